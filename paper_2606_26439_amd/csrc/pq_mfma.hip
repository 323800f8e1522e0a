// pq_mfma.hip -- fused PQ scoring by decoding into MFMA operands.
//
// The same scores as the table kernel (Sec. 4.2-4.3: by the ADC identity,
// sum_m T[i, m, c_jm] = q_i . concat_m C[m, c_jm]), computed the other way
// round: instead of a per-query table, the workgroup keeps the codebook
// itself in LDS (M x K x dsub FP16, 64 KiB at d = 128) and each wave
// rebuilds a 16-token document tile from it straight into the A operand of
// v_mfma_f32_16x16x32_f16: lane (r, g) of k-step c needs the 8 values
// c*32 + g*8 .. +8 of token r, which sit inside one centroid (dsub >= 8), so
// one ds_read_b128 fetches them. The decoded tile is then contracted with
// the query tokens held in VGPRs (B operand), several queries per wave, so
// one decode serves NQB x 16 query tokens. Running maxima stay in VGPRs; rows
// past a document's end are clamped to its last token; at the document's
// end two lane-row swaps finish the max over rows and four DPP rotations sum
// a query's tokens. FP16 products are exact and accumulate in FP32.
//
// A work position is (query group, document), or a candidate; every wave takes
// an equal share of them (document tokens, or candidates). Without candidate
// lists a group holds NQB / BPQ queries (BPQ = 16-column blocks per query,
// from the query-length bound); with candidate lists a group is one query,
// scored with its own number of blocks. Codes arrive by direct-to-LDS loads
// four tiles ahead, document offsets sit in lane registers, and scores are
// written 64 documents at a time, so no step waits for an offset or a store.
//
// Bound: the matrix cores (2 * Nq * d per document token, 11% more on clamped
// rows). 64 queries of 32 tokens over 250K documents: 7.24-7.51 ms, 1.21-1.26
// PFLOP/s, the rate of a large FP16 matrix product on the same card (8.07 ms
// with one wave per strided document, a scalar offset load at each document
// and eight query blocks). Eight queries of 8 to 64 tokens with 1K to 100K
// candidates, top-k included: 425 us, 701 when every query had the same number
// of workgroups and the blocks of the longest query (both with a top-k of 65
// us; 390 with the present one).
#include "device_common.h"
#include "kernels.h"

namespace {

template <int M>
struct PqCodes;
template <>
struct PqCodes<4> {
  typedef uint32_t type;
  __device__ static uint32_t word(type v, int) { return v; }
};
template <>
struct PqCodes<8> {
  typedef uint2 type;
  __device__ static uint32_t word(type v, int w) { return w == 0 ? v.x : v.y; }
};
template <>
struct PqCodes<16> {
  typedef uint4 type;
  __device__ static uint32_t word(type v, int w) {
    return w == 0 ? v.x : (w == 1 ? v.y : (w == 2 ? v.z : v.w));
  }
};

constexpr int PF = PQ_RING;

// One wave's scores: positions [lo, hi) (position base + b is document b, or
// position p is candidate p) of the gsz queries from a0 on, whose tokens fill
// NB blocks of 16 columns, bpq of them per query. RING: codes and scores pass
// through this wave's LDS (ring, sc); else, where the codebooks leave none, they
// stay in registers.
template <int M, int DSUB, int NB, bool RING>
__device__ __forceinline__ void score_range(const PqParams& P, int64_t a0, int gsz, int bpq,
                                            int64_t base, int64_t lo, int64_t hi,
                                            const char* cbl, char* ring, float* sc,
                                            const char* zrow) {
  constexpr int SLOT = 16 * M;  // bytes of a ring slot
  constexpr int DIM = M * DSUB;
  constexpr int NKS = DIM / 32;  // k-steps of 32
  typedef typename PqCodes<M>::type cvec;
  const int lane = lane_id();
  const int r = lane & 15, g = lane >> 4;
  const int K = P.K;

  // ---- query operand registers: block nb = query a0 + nb / bpq, rows
  // (nb % bpq) * 16 + r of that query (zero past its end) ----
  f16x8 qb[NB][NKS];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int64_t a = a0 + nb / bpq;
    int nq = 0;
    int64_t q0 = 0;
    if (a < P.n_q && nb / bpq < gsz) {
      q0 = P.q_off[a];
      nq = (int)(P.q_off[a + 1] - q0);
    }
    const int t = (nb % bpq) * 16 + r;
    const bool live = t < nq;
    const _Float16* qrow = (const _Float16*)P.q_tok + (q0 + (live ? t : 0)) * DIM + g * 8;
#pragma unroll
    for (int c = 0; c < NKS; ++c) {
      u32x4 v = {0u, 0u, 0u, 0u};
      if (live) v = *(const u32x4*)(qrow + c * 32);
      qb[nb][c] = __builtin_bit_cast(f16x8, v);
    }
  }
  // per query of the group (bit gq): exists, has tokens, exceeds its bound
  uint32_t valid_m = 0, nonempty_m = 0, poison_m = 0;
#pragma unroll
  for (int gq = 0; gq < NB; ++gq) {
    const int64_t a = a0 + gq;
    if (gq < gsz && a < P.n_q) {
      const int nq = (int)(P.q_off[a + 1] - P.q_off[a]);
      valid_m |= 1u << gq;
      if (nq > 0) nonempty_m |= 1u << gq;
      if (nq > P.bpq * 16) poison_m |= 1u << gq;
    }
  }
  valid_m = __builtin_amdgcn_readfirstlane(valid_m);
  nonempty_m = __builtin_amdgcn_readfirstlane(nonempty_m);
  poison_m = __builtin_amdgcn_readfirstlane(poison_m);

  // per-lane decode constants of k-step c: subspace m = (c*32 + g*8) / DSUB,
  // offset o inside the centroid; the 32/DSUB subspaces of one k-step lie in
  // one 4-byte word of the code vector
  int lbase[NKS], lsh[NKS];
#pragma unroll
  for (int c = 0; c < NKS; ++c) {
    const int kk = c * 32 + g * 8;
    const int m = kk / DSUB, o = kk % DSUB;
    lbase[c] = (m * K * DSUB + o) * 2;
    lsh[c] = 8 * (m & 3);
  }

  // ---- cursor over (document, 16-row tile) steps of [lo, hi). The starts
  // and lengths of 64 documents at a time sit in the lanes' registers, so a
  // document change reads a lane instead of waiting for memory.
  const bool has_cand = P.cand_off != nullptr;
  const int span = (int)(hi - lo);
  int64_t m_start = 0;
  int m_len = 0;
  auto load_meta = [&](int first) {
    m_start = 0;
    m_len = 0;
    if (first + lane < span) {
      const int64_t p = lo + first + lane;
      const int64_t b = has_cand ? (int64_t)P.cand_ids[p] : p - base;
      m_start = P.d_off[b];
      m_len = (int)(P.d_off[b + 1] - m_start);
    }
    // waited for here, once in 64 documents, so no other path waits for it
    vmem_wait<0>();
  };
  int cp = 0, ctile = 0, cnd = 0;
  int64_t ct0 = 0;
  auto enter_doc = [&]() {  // document cp becomes the cursor's
    if ((cp & 63) == 0 && cp < span) load_meta(cp);
    ct0 = readlane64(m_start, cp & 63);
    cnd = __builtin_amdgcn_readlane(m_len, cp & 63);
    ctile = 0;
  };
  enter_doc();
  constexpr int F_VALID = 1, F_EMPTY = 2, F_DLAST = 4;
  // Codes come straight into a ring of PF tile slots in LDS (16 * M bytes
  // each, four bytes per lane), so their loads hold no registers and nothing
  // but this wave's own counted waits waits for them. Every refill issues one
  // load (from the zero row when there is nothing left).
  const uint32_t ring_at = RING ? lds_offset(ring) : 0u;
  const int crow = lane * 4 / M, ccol = lane * 4 % M;
  cvec code_reg[RING ? 1 : PF];
  auto refill = [&](int k) -> int {
    const char* src = zrow;
    int f = 0, lim = 0;
    bool last = false;
    if (cp < span) {
      last = true;
      if (cnd == 0) {
        f = F_VALID | F_EMPTY;
      } else {
        src = (const char*)P.codes + (ct0 + ctile * 16) * M;
        lim = cnd - ctile * 16 - 1;
        last = lim < 16;
        f = F_VALID | (last ? F_DLAST : 0);
      }
    }
    if constexpr (RING) {
      if (4 * M >= 64 || lane < 4 * M)
        load_to_lds<4, false>(src + (crow < lim ? crow : lim) * M + ccol, ring_at + k * SLOT);
    } else {
      code_reg[k] = *(const cvec*)(src + (r < lim ? r : lim) * M);
    }
    if (last) {
      ++cp;
      enter_doc();
    } else {
      ++ctile;
    }
    return f;
  };

  // 64 documents' scores are kept in LDS (or one per lane), a row of 64 for the
  // query whose last block is nb, and written a row at a time
  float* const out = P.scores + lo + (has_cand ? 0 : (a0 - base / P.n_docs) * P.n_docs);
  int n_out = 0;  // documents scored
  float sc_reg[RING ? 1 : NB];
  auto put = [&](int nb, float v) {
    if constexpr (RING) {
      if (lane == 0) sc[nb * 64 + (n_out & 63)] = v;
    } else {
      v = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
      sc_reg[nb] = lane == (n_out & 63) ? v : sc_reg[nb];
    }
  };
  auto flush = [&](int n) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      if ((nb + 1) % bpq == 0) {
        const int gq = nb / bpq;
        if (((valid_m >> gq) & 1u) && lane < n) {
          // query longer than its bound: NaN (as a bit pattern; this file
          // assumes no NaN arithmetic)
          float v;
          if constexpr (RING)
            v = sc[nb * 64 + lane];
          else
            v = sc_reg[nb];
          if ((poison_m >> gq) & 1u) v = __builtin_bit_cast(float, 0x7fc00000u);
          out[(int64_t)gq * P.n_docs + n_out - n + lane] = v;
        }
      }
    }
  };
  auto scored = [&]() {
    ++n_out;
    if ((n_out & 63) == 0) flush(64);
  };

  float mx[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) mx[nb] = -__builtin_inff();
  if constexpr (!RING)
    for (int nb = 0; nb < NB; ++nb) sc_reg[nb] = 0.f;

  auto consume = [&](const cvec& cv, int fl) {
    if (!(fl & F_VALID)) return;
    if (fl & F_EMPTY) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        put(nb, ((nonempty_m >> (nb / bpq)) & 1u) ? -__builtin_inff() : 0.f);
      scored();
      return;
    }
    f16x8 av[NKS];
#pragma unroll
    for (int c = 0; c < NKS; ++c) {
      const uint32_t code =
          __builtin_amdgcn_ubfe(PqCodes<M>::word(cv, (c * 32 / DSUB) >> 2), lsh[c], 8);
      av[c] = __builtin_bit_cast(f16x8, *(const u32x4*)(cbl + lbase[c] + code * (DSUB * 2)));
    }
    // CH query blocks at a time, k-step outer: independent accumulation
    // chains keep the matrix pipe busy between dependent MFMAs, and no more
    // accumulators than that are live
    constexpr int CH = NB % 2 == 0 ? 2 : NB;
#pragma unroll
    for (int b0 = 0; b0 < NB; b0 += CH) {
      f32x4 acc[CH];
#pragma unroll
      for (int nb = 0; nb < CH; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < NKS; ++c)
#pragma unroll
        for (int nb = 0; nb < CH; ++nb)
          acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av[c], qb[b0 + nb][c], acc[nb], 0, 0, 0);
#pragma unroll
      for (int nb = 0; nb < CH; ++nb)
        mx[b0 + nb] = fmaxf(fmaxf(fmaxf(fmaxf(mx[b0 + nb], acc[nb].x), acc[nb].y), acc[nb].z),
                            acc[nb].w);
    }
    if (fl & F_DLAST) {
      float qsum = 0.f;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const float v = max_rows4(mx[nb]);
        qsum += v;
        mx[nb] = -__builtin_inff();
        if ((nb + 1) % bpq == 0) {
          put(nb, row_sum16(qsum));
          qsum = 0.f;
        }
      }
      scored();
    }
  };

  vmem_wait<0>();  // the query operand is in its registers
  int fl[PF];
#pragma unroll
  for (int k = 0; k < PF; ++k) fl[k] = refill(k);
  if constexpr (RING) {
    vmem_wait<PF - 1>();
    cvec cv = *(const cvec*)(ring + r * M);
    // a step: the next tile's codes out of its slot, this tile's slot refilled
    // (its codes are in registers), then the arithmetic. The wait for LDS reads
    // is for this tile's codes, read a step ago, which the refill overwrites (it
    // comes before the next tile's read, so that one is not waited for).
    while (fl[0] & F_VALID) {
#pragma unroll
      for (int k = 0; k < PF; ++k) {
        lds_reads_wait();
        vmem_wait<PF - 2>();
        const cvec nx = *(const cvec*)(ring + ((k + 1) % PF) * SLOT + r * M);
        const int f = fl[k];
        fl[k] = refill(k);
        consume(cv, f);
        cv = nx;
      }
    }
    // the idle refills and the last read still use this wave's ring
    lds_reads_wait();
    vmem_wait<0>();
  } else {
    while (fl[0] & F_VALID) {
#pragma unroll
      for (int k = 0; k < PF; ++k) {
        const cvec cv = code_reg[k];
        const int f = fl[k];
        fl[k] = refill(k);
        consume(cv, f);
      }
    }
  }
  flush(n_out & 63);
}

// First position of wave w of W: equal shares of the document tokens of every
// query group (positions are group * n_docs + document), or of the candidates
// of all queries.
__device__ int64_t pq_range_begin(const PqParams& P, int64_t w, int64_t W, int64_t n) {
  if (w >= W) return n;
  if (P.cand_off != nullptr || P.tokens_per_query <= 0) return (n / W) * w + ((n % W) * w) / W;
  const int64_t T = P.tokens_per_query, total = (n / P.n_docs) * T;
  const int64_t tau = (total / W) * w + ((total % W) * w) / W;
  const int64_t u = tau / T;
  return u * P.n_docs + wave_lower_bound(P.d_off, P.n_docs, tau - u * T);
}

constexpr int NW = 8;  // waves per workgroup

template <int M, int DSUB, int NQB, bool RING>
__global__ __launch_bounds__(NW * 64, RING && NQB * M * DSUB <= 512 ? 4 : 2) void pq_mfma_kernel(PqParams P) {
  extern __shared__ u32x4 cb_lds[];  // codebooks [M][K][DSUB] FP16
  // ---- codebooks into LDS (16-byte copies) ----
  {
    const int n16 = M * P.K * DSUB * 2 / 16;
    const u32x4* src = (const u32x4*)P.codebooks;
    for (int e = threadIdx.x; e < n16; e += NW * 64) cb_lds[e] = src[e];
  }
  const int gsz = P.group;  // queries per group
  const int64_t n = P.cand_off != nullptr ? P.n_pairs : ((P.n_q + gsz - 1) / gsz) * P.n_docs;
  const int64_t w = (int64_t)blockIdx.x * NW + uniform(threadIdx.x >> 6);
  const int64_t W = (int64_t)gridDim.x * NW;
  int64_t pb = uniform64(pq_range_begin(P, w, W, n));
  const int64_t pe = uniform64(pq_range_begin(P, w + 1, W, n));
  __syncthreads();
  const char* cbl = (const char*)cb_lds;
  char* ring = (char*)cb_lds + M * P.K * DSUB * 2 +  // (only with RING)
               uniform(threadIdx.x >> 6) * pq_mfma_wave_lds(M, NQB);
  float* sc = (float*)(ring + PF * 16 * M);
  const char* const zrow = zero_row_ptr();
  // the group-sized pieces of this wave's range
  while (pb < pe) {
    int64_t a0, base, end;  // first query, the position documents count from
    if (P.cand_off == nullptr) {
      const int64_t u = pb / P.n_docs;
      a0 = u * gsz;
      base = u * P.n_docs;
      end = base + P.n_docs;
    } else {
      // (positions that no query owns, which only offsets breaking the
      // contract leave, are passed over)
      a0 = uniform64(wave_owner(P.cand_off, P.n_q, pb));
      base = 0;
      end = uniform64(P.cand_off[a0 + 1]);
      if (a0 < 0) {
        pb = end;
        continue;
      }
      if (end <= pb) break;
    }
    const int64_t hi = end < pe ? end : pe;
    // a query alone in its group runs with its own block count, not its
    // batch's longest query's
    int own = NQB;
    if (gsz == 1) {
      const int nq = uniform((int)(P.q_off[a0 + 1] - P.q_off[a0]));
      own = nq <= 16 ? 1 : (nq + 15) / 16;
    }
    if (NQB > 1 && NQB <= 4 && own == 1)
      score_range<M, DSUB, 1, RING>(P, a0, gsz, 1, base, pb, hi, cbl, ring, sc, zrow);
    else if (NQB > 2 && NQB <= 4 && own == 2)
      score_range<M, DSUB, 2, RING>(P, a0, gsz, 2, base, pb, hi, cbl, ring, sc, zrow);
    else if (NQB > 3 && NQB <= 4 && own == 3)
      score_range<M, DSUB, 3, RING>(P, a0, gsz, 3, base, pb, hi, cbl, ring, sc, zrow);
    else
      score_range<M, DSUB, NQB, RING>(P, a0, gsz, P.bpq, base, pb, hi, cbl, ring, sc, zrow);
    pb = hi;
  }
}

template <int M, int DSUB, int NQB, bool RING>
hipError_t launch_mfma_r(const PqParams& P, size_t lds, hipStream_t s) {
  auto k = pq_mfma_kernel<M, DSUB, NQB, RING>;
  if (lds > 64 * 1024) {
    hipError_t e =
        hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  int occ = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k, NW * 64, lds);
  if (e != hipSuccess) return e;
  // Every compute unit filled, down to about two documents per wave, and up
  // to eight times as many workgroups where a wave keeps 200 documents to
  // spread the copy of the codebooks over: 64 queries over 250K documents
  // 7.95 / 7.36 / 7.24 ms with one, four and eight workgroups per place; 400K
  // candidates of eight queries 422 / 424 / 443 us.
  const int64_t n =
      P.cand_off != nullptr ? P.n_pairs : (P.n_q + P.group - 1) / P.group * P.n_docs;
  const int64_t resident = (int64_t)(occ < 1 ? 1 : occ) * P.cus;
  int64_t times = n / (200 * NW * resident);
  times = times < 1 ? 1 : (times > 8 ? 8 : times);
  int64_t grid = times * resident;
  const int64_t most = (n + 2 * NW - 1) / (2 * NW);
  if (grid > most) grid = most;
  hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(NW * 64), lds, s, P);
  return hipGetLastError();
}

template <int M, int DSUB, int NQB>
hipError_t launch_mfma_t(const PqParams& P, size_t lds, hipStream_t s) {
  // no ring: only codebooks near the size of the LDS (M * dsub = 512)
  if constexpr (M * DSUB >= 512) {
    if (!P.ring) return launch_mfma_r<M, DSUB, NQB, false>(P, lds, s);
  }
  return launch_mfma_r<M, DSUB, NQB, true>(P, lds, s);
}

template <int M, int DSUB>
hipError_t launch_mfma_nqb(const PqParams& P, size_t lds, hipStream_t s) {
  constexpr int NKS = M * DSUB / 32;
  switch (P.nqb) {
    case 1: return launch_mfma_t<M, DSUB, 1>(P, lds, s);
    case 2: return launch_mfma_t<M, DSUB, 2>(P, lds, s);
    case 4:
      if constexpr (NKS <= 8) return launch_mfma_t<M, DSUB, 4>(P, lds, s);
      return hipErrorInvalidValue;
    default:
      if constexpr (NKS <= 4) return launch_mfma_t<M, DSUB, 8>(P, lds, s);
      return hipErrorInvalidValue;
  }
}

template <int M>
hipError_t launch_mfma_dsub(const PqParams& P, size_t lds, hipStream_t s) {
  switch (P.dsub) {
    case 8: return launch_mfma_nqb<M, 8>(P, lds, s);
    case 16: return launch_mfma_nqb<M, 16>(P, lds, s);
    default: return launch_mfma_nqb<M, 32>(P, lds, s);
  }
}

}  // namespace

hipError_t launch_pq_mfma(const PqParams& P, size_t lds, hipStream_t s) {
  switch (P.M) {
    case 4: return launch_mfma_dsub<4>(P, lds, s);
    case 8: return launch_mfma_dsub<8>(P, lds, s);
    default: return launch_mfma_dsub<16>(P, lds, s);
  }
}
