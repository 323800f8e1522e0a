// residual.hip -- MaxSim over residual-compressed documents.
//
// A document token is stored as a centroid id plus a residual quantized per
// dimension to NBITS bits (the compressed form of the PLAID/WARP indexes the
// paper compares with and plugs into): x_jk = C[id_j, k] + w[code_jk]. The
// score is Eq. (1) on these vectors, computed through the split
//   q_i . x_j = q_i . C[id_j] + q_i . r_j.
// The first term does not depend on the document, so one small MFMA kernel
// tabulates P[c, (a, t)] = C[c] . q_t of query a for every centroid c (FP32,
// in the caller's workspace; each query owns QW = 16 * NQB columns, NQB the
// 16-token blocks of the longest query rounded up to a power of two; the
// blocks that hold its tokens are written, zero past the last one). Where the table would cost more than it saves
// (maxsim_residual_score's rule), the kernel gathers the centroid itself and
// adds q_t . C[id] in the same order, so the scores have the same bits. The
// fused kernel then reads each
// document token's id (4 B) and packed residual (dim * NBITS / 8 B) once from
// HBM, decodes the residual codes into FP16 through a byte-indexed table in
// LDS, and computes q_t . r_j with v_mfma_f32_16x16x32_f16 whose accumulator
// starts from the gathered table entries; the running max over tokens and the
// sum over query tokens follow. Decoded vectors are never written.
//
// Operand layout. The MFMA's rows are query tokens and its columns document
// tokens, so lane (r, g) of the accumulator holds document row r of the tile
// against query tokens 16 nb + 4g .. 16 nb + 4g + 3 of query block nb: the
// table entries it needs are consecutive in the centroid's table row and
// arrive in one 16-byte load per block. The sum over query tokens runs per
// row position over the blocks in order, then over the positions in a fixed
// tree, so a query scores the same bits whatever block count its batch uses
// (extra blocks add exact zeros at the end). In the k dimension lane group g
// owns the contiguous quarter [g * dim/4, (g+1) * dim/4) of the dimensions
// and k-step s takes columns g * dim/4 + 8 s .. + 7 of both operands, so a
// lane's residual codes for all k-steps are one contiguous dim * NBITS / 32-byte
// piece of the packed row.
#include <map>
#include <mutex>

#include "device_common.h"
#include "kernels.h"

namespace {

// P[c, a * QW + t] = C[c] . q_t of query a (t < its length), 0 for t up to
// the end of its last block; later blocks are not read, so not written (eight
// queries of 8 to 64 tokens, 2^17 centroids: 86 us, 96 with all of them). One wave per 16 centroids and every 16-column block of every query;
// 4 waves per group.
template <int NKS>
__global__ __launch_bounds__(256) void centroid_table_kernel(ResParams P) {
  constexpr int DIM = NKS * 32;
  const int lane = lane_id();
  const int r = lane & 15, g = lane >> 4;
  const int64_t c0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16;
  const int64_t n_c = P.n_centroids;
  if (c0 >= n_c) return;  // uniform per wave
  const int64_t cr = c0 + r < n_c ? c0 + r : n_c - 1;
  const _Float16* crow = (const _Float16*)P.centroids + cr * DIM + g * (DIM / 4);
  f16x8 a[NKS];
#pragma unroll
  for (int s = 0; s < NKS; ++s) a[s] = *(const f16x8*)(crow + 8 * s);
  const int64_t ncols = P.n_cols;
  const int bpq = P.nqb;
  for (int64_t blk = 0; blk < P.n_q * bpq; ++blk) {
    const int64_t qa = blk / bpq;
    const int t = (int)(blk % bpq) * 16 + r;
    const int64_t q0 = sload_i64(P.q_off, qa);
    const int nq = (int)(sload_i64(P.q_off, qa + 1) - q0);
    if (blk % bpq > 0 && (int)(blk % bpq) * 16 >= nq) continue;
    const bool live = t < nq;
    const _Float16* qrow = (const _Float16*)P.q_tok + (live ? q0 + t : 0) * DIM + g * (DIM / 4);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NKS; ++s) {
      u32x4 v = {0u, 0u, 0u, 0u};
      if (live) v = *(const u32x4*)(qrow + 8 * s);
      acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[s], __builtin_bit_cast(f16x8, v), acc, 0, 0,
                                                   0);
    }
    // lane holds centroids c0 + 4g + v, column blk * 16 + r
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t c = c0 + 4 * g + v;
      if (c < n_c) P.table[c * ncols + blk * 16 + r] = acc[v];
    }
  }
}

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// Residual bytes of one lane for one token, as 32-bit words.
template <int RB>
struct ResWords {
  static constexpr int N = RB < 4 ? 1 : RB / 4;
  uint32_t w[N];
  __device__ void read(const char* p) {
    if constexpr (RB == 2) {
      w[0] = *(const uint16_t*)p;
    } else if constexpr (RB == 4) {
      w[0] = *(const uint32_t*)p;
    } else if constexpr (RB == 8) {
      const u32x2 v = *(const u32x2*)p;
      w[0] = v.x;
      w[1] = v.y;
    } else {
#pragma unroll
      for (int h = 0; h < RB / 16; ++h) {
        const u32x4 v = *(const u32x4*)(p + 16 * h);
        w[4 * h] = v.x;
        w[4 * h + 1] = v.y;
        w[4 * h + 2] = v.z;
        w[4 * h + 3] = v.w;
      }
    }
  }
  // byte j of the lane's piece shifted left by scale_log2 (a byte offset into
  // the LUT, whose entries are 2^scale_log2 bytes)
  __device__ uint32_t byte_offset(int j, int scale_log2) const {
    return __builtin_amdgcn_ubfe(w[j >> 2], 8 * (j & 3), 8) << scale_log2;
  }
};

// Shape of a wave's ring slot: the 16 gathered rows of a tile (table rows of
// NB query blocks, or the centroids themselves), its packed residual codes,
// and the centroid ids of the tile after it in that slot.
template <int NBITS, int NKS, int NB, bool DIRECT>
struct Slot {
  static constexpr int DIM = NKS * 32;
  static constexpr int ROW = DIRECT ? DIM * 2 : NB * 64;  // gathered bytes per token
  static constexpr int CPR = ROW / 16;                    // 16-byte pieces per gathered row
  static constexpr int NG = 16 * ROW / 1024;              // gather instructions per tile
  static constexpr int RB = NKS * NBITS;                  // code bytes per lane per token
  static constexpr int ROWB = 4 * RB;                     // code bytes per token
  static constexpr int CU = ROWB >= 16 ? 16 : 4;          // bytes of one code copy per lane
  static constexpr int NCODE = 16 * ROWB / CU;            // lanes' worth of code copies per tile
  static constexpr int NCI = (NCODE + 63) / 64;           // code instructions per tile
  static constexpr int ROWS_OFF = 0, CODES_OFF = 16 * ROW, IDS_OFF = CODES_OFF + 16 * ROWB;
  static constexpr int BYTES = IDS_OFF + 64;
  static constexpr int OPS = 1 + NCI + NG;  // vector memory operations per tile
  // 16-byte piece p of gathered row rho lies at rho * CPR + place(rho, p): the
  // 16 rows an operand read touches fall in 16 different bank groups (rows of
  // 12 pieces start at four of the 16 groups: a turn by rho / 4 separates the
  // rows that start alike)
  __device__ static int place(int rho, int p) {
    if constexpr (CPR == 12) {
      const int q = p + (rho >> 2);
      return q < CPR ? q : q - CPR;
    } else {
      return p ^ swz(rho);
    }
  }
  // the piece that lies at place q
  __device__ static int piece_at(int rho, int q) {
    if constexpr (CPR == 12) {
      const int p = q - (rho >> 2);
      return p >= 0 ? p : p + CPR;
    } else {
      return q ^ swz(rho);
    }
  }
  __device__ static int swz(int rho) {
    constexpr int SW = CPR < 16 ? CPR : 16;
    return (rho / (16 / SW)) & (SW - 1);
  }
};

// Whether a wave holds two tiles' operands, so that one's come out of LDS while
// the other's are contracted. At d = 256 the query operand of three and four
// blocks takes 96 and 128 registers and two tiles of the table's route no longer
// fit beside it (100K documents, one 64-token query, 2 bits, 2^12 centroids: 851
// us with what spilled, 333 with one tile); with two blocks one tile leaves
// three waves per SIMD instead of two (223 against 208 us).
constexpr bool two_tiles(int nb, int nks, bool direct) {
  return direct || (nb * nks < 24 && !(nb == 2 && nks == 8));
}
// Waves per SIMD that the registers are shared out for. Gathered centroids at
// d = 256 with four blocks: one, as the rings leave room for (2^17 centroids,
// 20,000 candidates of a 64-token query: 860 us with two and what spilled, 206);
// the table's four blocks at d = 64: two (2^17 centroids, 90,000 candidates of a
// 64-token query: 643 us with four and what spilled, 261).
constexpr int waves_per_simd(int nqb, int nks, bool direct) {
  if (direct) return nqb * nks <= 4 ? 4 : nqb * nks >= 32 ? 1 : 2;
  return nqb == 4 ? 2 : nqb * nks <= 8 ? 4 : nqb * nks == 16 ? 3 : 2;
}

// One wave's scores: work positions [lo, hi) of query a (position base + b is
// document b, or position p is candidate p), NB blocks of 16 query tokens.
//
// Everything a tile needs arrives by direct-to-LDS loads in a ring of PF slots
// per wave: the ids PF tiles ahead of the gathers they address, those and the
// codes PF tiles ahead of the arithmetic. A gather instruction's consecutive
// lanes take consecutive 16-byte pieces of one row, so four lanes share one
// 64-byte access of the vector cache: 41 accesses a tile instead of 143.
// Bound (1M documents, one 32-token query, 2 bits, d = 128): the vector cache's
// address path. It is 78% busy with a table that the L2s hold (2^12 centroids;
// LDS 53%, half of that conflicts, VALU 56%), a launch of 1.15 ms (1.38 with the
// gathers in registers), and 87% busy with 2^17 centroids (16.8 MB against 4 MB
// of L2 per XCD: three quarters of the gathered lines come over the fabric, 10 GB
// with the streams), 1.32 ms (1.44). A batch of eight queries of 8 to 64 tokens
// with 1K to 100K candidates, table and top-k included: 0.97 ms (1.83 before;
// most of it the queries' equal shares of workgroups whatever their lists'
// lengths, and 64 columns for each of them).
template <int NBITS, int NKS, int NB, int PF, bool DIRECT>
__device__ __forceinline__ void score_range(const ResParams& P, int64_t a, int64_t base,
                                            int64_t lo, int64_t hi, int64_t qa0, int nq, bool poison, const char* lutb,
                                            char* ring) {
  typedef Slot<NBITS, NKS, NB, DIRECT> L;
  constexpr int DIM = L::DIM, RB = L::RB, ROWB = L::ROWB, CPR = L::CPR;
  constexpr int FPB = 8 / NBITS;  // fields per byte
  constexpr int EB = 2 * FPB;     // LUT entry bytes (FPB FP16 values)
  constexpr int EB_LOG2 = EB == 16 ? 4 : (EB == 8 ? 3 : 2);
  static_assert((PF - 1) * L::OPS <= 63, "waits count up to 63 operations");
  const int lane = lane_id();
  const int r = lane & 15, g = lane >> 4;

  // query operand (the MFMA's rows): block nb, row r is query token
  // 16 nb + r of query a, zero past its end
  f16x8 qa[NB][NKS];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int t = 16 * nb + r;
    const bool live = t < nq;
    const _Float16* qrow = (const _Float16*)P.q_tok + (qa0 + (live ? t : 0)) * DIM + g * (DIM / 4);
#pragma unroll
    for (int s = 0; s < NKS; ++s) {
      u32x4 v = {0u, 0u, 0u, 0u};
      if (live) v = *(const u32x4*)(qrow + 8 * s);
      qa[nb][s] = __builtin_bit_cast(f16x8, v);
    }
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
  constexpr int F_VALID = 1, F_EMPTY = 2, F_DLAST = 4, F_TOK = 8;
  struct Tile {
    int64_t tok0;
    int rows, flags;
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
  auto next_tile = [&]() -> Tile {
    Tile t{0, 1, 0};
    if (cp < span) {
      bool last = true;
      if (cnd == 0) {
        t.flags = F_VALID | F_EMPTY;
      } else {
        const int left = cnd - ctile * 16;
        t.tok0 = ct0 + (int64_t)ctile * 16;
        t.rows = left < 16 ? left : 16;
        last = left <= 16;
        t.flags = F_VALID | F_TOK | (last ? F_DLAST : 0);
      }
      if (last) {
        ++cp;
        enter_doc();
      } else {
        ++ctile;
      }
    }
    return t;
  };

  // Every tile issues the same loads (a tile without tokens reads the zero
  // row, and row 0 of the gathered array, instead), so the count of loads in
  // flight is the same on every path. The document streams are read once:
  // non-temporal loads keep them from displacing the gathered array in the
  // caches. The host keeps n_centroids and the table's row length below 2^24
  // and the table below 2^32 entries.
  const char* zrow = P.zero_row;
  const uint32_t max_c = (uint32_t)(P.n_centroids - 1);
  const char* const gat = DIRECT ? (const char*)P.centroids
                                 : (const char*)(P.table + (uint32_t)a * (uint32_t)(16 * P.nqb));
  const uint32_t stride = DIRECT ? (uint32_t)(DIM * 2) : (uint32_t)P.n_cols * 4u;
  auto issue_ids = [&](const Tile& t, uint32_t slot) {
    const int row = r < t.rows ? r : t.rows - 1;
    const int32_t* src = (t.flags & F_TOK) ? P.ids + t.tok0 + row : (const int32_t*)zrow;
    if (lane < 16) load_to_lds<4, true>(src, slot + L::IDS_OFF);
  };
  // ids: the tile's centroid ids of the rows this lane gathers (clamped to
  // the table, so a bad id cannot read outside it)
  auto issue_rest = [&](const Tile& t, const uint32_t (&ids)[L::NG], uint32_t slot) {
    const char* cb = (t.flags & F_TOK) ? (const char*)P.residuals + t.tok0 * ROWB : zrow;
    const int lim = (t.flags & F_TOK) ? t.rows - 1 : 0;
#pragma unroll
    for (int i = 0; i < L::NCI; ++i) {
      const int byte = (i * 64 + lane) * L::CU;
      const int row = byte / ROWB, in = byte % ROWB;
      if (L::NCODE >= 64 * (i + 1) || lane < L::NCODE - 64 * i)
        load_to_lds<L::CU, true>(cb + (row < lim ? row : lim) * ROWB + in,
                                 slot + L::CODES_OFF + i * 64 * L::CU);
    }
#pragma unroll
    for (int w = 0; w < L::NG; ++w) {
      const int piece = w * 64 + lane;
      const int rho = piece / CPR, p = piece % CPR;
      const uint32_t id = ids[w] < max_c ? ids[w] : max_c;
      load_to_lds<16, false>(gat + (uint64_t)id * stride + L::piece_at(rho, p) * 16,
                             slot + w * 1024);
    }
  };

  // scores are kept one per lane and written 64 at a time
  float* const out = P.scores + lo;
  float sbuf = 0.f;
  int n_out = 0;  // documents scored
  auto flush = [&](int n) {
    if (lane < n) out[n_out - n + lane] = sbuf;
  };
  auto store = [&](float v) {
    // query longer than its bound: NaN (as a bit pattern; this file assumes
    // no NaN arithmetic)
    if (poison) v = __builtin_bit_cast(float, 0x7fc00000u);
    v = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
    sbuf = lane == (n_out & 63) ? v : sbuf;
    ++n_out;
    if ((n_out & 63) == 0) flush(64);
  };

  // running max per (query block, accumulator row) over this lane's document
  // rows; reduced over the 16 rows of the tile at the document's end
  f32x4 mx[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) mx[nb] = f32x4{-__builtin_inff(), -__builtin_inff(),
                                                 -__builtin_inff(), -__builtin_inff()};

  // max over the 16 lanes of a row group (rotations by 8, 4, 2, 1)
  auto row_max = [](float v) {
    v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                               0, __builtin_bit_cast(int, v), 0x128, 0xF, 0xF, false)));
    v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                               0, __builtin_bit_cast(int, v), 0x124, 0xF, 0xF, false)));
    v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                               0, __builtin_bit_cast(int, v), 0x122, 0xF, 0xF, false)));
    v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                               0, __builtin_bit_cast(int, v), 0x121, 0xF, 0xF, false)));
    return v;
  };

  // a tile's operands in registers: the decoded residuals of k-step s, and
  // this row's table entries (query tokens 16 nb + 4g .. + 3) or centroid
  // (the lane's k columns)
  constexpr int NR = DIRECT ? NKS : NB;
  auto contract = [&](const u32x4 (&res)[NKS], const u32x4 (&rows)[NR], f32x4 (&acc)[NB]) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      if constexpr (DIRECT)
        acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
      else
        acc[nb] = __builtin_bit_cast(f32x4, rows[nb]);
    }
    if constexpr (DIRECT) {
      // q . C in the order the table kernel adds it, so both forms give the
      // same bits
#pragma unroll
      for (int s = 0; s < NKS; ++s)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
              qa[nb][s], __builtin_bit_cast(f16x8, rows[s]), acc[nb], 0, 0, 0);
    }
#pragma unroll
    for (int s = 0; s < NKS; ++s)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
            qa[nb][s], __builtin_bit_cast(f16x8, res[s]), acc[nb], 0, 0, 0);
  };
  auto finish = [&](int fl, const f32x4 (&acc)[NB]) {
    if (fl & F_TOK) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int v = 0; v < 4; ++v) mx[nb][v] = fmaxf(mx[nb][v], acc[nb][v]);
      if (fl & F_DLAST) {
        // max over the document's rows (lanes r), then the sum over query
        // tokens: per row position 4g + v over the blocks in order, then over
        // v and g in a fixed tree
        float sv[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
          for (int v = 0; v < 4; ++v) sv[v] += row_max(mx[nb][v]);
          mx[nb] =
              f32x4{-__builtin_inff(), -__builtin_inff(), -__builtin_inff(), -__builtin_inff()};
        }
        store(sum_rows4((sv[0] + sv[1]) + (sv[2] + sv[3])));
      }
    } else if (fl & F_EMPTY) {
      store(nq > 0 ? -__builtin_inff() : 0.f);
    }
  };

  // Slot k of the ring holds the rows and codes of tile k, k + PF, ... and the
  // ids of the tile PF further on.
  Tile now[PF], ahead[PF];
  const uint32_t ring_at = lds_offset(ring);
  auto read_ids = [&](const char* slot, uint32_t (&ids)[L::NG]) {
#pragma unroll
    for (int w = 0; w < L::NG; ++w)
      ids[w] = *(const uint32_t*)(slot + L::IDS_OFF + ((w * 64 + lane) / CPR) * 4);
  };
#pragma unroll
  for (int k = 0; k < PF; ++k) {
    now[k] = next_tile();
    issue_ids(now[k], ring_at + k * L::BYTES);
  }
  vmem_wait<0>();
#pragma unroll
  for (int k = 0; k < PF; ++k) {
    const char* slot = ring + k * L::BYTES;
    uint32_t ids[L::NG];
    read_ids(slot, ids);
    lds_reads_wait();
    issue_rest(now[k], ids, ring_at + k * L::BYTES);
    ahead[k] = next_tile();
    issue_ids(ahead[k], ring_at + k * L::BYTES);
  }
  // A tile's operands move from its slot to registers: rows, and codes decoded
  // through the byte table; with them the ids of the slot's next tile.
  auto take_raw = [&](const char* slot, u32x4 (&rows)[NR], uint32_t (&ids)[L::NG],
                      ResWords<RB>& rw) {
    rw.read(slot + L::CODES_OFF + r * ROWB + g * RB);
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int p = DIRECT ? g * NKS + i : i * 4 + g;
      rows[i] = *(const u32x4*)(slot + (r * CPR + L::place(r, p)) * 16);
    }
    read_ids(slot, ids);
  };
  auto decode = [&](const ResWords<RB>& rw, u32x4 (&res)[NKS]) {
#pragma unroll
    for (int s = 0; s < NKS; ++s) {
      // bytes s*NBITS .. s*NBITS + NBITS - 1 of the lane's piece decode to
      // the 8 residual values of k-step s
      if constexpr (NBITS == 1) {
        res[s] = *(const u32x4*)(lutb + rw.byte_offset(s, EB_LOG2));
      } else if constexpr (NBITS == 2) {
        const uint2 lo2 = *(const uint2*)(lutb + rw.byte_offset(2 * s, EB_LOG2));
        const uint2 hi2 = *(const uint2*)(lutb + rw.byte_offset(2 * s + 1, EB_LOG2));
        res[s] = u32x4{lo2.x, lo2.y, hi2.x, hi2.y};
      } else {
        res[s] = u32x4{*(const uint32_t*)(lutb + rw.byte_offset(4 * s, EB_LOG2)),
                       *(const uint32_t*)(lutb + rw.byte_offset(4 * s + 1, EB_LOG2)),
                       *(const uint32_t*)(lutb + rw.byte_offset(4 * s + 2, EB_LOG2)),
                       *(const uint32_t*)(lutb + rw.byte_offset(4 * s + 3, EB_LOG2))};
      }
    }
  };
  // refill of slot k: the gathers of its ids' tile, the ids of the next one
  auto refill = [&](int k, const uint32_t (&ids)[L::NG]) {
    const uint32_t slot = ring_at + k * L::BYTES;
    // the slot's reads complete before its refill can land
    lds_reads_wait();
    issue_rest(ahead[k], ids, slot);
    now[k] = ahead[k];
    ahead[k] = next_tile();
    issue_ids(ahead[k], slot);
  };
  if constexpr (two_tiles(NB, NKS, DIRECT)) {
    u32x4 res[NKS], rows[NR];
    int fl = now[0].flags;
    {
      uint32_t ids[L::NG];
      ResWords<RB> rw;
      vmem_wait<(PF - 1) * L::OPS>();
      take_raw(ring, rows, ids, rw);
      decode(rw, res);
      refill(0, ids);
    }
    // Whole rounds of PF steps. A step's arithmetic runs on operands taken a
    // step earlier, while the next tile's come out of LDS (the codes, then the
    // byte-table reads they address), so a wave waits for neither; the table
    // reads come before the step's refill, because after it the compiler would
    // wait for every load in flight. The tiles after a wave's last one carry no
    // flags: their steps compute on what idle refills left and store nothing.
    while (fl & F_VALID) {
#pragma unroll
      for (int k = 0; k < PF; ++k) {
        const int kn = (k + 1) % PF;
        // the other slots' loads are younger; slot kn's have landed
        vmem_wait<(PF - 1) * L::OPS>();
        u32x4 res2[NKS], rows2[NR];
        uint32_t ids[L::NG];
        ResWords<RB> rw;
        f32x4 acc[NB];
        take_raw(ring + kn * L::BYTES, rows2, ids, rw);
        contract(res, rows, acc);
        decode(rw, res2);
        finish(fl, acc);
        fl = now[kn].flags;
        refill(kn, ids);
#pragma unroll
        for (int s = 0; s < NKS; ++s) res[s] = res2[s];
#pragma unroll
        for (int i = 0; i < NR; ++i) rows[i] = rows2[i];
      }
    }
  } else {
    while (now[0].flags & F_VALID) {
#pragma unroll
      for (int k = 0; k < PF; ++k) {
        vmem_wait<(PF - 1) * L::OPS>();
        u32x4 res[NKS], rows[NR];
        uint32_t ids[L::NG];
        ResWords<RB> rw;
        f32x4 acc[NB];
        take_raw(ring + k * L::BYTES, rows, ids, rw);
        decode(rw, res);
        const int fl = now[k].flags;
        refill(k, ids);
        contract(res, rows, acc);
        finish(fl, acc);
      }
    }
  }
  // the idle refills still target this wave's ring
  vmem_wait<0>();
  flush(n_out & 63);
}

template <int NBITS, int NKS, int NQB, int PF, bool DIRECT>
constexpr size_t wave_ring_bytes() {
  return (size_t)PF * Slot<NBITS, NKS, NQB, DIRECT>::BYTES;
}

// First work position of wave w of W: equal shares of the document tokens of
// every query (positions are query * n_docs + document), or of the candidates
// of all queries, so long and short lists of one batch load the waves alike.
__device__ int64_t res_range_begin(const ResParams& P, int64_t w, int64_t W) {
  const int64_t n = P.n_pairs;
  if (w >= W) return n;
  if (P.cand_off != nullptr || P.n_tokens <= 0) return (n / W) * w + ((n % W) * w) / W;
  const int64_t T = P.n_tokens, total = P.n_q * T;
  const int64_t tau = (total / W) * w + ((total % W) * w) / W;
  const int64_t a = tau / T;
  return a * P.n_docs + wave_lower_bound(P.d_off, P.n_docs, tau - a * T);
}

template <int NBITS, int NKS, int NQB, int NW, int PF, bool DIRECT>
__global__ __launch_bounds__(NW * 64, waves_per_simd(NQB, NKS, DIRECT)) void residual_maxsim_kernel(ResParams P) {
  constexpr int FPB = 8 / NBITS;
  __shared__ __attribute__((aligned(16))) _Float16 lut[256 * FPB];
  extern __shared__ u32x4 res_lds[];  // the waves' rings
  const int wave = uniform(threadIdx.x >> 6);

  // LUT: entry b holds the residual values of the FPB fields of byte b,
  // lowest field first (fields fill a byte from its least significant bit)
  for (int e = threadIdx.x; e < 256 * FPB; e += NW * 64) {
    const int b = e / FPB, f = e % FPB;
    lut[e] = ((const _Float16*)P.weights)[(b >> (f * NBITS)) & ((1 << NBITS) - 1)];
  }
  const int64_t w = (int64_t)blockIdx.x * NW + wave, W = (int64_t)gridDim.x * NW;
  int64_t pb = uniform64(res_range_begin(P, w, W));
  const int64_t pe = uniform64(res_range_begin(P, w + 1, W));
  __syncthreads();
  const char* lutb = (const char*)lut;
  char* ring = (char*)res_lds + wave * wave_ring_bytes<NBITS, NKS, NQB, PF, DIRECT>();
  // the query-sized pieces of this wave's range
  while (pb < pe) {
    int64_t a, base, end;  // the query, and the position its documents count from
    if (P.cand_off == nullptr) {
      a = pb / P.n_docs;
      base = a * P.n_docs;
      end = base + P.n_docs;
    } else {
      // (positions that no query owns, which only offsets breaking the
      // contract leave, are passed over)
      a = uniform64(wave_owner(P.cand_off, P.n_q, pb));
      base = 0;
      end = uniform64(P.cand_off[a + 1]);
      if (a < 0) {
        pb = end;
        continue;
      }
      if (end <= pb) break;
    }
    const int64_t hi = end < pe ? end : pe;
    const int64_t qa0 = uniform64(P.q_off[a]);
    const int nq = uniform((int)(P.q_off[a + 1] - qa0));
    const bool poison = nq > NQB * 16;
    // the query's own block count, not its batch's longest query's
    if (NQB >= 2 && nq <= 16) {
      score_range<NBITS, NKS, 1, PF, DIRECT>(P, a, base, pb, hi, qa0, nq, poison, lutb, ring);
    } else if (NQB >= 4 && nq <= 32) {
      score_range<NBITS, NKS, 2, PF, DIRECT>(P, a, base, pb, hi, qa0, nq, poison, lutb, ring);
    } else if (NQB >= 4 && nq <= 48) {
      score_range<NBITS, NKS, 3, PF, DIRECT>(P, a, base, pb, hi, qa0, nq, poison, lutb, ring);
    } else {
      score_range<NBITS, NKS, NQB, PF, DIRECT>(P, a, base, pb, hi, qa0, nq, poison, lutb, ring);
    }
    pb = hi;
  }
}

template <int NKS>
hipError_t launch_table_t(const ResParams& P, hipStream_t s) {
  const int64_t waves = (P.n_centroids + 15) / 16;
  hipLaunchKernelGGL(centroid_table_kernel<NKS>, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0,
                     s, P);
  return hipGetLastError();
}

template <int NBITS, int NKS, int NQB, bool DIRECT>
hipError_t launch_score_p(const ResParams& P, hipStream_t s) {
  constexpr int NW = 4;
  // Four tiles in flight per wave (two and three measured slower), or three
  // where that lets two workgroups share a compute unit (100K documents, one
  // 64-token query, d = 128, 4 bits: 423 -> 306 us) or where the widest gathered
  // rows leave no room for four.
  constexpr size_t lut = 512 * (8 / NBITS), unit = 160 * 1024;
  constexpr size_t four = lut + NW * wave_ring_bytes<NBITS, NKS, NQB, 4, DIRECT>();
  constexpr size_t three = lut + NW * wave_ring_bytes<NBITS, NKS, NQB, 3, DIRECT>();
  constexpr int PF = four > unit || (four > unit / 2 && three <= unit / 2) ? 3 : 4;
  auto k = residual_maxsim_kernel<NBITS, NKS, NQB, NW, PF, DIRECT>;
  constexpr size_t lds = NW * wave_ring_bytes<NBITS, NKS, NQB, PF, DIRECT>();
  static_assert(lut + lds <= unit, "the rings fit the LDS");
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds);
    if (e != hipSuccess) return e;
  }
  int occ = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k, NW * 64, lds);
  if (e != hipSuccess) return e;
  // Every compute unit filled, down to about two documents per wave; beyond
  // that several times as many workgroups (the tuned variant) of at least 16
  // documents a wave, so that the dispatch evens out what equal shares leave
  // uneven (the cost of a position follows its query's length; a batch of
  // eight queries of 8 to 64 tokens took 1.20 / 1.04 / 1.00 ms with one, four
  // and eight workgroups per place; one query over 1M documents 1.376 / 1.344
  // / 1.339 ms).
  constexpr int TIMES[RES_PIPES] = {1, 4, 16, 8};
  const int64_t resident = (int64_t)(occ < 1 ? 1 : occ) * P.cus;
  int64_t grid = (P.n_pairs + 16 * NW - 1) / (16 * NW);
  if (grid > TIMES[P.pipe] * resident) grid = TIMES[P.pipe] * resident;
  if (grid < resident) grid = resident;
  const int64_t most = (P.n_pairs + 2 * NW - 1) / (2 * NW);
  if (grid > most) grid = most;
  hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(NW * 64), lds, s, P);
  return hipGetLastError();
}

template <int NBITS, int NKS, int NQB>
hipError_t launch_score_t(const ResParams& P, hipStream_t s) {
  return P.direct ? launch_score_p<NBITS, NKS, NQB, true>(P, s)
                  : launch_score_p<NBITS, NKS, NQB, false>(P, s);
}

template <int NBITS, int NKS>
hipError_t launch_score_nqb(const ResParams& P, hipStream_t s) {
  switch (P.nqb) {
    case 1: return launch_score_t<NBITS, NKS, 1>(P, s);
    case 2: return launch_score_t<NBITS, NKS, 2>(P, s);
    default: return launch_score_t<NBITS, NKS, 4>(P, s);
  }
}

template <int NBITS>
hipError_t launch_score_dim(const ResParams& P, hipStream_t s) {
  switch (P.dim) {
    case 64: return launch_score_nqb<NBITS, 2>(P, s);
    case 128: return launch_score_nqb<NBITS, 4>(P, s);
    default: return launch_score_nqb<NBITS, 8>(P, s);
  }
}

}  // namespace

// Device address of this file's zero row, per device (the kernels take it as
// an argument).
hipError_t zero_row_address(const char** out) {
  static std::mutex mu;
  static std::map<int, const char*> addr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lk(mu);
  auto it = addr.find(dev);
  if (it == addr.end()) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_zero_row));
    if (e != hipSuccess) return e;
    it = addr.emplace(dev, (const char*)p).first;
  }
  *out = it->second;
  return hipSuccess;
}

hipError_t launch_residual(const ResParams& Pin, hipStream_t s) {
  ResParams P = Pin;
  hipError_t e = zero_row_address(&P.zero_row);
  if (e != hipSuccess) return e;
  if (!P.direct) {
    switch (P.dim) {
      case 64: e = launch_table_t<2>(P, s); break;
      case 128: e = launch_table_t<4>(P, s); break;
      default: e = launch_table_t<8>(P, s); break;
    }
    if (e != hipSuccess) return e;
  }
  switch (P.nbits) {
    case 1: return launch_score_dim<1>(P, s);
    case 2: return launch_score_dim<2>(P, s);
    default: return launch_score_dim<4>(P, s);
  }
}
