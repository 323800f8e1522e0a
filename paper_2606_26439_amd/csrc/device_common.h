// device_common.h -- shared device-side helpers of the gfx950 MaxSim kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

// Element types, same numbering as maxsim_dtype.
enum : int { DT_F32 = 0, DT_BF16 = 1, DT_F16 = 2, DT_FP8 = 3 };

template <int DT>
struct elem_size {
  static constexpr int value = DT == DT_F32 ? 4 : (DT == DT_FP8 ? 1 : 2);
};

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ int64_t uniform64(int64_t v) {
  uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)(uint64_t)v);
  uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ int64_t readlane64(int64_t v, int lane) {
  uint32_t lo = __builtin_amdgcn_readlane((uint32_t)(uint64_t)v, lane);
  uint32_t hi = __builtin_amdgcn_readlane((uint32_t)((uint64_t)v >> 32), lane);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ float xor_shfl(float v, int m) { return __shfl_xor(v, m, 64); }

// Cross-lane reductions of an MFMA 16x16 result without the LDS pipe (a
// ds_bpermute shuffle is an LDS round trip the wave waits for; register-to-
// register forms keep a wave that is alone on its SIMD issuing).
//
// Max over the four 16-lane rows (lanes i, i ^ 16, i ^ 32, i ^ 48), left in
// every lane: v_permlane16_swap exchanges odd and even rows between two
// copies of v, v_permlane32_swap the two half-waves. Written as assembly so
// the two swapped copies stay distinct values for the compiler. The
// compiler's hazard recognizer does not look inside inline assembly, so the
// block carries its own wait states. The CDNA4 ISA's table of manually
// inserted wait states requires, before a V_PERMLANE16_SWAP or
// V_PERMLANE32_SWAP, 2 wait states after a VALU write of a VGPR it reads and
// 4 after a V_CMPX write of EXEC; "s_nop 3" gives 4, covering both whatever
// the compiler schedules before the block. The "s_nop 1" after it keeps the
// swapped values two states away from their first reader. The whole wave
// executes it. (A CPU test builds kernels using it to gfx950 assembly and
// checks the wait states and that the max after each swap reads both
// registers.)
__device__ __forceinline__ float max_row_pairs(float v) {
  float a = v, b = v;
  asm volatile("s_nop 3\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
  return fmaxf(a, b);
}
__device__ __forceinline__ float max_half_waves(float v) {
  float a = v, b = v;
  asm volatile("s_nop 3\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
  return fmaxf(a, b);
}
__device__ __forceinline__ float max_rows4(float v) { return max_half_waves(max_row_pairs(v)); }
// Two values at once: lanes 0-31 get max(a_i, a_i+32), lanes 32-63 the same of
// b. The swap's two results are already different values, so no copies.
__device__ __forceinline__ float max_halves_of2(float a, float b) {
  asm volatile("s_nop 3\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
  return fmaxf(a, b);
}
// Four values at once: row q (16 lanes) gets value q's max over the four rows.
__device__ __forceinline__ float max_rows_of4(float v0, float v1, float v2, float v3) {
  float a = max_halves_of2(v0, v2), b = max_halves_of2(v1, v3);
  asm volatile("s_nop 3\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
  return fmaxf(a, b);
}

// Sum over the four 16-lane rows by the same two swaps, left in every lane:
// (v_r0 + v_r1) + (v_r2 + v_r3), the pairs and order of an xor butterfly
// over 16 then 32.
__device__ __forceinline__ float sum_rows4(float v) {
  float a = v, b = v;
  asm volatile("s_nop 3\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
  v = a + b;
  a = v;
  b = v;
  asm volatile("s_nop 3\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
  return a + b;
}

// Sum over the 16 lanes of each row, left in every lane of the row: four DPP
// row rotations (by 8, 4, 2, 1) with adds. Lane 0 adds the same pairs in the
// same order as an xor butterfly over 8, 4, 2, 1, so its value does not
// depend on which of the two forms a kernel uses.
__device__ __forceinline__ float row_sum16(float v) {
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x128,
                                                             0xF, 0xF, false));
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x124,
                                                             0xF, 0xF, false));
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x122,
                                                             0xF, 0xF, false));
  v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x121,
                                                             0xF, 0xF, false));
  return v;
}

// First index i in [0, n] with arr[i] >= key, for a non-decreasing arr of
// n + 1 entries with arr[n] >= key. Executed by a whole wavefront: each round
// probes 64 evenly spaced positions and keeps the bracket of the first hit,
// so a 1M-entry array takes 4 dependent loads instead of 20.
__device__ __forceinline__ int64_t wave_lower_bound(const int64_t* __restrict__ arr, int64_t n,
                                                    int64_t key) {
  const int lane = lane_id();
  int64_t lo = 0, hi = n;
  while (hi - lo + 1 > 64) {
    int64_t step = (hi - lo + 64) / 64;  // ceil((hi - lo + 1) / 64)
    int64_t pos = lo + step * lane;
    if (pos > hi) pos = hi;
    bool pred = arr[pos] >= key;
    uint64_t mask = __ballot(pred);
    if (mask & 1ull) return lo;  // arr[lo] >= key
    if (mask == 0) {
      lo = lo + step * 63 + 1;
    } else {
      int f = __ffsll((unsigned long long)mask) - 1;  // f >= 1
      int64_t pf = lo + step * f;
      if (pf > hi) pf = hi;
      lo = lo + step * (f - 1) + 1;
      hi = pf;
    }
  }
  int64_t pos = lo + lane;
  bool pred = pos <= hi && arr[pos < hi ? pos : hi] >= key;
  uint64_t mask = __ballot(pred);
  int f = mask ? __ffsll((unsigned long long)mask) - 1 : (int)(hi - lo);
  return lo + f;
}

// wave_lower_bound of two keys at once: every round's loads of both searches
// are in flight together.
__device__ __forceinline__ void wave_lower_bound2(const int64_t* __restrict__ arr, int64_t n,
                                                  int64_t key0, int64_t key1, int64_t& r0,
                                                  int64_t& r1) {
  const int lane = lane_id();
  int64_t lo0 = 0, hi0 = n, lo1 = 0, hi1 = n;
  // the bracket [lo, hi] of the first hit after a round of 64 probes
  auto narrow = [&](int64_t& lo, int64_t& hi, int64_t step, uint64_t mask) {
    if (mask & 1ull) {
      hi = lo;
    } else if (mask == 0) {
      lo = lo + step * 63 + 1;
    } else {
      const int f = __ffsll((unsigned long long)mask) - 1;  // f >= 1
      const int64_t pf = lo + step * f;
      hi = pf < hi ? pf : hi;
      lo = lo + step * (f - 1) + 1;
    }
  };
  while (hi0 - lo0 >= 64 || hi1 - lo1 >= 64) {
    const int64_t step0 = (hi0 - lo0 + 64) / 64, step1 = (hi1 - lo1 + 64) / 64;
    int64_t p0 = lo0 + step0 * lane, p1 = lo1 + step1 * lane;
    p0 = p0 < hi0 ? p0 : hi0;
    p1 = p1 < hi1 ? p1 : hi1;
    const int64_t v0 = arr[p0], v1 = arr[p1];
    const uint64_t m0 = __ballot(v0 >= key0), m1 = __ballot(v1 >= key1);
    narrow(lo0, hi0, step0, m0);
    narrow(lo1, hi1, step1, m1);
  }
  const int64_t p0 = lo0 + lane, p1 = lo1 + lane;
  const int64_t v0 = arr[p0 < hi0 ? p0 : hi0], v1 = arr[p1 < hi1 ? p1 : hi1];
  const uint64_t m0 = __ballot(p0 <= hi0 && v0 >= key0), m1 = __ballot(p1 <= hi1 && v1 >= key1);
  r0 = lo0 + (m0 ? __ffsll((unsigned long long)m0) - 1 : hi0 - lo0);
  r1 = lo1 + (m1 ? __ffsll((unsigned long long)m1) - 1 : hi1 - lo1);
}

// Last index a in [0, n) with arr[a] <= key for arr non-decreasing of n + 1
// entries, arr[0] <= key < arr[n]: the set that owns element `key`.
__device__ __forceinline__ int64_t wave_owner(const int64_t* __restrict__ arr, int64_t n,
                                              int64_t key) {
  // first i with arr[i] >= key + 1, minus one
  return wave_lower_bound(arr, n, key + 1) - 1;
}

// E8M0 exponent byte of a normal power-of-two float (2^k -> k + 127).
__device__ __forceinline__ int e8m0_of(float s) { return (int)((__float_as_uint(s) >> 23) & 0xFF); }

// Scalar (SMEM) loads of wave-uniform indices: reading through the constant
// address space makes the compiler use s_load, whose completion is tracked by
// lgkmcnt and therefore independent of the vector loads in flight.
typedef const __attribute__((address_space(4))) int64_t* const_i64_ptr;
typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;
__device__ __forceinline__ int64_t sload_i64(const int64_t* p, int64_t i) {
  return ((const_i64_ptr)p)[i];
}
__device__ __forceinline__ int sload_i32(const int32_t* p, int64_t i) {
  return ((const_i32_ptr)p)[i];
}

// 1 KiB of zeros (one wave's worth of 16-byte lanes; at least one chunk row
// of the widest element type): the target of the fixed-count loads a wave
// issues when it has nothing left to load, so those loads never depend on the
// caller's buffers being non-empty.
static __device__ __attribute__((aligned(16))) char g_zero_row[1024];

// The zero row's address, read once into scalar registers. The empty asm
// makes the value opaque, so the compiler keeps it in registers instead of
// re-reading it from the global offset table (a scalar load the wave must
// wait for) at every idle refill of a loop; the pointer stays typed as a
// global one through the asm, so loads from it remain global loads.
typedef const __attribute__((address_space(1))) char global_char;
__device__ __forceinline__ const char* zero_row_ptr() {
  global_char* p = (global_char*)g_zero_row;
  asm volatile("" : "+s"(p));
  return (const char*)p;
}

// Loads from global memory straight into LDS, and the waits that go with
// them. Lane l's B bytes (4 or 16) land at lds + l * B for the active lanes;
// lds is wave-uniform.
//
// Written as assembly because the compiler's wait insertion takes any LDS read
// that does not overlap a slot it can name as one that needs every such load
// in flight to have landed (a wait for all vector memory operations), which
// empties a ring of prefetched slots at each read of another table in LDS.
// The instruction has no register result, so nothing of it is in the
// register allocator's hands; the compiler only counts fewer operations in
// flight than there are, which makes its own waits stricter, never looser.
// The memory clobbers keep LDS accesses on their side of each load and wait.
// The loads take their LDS address from m0, which the compiler reserves and
// takes on no clobber list. Nothing else in a kernel that uses load_to_lds may
// use m0 (no LDS-DMA builtin, no indirect register index); a CPU test looks
// for it in the assembly.
// The wave's own count is the caller's: vmem_wait<N>() returns when at most N
// vector memory operations of the wave are in flight (they retire in order).
__device__ __forceinline__ uint32_t lds_offset(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)p;
}
template <int B, bool NT>
__device__ __forceinline__ void load_to_lds(const void* src, uint32_t lds) {
  static_assert(B == 4 || B == 16, "4 or 16 bytes per lane");
  lds = __builtin_amdgcn_readfirstlane(lds);
  if constexpr (B == 16 && NT)
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt"
                 :: "v"(src), "s"(lds) : "memory");
  else if constexpr (B == 16)
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :: "v"(src), "s"(lds) : "memory");
  else if constexpr (NT)
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off nt"
                 :: "v"(src), "s"(lds) : "memory");
  else
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off"
                 :: "v"(src), "s"(lds) : "memory");
}
template <int N>
__device__ __forceinline__ void vmem_wait() {
  static_assert(N >= 0 && N <= 63, "the counter has six bits");
  if constexpr (N == 0) {
    // visible to the compiler: its own loads need no further wait either
    // (vmcnt in bits 3:0 and 15:14, the other counters at their maxima)
    __builtin_amdgcn_s_waitcnt((0x7 << 4) | (0xF << 8));
    asm volatile("" ::: "memory");
  } else {
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
  }
}
// every LDS access issued so far is complete
__device__ __forceinline__ void lds_reads_wait() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
