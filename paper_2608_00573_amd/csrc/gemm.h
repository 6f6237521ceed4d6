// Arguments and lane helpers shared by the matrix kernels (gemm.hip, skinny.hip)
// and the routing (decide.hip).  Not part of the public ABI.
#pragma once

#include "common.h"

namespace trimmoe {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

static inline int cdiv(int a, int b) { return (a + b - 1) / b; }

typedef __attribute__((address_space(3))) char lds_byte;

__device__ __forceinline__ uint32_t lds_addr(const char* p) {
  return (uint32_t)(uintptr_t)(const lds_byte*)(p);
}

// 16-byte chunk c of row r sits at chunk c ^ swz16(r) of its LDS row: 8
// consecutive rows, or 16 consecutive rows split by parity, then touch distinct
// bank groups
__device__ __forceinline__ int swz16(int r) { return (r & 7) ^ ((r >> 3) & 1); }

// barrier for plain LDS traffic that leaves vector-memory operations in flight
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// ----------------------------------------------- activation helpers --
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float swap_pair(float v) {
  // lane l reads lane l ^ 1 (quad_perm [1, 0, 3, 2])
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xb1, 0xf,
                                                             0xf, false));
}

// The values of lanes l and l ^ 16 (lanes_xor16) or l and l ^ 32
// (lanes_xor32) in every lane, by gfx950's permlane swaps instead of an LDS
// exchange: (a, b) is (own, other) in lanes 0..15 (xor16: every even row of
// 16 lanes) or 0..31 (xor32) and (other, own) in the rest, so a commutative
// reduction of a and b gives every lane the pair's result.  The two results
// are copied out of the returned pair before the bit casts: a bit cast of
// the subscripted second element read the first one.
struct LanePair {
  float a, b;
};
__device__ __forceinline__ LanePair lanes_xor16(float x) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const unsigned r0 = r[0], r1 = r[1];
  return {__builtin_bit_cast(float, r0), __builtin_bit_cast(float, r1)};
}
__device__ __forceinline__ LanePair lanes_xor32(float x) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const unsigned r0 = r[0], r1 = r[1];
  return {__builtin_bit_cast(float, r0), __builtin_bit_cast(float, r1)};
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const bf16x2_t v = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, v);
}

// silu(g) u = g u / (1 + e^-g) with the hardware exp2 and reciprocal (about
// 1 ulp each in fp32; callers round the result to bf16)
__device__ __forceinline__ float silu_mul(float g, float u) {
  return g * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-g * 1.4426950408889634f)) * u;
}

// Engine-clock record (measurement only): with a record set, a block adds the
// core clock cycles (s_memtime) and the 100 MHz constant-clock ticks
// (s_memrealtime) between its start and the end of its work to rec[0] and
// rec[1]; their ratio is the mean engine clock under the kernel.  The start
// values are subtracted at once (modulo 2^64) and the end values added at
// the end, so nothing is held in registers in between.
__device__ __forceinline__ void clock_mark(unsigned long long* rec, bool start) {
  if (rec && threadIdx.x == 0) {
    const unsigned long long t = __builtin_amdgcn_s_memtime();
    const unsigned long long r = __builtin_amdgcn_s_memrealtime();
    atomicAdd(rec, start ? 0ull - t : t);
    atomicAdd(rec + 1, start ? 0ull - r : r);
  }
}

// arguments of a grouped (or dense) FFN GEMM
struct FfnArgs {
  const bf16_t* X;        // [rows, K], or h [T, K] when x_idx is set
  const int* x_idx;       // row -> source row of X (gather), or NULL
  const bf16_t* W0;       // expert 0 of [E, N, K] (up, or down)
  const bf16_t* W1;       // gate, same layout, or NULL
  size_t w_stride;        // elements between experts
  int K, N;
  const int4* tiles;      // grouped mode
  const int* n_tiles;     // grouped mode: live tiles (device)
  const int* dense_rows;  // dense mode: live rows (device), else NULL
  void* out;              // up: bf16 [rows, N]; down: f32 [split][rows, N]
  const int* n_rows;      // down GEMM: live rows (device), the rows of a split slice
  long long cap_rows;     // ... rows `out` holds (live_down_splits), or 0: one slice
  int act;                // up: TRIMMOE_ACT_*
  int* sk_flag;           // large-group down GEMM: per-tile piece words (see SkPlan), or NULL
  float* sk_part;         // ... and the compact partials of pieces 1.. of cut tiles
  unsigned long long* clk;  // engine-clock record of this class (see clock_mark), or NULL
};

// arguments of an exit-head GEMM
struct ExitArgs {
  const bf16_t* W;    // [V, K]
  const bf16_t* H;    // [n_x, K]
  const float* bias;  // [V] or NULL
  const int* n_exec;  // device
  int V, K, n_vtiles;
  float2* partials;   // [n_x, n_vtiles]
  unsigned long long* clk;  // engine-clock record (see clock_mark), or NULL
};

// decode-sized batches (skinny.hip)
hipError_t launch_ffn_skinny(const FfnArgs& a, bool up, bool dual, int n_cu, hipStream_t st);
hipError_t launch_exit_skinny(const ExitArgs& a, bool argmax, hipStream_t st);

}  // namespace trimmoe
