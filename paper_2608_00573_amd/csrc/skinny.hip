// Weight-streaming GEMMs for decode-sized batches (bf16): grouped up/gate and
// down projections of up to kSkinnyTokens tokens, the shared expert of up to
// kSkinnyDenseTokens, and exit heads of up to kSkinnyTokens tokens where they
// beat the 128 x 32 tiles (exit_streams).
//
// With a few rows per expert every weight is used once per row tile, so the
// kernels are bound by reading W from HBM, and by the texture path that
// every load passes: a load whose neighbouring lanes read different rows (what
// an MFMA operand needs in registers) takes four times the address cycles of
// one whose lanes run along a row.  So
//   * W goes to LDS by buffer-to-LDS DMA, lanes along the rows (runs of 64 U
//     bytes), into a ring of two sets that only its own wavefront reads: no
//     barrier and no staging registers, one vmcnt wait per set;
//   * the activations (B operand, 16 token rows per MFMA) come from L2 into
//     registers with the set.  A unit of two 16-column groups halves that
//     traffic, and their producers leave them in operand order (frag_order),
//     so that a load is one contiguous run; only the up projection gathers h
//     rows;
//   * a unit is 32 output columns (a group is the 16 rows of a
//     v_mfma_f32_16x16x32_bf16 A operand) over the whole K; the four
//     wavefronts of a block (one per SIMD) split its k-steps, keep the next
//     set in flight under the current one across unit boundaries, and add
//     their parts through LDS in wavefront order.
// A block takes a contiguous range of groups (of an odd one the last unit's
// second group has no records and costs no memory traffic), blocks of one XCD
// next to each other, so they share the activation rows in its L2.
// The DMA carries the non-temporal hint: single-use weights leave the
// activations in L2 (up/gate 5.7 -> 6.3 TB/s).
//
// Mixtral layer shapes on an MI355X, against the 128-row tiles (us, weights
// read): 1 token: up/gate 84 -> 76, down 58 -> 42, exit head 64 -> 45 (5.8 TB/s);
// 16 tokens: 210 -> 165 (6.4 TB/s), 108 -> 86 (6.1), 63 -> 45; 64 tokens: 216 ->
// 195, 112 -> 108, 79 -> 56, where four token tiles make the activations twice
// the weights' traffic.  A plain read kernel reaches 6.2-6.6 TB/s.  Qwen shapes,
// 16 tokens: up 54 -> 42, down 29 -> 27, shared expert 104 -> 27, exit 125 -> 97.
// Above kSkinnyTokens the activations would outweigh the weights further and
// the matrix cores no longer wait for them: the 128-row tiles take over (the
// shared expert's weights stay in the last-level cache for a second pass).
#include <math.h>

#include "gemm.h"

namespace trimmoe {

namespace skinny {
constexpr int COLS = 16;                         // output columns of a group
constexpr int WAVES = 4, THREADS = 64 * WAVES;
constexpr int MT_MAX = kSkinnyTokens / 16;
constexpr int RING = 128 * 1024;                 // the wavefronts' rings
constexpr int RED = 32 * 1024;                   // K parts of one group of columns
constexpr int LDS = RING + RED;
constexpr int KSTEP = 32;                        // K of one MFMA
}  // namespace skinny

// LDS reads and writes of the sums and fragments are asm: the compiler cannot
// tell that they never alias a DMA in flight and would wait for all of them.
// Every read waits for its own data in the same statement.
template <int N, int STRIDE>
struct LdsRead;
template <int STRIDE>
struct LdsRead<4, STRIDE> {
  template <class V>
  static __device__ __forceinline__ void get(uint32_t a, V (&v)[4]) {
    asm volatile(
        "ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:%5\n\tds_read_b128 %2, %4 offset:%6\n\t"
        "ds_read_b128 %3, %4 offset:%7\n\ts_waitcnt lgkmcnt(0)"
        : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
        : "v"(a), "n"(STRIDE), "n"(2 * STRIDE), "n"(3 * STRIDE)
        : "memory");
  }
};
template <int STRIDE>
struct LdsRead<1, STRIDE> {
  template <class V>
  static __device__ __forceinline__ void get(uint32_t a, V (&v)[1]) {
    asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(v[0]) : "v"(a) : "memory");
  }
};
// K parts of a sum; the remarks name the layout of the sum area (bytes of a
// wavefront's parts, whether the halves of the area alternate), by which the
// check of the generated code tells the streams apart
template <int PART, bool PAR>
__device__ __forceinline__ void part_put(uint32_t a, f32x4_t v) {
  asm volatile("ds_write_b128 %0, %1 ; part write %2 %3" ::"v"(a), "v"(v), "n"(PART), "n"(PAR)
               : "memory");
}
template <int PART, bool PAR>
__device__ __forceinline__ void parts_get(uint32_t a, f32x4_t (&v)[4]) {
  asm volatile(
      "ds_read_b128 %0, %4 ; part read %5 %8\n\tds_read_b128 %1, %4 offset:%5\n\t"
      "ds_read_b128 %2, %4 offset:%6\n\tds_read_b128 %3, %4 offset:%7\n\ts_waitcnt lgkmcnt(0)"
      : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
      : "v"(a), "n"(PART), "n"(2 * PART), "n"(3 * PART), "n"(PAR)
      : "memory");
}

// range of units of this block, blocks of one XCD (dealt b % 8) in a row
__device__ __forceinline__ void skinny_range(long total, long& u0, long& u1) {
  const int P = gridDim.x, nx = min(8, P), x = blockIdx.x % nx;
  const int v = x * (P / nx) + min(x, P % nx) + (int)blockIdx.x / nx;
  u0 = total * v / P;
  u1 = total * (v + 1) / P;
}

// set shapes: two groups of 512-byte runs, four of 256-byte runs (kMid), or
// the shortest K
enum { kLong, kMid, kShort };

// shape of a stream: NB weight operands, MT token tiles, G groups per unit, U
// k-steps per set (16 KB sets but for the shortest K)
template <int NB_, int MT_, int KIND>
struct Stream {
  static constexpr int NB = NB_, MT = MT_, G = NB == 1 && KIND == kMid ? 4 : 2,
                       U = KIND == kShort ? 2 : 16 / (NB * G);
  static constexpr int NW = NB * G;             // weight tiles of 16 rows
  static constexpr int SET = NW * U * 1024;     // LDS bytes of a set
  static constexpr int OPS = NW * U + MT * U;   // vector-memory operations of a set
  // K parts of GR groups meet at once, a wavefront adding the tile (group,
  // token tile) of its number; PAR: the buffer alternates, so that a round
  // needs one barrier (while the layout stays: between streams of different
  // shapes the block needs one more)
  static constexpr int GR = skinny::WAVES * NB * G * MT * 1024 <= skinny::RED && G * MT <= skinny::WAVES ? G : 1;
  static constexpr int PART = NB * GR * MT * 1024;
  static constexpr bool PAR = 2 * skinny::WAVES * PART <= skinny::RED;
  static constexpr int TILES = GR * MT;
  static_assert(2 * SET * skinny::WAVES <= skinny::RING, "two sets per wavefront");
  static_assert(skinny::WAVES * PART <= skinny::RED, "K parts of a round");
  static_assert(TILES <= skinny::WAVES, "a wavefront adds one tile");
  static_assert(OPS <= 63, "vmcnt field");
  static_assert(U == 2 || U == 4 || U == 8, "rows of whole swizzle groups");
};

// the lane's activation operand: element 0 of token tile m at k-step s is at
// p[m] + s * step[m]
template <int MT>
struct XSrc {
  const bf16_t* p[MT];
  int step[MT];
};

// Streams units 0 .. units - 1.  wbase(u, o) is operand o's first row of unit
// u (wave-uniform), wrows(u) the rows of it that exist; ks the k-steps of K
// (at least U); epi(u, acc) gets this wavefront's part of the unit's tiles
// (lane: token lane % 16, columns 4 (lane / 16) .. + 4 of group g).  Every
// wavefront calls epi once per unit.
template <class T, class WBase, class WRows, class Epi>
__device__ __forceinline__ void skinny_stream(char* lds, const XSrc<T::MT>& xs, int units, int ks,
                                              WBase wbase, WRows wrows, Epi epi) {
  constexpr int NB = T::NB, G = T::G, MT = T::MT, U = T::U;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  // (in pairs of k-steps: whole 128-byte lines)
  const int s0 = ks / 2 * wave / skinny::WAVES * 2, s1 = ks / 2 * (wave + 1) / skinny::WAVES * 2;
  const int nc = (s1 - s0 + U - 1) / U;  // sets per unit
  f32x4_t acc[NB][G][MT];
  auto zero = [&] {
#pragma unroll
    for (int o = 0; o < NB; ++o)
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[o][g][m] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  };
  zero();
  if (nc == 0) {  // K shorter than the wavefronts: this one only joins the sums
    for (int u = 0; u < units; ++u) epi(u, acc);
    return;
  }
  const uint32_t ring = lds_addr(lds) + wave * 2 * T::SET;
  // DMA lanes: LPR lanes run along a row of the set, RPI rows per operation
  constexpr int LPR = 4 * U, RPI = 64 / LPR;
  const uint32_t rowb = (uint32_t)ks * (skinny::KSTEP * 2);
  // the last set of a unit: chunks outside the wavefront's k-steps lie past
  // the records (they read zeros and cost no memory traffic)
  const int ls = s0 + (nc - 1) * U, lg = min(ls, ks - U);
  uint32_t voff[U], vlast[U];
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int r = j * RPI + lane / LPR, ch = (lane % LPR) ^ swz16(r), s = lg + ch / 4;
    voff[j] = r * rowb + (ch << 4);
    vlast[j] = s >= ls && s < s1 ? voff[j] : 0x80000000u;
  }
  // fragment reads: row lane % 16, chunk 4 s + lane / 16; even and odd k-steps
  const int fr = lane & 15, q = lane >> 4;
  const uint32_t fa0 = fr * (U * 64) + ((q ^ swz16(fr)) << 4);
  const uint32_t fa1 = fr * (U * 64) + (((4 + q) ^ swz16(fr)) << 4);

  struct Set {
    bf16x8_t x[MT][U];
    int lo, hi;  // k-steps of the set that belong to it
  };
  // load side: set lc of unit lu; a short last set starts earlier so that it
  // stays inside K (its leading k-steps are not used), and past the last
  // unit the last set is read again (never used)
  int lu = 0, lc = 0;
  auto load = [&](Set& S, int half) {
    const int st = s0 + lc * U, g0 = min(st, ks - U);
    S.lo = st - g0;
    S.hi = min(st + U, s1) - g0;
    const int rows = wrows(lu);
    const bool tail = lc == nc - 1;
#pragma unroll
    for (int o = 0; o < NB; ++o) {
      const bf16_t* base = wbase(lu, o);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        // rows past the end read zeros
        const int n =
            __builtin_amdgcn_readfirstlane(min(max(rows - g * skinny::COLS, 0), skinny::COLS));
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<bf16_t*>(base + (size_t)g * skinny::COLS * (rowb / 2)), (short)0,
            (int)(n * rowb), 0x00020000);
#pragma unroll
        for (int j = 0; j < U; ++j)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(
              rs,
              (lds_byte*)(uintptr_t)(ring + half * T::SET + ((o * G + g) * U + j) * 1024), 16,
              tail ? vlast[j] : voff[j], (uint32_t)g0 * (skinny::KSTEP * 2), 0, 2);
      }
    }
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const bf16_t* p = xs.p[m] + (size_t)g0 * xs.step[m];
#pragma unroll
      for (int s = 0; s < U; ++s)
        S.x[m][s] = *reinterpret_cast<const bf16x8_t*>(p + s * xs.step[m]);
    }
    if (++lc == nc) {
      lc = 0;
      if (lu + 1 < units)
        ++lu;
      else
        lc = nc - 1;
    }
  };
  int cu = 0, cc = 0;
  auto compute = [&](Set& S, int half) {
    // everything of this set has landed: only the next set's operations are
    // newer (the builtin, so that the compiler knows it of the activations)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((T::OPS & 15) | (T::OPS >> 4) << 14 | 0xf70);
    asm volatile("" ::: "memory");
    const uint32_t st = ring + half * T::SET;
#pragma unroll
    for (int o = 0; o < NB; ++o)
#pragma unroll
      for (int g = 0; g < G; ++g) {
        bf16x8_t w[U];
        const uint32_t t = st + (o * G + g) * U * 1024;
        if constexpr (U == 8) {
          bf16x8_t e[4], d[4];
          LdsRead<4, 128>::get(t + fa0, e);
          LdsRead<4, 128>::get(t + fa1, d);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            w[2 * i] = e[i];
            w[2 * i + 1] = d[i];
          }
        } else {
#pragma unroll
          for (int i = 0; i < U / 2; ++i) {
            bf16x8_t e[1], d[1];
            LdsRead<1, 0>::get(t + fa0 + 128 * i, e);
            LdsRead<1, 0>::get(t + fa1 + 128 * i, d);
            w[2 * i] = e[0];
            w[2 * i + 1] = d[0];
          }
        }
#pragma unroll
        for (int s = 0; s < U; ++s)
          if (s >= S.lo && s < S.hi) {
#pragma unroll
            for (int m = 0; m < MT; ++m)
              acc[o][g][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[s], S.x[m][s], acc[o][g][m],
                                                                     0, 0, 0);
          }
      }
    if (++cc == nc) {
      cc = 0;
      epi(cu, acc);
      zero();
      ++cu;
    }
  };
  Set A, B;
  const int total = units * nc;
  load(A, 0);
  for (int i = 0; i < total; i += 2) {
    load(B, 1);
    compute(A, 0);
    if (i + 1 >= total) break;
    load(A, 0);
    compute(B, 1);
  }
  // the ring is reused by the next stream of this wavefront
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// K parts of groups g0 .. g0 + GR - 1 of a unit through LDS: every wavefront
// leaves its tiles, and wavefront w < TILES gets the sums (in wavefront order)
// of group g0 + w / MT, token tile w % MT, in v
template <class T>
__device__ __forceinline__ bool skinny_sum(char* lds, int& par,
                                           const f32x4_t (&acc)[T::NB][T::G][T::MT], int g0,
                                           f32x4_t (&v)[T::NB]) {
  constexpr int NB = T::NB, MT = T::MT, GR = T::GR;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const uint32_t red =
      lds_addr(lds) + skinny::RING + lane * 16 + (T::PAR ? par * skinny::WAVES * T::PART : 0);
  par ^= 1;
  // the compiler does not see that the asm stores read the results of MFMAs
  // (19 wait states at most for these)
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7");
#pragma unroll
  for (int o = 0; o < NB; ++o)
#pragma unroll
    for (int g = 0; g < GR; ++g)
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        f32x4_t t = acc[o][g0 + g][m];
        part_put<T::PART, T::PAR>(red + wave * T::PART + ((o * GR + g) * MT + m) * 1024, t);
      }
  lds_barrier();
  if (wave < T::TILES) {
#pragma unroll
    for (int o = 0; o < NB; ++o) {
      f32x4_t p[4];
      parts_get<T::PART, T::PAR>(red + (o * T::TILES + wave) * 1024, p);
      v[o] = p[0];
#pragma unroll
      for (int w = 1; w < 4; ++w)
#pragma unroll
        for (int r = 0; r < 4; ++r) v[o][r] += p[w][r];
    }
  }
  if constexpr (!T::PAR) lds_barrier();
  return wave < T::TILES;
}

// ------------------------------------------------------ grouped FFN GEMMs --
// rows [m0, m0 + rows) of one tile, output columns [n0, n1).  The down
// projection reads X in operand order (frag_order), which the up projection
// writes.
template <class T, bool UP>
__device__ __forceinline__ void skinny_ffn_rows(const FfnArgs& a, char* lds, int& par, int e, int m0,
                                                int rows, int n0, int n1) {
  constexpr int NB = T::NB, G = T::G, MT = T::MT;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int fr = lane & 15, q = lane >> 4;
  XSrc<MT> xs;
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    if constexpr (!UP) {
      const int b = 16 * m < rows ? 16 * m : 0;  // tiles past the rows repeat the first
      const int n = min(16, rows - b);
      xs.p[m] = a.X + (size_t)(m0 + b) * a.K + frag_order(0, q, min(fr, n - 1), n);
      xs.step[m] = frag_order(1, 0, 0, n);
    } else {
      const int r = m0 + min(16 * m + fr, rows - 1);
      xs.p[m] = a.X + (size_t)(a.x_idx ? a.x_idx[r] : r) * a.K + 8 * q;
      xs.step[m] = skinny::KSTEP;
    }
  }
  const size_t wo = (size_t)e * a.w_stride + (size_t)n0 * a.K;
  const size_t ustride = (size_t)(skinny::COLS * G) * a.K;
  auto wbase = [&](int u, int o) { return (o ? a.W1 : a.W0) + wo + u * ustride; };
  auto wrows = [&](int u) { return n1 - n0 - u * skinny::COLS * G; };
  const int tm = wave % MT, tg = wave / MT;  // the tile this wavefront adds
  auto epi = [&](int u, const f32x4_t(&acc)[NB][G][MT]) {
#pragma unroll
    for (int g = 0; g < G; g += T::GR) {
      f32x4_t v[NB];
      const bool mine = skinny_sum<T>(lds, par, acc, g, v);
      const int row = 16 * tm + fr;
      const int c = n0 + (u * G + g + tg) * skinny::COLS + 4 * q;
      if (!mine || row >= rows || c >= n1) continue;
      if constexpr (UP) {
        float x[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if constexpr (NB == 2)
            x[r] = silu_mul(v[1][r], v[0][r]);
          else
            x[r] = fmaxf(v[0][r], 0.f);
        }
        // operand order of the down projection: k-step c / 32, group c % 32 / 8
        const int b = 16 * tm, n = min(16, rows - b);
        const size_t o = (size_t)(m0 + b) * a.N + frag_order(c >> 5, (c >> 3) & 3, fr, n) + (c & 7);
        *reinterpret_cast<uint2*>(static_cast<bf16_t*>(a.out) + o) =
            make_uint2(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]));
      } else {
        *reinterpret_cast<f32x4_t*>(static_cast<float*>(a.out) + (size_t)(m0 + row) * a.N + c) = v[0];
      }
    }
  };
  const int units = (n1 - n0 + skinny::COLS * G - 1) / (skinny::COLS * G);
  skinny_stream<T>(lds, xs, units, a.K / skinny::KSTEP, wbase, wrows, epi);
  // the block's next tile may be of another width, which lays the sums out
  // anew: every wavefront has to be past its reads of the last one first
  if constexpr (T::PAR) lds_barrier();
}

// the widest batches halve their activation traffic with four groups per unit
// (exit head of 64 tokens, K = 4096: 70 -> 59 us; below, 512-byte runs of W
// are worth more: 48 against 51 us at one token)
constexpr int wide_kind(int kind) { return kind == kLong ? kMid : kind; }

template <int NB, bool UP, int KIND>
__global__ __launch_bounds__(skinny::THREADS) void k_ffn_skinny(FfnArgs a) {
  __shared__ __align__(16) char lds[skinny::LDS];
  const int dense_m1 = a.dense_rows ? *a.dense_rows : 0;
  // (wave-uniform, as the addresses of the weights have to be)
  const int n_mt = __builtin_amdgcn_readfirstlane(
      a.dense_rows ? (dense_m1 + kSkinnyTokens - 1) / kSkinnyTokens : *a.n_tiles);
  const int npt = a.N / skinny::COLS;  // groups per row tile; N is a multiple of 64
  long u, u1;
  skinny_range((long)n_mt * npt, u, u1);
  if (u >= u1) return;
  clock_mark(a.clk, true);
  int par = 0;
  while (u < u1) {
    // the block's groups of one row tile
    const int mt = (int)(u / npt), c0 = (int)(u - (long)mt * npt);
    const int groups = min((int)(u1 - u), npt - c0);
    int e = 0, m0 = mt * kSkinnyTokens, m1 = dense_m1;
    if (!a.dense_rows) {
      const int4 tl = a.tiles[mt];
      e = __builtin_amdgcn_readfirstlane(tl.x);
      m0 = __builtin_amdgcn_readfirstlane(tl.y);
      m1 = __builtin_amdgcn_readfirstlane(tl.z);
    }
    // an expert's tile of a batch of at most kSkinnyTokens tokens has no more
    // rows; dense tiles are that long
    const int rows = min(m1 - m0, kSkinnyTokens);
    const int n0 = c0 * skinny::COLS, n1 = n0 + groups * skinny::COLS;
    if (rows <= 16)
      skinny_ffn_rows<Stream<NB, 1, KIND>, UP>(a, lds, par, e, m0, rows, n0, n1);
    else if (rows <= 32)
      skinny_ffn_rows<Stream<NB, 2, KIND>, UP>(a, lds, par, e, m0, rows, n0, n1);
    else
      skinny_ffn_rows<Stream<NB, 4, wide_kind(KIND)>, UP>(a, lds, par, e, m0, rows, n0, n1);
    u += groups;
  }
  clock_mark(a.clk, false);
}

// -------------------------------------------------------------- exit head --
// Block b of the grid takes the b-th run of 16-row vocabulary groups and keeps
// a running softmax partial (base 2: largest y = z log2 e, sum 2^(y - max))
// or, ARGMAX, the largest logit and its row, per token; one partial per token
// and block (n_vtiles is the grid).  The softmax reads hx in operand order,
// the argmax a caller's rows.
template <bool ARGMAX, class T>
__device__ __forceinline__ void skinny_exit_rows(const ExitArgs& a, char* lds, int n_x, int v0,
                                                 int v1) {
  constexpr int MT = T::MT, UC = T::G * skinny::COLS;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int fr = lane & 15, q = lane >> 4;
  XSrc<MT> xs;
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    if constexpr (ARGMAX) {
      xs.p[m] = a.H + (size_t)min(16 * m + fr, n_x - 1) * a.K + 8 * q;
      xs.step[m] = skinny::KSTEP;
    } else {
      const int b = 16 * m < n_x ? 16 * m : 0;
      const int n = min(16, n_x - b);
      xs.p[m] = a.H + (size_t)b * a.K + frag_order(0, q, min(fr, n - 1), n);
      xs.step[m] = frag_order(1, 0, 0, n);
    }
  }
  auto wbase = [&](int u, int) { return a.W + (size_t)(v0 + u * UC) * a.K; };
  auto wrows = [&](int u) { return v1 - v0 - u * UC; };
  const float ninf = -__builtin_inff();
  const float kLog2e = 1.4426950408889634f;
  float M = ninf, S = 0.f;  // of the lane's token (wavefront m < MT: tile m), its rows 4 q .. + 4
  int R = v0;  // ... while no logit is above -inf
  auto group = [&](int r0, const f32x4_t& v) {
    float y[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float z = v[r];
      if (a.bias) z += a.bias[min(r0 + r, a.V - 1)];
      if constexpr (!ARGMAX) z *= kLog2e;
      y[r] = r0 + r < v1 ? z : ninf;
    }
    if constexpr (ARGMAX) {
      // rows come in increasing order: ties keep the lower row
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (r0 + r < v1 && (y[r] > M || (y[r] == M && r0 + r < R))) {
          M = y[r];
          R = r0 + r;
        }
    } else {
      const float m = fmaxf(M, fmaxf(fmaxf(y[0], y[1]), fmaxf(y[2], y[3])));
      if (m != ninf) {
        float t = M != ninf ? S * __builtin_amdgcn_exp2f(M - m) : 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) t += __builtin_amdgcn_exp2f(y[r] - m);
        S = t;
        M = m;
      }
    }
  };
  int par = 0;
  auto epi = [&](int u, const f32x4_t(&acc)[1][T::G][MT]) {
#pragma unroll
    for (int g = 0; g < T::G; g += T::GR) {
      f32x4_t v[1];
      if (skinny_sum<T>(lds, par, acc, g, v))
        group(v0 + u * UC + (g + wave / MT) * skinny::COLS + 4 * q, v[0]);
    }
  };
  const int units = (v1 - v0 + UC - 1) / UC;
  skinny_stream<T>(lds, xs, units, a.K / skinny::KSTEP, wbase, wrows, epi);
  // the four row groups of a token (lanes l, l ^ 16, l ^ 32, l ^ 48), then the
  // wavefronts that added its tile
  auto merge = [&](float m0, float s0, int r0, float m1, float s1, int r1) {
    if constexpr (ARGMAX) {
      const bool take = m1 > m0 || (m1 == m0 && r1 < r0);
      M = take ? m1 : m0;
      R = take ? r1 : r0;
    } else {
      M = fmaxf(m0, m1);
      S = 0.f;
      if (s0 > 0.f) S += s0 * __builtin_amdgcn_exp2f(m0 - M);
      if (s1 > 0.f) S += s1 * __builtin_amdgcn_exp2f(m1 - M);
    }
  };
#pragma unroll
  for (int step = 0; step < 2; ++step) {
    const LanePair pm = step ? lanes_xor32(M) : lanes_xor16(M);
    const float x = ARGMAX ? __int_as_float(R) : S;
    const LanePair px = step ? lanes_xor32(x) : lanes_xor16(x);
    merge(pm.a, px.a, __float_as_int(px.a), pm.b, px.b, __float_as_int(px.b));
  }
  float2* fin = reinterpret_cast<float2*>(lds);  // the ring is drained
  __syncthreads();
  if (q == 0 && wave < T::TILES) fin[wave * 16 + fr] = make_float2(M, ARGMAX ? __int_as_float(R) : S);
  __syncthreads();
  const int t = 16 * wave + fr;
  if (q != 0 || wave >= MT || t >= n_x) return;
#pragma unroll
  for (int g = 1; g < T::GR; ++g) {
    const float2 o = fin[(g * MT + wave) * 16 + fr];
    merge(M, S, R, o.x, o.y, __float_as_int(o.y));
  }
  a.partials[(size_t)t * a.n_vtiles + blockIdx.x] = make_float2(M, ARGMAX ? __int_as_float(R) : S);
}

template <bool ARGMAX, int KIND>
__global__ __launch_bounds__(skinny::THREADS) void k_exit_skinny(ExitArgs a) {
  __shared__ __align__(16) char lds[skinny::LDS];
  const int n_x = min(*a.n_exec, kSkinnyTokens);
  if (n_x <= 0) return;
  clock_mark(a.clk, true);
  const long n_u = (a.V + skinny::COLS - 1) / skinny::COLS;
  const int u0 = (int)(n_u * blockIdx.x / gridDim.x), u1 = (int)(n_u * (blockIdx.x + 1) / gridDim.x);
  const int v0 = u0 * skinny::COLS, v1 = min(u1 * skinny::COLS, a.V);
  if (n_x <= 16)
    skinny_exit_rows<ARGMAX, Stream<1, 1, KIND>>(a, lds, n_x, v0, v1);
  else if (n_x <= 32)
    skinny_exit_rows<ARGMAX, Stream<1, 2, KIND>>(a, lds, n_x, v0, v1);
  else
    skinny_exit_rows<ARGMAX, Stream<1, 4, wide_kind(KIND)>>(a, lds, n_x, v0, v1);
  clock_mark(a.clk, false);
}

// -------------------------------------------------------------- launchers --
// set shape for a K of ks k-steps: sets must fit K
static int stream_kind(int ks) { return ks < 8 ? kShort : kLong; }

template <int NB, bool UP>
static void launch_ffn(const FfnArgs& a, int n_cu, hipStream_t st) {
  const dim3 grid(n_cu), block(skinny::THREADS);
  if (stream_kind(a.K / skinny::KSTEP) == kShort)
    hipLaunchKernelGGL((k_ffn_skinny<NB, UP, kShort>), grid, block, 0, st, a);
  else
    hipLaunchKernelGGL((k_ffn_skinny<NB, UP, kLong>), grid, block, 0, st, a);
}

hipError_t launch_ffn_skinny(const FfnArgs& a, bool up, bool dual, int n_cu, hipStream_t st) {
  if (up && dual)
    launch_ffn<2, true>(a, n_cu, st);
  else if (up)
    launch_ffn<1, true>(a, n_cu, st);
  else
    launch_ffn<1, false>(a, n_cu, st);
  return hipGetLastError();
}

template <bool ARGMAX>
static void launch_exit(const ExitArgs& a, hipStream_t st) {
  const dim3 grid(a.n_vtiles), block(skinny::THREADS);
  if (stream_kind(a.K / skinny::KSTEP) == kShort)
    hipLaunchKernelGGL((k_exit_skinny<ARGMAX, kShort>), grid, block, 0, st, a);
  else
    hipLaunchKernelGGL((k_exit_skinny<ARGMAX, kLong>), grid, block, 0, st, a);
}

hipError_t launch_exit_skinny(const ExitArgs& a, bool argmax, hipStream_t st) {
  if (argmax)
    launch_exit<true>(a, st);
  else
    launch_exit<false>(a, st);
  return hipGetLastError();
}

}  // namespace trimmoe
