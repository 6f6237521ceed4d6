// Exit-head training of Sec. IV-A on cached hidden states: the prediction of
// a representation (argmax of an output head, for the consistency labels of
// Eq. (22)) and full-batch gradient descent of the sigmoid exit head on the
// binary cross-entropy of Eq. (23).  Reductions run in a fixed order (fp64
// accumulators), so repeated runs give identical weights.
#include "common.h"

namespace trimmoe {

namespace {
inline int cdiv(int a, int b) { return (a + b - 1) / b; }
}  // namespace

__global__ void k_set_int(int32_t* p, int v) { *p = v; }

hipError_t launch_set_int(int32_t* p, int v, hipStream_t st) {
  hipLaunchKernelGGL(k_set_int, dim3(1), dim3(1), 0, st, p, v);
  return hipGetLastError();
}

// argmax over the vocabulary tiles of one row: the largest logit, ties to
// the lower vocabulary row.  One wavefront per row.
__global__ __launch_bounds__(256) void k_argmax_reduce(const float2* partials, int n_vtiles,
                                                       int n_rows, int32_t* out) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int q = blockIdx.x * 4 + wave;
  if (q >= n_rows) return;
  const float2* pr = partials + (size_t)q * n_vtiles;
  float m = -__builtin_inff();
  int mi = 0x7fffffff;
  for (int u = lane; u < n_vtiles; u += 64) {
    const float2 v = pr[u];
    const int r = __float_as_int(v.y);
    if (v.x > m || (v.x == m && r < mi)) {
      m = v.x;
      mi = r;
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    const float m2 = __shfl_xor(m, o);
    const int r2 = __shfl_xor(mi, o);
    if (m2 > m || (m2 == m && r2 < mi)) {
      m = m2;
      mi = r2;
    }
  }
  if (lane == 0) out[q] = mi;
}

hipError_t launch_argmax_reduce(const float2* partials, int n_vtiles, int n_rows, int32_t* out,
                                hipStream_t st) {
  if (n_rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_argmax_reduce, dim3(cdiv(n_rows, 4)), dim3(256), 0, st, partials,
                     n_vtiles, n_rows, out);
  return hipGetLastError();
}

// Eq. (22): labels[q] = 1 where the layer's prediction equals the full-depth one
__global__ void k_consistency(const int32_t* pred, const int32_t* ref, int n_rows,
                              uint8_t* labels) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < n_rows) labels[q] = pred[q] == ref[q] ? 1 : 0;
}

hipError_t launch_consistency(const int32_t* pred, const int32_t* ref, int n_rows,
                              uint8_t* labels, hipStream_t st) {
  if (n_rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_consistency, dim3(cdiv(n_rows, 256)), dim3(256), 0, st, pred, ref, n_rows,
                     labels);
  return hipGetLastError();
}

// Logit z = w . h + c of every row (one wavefront per row, fixed butterfly),
// the residual sigmoid(z) - y of the gradient and the row's loss
// max(z, 0) - y z + log(1 + exp(-|z|)) of Eq. (23).
template <typename T>
__global__ __launch_bounds__(256) void k_bce_logits(const T* H, const uint8_t* y, int n_rows, int d,
                                                    const float* w, const float* c, float* r,
                                                    double* row_loss) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int q = blockIdx.x * 4 + wave;
  if (q >= n_rows) return;
  const T* h = H + (size_t)q * d;
  float acc = 0.f;
  for (int k = lane; k < d; k += 64) acc = fmaf(w[k], to_f32<T>(h[k]), acc);
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
  if (lane == 0) {
    const float z = acc + *c;
    const float label = y[q] ? 1.f : 0.f;
    r[q] = 1.f / (1.f + expf(-z)) - label;
    const double zd = z;
    row_loss[q] = fmax(zd, 0.0) - (double)label * zd + log1p(exp(-fabs(zd)));
  }
}

// w[k] -= lr * sum_q r[q] h[q][k] / Q, one column per thread, rows in order;
// block 0 also moves c by lr * mean r and writes the mean loss.
template <typename T>
__global__ __launch_bounds__(256) void k_bce_update(const T* H, int n_rows, int d, float lr,
                                                    const float* r, const double* row_loss,
                                                    float* w, float* c, float* loss_out) {
  __shared__ double s_r[256], s_l[256];
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k < d) {
    double g = 0.0;
    for (int q = 0; q < n_rows; ++q) g += (double)r[q] * (double)to_f32<T>(H[(size_t)q * d + k]);
    w[k] -= lr * (float)(g / n_rows);
  }
  if (blockIdx.x != 0) return;
  double sr = 0.0, sl = 0.0;
  for (int q = threadIdx.x; q < n_rows; q += 256) {
    sr += (double)r[q];
    sl += row_loss[q];
  }
  s_r[threadIdx.x] = sr;
  s_l[threadIdx.x] = sl;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      s_r[threadIdx.x] += s_r[threadIdx.x + s];
      s_l[threadIdx.x] += s_l[threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *c -= lr * (float)(s_r[0] / n_rows);
    if (loss_out) *loss_out = (float)(s_l[0] / n_rows);
  }
}

hipError_t launch_bce_step(bool bf16, const void* H, const uint8_t* y, int n_rows, int d,
                           float lr, float* w, float* c, float* r, double* row_loss,
                           float* loss_out, hipStream_t st) {
  if (n_rows <= 0) return hipSuccess;
  const dim3 g1(cdiv(n_rows, 4)), g2(cdiv(d, 256)), b(256);
  if (bf16) {
    hipLaunchKernelGGL(k_bce_logits<bf16_t>, g1, b, 0, st, static_cast<const bf16_t*>(H), y,
                       n_rows, d, w, c, r, row_loss);
    hipLaunchKernelGGL(k_bce_update<bf16_t>, g2, b, 0, st, static_cast<const bf16_t*>(H), n_rows,
                       d, lr, r, row_loss, w, c, loss_out);
  } else {
    hipLaunchKernelGGL(k_bce_logits<float>, g1, b, 0, st, static_cast<const float*>(H), y, n_rows,
                       d, w, c, r, row_loss);
    hipLaunchKernelGGL(k_bce_update<float>, g2, b, 0, st, static_cast<const float*>(H), n_rows,
                       d, lr, r, row_loss, w, c, loss_out);
  }
  return hipGetLastError();
}

// ------------------------------------------ one pass over the rows per step --
// The two kernels above read H twice per step, and k_bce_update walks all rows
// serially with d threads (8 blocks at d = 2048: 555 us per step at 4096 rows,
// a chain of 4096 dependent fp64 adds behind 2-byte loads).  Here a wavefront
// takes whole rows: it holds the row in registers (16-byte loads, the next
// row's in flight), reduces the logit, and adds residual * row into its own
// fp64 column sums, so H is read once per step.  A block adds its wavefronts'
// sums in order through LDS and writes one fp64 row of partials; k_bce_finish
// adds the blocks' partials in order (repeated runs stay bit-identical).
// 4096 bf16 rows, d = 2048: 568 -> 17 us per step on an MI355X (12.5 us rows,
// 4.5 us finish); what is left is two launches and their dependent chains of a
// load, a lane reduction and a store.
constexpr int kBceWaves = 4;
// columns a lane sums: 64 doubles (128 VGPRs) cover d = 4096 per wavefront
constexpr int kBceLaneCols = kTrainMaxCols / 64;

// Columns of a row are dealt in chunks of 64 V: column (i 64 + lane) V + u is
// element u of the lane's load i.  Partials are kept in slot order,
// slot = (i V + u) 64 + lane, so that they are stored and read contiguously.
__device__ __forceinline__ int bce_column(int slot, int V) {
  const int lane = slot & 63, iu = slot >> 6;
  return ((iu / V) * 64 + lane) * V + iu % V;
}

// V: elements per load (8 bf16 or 4 fp32 when rows are 16-byte aligned, else
// 1); NC: chunks of 64 V columns that cover a row
template <typename T, int V, int NC>
__global__ __launch_bounds__(64 * kBceWaves) void k_bce_rows(const T* H, const uint8_t* y, int n_rows,
                                                             int d, const float* w, const float* c,
                                                             double* part, double2* part_rl) {
  constexpr int SLOTS = 64 * V * NC;
  __shared__ double s_col[kBceWaves][SLOTS];
  __shared__ double2 s_rl[kBceWaves];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // (unsigned: the row after the last one passes 2^31 - 1 in the largest batches)
  const unsigned q0 = blockIdx.x * kBceWaves + wave, step = gridDim.x * kBceWaves;
  const unsigned rows = n_rows;
  struct alignas(sizeof(T) * V) Vec {
    T e[V];
  };
  auto load_row = [&](Vec(&x)[NC], unsigned q) {
    const T* h = H + (size_t)q * d;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int k = (i * 64 + lane) * V;
      if (k < d)
        x[i] = *reinterpret_cast<const Vec*>(h + k);
      else
        x[i] = Vec{};
    }
  };
  Vec x[NC], xn[NC];
  load_row(x, min(q0, rows - 1));
  float wv[NC][V];
#pragma unroll
  for (int i = 0; i < NC; ++i)
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const int k = (i * 64 + lane) * V + u;
      wv[i][u] = k < d ? w[k] : 0.f;
    }
  const float cv = *c;
  double g[NC][V];
#pragma unroll
  for (int i = 0; i < NC; ++i)
#pragma unroll
    for (int u = 0; u < V; ++u) g[i][u] = 0.0;
  double sr = 0.0, sl = 0.0;
  for (unsigned q = q0; q < rows; q += step) {
    const float label = y[q] ? 1.f : 0.f;
    load_row(xn, min(q + step, rows - 1));
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
      for (int u = 0; u < V; ++u) acc = fmaf(wv[i][u], to_f32<T>(x[i].e[u]), acc);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    const float z = acc + cv;
    const float r = 1.f / (1.f + expf(-z)) - label;
    const double rd = r;
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
      for (int u = 0; u < V; ++u) g[i][u] = fma(rd, (double)to_f32<T>(x[i].e[u]), g[i][u]);
    if (lane == 0) {
      const double zd = z;
      sr += rd;
      sl += fmax(zd, 0.0) - (double)label * zd + log1p(exp(-fabs(zd)));
    }
#pragma unroll
    for (int i = 0; i < NC; ++i) x[i] = xn[i];
  }
  if (lane == 0) s_rl[wave] = make_double2(sr, sl);
#pragma unroll
  for (int i = 0; i < NC; ++i)
#pragma unroll
    for (int u = 0; u < V; ++u) s_col[wave][(i * V + u) * 64 + lane] = g[i][u];
  __syncthreads();
  for (int j = threadIdx.x; j < SLOTS; j += 64 * kBceWaves) {
    double t = s_col[0][j];
#pragma unroll
    for (int v = 1; v < kBceWaves; ++v) t += s_col[v][j];
    part[(size_t)blockIdx.x * SLOTS + j] = t;
  }
  if (threadIdx.x == 0) {
    double2 t = s_rl[0];
    for (int v = 1; v < kBceWaves; ++v) {
      t.x += s_rl[v].x;
      t.y += s_rl[v].y;
    }
    part_rl[blockIdx.x] = t;
  }
}

// w[k] -= lr * (sum of the nb partials of column k) / Q: 32 slots per block,
// 8 threads per slot over consecutive runs of partials (their loads in flight
// together), the runs added in order.  Block 0 also moves c and writes the
// mean loss.
__global__ __launch_bounds__(256) void k_bce_finish(const double* part, const double2* part_rl,
                                                    int nb, int slots, int V, int n_rows, int d,
                                                    float lr, float* w, float* c,
                                                    float* loss_out) {
  constexpr int CB = 32, SEG = 256 / CB;
  __shared__ double s_g[SEG][CB];
  __shared__ double2 s_rl[256];
  const int cx = threadIdx.x % CB, seg = threadIdx.x / CB;
  const int slot = blockIdx.x * CB + cx;  // slots is a multiple of CB
  const int per = (nb + SEG - 1) / SEG, b0 = seg * per, b1 = min(nb, b0 + per);
  double t = 0.0;
#pragma unroll 16
  for (int b = b0; b < b1; ++b) t += part[(size_t)b * slots + slot];
  s_g[seg][cx] = t;
  if (blockIdx.x == 0) {
    double2 v = make_double2(0.0, 0.0);
    for (int b = threadIdx.x; b < nb; b += 256) {
      const double2 x = part_rl[b];
      v.x += x.x;
      v.y += x.y;
    }
    s_rl[threadIdx.x] = v;
  }
  __syncthreads();
  const int k = bce_column(slot, V);
  if (seg == 0 && k < d) {
    double g = s_g[0][cx];
#pragma unroll
    for (int v = 1; v < SEG; ++v) g += s_g[v][cx];
    w[k] -= lr * (float)(g / n_rows);
  }
  if (blockIdx.x != 0) return;
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      s_rl[threadIdx.x].x += s_rl[threadIdx.x + s].x;
      s_rl[threadIdx.x].y += s_rl[threadIdx.x + s].y;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *c -= lr * (float)(s_rl[0].x / n_rows);
    if (loss_out) *loss_out = (float)(s_rl[0].y / n_rows);
  }
}

int bce_slots(bool bf16, const void* H, int d, int* vec) {
  const bool al16 = (reinterpret_cast<uintptr_t>(H) & 15) == 0;
  const int V = !al16 ? 1 : bf16 ? (d % 8 == 0 ? 8 : 1) : (d % 4 == 0 ? 4 : 1);
  int slots = 64 * V;
  while (slots < d) slots *= 2;
  if (vec) *vec = V;
  return slots;
}

// chunk counts 1, 2, 4, ... up to NMAX that cover the row (bce_slots)
template <typename T, int V, int NC, int NMAX>
static void bce_rows(int slots, const T* H, const uint8_t* y, int n_rows, int d, const float* w,
                     const float* c, double* part, double2* part_rl, int nb, hipStream_t st) {
  if constexpr (NC < NMAX) {
    if (slots > 64 * V * NC)
      return bce_rows<T, V, 2 * NC, NMAX>(slots, H, y, n_rows, d, w, c, part, part_rl, nb, st);
  }
  hipLaunchKernelGGL((k_bce_rows<T, V, NC>), dim3(nb), dim3(64 * kBceWaves), 0, st, H, y, n_rows, d,
                     w, c, part, part_rl);
}

hipError_t launch_bce_rows_step(bool bf16, const void* H, const uint8_t* y, int n_rows, int d,
                                float lr, float* w, float* c, double* part, double2* part_rl,
                                int nb, float* loss_out, hipStream_t st) {
  int V = 1;
  const int slots = bce_slots(bf16, H, d, &V);
  const bf16_t* hb = static_cast<const bf16_t*>(H);
  const float* hf = static_cast<const float*>(H);
  if (bf16 && V == 8)
    bce_rows<bf16_t, 8, 1, kBceLaneCols / 8>(slots, hb, y, n_rows, d, w, c, part, part_rl, nb, st);
  else if (bf16)
    bce_rows<bf16_t, 1, 1, kBceLaneCols>(slots, hb, y, n_rows, d, w, c, part, part_rl, nb, st);
  else if (V == 4)
    bce_rows<float, 4, 1, kBceLaneCols / 4>(slots, hf, y, n_rows, d, w, c, part, part_rl, nb, st);
  else
    bce_rows<float, 1, 1, kBceLaneCols>(slots, hf, y, n_rows, d, w, c, part, part_rl, nb, st);
  hipLaunchKernelGGL(k_bce_finish, dim3(slots / 32), dim3(256), 0, st, part, part_rl, nb, slots, V,
                     n_rows, d, lr, w, c, loss_out);
  return hipGetLastError();
}

}  // namespace trimmoe
