// HBM-bound kernels of the CLT train step: decoder norms, loss reductions with
// their fused gradient by-products, the threshold (straight-through) column
// reductions and Adam.  Reductions are two-stage with a fixed summation order
// (per-block partials, then one pass over the partials), so results are
// bitwise reproducible run to run.
#include "common.h"

#include <algorithm>

namespace clt {
namespace {

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
// sum over a 256-lane block; result valid in thread 0
__device__ __forceinline__ double block_sum_256(double v) {
  __shared__ double sh[4];
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  return sh[0] + sh[1] + sh[2] + sh[3];
}

__global__ void zero_i32_kernel(int32_t* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}
// the same by the first workgroup of a kernel that runs anyway (n <= 128 <= its size)
__device__ __forceinline__ void zero_counters(int32_t* p, int n) {
  if (p && blockIdx.x == 0 && (int)threadIdx.x < n) p[threadIdx.x] = 0;
}

// ---- decode partial sums (see DecSplit): grid = (runs of 1024 elements of [B][d], targets) ----
__global__ __launch_bounds__(256) void decode_combine_kernel(Dims D, DecSplit sp, const float* __restrict__ part,
                                                             const float* __restrict__ b_dec, float* __restrict__ y_hat,
                                                             const int32_t* __restrict__ skip_flags, int kcap) {
  if (skip_flags && gather_selected(skip_flags, kcap)) return;
  const size_t n = (size_t)D.B * D.d, i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= n) return;
  const int lp = blockIdx.y;
  int slot = 0;
  for (int q = D.L - 1; q > lp; --q) slot += sp.chunks(q);
  const int end = slot + sp.chunks(lp);
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
  for (; slot < end; ++slot) {
    const float4 v = *reinterpret_cast<const float4*>(part + slot * n + i);
    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
  }
  const float4 b = *reinterpret_cast<const float4*>(b_dec + (size_t)lp * D.d + i % D.d);
  *reinterpret_cast<float4*>(y_hat + lp * n + i) = make_float4(s.x + b.x, s.y + b.y, s.z + b.z, s.w + b.w);
}

// ---- decoder norms (App. B): one wavefront per (source layer, feature) -----
// The L-l blocks that leave source l are contiguous in the source-major packing,
// so feature f's rows are L-l runs of d contiguous elements.
template <typename T>
__global__ __launch_bounds__(256) void decoder_norms_kernel(Dims D, const T* __restrict__ W_dec,
                                                            float* __restrict__ norms, int32_t* __restrict__ l0) {
  zero_counters(l0, D.L);
  const int lane = threadIdx.x & 63;
  const long row = (long)blockIdx.x * 4 + (threadIdx.x >> 6);   // l * F + f
  if (row >= (long)D.L * D.F) return;
  const int l = (int)(row / D.F), f = (int)(row - (long)l * D.F);
  const T* base = W_dec + ((size_t)packed_index(l, l, D.L) * D.F + f) * D.d;
  float acc = 0.f;
  for (int s = 0; s < D.L - l; ++s) {
    const T* r = base + (size_t)s * D.F * D.d;
    for (int j = lane * 4; j < D.d; j += 256) {
      const float4 v = Elem<T>::load4(r + j);
      acc += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
    }
  }
  acc = wave_sum(acc);
  if (lane == 0) norms[row] = sqrtf(acc);
}

// The same norms from sums of squares that the last fused update (or the decode of few tokens) left, in a fixed order.  The dense kernel leaves
// them per (block, column run, feature), [P][runs][F]; the list-driven row kernel per (block, feature, slot),
// [P][F][8 ceil(d / 2048)].  Which of the two ran is what the device-side switch decided in that step (flags).
__global__ __launch_bounds__(256) void norms_from_partials_kernel(Dims D, const float* __restrict__ n2_part, int runs,
                                                                  float* __restrict__ norms,
                                                                  const int32_t* __restrict__ flags, int kcap,
                                                                  int32_t* __restrict__ l0) {
  zero_counters(l0, D.L);
  const long i = (long)blockIdx.x * 256 + threadIdx.x;      // l * F + f
  if (i >= (long)D.L * D.F) return;
  const int l = (int)(i / D.F), f = (int)(i - (long)l * D.F);
  float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (flags && lists_backward_selected(flags, kcap)) {
    const int slots = 8 * ((D.d + 2047) / 2048);
    const float* base = n2_part + ((size_t)packed_index(l, l, D.L) * D.F + f) * slots;
    for (int j = 0; j < D.L - l; ++j)
      for (int q = 0; q < slots; q += 8) {
        const float4 u = *reinterpret_cast<const float4*>(base + (size_t)j * D.F * slots + q);
        const float4 w = *reinterpret_cast<const float4*>(base + (size_t)j * D.F * slots + q + 4);
        a[0] += u.x; a[1] += u.y; a[2] += u.z; a[3] += u.w; a[4] += w.x; a[5] += w.y; a[6] += w.z; a[7] += w.w;
      }
  } else {
    const float* base = n2_part + (size_t)packed_index(l, l, D.L) * runs * D.F + f;
    // eight independent chains keep eight loads in flight per lane; the order of the sum stays fixed
    const int n = (D.L - l) * runs;
    int j = 0;
    for (; j + 8 <= n; j += 8) {
#pragma unroll
      for (int q = 0; q < 8; ++q) a[q] += base[(size_t)(j + q) * D.F];
    }
    for (; j < n; ++j) a[j & 7] += base[(size_t)j * D.F];
  }
  norms[i] = sqrtf(((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7])));
}

// ---- reductions over token rows (losses, straight-through terms) --------------------------
// One workgroup takes `rows` token rows of one layer and 16 bytes of columns per lane (512 columns of bf16, 256 of
// fp32); its four wavefronts take a quarter of the rows each, eight rows in flight, and add their column sums up in LDS
// in a fixed order.  Walking one row after the other over all columns, with a workgroup per 32 rows only, left the small
// shapes bound by the latency of one load per row (sparsity sum, L = 12, F = 6144, 300 tokens: 129 us; L = 4, F = 256, 128
// tokens: 17) and wrote four times the partials for the large ones.
constexpr int ROWS_IN_FLIGHT = 8;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
template <typename T> struct Row16 { static constexpr int N = 16 / sizeof(T); };      // columns per lane
template <typename T> __device__ __forceinline__ u32x4 load16(const T* p) { return *reinterpret_cast<const u32x4*>(p); }
__device__ __forceinline__ void widen16(u32x4 r, float (&f)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) { f[2 * i] = __uint_as_float(r[i] << 16); f[2 * i + 1] = __uint_as_float(r[i] & 0xffff0000u); }
}
__device__ __forceinline__ void widen16(u32x4 r, float (&f)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) f[i] = __uint_as_float(r[i]);
}
__device__ __forceinline__ void store16(bf16_t* p, const float (&f)[8]) {
  const u32x4 r = {pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7])};
  *reinterpret_cast<u32x4*>(p) = r;
}
__device__ __forceinline__ void store16(float* p, const float (&f)[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(f[0], f[1], f[2], f[3]);
}
__device__ __forceinline__ void nt_store16(bf16_t* p, const float (&f)[8]) {
  const u32x4 r = {pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7])};
  CLT_NT_STORE(r, reinterpret_cast<u32x4*>(p));
}
__device__ __forceinline__ void nt_store16(float* p, const float (&f)[4]) { nt_store_f4(p, make_float4(f[0], f[1], f[2], f[3])); }
template <int N> __device__ __forceinline__ void load_floats(const float* p, float (&f)[N]) {
#pragma unroll
  for (int i = 0; i < N; i += 4) {
    const float4 v = *reinterpret_cast<const float4*>(p + i);
    f[i] = v.x; f[i + 1] = v.y; f[i + 2] = v.z; f[i + 3] = v.w;
  }
}
// the workgroup's part: rows [r0, r1) of the calling wavefront, first column c of the calling lane
template <int N> struct RowPart {
  int rb, l, r0, r1, c;
  __device__ __forceinline__ RowPart(Dims D, int block, int rows, int nchunks, int cols) {
    const int chunk = block % nchunks;
    rb = block / nchunks;
    l = blockIdx.y;
    const int w = threadIdx.x >> 6;
    r0 = min(D.B, rb * rows + w * (rows / 4));
    r1 = min(D.B, r0 + rows / 4);
    c = (chunk * 64 + (threadIdx.x & 63)) * N;
    if (c >= cols) r1 = r0;      // nothing to do, but the lane takes part in the barriers
  }
};
// column sums of the four wavefronts, written by the first one (all threads of the workgroup call it)
template <int N>
__device__ __forceinline__ void add_column_sums(float (&s)[N], float* dst, bool in, float (&lds)[3][64 * N]) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();
  if (w > 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) lds[w - 1][i * 64 + lane] = s[i];
  }
  __syncthreads();
  if (w == 0 && in) {
#pragma unroll
    for (int i = 0; i < N; ++i) s[i] = (s[i] + lds[0][i * 64 + lane]) + (lds[1][i * 64 + lane] + lds[2][i * 64 + lane]);
#pragma unroll
    for (int i = 0; i < N; i += 4) *reinterpret_cast<float4*>(dst + i) = make_float4(s[i], s[i + 1], s[i + 2], s[i + 3]);
  }
}

// reconstruction loss: r = y_hat - y; partial sum r^2; d_yhat = 2 r / B; column partial sums of d_yhat (for db_dec)
template <typename T, bool INT8>
__device__ __forceinline__ void loss_reconstruction(const Dims& D, int block, int nblocks, int rows, int nchunks, const float* __restrict__ y_hat,
                                                    const void* yv, const float* __restrict__ y_scale,
                                                    T* __restrict__ d_yhat, double* __restrict__ loss_part,
                                                    float* __restrict__ col_part, float (&lds)[3][64 * Row16<T>::N]) {
  constexpr int N = Row16<T>::N, R = ROWS_IN_FLIGHT / 2;      // (two more loads per row than the other kernels)
  const RowPart<N> p(D, block, rows, nchunks, D.d);
  const float two_over_b = 2.0f / (float)D.B;
  float cs[N];
#pragma unroll
  for (int i = 0; i < N; ++i) cs[i] = 0.f;
  double sq = 0.0;
  for (int r = p.r0; r < p.r1; r += R) {
    float yh[R][N], ys[R];
    u32x4 raw[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int rj = min(r + j, p.r1 - 1);
      const size_t o = ((size_t)p.l * D.B + rj) * D.d + p.c;
      load_floats(y_hat + o, yh[j]);
      if (INT8) {
        const uint2 q = *reinterpret_cast<const uint2*>(reinterpret_cast<const int8_t*>(yv) + o);
        raw[j] = u32x4{q.x, q.y, 0u, 0u};
        ys[j] = y_scale[(size_t)p.l * D.B + rj];
      } else {
        raw[j] = load16(reinterpret_cast<const T*>(yv) + o);
      }
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (r + j >= p.r1) break;
      float y[N], g[N];
      if (INT8) {
#pragma unroll
        for (int i = 0; i < N; ++i) y[i] = ys[j] * (float)(int8_t)(raw[j][i / 4] >> (8 * (i & 3)));
      } else {
        widen16(raw[j], y);
      }
#pragma unroll
      for (int i = 0; i < N; ++i) {
        y[i] = yh[j][i] - y[i];
        g[i] = two_over_b * y[i];
        cs[i] += g[i];
      }
#pragma unroll
      for (int i = 0; i < N; i += 4)
        sq += (double)(y[i] * y[i] + y[i + 1] * y[i + 1]) + (double)(y[i + 2] * y[i + 2] + y[i + 3] * y[i + 3]);
      store16(d_yhat + ((size_t)p.l * D.B + r + j) * D.d + p.c, g);
    }
  }
  add_column_sums(cs, col_part + ((size_t)p.rb * D.L + p.l) * D.d + p.c, p.c < D.d, lds);
  const double tot = block_sum_256(sq);
  if (threadIdx.x == 0) loss_part[(size_t)p.l * nblocks + block] = tot;
}

// sparsity loss: partial sum tanh(C z n); column partials of C z sech^2(C z n) (both from one hardware exponential).
// With DEAD also the App. B dead-feature term: partial sum relu(theta - pre) n and the
// column partials of relu(theta - pre) (its derivative w.r.t. the decoder norm).
template <typename T, bool DEAD>
__device__ __forceinline__ void loss_sparsity(const Dims& D, int block, int nblocks, int rows, int nchunks, const T* __restrict__ z,
                                              const float* __restrict__ norms, float C, double* __restrict__ loss_part,
                                              float* __restrict__ col_part, const T* __restrict__ pre,
                                              const float* __restrict__ theta, bool log_threshold,
                                              double* __restrict__ dead_part, float* __restrict__ dead_col_part,
                                              float (&lds)[3][64 * Row16<T>::N]) {
  constexpr int N = Row16<T>::N, R = DEAD ? ROWS_IN_FLIGHT / 2 : ROWS_IN_FLIGHT;
  const RowPart<N> p(D, block, rows, nchunks, D.F);
  const bool in = p.c < D.F;
  float ka[N], nn[N], th[N], cs[N], ds[N];
#pragma unroll
  for (int i = 0; i < N; ++i) ka[i] = nn[i] = th[i] = cs[i] = ds[i] = 0.f;
  if (in) {
    load_floats(norms + (size_t)p.l * D.F + p.c, nn);
    if (DEAD) load_floats(theta + (size_t)p.l * D.F + p.c, th);
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    ka[i] = -2.0f * 1.4426950408889634f * (C * nn[i]);
    if (DEAD) th[i] = threshold_value(th[i], log_threshold);
  }
  double sp = 0.0, dead = 0.0;
  for (int r = p.r0; r < p.r1; r += R) {
    u32x4 zr[R], pr[DEAD ? R : 1];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const size_t o = ((size_t)p.l * D.B + min(r + j, p.r1 - 1)) * D.F + p.c;
      zr[j] = load16(z + o);
      if (DEAD) pr[j] = load16(pre + o);
    }
    float ts = 0.f, dsum = 0.f;      // at most 8 rows of a lane's columns in fp32
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (r + j >= p.r1) break;
      float zz[N];
      widen16(zr[j], zz);
#pragma unroll
      for (int i = 0; i < N; ++i) {
        if (zz[i] != 0.f) {
          // u = C n z, e = exp(-2|u|): tanh|u| = (1 - e) / (1 + e), sech^2 u = 4 e / (1 + e)^2 (no cancellation for large u;
          // 1 - e is exact for e >= 1/2, so that small u keep their digits: 1 - 2 e / (1 + e) subtracts a rounded quotient and
          // is 4 times further off at |u| < 0.1)
          const float a = ka[i] * zz[i];      // -2 log2(e) u
          const float e = __builtin_amdgcn_exp2f(-fabsf(a));
          const float rc = __builtin_amdgcn_rcpf(1.0f + e);
          ts -= copysignf((1.0f - e) * rc, a);
          cs[i] = fmaf(zz[i], e * rc * rc, cs[i]);
        }
      }
      if (DEAD) {
        float pp[N];
        widen16(pr[j], pp);
#pragma unroll
        for (int i = 0; i < N; ++i) {
          const float g = fmaxf(th[i] - pp[i], 0.f);
          ds[i] += g;
          dsum += g * nn[i];
        }
      }
    }
    sp += (double)ts;
    dead += (double)dsum;
  }
#pragma unroll
  for (int i = 0; i < N; ++i) cs[i] *= 4.0f * C;
  const size_t po = ((size_t)p.rb * D.L + p.l) * D.F + p.c;
  add_column_sums(cs, col_part + po, in, lds);
  if (DEAD) add_column_sums(ds, dead_col_part + po, in, lds);
  const double tot = block_sum_256(sp);
  if (threadIdx.x == 0) loss_part[(size_t)p.l * nblocks + block] = tot;
  if (DEAD) {
    __syncthreads();
    const double dt = block_sum_256(dead);
    if (threadIdx.x == 0) dead_part[(size_t)p.l * nblocks + block] = dt;
  }
}

// Both losses in one launch, the sparsity term's workgroups first.  What bounds these kernels at small shapes is the launch, 2 to 5 us
// for each that waits for the one before: with the loss sums and G, and the vectors' gradients and their update, in one launch each
// as well and the encoder's counters cleared along the way, a training step has 11 launches instead of 19 (L = 4, d = 64, F = 256, 128
// tokens of fp32: 86 -> 69 us; L = 3, d = 136, F = 1032, 300 tokens of bf16: 184 -> 163).
struct LossArgs {
  int sp_rows, sp_chunks, sp_blocks, rec_rows, rec_chunks, rec_blocks;
  const void* z; const float* norms; float C; const void* pre; const float* theta; bool log_threshold;
  double* sp_part; float* sp_cols; double* dead_part; float* dead_cols;
  const float* y_hat; const void* y; const float* y_scale; void* d_yhat; double* rec_part; float* rec_cols;
};
template <typename T, bool INT8, bool DEAD>
__global__ __launch_bounds__(256) void loss_kernel(Dims D, LossArgs a) {
  __shared__ float lds[3][64 * Row16<T>::N];
  if ((int)blockIdx.x < a.sp_blocks)
    loss_sparsity<T, DEAD>(D, blockIdx.x, a.sp_blocks, a.sp_rows, a.sp_chunks, (const T*)a.z, a.norms, a.C, a.sp_part, a.sp_cols,
                           (const T*)a.pre, a.theta, a.log_threshold, a.dead_part, a.dead_cols, lds);
  else
    loss_reconstruction<T, INT8>(D, blockIdx.x - a.sp_blocks, a.rec_blocks, a.rec_rows, a.rec_chunks, a.y_hat, a.y, a.y_scale,
                                 (T*)a.d_yhat, a.rec_part, a.rec_cols, lds);
}

// Sum over the row partials of 64 columns by a workgroup: each wavefront adds a quarter of the partials, the quarters
// are added in order.  Valid in the first wavefront.  (One thread per column walking 128 partials: 34 us at 73728 columns,
// bound by the chain of loads; 5 us now, also because there are a quarter as many partials.)
__device__ __forceinline__ float sum_partials(const float* __restrict__ part, int nparts, int ncols, int c, float (&lds)[3][64]) {
  const int w = (threadIdx.x >> 6) & 3, lane = threadIdx.x & 63;      // (larger workgroups: four wavefronts each, with an lds of their own)
  const int per = (nparts + 3) / 4, r0 = min(nparts, w * per), r1 = min(nparts, r0 + per);
  float s = 0.f;
  if (c < ncols) {
#pragma unroll 8
    for (int r = r0; r < r1; ++r) s += part[(size_t)r * ncols + c];
  }
  __syncthreads();
  if (w > 0) lds[w - 1][lane] = s;
  __syncthreads();
  return w == 0 ? (s + lds[0][lane]) + (lds[1][lane] + lds[2][lane]) : 0.f;
}

// What is left of the loss after its row blocks: the first workgroup adds up the loss terms, the others the column partials
// of the norms' gradient, G[c] = sp_scale sum_r sp[r][c] (+ dead_scale sum_r dead[r][c]), scales lambda0/B and lambda1/B.
// The loss terms are one workgroup's chains of loads, which outlast the columns where there are many of them: L = 16, d = 2048, F = 8192,
// 4096 tokens 21.4 us with 256 lanes, 12.4 with 1024 (10.7 and 7.4 as two launches); L = 6, d = 2056, F = 8200 with the dead-feature term
// 18.0 and 11.1; L = 12, d = 768, F = 6144, 1024 tokens of fp32 9.0 and 7.2.  Up to 2048 terms each, one round of 256 lanes, the larger workgroup only
// costs its barriers (whole steps of 70 to 150 us are 0.7 to 1 us longer).
constexpr int LF_FEW = 2048;
template <int LF_LANES>
__global__ __launch_bounds__(LF_LANES) void loss_finish_kernel(const double* __restrict__ part_rec, int n_rec, const double* __restrict__ part_sp,
                                                          int n_sp, const double* __restrict__ part_dead, float inv_B, float lambda0,
                                                          float lambda1, float sp_scale, float dead_scale,
                                                          float* __restrict__ loss_dev, const float* __restrict__ sp_cols,
                                                          const float* __restrict__ dead_cols, int nparts, int ncols,
                                                          float* __restrict__ G) {
  if (blockIdx.x > 0) {
    __shared__ float lds[LF_LANES / 256][3][64];
    const int part = threadIdx.x >> 8, c = ((int)blockIdx.x - 1) * (LF_LANES / 4) + part * 64 + (threadIdx.x & 63);
    float g = sp_scale * sum_partials(sp_cols, nparts, ncols, c, lds[part]);
    if (part_dead) {
#pragma clang fp contract(off)
      const float q = dead_scale * sum_partials(dead_cols, nparts, ncols, c, lds[part]);
      g = g + q;
    }
    if ((threadIdx.x & 255) < 64 && c < ncols) G[c] = g;
    return;
  }
  __shared__ double sh[3][LF_LANES / 64];
  auto sum = [&](const double* p, int n, int slot) {
    constexpr int N = LF_LANES == 256 ? 8 : 4;      // chains, to keep as many loads in flight
    double s[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int i = threadIdx.x; i < n; i += N * LF_LANES) {
#pragma unroll
      for (int q = 0; q < N; ++q)
        if (i + LF_LANES * q < n) s[q] += p[i + LF_LANES * q];
    }
    const double t = wave_sum(((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7])));
    if ((threadIdx.x & 63) == 0) sh[slot][threadIdx.x >> 6] = t;
  };
  sum(part_rec, n_rec, 0);
  sum(part_sp, n_sp, 1);
  sum(part_dead, part_dead ? n_sp : 0, 2);
  __syncthreads();
  if (threadIdx.x == 0) {
    double a = 0.0, b = 0.0, c = 0.0;
    for (int i = 0; i < LF_LANES / 64; ++i) { a += sh[0][i]; b += sh[1][i]; c += sh[2][i]; }
    const double rec = a * (double)inv_B, sp = b * (double)inv_B * (double)lambda0;
    const double dead = c * (double)inv_B * (double)lambda1;
    loss_dev[0] = (float)(rec + sp + dead);
    loss_dev[1] = (float)rec;
    loss_dev[2] = (float)sp;
    loss_dev[3] = (float)dead;
  }
}

// Gradients of the three vectors from the column partials of the backward, and their Adam update where the caller wants it, in
// one launch.  d b_enc and d b_dec are plain sums.  Threshold: straight-through part -(theta/eps) * (sum over window entries of
// dz), plus the dead-feature part (lambda1/B) n * #(pre < theta); times theta when the parameter is tau = log(theta).  TopK has no
// threshold, the partials are zeros.
__global__ __launch_bounds__(256) void vector_gradients_kernel(VectorGradArgs a) {
  __shared__ float lds[3][64];
  const int nf = (a.nF + 63) / 64;
  auto update = [&](const VectorAdam& q, int c, float g) {
    if (!q.p) return;
    float p = q.p[c], m = q.m[c], v = q.v[c];
    adam_element(p, m, v, g, a.adam);
    q.p[c] = p; q.m[c] = m; q.v[c] = v;
  };
  if ((int)blockIdx.x >= nf) {
    const int c = ((int)blockIdx.x - nf) * 64 + (threadIdx.x & 63);
    const float g = sum_partials(a.part_bdec, a.nparts_bdec, a.nd, c, lds);
    if (threadIdx.x >= 64 || c >= a.nd) return;
    a.g_bdec[c] = g;
    update(a.b_dec, c, g);
    return;
  }
  const int c = (int)blockIdx.x * 64 + (threadIdx.x & 63);
  const int nparts = a.sw.flags && lists_backward_selected(a.sw.flags, a.sw.kcap) ? a.sw.nparts_lists : a.nparts;
  const float w = sum_partials(a.part_win, nparts, a.nF, c, lds);
  const float nb = a.lam1_over_b != 0.f ? sum_partials(a.part_below, nparts, a.nF, c, lds) : 0.f;
  const float gb = sum_partials(a.part_benc, nparts, a.nF, c, lds);
  if (threadIdx.x >= 64 || c >= a.nF) return;
  float g = w;
  if (!a.topk) {
    const float th = threshold_value(a.theta[c], a.log_threshold);
    g = (w == 0.f) ? 0.f : w * -(th * a.inv_eps);   // empty window: exactly 0, also for theta = inf
    if (a.lam1_over_b != 0.f) g += a.lam1_over_b * a.norms[c] * nb;
    if (a.log_threshold) g *= th;
  }
  a.g_theta[c] = g;
  a.g_benc[c] = gb;
  update(a.th, c, g);
  update(a.b_enc, c, gb);
}

// ---- straight-through reductions over the buffer that holds dz where a feature
// is active or in the threshold window, and the dead-feature gradient elsewhere
// below the threshold: column partials of dz over the window (-> dtheta), of the
// final dpre (-> db_enc) and of the below-threshold count; entries that are in the
// window but inactive are rewritten to their dpre value (dead-feature gradient or 0),
// so the buffer becomes dpre.  With a row scale (int8 inputs) dpre rows are also
// multiplied by it, because the encoder-weight gradient contracts them with the
// integer codes.
template <typename T>
__global__ __launch_bounds__(256) void ste_reduce_kernel(Dims D, int rows, int nchunks, T* __restrict__ dpre,
                                                         const uint8_t* __restrict__ cls,
                                                         const float* __restrict__ row_scale,
                                                         const float* __restrict__ norms, float lam1_over_b,
                                                         float* __restrict__ part_theta,
                                                         float* __restrict__ part_benc,
                                                         float* __restrict__ part_below,
                                                         const int32_t* __restrict__ only_if_lists, int kcap) {
  if (only_if_lists && !lists_backward_selected(only_if_lists, kcap)) return;
  constexpr int N = Row16<T>::N, W = N / 4, R = ROWS_IN_FLIGHT;      // W words of classes per row
  __shared__ float lds[3][64 * N];
  const RowPart<N> p(D, blockIdx.x, rows, nchunks, D.F);
  const bool dead = lam1_over_b != 0.f, in = p.c < D.F;
  float st[N], sb[N], nb[N], dg[N];
#pragma unroll
  for (int i = 0; i < N; ++i) st[i] = sb[i] = nb[i] = dg[i] = 0.f;
  if (dead && in) {
    load_floats(norms + (size_t)p.l * D.F + p.c, dg);
#pragma unroll
    for (int i = 0; i < N; ++i) dg[i] *= -lam1_over_b;
  }
  const uint32_t care = dead ? 0xffffffffu : 0x03030303u;   // without the dead-feature term only active / window entries matter
  for (int r = p.r0; r < p.r1; r += R) {
    uint32_t cw[R][W];
    u32x4 raw[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const uint32_t* q = reinterpret_cast<const uint32_t*>(cls + ((size_t)p.l * D.B + min(r + j, p.r1 - 1)) * D.F + p.c);
#pragma unroll
      for (int k = 0; k < W; ++k) cw[j][k] = q[k];
    }
    uint32_t any[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      any[j] = 0u;
#pragma unroll
      for (int k = 0; k < W; ++k) any[j] |= (cw[j][k] &= care);
      if (r + j >= p.r1) any[j] = 0u;
      raw[j] = u32x4{0u, 0u, 0u, 0u};
      if (any[j]) raw[j] = load16(dpre + ((size_t)p.l * D.B + r + j) * D.F + p.c);
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (!any[j]) continue;
      float g[N];
      widen16(raw[j], g);
      bool rewrite = row_scale != nullptr;
      const float s = row_scale ? row_scale[(size_t)p.l * D.B + r + j] : 1.0f;
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const uint32_t ci = (cw[j][i / 4] >> (8 * (i & 3))) & 7u;
        if (ci & CLS_WINDOW) st[i] += g[i];
        if (ci & CLS_BELOW) nb[i] += 1.0f;
        if (!(ci & CLS_ACTIVE) && (ci & CLS_WINDOW)) {   // held dz for the threshold gradient only
          g[i] = (ci & CLS_BELOW) ? dg[i] : 0.f;
          rewrite = true;
        }
        if (ci) {
          sb[i] += g[i];
          g[i] *= s;
        }
      }
      if (rewrite) store16(dpre + ((size_t)p.l * D.B + r + j) * D.F + p.c, g);
    }
  }
  const size_t po = ((size_t)p.rb * D.L + p.l) * D.F + p.c;
  add_column_sums(st, part_theta + po, in, lds);
  add_column_sums(sb, part_benc + po, in, lds);
  if (dead) add_column_sums(nb, part_below + po, in, lds);
}

// ---- Adam (App. C Table 1), ADAM_QUADS x 4 elements per lane, one workgroup per run ----
// (396 M parameters in fp32, 28 bytes each: 2.69 ms as a grid-stride loop of one quad per lane, 2.39 now, 4.6 TB/s)
constexpr int ADAM_QUADS = 2;
template <typename T, bool MASTER>
__global__ __launch_bounds__(256) void adam_kernel(size_t n4, T* __restrict__ p, const T* __restrict__ g,
                                                   float* __restrict__ m, float* __restrict__ v,
                                                   float* __restrict__ master, AdamScalars a) {
  typedef typename Elem<T>::Raw4 Raw4;
  constexpr int R = ADAM_QUADS;      // quads of a lane, all their loads in flight
  const size_t i0 = (size_t)blockIdx.x * (256 * R) + threadIdx.x;
  Raw4 g4[R], w4[R];
  float4 m4[R], v4[R], p4[R];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    if (i0 + 256 * j >= n4) break;
    const size_t o = (i0 + 256 * j) * 4;
    g4[j] = Elem<T>::load_raw4(g + o);
    m4[j] = *reinterpret_cast<const float4*>(m + o);
    v4[j] = *reinterpret_cast<const float4*>(v + o);
    if (MASTER) p4[j] = *reinterpret_cast<const float4*>(master + o);
    else w4[j] = Elem<T>::load_raw4(p + o);
  }
#pragma unroll
  for (int j = 0; j < R; ++j) {
    if (i0 + 256 * j >= n4) break;
    const size_t o = (i0 + 256 * j) * 4;
    if (!MASTER) p4[j] = Elem<T>::widen4(w4[j]);
    const float4 gw = Elem<T>::widen4(g4[j]);
    const float gg[4] = {gw.x, gw.y, gw.z, gw.w};
    float mm[4] = {m4[j].x, m4[j].y, m4[j].z, m4[j].w}, vv[4] = {v4[j].x, v4[j].y, v4[j].z, v4[j].w};
    float pp[4] = {p4[j].x, p4[j].y, p4[j].z, p4[j].w};
#pragma unroll
    for (int k = 0; k < 4; ++k) adam_element(pp[k], mm[k], vv[k], gg[k], a);
    *reinterpret_cast<float4*>(m + o) = make_float4(mm[0], mm[1], mm[2], mm[3]);
    *reinterpret_cast<float4*>(v + o) = make_float4(vv[0], vv[1], vv[2], vv[3]);
    const float4 pn = make_float4(pp[0], pp[1], pp[2], pp[3]);
    if (MASTER) *reinterpret_cast<float4*>(master + o) = pn;
    Elem<T>::store4(p + o, pn);
  }
}

// ---- weight gradients whose tokens were cut into chunks (see SplitTokens): the chunks' partial sums in order, then what the
// contraction's epilogue does otherwise.  grid = (runs of 1024 elements of [M][N], groups); DEC: groups are decoder blocks, rows
// features, with the norm term and, for the next step's norms, the sums of squares of runs of 64 updated weights.  Bound by its traffic
// (16 bytes per lane, everything fp32 but the weights): 3 blocks of 2048 features x 1024 in 2 chunks with the update 32 us, 5.5 TB/s; 10
// blocks of 1024 x 256 12.7 us.
struct CombineArgs {
  int chunks, M, N; const float* part; bf16_t* w; bf16_t* grad; AdamFuseArgs fuse;
  const float* G; const float* norms; float* n2_part; const int32_t* skip_flags; int kcap;
};
template <bool DEC>
__global__ __launch_bounds__(256) void combine_weight_gradient_kernel(Dims D, CombineArgs a) {
  if (DEC && a.skip_flags && lists_backward_selected(a.skip_flags, a.kcap)) return;
  typedef Elem<bf16_t> E;
  const size_t n = (size_t)a.M * a.N, i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= n) return;      // (with n2_part n is a multiple of a workgroup's 1024)
  const int g = blockIdx.y;
  const size_t o = g * n + i;
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
  for (int c = 0; c < a.chunks; ++c) {
    const float4 q = *reinterpret_cast<const float4*>(a.part + ((size_t)g * a.chunks + c) * n + i);
    v.x += q.x; v.y += q.y; v.z += q.z; v.w += q.w;
  }
  float4 w4 = make_float4(0.f, 0.f, 0.f, 0.f);
  if (DEC || (a.fuse.m && !a.fuse.master)) w4 = E::load4(a.w + o);
  const int f = (int)(i / a.N);
  if (DEC) {
    int l = 0, q = g;
    while (q >= D.L - l) { q -= D.L - l; ++l; }
    const float coef = a.G[(size_t)l * D.F + f] * __builtin_amdgcn_rcpf(fmaxf(a.norms[(size_t)l * D.F + f], 1e-30f));
    v = make_float4(fmaf(coef, w4.x, v.x), fmaf(coef, w4.y, v.y), fmaf(coef, w4.z, v.z), fmaf(coef, w4.w, v.w));
  }
  if (a.grad) E::store4(a.grad + o, v);
  if (!a.fuse.m) return;
  const float4 m4 = *reinterpret_cast<const float4*>(a.fuse.m + o), v4 = *reinterpret_cast<const float4*>(a.fuse.v + o),
               p4 = a.fuse.master ? *reinterpret_cast<const float4*>(a.fuse.master + o) : w4;
  const float gg[4] = {v.x, v.y, v.z, v.w};
  float mm[4] = {m4.x, m4.y, m4.z, m4.w}, vv[4] = {v4.x, v4.y, v4.z, v4.w}, pp[4] = {p4.x, p4.y, p4.z, p4.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) adam_element(pp[k], mm[k], vv[k], gg[k], a.fuse.a);
  *reinterpret_cast<float4*>(a.fuse.m + o) = make_float4(mm[0], mm[1], mm[2], mm[3]);
  *reinterpret_cast<float4*>(a.fuse.v + o) = make_float4(vv[0], vv[1], vv[2], vv[3]);
  const float4 pn = make_float4(pp[0], pp[1], pp[2], pp[3]);
  if (a.fuse.master) *reinterpret_cast<float4*>(a.fuse.master + o) = pn;
  const E::Raw4 stored = E::narrow4(pn);
  *reinterpret_cast<E::Raw4*>(a.w + o) = stored;
  if (DEC && a.n2_part) {      // 16 lanes hold a run of 64 columns
    const float4 wn = E::widen4(stored);
    const float s2 = row16_sum((wn.x * wn.x + wn.y * wn.y) + (wn.z * wn.z + wn.w * wn.w));
    if ((threadIdx.x & 15) == 0) a.n2_part[((size_t)g * (a.N >> 6) + (i % a.N >> 6)) * a.M + f] = s2;
  }
}

// the three vectors in one launch, four elements per lane
__global__ __launch_bounds__(256) void adam_vectors_kernel(AdamVectors q, AdamScalars a) {
  const int t = blockIdx.y, i = ((int)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= q.n[t]) return;
  const float4 g4 = *reinterpret_cast<const float4*>(q.g[t] + i);
  const float4 p4 = *reinterpret_cast<const float4*>(q.p[t] + i), m4 = *reinterpret_cast<const float4*>(q.m[t] + i),
               v4 = *reinterpret_cast<const float4*>(q.v[t] + i);
  const float g[4] = {g4.x, g4.y, g4.z, g4.w};
  float p[4] = {p4.x, p4.y, p4.z, p4.w}, m[4] = {m4.x, m4.y, m4.z, m4.w}, v[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) adam_element(p[k], m[k], v[k], g[k], a);
  *reinterpret_cast<float4*>(q.p[t] + i) = make_float4(p[0], p[1], p[2], p[3]);
  *reinterpret_cast<float4*>(q.m[t] + i) = make_float4(m[0], m[1], m[2], m[3]);
  *reinterpret_cast<float4*>(q.v[t] + i) = make_float4(v[0], v[1], v[2], v[3]);
}

// ---- TopK activation: the k largest of a row's F fp32 pre-activations ----------------
// One workgroup per (layer, token) row.  A radix select over the order-preserving integer image
// of the floats finds the k-th largest value in four 8-bit passes (LDS histograms); a last pass
// writes z and the class bytes.  Entries equal to the k-th value are taken in index order until
// k entries are selected; that ordered count runs only for rows that have such ties to break.
#ifndef TOPK_HIST_COPIES
#define TOPK_HIST_COPIES 4
#endif
__device__ __forceinline__ uint32_t order_key(float x) {
  const uint32_t u = __float_as_uint(x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);     // larger float <=> larger key (NaN sorts by its bits)
}

// NV4 > 0: the row (F <= 1024 * NV4) is held in registers, NV4 float4 per lane, and read from memory once;
// NV4 = 0: any F, every pass re-reads the row (it stays in the L2).
template <typename T, int NV4>
__global__ __launch_bounds__(256) void topk_select_kernel(Dims D, const float* __restrict__ pre32, int k,
                                                          T* __restrict__ z, uint8_t* __restrict__ cls,
                                                          int32_t* __restrict__ l0) {
  // (TOPK_HIST_COPIES histograms, one per lane residue: pre-activations share a few exponents, so most keys of the
  //  first pass fall into a handful of bins and atomics on one LDS word serialise)
  __shared__ int hist[TOPK_HIST_COPIES][256];
  __shared__ int sh_bin, sh_rem, scan[256], wtot[4];
  const int tid = threadIdx.x;
  const size_t row = blockIdx.x;
  const float* pr = pre32 + row * D.F;
  const int F4 = D.F / 4;
  const int rounds = NV4 > 0 ? NV4 : (F4 + 255) / 256;
  float4 held[NV4 > 0 ? NV4 : 1];
  if (NV4 > 0) {
#pragma unroll
    for (int j = 0; j < NV4; ++j) {
      const int q = tid + 256 * j;
      // padding sorts below every float (no float maps to key 0), so it is never selected
      held[j] = q < F4 ? *reinterpret_cast<const float4*>(pr + 4 * q) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  auto value4 = [&](int j) -> float4 {        // the lane's j-th float4 (index 4 * (tid + 256 j)); in range only
    if (NV4 > 0) return held[j];
    return *reinterpret_cast<const float4*>(pr + 4 * (tid + 256 * j));
  };
  auto key4 = [&](int j, uint32_t (&key)[4]) {
    const int q = tid + 256 * j;
    if (q < F4) {
      const float4 v = value4(j);
      key[0] = order_key(v.x); key[1] = order_key(v.y); key[2] = order_key(v.z); key[3] = order_key(v.w);
    } else {
      key[0] = key[1] = key[2] = key[3] = 0u;
    }
  };

  uint32_t prefix = 0;
  int remaining = k;            // entries still to take among those whose key matches the prefix so far
  if (k > 0 && k < D.F) {
    for (int shift = 24; shift >= 0; shift -= 8) {
#pragma unroll
      for (int c = 0; c < TOPK_HIST_COPIES; ++c) hist[c][tid] = 0;
      __syncthreads();
      const uint32_t himask = shift == 24 ? 0u : (0xffffffffu << (shift + 8));
#pragma unroll NV4 > 0 ? NV4 : 1
      for (int j = 0; j < rounds; ++j) {
        uint32_t key[4];
        key4(j, key);
        if (tid + 256 * j < F4) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if ((key[i] & himask) == prefix) atomicAdd(&hist[tid & (TOPK_HIST_COPIES - 1)][(key[i] >> shift) & 255u], 1);
        }
      }
      __syncthreads();
      // the bin that holds the `remaining`-th largest entry: suffix sums over the 256 bins (lane = bin),
      // wave scans plus the totals of the higher waves
      {
        int h = 0;
#pragma unroll
        for (int c = 0; c < TOPK_HIST_COPIES; ++c) h += hist[c][tid];
        const int lane = tid & 63, wv = tid >> 6;
        int sfx = h;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const int u = __shfl_down(sfx, off, 64);
          if (lane + off < 64) sfx += u;
        }
        if (lane == 0) wtot[wv] = sfx;
        __syncthreads();
        for (int w2 = wv + 1; w2 < 4; ++w2) sfx += wtot[w2];
        const int above = sfx - h;                  // entries in higher bins
        if (above < remaining && remaining <= sfx) { sh_bin = tid; sh_rem = remaining - above; }
      }
      __syncthreads();
      prefix |= (uint32_t)sh_bin << shift;
      remaining = sh_rem;
      __syncthreads();
    }
  }
  // prefix = key of the k-th largest value; `remaining` of the entries equal to it are selected
  const bool all = k >= D.F, none = k <= 0;
  int eq_total = 0;
  if (!all && !none) {
    int c = 0;
#pragma unroll NV4 > 0 ? NV4 : 1
    for (int j = 0; j < rounds; ++j) {
      uint32_t key[4];
      key4(j, key);
      if (tid + 256 * j < F4) c += (key[0] == prefix) + (key[1] == prefix) + (key[2] == prefix) + (key[3] == prefix);
    }
    scan[tid] = c;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
      if (tid < off) scan[tid] += scan[tid + off];
      __syncthreads();
    }
    eq_total = scan[0];
    __syncthreads();
  }
  const bool ties = !all && !none && eq_total > remaining;     // uniform over the workgroup
  int taken_before = 0;                                         // equal entries in earlier float4 rounds
#pragma unroll NV4 > 0 ? NV4 : 1
  for (int j = 0; j < rounds; ++j) {
    const int q = tid + 256 * j;
    const bool in = q < F4;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (in) v = value4(j);
    const float vv[4] = {v.x, v.y, v.z, v.w};
    uint32_t key[4];
    key4(j, key);
    int rank0 = 0;                                              // equal entries before this lane's first one
    if (ties) {
      const int c = in ? (key[0] == prefix) + (key[1] == prefix) + (key[2] == prefix) + (key[3] == prefix) : 0;
      scan[tid] = c;
      __syncthreads();
      for (int off = 1; off < 256; off <<= 1) {                 // inclusive scan over the 256 lanes
        const int u = tid >= off ? scan[tid - off] : 0;
        __syncthreads();
        scan[tid] += u;
        __syncthreads();
      }
      rank0 = taken_before + scan[tid] - c;
      taken_before += scan[255];
      __syncthreads();
    }
    if (in) {
      float zz[4];
      uint32_t c4 = 0;
      int r = rank0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        bool sel = all || (!none && key[i] > prefix);
        if (!all && !none && key[i] == prefix) {
          sel = !ties || r < remaining;
          ++r;
        }
        zz[i] = sel ? vv[i] : 0.f;
        c4 |= (sel ? (uint32_t)CLS_ACTIVE : 0u) << (8 * i);
      }
      Elem<T>::store4(z + row * D.F + 4 * q, make_float4(zz[0], zz[1], zz[2], zz[3]));
      *reinterpret_cast<uint32_t*>(cls + row * D.F + 4 * q) = c4;
    }
  }
  // every row selects the same number of entries, so one row per layer books the whole layer
  // (a per-row add would send all B*L atomics of the launch to 16 addresses, one after the other)
  if (tid == 0 && l0 && row % D.B == 0) atomicAdd(l0 + (int)(row / D.B), D.B * (all ? D.F : (none ? 0 : k)));
}

// ---- activation normalisation (Sec. 3.1): the factor of a layer is the mean L2 norm of its
// token vectors over the first batches.  Stage 1: grid = (row blocks, L), one wave per row, each
// block leaves the sum of its rows' norms; stage 2 adds the blocks of a layer, in order, to the
// running sum.  int8 rows: the norm of the codes times |row scale|.
// A wave takes four rows at a time, 16 bytes (int8: 8) per lane and row in flight.  L = 16, d = 2048, 4096 tokens of bf16: both
// stages read 268 MB in 59 us, 81 behind plain stores of another 268 MB; the second stage was one chain of loads per layer before, 12 us.
template <typename T, bool INT8>
__global__ __launch_bounds__(256) void row_norm_sum_kernel(Dims D, const void* __restrict__ av,
                                                           const float* __restrict__ a_scale,
                                                           double* __restrict__ part) {
  constexpr int N = INT8 ? 8 : Row16<T>::N, R = 4;
  const int rb = blockIdx.x, l = blockIdx.y, lane = threadIdx.x & 63;
  const int r0 = rb * LOSS_ROWS_PER_BLOCK, r1 = min(D.B, r0 + LOSS_ROWS_PER_BLOCK);
  double s = 0.0;   // the same value in every lane of a wave
  for (int r = r0 + (threadIdx.x >> 6) * R; r < r1; r += 4 * R) {
    float acc[R] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
    for (int c = lane * N; c < D.d; c += 64 * N) {
      u32x4 raw[R];
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const size_t o = ((size_t)l * D.B + min(r + j, r1 - 1)) * D.d + c;
        if (INT8) {
          const uint2 q = *reinterpret_cast<const uint2*>(reinterpret_cast<const int8_t*>(av) + o);
          raw[j] = u32x4{q.x, q.y, 0u, 0u};
        } else {
          raw[j] = load16(reinterpret_cast<const T*>(av) + o);
        }
      }
#pragma unroll
      for (int j = 0; j < R; ++j) {
        float v[N];
        if constexpr (INT8) {
#pragma unroll
          for (int i = 0; i < N; ++i) v[i] = (float)(int8_t)(raw[j][i / 4] >> (8 * (i & 3)));
        } else {
          widen16(raw[j], v);
        }
#pragma unroll
        for (int i = 0; i < N; i += 4) acc[j] += (v[i] * v[i] + v[i + 1] * v[i + 1]) + (v[i + 2] * v[i + 2] + v[i + 3] * v[i + 3]);
      }
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (r + j >= r1) break;
      float n = sqrtf(wave_sum(acc[j]));
      if (INT8) n *= fabsf(a_scale[(size_t)l * D.B + r + j]);
      s += (double)n;
    }
  }
  __shared__ double sh[4];
  if (lane == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) part[(size_t)l * gridDim.x + rb] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// one wavefront per layer
__global__ __launch_bounds__(64) void norm_sum_final_kernel(int nrb, const double* __restrict__ part, double* __restrict__ norm_sum) {
  const int l = blockIdx.x;
  double s = 0.0;
#pragma unroll 4
  for (int i = threadIdx.x; i < nrb; i += 64) s += part[(size_t)l * nrb + i];
  s = wave_sum(s);
  if (threadIdx.x == 0) norm_sum[l] += s;
}

// 1 / c[l] = n_tokens / norm_sum[l]; a layer that summed to zero has no scale and keeps factor 1
__device__ __forceinline__ float inv_norm_factor(const double* norm_sum, int l, double n_tokens) {
  const double s = norm_sum[l];
  return s > 0.0 ? (float)(n_tokens / s) : 1.0f;
}

// int8 rows: the division folds into the dequantisation scale, the codes stay as they are
__global__ void normalise_scale_kernel(Dims D, const double* __restrict__ norm_sum, double n_tokens,
                                       const float* __restrict__ scale_in, float* __restrict__ scale_out) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (size_t)D.L * D.B) return;
  scale_out[i] = scale_in[i] * inv_norm_factor(norm_sum, (int)(i / D.B), n_tokens);
}

// native rows: a_out = a_in / c[l] (a_out may be a_in); grid = (chunks of a layer, L).  Bound by memory.  STREAM: non-temporal stores,
// for batches that do not fit the 256 MB Infinity Cache together with the result.  The division itself hardly gains (L = 16, d = 2048, 4096
// tokens of bf16: 81.5 -> 79.6 us); what gains is the next reading, here the norm sum of the batch after, which does not wait behind the
// write-back any more (81 -> 59 us).  Both, another batch each time: 159.9 -> 135.4 us, in fp32 with L = 8 153.2 -> 133.6; the same batch
// again, part of it still in the cache, 154.5 -> 124.4 and 143.5 -> 127.7.  75 MB: 51 and 41 us with either, and the forward pass that follows may
// find the result in the cache.
constexpr int NORM_LOADS = 4;      // 16-byte pieces per lane
template <typename T, bool STREAM>
__global__ __launch_bounds__(256) void normalise_rows_kernel(Dims D, const double* __restrict__ norm_sum,
                                                             double n_tokens, const T* a_in, T* a_out) {
  constexpr int N = Row16<T>::N, R = NORM_LOADS;
  const int l = blockIdx.y;
  const float k = inv_norm_factor(norm_sum, l, n_tokens);
  const size_t n = (size_t)D.B * D.d / N, base = (size_t)l * D.B * D.d, i0 = (size_t)blockIdx.x * (256 * R) + threadIdx.x;
  u32x4 raw[R];
#pragma unroll
  for (int j = 0; j < R; ++j)
    if (i0 + 256 * j < n) raw[j] = load16(a_in + base + (i0 + 256 * j) * N);
#pragma unroll
  for (int j = 0; j < R; ++j) {
    if (i0 + 256 * j >= n) break;
    float v[N];
    widen16(raw[j], v);
#pragma unroll
    for (int q = 0; q < N; ++q) v[q] *= k;
    if (STREAM) nt_store16(a_out + base + (i0 + 256 * j) * N, v); else store16(a_out + base + (i0 + 256 * j) * N, v);
  }
}

// Scratch of the entry point that allocates nothing: the per-block partial sums of the activation-norm
// reduction, held in the library's own device memory instead of a caller workspace.  One copy per GPU
// for the life of the process (512 KB); every call on a GPU uses that GPU's copy.
static __device__ __align__(256) double scratch[STATIC_SCRATCH_DOUBLES];
constexpr int MAX_DEVICES = 64;
double* g_scratch_ptr[MAX_DEVICES] = {};   // device address of `scratch` on each GPU, resolved once

}  // namespace

hipError_t launch_zero_i32(hipStream_t s, int32_t* p, int n) {
  hipLaunchKernelGGL(zero_i32_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

hipError_t launch_topk_select(hipStream_t s, bool bf16, Dims D, const float* pre32, int k, void* z, uint8_t* cls,
                              int32_t* l0) {
  const dim3 grid((unsigned)((size_t)D.L * D.B));
#define CLT_TOPK(T, NV4) \
  hipLaunchKernelGGL((topk_select_kernel<T, NV4>), grid, dim3(256), 0, s, D, pre32, k, (T*)z, cls, l0)
  const int nv4 = D.F <= 2048 ? 2 : (D.F <= 8192 ? 8 : 0);     // registers for rows up to 8192 features
  if (bf16) { if (nv4 == 2) CLT_TOPK(bf16_t, 2); else if (nv4 == 8) CLT_TOPK(bf16_t, 8); else CLT_TOPK(bf16_t, 0); }
  else { if (nv4 == 2) CLT_TOPK(float, 2); else if (nv4 == 8) CLT_TOPK(float, 8); else CLT_TOPK(float, 0); }
#undef CLT_TOPK
  return hipGetLastError();
}

hipError_t launch_decode_combine(hipStream_t s, Dims D, DecSplit sp, const float* part, const float* b_dec, float* y_hat,
                                 const int32_t* skip_flags, int kcap) {
  const dim3 grid((unsigned)(((size_t)D.B * D.d + 1023) / 1024), D.L);
  hipLaunchKernelGGL(decode_combine_kernel, grid, dim3(256), 0, s, D, sp, part, b_dec, y_hat, skip_flags, kcap);
  return hipGetLastError();
}

hipError_t launch_decoder_norms(hipStream_t s, bool bf16, Dims D, const void* W_dec, float* norms, int32_t* l0) {
  const long rows = (long)D.L * D.F;
  const dim3 grid((unsigned)((rows + 3) / 4));
  if (bf16)
    hipLaunchKernelGGL((decoder_norms_kernel<bf16_t>), grid, dim3(256), 0, s, D, (const bf16_t*)W_dec, norms, l0);
  else
    hipLaunchKernelGGL((decoder_norms_kernel<float>), grid, dim3(256), 0, s, D, (const float*)W_dec, norms, l0);
  return hipGetLastError();
}

hipError_t launch_norms_from_partials(hipStream_t s, Dims D, const float* n2_part, int runs, float* norms,
                                      const int32_t* flags, int kcap, int32_t* l0) {
  const long rows = (long)D.L * D.F;
  hipLaunchKernelGGL(norms_from_partials_kernel, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, s, D, n2_part, runs, norms,
                     flags, kcap, l0);
  return hipGetLastError();
}

hipError_t launch_loss(hipStream_t s, bool bf16, bool int8_y, Dims D, const void* z, const float* norms, float C, const void* pre,
                       const float* theta, bool log_threshold, double* sp_part, float* sp_cols, double* dead_part, float* dead_cols,
                       const float* y_hat, const void* y, const float* y_scale, void* d_yhat, double* rec_part, float* rec_cols) {
  const ReduceGrid rf = reduce_grid(bf16, D, D.F), rd = reduce_grid(bf16, D, D.d);
  const LossArgs a{rf.rows, rf.chunks, rf.blocks(), rd.rows, rd.chunks, rd.blocks(), z, norms, C, pre, theta, log_threshold,
                   sp_part, sp_cols, dead_part, dead_cols, y_hat, y, y_scale, d_yhat, rec_part, rec_cols};
  const dim3 grid(rf.blocks() + rd.blocks(), D.L);
#define CLT_LOSS(T, INT8)                                                                              \
  do {                                                                                                 \
    if (pre) hipLaunchKernelGGL((loss_kernel<T, INT8, true>), grid, dim3(256), 0, s, D, a);            \
    else hipLaunchKernelGGL((loss_kernel<T, INT8, false>), grid, dim3(256), 0, s, D, a);               \
  } while (0)
  if (!bf16) CLT_LOSS(float, false); else if (int8_y) CLT_LOSS(bf16_t, true); else CLT_LOSS(bf16_t, false);
#undef CLT_LOSS
  return hipGetLastError();
}

hipError_t launch_loss_finish(hipStream_t s, Dims D, const double* part_rec, int n_rec, const double* part_sp, int n_sp,
                              const double* part_dead_or_null, float inv_B, float lambda0, float lambda1, float* loss_dev,
                              const float* sp_cols, const float* dead_cols, int nparts, float* G) {
  const int ncols = D.L * D.F;
  const bool few = std::max(n_rec, n_sp) <= LF_FEW;
  const int cols = few ? 64 : 256;
  hipLaunchKernelGGL(few ? loss_finish_kernel<256> : loss_finish_kernel<1024>, dim3(1 + (ncols + cols - 1) / cols), dim3(4 * cols), 0, s,
                     part_rec, n_rec, part_sp, n_sp, part_dead_or_null, inv_B, lambda0, lambda1, lambda0 / (float)D.B, lambda1 / (float)D.B,
                     loss_dev, sp_cols, dead_cols, nparts, ncols, G);
  return hipGetLastError();
}

hipError_t launch_vector_gradients(hipStream_t s, const VectorGradArgs& a) {
  hipLaunchKernelGGL(vector_gradients_kernel, dim3((a.nF + 63) / 64 + (a.nd + 63) / 64), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_ste_reduce(hipStream_t s, bool bf16, Dims D, void* dpre, const uint8_t* cls,
                             const float* row_scale_or_null, const float* norms, float lam1_over_b,
                             float* part_theta, float* part_benc, float* part_below,
                             const int32_t* only_if_lists, int kcap) {
  const ReduceGrid rg = reduce_grid(bf16, D, D.F);
  const dim3 grid(rg.blocks(), D.L);
  if (bf16)
    hipLaunchKernelGGL((ste_reduce_kernel<bf16_t>), grid, dim3(256), 0, s, D, rg.rows, rg.chunks, (bf16_t*)dpre, cls, row_scale_or_null,
                       norms, lam1_over_b, part_theta, part_benc, part_below, only_if_lists, kcap);
  else
    hipLaunchKernelGGL((ste_reduce_kernel<float>), grid, dim3(256), 0, s, D, rg.rows, rg.chunks, (float*)dpre, cls, row_scale_or_null,
                       norms, lam1_over_b, part_theta, part_benc, part_below, only_if_lists, kcap);
  return hipGetLastError();
}

hipError_t launch_adam_matrix(hipStream_t s, bool bf16, size_t n, void* p, const void* g, float* m, float* v,
                              float* master, AdamScalars a) {
  const size_t n4 = n / 4;   // matrices have a multiple of 64 elements (d, F multiples of 8)
  const dim3 grid((unsigned)((n4 + 256 * ADAM_QUADS - 1) / (256 * ADAM_QUADS)));
  if (bf16) {
    if (master)
      hipLaunchKernelGGL((adam_kernel<bf16_t, true>), grid, dim3(256), 0, s, n4, (bf16_t*)p, (const bf16_t*)g, m, v,
                         master, a);
    else
      hipLaunchKernelGGL((adam_kernel<bf16_t, false>), grid, dim3(256), 0, s, n4, (bf16_t*)p, (const bf16_t*)g, m, v,
                         master, a);
  } else {
    if (master)
      hipLaunchKernelGGL((adam_kernel<float, true>), grid, dim3(256), 0, s, n4, (float*)p, (const float*)g, m, v,
                         master, a);
    else
      hipLaunchKernelGGL((adam_kernel<float, false>), grid, dim3(256), 0, s, n4, (float*)p, (const float*)g, m, v,
                         master, a);
  }
  return hipGetLastError();
}

hipError_t launch_combine_dwdec(hipStream_t s, Dims D, int chunks, const DWdecArgs& a) {
  const CombineArgs c{chunks, D.F, D.d, a.split_part, (bf16_t*)a.W_dec, (bf16_t*)a.dW_dec, a.fuse, a.G, a.norms,
                      a.fuse.m && D.F % 256 == 0 && D.d % 256 == 0 ? a.n2_part : nullptr, a.skip_flags, a.kcap};
  const dim3 grid((unsigned)(((size_t)D.F * D.d + 1023) / 1024), D.P());
  hipLaunchKernelGGL((combine_weight_gradient_kernel<true>), grid, dim3(256), 0, s, D, c);
  return hipGetLastError();
}
hipError_t launch_combine_dwenc(hipStream_t s, Dims D, int chunks, const DWencArgs& a) {
  const CombineArgs c{chunks, D.d, D.F, a.split_part, (bf16_t*)a.W_enc, (bf16_t*)a.dW_enc, a.fuse, nullptr, nullptr, nullptr, nullptr, 0};
  const dim3 grid((unsigned)(((size_t)D.F * D.d + 1023) / 1024), D.L);
  hipLaunchKernelGGL((combine_weight_gradient_kernel<false>), grid, dim3(256), 0, s, D, c);
  return hipGetLastError();
}

hipError_t launch_adam_vectors(hipStream_t s, const AdamVectors& a, AdamScalars sc) {
  const int most = (std::max(a.n[0], std::max(a.n[1], a.n[2])) / 4 + 255) / 256;      // vectors have L*F or L*d elements, multiples of 8
  hipLaunchKernelGGL(adam_vectors_kernel, dim3(most, 3), dim3(256), 0, s, a, sc);
  return hipGetLastError();
}

hipError_t launch_norm_accumulate(hipStream_t s, bool bf16, bool int8_a, Dims D, const void* a, const float* a_scale,
                                  double* part, double* norm_sum) {
  const dim3 grid(row_blocks(D.B), D.L);
  if (!bf16)
    hipLaunchKernelGGL((row_norm_sum_kernel<float, false>), grid, dim3(256), 0, s, D, a, a_scale, part);
  else if (int8_a)
    hipLaunchKernelGGL((row_norm_sum_kernel<bf16_t, true>), grid, dim3(256), 0, s, D, a, a_scale, part);
  else
    hipLaunchKernelGGL((row_norm_sum_kernel<bf16_t, false>), grid, dim3(256), 0, s, D, a, a_scale, part);
  hipLaunchKernelGGL(norm_sum_final_kernel, dim3(D.L), dim3(64), 0, s, (int)grid.x, part, norm_sum);
  return hipGetLastError();
}

// Device address of this GPU's `scratch` array (the array's name is only a host-side handle for
// hipGetSymbolAddress; kernels get the resolved pointer as an argument).  Resolved once per device,
// with that device current.
hipError_t static_scratch(double** ptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  double* p = __atomic_load_n(&g_scratch_ptr[dev], __ATOMIC_ACQUIRE);
  if (!p) {
    e = hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    __atomic_store_n(&g_scratch_ptr[dev], p, __ATOMIC_RELEASE);   // every thread resolves the same address
  }
  *ptr = p;
  return hipSuccess;
}

hipError_t launch_normalise(hipStream_t s, bool bf16, bool int8_a, Dims D, const double* norm_sum, double n_tokens,
                            const void* a_in, const float* scale_in, void* a_out, float* scale_out) {
  if (int8_a) {
    const size_t n = (size_t)D.L * D.B;
    hipLaunchKernelGGL(normalise_scale_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, D, norm_sum,
                       n_tokens, scale_in, scale_out);
  } else {
    const size_t per_wg = 256 * NORM_LOADS * (bf16 ? 8 : 4), n = (size_t)D.B * D.d;      // elements (rows are multiples of 8 elements)
    const dim3 grid((unsigned)((n + per_wg - 1) / per_wg), D.L);
    const bool stream = (double)D.L * n * (bf16 ? 2 : 4) > 128e6;
#define CLT_NORM(T, STREAM) \
  hipLaunchKernelGGL((normalise_rows_kernel<T, STREAM>), grid, dim3(256), 0, s, D, norm_sum, n_tokens, (const T*)a_in, (T*)a_out)
    if (bf16) { if (stream) CLT_NORM(bf16_t, true); else CLT_NORM(bf16_t, false); }
    else { if (stream) CLT_NORM(float, true); else CLT_NORM(float, false); }
#undef CLT_NORM
  }
  return hipGetLastError();
}

}  // namespace clt
