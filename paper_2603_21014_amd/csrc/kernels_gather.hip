// Active-feature gather paths (paper Sec. 3.2 "Sparse Decode"): once training
// has pushed the activations into the sparse regime, each token looks up only
// the decoder rows of its active features, O(k d) instead of the dense O(F d)
// contraction.  The paper does this for the forward decode; the same lists also
// drive the two backward contractions through the decoder here.
//   decide    reads the per-layer active counts of the encoder epilogue and sets
//             the device-side switch (no host round trip);
//   compact   turns every (layer, token) row of z into an ordered list of
//             (feature, value) pairs, plus the inactive features inside the
//             threshold window (needed by the threshold gradient);
//   gather decode   one wavefront per (token, target layer, run of 256 columns): walks
//             the sources l <= l' and their lists, four columns of the listed decoder
//             rows per lane, and accumulates in fp32 registers;
//   stepped gather decode   the same sums with all tokens of the batch at one (source,
//             target) block at a time, so that its rows come out of the L2;
//   gather dz       one workgroup per (layer, token): dot products of the listed
//             features' decoder rows with the token's d y_hat rows;
//   feature lists   transpose of the row lists: per (layer, feature) the tokens on
//             which it is active, built by a column scan in token order;
//   sparse dW_dec   one wavefront per (source, target, feature, slice of columns): sums
//             the d y_hat rows of the feature's tokens, adds the norm term and runs
//             the fused Adam update of the row; takes the partial dot products of dz along.
// Every order of summation is fixed, so the results are bitwise reproducible
// (no floating-point atomics).  Decode and dz read B * k * P * d * sizeof(T)
// bytes of decoder rows (HBM/L2-bound); sparse dW_dec streams the optimizer
// state once, like a plain Adam pass, and reads its d y_hat rows out of the L2.
#include "common.h"

#include <cstdlib>

#include <type_traits>

namespace clt {
namespace {

constexpr int SGD_WAVES = 16, SGD_WGS = 64, SGD_TPW = 4;      // wavefronts per workgroup, workgroups per XCD, tokens per wavefront
constexpr int SGD_TOKENS = SGD_TPW * SGD_WAVES;

// Whether the decode that goes through the blocks in step is the faster one, by the times (us) of both; pairs: (entry, target) pairs of
// the batch, k: entries per (layer, token).  In step: an XCD takes an eighth of the P x ns (block, slice of 128 columns) steps, each for the
// whole batch; a step has its price for every pass over the tokens and for every token whatever they list, entries come on top
// (below 256 tokens their chains are too few to hide their latency).  Otherwise: entries by their columns, cheaper where a
// source's 256 columns stay in the L2 (F of a few thousand), but no faster than the chain of the last target.  Over 95 sizes (L = 8 to 16,
// d = 136 to 2304, F = 1024 to 8192, 70 to 8192 tokens, 4 to 900 entries) the pick is the faster one or within 8 % of it.  A rule on the tokens per
// feature alone (six or more) took 1333 tokens of 4.7 entries at L = 16, d = 2048, F = 1024 in step, 1193 us against 393, and left
// 2500 tokens of 12 at L = 12, d = 768, F = 6144 out of step, 498 against 458.
__host__ __device__ inline bool stepping_pays(Dims D, double pairs, double k) {
  const int ns = (D.d + 127) / 128, passes = (D.B + SGD_WGS * SGD_TOKENS - 1) / (SGD_WGS * SGD_TOKENS);
  const double slots = 0.25 + D.F / 4500.0, chain = 0.075 * D.L * k;
  const double apart = 3.3e-5 * pairs * D.d / 128.0 * (slots < 1.0 ? slots : 1.0);
  const double in_step = 0.125 * D.P() * ns * (1.5 + 1.7 * passes + 0.9e-3 * D.B) + 1e-5 * pairs * ns * (D.B < 256 ? 256.0 / D.B : 1.0);
  return in_step < (apart > chain ? apart : chain);
}

__global__ __launch_bounds__(512) void decode_decide_kernel(Dims D, const int32_t* __restrict__ l0, float thr, float thr_bwd, int forced,
                                                            int rows_free, int can_step, int32_t* __restrict__ flags,
                                                            uint32_t* __restrict__ step_ctr) {
  step_ctr[threadIdx.x] = 0u;      // pacing of the stepped decode: 8 lines of 64 words
  if (threadIdx.x != 0) return;
  long long tot = 0, pairs = 0;
  for (int l = 0; l < D.L; ++l) { tot += l0[l]; pairs += (long long)l0[l] * (D.L - l); }
  const double dens = (double)tot / ((double)D.L * D.B * D.F);
  flags[0] = ((forced || dens <= (double)thr) ? 1 : 0) | ((forced || dens <= (double)thr_bwd) ? 2 : 0) |
             (rows_free ? 4 : 0);
  flags[1] = 0;
  flags[2] = 1;
  flags[3] = 0;
  flags[4] = can_step && stepping_pays(D, (double)pairs, dens * D.F) ? (int)(4.0 * dens * D.F) + 64 : -1;
}

// One wavefront per (layer, token) row; lanes take 16 consecutive features per pass (two 8-byte
// loads of class bytes: F is a multiple of 8, so a row start is 8-byte aligned), positions come
// from wave-wide exclusive scans of the per-lane counts: 8 passes and 16 scans for 8192 features.
// Active features fill the row's slots from the front, window-only features from the back.
// z is read only where a group of 4 features holds an active one.
__device__ __forceinline__ int wave_incl_scan(int v, int lane) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int u = __shfl_up(v, off, 64);
    if (lane >= off) v += u;
  }
  return v;
}

template <typename T>
__global__ __launch_bounds__(256) void compact_active_kernel(Dims D, const T* __restrict__ z,
                                                             const uint8_t* __restrict__ cls, GatherLists g,
                                                             int32_t* __restrict__ flags) {
  // the row lists serve the gather decode, and the backward unless it works from the per-feature lists alone
  if (!((flags[0] & 1) || ((flags[0] & 2) && !(flags[0] & 4)))) return;
  const int lane = threadIdx.x & 63;
  const long row = (long)blockIdx.x * 4 + (threadIdx.x >> 6);   // l * B + b
  if (row >= (long)D.L * D.B) return;
  const T* zr = z + (size_t)row * D.F;
  const uint8_t* cr = cls + (size_t)row * D.F;
  int32_t* oi = g.idx + (size_t)row * g.stride;
  float* ov = g.val + (size_t)row * g.stride;
  int base = 0, base_w = 0;
  for (int f0 = 0; f0 < D.F; f0 += 1024) {
    const int f = f0 + lane * 16;
    uint32_t c[4] = {0u, 0u, 0u, 0u};
    if (f < D.F) {
      const uint2 lo = *reinterpret_cast<const uint2*>(cr + f);
      c[0] = lo.x; c[1] = lo.y;
    }
    if (f + 8 < D.F) {
      const uint2 hi = *reinterpret_cast<const uint2*>(cr + f + 8);
      c[2] = hi.x; c[3] = hi.y;
    }
    uint32_t a[4], w[4];
    int n = 0, nw = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      a[j] = c[j] & 0x01010101u;                          // active
      w[j] = ((c[j] >> 1) & 0x01010101u) & ~a[j];         // in the window, not active
      n += __popc(a[j]);
      nw += __popc(w[j]);
    }
    const int incl = wave_incl_scan(n, lane), incl_w = wave_incl_scan(nw, lane);
    int pos = base + incl - n, pos_w = base_w + incl_w - nw;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if ((a[j] | w[j]) == 0u) continue;
      float4 z4 = make_float4(0.f, 0.f, 0.f, 0.f);
      if (a[j]) z4 = Elem<T>::load4(zr + f + 4 * j);
      const float zz[4] = {z4.x, z4.y, z4.z, z4.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if ((a[j] >> (8 * i)) & 1u) {
          if (pos < g.kcap) { oi[pos] = f + 4 * j + i; ov[pos] = zz[i]; }
          ++pos;
        }
        if ((w[j] >> (8 * i)) & 1u) {
          if (pos_w < g.kcap) { oi[g.kcap - 1 - pos_w] = f + 4 * j + i; ov[g.kcap - 1 - pos_w] = 0.f; }
          ++pos_w;
        }
      }
    }
    base += __shfl(incl, 63, 64);
    base_w += __shfl(incl_w, 63, 64);
  }
  if (lane == 0) {
    g.counts[row] = base;
    g.counts_w[row] = base_w;
    // longest list so far; lists that collide make every gather kernel stand down.  The value only
    // grows, so a row that does not exceed what is already there (a stale read at worst costs an
    // atomic that changes nothing) leaves the one hot address alone.
    const int mine = base + base_w;
    if (mine > *reinterpret_cast<volatile const int32_t*>(flags + 1)) atomicMax(flags + 1, mine);
  }
}

// Address = wave-uniform base + the lane's fixed element offset (one 32-bit register per lane).
template <typename X>
__device__ __forceinline__ X* lane_ptr(X* uniform_base, uint32_t lane_elems) {   // base + lane offset, 32-bit lane part
  typedef typename std::conditional<std::is_const<X>::value, const char, char>::type Byte;
  return reinterpret_cast<X*>(reinterpret_cast<Byte*>(uniform_base) + lane_elems * (uint32_t)sizeof(X));
}

// 8 consecutive elements kept as loaded (16 bytes of bf16 or 32 bytes of fp32) until they are used
template <typename T> struct Raw8;
template <> struct Raw8<bf16_t> {
  typedef uint4 type;
  static __device__ __forceinline__ type load(const bf16_t* p) { return *reinterpret_cast<const uint4*>(p); }
  static __device__ __forceinline__ float dot(const type& a, const type& b, float acc) {
    const uint32_t x[4] = {a.x, a.y, a.z, a.w}, y[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      acc = fmaf(__uint_as_float(x[i] << 16), __uint_as_float(y[i] << 16), acc);
      acc = fmaf(__uint_as_float(x[i] & 0xffff0000u), __uint_as_float(y[i] & 0xffff0000u), acc);
    }
    return acc;
  }
};
template <> struct Raw8<float> {
  struct type { float4 lo, hi; };
  static __device__ __forceinline__ type load(const float* p) {
    return type{*reinterpret_cast<const float4*>(p), *reinterpret_cast<const float4*>(p + 4)};
  }
  static __device__ __forceinline__ float dot(const type& a, const type& b, float acc) {
    acc = fmaf(a.lo.x, b.lo.x, acc); acc = fmaf(a.lo.y, b.lo.y, acc); acc = fmaf(a.lo.z, b.lo.z, acc);
    acc = fmaf(a.lo.w, b.lo.w, acc); acc = fmaf(a.hi.x, b.hi.x, acc); acc = fmaf(a.hi.y, b.hi.y, acc);
    acc = fmaf(a.hi.z, b.hi.z, acc); acc = fmaf(a.hi.w, b.hi.w, acc);
    return acc;
  }
};

// One wavefront per (token, target, run of 256 columns): 4 columns per lane, the sources l <= l' and their lists in
// order.  Feature ids and values are wave-uniform, so a decoder row is a scalar base plus the lane's fixed column
// offset; eight rows are in flight for long lists, four for short ones.  The runs of a row are neighbours in the
// grid, and workgroups go round-robin to the XCDs: with d = 2048 an XCD always gets the same eighth of the columns,
// so the eight L2s hold disjoint parts of the decoder instead of eight copies of what is hot, and the long rows of
// a heavy-tailed batch are spread over eight CUs instead of going through one.
template <typename T, int U>
__device__ __forceinline__ void gather_rows(float (&acc)[4], const T* __restrict__ Wp, int ld, uint32_t col,
                                            const int32_t* __restrict__ ii, const float* __restrict__ vv, int j) {
  typename Elem<T>::Raw4 r[U];
  float v[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int f = __builtin_amdgcn_readfirstlane(ii[j + u]);
    v[u] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(vv[j + u])));
    r[u] = Elem<T>::load_raw4(lane_ptr(Wp + (size_t)f * ld, col));
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const float4 q = Elem<T>::widen4(r[u]);
    acc[0] = fmaf(v[u], q.x, acc[0]);
    acc[1] = fmaf(v[u], q.y, acc[1]);
    acc[2] = fmaf(v[u], q.z, acc[2]);
    acc[3] = fmaf(v[u], q.w, acc[3]);
  }
}

constexpr int GD_COLS = 256;      // columns per wavefront
// (four wavefronts, of consecutive tokens, per workgroup: a launch that stands down costs a quarter of the empty workgroups)
template <typename T>
__global__ __launch_bounds__(256) void gather_decode_kernel(Dims D, GatherLists g, const T* __restrict__ W_dec,
                                                          const float* __restrict__ b_dec,
                                                          float* __restrict__ y_hat, int32_t* __restrict__ flags) {
  if (!gather_selected(flags, g.kcap) || stepped_decode_selected(flags)) return;
  const int ncs = (D.d + GD_COLS - 1) / GD_COLS, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cs = (int)(blockIdx.x % ncs);
  const size_t bt = (size_t)(blockIdx.x / ncs) * 4 + wv;
  if (blockIdx.x == 0 && threadIdx.x == 0) flags[2] = 2;
  if (bt >= (size_t)D.L * D.B) return;
  const int lp = D.L - 1 - (int)(bt / D.B);   // heaviest targets first
  const int b = (int)(bt % D.B);
  const int col = cs * GD_COLS + (threadIdx.x & 63) * 4;
  if (col >= D.d) return;
  float acc[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i] = b_dec[(size_t)lp * D.d + col + i];
  for (int l = 0; l <= lp; ++l) {
    const size_t row = (size_t)l * D.B + b;
    const int cnt = g.counts[row];
    const int32_t* ii = g.idx + row * g.stride;
    const float* vv = g.val + row * g.stride;
    const T* Wp = W_dec + (size_t)packed_index(l, lp, D.L) * D.F * D.d;
    int j = 0;
    for (; j + 8 <= cnt; j += 8) gather_rows<T, 8>(acc, Wp, D.d, (uint32_t)col, ii, vv, j);
    if (j + 4 <= cnt) { gather_rows<T, 4>(acc, Wp, D.d, (uint32_t)col, ii, vv, j); j += 4; }
    for (; j < cnt; ++j) gather_rows<T, 1>(acc, Wp, D.d, (uint32_t)col, ii, vv, j);
  }
  *reinterpret_cast<float4*>(y_hat + ((size_t)lp * D.B + b) * D.d + col) = make_float4(acc[0], acc[1], acc[2], acc[3]);
}

typedef unsigned int u32x4_lds __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_mfma __attribute__((ext_vector_type(8)));
typedef float f32x4_mfma __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void wave_lds_order() {      // a wave's LDS accesses complete in order; this keeps the compiler to it
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Streaming accesses of a wavefront to `bytes` bytes from a uniform address on: base and bounds in scalar registers, the lane's
// 32-bit offset as it is; lanes beyond the end load zeros and store nothing.  (With pointers, base + lane of every array was hoisted
// out of the item loop, two registers per lane each, and spilled.)
// The descriptor is put into scalar registers here, whatever the compiler makes of its parts.  A descriptor that it takes for
// different from lane to lane costs a loop over the lanes around every access, which ends with no lane at work; the register
// allocator then puts copies and spill stores behind such a loop before the lanes come back, and their values are lost (a row kernel of
// dW_dec like that, limited to 80 or 72 registers, gave wrong updates).  build.py refuses a listing that shows it.
struct UniformRun {
  __amdgpu_buffer_rsrc_t d;
  static constexpr int NT = 2;      // cache policy: non-temporal
  __device__ __forceinline__ UniformRun(const void* p, int bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    d = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>((uint64_t)hi << 32 | lo), 0, __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
  }
  __device__ __forceinline__ nt_f32x4 load_f4(uint32_t o) const { return __builtin_bit_cast(nt_f32x4, __builtin_amdgcn_raw_buffer_load_b128(d, (int)o, 0, NT)); }
  __device__ __forceinline__ nt_u32x2 load8(uint32_t o) const { return __builtin_bit_cast(nt_u32x2, __builtin_amdgcn_raw_buffer_load_b64(d, (int)o, 0, NT)); }
  __device__ __forceinline__ uint32_t load4(uint32_t o) const { return __builtin_amdgcn_raw_buffer_load_b32(d, (int)o, 0, 0); }
  __device__ __forceinline__ void store_f4(uint32_t o, nt_f32x4 v) const {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(__attribute__((__vector_size__(16))) unsigned int, v), d, (int)o, 0, NT);
  }
  __device__ __forceinline__ void store8(uint32_t o, nt_u32x2 v, int policy) const {
    const __attribute__((__vector_size__(8))) unsigned int t = {v[0], v[1]};
    if (policy) __builtin_amdgcn_raw_buffer_store_b64(t, d, (int)o, 0, NT); else __builtin_amdgcn_raw_buffer_store_b64(t, d, (int)o, 0, 0);
  }
  __device__ __forceinline__ void store4(uint32_t o, uint32_t v) const { __builtin_amdgcn_raw_buffer_store_b32(v, d, (int)o, 0, 0); }
};

// The decode of a batch whose features are active on several tokens each, bf16 storage: all tokens of the batch go through the
// (source, target) blocks in step, so that a block's rows come out of the L2 from the second token on.
// An XCD works on one target and 128 columns at a time: the slice of a block is F x 256 bytes (2 MB at F = 8192, half of its L2), all
// 4096 tokens of a batch are spread over its wavefronts and keep their sums in LDS across the sources.  At every source the
// workgroup books itself on its XCD's counter and waits, for a bounded time, until all of the XCD have begun the source before:
// a pacing aid that no result depends on.  (The counter is only touched from one XCD, in its L2; an atomic that has to be seen by
// the whole device takes ten times as long here.)  The sums are taken as in the row kernel of dW_dec below: four entries and 128
// columns per load and MFMA.
// What bounds it: a step takes about 7 us at 4096 tokens for the pacing, the latency of lists and rows and the 2 MB per XCD that come
// from memory, 3.3 at 512; the entries come on top at 20 to 25 TB/s of rows.  L = 16, d = 2048, F = 8192, against the kernel above: 4096 tokens, 4
// active features each 1.42 -> 2.47 ms, 8: 2.41 -> 2.57, 16: 4.66 -> 3.30, 32: 9.01 -> 5.00; 4100 tokens (a second pass for four of them) 4.52 -> 3.83 at
// 16; 8192: 8.85 -> 6.12; 2048: 2.28 -> 2.16; 512: 0.63 -> 1.07.  L = 12, d = 768, F = 6144, 4096 tokens, 6: 0.40 -> 0.54, 12: 0.81 ->
// 0.60.  F = 1024 and 10 at L = 16, d = 2048: 1.59 -> 2.06.  Long-tailed lists (25 on average, 300 at most): 2.36 -> 2.59, one wavefront
// holds up its XCD.  72 MB of decoder in all (L = 5, d = 776, F = 3080, 3001 tokens), 14: 0.114 -> 0.133, 41: 0.265 -> 0.228.  Hence the rule:
// stepping_pays, no list longer than four times the mean + 64, a slice that fits half an L2 and a decoder of several L2s.
__global__ __launch_bounds__(64 * SGD_WAVES, 8) void stepped_gather_decode_kernel(
    Dims D, int kcap, int stride, const int32_t* __restrict__ counts, const int32_t* __restrict__ idx, const float* __restrict__ val,
    const bf16_t* __restrict__ W_dec, const float* __restrict__ b_dec, float* __restrict__ y_hat, int32_t* __restrict__ flags,
    uint32_t* __restrict__ ctr0, int nw) {
  if (!gather_selected(flags, kcap) || !stepped_decode_selected(flags)) return;
  __shared__ __align__(16) float acc_s[SGD_TOKENS][128];
  __shared__ __align__(16) nt_u32x2 win_s[SGD_WAVES][64];
  if (blockIdx.x == 0 && threadIdx.x == 0) flags[2] = 2;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = lane >> 4, i16 = lane & 15;
  const int xcd = blockIdx.x & 7, wg = blockIdx.x >> 3;
  const uint32_t half = i16 >= 8 ? 0u : (i16 & 1) ? 0xffff0000u : 0x0000ffffu;
  nt_u32x2* const win = win_s[wv];
  const int ns = (D.d + 127) / 128, units = D.L * ns;
  const uint32_t row_bytes = (uint32_t)D.d * 2;
  const int per_batch = nw * SGD_TOKENS;
  uint32_t step = 0;
  bool pace = true;
  uint32_t* const ctr = ctr0 + xcd * 64;
  for (int r = 0; r * 8 < units; ++r) {
    const int u = r * 8 + ((r & 1) ? 7 - xcd : xcd);
    if (u >= units) continue;
    const int lp = D.L - 1 - u / ns, c0 = (u % ns) * 128;
    const uint32_t voff = c0 + i16 * 8 < D.d ? (uint32_t)(c0 + i16 * 8) * 2u : 0x7ffffff0u;
    for (int tb = 0; tb < D.B; tb += per_batch) {
      const int t0 = tb + wv * nw + wg;      // the wavefront's tokens: t0, t0 + SGD_WAVES * nw, ...
      int cn[SGD_TPW];
#pragma unroll
      for (int i = 0; i < SGD_TPW; ++i) {
        *reinterpret_cast<float2*>(&acc_s[wv * SGD_TPW + i][lane * 2]) = make_float2(0.f, 0.f);
        const int t = t0 + i * SGD_WAVES * nw;
        cn[i] = counts[t < D.B ? t : 0];
        if (t >= D.B) cn[i] = 0;
      }
      uint32_t fn = UniformRun(idx + (size_t)t0 * stride, cn[0] * 4).load4(lane * 4u), zn = UniformRun(val + (size_t)t0 * stride, cn[0] * 4).load4(lane * 4u);
      for (int l = 0; l <= lp; ++l) {
        int cc[SGD_TPW];
        const int ln = l < lp ? l + 1 : l;
#pragma unroll
        for (int i = 0; i < SGD_TPW; ++i) {
          cc[i] = cn[i];
          const int t = t0 + i * SGD_WAVES * nw;
          cn[i] = counts[(size_t)ln * D.B + (t < D.B ? t : 0)];
          if (t >= D.B) cn[i] = 0;
        }
        {
          ++step;
          __syncthreads();
          if (threadIdx.x == 0) {
            uint32_t seen = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) + 1u;
            const uint32_t want = (step - 1u) * (uint32_t)nw;      // (the count in the low 20 bits; the polls go into the rest)
#pragma unroll 1
            for (int spin = 0; pace && (int)((seen - want) << 12) < 0; ++spin) {
              __builtin_amdgcn_s_sleep(2);
              seen = __hip_atomic_fetch_add(ctr, 1u << 20, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
              pace = spin < 400;      // (after one wait in vain -- fewer CUs, another partition -- none any more)
            }
          }
          __syncthreads();
        }
        const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<bf16_t*>(W_dec + (size_t)packed_index(l, lp, D.L) * D.F * D.d), 0, (int)((size_t)D.F * D.d * 2), 0x00020000);
#pragma unroll
        for (int i = 0; i < SGD_TPW; ++i) {
          const size_t row = (size_t)l * D.B + (t0 + i * SGD_WAVES * nw);
          const uint32_t f0 = fn, z0 = zn;
          {
            const size_t next = i + 1 < SGD_TPW ? row + SGD_WAVES * nw : (size_t)ln * D.B + t0;
            const int cnext = i + 1 < SGD_TPW ? cc[i + 1 < SGD_TPW ? i + 1 : 0] : cn[0];
            fn = UniformRun(idx + next * stride, cnext * 4).load4(lane * 4u);
            zn = UniformRun(val + next * stride, cnext * 4).load4(lane * 4u);
          }
          const int cnt = cc[i];
          if (cnt == 0) continue;
          f32x4_mfma acc = {0.f, 0.f, 0.f, 0.f};
          float* const as = &acc_s[wv * SGD_TPW + i][(4 * grp) * 8 + (i16 & 7)];
#pragma unroll
          for (int k = 0; k < 4; ++k) acc[k] = as[8 * k];
          uint32_t f = f0, zb = z0;
#pragma unroll 1
          for (int w0 = 0; w0 < cnt; w0 += 64) {
            const int n = __builtin_amdgcn_readfirstlane(min(64, cnt - w0));
            if (w0 > 0) {
              f = UniformRun(idx + row * stride + w0, n * 4).load4(lane * 4u);
              zb = UniformRun(val + row * stride + w0, n * 4).load4(lane * 4u);
            }
            wave_lds_order();
            win[lane] = nt_u32x2{lane < n ? f * row_bytes : 0x80000000u, __builtin_amdgcn_perm(zb, zb, 0x07060706u)};
            wave_lds_order();
#pragma unroll 1
            for (int j = 0; j < n; j += 16) {
              nt_u32x2 en[4];
              u32x4_lds q[4];
#pragma unroll
              for (int s4 = 0; s4 < 4; ++s4) en[s4] = win[j + 4 * s4 + grp];
#pragma unroll
              for (int s4 = 0; s4 < 4; ++s4)
                q[s4] = __builtin_bit_cast(u32x4_lds, __builtin_amdgcn_raw_buffer_load_b128(rows, (int)(en[s4][0] + voff), 0, 0));
#pragma unroll
              for (int s4 = 0; s4 < 4; ++s4) {
                const uint32_t zs = en[s4][1] & half;
                const u32x4_lds zd = {(i16 >> 1) == 0 ? zs : 0u, (i16 >> 1) == 1 ? zs : 0u, (i16 >> 1) == 2 ? zs : 0u, (i16 >> 1) == 3 ? zs : 0u};
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_mfma, q[s4]), __builtin_bit_cast(bf16x8_mfma, zd), acc, 0, 0, 0);
              }
            }
          }
          wave_lds_order();
          if (i16 < 8) {
#pragma unroll
            for (int k = 0; k < 4; ++k) as[8 * k] = acc[k];
          }
          wave_lds_order();
        }
      }
      wave_lds_order();
      const int col = c0 + lane * 2;
      if (col < D.d) {
        const float2 b = *reinterpret_cast<const float2*>(b_dec + (size_t)lp * D.d + col);
#pragma unroll
        for (int i = 0; i < SGD_TPW; ++i) {
          const int t = t0 + i * SGD_WAVES * nw;
          if (t >= D.B) break;
          float2 a = *reinterpret_cast<const float2*>(&acc_s[wv * SGD_TPW + i][lane * 2]);
          // (an infinity or a NaN in one weight reaches the sums of the other seven columns of its run through the zeros beside
          //  z: where a sum is not finite the token's columns are summed up one by one)
          if (__builtin_amdgcn_ballot_w64(!(fabsf(a.x) + fabsf(a.y) < __builtin_inff()))) {
            a = make_float2(0.f, 0.f);
            for (int l = 0; l <= lp; ++l) {
              const size_t row = (size_t)l * D.B + t;
              const bf16_t* w = W_dec + (size_t)packed_index(l, lp, D.L) * D.F * D.d + col;
              for (int e = 0; e < counts[row]; ++e) {
                const uint32_t w2 = *reinterpret_cast<const uint32_t*>(w + (size_t)idx[row * stride + e] * D.d);
                const float z = val[row * stride + e];
                a = make_float2(fmaf(z, __uint_as_float(w2 << 16), a.x), fmaf(z, __uint_as_float(w2 & 0xffff0000u), a.y));
              }
            }
          }
          *reinterpret_cast<float2*>(y_hat + ((size_t)lp * D.B + t) * D.d + col) = make_float2(a.x + b.x, a.y + b.y);
        }
      }
      wave_lds_order();
    }
  }
}

// ---------------------------------------------------------------------------
// Sparse backward
// ---------------------------------------------------------------------------
template <typename T> struct Row8;      // 8 consecutive elements of a row as floats
template <> struct Row8<bf16_t> {
  static __device__ __forceinline__ void load(const bf16_t* p, float (&o)[8]) {
    const uint4 u = *reinterpret_cast<const uint4*>(p);
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) { o[2 * i] = __uint_as_float(w[i] << 16); o[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u); }
  }
};
template <> struct Row8<float> {
  static __device__ __forceinline__ void load(const float* p, float (&o)[8]) {
    const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
    o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w; o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
  }
};

// dpre := 0 (or the dead-feature gradient below the threshold); the listed entries are overwritten by gather_dz.
template <typename T>
__global__ __launch_bounds__(256) void sparse_dpre_fill_kernel(Dims D, const uint8_t* __restrict__ cls,
                                                               const float* __restrict__ norms, float lam1_over_b,
                                                               T* __restrict__ dpre, const int32_t* __restrict__ flags,
                                                               int kcap) {
  if (!lists_backward_selected(flags, kcap)) return;
  const size_t n4 = (size_t)D.L * D.B * D.F / 4, per_layer4 = (size_t)D.B * D.F / 4;
  const int F4 = D.F / 4;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (size_t)gridDim.x * 256) {
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
    if (lam1_over_b != 0.f) {
      const uint32_t c4 = *reinterpret_cast<const uint32_t*>(cls + i * 4);
      if (c4 & 0x04040404u) {
        const int l = (int)(i / per_layer4), f = (int)(i % F4) * 4;
        const float4 n = *reinterpret_cast<const float4*>(norms + (size_t)l * D.F + f);
        o = make_float4((c4 & 0x4u) ? -lam1_over_b * n.x : 0.f, (c4 & 0x400u) ? -lam1_over_b * n.y : 0.f,
                        (c4 & 0x40000u) ? -lam1_over_b * n.z : 0.f, (c4 & 0x4000000u) ? -lam1_over_b * n.w : 0.f);
      }
    }
    Elem<T>::store4(dpre + i * 4, o);
  }
}

// One wavefront per listed entry: for each target l' >= l it streams the entry's decoder row and
// the token's d y_hat row (64 lanes x 8 columns, 4 passes in flight), keeps one partial dot
// product per lane and reduces over the wave at the end.  No workgroup barrier, few registers
// (93 registers with bf16 storage: five waves per SIMD), so many independent latency chains overlap.  A row's entries are dealt
// to GDZ_PARTS workgroups of 4 waves, so that the few very long rows of a heavy-tailed batch do
// not serialise on one workgroup.
constexpr int GDZ_PARTS = 8;
template <typename T>
__global__ __launch_bounds__(256) void gather_dz_kernel(Dims D, GatherLists g, const T* __restrict__ d_yhat,
                                                        const T* __restrict__ W_dec, const float* __restrict__ norms,
                                                        float lam_c_over_b, float C, T* __restrict__ dpre,
                                                        const int32_t* __restrict__ flags, FeatureLists fused) {
  if (!lists_backward_selected(flags, g.kcap) || fused_dz_selected(flags, fused)) return;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long items = ((long)D.L * D.B + 7) / 8 * 8 * GDZ_PARTS;
  for (long it = blockIdx.x; it < items; it += gridDim.x) {      // layer 0 (most targets) first
    // items in groups of 8 rows x GDZ_PARTS parts, the row index fastest: workgroups go round-robin
    // to the 8 XCDs, so all parts of a row run on one XCD and share its L2
    const long grp = it / (8 * GDZ_PARTS);
    const int within = (int)(it % (8 * GDZ_PARTS));
    const long row = grp * 8 + (within & 7);
    const int part = within >> 3;
    if (row >= (long)D.L * D.B) continue;
    const int l = (int)(row / D.B), b = (int)(row % D.B);
    const int na = g.counts[row], n = na + g.counts_w[row];
    const int32_t* ii = g.idx + (size_t)row * g.stride;
    const float* vv = g.val + (size_t)row * g.stride;
    for (int e = part * 4 + wv; e < n; e += 4 * GDZ_PARTS) {
      const int slot = e < na ? e : g.kcap - 1 - (e - na);      // front: active entries, back: window-only
      const int fe = __builtin_amdgcn_readfirstlane(ii[slot]);
      float part_sum = 0.f;
      // the loads of two targets are in flight together
      auto targets = [&](auto nt_tag, int lp) {
        constexpr int NTG = decltype(nt_tag)::value;
        for (int c0 = 0; c0 < D.d; c0 += 2048) {
          typename Raw8<T>::type dy[NTG][4], wq[NTG][4];
#pragma unroll
          for (int t = 0; t < NTG; ++t) {
            const T* dyr = d_yhat + ((size_t)(lp + t) * D.B + b) * D.d;
            const T* wr = W_dec + ((size_t)packed_index(l, lp + t, D.L) * D.F + fe) * D.d;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const uint32_t col = (uint32_t)(c0 + q * 512 + lane * 8);
              if ((int)col < D.d) { dy[t][q] = Raw8<T>::load(lane_ptr(dyr, col)); wq[t][q] = Raw8<T>::load(lane_ptr(wr, col)); }
            }
          }
#pragma unroll
          for (int t = 0; t < NTG; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const uint32_t col = (uint32_t)(c0 + q * 512 + lane * 8);
              if ((int)col < D.d) part_sum = Raw8<T>::dot(wq[t][q], dy[t][q], part_sum);
            }
        }
      };
      int lp = l;
      for (; lp + 2 <= D.L; lp += 2) targets(std::integral_constant<int, 2>{}, lp);
      if (lp < D.L) targets(std::integral_constant<int, 1>{}, lp);
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) part_sum += __shfl_xor(part_sum, off, 64);
      if (lane == 0) {
        const float zv = vv[slot];
        const float nn = norms[(size_t)l * D.F + fe];
        const float ex = __builtin_amdgcn_exp2f(-2.0f * 1.4426950408889634f * C * nn * fabsf(zv));
        const float sden = 1.0f + ex;
        const float gsp = 4.0f * lam_c_over_b * nn * ex * __builtin_amdgcn_rcpf(sden * sden);
        Elem<T>::store(dpre + (size_t)row * D.F + fe, part_sum + gsp);
      }
    }
  }
}

// The same entries with the token's d y_hat rows staged in LDS: one workgroup of 16 waves per (layer, token) row,
// the rows of up to `tcap` targets (at most 64 KB) are copied to LDS once and every wave streams the decoder rows
// of its entries (four per batch of 64) against them, two targets' rows in flight.  Only decoder rows are left on the
// vector-memory path (d y_hat is fetched once per row instead of once per entry), and 64 registers allow eight waves
// per SIMD.  Launched with one workgroup per row, so long and short rows are balanced by the dispatcher; this is the
// kernel the library uses whenever a row of d y_hat fits LDS, gather_dz_kernel above is the fallback.
template <typename T> struct Raw8Lds;
template <> struct Raw8Lds<bf16_t> {
  static __device__ __forceinline__ Raw8<bf16_t>::type load(const bf16_t* p) { return *reinterpret_cast<const uint4*>(p); }
};
template <> struct Raw8Lds<float> {
  static __device__ __forceinline__ Raw8<float>::type load(const float* p) {
    return Raw8<float>::type{*reinterpret_cast<const float4*>(p), *reinterpret_cast<const float4*>(p + 4)};
  }
};
template <typename T>
__global__ __launch_bounds__(1024, 2) void gather_dz_lds_kernel(Dims D, GatherLists g, const T* __restrict__ d_yhat,
                                                                const T* __restrict__ W_dec,
                                                                const float* __restrict__ norms, float lam_c_over_b,
                                                                float C, T* __restrict__ dpre,
                                                                const int32_t* __restrict__ flags, int tcap,
                                                                FeatureLists fused) {
  extern __shared__ __align__(16) unsigned char gdz_smem[];
  T* dys = reinterpret_cast<T*>(gdz_smem);      // [tcap][d]
  if (!lists_backward_selected(flags, g.kcap) || fused_dz_selected(flags, fused)) return;
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int PIECE = 16 / (int)sizeof(T);      // elements per 16-byte piece
  const int ppr = D.d / PIECE;                    // pieces per row
  const long rows = (long)D.L * D.B;
  for (long row = blockIdx.x; row < rows; row += gridDim.x) {      // layer 0 (most targets) first
    const int l = (int)(row / D.B), b = (int)(row % D.B);
    const int na = g.counts[row], n = na + g.counts_w[row];
    const int32_t* ii = g.idx + (size_t)row * g.stride;
    const float* vv = g.val + (size_t)row * g.stride;
    for (int e0 = 0; e0 < n; e0 += 64) {
      float sum[4] = {0.f, 0.f, 0.f, 0.f};
      int slot[4], fe[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = e0 + u * 16 + wv;
        const int ec = e < n ? e : e0;                               // (a valid slot; nothing is computed or stored for it)
        slot[u] = ec < na ? ec : g.kcap - 1 - (ec - na);             // front: active entries, back: window-only
        fe[u] = __builtin_amdgcn_readfirstlane(ii[slot[u]]);
      }
      for (int lp0 = l; lp0 < D.L; lp0 += tcap) {
        const int tc = min(tcap, D.L - lp0);
        __syncthreads();                                             // the previous chunk's rows are no longer read
        for (int i = tid; i < tc * ppr; i += 1024) {
          const int t = i / ppr, c = (i - t * ppr) * PIECE;
          *reinterpret_cast<uint4*>(dys + (size_t)t * D.d + c) =
              *reinterpret_cast<const uint4*>(d_yhat + ((size_t)(lp0 + t) * D.B + b) * D.d + c);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (e0 + u * 16 + wv >= n) continue;                       // wave-uniform
          float ps = sum[u];
          const T* wrow0 = W_dec + ((size_t)packed_index(l, lp0, D.L) * D.F + fe[u]) * D.d;
          const size_t blk = (size_t)D.F * D.d;
          for (int t = 0; t < tc; t += 2) {
            const bool two = t + 1 < tc;
            for (int c0 = 0; c0 < D.d; c0 += 2048) {
              typename Raw8<T>::type wq[2][4];
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const uint32_t col = (uint32_t)(c0 + q * 512 + lane * 8);
                if ((int)col < D.d) {
                  wq[0][q] = Raw8<T>::load(lane_ptr(wrow0 + (size_t)t * blk, col));
                  wq[1][q] = Raw8<T>::load(lane_ptr(wrow0 + (size_t)(two ? t + 1 : t) * blk, col));
                }
              }
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const uint32_t col = (uint32_t)(c0 + q * 512 + lane * 8);
                if ((int)col < D.d) {
                  ps = Raw8<T>::dot(wq[0][q], Raw8Lds<T>::load(dys + (size_t)t * D.d + col), ps);
                  if (two) ps = Raw8<T>::dot(wq[1][q], Raw8Lds<T>::load(dys + (size_t)(t + 1) * D.d + col), ps);
                }
              }
            }
          }
          sum[u] = ps;
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (e0 + u * 16 + wv >= n) continue;
        float ps = sum[u];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) ps += __shfl_xor(ps, off, 64);
        if (lane == 0) {
          const float zv = vv[slot[u]];
          const float nn = norms[(size_t)l * D.F + fe[u]];
          const float ex = __builtin_amdgcn_exp2f(-2.0f * 1.4426950408889634f * C * nn * fabsf(zv));
          const float sden = 1.0f + ex;
          const float gsp = 4.0f * lam_c_over_b * nn * ex * __builtin_amdgcn_rcpf(sden * sden);
          Elem<T>::store(dpre + (size_t)row * D.F + fe[u], ps + gsp);
        }
      }
    }
  }
}

// ---- feature lists: column scan of the class bytes in FL_SEGS token segments ----
// Each thread owns 8 consecutive features of one layer and one token segment (F is a multiple of 8), the class bytes of
// eight tokens in flight.
__global__ __launch_bounds__(256) void fl_count_kernel(Dims D, const uint8_t* __restrict__ cls, FeatureLists fl,
                                                       const int32_t* __restrict__ flags) {
  if (!lists_backward_selected(flags, fl.kcap)) return;
  const int LF8 = D.L * D.F / 8;
  const int q = blockIdx.x * 256 + threadIdx.x, sgm = blockIdx.y;
  if (q >= LF8) return;
  const int l = (q * 8) / D.F, f = (q * 8) % D.F;
  const int seg_len = (D.B + FL_SEGS - 1) / FL_SEGS;
  const int b0 = sgm * seg_len, b1 = min(D.B, b0 + seg_len);
  int c[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll 8
  for (int b = b0; b < b1; ++b) {
    const uint2 a8 = *reinterpret_cast<const uint2*>(cls + ((size_t)l * D.B + b) * D.F + f);
    const uint32_t lo = (a8.x | (a8.x >> 1)) & 0x01010101u, hi = (a8.y | (a8.y >> 1)) & 0x01010101u;      // active, or inside the threshold window
#pragma unroll
    for (int i = 0; i < 4; ++i) { c[i] += (int)((lo >> (8 * i)) & 1u); c[4 + i] += (int)((hi >> (8 * i)) & 1u); }
  }
  int4* o = reinterpret_cast<int4*>(fl.seg + (size_t)sgm * D.L * D.F + (size_t)q * 8);
  o[0] = make_int4(c[0], c[1], c[2], c[3]);
  o[1] = make_int4(c[4], c[5], c[6], c[7]);
}

// One workgroup of 1024 lanes per layer: layer-local exclusive scan over the features of the summed segment counts; the
// segment counts are turned into each segment's first slot.  The lanes take 1024 consecutive features at a time, so that
// every access is one run of memory (a lane with a run of 8 features of its own: 152 us at 16 x 8192 features, each access of
// a wavefront spread over 2 KB).
constexpr int FL_SCAN_THREADS = 1024;
__global__ __launch_bounds__(FL_SCAN_THREADS) void fl_scan_kernel(Dims D, FeatureLists fl,
                                                                  int32_t* __restrict__ flags, int dense_beyond) {
  if (!lists_backward_selected(flags, fl.kcap)) return;
  constexpr int WAVES = FL_SCAN_THREADS / 64;
  __shared__ int wtot[WAVES];
  const int l = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const size_t LF = (size_t)D.L * D.F;
  int run = 0;      // entries of the features before this chunk
  for (int f0 = 0; f0 < D.F; f0 += FL_SCAN_THREADS) {
    const int f = f0 + threadIdx.x;
    const bool in = f < D.F;
    const size_t lf = (size_t)l * D.F + (in ? f : 0);
    int v[FL_SEGS], c = 0;
#pragma unroll
    for (int sgm = 0; sgm < FL_SEGS; ++sgm) v[sgm] = in ? fl.seg[(size_t)sgm * LF + lf] : 0;
#pragma unroll
    for (int sgm = 0; sgm < FL_SEGS; ++sgm) c += v[sgm];
    int incl = c;      // inclusive scan over the wavefront
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int u = __shfl_up(incl, off, 64);
      if (lane >= off) incl += u;
    }
    if (lane == 63) wtot[w] = incl;
    __syncthreads();
    int before = run, total = 0;
#pragma unroll
    for (int q = 0; q < WAVES; ++q) {
      if (q < w) before += wtot[q];
      total += wtot[q];
    }
    __syncthreads();      // the next chunk writes wtot again
    if (in) {
      int pos = before + incl - c;
      fl.off[lf] = pos;
      fl.cnt[lf] = c;
#pragma unroll
      for (int sgm = 0; sgm < FL_SEGS; ++sgm) {
        fl.seg[(size_t)sgm * LF + lf] = pos;
        pos += v[sgm];
      }
    }
    run += total;
  }
  if (threadIdx.x == 0) {
    atomicMax(&flags[3], run);      // the longest layer decides whether the fused dz has room
    // Automatic mode: lists too long for the fused dz are long enough for the dense kernels to win, so the backward
    // is handed back to them (they run after this kernel and look at the same bit; so do the list kernels).
    if (dense_beyond > 0 && run > dense_beyond) atomicAnd(&flags[0], ~2);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void fl_fill_kernel(Dims D, const uint8_t* __restrict__ cls, const T* __restrict__ z,
                                                      FeatureLists fl, const int32_t* __restrict__ flags) {
  if (!lists_backward_selected(flags, fl.kcap)) return;
  const int LF4 = D.L * D.F / 4;
  const int q = blockIdx.x * 256 + threadIdx.x, sgm = blockIdx.y;
  if (q >= LF4) return;
  const int l = (q * 4) / D.F, f = (q * 4) % D.F;
  const int seg_len = (D.B + FL_SEGS - 1) / FL_SEGS;
  const int b0 = sgm * seg_len, b1 = min(D.B, b0 + seg_len);
  const int32_t* so = fl.seg + (size_t)sgm * D.L * D.F + (size_t)q * 4;
  int pos[4] = {so[0], so[1], so[2], so[3]};
  const size_t base = (size_t)l * D.B * fl.kcap;        // layer l's region of the lists
  for (int bb = b0; bb < b1; bb += 8) {      // the class words of eight tokens in flight, then the (few) listed entries
    uint32_t c8[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      c8[u] = bb + u < b1 ? *reinterpret_cast<const uint32_t*>(cls + ((size_t)l * D.B + bb + u) * D.F + f) : 0u;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint32_t a4 = (c8[u] | (c8[u] >> 1)) & 0x01010101u;      // as counted: active or in the window (z = 0 there)
      if (!a4) continue;
      const int b = bb + u;
      const float4 z4 = Elem<T>::load4(z + ((size_t)l * D.B + b) * D.F + f);
      const float zz[4] = {z4.x, z4.y, z4.z, z4.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if ((a4 >> (8 * i)) & 1u) {
          fl.tok[base + pos[i]] = b;
          // (bf16 storage: the class travels in the low bits that a bf16 value leaves free)
          fl.val[base + pos[i]] = sizeof(T) == 2 ? __uint_as_float(__float_as_uint(zz[i]) | ((c8[u] >> (8 * i)) & 3u)) : zz[i];
          ++pos[i];
        }
    }
  }
}

// z of a feature-list entry (see fl_fill_kernel)
template <typename T> __device__ __forceinline__ float list_z(float v) {
  return sizeof(T) == 2 ? __uint_as_float(__float_as_uint(v) & 0xffff0000u) : v;
}

// One item = (layer l, feature f, pair of targets): a workgroup of 256 lanes, 8 columns each,
// requests the rows' weights and optimizer state, sums z * d y_hat rows over the feature's tokens (four tokens in
// flight) meanwhile, then finishes the row of both targets: norm term, optional gradient store, optional Adam update.  Most rows of a
// sparse step have no token at all and only stream their optimizer state.  Token indices and
// values are wave-uniform, so every address is a scalar base plus the lane's fixed column offset.
constexpr int SD_TCH = 2;

template <typename T, int NT, bool MASTER>
__device__ __forceinline__ void sparse_dwdec_rows(const Dims& D, int l, int f, int lp0, int cnt,
                                                  const int32_t* __restrict__ tk, const float* __restrict__ tv,
                                                  float coef, const T* __restrict__ d_yhat, T* __restrict__ W_dec,
                                                  T* __restrict__ dW_dec, const AdamFuseArgs& fuse, uint32_t col,
                                                  bool ok1, float* __restrict__ n2_part, int n2_slots, int n2_slot0) {
  // the lane owns columns col..col+3 and, when ok1, col+1024..col+1027: every access of the
  // workgroup is one contiguous run of 256 x 4 elements.
  // The rows' weights and optimizer state are requested first: they come from HBM and do not depend on the
  // token lists, so their latency lies under the gathering of the d y_hat rows below.
  // (native vector types: selects on the float4 class type would go through scratch memory)
  typename Elem<T>::Raw4 wr[NT][2];
  nt_f32x4 m4[NT][2], v4[NT][2], p4[NT][2];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const size_t o = ((size_t)packed_index(l, lp0 + t, D.L) * D.F + f) * D.d;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      m4[t][h] = v4[t][h] = p4[t][h] = nt_f32x4{0.f, 0.f, 0.f, 0.f};
      wr[t][h] = Elem<T>::narrow4(make_float4(0.f, 0.f, 0.f, 0.f));
      if (h == 1 && !ok1) continue;
      const uint32_t ch = col + 1024 * h;
      wr[t][h] = Elem<T>::load_raw4(lane_ptr(W_dec + o, ch));
      if (fuse.m) {
        m4[t][h] = *reinterpret_cast<const nt_f32x4*>(lane_ptr(fuse.m + o, ch));
        v4[t][h] = *reinterpret_cast<const nt_f32x4*>(lane_ptr(fuse.v + o, ch));
        if (MASTER) p4[t][h] = *reinterpret_cast<const nt_f32x4*>(lane_ptr(fuse.master + o, ch));
      }
    }
  }
  float acc[NT][2][4];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[t][h][k] = 0.f;
  int j = 0;
  for (; j + 4 <= cnt; j += 4) {
    // (the gathered rows stay in their storage type until they are used: half the registers for bf16)
    typename Elem<T>::Raw4 r[4][NT][2];
    float zv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int b = __builtin_amdgcn_readfirstlane(tk[j + u]);
      zv[u] = list_z<T>(__int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(tv[j + u]))));
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const T* row = d_yhat + ((size_t)(lp0 + t) * D.B + b) * D.d;
        r[u][t][0] = Elem<T>::load_raw4(lane_ptr(row, col));
        r[u][t][1] = Elem<T>::load_raw4(lane_ptr(row, ok1 ? col + 1024 : col));
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const float4 q = Elem<T>::widen4(r[u][t][h]);
          acc[t][h][0] = fmaf(zv[u], q.x, acc[t][h][0]);
          acc[t][h][1] = fmaf(zv[u], q.y, acc[t][h][1]);
          acc[t][h][2] = fmaf(zv[u], q.z, acc[t][h][2]);
          acc[t][h][3] = fmaf(zv[u], q.w, acc[t][h][3]);
        }
  }
  for (; j < cnt; ++j) {
    const int b = __builtin_amdgcn_readfirstlane(tk[j]);
    const float zv = list_z<T>(__int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(tv[j]))));
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const T* row = d_yhat + ((size_t)(lp0 + t) * D.B + b) * D.d;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (h == 1 && !ok1) continue;
        const float4 r = Elem<T>::load4(lane_ptr(row, col + 1024 * h));
        acc[t][h][0] = fmaf(zv, r.x, acc[t][h][0]);
        acc[t][h][1] = fmaf(zv, r.y, acc[t][h][1]);
        acc[t][h][2] = fmaf(zv, r.z, acc[t][h][2]);
        acc[t][h][3] = fmaf(zv, r.w, acc[t][h][3]);
      }
    }
  }
  nt_f32x4 w[NT][2];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float4 wl = Elem<T>::widen4(wr[t][h]);
      w[t][h] = nt_f32x4{wl.x, wl.y, wl.z, wl.w};
      if (!MASTER) p4[t][h] = w[t][h];
    }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const size_t o = ((size_t)packed_index(l, lp0 + t, D.L) * D.F + f) * D.d;
    float n2_half[2] = {0.f, 0.f};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (h == 1 && !ok1) continue;
      const uint32_t ch = col + 1024 * h;
      const nt_f32x4 wq = w[t][h];
      const float g4[4] = {fmaf(coef, wq[0], acc[t][h][0]), fmaf(coef, wq[1], acc[t][h][1]),
                           fmaf(coef, wq[2], acc[t][h][2]), fmaf(coef, wq[3], acc[t][h][3])};
      if (dW_dec) Elem<T>::store4(lane_ptr(dW_dec + o, ch), make_float4(g4[0], g4[1], g4[2], g4[3]));
      if (fuse.m) {
        float mm[4] = {m4[t][h][0], m4[t][h][1], m4[t][h][2], m4[t][h][3]};
        float vv[4] = {v4[t][h][0], v4[t][h][1], v4[t][h][2], v4[t][h][3]};
        float pp[4] = {p4[t][h][0], p4[t][h][1], p4[t][h][2], p4[t][h][3]};
#pragma unroll
        for (int k = 0; k < 4; ++k) adam_element(pp[k], mm[k], vv[k], g4[k], fuse.a);
        *reinterpret_cast<float4*>(lane_ptr(fuse.m + o, ch)) = make_float4(mm[0], mm[1], mm[2], mm[3]);
        *reinterpret_cast<float4*>(lane_ptr(fuse.v + o, ch)) = make_float4(vv[0], vv[1], vv[2], vv[3]);
        const float4 pn = make_float4(pp[0], pp[1], pp[2], pp[3]);
        if (MASTER) *reinterpret_cast<float4*>(lane_ptr(fuse.master + o, ch)) = pn;
        const typename Elem<T>::Raw4 stored = Elem<T>::narrow4(pn);
        *reinterpret_cast<typename Elem<T>::Raw4*>(lane_ptr(W_dec + o, ch)) = stored;
        if (n2_part) {   // sum of squares of the wave's 256 weights as stored, for the next step's norms: one slot per wave and half
          const float4 wn = Elem<T>::widen4(stored);
          const int b16 = __float_as_int(row16_sum((wn.x * wn.x + wn.y * wn.y) + (wn.z * wn.z + wn.w * wn.w)));
          n2_half[h] = (__int_as_float(__builtin_amdgcn_readlane(b16, 0)) + __int_as_float(__builtin_amdgcn_readlane(b16, 16))) +
                       (__int_as_float(__builtin_amdgcn_readlane(b16, 32)) + __int_as_float(__builtin_amdgcn_readlane(b16, 48)));
        }
      }
    }
    if (n2_part && fuse.m && (threadIdx.x & 63) == 0)     // both halves of the wave's slot pair at once
      *reinterpret_cast<float2*>(n2_part + ((size_t)packed_index(l, lp0 + t, D.L) * D.F + f) * n2_slots + n2_slot0) =
          make_float2(n2_half[0], n2_half[1]);
  }
}

// MASTER: fp32 master weights travel with the moments (compile-time: their 16 registers are not held otherwise)
template <typename T, bool MASTER>
__global__ __launch_bounds__(256, 4) void sparse_dwdec_kernel(Dims D, FeatureLists fl, const T* __restrict__ d_yhat,
                                                           T* __restrict__ W_dec, const float* __restrict__ G,
                                                           const float* __restrict__ norms, T* __restrict__ dW_dec,
                                                           AdamFuseArgs fuse, const int32_t* __restrict__ flags,
                                                           float* __restrict__ n2_part) {
  if (!lists_backward_selected(flags, fl.kcap)) return;
  const int tid = threadIdx.x;
  const int chunks = (D.L + SD_TCH - 1) / SD_TCH;          // chunk slots per (l, f); those past L - l are empty
  const long items = (long)D.L * D.F * chunks;
  // what an item needs before its rows can be touched; fetched one item ahead
  struct Meta { int l, f, lp0, cnt, off; float Gf, nf; };
  auto fetch_meta = [&](long it) {
    Meta mt;
    // order (l, target pair, f): the workgroups in flight walk a few long contiguous row ranges
    mt.f = (int)(it % D.F);
    const long lc = it / D.F;
    const int c = (int)(lc % chunks);
    mt.l = (int)(lc / chunks);
    const long lf = (long)mt.l * D.F + mt.f;
    mt.lp0 = mt.l + c * SD_TCH;
    mt.cnt = 0; mt.off = 0; mt.Gf = 0.f; mt.nf = 1.f;
    if (mt.lp0 < D.L) { mt.cnt = fl.cnt[lf]; mt.off = fl.off[lf]; mt.Gf = G[lf]; mt.nf = norms[lf]; }
    return mt;
  };
  long it = blockIdx.x;
  if (it >= items) return;
  Meta cur = fetch_meta(it);
  for (; it < items; it += gridDim.x) {
    const long nx = it + gridDim.x;
    Meta nxt = cur;
    if (nx < items) nxt = fetch_meta(nx);
    if (cur.lp0 < D.L) {
      const int32_t* tk = fl.tok + (size_t)cur.l * D.B * fl.kcap + cur.off;
      const float* tv = fl.val + (size_t)cur.l * D.B * fl.kcap + cur.off;
      const float coef = cur.Gf * __builtin_amdgcn_rcpf(fmaxf(cur.nf, 1e-30f));
      // row sums of squares of the updated weights (n2_part, d a multiple of 256): [P][F][8 slots per 2048 columns],
      // slot = (wave, half) of the lanes that own the columns; slots whose columns do not exist hold zero
      const int n2_slots = 8 * ((D.d + 2047) / 2048);
      for (int c0 = 0; c0 < D.d; c0 += 2048) {
        const int col = c0 + tid * 4;
        const bool ok1 = col + 1024 < D.d;
        const int slot0 = (c0 >> 11) * 8 + (tid >> 6) * 2;
        if (n2_part && (tid & 63) == 0) {
          const int nt = cur.lp0 + 1 < D.L ? 2 : 1;
          for (int t = 0; t < nt; ++t) {
            float* q = n2_part + ((size_t)packed_index(cur.l, cur.lp0 + t, D.L) * D.F + cur.f) * n2_slots + slot0;
            if (col >= D.d) { q[0] = 0.f; q[1] = 0.f; }
          }
        }
        if (col >= D.d) continue;
        if (cur.lp0 + 1 < D.L)
          sparse_dwdec_rows<T, 2, MASTER>(D, cur.l, cur.f, cur.lp0, cur.cnt, tk, tv, coef, d_yhat, W_dec, dW_dec, fuse,
                                  (uint32_t)col, ok1, n2_part, n2_slots, slot0);
        else
          sparse_dwdec_rows<T, 1, MASTER>(D, cur.l, cur.f, cur.lp0, cur.cnt, tk, tv, coef, d_yhat, W_dec, dW_dec, fuse,
                                  (uint32_t)col, ok1, n2_part, n2_slots, slot0);
      }
    }
    cur = nxt;
  }
}

// Sums of four values over the wave at once: on return the lanes with lane % 4 == u hold the sum of the u-th value.
// Two exchange steps inside quads halve the values each lane carries, two rotations finish the rows of 16 lanes,
// two shuffles the four rows.
__device__ __forceinline__ float wave_sum4(float a, float b, float c, float d, int lane, int addr16, int addr32) {
  const bool o1 = lane & 1, o2 = lane & 2;
  const float r1 = (o1 ? b : a) + dpp_move<0xB1>(o1 ? a : b);      // even lanes: a of the pair, odd lanes: b
  const float r2 = (o1 ? d : c) + dpp_move<0xB1>(o1 ? c : d);
  float r = (o2 ? r2 : r1) + dpp_move<0x4E>(o2 ? r1 : r2);         // lane % 4 = 0, 1, 2, 3: a, b, c, d of the quad
  r += dpp_move<0x128>(r);                                          // row_ror:8
  r += dpp_move<0x124>(r);                                          // row_ror:4
  // (addr16 / addr32: byte addresses of lanes lane ^ 16 and lane ^ 32, computed once by the caller)
  r += __int_as_float(__builtin_amdgcn_ds_bpermute(addr16, __float_as_int(r)));
  r += __int_as_float(__builtin_amdgcn_ds_bpermute(addr32, __float_as_int(r)));
  return r;
}

// bf16 pairs as the dot-product instruction takes them
typedef __bf16 bf16x2_hw __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_hw, a), __builtin_bit_cast(bf16x2_hw, b), c, false);
}

// The same rows cut into eight column slices, one per XCD (workgroups go round-robin to the XCDs, so blockIdx & 7
// names the slice): an XCD's L2 then only ever sees its d/8 columns of d y_hat, and with the (source, target) pairs
// walked target-major that is B * d/8 elements at a time (2 MB of bf16 at L=16 d=2048 B=4096), so the gathered d y_hat rows
// come out of the L2.  One wave per (pair, feature, slice), four consecutive features per workgroup.  The weights and optimizer
// state, touched once, are streamed with non-temporal accesses so that they do not displace the slice (plain accesses: 10 %
// slower).  The sums run over the feature's tokens in list order.
// fp32 storage: lanes own 4 columns per pass of 256; sums exactly as in the kernel above (same gradient and update, bit for
// bit).  Used whenever d is a multiple of 32.
constexpr int SD_ITEMS_PER_WG = 2;
template <bool MASTER>
__global__ __launch_bounds__(256, MASTER ? 5 : 6) void sparse_dwdec_sliced_kernel(Dims D, FeatureLists fl, const float* __restrict__ d_yhat,
                                                                     float* __restrict__ W_dec, const float* __restrict__ G,
                                                                     const float* __restrict__ norms, float* __restrict__ dW_dec,
                                                                     AdamFuseArgs fuse, const int32_t* __restrict__ flags,
                                                                     const int32_t* __restrict__ fl_tok,
                                                                     const float* __restrict__ fl_val) {
  typedef float T;
  // (fl_tok, fl_val: fl.tok and fl.val once more, as parameters of their own that nothing else aliases: the wave-uniform
  //  reads of the token lists can then go through the scalar unit)
  if (!lists_backward_selected(flags, fl.kcap)) return;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int addr16 = (lane ^ 16) << 2, addr32 = (lane ^ 32) << 2;
  const int slice = blockIdx.x & 7, wg = blockIdx.x >> 3, nwg = gridDim.x >> 3;      // (the grid is a multiple of 8)
  const int sw = D.d / 8, q4 = sw / 4;                     // slice width in columns and in lane quads (d % 32 == 0)
  const int passes = (q4 + 63) / 64;
  const int F4 = (D.F + 3) / 4;
  const long items = (long)(D.L * (D.L + 1) / 2) * F4;
  const bool dz_on = fused_dz_selected(flags, fl);
  struct Meta { int l, lp, f, cnt, off; float Gf, nf; };
  // (SD_ITEMS_PER_WG consecutive items per workgroup as long as the grid allows it: handed out in order by the
  //  dispatcher, the workgroups in flight stay within a narrow window of items, which is what keeps their d y_hat rows
  //  in the L2; more than one item, so that a launch that stands down costs fewer empty workgroups)
  for (long itb = (long)wg * SD_ITEMS_PER_WG; itb < items; itb += (long)nwg * SD_ITEMS_PER_WG)
  for (long it = itb; it < itb + SD_ITEMS_PER_WG && it < items; ++it) {
    Meta cur;
    const int pq = (int)(it / F4);                         // pair ordinal, target-major: (0,0) (0,1) (1,1) (0,2) ...
    cur.f = (int)(it % F4) * 4 + wv;
    int lpq = (int)((__builtin_amdgcn_sqrtf(8.0f * (float)pq + 1.0f) - 1.0f) * 0.5f);
    while ((lpq + 1) * (lpq + 2) / 2 <= pq) ++lpq;
    while (lpq * (lpq + 1) / 2 > pq) --lpq;
    cur.lp = lpq;
    cur.l = pq - lpq * (lpq + 1) / 2;
    if (cur.f < D.F) {
      const long lf = (long)cur.l * D.F + cur.f;
      cur.cnt = fl.cnt[lf]; cur.off = fl.off[lf]; cur.Gf = G[lf]; cur.nf = norms[lf];
      const int32_t* tk = fl_tok + (size_t)cur.l * D.B * fl.kcap + cur.off;
      const float* tv = fl_val + (size_t)cur.l * D.B * fl.kcap + cur.off;
      const float coef = cur.Gf * __builtin_amdgcn_rcpf(fmaxf(cur.nf, 1e-30f));
      const size_t o = ((size_t)packed_index(cur.l, cur.lp, D.L) * D.F + cur.f) * D.d;
      const T* dyt = d_yhat + (size_t)cur.lp * D.B * D.d;
      float* dz_out = dz_on ? fl.dz_part + ((size_t)packed_index(cur.l, cur.lp, D.L) * 8 + slice) * fl.ecap + cur.off : nullptr;
      for (int ps = 0; ps < passes; ++ps) {
        const int qd = ps * 64 + lane;
        const bool on = qd < q4;
        const uint32_t col = (uint32_t)(slice * sw + (on ? qd : 0) * 4);      // (idle lanes shadow quad 0, store nothing)
        typename Elem<T>::Raw4 wr;
        nt_f32x4 m4 = {0.f, 0.f, 0.f, 0.f}, v4 = m4, p4 = m4;
        wr = Elem<T>::nt_load_raw4(lane_ptr(W_dec + o, col));
        if (fuse.m) {
          m4 = nt_load_v4(lane_ptr(fuse.m + o, col));
          v4 = nt_load_v4(lane_ptr(fuse.v + o, col));
          if (MASTER) p4 = nt_load_v4(lane_ptr(fuse.master + o, col));
        }
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        // Fused dz: the token's d y_hat columns are in registers anyway, so their dot product with the row's weights
        // (before the update) costs four multiply-adds per lane and, for four tokens at a time, one sum over the
        // wave; lane t % 64 keeps token t's sum and the wave stores 64 of them at a time, one slot per
        // (pair, slice, entry).
        float dz_keep = 0.f;
        const float4 wl = Elem<T>::widen4(wr);
        auto dz_group = [&](int j0, int nval, const float (&pd)[4]) {      // tokens j0 .. j0 + nval - 1, j0 % 4 == 0
          const float r = wave_sum4(pd[0], pd[1], pd[2], pd[3], lane, addr16, addr32);
          if ((lane & 60) == (j0 & 63)) dz_keep = r;
          const int last = j0 + nval - 1;
          if ((last & 63) == 63 || last == cur.cnt - 1) {
            if (lane <= (last & 63)) {
              float* slot = dz_out + (last & ~63) + lane;
              *slot = ps == 0 ? dz_keep : *slot + dz_keep;      // (a slice wider than 256 columns: one pass after the other)
            }
          }
        };
        {
          const float4 wz = on ? wl : make_float4(0.f, 0.f, 0.f, 0.f);
          int j = 0;
          for (; j + 4 <= cur.cnt; j += 4) {
            typename Elem<T>::Raw4 r[4];
            float zv[4], pd[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const int b = __builtin_amdgcn_readfirstlane(tk[j + u]);
              zv[u] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(tv[j + u])));
              r[u] = Elem<T>::load_raw4(lane_ptr(dyt + (size_t)b * D.d, col));
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const float4 q = Elem<T>::widen4(r[u]);
              acc[0] = fmaf(zv[u], q.x, acc[0]);
              acc[1] = fmaf(zv[u], q.y, acc[1]);
              acc[2] = fmaf(zv[u], q.z, acc[2]);
              acc[3] = fmaf(zv[u], q.w, acc[3]);
              pd[u] = fmaf(wz.x, q.x, fmaf(wz.y, q.y, fmaf(wz.z, q.z, wz.w * q.w)));
            }
            if (dz_out) dz_group(j, 4, pd);
          }
          if (j < cur.cnt) {
            const int nval = cur.cnt - j;
            float pd[4] = {0.f, 0.f, 0.f, 0.f};
            for (int u = 0; u < nval; ++u) {
              const int b = __builtin_amdgcn_readfirstlane(tk[j + u]);
              const float zv = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(tv[j + u])));
              const float4 q = Elem<T>::widen4(Elem<T>::load_raw4(lane_ptr(dyt + (size_t)b * D.d, col)));
              acc[0] = fmaf(zv, q.x, acc[0]);
              acc[1] = fmaf(zv, q.y, acc[1]);
              acc[2] = fmaf(zv, q.z, acc[2]);
              acc[3] = fmaf(zv, q.w, acc[3]);
              const float pu = fmaf(wz.x, q.x, fmaf(wz.y, q.y, fmaf(wz.z, q.z, wz.w * q.w)));
              pd[0] = u == 0 ? pu : pd[0];
              pd[1] = u == 1 ? pu : pd[1];
              pd[2] = u == 2 ? pu : pd[2];
            }
            if (dz_out) dz_group(j, nval, pd);
          }
        }
        const float w4[4] = {wl.x, wl.y, wl.z, wl.w};
        float g4[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) g4[k] = fmaf(coef, w4[k], acc[k]);
        if (dW_dec && on) Elem<T>::store4(lane_ptr(dW_dec + o, col), make_float4(g4[0], g4[1], g4[2], g4[3]));
        if (fuse.m) {
          float mm[4] = {m4[0], m4[1], m4[2], m4[3]};
          float vv[4] = {v4[0], v4[1], v4[2], v4[3]};
          float pp[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) pp[k] = MASTER ? p4[k] : w4[k];
#pragma unroll
          for (int k = 0; k < 4; ++k) adam_element(pp[k], mm[k], vv[k], g4[k], fuse.a);
          const float4 pn = make_float4(pp[0], pp[1], pp[2], pp[3]);
          const typename Elem<T>::Raw4 stored = Elem<T>::narrow4(pn);
          if (on) {
            nt_store_f4(lane_ptr(fuse.m + o, col), make_float4(mm[0], mm[1], mm[2], mm[3]));
            nt_store_f4(lane_ptr(fuse.v + o, col), make_float4(vv[0], vv[1], vv[2], vv[3]));
            if (MASTER) nt_store_f4(lane_ptr(fuse.master + o, col), pn);
            Elem<T>::nt_store_raw4(lane_ptr(W_dec + o, col), stored);
          }
        }
      }
    }
  }
}

// bf16 storage: slices of at most 256 columns where eight of them make up d, fewer slices for smaller d (with eight of 32 columns at d =
// 256 a wavefront's 64 lanes held 8 quads of columns): slices, and columns of a slice in whole runs of 8.
__host__ __device__ inline int slice_cols(Dims D) { const int S = dz_slices(true, D.d, D.B); return (D.d + 8 * S - 1) / (8 * S) * 8; }

// bf16 storage.  What bounds it: the bytes that come back through the vector caches, state and gathered rows added up (a wavefront's
// loads return in order, so rows that wait in the L2 do not overtake state on its way from HBM), and below a few tokens per
// feature the state alone at 6 TB/s.  Hence 16 bytes per lane and load for the rows (rows that lie in the L2 come at 18 TB/s with 8 bytes
// per lane, at 28 to 31 with 16, whatever their stride), and every weight loaded once: as quads of columns for the update,
// turned into runs of 8 through LDS for the dot products.
// A load takes 4 entries of the feature's list at a time, one per row of 16 lanes, 128 columns each.  The sum z * row
// goes to the matrix cores: as A operand of v_mfma_f32_16x16x32 the load's registers are a 16 x 32 matrix whose row m is column run m
// (8 columns) and whose k = 8 t + c is column c of entry t's run; with B[8 t + c][n] = z_t where c = n, else 0, entry (m, n) of
// the product is column 8 m + n of the sum over the 4 entries: products exact, sums fp32.  The dot products for dz stay on the
// vector unit (packed, 16 lanes per entry, four entries per cross-lane sum).  z is a bf16 value: nothing is rounded.
// L = 16, d = 2048, F = 8192, 4096 tokens with the update, against one entry at a time with 8 bytes per lane: 82 active features per
// token 19.1 -> 15.0 ms, 16: 9.05 -> 8.35, 2.5: 7.4 either way.  Whole steps (with the other changes to the list-driven path) at L = 12,
// d = 768, F = 6144: 12.2 -> 7.5 ms at 1 % active, 8.4 -> 5.0 at 0.4 %; of that from four slices instead of eight: 8.5 -> 7.5, 5.7 -> 5.0.
// L = 8, d = 200, F = 2000, 1000 tokens, 1 %: 725 -> 361 us, 555 with eight slices.  More rows or the next feature's state in flight per wavefront: no faster (16.4 to 18.3 ms).
// NH: runs of 128 columns per pass.  ADAM: 0 gradient only, 1 with the update, 2 with fp32 master weights.
constexpr int SDM_ITEMS = 4;      // quads of features per workgroup; 2: 1.5 % slower, 8: 3 %
template <int NH, int ADAM>
__global__ __launch_bounds__(256, (NH == 1 ? 7 : NH == 2 ? 5 : 3) - (ADAM == 2 ? 1 : 0)) void sparse_dwdec_mfma_kernel(
    Dims D, FeatureLists fl, const bf16_t* __restrict__ d_yhat, bf16_t* __restrict__ W_dec, const float* __restrict__ G,
    const float* __restrict__ norms, bf16_t* __restrict__ dW_dec, AdamFuseArgs fuse, const int32_t* __restrict__ flags,
    float* __restrict__ n2_part, const int32_t* __restrict__ fl_tok, const float* __restrict__ fl_val,
    const int32_t* __restrict__ fl_cnt, const int32_t* __restrict__ fl_off) {
  if (!lists_backward_selected(flags, fl.kcap)) return;
  typedef Elem<bf16_t> E;
  constexpr int IT = SDM_ITEMS, R = NH > 2 ? 2 : 1;      // column quads per lane in the update
  constexpr int COLS = 128 * NH;
  __shared__ __align__(16) unsigned char smem[4][3072];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = lane >> 4, i16 = lane & 15;
  float* const sums = reinterpret_cast<float*>(smem[wv]);                       // [COLS] after the token loop
  nt_u32x2* const win = reinterpret_cast<nt_u32x2*>(smem[wv]);                  // [64] list window during it
  const u32x4_lds* const wts = reinterpret_cast<const u32x4_lds*>(smem[wv] + 2048);      // [COLS] weights, by runs of 8
  nt_u32x2* const wts8 = reinterpret_cast<nt_u32x2*>(smem[wv] + 2048);                   // and as the lanes load them
  // the B operand's diagonal: lane (t, n) holds z_t at k = n of its run of 8
  const uint32_t half = i16 >= 8 ? 0u : (i16 & 1) ? 0xffff0000u : 0x0000ffffu;
  // (gridDim.x is a multiple of 8.  With fewer slices than XCDs 8 / S of them take the same slice, each its share of the features)
  const int S = dz_slices(true, D.d, D.B), slice = blockIdx.x & (S - 1), wg = blockIdx.x / S, nwg = gridDim.x / S;
  const int sw = slice_cols(D), slots = 8 * ((D.d + 2047) / 2048) / S, passes = NH == 4 ? (sw + COLS - 1) / COLS : 1;
  const int F4 = (D.F + 3) / 4;
  const bool dz_on = fused_dz_selected(flags, fl);
  const uint32_t row_bytes = (uint32_t)D.d * 2;
  const int pq = blockIdx.y;                               // pair ordinal, target-major: (0,0) (0,1) (1,1) (0,2) ...
  int lp = __builtin_amdgcn_readfirstlane((int)((__builtin_amdgcn_sqrtf(8.0f * (float)pq + 1.0f) - 1.0f) * 0.5f));
  while ((lp + 1) * (lp + 2) / 2 <= pq) ++lp;
  while (lp * (lp + 1) / 2 > pq) --lp;
  const int l = pq - lp * (lp + 1) / 2;
  const int pair = packed_index(l, lp, D.L);
  const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(d_yhat + (size_t)lp * D.B * D.d), 0, (int)((size_t)D.B * D.d * 2), 0x00020000);
  const size_t pairF = (size_t)pair * D.F;
  const int32_t* const tkl = fl_tok + (size_t)l * D.B * fl.kcap;
  const float* const tvl = fl_val + (size_t)l * D.B * fl.kcap;
  const size_t lF = (size_t)l * D.F;
  for (int q0 = wg * IT; q0 < F4; q0 += nwg * IT) {
    const int f_first = q0 * 4 + wv;
    if (f_first >= D.F) break;
    const int f_end = min(D.F, (q0 + IT) * 4);
    // the list heads of an item are requested one item ahead
    int cnt = fl_cnt[lF + f_first], off = fl_off[lF + f_first];
    uint32_t tok = UniformRun(tkl + off, cnt * 4).load4(lane * 4u), val = UniformRun(tvl + off, cnt * 4).load4(lane * 4u);
#pragma unroll 1
    for (int fi = f_first; fi < f_end; fi += 4) {
      int f = fi;      // (opaque: addresses are formed from it anew instead of being carried along per lane)
      asm volatile("" : "+s"(f));
      const bool more = f + 4 < f_end;
      const int fn = more ? f + 4 : f;
      const int cnt_n = fl_cnt[lF + fn], off_n = fl_off[lF + fn];
      const float Gf = G[lF + f], nf = norms[lF + f];
      const size_t o = ((size_t)pair * D.F + f) * D.d;
      float* dz_out = dz_on ? fl.dz_part + ((size_t)pair * S + slice) * fl.ecap + off : nullptr;
      uint32_t tok_n = 0, val_n = 0;
      for (int ps = 0; ps < passes; ++ps) {
        const int c0 = slice * sw + ps * COLS;
        const int cols = __builtin_amdgcn_readfirstlane(max(min(min(sw - ps * COLS, COLS), D.d - c0), 0));
        const UniformRun pw(W_dec + o + c0, cols * 2);
        E::Raw4 wq[R];      // a lane's quads of columns: the weights, then the optimizer state
        nt_f32x4 m4[R], v4[R], p4[R];
#pragma unroll
        for (int r = 0; r < R; ++r) wq[r] = pw.load8((uint32_t)(r * 64 + lane) * 8u);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (ADAM) {
            m4[r] = UniformRun(fuse.m + o + c0, cols * 4).load_f4((uint32_t)(r * 64 + lane) * 16u);
            v4[r] = UniformRun(fuse.v + o + c0, cols * 4).load_f4((uint32_t)(r * 64 + lane) * 16u);
            if (ADAM == 2) p4[r] = UniformRun(fuse.master + o + c0, cols * 4).load_f4((uint32_t)(r * 64 + lane) * 16u);
          }
        }
        tok_n = UniformRun(tkl + off_n, cnt_n * 4).load4(lane * 4u);
        val_n = UniformRun(tvl + off_n, cnt_n * 4).load4(lane * 4u);
        float4 a4[R];
#pragma unroll
        for (int r = 0; r < R; ++r) a4[r] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (cnt > 0) {
          wave_lds_order();
#pragma unroll
          for (int r = 0; r < R; ++r) wts8[r * 64 + lane] = wq[r];
          wave_lds_order();
          uint32_t voff[NH];
          u32x4_lds w8[NH];
          f32x4_mfma acc[NH];
#pragma unroll
          for (int h = 0; h < NH; ++h) {      // (lanes past the slice: zeros, no descriptor covers their offset)
            voff[h] = h * 128 + i16 * 8 < cols ? (uint32_t)(c0 + h * 128 + i16 * 8) * 2u : 0x7ffffff0u;
            w8[h] = wts[h * 16 + i16];
            acc[h] = f32x4_mfma{0.f, 0.f, 0.f, 0.f};
          }
          for (int w0 = 0; w0 < cnt; w0 += 64) {
            const int n = __builtin_amdgcn_readfirstlane(min(64, cnt - w0));
            if (w0 > 0 || (NH == 4 && ps > 0)) {      // (the head came with the item; a later pass has another window in its place)
              tok = UniformRun(tkl + off + w0, n * 4).load4(lane * 4u);
              val = UniformRun(tvl + off + w0, n * 4).load4(lane * 4u);
            }
            wave_lds_order();
            win[lane] = nt_u32x2{lane < n ? tok * row_bytes : 0x80000000u, __builtin_amdgcn_perm(val, val, 0x07060706u)};
            wave_lds_order();
            float dz_keep = 0.f;
            for (int j = 0; j < n; j += 16) {
              const bool o1 = lane & 1, o2 = lane & 2;
              auto sets = [&](int u0) -> float {      // two sets of 4 entries, one entry per row of 16 lanes; their dot products in turn
                float pd[2] = {0.f, 0.f};
                nt_u32x2 en[2];
                u32x4_lds q[2][NH];
#pragma unroll
                for (int u = 0; u < 2; ++u) en[u] = win[j + 4 * (u0 + u) + grp];
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                  for (int h = 0; h < NH; ++h)
                    q[u][h] = __builtin_bit_cast(u32x4_lds, __builtin_amdgcn_raw_buffer_load_b128(rows, (int)(en[u][0] + voff[h]), 0, 0));
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                  const uint32_t zs = en[u][1] & half;
                  const u32x4_lds zd = {(i16 >> 1) == 0 ? zs : 0u, (i16 >> 1) == 1 ? zs : 0u, (i16 >> 1) == 2 ? zs : 0u, (i16 >> 1) == 3 ? zs : 0u};
#pragma unroll
                  for (int h = 0; h < NH; ++h) {
                    acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_mfma, q[u][h]), __builtin_bit_cast(bf16x8_mfma, zd), acc[h], 0, 0, 0);
#pragma unroll
                    for (int k = 0; k < 4; ++k) pd[u] = dot2_bf16(q[u][h][k], w8[h][k], pd[u]);
                  }
                }
                return (o1 ? pd[1] : pd[0]) + dpp_move<0xB1>(o1 ? pd[0] : pd[1]);
              };
              const float r1 = sets(0);
              const float r2 = j + 8 < n ? sets(2) : 0.f;
              float r = (o2 ? r2 : r1) + dpp_move<0x4E>(o2 ? r1 : r2);
              r += dpp_move<0x128>(r);      // row_ror:8
              r += dpp_move<0x124>(r);      // row_ror:4
              if ((i16 >> 2) == (j >> 4)) dz_keep = r;
            }
            const int td = (i16 >> 2) * 16 + (i16 & 3) * 4 + grp;      // the entry whose sum the lane kept
            if (dz_out) {
              const UniformRun out(dz_out + w0, n * 4);
              if (NH == 4 && ps > 0) dz_keep += __uint_as_float(out.load4(td * 4u));      // (a slice wider than a pass: one after the other)
              out.store4(td * 4u, __float_as_uint(dz_keep));
            }
          }
          wave_lds_order();
#pragma unroll
          for (int h = 0; h < NH; ++h)
            if (i16 < 8) {
#pragma unroll
              for (int r = 0; r < 4; ++r) sums[h * 128 + (4 * grp + r) * 8 + i16] = acc[h][r];
            }
          wave_lds_order();
#pragma unroll
          for (int r = 0; r < R; ++r) {
            a4[r] = *reinterpret_cast<const float4*>(sums + (r * 64 + lane) * 4);
            wq[r] = wts8[r * 64 + lane];      // (not held through the loop)
          }
          // The zeros beside z in the B operand meet the other seven columns of a run, so an infinity or a NaN in one column of
          // d y_hat would reach them.  Where a sum is not finite the columns are summed up one by one.
          float nan = 0.f;
#pragma unroll
          for (int r = 0; r < R; ++r)
            if ((r * 64 + lane) * 4 < cols) nan = fmaf(a4[r].x, 0.f, fmaf(a4[r].y, 0.f, fmaf(a4[r].z, 0.f, fmaf(a4[r].w, 0.f, nan))));
          if (__builtin_amdgcn_ballot_w64(nan != nan)) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
              a4[r] = make_float4(0.f, 0.f, 0.f, 0.f);
              for (int e = 0; e < cnt; ++e) {
                const uint32_t at = (r * 64 + lane) * 4 < cols ? (uint32_t)tkl[off + e] * row_bytes + (uint32_t)(c0 + (r * 64 + lane) * 4) * 2u : 0x80000000u;
                const nt_u32x2 raw = __builtin_bit_cast(nt_u32x2, __builtin_amdgcn_raw_buffer_load_b64(rows, (int)at, 0, 0));
                const float4 y = E::widen4(raw);
                const float z = list_z<bf16_t>(tvl[off + e]);
                a4[r] = make_float4(fmaf(z, y.x, a4[r].x), fmaf(z, y.y, a4[r].y), fmaf(z, y.z, a4[r].z), fmaf(z, y.w, a4[r].w));
              }
            }
          }
        }
        const float coef = Gf * __builtin_amdgcn_rcpf(fmaxf(nf, 1e-30f));
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int qd = r * 64 + lane;
          const bool on = qd * 4 < cols;
          const float4 wl = E::widen4(wq[r]);
          const float w4[4] = {wl.x, wl.y, wl.z, wl.w};
          const float g4[4] = {fmaf(coef, w4[0], a4[r].x), fmaf(coef, w4[1], a4[r].y), fmaf(coef, w4[2], a4[r].z), fmaf(coef, w4[3], a4[r].w)};
          if (dW_dec) UniformRun(dW_dec + o + c0, cols * 2).store8((uint32_t)qd * 8u, E::narrow4(make_float4(g4[0], g4[1], g4[2], g4[3])), 0);
          if (ADAM) {
            float mm[4] = {m4[r][0], m4[r][1], m4[r][2], m4[r][3]};
            float vv[4] = {v4[r][0], v4[r][1], v4[r][2], v4[r][3]};
            float pp[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) pp[k] = ADAM == 2 ? p4[r][k] : w4[k];
#pragma unroll
            for (int k = 0; k < 4; ++k) adam_element(pp[k], mm[k], vv[k], g4[k], fuse.a);
            const float4 pn = make_float4(pp[0], pp[1], pp[2], pp[3]);
            const E::Raw4 stored = E::narrow4(pn);
            UniformRun(fuse.m + o + c0, cols * 4).store_f4((uint32_t)qd * 16u, nt_f32x4{mm[0], mm[1], mm[2], mm[3]});
            UniformRun(fuse.v + o + c0, cols * 4).store_f4((uint32_t)qd * 16u, nt_f32x4{vv[0], vv[1], vv[2], vv[3]});
            if (ADAM == 2) UniformRun(fuse.master + o + c0, cols * 4).store_f4((uint32_t)qd * 16u, nt_f32x4{pp[0], pp[1], pp[2], pp[3]});
            pw.store8((uint32_t)qd * 8u, stored, 1);
            if (n2_part && ps * R + r < slots) {      // sum of squares of 256 weights as stored, for the next step's norms
              const float4 wn = E::widen4(stored);
              const float sq = on ? (wn.x * wn.x + wn.y * wn.y) + (wn.z * wn.z + wn.w * wn.w) : 0.f;
              const int b16 = __float_as_int(row16_sum(sq));
              const float tot = (__int_as_float(__builtin_amdgcn_readlane(b16, 0)) + __int_as_float(__builtin_amdgcn_readlane(b16, 16))) +
                                (__int_as_float(__builtin_amdgcn_readlane(b16, 32)) + __int_as_float(__builtin_amdgcn_readlane(b16, 48)));
              // (the slice's slots are written by its last sums: those that no columns belong to with zeros)
              const int at = ps * R + r, end = ps + 1 == passes && r + 1 == R ? slots : at + 1;
              if (lane < end - at) n2_part[(pairF + f) * (S * slots) + slice * slots + at + lane] = lane == 0 ? tot : 0.f;
            }
          }
        }
        wave_lds_order();
      }
      cnt = cnt_n; off = off_n; tok = tok_n; val = val_n;
    }
  }
}

// Fused dz, second half: an entry's partial dot products summed over the targets and the column slices, always in that
// order, plus the gradient of the sparsity term.  Bound by the partials, a float per entry, target and slice: a workgroup takes the
// entries of 64 consecutive features one per lane, which reads them in whole lines (16 lanes per feature, in pieces of 64 bytes at
// 4 KB and more from each other: 0.80 ms at L = 16, 41 entries per feature and layer; 0.40 now).
// FINAL (bf16 storage, no dead-feature term): what ste_reduce_kernel does elsewhere in a scan of the dense arrays (0.43 ms there): the
// final d pre (times the x scale for int8 inputs) and the column sums for d theta and d b_enc, an entry's dz going through its first
// partial's place.
template <typename T, bool FINAL>
__global__ __launch_bounds__(256) void dz_from_partials_kernel(Dims D, FeatureLists fl, const float* __restrict__ norms,
                                                               float lam_c_over_b, float C, T* __restrict__ dpre,
                                                               const int32_t* __restrict__ flags, const float* __restrict__ x_scale,
                                                               float* __restrict__ sum_theta, float* __restrict__ sum_benc) {
  if (!fused_dz_selected(flags, fl)) return;
  __shared__ int off_s[64], cnt_s[64];
  __shared__ float nn_s[64];
  const int groups = (D.F + 63) / 64, l = (int)(blockIdx.x / groups), f0 = (int)(blockIdx.x % groups) * 64, nf = min(64, D.F - f0);
  if (threadIdx.x < 64) {
    const size_t lf = (size_t)l * D.F + f0 + min((int)threadIdx.x, nf - 1);
    off_s[threadIdx.x] = fl.off[lf];
    cnt_s[threadIdx.x] = (int)threadIdx.x < nf ? fl.cnt[lf] : 0;
    nn_s[threadIdx.x] = norms[lf];
  }
  __syncthreads();
  const int e0 = off_s[0], e1 = off_s[nf - 1] + cnt_s[nf - 1];
  const size_t lists = (size_t)l * D.B * fl.kcap;
  const int S = dz_slices(sizeof(T) == 2, D.d, D.B);
  float* const part = fl.dz_part + (size_t)packed_index(l, l, D.L) * S * fl.ecap;      // the targets' partials follow each other
  const int n = (D.L - l) * S;
  for (int e = e0 + threadIdx.x; e < e1; e += 256) {
    float acc = 0.f;
    const float* q = part + e;
    int i = 0;
    for (; i + 32 <= n; i += 32) {      // four targets' partials in flight
      float p[32];
#pragma unroll
      for (int u = 0; u < 32; ++u) p[u] = q[(size_t)(i + u) * fl.ecap];
#pragma unroll
      for (int u = 0; u < 32; ++u) acc += p[u];
    }
    for (; i + 8 <= n; i += 8) {
      float p[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) p[u] = q[(size_t)(i + u) * fl.ecap];
#pragma unroll
      for (int u = 0; u < 8; ++u) acc += p[u];
    }
    for (; i < n; ++i) acc += q[(size_t)i * fl.ecap];
    int k = 0;      // the last feature that starts at or before e (empty ones before it start there too)
#pragma unroll
    for (int step = 32; step > 0; step >>= 1)
      if (k + step < nf && off_s[k + step] <= e) k += step;
    const float v = fl.val[lists + e], zv = list_z<T>(v), nn = nn_s[k];
    const int b = fl.tok[lists + e];
    const float ex = __builtin_amdgcn_exp2f(-2.0f * 1.4426950408889634f * C * nn * fabsf(zv));
    const float sden = 1.0f + ex;
    const float gsp = 4.0f * lam_c_over_b * nn * ex * __builtin_amdgcn_rcpf(sden * sden);
    const float dz = acc + gsp;
    T* const out = dpre + ((size_t)l * D.B + b) * D.F + f0 + k;
    if (!FINAL) {
      Elem<T>::store(out, dz);
    } else {
      part[e] = dz;
      if (__float_as_uint(v) & CLS_ACTIVE) Elem<T>::store(out, x_scale ? dz * x_scale[(size_t)l * D.B + b] : dz);
    }
  }
  if (!FINAL) return;
  __threadfence_block();
  __syncthreads();
  for (int k = threadIdx.x >> 4; k < nf; k += 16) {      // 16 lanes per feature
    float st = 0.f, sb = 0.f;
    for (int j = threadIdx.x & 15; j < cnt_s[k]; j += 16) {
      const float dz = part[off_s[k] + j];
      const uint32_t c = __float_as_uint(fl.val[lists + off_s[k] + j]);
      st += (c & CLS_WINDOW) ? dz : 0.f;
      sb += (c & CLS_ACTIVE) ? dz : 0.f;
    }
    st = row16_sum(st);
    sb = row16_sum(sb);
    if ((threadIdx.x & 15) == 0) {
      sum_theta[(size_t)l * D.F + f0 + k] = st;
      sum_benc[(size_t)l * D.F + f0 + k] = sb;
    }
  }
}

}  // namespace

// Whether the decode may go in step: what the host knows of the rule at stepped_gather_decode_kernel (max_density: up to which the
// lists are used at all; what pays at some density pays at every larger one)
static bool stepped_decode_possible(bool bf16, Dims D, double max_density) {
  return bf16 && D.F <= 8192 && (double)D.P() * D.F * D.d * 2.0 >= 128e6 && (size_t)D.F * D.d * 2 < ((size_t)1 << 31) &&
         stepping_pays(D, max_density * D.B * D.F * D.P(), max_density * D.F);
}

hipError_t launch_decode_decide(hipStream_t s, bool bf16, Dims D, const int32_t* l0, float density_threshold,
                                float backward_density_threshold, int forced, bool backward_without_row_lists,
                                int32_t* flags, uint32_t* step_ctr) {
  hipLaunchKernelGGL(decode_decide_kernel, dim3(1), dim3(512), 0, s, D, l0, density_threshold,
                     backward_density_threshold, forced, backward_without_row_lists ? 1 : 0,
                     stepped_decode_possible(bf16, D, forced ? 1.0 : (double)density_threshold) ? 1 : 0, flags, step_ctr);
  return hipGetLastError();
}

hipError_t launch_compact_active(hipStream_t s, bool bf16, Dims D, const void* z, const uint8_t* cls, GatherLists g,
                                 int32_t* flags) {
  const long rows = (long)D.L * D.B;
  const dim3 grid((unsigned)((rows + 3) / 4));
  if (bf16)
    hipLaunchKernelGGL((compact_active_kernel<bf16_t>), grid, dim3(256), 0, s, D, (const bf16_t*)z, cls, g, flags);
  else
    hipLaunchKernelGGL((compact_active_kernel<float>), grid, dim3(256), 0, s, D, (const float*)z, cls, g, flags);
  return hipGetLastError();
}

hipError_t launch_gather_decode(hipStream_t s, bool bf16, Dims D, GatherLists g, const void* W_dec,
                                const float* b_dec, float* y_hat, int32_t* flags, uint32_t* step_ctr, double max_density) {
  const size_t ncs = ((size_t)D.d + GD_COLS - 1) / GD_COLS;
  const dim3 grid((unsigned)(((size_t)D.L * D.B + 3) / 4 * ncs));
  if (bf16)
    hipLaunchKernelGGL((gather_decode_kernel<bf16_t>), grid, dim3(256), 0, s, D, g, (const bf16_t*)W_dec, b_dec, y_hat,
                       flags);
  else
    hipLaunchKernelGGL((gather_decode_kernel<float>), grid, dim3(256), 0, s, D, g, (const float*)W_dec, b_dec, y_hat,
                       flags);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || !stepped_decode_possible(bf16, D, max_density)) return e;
  hipLaunchKernelGGL(stepped_gather_decode_kernel, dim3(8 * SGD_WGS), dim3(64 * SGD_WAVES), 0, s, D, g.kcap, g.stride, g.counts,
                     g.idx, g.val, (const bf16_t*)W_dec, b_dec, y_hat, flags, step_ctr, SGD_WGS);
  return hipGetLastError();
}

hipError_t launch_sparse_dpre_fill(hipStream_t s, bool bf16, Dims D, const uint8_t* cls, const float* norms,
                                   float lam1_over_b, void* dpre, const int32_t* flags, int kcap) {
  const dim3 grid(256 * 16);
  if (bf16)
    hipLaunchKernelGGL((sparse_dpre_fill_kernel<bf16_t>), grid, dim3(256), 0, s, D, cls, norms, lam1_over_b,
                       (bf16_t*)dpre, flags, kcap);
  else
    hipLaunchKernelGGL((sparse_dpre_fill_kernel<float>), grid, dim3(256), 0, s, D, cls, norms, lam1_over_b,
                       (float*)dpre, flags, kcap);
  return hipGetLastError();
}

hipError_t launch_gather_dz(hipStream_t s, bool bf16, Dims D, GatherLists g, const void* d_yhat, const void* W_dec,
                            const float* norms, float lam_c_over_b, float C, void* dpre, const int32_t* flags,
                            const FeatureLists* fused) {
  FeatureLists fz{};
  if (fused) fz = *fused;
  const size_t esz = bf16 ? 2 : 4;
  int tcap = (int)(65536 / ((size_t)D.d * esz));      // targets whose d y_hat rows fit 64 KB of LDS
  if (tcap > D.L) tcap = D.L;
  if (D.d % 8 == 0 && tcap >= 1 && !getenv("CLT_GDZ_NO_LDS")) {
    // One workgroup per row, no loop over rows: the dispatcher hands rows out as workgroups retire, so the long
    // rows of a heavy-tailed batch (the same tokens in every layer) do not pile up on a few resident workgroups.
    const size_t rows = (size_t)D.L * D.B;
    const dim3 grid((unsigned)(rows < ((size_t)1 << 30) ? rows : ((size_t)1 << 30)));
    const size_t lds = (size_t)tcap * D.d * esz;
    if (bf16)
      hipLaunchKernelGGL((gather_dz_lds_kernel<bf16_t>), grid, dim3(1024), lds, s, D, g, (const bf16_t*)d_yhat,
                         (const bf16_t*)W_dec, norms, lam_c_over_b, C, (bf16_t*)dpre, flags, tcap, fz);
    else
      hipLaunchKernelGGL((gather_dz_lds_kernel<float>), grid, dim3(1024), lds, s, D, g, (const float*)d_yhat,
                         (const float*)W_dec, norms, lam_c_over_b, C, (float*)dpre, flags, tcap, fz);
    return hipGetLastError();
  }
  // rows too wide for LDS staging, or not a multiple of 8 columns (or CLT_GDZ_NO_LDS set, for comparison runs)
  const size_t items = ((size_t)D.L * D.B + 7) / 8 * 8 * GDZ_PARTS;
  const dim3 grid((unsigned)(items < 256 * 64 ? items : 256 * 64));
  if (bf16)
    hipLaunchKernelGGL((gather_dz_kernel<bf16_t>), grid, dim3(256), 0, s, D, g, (const bf16_t*)d_yhat,
                       (const bf16_t*)W_dec, norms, lam_c_over_b, C, (bf16_t*)dpre, flags, fz);
  else
    hipLaunchKernelGGL((gather_dz_kernel<float>), grid, dim3(256), 0, s, D, g, (const float*)d_yhat,
                       (const float*)W_dec, norms, lam_c_over_b, C, (float*)dpre, flags, fz);
  return hipGetLastError();
}
hipError_t init_gather() {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&gather_dz_lds_kernel<bf16_t>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, 65536);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&gather_dz_lds_kernel<float>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, 65536);
}

hipError_t launch_feature_lists(hipStream_t s, bool bf16, Dims D, const uint8_t* cls, const void* z, FeatureLists fl,
                                int32_t* flags, bool dense_when_too_long) {
  const int LF4 = D.L * D.F / 4;
  const dim3 grid((LF4 + 255) / 256, FL_SEGS), grid8((LF4 / 2 + 255) / 256, FL_SEGS);
  hipLaunchKernelGGL(fl_count_kernel, grid8, dim3(256), 0, s, D, cls, fl, flags);
  hipLaunchKernelGGL(fl_scan_kernel, dim3(D.L), dim3(FL_SCAN_THREADS), 0, s, D, fl, flags,
                     dense_when_too_long && fl.dz_part ? fl.ecap : 0);
  if (bf16)
    hipLaunchKernelGGL((fl_fill_kernel<bf16_t>), grid, dim3(256), 0, s, D, cls, (const bf16_t*)z, fl, flags);
  else
    hipLaunchKernelGGL((fl_fill_kernel<float>), grid, dim3(256), 0, s, D, cls, (const float*)z, fl, flags);
  return hipGetLastError();
}

// The sliced kernels: d in slices (fp32: eight of whole lane quads), and one target's d y_hat within reach of a 32-bit byte offset
static bool sparse_dwdec_sliced(bool bf16, Dims D) {
  return (bf16 || D.d % 32 == 0) && (size_t)D.B * D.d * 2 < ((size_t)1 << 31) && !getenv("CLT_SD_ROWS");
}
bool sparse_dwdec_takes_dz(bool bf16, Dims D) { return sparse_dwdec_sliced(bf16, D) && !getenv("CLT_NO_FUSED_DZ"); }

hipError_t launch_dz_from_partials(hipStream_t s, bool bf16, Dims D, FeatureLists fl, const float* norms,
                                   float lam_c_over_b, float C, void* dpre, const int32_t* flags, bool final, const float* x_scale,
                                   float* sum_theta, float* sum_benc) {
  if (!fl.dz_part) return hipSuccess;
  const dim3 grid((unsigned)((size_t)D.L * ((D.F + 63) / 64)));
#define CLT_DZP(T, FINAL)                                                                                             \
  hipLaunchKernelGGL((dz_from_partials_kernel<T, FINAL>), grid, dim3(256), 0, s, D, fl, norms, lam_c_over_b, C, (T*)dpre, flags, \
                     x_scale, sum_theta, sum_benc)
  if (!bf16) CLT_DZP(float, false); else if (final) CLT_DZP(bf16_t, true); else CLT_DZP(bf16_t, false);
#undef CLT_DZP
  return hipGetLastError();
}

template <int NH>
static hipError_t launch_sparse_dwdec_mfma(hipStream_t s, Dims D, const FeatureLists& fl, const DWdecArgs& a, float* n2,
                                           const int32_t* flags) {
  // (every workgroup takes SDM_ITEMS quads of features while the grid allows it)
  const size_t wgs = (((D.F + 3) / 4 + SDM_ITEMS - 1) / SDM_ITEMS * dz_slices(true, D.d, D.B) + 7) / 8, most = (size_t)1 << 19;
  const dim3 grid(8 * (unsigned)(wgs < most ? wgs : most), D.P());
#define CLT_SDM(ADAM)                                                                                                 \
  hipLaunchKernelGGL((sparse_dwdec_mfma_kernel<NH, ADAM>), grid, dim3(256), 0, s, D, fl, (const bf16_t*)a.d_yhat,     \
                     (bf16_t*)a.W_dec, a.G, a.norms, (bf16_t*)a.dW_dec, a.fuse, flags, n2, fl.tok, fl.val, fl.cnt, fl.off)
  if (!a.fuse.m) CLT_SDM(0); else if (!a.fuse.master) CLT_SDM(1); else CLT_SDM(2);
#undef CLT_SDM
  return hipGetLastError();
}

hipError_t launch_sparse_dwdec(hipStream_t s, bool bf16, Dims D, FeatureLists fl, const DWdecArgs& a,
                               const int32_t* flags) {
  const bool master = a.fuse.m && a.fuse.master;
  float* n2 = (bf16 && a.fuse.m && D.d % 256 == 0) ? a.n2_part : nullptr;
  if (sparse_dwdec_sliced(bf16, D)) {
    if (bf16) {
      const int runs = (slice_cols(D) + 127) / 128;
      return runs <= 1 ? launch_sparse_dwdec_mfma<1>(s, D, fl, a, n2, flags) : runs == 2 ? launch_sparse_dwdec_mfma<2>(s, D, fl, a, n2, flags)
             : runs == 3 ? launch_sparse_dwdec_mfma<3>(s, D, fl, a, n2, flags) : launch_sparse_dwdec_mfma<4>(s, D, fl, a, n2, flags);
    }
    const size_t per_xcd = ((size_t)(D.L * (D.L + 1) / 2) * ((D.F + 3) / 4) + SD_ITEMS_PER_WG - 1) / SD_ITEMS_PER_WG,
                 gx = (size_t)1 << 27;
    const dim3 grid((unsigned)(8 * (per_xcd < gx ? per_xcd : gx)));
#define CLT_SDS(M)                                                                                                 \
  hipLaunchKernelGGL((sparse_dwdec_sliced_kernel<M>), grid, dim3(256), 0, s, D, fl, (const float*)a.d_yhat,        \
                     (float*)a.W_dec, a.G, a.norms, (float*)a.dW_dec, a.fuse, flags, fl.tok, fl.val)
    if (master) CLT_SDS(true); else CLT_SDS(false);
#undef CLT_SDS
    return hipGetLastError();
  }
  // fp32 with d not a multiple of 32, a batch beyond that reach (or CLT_SD_ROWS set, for comparison runs): whole rows per workgroup
  const size_t items = (size_t)D.L * D.F * ((D.L + SD_TCH - 1) / SD_TCH), gcap = (size_t)1 << 30;
  const dim3 grid((unsigned)(items < gcap ? items : gcap));
#define CLT_SD(T, M)                                                                                              \
  hipLaunchKernelGGL((sparse_dwdec_kernel<T, M>), grid, dim3(256), 0, s, D, fl, (const T*)a.d_yhat, (T*)a.W_dec, a.G, \
                     a.norms, (T*)a.dW_dec, a.fuse, flags, n2)
  if (bf16) { if (master) CLT_SD(bf16_t, true); else CLT_SD(bf16_t, false); }
  else { if (master) CLT_SD(float, true); else CLT_SD(float, false); }
#undef CLT_SD
  return hipGetLastError();
}

}  // namespace clt
