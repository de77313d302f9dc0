// fp32 path of the five CLT contractions on gfx950: fp32 storage, fp32 products and fp32 accumulation on the
// matrix cores (v_mfma_f32_16x16x4_f32, a full-precision fused multiply-add; no reduced-precision mode).  The bf16
// path lives in kernels_gemm_bf16.hip.
//
// What bounds it: the fp32 matrix rate (157 TFLOP/s nominal; a large library product reaches 153 here).  Vector FMAs
// without packed arithmetic end at half of that, and the operand traffic is small beside either.
//
// Against the vector-FMA kernel before it (64x64x16 tiles, scalar loads): L = 12, d = 768, F = 6144, B = 1024: decode
// 16.6 -> 6.0 ms (126 TFLOP/s; 7.9 without its K ranges cut), dz 12.0 -> 5.6 (135), dW_dec 12.2 -> 6.2 (121); L = 4, d = 64,
// F = 256, B = 128: decode 186 -> 5 us, dz 42 -> 12, dW_dec 72 -> 10.
//
// One workgroup = 4 wavefronts computes a TxT tile (T = 128: 64x64 per wavefront as 4x4 accumulators; T = 64: 32x32),
// K advances in steps of 32 through two LDS stages, two workgroups per CU cover each other's barriers.  Operands keep
// their memory order in LDS: one that is contiguous along K as [row][32 k] (a lane reads four consecutive k of its
// row in one go), one that is strided along K as [k][T rows] (four single reads).  Both leave the lane with k = 4 * (lane
// / 16) + q for MFMA q of a 16-wide slice, so any pair of layouts agrees and nothing is transposed.
// Loads go through buffer descriptors: a chunk outside the matrix gets an offset beyond the descriptor's range and
// reads as zero, so sizes that fit no tile run the same code as those that do.
// IN_ORDER (the encoder): one running sum per entry, in the order of K.  The MFMA adds its four products one after the other,
// each with one rounding, so the pre-activations are exactly a chain of FMAs over k = 0, 1, 2, ...  The active set, the window
// and the TopK selection are decided on them and jump where one lies within rounding of its threshold: another order of
// the sum would give a trained model another set for some inputs.  A lane then reads k = 4 q + lane / 16 for MFMA q,
// four single reads in both layouts; no slower (L = 12, d = 768, F = 6144, B = 1024: step 22.68 and 22.70 ms).
// The MFMA's operands are swapped (D = B^T A^T): a lane then holds four consecutive columns of one row, which is what
// the policies' epilogues take.
#include "common.h"
#include "gemm_policies.h"

namespace clt {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int FTK = 32;
constexpr uint32_t OUT_OF_RANGE = 0xffffff00u;      // lane offset that no descriptor below covers

__device__ __forceinline__ f32x4 load_chunk(const float* base, uint32_t voff) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, 0xffffff00u, 0x00027000);
  return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, 0, 0));
}

// One operand's T x 32 tile: staging by 256 lanes (T / 32 chunks of 16 bytes each) and fragment reads.
template <bool KC, int T, bool IN_ORDER>
struct Operand {
  static constexpr int NCH = T / 32;                       // chunks per lane
  // floats; the padding spreads the fragment reads over all banks (16 lanes' rows of four k, 4 apart or next to each other)
  static constexpr int PITCH = KC ? FTK + 4 : IN_ORDER ? T + 16 : T + 4;
  static constexpr int LDS_FLOATS = KC ? T * PITCH : FTK * PITCH;
  static constexpr int RSTEP = KC ? 32 : 1024 / T;         // rows (KC) or k (strided) between a lane's chunks
  uint32_t voff, ok;      // lane byte offset inside the tile; bit i: chunk i's row lies inside the matrix
  int klane, lds;         // KC: first k of the lane's chunks; strided: the k of its first chunk
  size_t step;            // elements between a lane's consecutive chunks (uniform)
  __device__ __forceinline__ void init(int t, int ld, int rows_left) {
    const int a = KC ? t >> 3 : t / (T / 4), b = KC ? (t & 7) * 4 : (t % (T / 4)) * 4;
    voff = (uint32_t)((size_t)a * ld + b) * 4u;
    lds = a * PITCH + b;
    step = (size_t)RSTEP * ld;
    klane = KC ? b : a;
    ok = 0;
#pragma unroll
    for (int i = 0; i < NCH; ++i)
      if ((KC ? a + RSTEP * i : b) < rows_left) ok |= 1u << i;
  }
  __device__ __forceinline__ void load(f32x4 (&r)[NCH], const float* base, int k_left) const {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const bool in = ((ok >> i) & 1u) && (KC ? klane : klane + RSTEP * i) < k_left;
      r[i] = load_chunk(base + i * step, in ? voff : OUT_OF_RANGE);
    }
  }
  __device__ __forceinline__ void store(float* s, const f32x4 (&r)[NCH]) const {
#pragma unroll
    for (int i = 0; i < NCH; ++i) *reinterpret_cast<f32x4*>(s + lds + i * RSTEP * PITCH) = r[i];
  }
  // fragment of the 16 rows from `row0` on for k slice `sl` (16 wide): element q is k = 16 sl + 4 (lane / 16) + q, or
  // 16 sl + 4 q + lane / 16 where the products are added in the order of k
  __device__ __forceinline__ static f32x4 frag(const float* s, int row0, int sl, int lane) {
    const int row = row0 + (lane & 15), k = 16 * sl + (IN_ORDER ? lane >> 4 : 4 * (lane >> 4));
    if (KC && !IN_ORDER) return *reinterpret_cast<const f32x4*>(s + row * PITCH + k);
    f32x4 v;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int kq = k + (IN_ORDER ? 4 * q : q);
      v[q] = s[KC ? row * PITCH + kq : kq * PITCH + row];
    }
    return v;
  }
};

template <class P, int T>
__global__ __launch_bounds__(256, 2) void gemm_f32_kernel(P p, TileGrid tg) {
  constexpr int NB = T / 32, W = T / 2;      // 16-blocks per wavefront and direction, wavefront block edge
  typedef Operand<P::A_KC, T, P::IN_ORDER> OA;
  typedef Operand<P::B_KC, T, P::IN_ORDER> OB;
  __shared__ __align__(16) float smem[2 * (OA::LDS_FLOATS + OB::LDS_FLOATS)];
  int gorder, tm, tn;
  if (!tg.decode(blockIdx.x, gorder, tm, tn) || p.skip()) return;
  const typename P::GInfo gi = p.ginfo(gorder);
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = (w >> 1) * W, wn = (w & 1) * W;
  const int m0 = tm * T, n0 = tn * T;
  const int M = p.M, N = p.N, kseg = p.kseg;
  const int spseg = (kseg + FTK - 1) / FTK;
  const KRange kr = p.krange(gi, spseg);

  OA oa;
  OB ob;
  oa.init(t, p.lda, M - m0);
  ob.init(t, p.ldb, N - n0);
  int seg = kr.first / spseg, k0 = (kr.first - seg * spseg) * FTK;
  const size_t a0 = P::A_KC ? (size_t)m0 * p.lda : (size_t)m0, b0 = P::B_KC ? (size_t)n0 * p.ldb : (size_t)n0;
  const float* Aseg = p.a_seg(gi, seg) + a0;
  const float* Bseg = p.b_seg(gi, seg) + b0;
  const int last = kr.first + kr.count - 1;
  f32x4 ra[OA::NCH], rb[OB::NCH];
  auto fetch = [&](int s) {      // step s (absolute), then the cursor moves on
    oa.load(ra, Aseg + (P::A_KC ? (size_t)k0 : (size_t)k0 * p.lda), kseg - k0);
    ob.load(rb, Bseg + (P::B_KC ? (size_t)k0 : (size_t)k0 * p.ldb), kseg - k0);
    k0 += FTK;
    if (k0 >= kseg && s < last) {
      k0 = 0;
      ++seg;
      Aseg = p.a_seg(gi, seg) + a0;
      Bseg = p.b_seg(gi, seg) + b0;
    }
  };

  // sums over 128 k at a time, added up in `tot`: the rounding errors of a long K grow with the number of partial
  // sums and the length of one, not with K (K = 768: rms error 2.1e-7 instead of 5.0e-7 with one running sum)
  constexpr int STEPS_PER_SUM = 4;
  f32x4 acc[NB][NB], tot[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = tot[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto flush = [&]() {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) { tot[i][j][q] += acc[i][j][q]; acc[i][j][q] = 0.f; }
  };

  constexpr int STAGE = OA::LDS_FLOATS + OB::LDS_FLOATS;
  fetch(kr.first);
  oa.store(smem, ra);
  ob.store(smem + OA::LDS_FLOATS, rb);
  if (kr.count > 1) fetch(kr.first + 1);
  __syncthreads();
  // A K step: the MFMAs on the last four k of the step before (held back, their operands stay in registers) cover the latency
  // of the first fragment reads; the next tile goes to LDS and the one after it is fetched between the two slices, so
  // that only the barrier itself stands between two steps' MFMAs.  (With the stores right before the barrier and nothing
  // held back the matrix cores were busy 76 to 82 % of the time, at full clock; decode 6.19 -> 6.01 ms, dz 5.93 -> 5.60,
  // dW_dec 6.39 -> 6.21 at the sizes above.)
  constexpr int NSL = FTK / 16;
  static_assert(NSL == 2, "two slices");
  f32x4 fa[NSL][NB], fb[NSL][NB];
  auto mfma = [&](int sl, int q) {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[sl][j][q], fa[sl][i][q], acc[i][j], 0, 0, 0);
  };
  for (int kt = 0; kt < kr.count; ++kt) {
    const float* sa = smem + (kt & 1) * STAGE;
    const float* sb = sa + OA::LDS_FLOATS;
    auto read = [&](int sl) {
#pragma unroll
      for (int i = 0; i < NB; ++i) fa[sl][i] = OA::frag(sa, wm + 16 * i, sl, lane);
#pragma unroll
      for (int j = 0; j < NB; ++j) fb[sl][j] = OB::frag(sb, wn + 16 * j, sl, lane);
    };
    read(0);
    if (kt > 0) mfma(1, 3);
    if (!P::IN_ORDER && (kt & (STEPS_PER_SUM - 1)) == 0) flush();
    read(1);
#pragma unroll
    for (int q = 0; q < 4; ++q) mfma(0, q);
    // the other stage was last read before the barrier that ended the previous step
    if (kt + 1 < kr.count) {
      float* s = smem + ((kt + 1) & 1) * STAGE;
      oa.store(s, ra);
      ob.store(s + OA::LDS_FLOATS, rb);
      if (kt + 2 < kr.count) fetch(kr.first + kt + 2);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) mfma(1, q);
    __syncthreads();
  }
  if (kr.count > 0) mfma(1, 3);

  flush();
  // a lane's four columns of block j and row lane % 16 of block i
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    typename P::Epi est;
    EpiPos pos{m0 + wm, n0 + wn + 16 * j, lane & 15, 4 * (lane >> 4)};
    const bool col_ok = pos.col() < N;
    p.epi_begin(est, gi, pos.col(), col_ok, m0 + wm, 0);
    typename P::EpiRegs er[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      pos.ru = m0 + wm + 16 * i;
      if (col_ok && pos.row() < M) p.epi_load(er[i], gi, pos);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      pos.ru = m0 + wm + 16 * i;
      const f32x4 v = tot[i][j];
      if (col_ok && pos.row() < M) p.epi4(est, gi, pos, make_float4(v[0], v[1], v[2], v[3]), er[i]);
    }
    p.epi_end(est, gi, nullptr);
  }
}

constexpr int CUS = 256;      // a literal like the one in few_rows

template <class P>
hipError_t launch(hipStream_t s, const P& p, int G, int tile = 0) {
  const TileGrid big = TileGrid::make(G, p.M, p.N, 128, 128);
  // 128x128 tiles read each operand half as often, 64x64 tiles fill the chip at a quarter of the size: the small
  // tile where the large one leaves half of the two workgroups per CU without work
  if (tile ? tile == 128 : (long)big.mt * big.nt * G >= CUS) {
    hipLaunchKernelGGL((gemm_f32_kernel<P, 128>), dim3(big.num_wg()), dim3(256), 0, s, p, big);
  } else {
    const TileGrid tg = TileGrid::make(G, p.M, p.N, 64, 64);
    hipLaunchKernelGGL((gemm_f32_kernel<P, 64>), dim3(tg.num_wg()), dim3(256), 0, s, p, tg);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_enc_f32(hipStream_t s, Dims D, const EncArgs& a) {
  EncPolicy<float> p{D, D.B, D.F, D.d, D.d, D.F,
                     (const float*)a.x, (const float*)a.W_enc, a.b_enc, a.theta, nullptr,
                     0.5f * a.ste_eps, (float*)a.z, (float*)a.pre, a.cls, a.l0, a.log_threshold, a.pre32};
  return launch(s, p, D.L);
}
// The tile that the decode is cut for: with less than 32 of the large tile's K steps per CU there is too little work to
// share out in large tiles.
static int dec_tile(Dims D) {
  const double steps = (double)D.P() * ((D.F + FTK - 1) / FTK) * ((D.B + 127) / 128) * ((D.d + 127) / 128);
  return steps >= 32.0 * CUS ? 128 : 64;
}
DecSplit dec_split_f32(Dims D) {
  const int T = dec_tile(D);
  return choose_dec_split(D, T, T, FTK, (T == 128 ? 2 : 4) * CUS / 8, T == 128 ? 3.4 : 1.0);
}
hipError_t launch_dec_f32(hipStream_t s, Dims D, const DecArgs& a) {
  if (a.split.groups > 0) {
    DecPolicy<float, true> p{D, D.B, D.d, D.F, D.F, D.d, (const float*)a.z, (const float*)a.W_dec, a.b_dec, a.y_hat, a.skip_flags,
                             a.kcap, nullptr, a.split, a.split_part, nullptr};
    const hipError_t e = launch(s, p, a.split.groups, dec_tile(D));
    return e != hipSuccess ? e : launch_decode_combine(s, D, a.split, a.split_part, a.b_dec, a.y_hat, a.skip_flags, a.kcap);
  }
  DecPolicy<float> p{D, D.B, D.d, D.F, D.F, D.d, (const float*)a.z, (const float*)a.W_dec, a.b_dec, a.y_hat, a.skip_flags, a.kcap,
                     nullptr, a.split, nullptr, nullptr};
  return launch(s, p, D.L);
}
hipError_t launch_dz_f32(hipStream_t s, Dims D, const DzArgs& a) {
  DzPolicy<float> p{D, D.B, D.F, D.d, D.d, D.d,
                    (const float*)a.d_yhat, (const float*)a.W_dec, (const float*)a.z, a.cls, a.norms,
                    a.lam_c_over_b, a.C, (float*)a.dpre, a.lam1_over_b, a.skip_flags, a.kcap,
                    nullptr, nullptr, nullptr, nullptr};
  return launch(s, p, D.L);
}
template <bool ADAM>
static hipError_t launch_dwdec_mode(hipStream_t s, Dims D, const DWdecArgs& a) {
  DWdecPolicy<float, ADAM> p{D, D.F, D.d, D.B, D.F, D.d,
                             (const float*)a.z, (const float*)a.d_yhat, (float*)a.W_dec, a.G, a.norms,
                             (float*)a.dW_dec, AdamFuse{a.fuse.m, a.fuse.v, a.fuse.master, a.fuse.a}, a.skip_flags, a.kcap, 0, nullptr};
  // launches of whole source layers, like the bf16 path, each of at least 8 rounds of tiles for the chip (L = 4, d = 64,
  // F = 256, 128 tokens: one launch instead of four of 9 us)
  const long tiles = (long)((D.F + 127) / 128) * ((D.d + 127) / 128), want = 8L * 2 * CUS;
  for (int l = 0; l < D.L;) {
    int l1 = l;
    long blocks = 0;
    do { blocks += D.L - l1; ++l1; } while (l1 < D.L && blocks * tiles < want);
    p.p0 = packed_index(l, l, D.L);
    const hipError_t e = launch(s, p, (int)blocks);
    if (e != hipSuccess) return e;
    l = l1;
  }
  return hipSuccess;
}
hipError_t launch_dwdec_f32(hipStream_t s, Dims D, const DWdecArgs& a) {
  return a.fuse.m ? launch_dwdec_mode<true>(s, D, a) : launch_dwdec_mode<false>(s, D, a);
}
template <bool ADAM>
static hipError_t launch_dwenc_mode(hipStream_t s, Dims D, const DWencArgs& a) {
  DWencPolicy<float, ADAM> p{D, D.d, D.F, D.B, D.d, D.F, (const float*)a.x, (const float*)a.dpre, (float*)a.dW_enc,
                             (float*)a.W_enc, AdamFuse{a.fuse.m, a.fuse.v, a.fuse.master, a.fuse.a}};
  return launch(s, p, D.L);
}
hipError_t launch_dwenc_f32(hipStream_t s, Dims D, const DWencArgs& a) {
  return a.fuse.m ? launch_dwenc_mode<true>(s, D, a) : launch_dwenc_mode<false>(s, D, a);
}

}  // namespace clt
