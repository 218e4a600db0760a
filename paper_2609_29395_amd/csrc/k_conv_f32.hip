// fp32 convolutions on the bf16 matrix cores (gfx950).
//
// The fp32 MFMA (v_mfma_f32_16x16x4_f32) runs at 1/16 of the bf16 rate, so an
// fp32 product of the layers here was bound by the matrix cores at 80-90 of
// their 157 TFLOP/s.  An fp32 value is instead written exactly as the sum of
// three bf16 values,
//
//   x = h + m + l,  h = bf16(x), m = bf16(x - h), l = x - h - m
//
// (8 + 8 + 8 significant bits; each difference is exact, rounding to nearest
// leaves |m| <= 2^-8 |x| and |l| <= 2^-17 |x|), and a product x y is the six
// terms l h' + h l' + m m' + m h' + h m' + h h' on v_mfma_f32_16x16x32_bf16,
// accumulated in fp32.  The three terms left out, m l' + l m' + l l', reach
// 2^-24 |x y| at worst, the fp32 rounding of one product (what the sums are off
// as a whole: Sums below).  (Below 2^-110 the last parts run out of the bf16
// exponent range: absolute precision 2^-133.)
//
// Sums that are not finite: a NaN gives NaN in all six terms, as in fp32.
// But an infinity has no such split (inf - inf), a value within half a bf16
// spacing of FLT_MAX rounds to one, and terms of opposite sign may overflow
// here and not in the order of k.  So the staging threads keep the largest
// magnitude they split; where it is kHuge or more, a wave whose tile holds a
// sum that is not finite takes it again in plain fp32 (sum_* below), and
// infinities come out as fp32 arithmetic gives them.
//
// Tiles are staged per 32 k values: every thread loads fp32 values into
// registers one k step ahead, splits them and writes three bf16 planes, so an
// element is split once per workgroup and the fragment reads are plain
// 16-byte LDS reads.  One LDS buffer per workgroup: two or more workgroups
// share a CU and one's staging overlaps the other's MFMAs.
#include "runtime.h"

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// Two fp32 values -> their three bf16 parts, packed (a in the low half).
__device__ __forceinline__ void split2(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l) {
  h = pack2_bf16(a, b);
  a -= __uint_as_float(h << 16);
  b -= __uint_as_float(h & 0xffff0000u);
  m = pack2_bf16(a, b);
  a -= __uint_as_float(m << 16);
  b -= __uint_as_float(m & 0xffff0000u);
  l = pack2_bf16(a, b);
}

// Eight fp32 values -> three 16-byte vectors of bf16 parts (h, m, l); top: the
// largest magnitude so far (a NaN does not count).
__device__ __forceinline__ void split8(const float (&v)[8], uint4 (&p)[3], float &top) {
  uint32_t w[3][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    split2(v[2 * i], v[2 * i + 1], w[0][i], w[1][i], w[2][i]);
    top = fmaxf(fmaxf(top, fabsf(v[2 * i])), fabsf(v[2 * i + 1]));
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) p[k] = make_uint4(w[k][0], w[k][1], w[k][2], w[k][3]);
}

struct Frag3 {
  bf16x8_t p[3];
};

// Sums of a wave's outputs: of the h h' terms, and of the five small ones.
// An MFMA rounds its accumulator about once per 8 products, so all six terms
// on one accumulator would round it 24 times per 32 values: on ReLU outputs
// (half of them zeros, at which an fp32 FMA chain does not round) 1.15 times
// the fp32 MFMA's error.  With the small terms apart the large sum is rounded
// 4 times per 32 values: 0.4 to 0.5 of the fp32 MFMA's error, measured
// against 64 bits from 8 to 512 channels.
template <int TM, int TN> struct Sums {
  f32x4_t hh[TM][TN], lo[TM][TN];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) hh[i][j] = lo[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
  // [i][j0 + j] += a_i b_j over 32 k values, the smallest terms first
  template <int NB>
  __device__ __forceinline__ void add(const Frag3 (&a)[TM], const Frag3 (&b)[NB], int j0 = 0) {
    constexpr int pa[5] = {2, 0, 1, 1, 0}, pb[5] = {0, 2, 1, 0, 1};
#pragma unroll
    for (int t = 0; t < 5; ++t)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          lo[i][j0 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i].p[pa[t]], b[j].p[pb[t]], lo[i][j0 + j], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
        hh[i][j0 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i].p[0], b[j].p[0], hh[i][j0 + j], 0, 0, 0);
  }
  // hh: the whole sums
  __device__ __forceinline__ void finish() {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) hh[i][j] += lo[i][j];
  }
};

// Whether every accumulator of the wave is finite.
template <int TM, int TN> __device__ __forceinline__ bool all_finite(const f32x4_t (&acc)[TM][TN]) {
  float z = 0.f;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) z = fmaf(acc[i][j][r], 0.f, z);  // 0, or NaN from an infinity or NaN on
  return __ballot(z != 0.f) == 0;
}

// Whether a stored value is finite.
__device__ __forceinline__ bool finite(const float *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) * 0.f == 0.f;
}

// Below this no sum overflows: products stay below 2^100, and no sum has 2^27
// terms (a layer's tensors are below 2 GiB, so a weight gradient has at most
// 2^26 pixels of 8 channels; the others have 9 taps of fewer than 2^14 channels).
constexpr float kHuge = 0x1p50f;
constexpr int kHaloW = 32;  // widest image of the halo kernel
constexpr int kStep = 32;  // k values per stage

// ------------------------------------------------------ forward / dgrad
// Rows of a plane: 32 bf16 (64 bytes) of one pixel or output channel, 16-byte
// chunk c at c ^ ((row >> 1) & 3), so that 8 consecutive lanes of a write
// (two rows) and of a fragment read (8 rows, one chunk) use every bank once.
template <int ROWS> __device__ __forceinline__ int lds_at(int plane, int row, int chunk) {
  return (plane * ROWS + row) * 64 + ((chunk ^ ((row >> 1) & 3)) << 4);
}

// One output of the conv in plain fp32 (k ascending, padding as zeros): m's
// pixel (b, h, w), output channel n.  (Only values that are not finite are
// taken again, and a sum ends at the first NaN, which stays one: a network that
// has diverged takes every round this way.  Narrow network, 10 replicas of 21
// examples: 4.42 ms a round with whole tiles of whole sums, 0.83 so.)
__device__ float sum_conv(const ConvArgs &a, const float *src, const float *wt, int b, int h, int w, int n) {
  float s = 0.f;
  const float *wr = wt + (int64_t)n * a.Kp;
  for (int rs = 0; rs < (a.taps == 1 ? 1 : 9); ++rs) {
    const int hh = h + (a.taps == 1 ? 0 : rs / 3 - 1), ww = w + (a.taps == 1 ? 0 : rs % 3 - 1);
    const bool in = (unsigned)hh < (unsigned)a.H && (unsigned)ww < (unsigned)a.W;
    const float *x = src + ((int64_t)(b * a.H + hh) * a.W + ww) * a.Csrc;
    for (int c = 0; c < a.Csrc; ++c) {
      s = fmaf(in ? x[c] : 0.f, wr[rs * a.Csrc + c], s);
      if (s != s) return s;
    }
  }
  return s;
}

// The same of a stride-2 input gradient: (b, h, w) the class's pixel on the
// output gradient's grid.
__device__ float sum_conv(const ConvArgs &a, const float *src, const float *wt, int b, int h, int w, int n,
                          const S2Class &cls) {
  float s = 0.f;
  for (int u = 0; u < cls.n; ++u) {
    const float *wr = wt + (int64_t)n * a.Kp + cls.wtap(u) * a.Csrc;
    const int hh = h + cls.di(u), ww = w + cls.dj(u);
    const bool in = hh < a.H && ww < a.W;
    const float *x = src + ((int64_t)(b * a.H + hh) * a.W + ww) * a.Csrc;
    for (int c = 0; c < a.Csrc; ++c) {
      s = fmaf(in ? x[c] : 0.f, wr[c], s);
      if (s != s) return s;
    }
  }
  return s;
}

// The tile's outputs from its sums: bias, residual, ReLU (forward) or
// residual and ReLU mask (input gradient).
template <int BM, int BN, int WM, int WN, int EPI, bool S2 = false>
__device__ __forceinline__ void conv_store(const ConvArgs &a, const f32x4_t (&acc)[BN / WN / 16][BM / WM / 16],
                                           const float *src, const float *wt, int rep, int m0, int n0, bool huge,
                                           const FastDiv &fd_w, const FastDiv &fd_h, const S2Class &cls = S2Class(0, 9)) {
  constexpr int TM = BM / WM / 16, TN = BN / WN / 16;
  // output pixel of the tile's pixel m (classes: on the doubled grid)
  auto opix = [&](int m) -> int64_t {
    if constexpr (!S2) return m;
    const int q1 = (int)fdiv((uint32_t)m, fd_w);
    return (int64_t)(2 * q1 + cls.y) * (2 * a.W) + 2 * (m - q1 * a.W) + cls.x;
  };
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, lg = lane >> 4;
  const int wm0 = (wave / WN) * (BM / WM), wn0 = (wave % WN) * (BN / WN);
  const int M = a.Bt * a.H * a.W;
  float *out = reinterpret_cast<float *>(a.out) + rep * a.out_rs;
  const float *res = a.res ? reinterpret_cast<const float *>(a.res) + rep * a.out_rs : nullptr;
  const float *msk = a.mask ? reinterpret_cast<const float *>(a.mask) + rep * a.out_rs : nullptr;
  const float *bias = EPI == EPI_FWD ? a.bias + rep * a.bias_rs : nullptr;
  // sums that are not finite where an operand is huge, one bit per value of the
  // lane: taken again in plain fp32 after the others are stored
  uint64_t again = 0;
  if (huge) {
    static_assert(TM * TN * 4 <= 64, "one bit per value");
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (!(acc[j][i][r] * 0.f == 0.f)) again |= 1ull << ((j * TM + i) * 4 + r);
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = n0 + wn0 + j * 16 + lg * 4;
    const bool nok = n < a.N;  // N is a multiple of 8
    f32x4_t bv = {0.f, 0.f, 0.f, 0.f};
    if (EPI == EPI_FWD && nok) {
#pragma unroll
      for (int r = 0; r < 4; ++r) bv[r] = bias[n + r];
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = m0 + wm0 + i * 16 + li;
      if (m >= M || !nok) continue;
      const int64_t o = opix(m) * a.N + n;
      f32x4_t v = acc[j][i];
      f32x4_t rv = {0.f, 0.f, 0.f, 0.f};
      if (res) rv = *reinterpret_cast<const f32x4_t *>(res + o);
      if constexpr (EPI == EPI_FWD) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          v[r] += bv[r];
          if (res) v[r] += rv[r];
          if (!a.no_relu) v[r] = fmaxf(v[r], 0.f);
        }
      } else {
        f32x4_t mv = {1.f, 1.f, 1.f, 1.f};
        if (msk) mv = *reinterpret_cast<const f32x4_t *>(msk + o);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (res) v[r] += rv[r];
          if (!(mv[r] > 0.f)) v[r] = 0.f;
        }
      }
      *reinterpret_cast<f32x4_t *>(out + o) = v;
    }
  }
  for (; again; again &= again - 1) {
    const int bit = __ffsll((unsigned long long)again) - 1, ij = bit >> 2;
    const int m = m0 + wm0 + ij % TM * 16 + li, n = n0 + wn0 + ij / TM * 16 + lg * 4 + (bit & 3);
    if (m >= M || n >= a.N) continue;
    const uint32_t q = fdiv((uint32_t)m, fd_w), b = fdiv(q, fd_h);
    const int h = (int)(q - b * (uint32_t)a.H), w = (int)((uint32_t)m - q * (uint32_t)a.W);
    float v = S2 ? sum_conv(a, src, wt, (int)b, h, w, n, cls) : sum_conv(a, src, wt, (int)b, h, w, n);
    const int64_t o = opix(m) * a.N + n;
    if (EPI == EPI_FWD) v += bias[n];
    if (res) v += res[o];
    if (EPI == EPI_FWD && !a.no_relu) v = fmaxf(v, 0.f);
    if (EPI == EPI_DGRAD && msk && !(msk[o] > 0.f)) v = 0.f;
    out[o] = v;
  }
}

// BM pixels x BN output channels per workgroup, WM x WN waves.  The weights
// are the MFMA's first operand, so a lane ends with four consecutive channels
// of one pixel: 16-byte stores, residual and mask loads.  S2: the input gradient
// of a stride-2 conv by classes of input pixels (ConvArgs::stride2), the class
// of most taps first.
template <int BM, int BN, int WM, int WN, int EPI, int OCC, bool S2 = false>
__global__ void __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(OCC)))
conv_f32_kernel(ConvArgs a, FastDiv fd_w, FastDiv fd_h, FastDiv fd_c, int MT, int NT) {
  constexpr int NTH = 64 * WM * WN, TM = BM / WM / 16, TN = BN / WN / 16;
  constexpr int RP = NTH / 4;  // rows per staging pass (four 8-value chunks per row)
  constexpr int AV = (BM + RP - 1) / RP, BV = (BN + RP - 1) / RP;
  __shared__ __attribute__((aligned(16))) char Xs[3 * BM * 64];
  __shared__ __attribute__((aligned(16))) char Ws[3 * BN * 64];
  __shared__ int huge;

  const int tid = threadIdx.x;
  const uint32_t ntiles = (uint32_t)(MT * NT * a.C);
  const S2Class cls(S2 ? __builtin_amdgcn_readfirstlane((int)(blockIdx.x / ntiles)) : 0, a.taps);
  const uint32_t t = xcd_swizzle(S2 ? blockIdx.x % ntiles : blockIdx.x, ntiles);
  const int nt = __builtin_amdgcn_readfirstlane((int)(t % (uint32_t)NT));
  const uint32_t rest = t / (uint32_t)NT;
  const int mt = __builtin_amdgcn_readfirstlane((int)(rest % (uint32_t)MT));
  const int rep = replica_of(a.rmap, __builtin_amdgcn_readfirstlane((int)(rest / (uint32_t)MT)));
  const int M = a.Bt * a.H * a.W;
  const int m0 = mt * BM, n0 = nt * BN;
  const float *src = reinterpret_cast<const float *>(a.src) + rep * a.src_rs;
  const float *wt = reinterpret_cast<const float *>(a.wt) + rep * a.wt_rs;
  const __amdgpu_buffer_rsrc_t rsa = make_rsrc(src, (uint32_t)(a.src_rs * 4));
  const __amdgpu_buffer_rsrc_t rsb = make_rsrc(wt, (uint32_t)((int64_t)a.N * a.Kp * 4));

  const int chunk = tid & 3, rrow = tid >> 2;
  // byte offset of each staged pixel row's centre pixel and the mask of
  // kernel taps inside its image (taps 1: the centre tap); weight rows
  uint32_t rowoff[AV], tapmask[AV], offb[BV];
#pragma unroll
  for (int j = 0; j < AV; ++j) {
    const int row = rrow + RP * j, m = m0 + row;
    const bool ok = m < M && row < BM;
    const uint32_t mm = ok ? (uint32_t)m : 0u;
    const uint32_t q = fdiv(mm, fd_w);
    const int w = (int)(mm - q * (uint32_t)a.W), h = (int)(q - fdiv(q, fd_h) * (uint32_t)a.H);
    uint32_t mk = 0;
#pragma unroll
    for (int rs = 0; rs < 9; ++rs) {
      const int hh = h + rs / 3 - 1, ww = w + rs % 3 - 1;
      if ((unsigned)hh < (unsigned)a.H && (unsigned)ww < (unsigned)a.W) mk |= 1u << rs;
    }
    rowoff[j] = mm * (uint32_t)a.Csrc * 4u;
    tapmask[j] = ok ? mk : 0u;
  }
#pragma unroll
  for (int j = 0; j < BV; ++j) {
    const int row = rrow + RP * j, n = n0 + row;
    offb[j] = (n < a.N && row < BN) ? ((uint32_t)n * (uint32_t)a.Kp + (uint32_t)(chunk * 8)) * 4u : kOob;
  }

  const int K = S2 ? cls.n * a.Csrc : a.K;
  float top = 0.f;
  uint4 ra[AV][2], rb[BV][2];
  auto load = [&](int kt) {
    const int k0 = kt * kStep + chunk * 8;
    // tap and channel of the thread's 8 values (channels come in multiples of
    // 8 with 9 taps; im2col rows: multiples of 4, checked per 4 values)
    int rs = !S2 && a.taps == 1 ? 4 : (int)fdiv((uint32_t)k0, fd_c);
    const int c = k0 - (!S2 && a.taps == 1 ? 0 : rs * a.Csrc);
    int kw = k0;  // weight column
    if constexpr (S2) {
      kw = cls.wtap(rs) * a.Csrc + c;
      rs = 4 + 3 * cls.di(rs) + cls.dj(rs);
    }
    const int r = (rs * 11) >> 5;  // rs / 3 for rs < 9
    const uint32_t tap = (uint32_t)((((r - 1) * a.W + (rs - 3 * r - 1)) * a.Csrc + c) * 4);
    const bool live0 = k0 < K, live1 = k0 + 4 < K;  // (past the last stage: nothing is read)
#pragma unroll
    for (int j = 0; j < AV; ++j) {
      const bool in = ((tapmask[j] >> (rs & 31)) & 1u) != 0u;
      ra[j][0] = buffer_load16(rsa, in && live0 ? rowoff[j] + tap : kOob);
      ra[j][1] = buffer_load16(rsa, in && live1 ? rowoff[j] + tap + 16u : kOob);
    }
#pragma unroll
    for (int j = 0; j < BV; ++j) {
      const uint32_t o = S2 ? (k0 < K ? offb[j] + (uint32_t)((kw - chunk * 8) * 4) : kOob)
                            : k0 < a.Kp ? offb[j] + (uint32_t)(kt * kStep * 4) : kOob;
      rb[j][0] = buffer_load16(rsb, o);
      rb[j][1] = buffer_load16(rsb, o + 16u);
    }
  };
  auto stage = [&]() {
    auto put = [&](char *dst, const uint4 (&q)[2], auto at) {
      const float v[8] = {__uint_as_float(q[0].x), __uint_as_float(q[0].y), __uint_as_float(q[0].z),
                          __uint_as_float(q[0].w), __uint_as_float(q[1].x), __uint_as_float(q[1].y),
                          __uint_as_float(q[1].z), __uint_as_float(q[1].w)};
      uint4 p[3];
      split8(v, p, top);
#pragma unroll
      for (int k = 0; k < 3; ++k) *reinterpret_cast<uint4 *>(dst + at(k)) = p[k];
    };
#pragma unroll
    for (int j = 0; j < AV; ++j) {
      const int row = rrow + RP * j;
      if (BM % RP == 0 || row < BM) put(Xs, ra[j], [&](int k) { return lds_at<BM>(k, row, chunk); });
    }
#pragma unroll
    for (int j = 0; j < BV; ++j) {
      const int row = rrow + RP * j;
      if (BN % RP == 0 || row < BN) put(Ws, rb[j], [&](int k) { return lds_at<BN>(k, row, chunk); });
    }
  };

  const int lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lg = lane >> 4;
  const int wm0 = (wave / WN) * (BM / WM), wn0 = (wave % WN) * (BN / WN);
  Sums<TN, TM> sums;
  sums.clear();

  const int nk = (K + kStep - 1) / kStep;
  if (tid == 0) huge = 0;
  load(0);
  for (int kt = 0; kt < nk; ++kt) {
    stage();
    __syncthreads();
    load(kt + 1);
    Frag3 x[TM], w[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int k = 0; k < 3; ++k)
        x[i].p[k] = *reinterpret_cast<const bf16x8_t *>(Xs + lds_at<BM>(k, wm0 + i * 16 + li, lg));
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int k = 0; k < 3; ++k)
        w[j].p[k] = *reinterpret_cast<const bf16x8_t *>(Ws + lds_at<BN>(k, wn0 + j * 16 + li, lg));
    sums.add(w, x);
    __syncthreads();
  }

  if (top >= kHuge) huge = 1;
  sums.finish();
  __syncthreads();
  conv_store<BM, BN, WM, WN, EPI, S2>(a, sums.hh, src, wt, rep, m0, n0, huge != 0, fd_w, fd_h, cls);
}

// The same contraction for 3 x 3 convs whose input channels fill 32-channel
// blocks: per block, the BM + 2 W + 2 pixels that all nine taps of the tile
// read (rows of 32 channels, by flat pixel index) are staged and split once,
// and tap (r, s) reads its fragments r W + s rows further; a lane whose tap
// leaves the image reads a row of zeros instead.  The pixels' share of the
// splitting falls from nine times per block to about once and a half, so the
// stages are the weights' (one tap of the block each).  A tap's weights are
// loaded RD taps ahead (a ring of registers) and staged in two LDS buffers, one
// barrier per tap: a tap of a small tile is 12 or 24 MFMAs of a wave, far less
// than a load's latency, so the smaller tiles take RD = 3; the 256-pixel ones
// have no registers for it.
template <int BM, int BN, int WM, int WN, int EPI, int OCC, int RD>
__global__ void __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(OCC)))
conv_f32_halo_kernel(ConvArgs a, FastDiv fd_w, FastDiv fd_h, int MT, int NT) {
  constexpr int NTH = 64 * WM * WN, TM = BM / WM / 16, TN = BN / WN / 16;
  constexpr int HR = BM + 2 * kHaloW + 2;  // halo rows, at most; row HR holds zeros
  constexpr int RP = NTH / 4;
  constexpr int HV = (HR + RP - 1) / RP, BV = (BN + RP - 1) / RP;
  __shared__ __attribute__((aligned(16))) char Xs[3 * (HR + 1) * 64];
  __shared__ __attribute__((aligned(16))) char Ws[2][3 * BN * 64];
  __shared__ int huge;

  const int tid = threadIdx.x;
  const uint32_t t = xcd_swizzle(blockIdx.x, (uint32_t)(MT * NT * a.C));
  const int nt = __builtin_amdgcn_readfirstlane((int)(t % (uint32_t)NT));
  const uint32_t rest = t / (uint32_t)NT;
  const int mt = __builtin_amdgcn_readfirstlane((int)(rest % (uint32_t)MT));
  const int rep = replica_of(a.rmap, __builtin_amdgcn_readfirstlane((int)(rest / (uint32_t)MT)));
  const int M = a.Bt * a.H * a.W;
  const int m0 = mt * BM, n0 = nt * BN;
  const float *src = reinterpret_cast<const float *>(a.src) + rep * a.src_rs;
  const float *wt = reinterpret_cast<const float *>(a.wt) + rep * a.wt_rs;
  const __amdgpu_buffer_rsrc_t rsa = make_rsrc(src, (uint32_t)(a.src_rs * 4));
  const __amdgpu_buffer_rsrc_t rsb = make_rsrc(wt, (uint32_t)((int64_t)a.N * a.Kp * 4));

  const int chunk = tid & 3, rrow = tid >> 2;
  const int rows = BM + 2 * a.W + 2;  // halo rows of this width (later passes are skipped)
  uint32_t offx[HV], offb[BV];
#pragma unroll
  for (int j = 0; j < HV; ++j) {
    const int row = rrow + RP * j, p = m0 - a.W - 1 + row;
    offx[j] = (row < rows && p >= 0 && p < M) ? ((uint32_t)p * (uint32_t)a.Csrc + (uint32_t)(chunk * 8)) * 4u
                                                          : kOob;
  }
#pragma unroll
  for (int j = 0; j < BV; ++j) {
    const int row = rrow + RP * j, n = n0 + row;
    offb[j] = (n < a.N && row < BN) ? ((uint32_t)n * (uint32_t)a.Kp + (uint32_t)(chunk * 8)) * 4u : kOob;
  }
  float top = 0.f;
  uint4 rx[HV][2], rb[RD][BV][2];  // rb[s]: the weights of tap s of the next RD
  static_assert(9 % RD == 0, "ring");
  auto load_halo = [&](int c0) {
    const bool live = c0 + chunk * 8 < a.Csrc;  // channels come in multiples of 8
#pragma unroll
    for (int j = 0; j < HV; ++j) {
      if (RP * j >= rows) break;
      const uint32_t o = live ? offx[j] + (uint32_t)(c0 * 4) : kOob;
      rx[j][0] = buffer_load16(rsa, o);
      rx[j][1] = buffer_load16(rsa, o + 16u);
    }
  };
  auto load_w = [&](uint4 (&q)[BV][2], int c0, int rs) {
    const bool live = c0 + chunk * 8 < a.Csrc;
#pragma unroll
    for (int j = 0; j < BV; ++j) {
      const uint32_t o = live ? offb[j] + (uint32_t)((rs * a.Csrc + c0) * 4) : kOob;
      q[j][0] = buffer_load16(rsb, o);
      q[j][1] = buffer_load16(rsb, o + 16u);
    }
  };
  auto put = [&](char *dst, const uint4 (&q)[2], auto at) {
    const float v[8] = {__uint_as_float(q[0].x), __uint_as_float(q[0].y), __uint_as_float(q[0].z),
                        __uint_as_float(q[0].w), __uint_as_float(q[1].x), __uint_as_float(q[1].y),
                        __uint_as_float(q[1].z), __uint_as_float(q[1].w)};
    uint4 p[3];
    split8(v, p, top);
#pragma unroll
    for (int k = 0; k < 3; ++k) *reinterpret_cast<uint4 *>(dst + at(k)) = p[k];
  };

  const int lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lg = lane >> 4;
  const int wm0 = (wave / WN) * (BM / WM), wn0 = (wave % WN) * (BN / WN);
  uint32_t tapmask[TM];  // taps inside the image, of this lane's pixel of each fragment
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m0 + wm0 + i * 16 + li;
    const uint32_t mm = m < M ? (uint32_t)m : 0u, q = fdiv(mm, fd_w);
    const int w = (int)(mm - q * (uint32_t)a.W), h = (int)(q - fdiv(q, fd_h) * (uint32_t)a.H);
    uint32_t mk = 0;
#pragma unroll
    for (int rs = 0; rs < 9; ++rs) {
      const int hh = h + rs / 3 - 1, ww = w + rs % 3 - 1;
      if ((unsigned)hh < (unsigned)a.H && (unsigned)ww < (unsigned)a.W) mk |= 1u << rs;
    }
    tapmask[i] = m < M ? mk : 0u;
  }
  Sums<TN, TM> sums;
  sums.clear();

  if (tid == 0) huge = 0;
  if (tid < 12) *reinterpret_cast<uint4 *>(Xs + lds_at<HR + 1>(tid >> 2, HR, tid & 3)) = make_uint4(0, 0, 0, 0);
  const int ncb = (a.Csrc + 31) / 32;
  load_halo(0);
#pragma unroll
  for (int s = 0; s < RD; ++s) load_w(rb[s], 0, s);
  int buf = 0;
  for (int cb = 0; cb < ncb; ++cb) {
    if (cb) __syncthreads();  // every wave has read the block before
#pragma unroll
    for (int j = 0; j < HV; ++j) {
      const int row = rrow + RP * j;
      if (RP * j >= rows) break;
      if (HR % RP == 0 || row < HR) put(Xs, rx[j], [&](int k) { return lds_at<HR + 1>(k, row, chunk); });
    }
#pragma unroll 1
    for (int t0 = 0; t0 < 9; t0 += RD)
#pragma unroll
    for (int s = 0; s < RD; ++s) {
      const int rs = t0 + s;
      char *wb = Ws[buf];
      buf ^= 1;
#pragma unroll
      for (int j = 0; j < BV; ++j) {
        const int row = rrow + RP * j;
        if (BN % RP == 0 || row < BN) put(wb, rb[s][j], [&](int k) { return lds_at<BN>(k, row, chunk); });
      }
      // (the other buffer's readers have passed this barrier before it is
      // written again)
      __syncthreads();
      if (rs == 6) load_halo((cb + 1) * 32);  // (past the last block: nothing is read)
      load_w(rb[s], rs < 9 - RD ? cb * 32 : cb * 32 + 32, rs < 9 - RD ? rs + RD : rs + RD - 9);
      const int r = (rs * 11) >> 5, shift = r * a.W + rs - 3 * r;
      const int row0 = wm0 + li + shift;
      const int at0 = lds_at<HR + 1>(0, row0, lg), zero = lds_at<HR + 1>(0, HR, lg);
      Frag3 w[TN];
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int k = 0; k < 3; ++k)
          w[j].p[k] = *reinterpret_cast<const bf16x8_t *>(wb + lds_at<BN>(k, wn0 + j * 16 + li, lg));
      // pixel fragments two at a time (fewer registers; the other waves cover the reads)
      constexpr int XB = TM > 2 ? 2 : TM;
#pragma unroll
      for (int i0 = 0; i0 < TM; i0 += XB) {
        Frag3 x[XB];
#pragma unroll
        for (int i = 0; i < XB; ++i) {
          const int at = (tapmask[i0 + i] >> rs) & 1u ? at0 + (i0 + i) * 16 * 64 : zero;
#pragma unroll
          for (int k = 0; k < 3; ++k) x[i].p[k] = *reinterpret_cast<const bf16x8_t *>(Xs + at + k * (HR + 1) * 64);
        }
        sums.add(w, x, i0);
        if (i0 + XB < TM) __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  if (top >= kHuge) huge = 1;
  sums.finish();
  __syncthreads();
  conv_store<BM, BN, WM, WN, EPI>(a, sums.hh, src, wt, rep, m0, n0, huge != 0, fd_w, fd_h);
}
// --------------------------------------------------------------- wgrad
// Rows of a plane: 32 pixels (64 bytes) of one channel, 80 bytes apart: 8
// consecutive lanes of a write (four pixel chunks of two rows four apart) and
// of a fragment read (8 rows, one chunk) use every bank once.
constexpr int kRow = 80;
template <int ROWS> __device__ __forceinline__ int wlds_at(int plane, int row, int chunk) {
  return (plane * ROWS + row) * kRow + (chunk << 4);
}

// One weight gradient in plain fp32 (pixels ascending, padding as zeros) over
// [p_begin, p_end).
__device__ float sum_wgrad(const WgradArgs &a, const float *G, const float *X, int co, int kk, int p_begin, int p_end,
                           const FastDiv &fd_w, const FastDiv &fd_h) {
  const int rs = a.taps == 1 ? 4 : kk / a.Ci, c = a.taps == 1 ? kk : kk - rs * a.Ci;
  float s = 0.f;
  for (int p = p_begin; p < p_end; ++p) {
    const uint32_t q = fdiv((uint32_t)p, fd_w), b = fdiv(q, fd_h);
    const int hh = (int)(q - b * (uint32_t)a.H) + rs / 3 - 1, ww = (int)((uint32_t)p - q * (uint32_t)a.W) + rs % 3 - 1;
    const bool in = (unsigned)hh < (unsigned)a.H && (unsigned)ww < (unsigned)a.W;
    s = fmaf(G[(int64_t)p * a.Co + co], in ? X[((int64_t)((int)b * a.H + hh) * a.W + ww) * a.Ci + c] : 0.f, s);
    if (s != s) return s;
  }
  return s;
}

// BM output channels x BN columns (r, s, ci) per workgroup over a chunk of
// pixels, 32 per stage.  A thread stages 8 pixels x 4 channels of one operand
// (eight 16-byte loads): transposed in registers, split, written as 16-byte
// runs of 8 pixels.  Any image width: a block's pixels step (w, h, b).
template <int BM, int BN, int WM, int WN, int OCC>
__global__ void __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(OCC)))
wgrad_f32_kernel(WgradArgs a, FastDiv fd_w, FastDiv fd_h, FastDiv fd_c, int MT, int NT) {
  constexpr int NTH = 64 * WM * WN, TM = BM / WM / 16, TN = BN / WN / 16;
  static_assert(BM + BN <= NTH, "one staging task per thread");
  __shared__ __attribute__((aligned(16))) char Gs[3 * BM * kRow];
  __shared__ __attribute__((aligned(16))) char Xs[3 * BN * kRow];
  __shared__ float red[4][BM];
  __shared__ int huge;

  const int tid = threadIdx.x;
  const uint32_t t = xcd_swizzle(blockIdx.x, (uint32_t)(MT * NT * a.splits * a.C));
  const int nt = __builtin_amdgcn_readfirstlane((int)(t % (uint32_t)NT));
  uint32_t rest = t / (uint32_t)NT;
  const int mt = __builtin_amdgcn_readfirstlane((int)(rest % (uint32_t)MT));
  rest /= (uint32_t)MT;
  const int split = __builtin_amdgcn_readfirstlane((int)(rest % (uint32_t)a.splits));
  const int rep = replica_of(a.rmap, __builtin_amdgcn_readfirstlane((int)(rest / (uint32_t)a.splits)));
  const int M = a.Bt * a.H * a.W;
  const int NW = a.taps == 1 ? a.Ci : 9 * a.Ci;
  const int p_begin = split * a.chunk, p_end = min(M, p_begin + a.chunk);
  const int nk = (p_end - p_begin + kStep - 1) / kStep;
  const int m0 = mt * BM, n0 = nt * BN;
  const float *G = reinterpret_cast<const float *>(a.g) + rep * a.g_rs;
  const float *X = reinterpret_cast<const float *>(a.x) + rep * a.x_rs;
  const bool do_bias = nt == 0 && a.db != nullptr;
  const __amdgpu_buffer_rsrc_t rsg = make_rsrc(G, (uint32_t)((int64_t)M * a.Co * 4));
  const __amdgpu_buffer_rsrc_t rsx = make_rsrc(X, (uint32_t)((int64_t)M * a.Ci * 4));

  // this thread's task: pixels 8 pc .. 8 pc + 7 of a stage, rows row .. row + 3
  const bool is_g = tid < BM, is_x = !is_g && tid < BM + BN;
  const int task = is_g ? tid : tid - BM;
  const int pc = task & 3, row = (task >> 2) << 2;
  const int kk = n0 + row;
  const int rs = a.taps == 1 || !is_x ? 4 : (int)fdiv((uint32_t)kk, fd_c);
  const int dr = ((rs * 11) >> 5) - 1, ds = rs - 3 * (dr + 1) - 1;
  const bool live = is_g ? m0 + row < a.Co : is_x && kk < NW;
  const int ch = is_g ? m0 + row : a.taps == 1 ? kk : kk - rs * a.Ci;  // first of the 4 channels
  const int stride = is_g ? a.Co : a.Ci;
  const int shift = is_g ? 0 : dr * a.W + ds;  // tap, in pixels

  float top = 0.f;
  uint4 reg[8];
  auto load = [&](int kt) {
    const int p0 = p_begin + kt * kStep + pc * 8;
    const uint32_t base = (uint32_t)((p0 + shift) * stride + ch) * 4u;
    const uint32_t step = (uint32_t)stride * 4u;
    if (is_g) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        reg[e] = buffer_load16(rsg, live && p0 + e < p_end ? base + (uint32_t)e * step : kOob);
    } else if (is_x) {
      const uint32_t q = fdiv((uint32_t)p0, fd_w);
      int w = (int)((uint32_t)p0 - q * (uint32_t)a.W), h = (int)(q - fdiv(q, fd_h) * (uint32_t)a.H);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bool ok = live && p0 + e < p_end && (unsigned)(h + dr) < (unsigned)a.H && (unsigned)(w + ds) < (unsigned)a.W;
        reg[e] = buffer_load16(rsx, ok ? base + (uint32_t)e * step : kOob);
        const bool wrap = ++w == a.W;
        w = wrap ? 0 : w;
        h += wrap ? 1 : 0;
        h = h == a.H ? 0 : h;
      }
    }
  };
  float bsum[4] = {0.f, 0.f, 0.f, 0.f};
  auto stage = [&]() {
    if (!is_g && !is_x) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e)
        v[e] = __uint_as_float(q == 0 ? reg[e].x : q == 1 ? reg[e].y : q == 2 ? reg[e].z : reg[e].w);
      if (do_bias && is_g) {
#pragma unroll
        for (int e = 0; e < 8; ++e) bsum[q] += v[e];
      }
      uint4 p[3];
      split8(v, p, top);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        if (is_g)
          *reinterpret_cast<uint4 *>(Gs + wlds_at<BM>(k, row + q, pc)) = p[k];
        else
          *reinterpret_cast<uint4 *>(Xs + wlds_at<BN>(k, row + q, pc)) = p[k];
      }
    }
  };

  const int lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lg = lane >> 4;
  const int wm0 = (wave / WN) * (BM / WM), wn0 = (wave % WN) * (BN / WN);
  Sums<TM, TN> sums;
  sums.clear();
  if (tid == 0) huge = 0;
  if (nk > 0) load(0);
  for (int kt = 0; kt < nk; ++kt) {
    stage();
    __syncthreads();
    load(kt + 1);
    Frag3 g[TM], x[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int k = 0; k < 3; ++k)
        g[i].p[k] = *reinterpret_cast<const bf16x8_t *>(Gs + wlds_at<BM>(k, wm0 + i * 16 + li, lg));
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int k = 0; k < 3; ++k)
        x[j].p[k] = *reinterpret_cast<const bf16x8_t *>(Xs + wlds_at<BN>(k, wn0 + j * 16 + li, lg));
    sums.add(g, x);
    __syncthreads();
  }

  if (top >= kHuge) huge = 1;
  sums.finish();
  __syncthreads();
  float *dw = a.dw + split * a.dw_ss + rep * a.dw_rs;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = n0 + wn0 + j * 16 + li;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm0 + i * 16 + lg * 4 + r;
        if (m < a.Co && n < a.nw) dw[(int64_t)m * a.nw + n] = sums.hh[i][j][r];
      }
  }
  if (huge && !all_finite(sums.hh)) {
    __threadfence_block();  // the wave's own stores, read by other lanes of it
    for (int e = lane; e < (BM / WM) * (BN / WN); e += 64) {
      const int m = m0 + wm0 + e / (BN / WN), n = n0 + wn0 + e % (BN / WN);
      if (m < a.Co && n < a.nw && !finite(dw + (int64_t)m * a.nw + n))
        dw[(int64_t)m * a.nw + n] = sum_wgrad(a, G, X, m, n, p_begin, p_end, fd_w, fd_h);
    }
  }

  if (do_bias) {
    if (is_g) {
#pragma unroll
      for (int q = 0; q < 4; ++q) red[pc][row + q] = bsum[q];
    }
    __syncthreads();
    if (tid < BM && m0 + tid < a.Co)
      a.db[split * a.db_ss + rep * a.db_rs + m0 + tid] = ((red[0][tid] + red[1][tid]) + red[2][tid]) + red[3][tid];
  }
}

// The same contraction for layers whose channels fill 64 x 32 blocks: 64
// output channels x one 32-channel input block x all nine taps (64 x 288
// outputs) per workgroup of 4 waves (32 output x 16 input channels x 9 taps
// each).  Both operands stay pixel-major in LDS and are read with the
// transposing LDS read; a tap reads its pixels r W + s rows further, so a
// pixel is staged and split once for nine taps.  Input rows live in a ring of
// 128 (pixel u of the chunk, counted from W + 1 before its first, in row
// u mod 128): a stage adds the 32 that the next 32 output pixels reach.  A
// lane whose tap leaves the image reads a row of zeros.
//
// An operand element is split once per 108 MFMAs of its 32 pixels where the
// 128 x 128 tile above splits it per 96 MFMAs of a tap: 90 against 133 us on
// 128 -> 128 at 16 x 16 (4 replicas of 64 examples; the fp32 MFMA kernel 230).
namespace wh {
constexpr int RING = 128, XROW = 64, GROW = 128;  // ring rows; bytes of an x and a g row (32, 64 channels)
constexpr int XPL = (RING + 1) * XROW, GPL = kStep * GROW;  // bytes of a plane
constexpr int ZERO = RING * XROW;
// 16-byte chunk c of ring row `row`: the four rows that 16 lanes of a
// transposing read take (32 bytes each) and the four rows 8 further, which
// the next 16 lanes take, fall on distinct banks.
__device__ __forceinline__ int x_at(int row, int c) { return row * XROW + ((c ^ ((row >> 2) & 2)) << 4); }
__device__ __forceinline__ int g_at(int row, int c) {
  return row * GROW + ((c ^ ((row & 2) | ((row >> 1) & 4))) << 4);
}
}  // namespace wh

typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8_t read_tr(const char *lo, const char *hi) {
  typedef __attribute__((address_space(3))) s16x4_t *lds_t;
  const bf16x4_t a = __builtin_bit_cast(bf16x4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)lo));
  const bf16x4_t b = __builtin_bit_cast(bf16x4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)hi));
  return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
wgrad_f32_halo_kernel(WgradArgs a, FastDiv fd_w, FastDiv fd_h, int MT, int NT) {
  using namespace wh;
  __shared__ __attribute__((aligned(16))) char Xs[3 * XPL];
  __shared__ __attribute__((aligned(16))) char Gs[3 * GPL];
  __shared__ int huge;
  static_assert(sizeof(Xs) >= 32 * 64 * sizeof(float), "bias sums reuse the ring");

  const int tid = threadIdx.x;
  const uint32_t t = xcd_swizzle(blockIdx.x, (uint32_t)(MT * NT * a.splits * a.C));
  const int nt = __builtin_amdgcn_readfirstlane((int)(t % (uint32_t)NT));
  uint32_t rest = t / (uint32_t)NT;
  const int mt = __builtin_amdgcn_readfirstlane((int)(rest % (uint32_t)MT));
  rest /= (uint32_t)MT;
  const int split = __builtin_amdgcn_readfirstlane((int)(rest % (uint32_t)a.splits));
  const int rep = replica_of(a.rmap, __builtin_amdgcn_readfirstlane((int)(rest / (uint32_t)a.splits)));
  const int M = a.Bt * a.H * a.W, W = a.W;
  const int p_begin = split * a.chunk, p_end = min(M, p_begin + a.chunk);
  const int nk = (p_end - p_begin + kStep - 1) / kStep;
  const int m0 = mt * 64, n0 = nt * 32;
  const float *G = reinterpret_cast<const float *>(a.g) + rep * a.g_rs;
  const float *X = reinterpret_cast<const float *>(a.x) + rep * a.x_rs;
  const bool do_bias = nt == 0 && a.db != nullptr;
  const __amdgpu_buffer_rsrc_t rsg = make_rsrc(G, (uint32_t)((int64_t)M * a.Co * 4));
  const __amdgpu_buffer_rsrc_t rsx = make_rsrc(X, (uint32_t)((int64_t)M * a.Ci * 4));

  // staging: g pixel tid / 8 of a stage, channels 8 (tid mod 8) on; the ring
  // rows 64 at a time (prologue) or 32 (stages: the first 128 threads),
  // channels 8 (tid mod 4) on
  const int gpx = tid >> 3, gc = tid & 7, xr = tid >> 2, xc = tid & 3;
  const bool glive = m0 + gc * 8 < a.Co, xlive = n0 + xc * 8 < a.Ci;  // channels come in multiples of 8
  float top = 0.f;
  uint4 rg[2], rx[2];
  auto load_g = [&](int kt) {
    const int p = p_begin + kt * kStep + gpx;
    const uint32_t o = glive && p < p_end ? ((uint32_t)p * (uint32_t)a.Co + (uint32_t)(m0 + gc * 8)) * 4u : kOob;
    rg[0] = buffer_load16(rsg, o);
    rg[1] = buffer_load16(rsg, o + 16u);
  };
  auto load_x = [&](int u) {  // ring row u + xr
    const int p = p_begin - W - 1 + u + xr;
    const uint32_t o =
        xlive && p >= 0 && p < M ? ((uint32_t)p * (uint32_t)a.Ci + (uint32_t)(n0 + xc * 8)) * 4u : kOob;
    rx[0] = buffer_load16(rsx, o);
    rx[1] = buffer_load16(rsx, o + 16u);
  };
  auto put = [&](char *dst, int plane, const uint4 (&q)[2]) {
    const float v[8] = {__uint_as_float(q[0].x), __uint_as_float(q[0].y), __uint_as_float(q[0].z),
                        __uint_as_float(q[0].w), __uint_as_float(q[1].x), __uint_as_float(q[1].y),
                        __uint_as_float(q[1].z), __uint_as_float(q[1].w)};
    uint4 p[3];
    split8(v, p, top);
#pragma unroll
    for (int k = 0; k < 3; ++k) *reinterpret_cast<uint4 *>(dst + k * plane) = p[k];
  };
  float bsum[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) bsum[e] = 0.f;

  const int lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lg = lane >> 4;
  const int wm0 = (wave >> 1) * 32, wn0 = (wave & 1) * 16;  // this wave's output and input channels
  // transposing reads: lane 4 r + q of 16 reads channels 4 q on of pixel r
  // (and r + 4) of its group's eight, and receives channel 4 r + q of all four
  const int pr = 8 * lg + (li >> 2), q8 = (li & 3) * 8;
  int ga[2][2];  // [row block][pixel r, r + 4]
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 2; ++e) ga[i][e] = g_at(pr + 4 * e, (wm0 + 16 * i) / 8 + (q8 >> 4)) + (q8 & 8);
  int xa[9][2];  // ring address of tap t at stage 0 (adding 32 rows keeps the bank key, bit 3 of the row)
#pragma unroll
  for (int rs = 0; rs < 9; ++rs)
#pragma unroll
    for (int e = 0; e < 2; ++e)
      xa[rs][e] = x_at(pr + 4 * e + (rs / 3) * W + rs % 3, wn0 / 8 + (q8 >> 4)) + (q8 & 8);
  Sums<2, 9> sums;
  sums.clear();

  if (tid == 0) huge = 0;
  if (tid < 12) *reinterpret_cast<uint4 *>(Xs + (tid >> 2) * XPL + ZERO + (tid & 3) * 16) = make_uint4(0, 0, 0, 0);
  // ring rows before the first stage's 32: 2 W + 2
  for (int u = 0; u < 2 * W + 2; u += 64) {
    load_x(u);
    if (u + xr < 2 * W + 2) put(Xs + x_at(u + xr, xc), XPL, rx);
  }
  load_g(0);
  load_x(2 * W + 2);
  for (int kt = 0; kt < nk; ++kt) {
    put(Gs + g_at(gpx, gc), GPL, rg);
    if (do_bias) {
      const uint4 b0 = rg[0], b1 = rg[1];
      bsum[0] += __uint_as_float(b0.x); bsum[1] += __uint_as_float(b0.y);
      bsum[2] += __uint_as_float(b0.z); bsum[3] += __uint_as_float(b0.w);
      bsum[4] += __uint_as_float(b1.x); bsum[5] += __uint_as_float(b1.y);
      bsum[6] += __uint_as_float(b1.z); bsum[7] += __uint_as_float(b1.w);
    }
    if (xr < kStep) put(Xs + x_at((2 * W + 2 + kt * kStep + xr) & (RING - 1), xc), XPL, rx);
    __syncthreads();
    load_g(kt + 1);
    load_x(2 * W + 2 + (kt + 1) * kStep);
    // which taps of this lane's two pixels stay inside the image
    bool up[2], dn[2], lf[2], rt[2], in[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int p = p_begin + kt * kStep + pr + 4 * e;
      const uint32_t q = fdiv((uint32_t)p, fd_w);
      const int w = (int)((uint32_t)p - q * (uint32_t)W), h = (int)(q - fdiv(q, fd_h) * (uint32_t)a.H);
      in[e] = p < p_end;
      up[e] = h > 0, dn[e] = h < a.H - 1, lf[e] = w > 0, rt[e] = w < W - 1;
    }
    Frag3 g[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int k = 0; k < 3; ++k) g[i].p[k] = read_tr(Gs + k * GPL + ga[i][0], Gs + k * GPL + ga[i][1]);
#pragma unroll
    for (int rs = 0; rs < 9; ++rs) {
      const int r = rs / 3, c = rs % 3;
      int at[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const bool ok = in[e] && (r == 1 || (r == 0 ? up[e] : dn[e])) && (c == 1 || (c == 0 ? lf[e] : rt[e]));
        at[e] = ok ? (xa[rs][e] + kt * (kStep * XROW)) & (RING * XROW - 1) : ZERO;
      }
      Frag3 x[1];
#pragma unroll
      for (int k = 0; k < 3; ++k) x[0].p[k] = read_tr(Xs + k * XPL + at[0], Xs + k * XPL + at[1]);
      sums.add(g, x, rs);
    }
    __syncthreads();
  }

  if (top >= kHuge) huge = 1;
  sums.finish();
  __syncthreads();
  float *dw = a.dw + split * a.dw_ss + rep * a.dw_rs;
  const bool plain = huge != 0 && !all_finite(sums.hh);
#pragma unroll
  for (int rs = 0; rs < 9; ++rs) {
    const int n = n0 + wn0 + li;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm0 + i * 16 + lg * 4 + r;
        if (m < a.Co && n < a.Ci) dw[(int64_t)m * a.nw + rs * a.Ci + n] = sums.hh[i][rs][r];
      }
  }
  if (plain) {
    __threadfence_block();  // the wave's own stores, read by other lanes of it
    for (int e = lane; e < 32 * 9 * 16; e += 64) {
      const int m = m0 + wm0 + e / 144, rs = e % 144 / 16, n = n0 + wn0 + e % 16;
      if (m < a.Co && n < a.Ci && !finite(dw + (int64_t)m * a.nw + rs * a.Ci + n))
        dw[(int64_t)m * a.nw + rs * a.Ci + n] = sum_wgrad(a, G, X, m, rs * a.Ci + n, p_begin, p_end, fd_w, fd_h);
    }
  }
  if (do_bias) {
    float *red = reinterpret_cast<float *>(Xs);  // [32 pixels][64 channels]
#pragma unroll
    for (int e = 0; e < 8; ++e) red[gpx * 64 + gc * 8 + e] = bsum[e];
    __syncthreads();
    if (tid < 64 && m0 + tid < a.Co) {
      float s = 0.f;
      for (int i = 0; i < 32; ++i) s += red[i * 64 + tid];
      a.db[split * a.db_ss + rep * a.db_rs + m0 + tid] = s;
    }
  }
}

hipError_t run_wgrad_halo(const WgradArgs &a, hipStream_t s, std::string *label) {
  const int MT = (a.Co + 63) / 64, NT = (a.Ci + 31) / 32;
  if (label) *label = "conv_wgrad<f32,64x288,w4,halo,split>";
  hipLaunchKernelGGL(wgrad_f32_halo_kernel, dim3((uint32_t)MT * NT * a.splits * a.C), dim3(256), 0, s, a,
                     make_fastdiv(a.W), make_fastdiv(a.H), MT, NT);
  return hipGetLastError();
}

template <int BM, int BN, int WM, int WN, int OCC>
hipError_t run_conv(const ConvArgs &a, hipStream_t s, std::string *label) {
  const int M = a.Bt * a.H * a.W;
  const int MT = (M + BM - 1) / BM, NT = (a.N + BN - 1) / BN;
  const FastDiv fw = make_fastdiv(a.W), fh = make_fastdiv(a.H), fc = make_fastdiv(a.Csrc);
  const uint32_t blocks = (uint32_t)MT * NT * a.C;
  if (label)
    *label = std::string(a.epi == EPI_FWD ? "conv_fwd<f32," : "conv_dgrad<f32,") + std::to_string(BM) + "x" +
             std::to_string(BN) + ",w" + std::to_string(WM * WN) + ",split>";
  const dim3 threads(64 * WM * WN);
  if (a.epi == EPI_FWD)
    hipLaunchKernelGGL((conv_f32_kernel<BM, BN, WM, WN, EPI_FWD, OCC>), dim3(blocks), threads, 0, s, a, fw, fh, fc, MT,
                       NT);
  else
    hipLaunchKernelGGL((conv_f32_kernel<BM, BN, WM, WN, EPI_DGRAD, OCC>), dim3(blocks), threads, 0, s, a, fw, fh, fc,
                       MT, NT);
  return hipGetLastError();
}

template <int BM, int BN, int WM, int WN, int OCC>
hipError_t run_stride2(const ConvArgs &a, hipStream_t s, std::string *label) {
  const int M = a.Bt * a.H * a.W;
  const int MT = (M + BM - 1) / BM, NT = (a.N + BN - 1) / BN;
  if (label)
    *label = "conv_dgrad<f32," + std::to_string(BM) + "x" + std::to_string(BN) + ",w" + std::to_string(WM * WN) +
             ",stride2,split>";
  hipLaunchKernelGGL((conv_f32_kernel<BM, BN, WM, WN, EPI_DGRAD, OCC, true>), dim3((uint32_t)MT * NT * a.C * 4),
                     dim3(64 * WM * WN), 0, s, a, make_fastdiv(a.W), make_fastdiv(a.H), make_fastdiv(a.Csrc), MT, NT);
  return hipGetLastError();
}

template <int BM, int BN, int WM, int WN, int OCC, int RD>
hipError_t run_conv_halo(const ConvArgs &a, hipStream_t s, std::string *label) {
  const int M = a.Bt * a.H * a.W;
  const int MT = (M + BM - 1) / BM, NT = (a.N + BN - 1) / BN;
  const FastDiv fw = make_fastdiv(a.W), fh = make_fastdiv(a.H);
  const uint32_t blocks = (uint32_t)MT * NT * a.C;
  if (label)
    *label = std::string(a.epi == EPI_FWD ? "conv_fwd<f32," : "conv_dgrad<f32,") + std::to_string(BM) + "x" +
             std::to_string(BN) + ",w" + std::to_string(WM * WN) + ",halo,split>";
  const dim3 threads(64 * WM * WN);
  if (a.epi == EPI_FWD)
    hipLaunchKernelGGL((conv_f32_halo_kernel<BM, BN, WM, WN, EPI_FWD, OCC, RD>), dim3(blocks), threads, 0, s, a, fw,
                       fh, MT, NT);
  else
    hipLaunchKernelGGL((conv_f32_halo_kernel<BM, BN, WM, WN, EPI_DGRAD, OCC, RD>), dim3(blocks), threads, 0, s, a,
                       fw, fh, MT, NT);
  return hipGetLastError();
}

template <int BM, int BN, int WM, int WN, int OCC>
hipError_t run_wgrad(const WgradArgs &a, hipStream_t s, std::string *label) {
  const int MT = (a.Co + BM - 1) / BM, NT = ((a.taps == 1 ? a.Ci : 9 * a.Ci) + BN - 1) / BN;
  const FastDiv fw = make_fastdiv(a.W), fh = make_fastdiv(a.H), fc = make_fastdiv(a.Ci);
  if (label)
    *label = std::string("conv_wgrad<f32,") + std::to_string(BM) + "x" + std::to_string(BN) + ",w" +
             std::to_string(WM * WN) + ",split>";
  hipLaunchKernelGGL((wgrad_f32_kernel<BM, BN, WM, WN, OCC>), dim3((uint32_t)MT * NT * a.splits * a.C),
                     dim3(64 * WM * WN), 0, s, a, fw, fh, fc, MT, NT);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_conv_f32(const ConvArgs &a, hipStream_t s, std::string *label) {
  // 16-byte loads of 4 channels; 8 values of one tap per thread
  if (a.Csrc % 4 != 0 || (a.taps != 1 && a.Csrc % 8 != 0) || a.N % 4 != 0) return hipErrorInvalidValue;
  const int64_t M = (int64_t)a.Bt * a.H * a.W;
  auto blocks = [&](int bm, int bn) { return (M + bm - 1) / bm * ((a.N + bn - 1) / bn) * a.C; };
  if (a.stride2) {
    // (the grid holds four classes; tiles as below, by the class of most taps)
    if (a.N > 64 && blocks(128, 128) >= 256) return run_stride2<128, 128, 4, 2, 4>(a, s, label);
    if (a.N > 32) return blocks(128, 64) >= 256 ? run_stride2<128, 64, 2, 2, 3>(a, s, label)
                                                : run_stride2<64, 64, 2, 2, 4>(a, s, label);
    return run_stride2<32, 32, 2, 2, 4>(a, s, label);
  }
  // Halo staging where 32-channel blocks waste less than a fifth of their
  // stages.  The largest tile that gives every CU a workgroup: a smaller one
  // reads and splits its operands more often per product, a larger one leaves
  // CUs idle (64 examples, us per launch on one box; 256 x 128 / 128 x 64 /
  // 64 x 64 / 32 x 64, and the fp32 MFMA kernel these replaced):
  //   4 replicas, 128 -> 128 at 16 x 16    95 / 108 / 118 / 169   (122)
  //   4 replicas, 256 -> 256 at 8 x 8     161 / 107 / 119 / 163   (132)
  //   4 replicas, 512 -> 512 at 4 x 4     288 / 142 / 133 / 163   (241)
  //   1 replica,  128 -> 128 at 16 x 16    80 /  36 /  38 /  48
  //   1 replica,  512 -> 512 at 4 x 4     283 / 137 / 114 / 102
  //   4 replicas,  64 ->  64 at 32 x 32     - / 112 / 119         (162)
  // The table is with the weights loaded one tap ahead.  Three taps ahead, the
  // chosen tiles (forward): 256 -> 256 at 8 x 8 95 -> 92, 512 -> 512 at 4 x 4 143
  // -> 117, 64 -> 64 at 32 x 32 103 -> 97; 1 replica, 128 -> 128 at 16 x 16 36 ->
  // 31; 32 x 64 (3 replicas of 20 examples, 136 -> 136 at 6 x 6) 34 -> 28; 64 x 32
  // (24 -> 8 at 12 x 12) 33 -> 27.
  // (4 x 4 images: a 128-pixel tile's taps read eight images' borders, mostly
  // zeros, so 64 pixels do better.)
  if (a.taps == 9 && a.W <= kHaloW && a.Csrc >= 32 && 45 * ((a.Csrc + 31) / 32) <= 6 * ((9 * a.Csrc + 31) / 32)) {
    if (a.N > 32) {
      if (a.N > 64 && blocks(256, 128) >= 256) return run_conv_halo<256, 128, 4, 2, 2, 1>(a, s, label);
      if (blocks(128, 64) >= 256 && a.W > 4) return run_conv_halo<128, 64, 4, 2, 4, 3>(a, s, label);
      if (blocks(64, 64) >= 256) return run_conv_halo<64, 64, 2, 2, 3, 3>(a, s, label);
      return run_conv_halo<32, 64, 1, 4, 3, 3>(a, s, label);
    }
    // 64 -> 32 at 32 x 32, 4 replicas: 59 us (128 x 32: 67; fp32 MFMA 107)
    if (blocks(256, 32) >= 256) return run_conv_halo<256, 32, 8, 1, 4, 1>(a, s, label);
    return run_conv_halo<64, 32, 4, 1, 4, 3>(a, s, label);
  }
  if (a.N > 64) {
    if (blocks(128, 128) >= 256) return run_conv<128, 128, 4, 2, 4>(a, s, label);
    return run_conv<64, 64, 2, 2, 4>(a, s, label);
  }
  if (a.N > 32) {
    if (blocks(128, 64) >= 256) return run_conv<128, 64, 2, 2, 3>(a, s, label);
    return run_conv<64, 64, 2, 2, 4>(a, s, label);
  }
  if (blocks(128, 32) >= 256) return run_conv<128, 32, 4, 1, 3>(a, s, label);
  return run_conv<32, 32, 2, 2, 4>(a, s, label);
}

// Halo staging for the weight gradient: the padding of the channels to 64 x
// 32 blocks must cost less than the halo's rate gains (measured 220-230
// against 130-150 TFLOP/s of fp32 products on 64-channel multiples).
bool wgrad_f32_halo(int Co, int Ci, int W, int taps) {
  if (taps != 9 || W > kHaloW || Ci % 8 != 0 || Co % 8 != 0) return false;
  int bm, bn;
  wgrad_tile(GCPSL_F32, Co, 9 * Ci, &bm, &bn);
  const int64_t halo = (int64_t)((Co + 63) / 64) * 64 * ((Ci + 31) / 32) * 288;
  const int64_t flat = (int64_t)((Co + bm - 1) / bm) * bm * ((9 * Ci + bn - 1) / bn) * bn;
  return 2 * halo <= 3 * flat;
}

int64_t wgrad_f32_tiles(int Co, int Ci, int W, int taps) {
  if (wgrad_f32_halo(Co, Ci, W, taps)) return (int64_t)((Co + 63) / 64) * ((Ci + 31) / 32);
  const int nw = taps == 1 ? Ci : 9 * Ci;
  int bm, bn;
  wgrad_tile(GCPSL_F32, Co, nw, &bm, &bn);
  return (int64_t)((Co + bm - 1) / bm) * ((nw + bn - 1) / bn);
}

hipError_t launch_wgrad_f32(const WgradArgs &a, hipStream_t s, std::string *label) {
  if (a.Ci % 4 != 0 || a.Co % 4 != 0 || a.chunk % kStep != 0) return hipErrorInvalidValue;
  if (wgrad_f32_halo(a.Co, a.Ci, a.W, a.taps)) return run_wgrad_halo(a, s, label);
  int bm, bn;
  wgrad_tile(GCPSL_F32, a.Co, a.taps == 1 ? a.Ci : 9 * a.Ci, &bm, &bn);
  if (bm == 128) {
    if (bn == 128) return run_wgrad<128, 128, 2, 2, 2>(a, s, label);
    if (bn == 64) return run_wgrad<128, 64, 2, 2, 2>(a, s, label);
    return run_wgrad<128, 32, 4, 1, 3>(a, s, label);
  }
  if (bm == 64) {
    if (bn == 128) return run_wgrad<64, 128, 2, 2, 2>(a, s, label);
    if (bn == 64) return run_wgrad<64, 64, 2, 2, 3>(a, s, label);
    return run_wgrad<64, 32, 2, 2, 3>(a, s, label);
  }
  if (bn == 128) return run_wgrad<32, 128, 1, 4, 3>(a, s, label);
  if (bn == 64) return run_wgrad<32, 64, 1, 4, 3>(a, s, label);
  return run_wgrad<32, 32, 2, 2, 3>(a, s, label);
}
