// Normalisation layers of the split CNN (Sec. IV-B): GroupNorm in the client
// segment, BatchNorm in the server segment, each followed by ReLU, over the
// raw output z [Bt][H][W][Ch] (NHWC) of the conv before it:
//
//   x_hat = (z - mean) * rstd,  rstd = 1 / sqrt(var + 1e-5),  var biased,
//   u = gamma_c x_hat + beta_c,  a = ReLU(u);
//
// batch norm takes mean and var per channel over (Bt, H, W), group norm per
// example over (H, W, the channels of a group).  Backward, from du = dL/du:
//
//   dgamma_c = sum du x_hat,  dbeta_c = sum du        (over Bt, H, W)
//   dz = rstd (du gamma_c - S1 / n - x_hat S2 / n),
//   S1 = sum du gamma_c,  S2 = sum du gamma_c x_hat   (over the set of n values)
//
// Batch norm also updates its replica's running statistics (momentum 0.1,
// unbiased variance for the running value) and batch counter.
//
// Every sum runs in fp64 in a fixed order (per-thread pixel strides, then
// pixel-lane order within a workgroup; across the chunks of a channel
// reduction, eight strided chunk lanes, then lane order), so results do not
// depend on scheduling or on which replicas share a launch.  A thread owns
// one 16-byte vector of VEC channels.
//
// Group norm is one launch each way (and chan_finish for dgamma, dbeta): a
// workgroup takes whole examples, so it has every value of its statistics,
// and keeps the example in registers between the sums and the result where it
// fits; a few examples that don't take the result in a second launch over the
// chip.  Batch norm of few pixels (bn_one_launch) is one launch each
// way too: a workgroup takes a few channels of every pixel and holds them.
// Larger batch norms reduce chunks of pixels, finish the sums and apply them in
// three launches; their chunks shrink for small tensors (16 to 256 pixels) so
// that the launches still spread over the chip.
#include "runtime.h"

namespace {

constexpr double kEps = 1e-5;
constexpr double kMomentum = 0.1;

template <typename T> struct V16 {
  T v[ElemT<T>::VEC];
};
template <typename T> __device__ __forceinline__ V16<T> load16(const T *p) {
  return __builtin_bit_cast(V16<T>, *reinterpret_cast<const uint4 *>(p));
}
template <typename T> __device__ __forceinline__ void store16(T *p, const V16<T> &v) {
  *reinterpret_cast<uint4 *>(p) = __builtin_bit_cast(uint4, v);
}

// Per-channel sums over one chunk of pixels: MODE 0 sum z and z^2 (batch
// statistics), MODE 1 sum du and du x_hat (gradients of gamma and beta).
// Partials part[rep][chunk][c][2].
template <typename T, int MODE>
__global__ void __launch_bounds__(256)
chan_reduce_kernel(NormArgs a) {
  constexpr int VEC = ElemT<T>::VEC;
  __shared__ double red[256][2 * VEC];
  const int rep = replica_of(a.rmap, blockIdx.y);
  const int CV = a.Ch / VEC, PL = 256 / CV;
  const int tid = threadIdx.x, cv = tid % CV, pl = tid / CV;
  const int64_t M = (int64_t)a.Bt * a.H * a.W;
  const int64_t p0 = (int64_t)blockIdx.x * a.chunk_px, p1 = min(M, p0 + a.chunk_px);
  const T *z = reinterpret_cast<const T *>(a.z) + rep * a.z_rs;
  const T *du = reinterpret_cast<const T *>(a.du) + rep * a.z_rs;
  const float *mean = a.mean + (int64_t)rep * a.nstat, *rstd = a.rstd + (int64_t)rep * a.nstat;
  double s0[VEC], s1[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) s0[e] = s1[e] = 0.0;
  float km[VEC], kr[VEC];  // MODE 1: the statistics of this thread's channels
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    km[e] = MODE == 1 && pl < PL ? mean[cv * VEC + e] : 0.f;
    kr[e] = MODE == 1 && pl < PL ? rstd[cv * VEC + e] : 0.f;
  }
  auto add = [&](const V16<T> &zv, const V16<T> &gv) {
    if constexpr (MODE == 0) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const double v = ElemT<T>::to_f(zv.v[e]);
        s0[e] += v;
        s1[e] += v * v;
      }
    } else {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const float xh = (ElemT<T>::to_f(zv.v[e]) - km[e]) * kr[e];
        const double g = ElemT<T>::to_f(gv.v[e]);
        s0[e] += g;
        s1[e] += g * (double)xh;
      }
    }
  };
  if (pl < PL) {
    // four pixels' loads in flight, added in pixel order
    int64_t p = p0 + pl;
    for (; p + 3 * PL < p1; p += 4 * PL) {
      V16<T> zv[4], gv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        zv[u] = load16(z + (p + u * PL) * a.Ch + cv * VEC);
        if constexpr (MODE == 1) gv[u] = load16(du + (p + u * PL) * a.Ch + cv * VEC);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) add(zv[u], gv[u]);
    }
    for (; p < p1; p += PL) {
      V16<T> zv = load16(z + p * a.Ch + cv * VEC), gv{};
      if constexpr (MODE == 1) gv = load16(du + p * a.Ch + cv * VEC);
      add(zv, gv);
    }
  }
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    red[tid][e] = s0[e];
    red[tid][VEC + e] = s1[e];
  }
  __syncthreads();
  // the chunk's sums: one (channel, sum) per thread, over the pixel lanes in
  // lane order
  double *out = a.part + ((int64_t)rep * a.chunks + blockIdx.x) * a.Ch * 2;
  for (int o = tid; o < 2 * a.Ch; o += 256) {
    const int c = o >> 1, k = o & 1, ocv = c / VEC, e = c - ocv * VEC;
    double t = 0.0;
    for (int l = 0; l < PL; ++l) t += red[l * CV + ocv][k * VEC + e];
    out[o] = t;
  }
}

// Chunk partials -> per-channel sums.  A workgroup takes 32 channels: lane j
// of a channel adds chunks j, j + 8, j + 16, ... in order (four loads in
// flight), and the 8 lanes' sums are added in lane order.  MODE 0:
// batch-norm mean and rstd, and the running statistics; MODE 1: dbeta,
// dgamma into grad and (batch norm) the sums for the input gradient.
constexpr int kFinishCh = 32, kFinishLanes = 8;

template <int MODE>
__global__ void __launch_bounds__(256)
chan_finish_kernel(NormArgs a) {
  __shared__ double red[kFinishLanes][kFinishCh][2];
  const int rep = replica_of(a.rmap, blockIdx.y);
  const int cl = threadIdx.x % kFinishCh, j = threadIdx.x / kFinishCh;
  const int c = blockIdx.x * kFinishCh + cl;
  double S0 = 0.0, S1 = 0.0;
  if (c < a.Ch) {
    const double *pp = a.part + ((int64_t)rep * a.chunks * a.Ch + c) * 2;
    const int64_t step = (int64_t)a.Ch * 2;
    int k = j;
    for (; k + 3 * kFinishLanes < a.chunks; k += 4 * kFinishLanes) {
      double v[4][2];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        v[u][0] = pp[(k + u * kFinishLanes) * step];
        v[u][1] = pp[(k + u * kFinishLanes) * step + 1];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        S0 += v[u][0];
        S1 += v[u][1];
      }
    }
    for (; k < a.chunks; k += kFinishLanes) {
      S0 += pp[k * step];
      S1 += pp[k * step + 1];
    }
  }
  red[j][cl][0] = S0;
  red[j][cl][1] = S1;
  __syncthreads();
  if (j != 0 || c >= a.Ch) return;
  S0 = red[0][cl][0];
  S1 = red[0][cl][1];
#pragma unroll
  for (int l = 1; l < kFinishLanes; ++l) {
    S0 += red[l][cl][0];
    S1 += red[l][cl][1];
  }
  const double n = (double)a.Bt * a.H * a.W;
  if constexpr (MODE == 0) {
    const double mean = S0 / n;
    const double var = fmax(S1 / n - mean * mean, 0.0);
    a.mean[(int64_t)rep * a.nstat + c] = (float)mean;
    a.rstd[(int64_t)rep * a.nstat + c] = (float)(1.0 / sqrt(var + kEps));
    float *st = a.state + rep * a.S + a.st_off;
    st[c] = (float)((1.0 - kMomentum) * (double)st[c] + kMomentum * mean);
    st[a.Ch + c] = (float)((1.0 - kMomentum) * (double)st[a.Ch + c] + kMomentum * var * n / (n - 1.0));
    if (c == 0) st[2 * a.Ch] = (float)((double)st[2 * a.Ch] + 1.0);
  } else {
    a.grad[rep * a.P + a.b_off + c] = (float)S0;
    a.grad[rep * a.P + a.g_off + c] = (float)S1;
    if (!a.groups) {
      a.sums[((int64_t)rep * a.nstat + c) * 2] = S0;
      a.sums[((int64_t)rep * a.nstat + c) * 2 + 1] = S1;
    }
  }
}

// ------------------------------------------------ whole sets per workgroup
// Sums over a workgroup's pixel lanes.  Thread tid = pl CV + cv holds partial
// sums of channels VEC cv on over pixels pl, pl + PL, ... (threads past PL CV
// hold zeros).  Output (channel, sum) o is added by S threads of one wave (a
// power of two), each over every S-th pixel lane, then by a butterfly: a fixed
// order.  Rows are padded to an odd number of doubles against bank conflicts.
template <int VEC, int NT, int MAXC> struct LaneSums {
  double red[NT][2 * VEC + 1];
  double chs[2][MAXC];  // per-channel sums
  __device__ __forceinline__ void reduce(const double (&s0)[VEC], const double (&s1)[VEC], int CV, int PL) {
    const int tid = threadIdx.x, O = 2 * CV * VEC;
#pragma unroll
    for (int e = 0; e < VEC; ++e) red[tid][e] = s0[e], red[tid][VEC + e] = s1[e];
    __syncthreads();
    int lgS = 0;
    while ((2 << lgS) * O <= NT && lgS < 6) ++lgS;
    const int S = 1 << lgS, seg = tid & (S - 1);
    for (int o = tid >> lgS; o < O; o += NT >> lgS) {  // (the S threads of an output share o: they leave together)
      const int c = o >> 1, k = o & 1;
      const int cc = c / VEC, at = k * VEC + c % VEC;
      double t = 0.0;
#pragma unroll 4
      for (int l = seg; l < PL; l += S) t += red[l * CV + cc][at];
      for (int d = 1; d < S; d <<= 1) t += __shfl_xor(t, d);
      if (seg == 0) chs[k][c] = t;
    }
    __syncthreads();
  }
};

// f(i, p) for this thread's pixels p = pl + i PL < n, U loads in flight:
// get(p) loads, use(value, p) takes the values in pixel order.
template <int U, typename G, typename F> __device__ __forceinline__ void stream_pixels(int pl, int PL, int n, G get, F use) {
  for (int p = pl; p < n; p += U * PL) {
    decltype(get(0)) v[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (p + u * PL < n) v[u] = get(p + u * PL);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (p + u * PL < n) use(v[u], p + u * PL);
  }
}
template <typename T> struct Pair {
  V16<T> x, g;
};

// Hides a held vector's value from the compiler, which would otherwise keep
// the converted values of the sums for the result (twice the registers).
template <typename T> __device__ __forceinline__ void opaque(V16<T> &v) {
  uint4 q = __builtin_bit_cast(uint4, v);
  asm volatile("" : "+v"(q.x), "+v"(q.y), "+v"(q.z), "+v"(q.w));
  v = __builtin_bit_cast(V16<T>, q);
}

// APPLY false: the statistics only (norm_apply_* write the result).
template <typename T, int NT, int NV, int MAXC, bool APPLY = true>
__global__ void __launch_bounds__(NT)
group_fwd_kernel(NormArgs a) {
  constexpr int VEC = ElemT<T>::VEC, N = NV > 0 ? NV : 1;
  __shared__ LaneSums<VEC, NT, MAXC> ls;
  __shared__ float gm[MAXC], gr[MAXC];  // mean and rstd of each group
  const int rep = replica_of(a.rmap, blockIdx.y), b = blockIdx.x;
  const int CV = a.Ch / VEC, PL = NT / CV;
  const int tid = threadIdx.x, cv = tid % CV, pl = tid / CV;
  const int HW = a.H * a.W, G = a.groups, CG = a.Ch / G;
  const int64_t base = rep * a.z_rs + (int64_t)b * HW * a.Ch + cv * VEC;
  const T *z = reinterpret_cast<const T *>(a.z) + base;
  const T *res = a.res ? reinterpret_cast<const T *>(a.res) + base : nullptr;
  T *out = reinterpret_cast<T *>(a.a) + base;
  V16<T> zv[N];
  double s0[VEC], s1[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) s0[e] = s1[e] = 0.0;
  auto add = [&](const V16<T> &v) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const double x = ElemT<T>::to_f(v.v[e]);
      s0[e] += x;
      s1[e] += x * x;
    }
  };
  if (NV > 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int p = pl + i * PL;
      zv[i] = V16<T>{};
      if (pl < PL && p < HW) zv[i] = load16(z + (int64_t)p * a.Ch);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) add(zv[i]);
  } else if (pl < PL) {
    stream_pixels<4>(pl, PL, HW, [&](int p) { return load16(z + (int64_t)p * a.Ch); },
                     [&](const V16<T> &v, int) { add(v); });
  }
  ls.reduce(s0, s1, CV, PL);
  for (int g = tid; g < G; g += NT) {
    double S0 = 0.0, S1 = 0.0;
    for (int c = g * CG; c < (g + 1) * CG; ++c) S0 += ls.chs[0][c], S1 += ls.chs[1][c];
    const double n = (double)HW * CG, m = S0 / n, var = fmax(S1 / n - m * m, 0.0);
    const int64_t si = (int64_t)rep * a.nstat + b * G + g;
    a.mean[si] = gm[g] = (float)m;
    a.rstd[si] = gr[g] = (float)(1.0 / sqrt(var + kEps));
  }
  if (!APPLY) return;
  __syncthreads();
  if (pl >= PL) return;
  const float *gamma = a.theta + rep * a.P + a.g_off, *beta = a.theta + rep * a.P + a.b_off;
  float km[VEC], kr[VEC], kg[VEC], kb[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    const int c = cv * VEC + e, g = c / CG;
    km[e] = gm[g], kr[e] = gr[g], kg[e] = gamma[c], kb[e] = beta[c];
  }
  if (NV > 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) opaque(zv[i]);
  }
  auto put = [&](const V16<T> &v, const V16<T> &r, int p) {
    V16<T> o;
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      float u = kg[e] * ((ElemT<T>::to_f(v.v[e]) - km[e]) * kr[e]) + kb[e];
      if (res) u += ElemT<T>::to_f(r.v[e]);
      o.v[e] = ElemT<T>::from_f(a.relu ? fmaxf(u, 0.f) : u);
    }
    store16(out + (int64_t)p * a.Ch, o);
  };
  if (NV > 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int p = pl + i * PL;
      if (p < HW) put(zv[i], res ? load16(res + (int64_t)p * a.Ch) : V16<T>{}, p);
    }
  } else {
    stream_pixels<4>(pl, PL, HW,
                     [&](int p) {
                       return Pair<T>{load16(z + (int64_t)p * a.Ch), res ? load16(res + (int64_t)p * a.Ch) : V16<T>{}};
                     },
                     [&](const Pair<T> &v, int p) { put(v.x, v.g, p); });
  }
}

// Backward: dz, and the channel sums of du and du x_hat of each workgroup's
// `per` consecutive examples in part[rep][workgroup][c][2] (chan_finish adds
// the workgroups in order).  APPLY false: S1 and S2 of each group in sums[rep]
// instead of dz.
template <typename T, int NT, int NV, int MAXC, bool APPLY = true>
__global__ void __launch_bounds__(NT)
group_bwd_kernel(NormArgs a, int per) {
  constexpr int VEC = ElemT<T>::VEC, N = NV > 0 ? NV : 1;
  __shared__ LaneSums<VEC, NT, MAXC> ls;
  __shared__ float g1[MAXC], g2[MAXC];  // S1 / n and S2 / n of each group
  const int rep = replica_of(a.rmap, blockIdx.y);
  const int CV = a.Ch / VEC, PL = NT / CV;
  const int tid = threadIdx.x, cv = tid % CV, pl = tid / CV;
  const int HW = a.H * a.W, G = a.groups, CG = a.Ch / G;
  const float *gamma = a.theta + rep * a.P + a.g_off;
  float kg[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) kg[e] = pl < PL ? gamma[cv * VEC + e] : 0.f;
  constexpr int MC = MAXC > NT ? MAXC / NT : 1;
  double t0[MC] = {}, t1[MC] = {};  // sums over the examples, of channels tid, tid + NT, ...
  auto both = [&](const T *z, const T *du, auto use) {
    stream_pixels<4>(pl, PL, HW,
                     [&](int p) { return Pair<T>{load16(z + (int64_t)p * a.Ch), load16(du + (int64_t)p * a.Ch)}; },
                     [&](const Pair<T> &v, int p) { use(v.x, v.g, p); });
  };
  for (int b = blockIdx.x * per; b < min(a.Bt, (int)(blockIdx.x + 1) * per); ++b) {
    const int64_t base = rep * a.z_rs + (int64_t)b * HW * a.Ch + cv * VEC;
    const T *z = reinterpret_cast<const T *>(a.z) + base;
    const T *du = reinterpret_cast<const T *>(a.du) + base;
    T *dz = reinterpret_cast<T *>(a.dz) + base;
    float km[VEC], kr[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const int64_t si = (int64_t)rep * a.nstat + b * G + (pl < PL ? (cv * VEC + e) / CG : 0);
      km[e] = a.mean[si], kr[e] = a.rstd[si];
    }
    V16<T> zv[N], gv[N];
    double s0[VEC], s1[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) s0[e] = s1[e] = 0.0;
    auto add = [&](const V16<T> &x, const V16<T> &g) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const float xh = (ElemT<T>::to_f(x.v[e]) - km[e]) * kr[e];
        const double d = ElemT<T>::to_f(g.v[e]);
        s0[e] += d;
        s1[e] += d * (double)xh;
      }
    };
    if (NV > 0) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int p = pl + i * PL;
        zv[i] = gv[i] = V16<T>{};
        if (pl < PL && p < HW) zv[i] = load16(z + (int64_t)p * a.Ch), gv[i] = load16(du + (int64_t)p * a.Ch);
      }
#pragma unroll
      for (int i = 0; i < N; ++i)
        if (pl < PL && pl + i * PL < HW) add(zv[i], gv[i]);
#pragma unroll
      for (int i = 0; i < N; ++i) opaque(zv[i]), opaque(gv[i]);
    } else if (pl < PL) {
      both(z, du, [&](const V16<T> &x, const V16<T> &g, int) { add(x, g); });
    }
    ls.reduce(s0, s1, CV, PL);
#pragma unroll
    for (int i = 0; i < MC; ++i)
      if (tid + i * NT < a.Ch) t0[i] += ls.chs[0][tid + i * NT], t1[i] += ls.chs[1][tid + i * NT];
    for (int g = tid; g < G; g += NT) {
      double S1 = 0.0, S2 = 0.0;
      for (int c = g * CG; c < (g + 1) * CG; ++c) {
        S1 += ls.chs[0][c] * gamma[c];
        S2 += ls.chs[1][c] * gamma[c];
      }
      const double n = (double)HW * CG;
      if (APPLY) {
        g1[g] = (float)(S1 / n), g2[g] = (float)(S2 / n);
      } else {
        double *o = a.sums + ((int64_t)rep * a.nstat + b * G + g) * 2;
        o[0] = S1, o[1] = S2;
      }
    }
    __syncthreads();
    if (!APPLY) continue;
    float k1[VEC], k2[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const int g = pl < PL ? (cv * VEC + e) / CG : 0;
      k1[e] = g1[g], k2[e] = g2[g];
    }
    auto put = [&](const V16<T> &x, const V16<T> &g, int p) {
      V16<T> o;
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const float xh = (ElemT<T>::to_f(x.v[e]) - km[e]) * kr[e];
        o.v[e] = ElemT<T>::from_f(kr[e] * (ElemT<T>::to_f(g.v[e]) * kg[e] - k1[e] - xh * k2[e]));
      }
      store16(dz + (int64_t)p * a.Ch, o);
    };
    if (NV > 0) {
#pragma unroll
      for (int i = 0; i < N; ++i)
        if (pl < PL && pl + i * PL < HW) put(zv[i], gv[i], pl + i * PL);
    } else if (pl < PL) {
      both(z, du, put);
    }
    __syncthreads();  // g1, g2 and the sums are read before the next example's
  }
#pragma unroll
  for (int i = 0; i < MC; ++i) {
    const int c = tid + i * NT;
    if (c >= a.Ch) break;
    double *out = a.part + (((int64_t)rep * gridDim.x + blockIdx.x) * a.Ch + c) * 2;
    out[0] = t0[i], out[1] = t1[i];
  }
}

// Batch norm of few pixels: a workgroup of 1024 threads takes SV vectors of
// channels of every pixel of its replica and holds them (NV vectors per
// thread), MODE 0 forward (statistics, running state, output), MODE 1 backward
// (dgamma, dbeta, dz).
constexpr int kBnThreads = 1024;
template <typename T, int SV, int MODE, int NV>
__global__ void __launch_bounds__(kBnThreads)
batch_norm_kernel(NormArgs a) {
  constexpr int VEC = ElemT<T>::VEC, NT = kBnThreads, PL = NT / SV;
  __shared__ LaneSums<VEC, NT, SV * VEC> ls;
  // the workgroups that share cache lines (neighbouring channels) on one XCD
  const uint32_t t = xcd_swizzle(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int slice = __builtin_amdgcn_readfirstlane((int)(t % gridDim.x));
  const int rep = replica_of(a.rmap, __builtin_amdgcn_readfirstlane((int)(t / gridDim.x)));
  const int tid = threadIdx.x, cv = tid % SV, pl = tid / SV;
  const int M = a.Bt * a.H * a.W, c0 = (slice * SV + cv) * VEC;  // (Ch is a multiple of SV VEC)
  const T *z = reinterpret_cast<const T *>(a.z) + rep * a.z_rs + c0;
  const T *du = reinterpret_cast<const T *>(a.du) + rep * a.z_rs + c0;
  const T *res = MODE == 0 && a.res ? reinterpret_cast<const T *>(a.res) + rep * a.z_rs + c0 : nullptr;
  float *mean = a.mean + (int64_t)rep * a.nstat, *rstd = a.rstd + (int64_t)rep * a.nstat;
  double s0[VEC], s1[VEC];
  float km[VEC], kr[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    s0[e] = s1[e] = 0.0;
    km[e] = MODE == 1 ? mean[c0 + e] : 0.f;
    kr[e] = MODE == 1 ? rstd[c0 + e] : 0.f;
  }
  auto get = [&](int p) {
    Pair<T> v{load16(z + (int64_t)p * a.Ch), V16<T>{}};
    if (MODE == 1) v.g = load16(du + (int64_t)p * a.Ch);
    return v;
  };
  auto add = [&](const Pair<T> &v) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const float x = ElemT<T>::to_f(v.x.v[e]);
      if (MODE == 0) {
        s0[e] += (double)x;
        s1[e] += (double)x * x;
      } else {
        const double d = ElemT<T>::to_f(v.g.v[e]);
        s0[e] += d;
        s1[e] += d * (double)((x - km[e]) * kr[e]);
      }
    }
  };
  V16<T> hx[NV], hg[MODE == 1 ? NV : 1];
#pragma unroll
  for (int i = 0; i < NV; ++i)
    if (pl + i * PL < M) {
      const Pair<T> v = get(pl + i * PL);
      hx[i] = v.x;
      if (MODE == 1) hg[MODE == 1 ? i : 0] = v.g;
    }
#pragma unroll
  for (int i = 0; i < NV; ++i)
    if (pl + i * PL < M) add(Pair<T>{hx[i], hg[MODE == 1 ? i : 0]});
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    opaque(hx[i]);
    if (MODE == 1) opaque(hg[MODE == 1 ? i : 0]);
  }
  ls.reduce(s0, s1, SV, PL);
  const double n = (double)M;
  if (tid < SV * VEC) {
    const int c = slice * SV * VEC + tid;
    const double S0 = ls.chs[0][tid], S1 = ls.chs[1][tid];
    if (MODE == 0) {
      const double m = S0 / n, var = fmax(S1 / n - m * m, 0.0);
      mean[c] = (float)m;
      rstd[c] = (float)(1.0 / sqrt(var + kEps));
      ls.chs[0][tid] = (double)(float)m;
      ls.chs[1][tid] = (double)(float)(1.0 / sqrt(var + kEps));
      float *st = a.state + rep * a.S + a.st_off;
      st[c] = (float)((1.0 - kMomentum) * (double)st[c] + kMomentum * m);
      st[a.Ch + c] = (float)((1.0 - kMomentum) * (double)st[a.Ch + c] + kMomentum * var * n / (n - 1.0));
      if (c == 0) st[2 * a.Ch] = (float)((double)st[2 * a.Ch] + 1.0);
    } else {
      a.grad[rep * a.P + a.b_off + c] = (float)S0;
      a.grad[rep * a.P + a.g_off + c] = (float)S1;
    }
  }
  __syncthreads();
  float kg[VEC], k1[VEC], k2[VEC];
  const float *gamma = a.theta + rep * a.P + a.g_off, *beta = a.theta + rep * a.P + a.b_off;
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    const double S0 = ls.chs[0][cv * VEC + e], S1 = ls.chs[1][cv * VEC + e];
    kg[e] = gamma[c0 + e];
    if (MODE == 0) {
      km[e] = (float)S0, kr[e] = (float)S1, k1[e] = beta[c0 + e];
    } else {
      k1[e] = (float)(S0 / n), k2[e] = (float)(S1 / n);
    }
  }
  T *out = reinterpret_cast<T *>(MODE == 0 ? a.a : a.dz) + rep * a.z_rs + c0;
  auto put = [&](const Pair<T> &v, int p) {
    V16<T> o;
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const float xh = (ElemT<T>::to_f(v.x.v[e]) - km[e]) * kr[e];
      float u;
      if (MODE == 0) {
        u = kg[e] * xh + k1[e];
        if (res) u += ElemT<T>::to_f(v.g.v[e]);
        u = a.relu ? fmaxf(u, 0.f) : u;
      } else {
        u = kr[e] * kg[e] * (ElemT<T>::to_f(v.g.v[e]) - k1[e] - xh * k2[e]);
      }
      o.v[e] = ElemT<T>::from_f(u);
    }
    store16(out + (int64_t)p * a.Ch, o);
  };
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int p = pl + i * PL;
    if (p < M)
      put(Pair<T>{hx[i], MODE == 1 ? hg[MODE == 1 ? i : 0]
                                   : (res ? load16(res + (int64_t)p * a.Ch) : V16<T>{})}, p);
  }
}

// The elementwise passes of large batch norms, and of group norms (GROUPS) of a
// few large examples: a workgroup takes kApplyUnroll consecutive runs of 256
// 16-byte vectors (four loads in flight per thread), so a thread keeps the same
// VEC channels (where 256 is a multiple of the vectors per pixel) and walks
// neighbouring pixels.  The values it needs (gamma, beta, the statistics) are
// loaded when its channels or its example change, not per element.
constexpr int kApplyUnroll = 4;

// statistics index of channel c of example b
template <bool GROUPS> __device__ __forceinline__ int stat_index(const NormArgs &a, int b, int c) {
  return GROUPS ? b * a.groups + c / (a.Ch / a.groups) : c;
}

// a = ReLU(gamma (z - mean) rstd + beta (+ res)) (without the ReLU for a
// shortcut's norm).
template <typename T, bool GROUPS>
__global__ void __launch_bounds__(256)
norm_apply_fwd_kernel(NormArgs a, uint32_t total, FastDiv fcv, FastDiv fhw) {
  constexpr int VEC = ElemT<T>::VEC;
  const int rep = replica_of(a.rmap, blockIdx.y);
  const int CV = a.Ch / VEC;
  const T *z = reinterpret_cast<const T *>(a.z) + rep * a.z_rs;
  const T *res = a.res ? reinterpret_cast<const T *>(a.res) + rep * a.z_rs : nullptr;
  T *out = reinterpret_cast<T *>(a.a) + rep * a.z_rs;
  const float *mean = a.mean + (int64_t)rep * a.nstat, *rstd = a.rstd + (int64_t)rep * a.nstat;
  const float *gamma = a.theta + rep * a.P + a.g_off, *beta = a.theta + rep * a.P + a.b_off;
  constexpr uint32_t stride = 256u;
  int kc = -1, kb = 0;  // channel vector and example of the cached values
  float km[VEC], kr[VEC], kg[VEC], kbt[VEC];
  {
    const uint32_t i0 = blockIdx.x * (256u * kApplyUnroll) + threadIdx.x;
    V16<T> zv[kApplyUnroll], rv[kApplyUnroll];
#pragma unroll
    for (int u = 0; u < kApplyUnroll; ++u) {
      const uint32_t i = i0 + u * stride;
      if (i < total) {
        zv[u] = load16(z + (int64_t)i * VEC);
        if (res) rv[u] = load16(res + (int64_t)i * VEC);
      }
    }
#pragma unroll
    for (int u = 0; u < kApplyUnroll; ++u) {
      const uint32_t i = i0 + u * stride;
      if (i >= total) break;
      const uint32_t p = fdiv(i, fcv);
      const int cv = (int)(i - p * CV), b = GROUPS ? (int)fdiv(p, fhw) : 0;
      if (cv != kc || b != kb) {
        kc = cv, kb = b;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const int c = cv * VEC + e, si = stat_index<GROUPS>(a, b, c);
          km[e] = mean[si], kr[e] = rstd[si], kg[e] = gamma[c], kbt[e] = beta[c];
        }
      }
      V16<T> o;
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        float uu = kg[e] * ((ElemT<T>::to_f(zv[u].v[e]) - km[e]) * kr[e]) + kbt[e];
        if (res) uu += ElemT<T>::to_f(rv[u].v[e]);
        o.v[e] = ElemT<T>::from_f(a.relu ? fmaxf(uu, 0.f) : uu);
      }
      store16(out + (int64_t)i * VEC, o);
    }
  }
}

// dz = rstd (du gamma - S1 / n - x_hat S2 / n); batch norm's S1, S2 are gamma
// times the per-channel sums.
template <typename T, bool GROUPS>
__global__ void __launch_bounds__(256)
norm_apply_bwd_kernel(NormArgs a, uint32_t total, FastDiv fcv, FastDiv fhw) {
  constexpr int VEC = ElemT<T>::VEC;
  const int rep = replica_of(a.rmap, blockIdx.y);
  const int CV = a.Ch / VEC;
  const T *z = reinterpret_cast<const T *>(a.z) + rep * a.z_rs;
  const T *du = reinterpret_cast<const T *>(a.du) + rep * a.z_rs;
  T *dz = reinterpret_cast<T *>(a.dz) + rep * a.z_rs;
  const float *mean = a.mean + (int64_t)rep * a.nstat, *rstd = a.rstd + (int64_t)rep * a.nstat;
  const float *gamma = a.theta + rep * a.P + a.g_off;
  const double *sums = a.sums + (int64_t)rep * a.nstat * 2;
  const double n = GROUPS ? (double)a.H * a.W * (a.Ch / a.groups) : (double)a.Bt * a.H * a.W;
  constexpr uint32_t stride = 256u;
  int kc = -1, kb = 0;
  float km[VEC], kr[VEC], kg[VEC], k1[VEC], k2[VEC];
  {
    const uint32_t i0 = blockIdx.x * (256u * kApplyUnroll) + threadIdx.x;
    V16<T> zv[kApplyUnroll], gv[kApplyUnroll];
#pragma unroll
    for (int u = 0; u < kApplyUnroll; ++u) {
      const uint32_t i = i0 + u * stride;
      if (i < total) {
        zv[u] = load16(z + (int64_t)i * VEC);
        gv[u] = load16(du + (int64_t)i * VEC);
      }
    }
#pragma unroll
    for (int u = 0; u < kApplyUnroll; ++u) {
      const uint32_t i = i0 + u * stride;
      if (i >= total) break;
      const uint32_t p = fdiv(i, fcv);
      const int cv = (int)(i - p * CV), b = GROUPS ? (int)fdiv(p, fhw) : 0;
      if (cv != kc || b != kb) {
        kc = cv, kb = b;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const int c = cv * VEC + e, si = stat_index<GROUPS>(a, b, c);
          km[e] = mean[si], kr[e] = rstd[si], kg[e] = gamma[c];
          k1[e] = (float)(sums[2 * si] / n), k2[e] = (float)(sums[2 * si + 1] / n);
        }
      }
      V16<T> o;
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const float xh = (ElemT<T>::to_f(zv[u].v[e]) - km[e]) * kr[e];
        const float g = ElemT<T>::to_f(gv[u].v[e]);
        o.v[e] = ElemT<T>::from_f(GROUPS ? kr[e] * (g * kg[e] - k1[e] - xh * k2[e])
                                         : kr[e] * kg[e] * (g - k1[e] - xh * k2[e]));
      }
      store16(dz + (int64_t)i * VEC, o);
    }
  }
}

// workgroups of an elementwise pass over `total` vectors of one replica:
// about kApplyUnroll vectors per thread
uint32_t apply_blocks(uint32_t total) {
  return std::max<uint32_t>(1u, (total + 256u * kApplyUnroll - 1) / (256u * kApplyUnroll));
}

// Threads and vectors per thread that hold an example: the fewest threads (a
// workgroup is bound by its loads in flight, and several then share a CU).  A
// larger example, or more channels than threads, is read again instead (on
// 64 channels of 32 x 32, 256 examples: forward 21 us held / bf16, 37 us read
// again / fp32, 38 held; backward 37 read again / 53 held in bf16, 53 / 64 in
// fp32: the second reading comes from the last-level cache, and the registers
// of the held one spill).
// group_vectors: the vectors of an example that a thread of NT then holds.
int group_vectors(const NormArgs &a, int CV, int NT) {
  const int PL = NT / CV;
  return a.Ch <= NT ? (a.H * a.W + PL - 1) / PL : 1 << 20;
}
#define GCPSL_HOLD(MOST, CALL)                 \
  do {                                         \
    if (group_vectors(a, CV, 256) <= 4)        \
      CALL(256, 4, 256);                       \
    else if (group_vectors(a, CV, 512) <= 8)   \
      CALL(512, 8, 512);                       \
    else if (group_vectors(a, CV, 512) <= MOST) \
      CALL(512, MOST, 512);                    \
    else                                       \
      CALL(512, 0, 2048);                      \
  } while (0)

// Whether a group norm takes its result in an elementwise pass of its own: the
// workgroup that has an example's sums would read it again and write it alone,
// so fewer examples than kGroupSplit (of all the context's replicas) leave the
// chip idle.  Forward and backward, us, in one kernel / with the pass, bf16 (fp32):
//   64 channels of 64 x 64,    2 examples 105 /  78 (101 /  63)
//                             32 examples 114 /  94 (115 /  83)
//                             96 examples 122 / 122 (200 / 172)
//   192 channels of 32 x 32,  32 examples  94 /  91  (96 /  81)
//                             64 examples  99 / 110 (101 / 106)
constexpr int kGroupSplit = 64;
bool group_split(const NormArgs &a, int CV, int most) {
  return (int64_t)a.Bt * a.Call < kGroupSplit && group_vectors(a, CV, 256) > 4 && group_vectors(a, CV, 512) > most;
}
// vectors a thread holds at most, forward and backward (where the registers end)
constexpr int kHoldFwd = 16;
template <typename T> constexpr int kHoldBwd = ElemT<T>::VEC == 4 ? 16 : 8;

// Pixels per replica up to which a batch norm runs in one launch.  Its time is
// that of one workgroup (M pixels at a CU's rate and the fp64 sums), whatever
// the replicas, while the three launches' grows with all of them from 28 us
// forward and backward.  Rows of more than 64 bytes cost the workgroup more: it
// takes 16 bytes of every line.  Forward and backward, us, one launch / three:
//                             4,096        6,144        8,192 pixels
//   fp32,  16 channels, 1   22 / 29      27 / 31      32 / 34
//          64 channels, 1   29 / 30      38 / 33      47 / 36   of 1 replica
//                       4   28 / 32      36 / 38      45 / 42   of 4
//   bf16,  64 channels, 1   33 / 33      43 / 35      54 / 39
//                       4   31 / 39      39 / 49      48 / 54
//                       3   33 / 36      44 / 44      55 / 51
// So wide rows may have more pixels with every replica of the context, by the
// points where the two times meet, up to what a thread holds (fp32, whose rows
// are twice as long: fewer).
constexpr int kBnHold = 8;  // pixels that a thread holds at most
constexpr int kBnPixels = kBnHold * kBnThreads, kBnPixelsWide = 4096;

template <typename T> bool bn_one_launch(const NormArgs &a) {
  const int64_t M = (int64_t)a.Bt * a.H * a.W;
  if (a.groups != 0 || M > kBnPixels) return false;
  if (a.Ch * sizeof(T) <= 64) return true;
  const int64_t more = a.Call - 1;
  return M <= (sizeof(T) == 4 ? std::min<int64_t>(kBnPixelsWide + 768 * more, 7168)
                              : std::min<int64_t>(kBnPixelsWide + 1366 * more, kBnPixels));
}
template <typename T, int SV, int MODE> void run_bn_sv(const NormArgs &a, hipStream_t s) {
  const dim3 grid(a.Ch / ElemT<T>::VEC / SV, a.C);
  if (a.Bt * a.H * a.W <= 2 * kBnThreads / SV)
    hipLaunchKernelGGL((batch_norm_kernel<T, SV, MODE, 2>), grid, dim3(kBnThreads), 0, s, a);
  else
    hipLaunchKernelGGL((batch_norm_kernel<T, SV, MODE, kBnHold>), grid, dim3(kBnThreads), 0, s, a);
}
template <typename T, int MODE> void run_bn(const NormArgs &a, hipStream_t s) {
  // (the fp64 sums bound a workgroup: two vectors each only where that still
  // gives 128 of them in a launch of all the context's replicas; a launch of
  // fewer takes the same slices, whose pixel lanes set the order of the sums.
  // And only where a thread still holds its pixels: read twice, 256 channels of
  // 8,192 pixels took 119 us of 4 fp32 replicas and 103 of 8 bf16 ones, where one
  // vector each takes 68 and 75)
  const int CV = a.Ch / ElemT<T>::VEC;
  if (CV % 2 == 0 && CV / 2 * a.Call >= 128 && a.Bt * a.H * a.W <= kBnHold * kBnThreads / 2)
    run_bn_sv<T, 2, MODE>(a, s);
  else
    run_bn_sv<T, 1, MODE>(a, s);
}

template <typename T>
hipError_t norm_fwd_t(const NormArgs &a, hipStream_t s) {
  constexpr int VEC = ElemT<T>::VEC;
  const int CV = a.Ch / VEC;
  const uint32_t total = (uint32_t)((int64_t)a.Bt * a.H * a.W * CV);
  const FastDiv fcv = make_fastdiv((uint32_t)CV), fhw = make_fastdiv((uint32_t)(a.H * a.W));
  const dim3 apply(apply_blocks(total), a.C);
  if (a.groups && group_split(a, CV, kHoldFwd)) {
    hipLaunchKernelGGL((group_fwd_kernel<T, 512, 0, 2048, false>), dim3(a.Bt, a.C), dim3(512), 0, s, a);
    hipLaunchKernelGGL((norm_apply_fwd_kernel<T, true>), apply, dim3(256), 0, s, a, total, fcv, fhw);
  } else if (a.groups) {
#define FWD(NT, NV, MC) hipLaunchKernelGGL((group_fwd_kernel<T, NT, NV, MC>), dim3(a.Bt, a.C), dim3(NT), 0, s, a)
    GCPSL_HOLD(kHoldFwd, FWD);
#undef FWD
  } else if (bn_one_launch<T>(a)) {
    run_bn<T, 0>(a, s);
  } else {
    hipLaunchKernelGGL((chan_reduce_kernel<T, 0>), dim3(a.chunks, a.C), dim3(256), 0, s, a);
    hipLaunchKernelGGL((chan_finish_kernel<0>), dim3((a.Ch + kFinishCh - 1) / kFinishCh, a.C), dim3(256), 0, s, a);
    hipLaunchKernelGGL((norm_apply_fwd_kernel<T, false>), apply, dim3(256), 0, s, a, total, fcv, fhw);
  }
  return hipGetLastError();
}

template <typename T>
hipError_t norm_bwd_t(const NormArgs &a, hipStream_t s) {
  constexpr int VEC = ElemT<T>::VEC;
  const int CV = a.Ch / VEC;
  const uint32_t total = (uint32_t)((int64_t)a.Bt * a.H * a.W * CV);
  const FastDiv fcv = make_fastdiv((uint32_t)CV), fhw = make_fastdiv((uint32_t)(a.H * a.W));
  const dim3 fin((a.Ch + kFinishCh - 1) / kFinishCh, a.C), apply(apply_blocks(total), a.C);
  if (a.groups) {
    // examples per workgroup: its partial sums fill at most the chunks' rows
    NormArgs f = a;
    const int per = (a.Bt + a.chunks - 1) / a.chunks;
    f.chunks = (a.Bt + per - 1) / per;
    const bool split = group_split(a, CV, kHoldBwd<T>);
    if (split) {
      hipLaunchKernelGGL((group_bwd_kernel<T, 512, 0, 2048, false>), dim3(f.chunks, a.C), dim3(512), 0, s, f, per);
    } else {
#define BWD(NT, NV, MC) \
  hipLaunchKernelGGL((group_bwd_kernel<T, NT, NV, MC>), dim3(f.chunks, a.C), dim3(NT), 0, s, f, per)
      GCPSL_HOLD(kHoldBwd<T>, BWD);
#undef BWD
    }
    hipLaunchKernelGGL((chan_finish_kernel<1>), fin, dim3(256), 0, s, f);
    if (split) hipLaunchKernelGGL((norm_apply_bwd_kernel<T, true>), apply, dim3(256), 0, s, a, total, fcv, fhw);
  } else if (bn_one_launch<T>(a)) {
    run_bn<T, 1>(a, s);
  } else {
    hipLaunchKernelGGL((chan_reduce_kernel<T, 1>), dim3(a.chunks, a.C), dim3(256), 0, s, a);
    hipLaunchKernelGGL((chan_finish_kernel<1>), fin, dim3(256), 0, s, a);
    hipLaunchKernelGGL((norm_apply_bwd_kernel<T, false>), apply, dim3(256), 0, s, a, total, fcv, fhw);
  }
  return hipGetLastError();
}

}  // namespace

bool norm_ok(int dtype, int Ch, int groups) {
  const int vec = dtype == GCPSL_BF16 ? 8 : 4;
  return Ch % vec == 0 && Ch / vec <= 256 && Ch <= 2048 && (groups == 0 || Ch % groups == 0);
}

hipError_t launch_norm_fwd(int dtype, const NormArgs &a, hipStream_t s) {
  return dtype == GCPSL_BF16 ? norm_fwd_t<bf16_t>(a, s) : norm_fwd_t<float>(a, s);
}

hipError_t launch_norm_bwd(int dtype, const NormArgs &a, hipStream_t s) {
  return dtype == GCPSL_BF16 ? norm_bwd_t<bf16_t>(a, s) : norm_bwd_t<float>(a, s);
}
