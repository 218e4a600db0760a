// Replica-batched implicit-GEMM 3x3 convolutions on MFMA (gfx950): the choice of
// the kernel for a layer's pass, and the general bf16 weight gradient.
//
// Every pass of a conv layer is a dense contraction:
//   forward  out[m][co] = sum_{(r,s,ci)} x[m + (r-1, s-1)][ci] W[co][r][s][ci]
//   dgrad    dx[m][ci]  = sum_{(r,s,co)} g[m + (r-1, s-1)][co] W[co][2-r][2-s][ci]
//            (a forward conv of g with the flipped, transposed weights)
//   wgrad    dW[co][(r,s,ci)] = sum_m g[m][co] x[m + (r-1, s-1)][ci]
// with m = (b, h, w) over the batch and the image.  One workgroup computes a
// BM x BN output tile of one replica; replicas are folded into the linear
// workgroup index, so one launch covers all C clusters.
//
// fp32 layers run in k_conv_f32.hip; bf16 ones in k_conv_img.hip (the image
// side) and k_conv_lds.hip (every other forward and input gradient), their
// weight gradients in k_wgrad_lds.hip, or here for fewer than 64 output
// channels.  Tiles here are staged through LDS in "k-contiguous" rows of 128
// bytes (64 pixels) plus 16 bytes of padding, double buffered with one barrier
// per k tile.  The waves each own a sub-tile of 16x16 MFMA blocks.  A lane's
// operand fragment is 8 consecutive k values of one row: one
// v_mfma_f32_16x16x32_bf16.
#include "runtime.h"

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8_t load_frag(const bf16_t *p) {
  return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4 *>(p));
}

struct Pack {
  bf16_t v[8];
};

// Tile geometry and the MFMA loop over one staged k tile, one k group at a time
// (few registers).
template <int BM, int BN, int WM, int WN> struct Tile {
  static constexpr int VEC = ElemT<bf16_t>::VEC;
  static constexpr int BK = 64;         // k values per staged row (128 bytes)
  static constexpr int LDR = BK + 8;
  static constexpr int NT = 64 * WM * WN;  // threads per workgroup
  static constexpr int TM = BM / WM / 16, TN = BN / WN / 16;
  static_assert(TM >= 1 && TN >= 1, "wave tile must hold a 16x16 block");

  __device__ static __forceinline__ void compute(f32x4_t (&acc)[TM][TN], const bf16_t *As, const bf16_t *Bs, int wm0,
                                                 int wn0, int lane) {
    const int li = lane & 15, lg = lane >> 4;
#pragma unroll
    for (int kg = 0; kg < BK / 32; ++kg) {
      bf16x8_t a[TM], b[TN];
#pragma unroll
      for (int tm = 0; tm < TM; ++tm) a[tm] = load_frag(As + (wm0 + tm * 16 + li) * LDR + kg * 32 + lg * 8);
#pragma unroll
      for (int tn = 0; tn < TN; ++tn) b[tn] = load_frag(Bs + (wn0 + tn * 16 + li) * LDR + kg * 32 + lg * 8);
#pragma unroll
      for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
          acc[tm][tn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[tm], b[tn], acc[tm][tn], 0, 0, 0);
    }
  }
};

// Transpose an 8 x 8 (pixel x channel) block and store channel row q at dst +
// q * ldr, one row at a time (keeps few registers live): word j of row q packs
// channel q of pixels 2j (low half) and 2j + 1, one byte permute per word.
__device__ __forceinline__ void store_transposed(const uint4 (&in)[8], bf16_t *dst, int ldr) {
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const uint32_t sel = (q & 1) ? 0x07060302u : 0x05040100u;
    uint32_t o[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint4 &lo4 = in[2 * j], &hi4 = in[2 * j + 1];
      const uint32_t lo = (q >> 1) == 0 ? lo4.x : (q >> 1) == 1 ? lo4.y : (q >> 1) == 2 ? lo4.z : lo4.w;
      const uint32_t hi = (q >> 1) == 0 ? hi4.x : (q >> 1) == 1 ? hi4.y : (q >> 1) == 2 ? hi4.z : hi4.w;
      o[j] = __builtin_amdgcn_perm(hi, lo, sel);
    }
    *reinterpret_cast<uint4 *>(dst + q * ldr) = make_uint4(o[0], o[1], o[2], o[3]);
  }
}

template <int BM, int BN, bool VB>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
wgrad_kernel(WgradArgs a, FastDiv fd_w, FastDiv fd_h, FastDiv fd_c, int MT, int NT) {
  typedef bf16_t T;
  constexpr int WM = 2, WN = 2;
  using TL = Tile<BM, BN, WM, WN>;
  constexpr int VEC = TL::VEC, BK = TL::BK, LDR = TL::LDR;
  constexpr int NTH = TL::NT;
  constexpr int PB = BK / VEC;  // pixel blocks per k tile
  constexpr int NA = (BM / VEC) * PB, NB = (BN / VEC) * PB;
  constexpr int ITER = (NA + NB + NTH - 1) / NTH;
  static_assert(NA <= NTH, "A blocks must fit one pass");
  __shared__ __attribute__((aligned(16))) T As[2][BM * LDR];
  __shared__ __attribute__((aligned(16))) T Bs[2][BN * LDR];
  __shared__ float red[PB][BM];

  const int tid = threadIdx.x;
  const uint32_t total = (uint32_t)(MT * NT * a.splits * a.C);
  const uint32_t t = xcd_swizzle(blockIdx.x, total);
  const int nt = __builtin_amdgcn_readfirstlane((int)(t % (uint32_t)NT));
  uint32_t rest = t / (uint32_t)NT;
  const int mt = __builtin_amdgcn_readfirstlane((int)(rest % (uint32_t)MT));
  rest /= (uint32_t)MT;
  const int split = __builtin_amdgcn_readfirstlane((int)(rest % (uint32_t)a.splits));
  const int rep = replica_of(a.rmap, __builtin_amdgcn_readfirstlane((int)(rest / (uint32_t)a.splits)));
  const int M = a.Bt * a.H * a.W;
  const int NW = a.taps == 1 ? a.Ci : 9 * a.Ci;  // columns of the (padded) im2col operand
  const int p_begin = split * a.chunk;
  const int p_end = min(M, p_begin + a.chunk);
  const int nk = (p_end - p_begin + BK - 1) / BK;
  const int m0 = mt * BM, n0 = nt * BN;
  const T *G = reinterpret_cast<const T *>(a.g) + rep * a.g_rs;
  const T *X = reinterpret_cast<const T *>(a.x) + rep * a.x_rs;
  const bool do_bias = (nt == 0) && a.db != nullptr;

  // blocks owned by this thread
  int kind[ITER], rowb[ITER], pb[ITER], br[ITER], bs[ITER], bc[ITER];
  bool bvalid[ITER];
#pragma unroll
  for (int it = 0; it < ITER; ++it) {
    const int i = tid + NTH * it;
    if (i < NA) {
      kind[it] = 0;
      rowb[it] = i / PB;
      pb[it] = i % PB;
    } else if (i < NA + NB) {
      kind[it] = 1;
      rowb[it] = (i - NA) / PB;
      pb[it] = (i - NA) % PB;
    } else {
      kind[it] = 2;
      rowb[it] = 0;
      pb[it] = 0;
    }
    br[it] = bs[it] = bc[it] = 0;
    bvalid[it] = false;
    if (kind[it] == 1) {
      const int kk0 = n0 + rowb[it] * VEC;
      bvalid[it] = kk0 < NW;
      if (bvalid[it]) {
        const int rs = a.taps == 1 ? 4 : (int)fdiv((uint32_t)kk0, fd_c);
        bc[it] = kk0 - (a.taps == 1 ? 0 : rs * a.Ci);
        br[it] = (rs * 11) >> 5;
        bs[it] = rs - 3 * br[it];
      }
    }
  }

  // two register sets of prefetched blocks (tile kt + 2 is in flight while
  // tile kt is multiplied)
  uint4 reg0[ITER][VEC], reg1[ITER][VEC];
  float bsum[VEC];
#pragma unroll
  for (int q = 0; q < VEC; ++q) bsum[q] = 0.f;

  // Gradient rows: contiguous pixels, so one buffer offset per pixel; pixels
  // past the tensor read zero.  Input rows (VB: W % VEC == 0): a block's VEC
  // pixels share (b, h), only its first or last pixel can leave the image row
  // for kernel column s = 0 or 2.  Other widths follow each pixel's row and
  // column (12 x 12 images, 8 -> 24 channels, 3 replicas of 20 examples: 10.9 us
  // instead of 38.5 with one load per channel).
  constexpr uint32_t ESZ = sizeof(T);
  const __amdgpu_buffer_rsrc_t rsg = make_rsrc(G, (uint32_t)((int64_t)M * a.Co * ESZ));
  const __amdgpu_buffer_rsrc_t rsx = make_rsrc(X, (uint32_t)((int64_t)M * a.Ci * ESZ));
  auto load_tiles = [&](int kt, auto &reg) {
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
      const int pbase = p_begin + kt * BK + pb[it] * VEC;
      if (kind[it] == 0) {
        const int c0 = m0 + rowb[it] * VEC;
        const uint32_t o0 = c0 < a.Co ? ((uint32_t)pbase * (uint32_t)a.Co + (uint32_t)c0) * ESZ : kOob;
#pragma unroll
        for (int e = 0; e < VEC; ++e) reg[it][e] = buffer_load16(rsg, o0 + (uint32_t)(e * a.Co) * ESZ);
        continue;
      }
      if constexpr (VB) {
        if (kind[it] == 1 && a.taps == 1) {
          // im2col rows: contiguous pixels, like the gradient operand
          const uint32_t o0 = bvalid[it] ? ((uint32_t)pbase * (uint32_t)a.Ci + (uint32_t)bc[it]) * ESZ : kOob;
#pragma unroll
          for (int e = 0; e < VEC; ++e) reg[it][e] = buffer_load16(rsx, o0 + (uint32_t)(e * a.Ci) * ESZ);
        } else if (kind[it] == 1) {
          const uint32_t q1 = fdiv((uint32_t)pbase, fd_w);
          const int w0 = (int)((uint32_t)pbase - q1 * (uint32_t)a.W);
          const int b = (int)fdiv(q1, fd_h);
          const int h = (int)(q1 - (uint32_t)b * (uint32_t)a.H);
          const int hh = h + br[it] - 1;
          const bool rowok = bvalid[it] && pbase < M && (unsigned)hh < (unsigned)a.H;
          const int base = ((b * a.H + hh) * a.W + w0 + bs[it] - 1) * a.Ci + bc[it];
#pragma unroll
          for (int e = 0; e < VEC; ++e) {
            bool ok = rowok;
            if (e == 0) ok = ok && (w0 + bs[it] - 1 >= 0);
            if (e == VEC - 1) ok = ok && (w0 + VEC - 1 + bs[it] - 1 < a.W);
            reg[it][e] = buffer_load16(rsx, ok ? (uint32_t)(base + e * a.Ci) * ESZ : kOob);
          }
        } else {
#pragma unroll
          for (int e = 0; e < VEC; ++e) reg[it][e] = make_uint4(0, 0, 0, 0);
        }
      } else {
        // any image width: each pixel's own row and column
        const uint32_t q1 = fdiv((uint32_t)pbase, fd_w);
        int w = pbase - (int)q1 * a.W, h = (int)(q1 - fdiv(q1, fd_h) * (uint32_t)a.H);
        const int shift = (br[it] - 1) * a.W + bs[it] - 1;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const bool ok = kind[it] == 1 && bvalid[it] && pbase + e < p_end &&
                          (unsigned)(h + br[it] - 1) < (unsigned)a.H && (unsigned)(w + bs[it] - 1) < (unsigned)a.W;
          reg[it][e] = buffer_load16(
              rsx, ok ? (uint32_t)((pbase + e + shift) * a.Ci + bc[it]) * ESZ : kOob);
          if (++w == a.W) {
            w = 0;
            if (++h == a.H) h = 0;
          }
        }
      }
    }
  };
  auto store_tiles = [&](int buf, auto &reg) {
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
      if (kind[it] == 2) continue;
      if (kind[it] == 0 && do_bias) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const Pack p = __builtin_bit_cast(Pack, reg[it][e]);
#pragma unroll
          for (int q = 0; q < VEC; ++q) bsum[q] += bf16_to_f32(p.v[q]);
        }
      }
      T *dst = kind[it] == 0 ? As[buf] : Bs[buf];
      store_transposed(reg[it], dst + rowb[it] * VEC * LDR + pb[it] * VEC, LDR);
    }
  };

  const int lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave / WN) * (BM / WM), wn0 = (wave % WN) * (BN / WN);
  f32x4_t acc[TL::TM][TL::TN];
#pragma unroll
  for (int i = 0; i < TL::TM; ++i)
#pragma unroll
    for (int j = 0; j < TL::TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  if (nk > 0) {
    load_tiles(0, reg0);
    if (nk > 1) load_tiles(1, reg1);
    store_tiles(0, reg0);
  }
  __syncthreads();
  for (int kt = 0; kt < nk; kt += 2) {
    if (kt + 2 < nk) load_tiles(kt + 2, reg0);
    TL::compute(acc, As[0], Bs[0], wm0, wn0, lane);
    if (kt + 1 < nk) store_tiles(1, reg1);
    __syncthreads();
    if (kt + 1 < nk) {
      if (kt + 3 < nk) load_tiles(kt + 3, reg1);
      TL::compute(acc, As[1], Bs[1], wm0, wn0, lane);
      if (kt + 2 < nk) store_tiles(0, reg0);
      __syncthreads();
    }
  }

  const int li = lane & 15, lg = lane >> 4;
  float *dw = a.dw + split * a.dw_ss + rep * a.dw_rs;
#pragma unroll
  for (int tn = 0; tn < TL::TN; ++tn) {
    const int n = n0 + wn0 + tn * 16 + li;
#pragma unroll
    for (int tm = 0; tm < TL::TM; ++tm)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm0 + tm * 16 + lg * 4 + r;
        if (m < a.Co && n < a.nw) dw[(int64_t)m * a.nw + n] = acc[tm][tn][r];
      }
  }

  if (do_bias) {
    if (kind[0] == 0) {
#pragma unroll
      for (int q = 0; q < VEC; ++q) red[pb[0]][rowb[0] * VEC + q] = bsum[q];
    }
    __syncthreads();
    if (tid < BM) {
      const int co = m0 + tid;
      if (co < a.Co) {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < PB; ++i) s += red[i][tid];
        a.db[split * a.db_ss + rep * a.db_rs + co] = s;
      }
    }
  }
}

template <int BM, int BN, bool VB> hipError_t run_wgrad(const WgradArgs &a, hipStream_t s, std::string *label) {
  const int MT = (a.Co + BM - 1) / BM, NT = ((a.taps == 1 ? a.Ci : 9 * a.Ci) + BN - 1) / BN;
  const FastDiv fw = make_fastdiv(a.W), fh = make_fastdiv(a.H), fc = make_fastdiv(a.Ci);
  if (label)
    *label = "conv_wgrad<bf16," + std::to_string(BM) + "x" + std::to_string(BN) + ",w4" + (VB ? ",vec>" : ",anywidth>");
  hipLaunchKernelGGL((wgrad_kernel<BM, BN, VB>), dim3((uint32_t)MT * NT * a.splits * a.C), dim3(256), 0, s, a, fw, fh,
                     fc, MT, NT);
  return hipGetLastError();
}

template <bool VB> hipError_t pick_wgrad(const WgradArgs &a, hipStream_t s, std::string *label) {
  int bm, bn;
  wgrad_tile(GCPSL_BF16, a.Co, a.taps == 1 ? a.Ci : 9 * a.Ci, &bm, &bn);
  if (bm == 64) {
    if (bn == 128) return run_wgrad<64, 128, VB>(a, s, label);
    return bn == 64 ? run_wgrad<64, 64, VB>(a, s, label) : run_wgrad<64, 32, VB>(a, s, label);
  }
  if (bn == 128) return run_wgrad<32, 128, VB>(a, s, label);
  return bn == 64 ? run_wgrad<32, 64, VB>(a, s, label) : run_wgrad<32, 32, VB>(a, s, label);
}

}  // namespace

int wgrad_k_tile(int dtype) { return dtype == GCPSL_BF16 ? 64 : 32; }

void wgrad_tile(int dtype, int Co, int ncols, int *bm, int *bn) {
  const int nw = ncols;
  *bm = Co > 64 ? 128 : (Co > 32 ? 64 : 32);
  *bn = nw > 64 ? 128 : (nw > 32 ? 64 : 32);
}

bool conv_stride2(int dtype, int Csrc) { return Csrc % (dtype == GCPSL_BF16 ? 64 : 8) == 0; }

hipError_t launch_conv(int dtype, const ConvArgs &a, hipStream_t s, std::string *label) {
  if (a.stride2) {
    if (a.epi != EPI_DGRAD || !conv_stride2(dtype, a.Csrc) || a.N % 8 != 0) return hipErrorInvalidValue;
    return dtype == GCPSL_BF16 ? launch_conv_lds(a, s, label) : launch_conv_f32(a, s, label);
  }
  // routing codes: the head's pooling epilogue (halo tile) and the
  // image-side kernels take them
  if (a.pool_code) {
    if (a.epi == EPI_FWD && a.pool_max && a.pool_out && conv_fuses_avg(dtype, a)) return launch_conv_lds(a, s, label);
    return (conv_pool_codes(dtype, a) && (a.epi == EPI_DGRAD || a.pool_out)) ? launch_conv_img(a, s, label)
                                                                              : hipErrorInvalidValue;
  }
  if (a.taps == 9 && a.epi == EPI_FWD && a.res == nullptr && conv_im3_ok(dtype, a.Csrc, a.N, a.H, a.W))
    return launch_conv_col(a, s, label);
  if (conv_img_ok(dtype, a)) return launch_conv_img(a, s, label);
  if (a.epi == EPI_FWD && conv_col_ok(dtype, a)) return launch_conv_col(a, s, label);
  if (dtype != GCPSL_BF16) return launch_conv_f32(a, s, label);
  return conv_lds_ok(dtype, a) ? launch_conv_lds(a, s, label) : hipErrorInvalidValue;
}

hipError_t launch_wgrad(int dtype, const WgradArgs &a, hipStream_t s, std::string *label) {
  if (a.gcode)
    return (wgrad_pool_codes(dtype, a.Co, a.Ci, a.H, a.W, a.taps) && wgrad_lds_ok(dtype, a.Co, a.Ci) &&
            a.chunk % 64 == 0)
               ? launch_wgrad_lds(a, s, label)
               : hipErrorInvalidValue;
  if ((wgrad_col_ok(dtype, a.Co, a.Ci, a.taps) ||
       (a.taps == 9 && conv_im3_ok(dtype, a.Ci, a.Co, a.H, a.W))) && a.chunk % 128 == 0)
    return launch_wgrad_col(a, s, label);
  if (wgrad_lds_ok(dtype, a.Co, a.Ci) && a.chunk % 64 == 0) return launch_wgrad_lds(a, s, label);
  if (dtype != GCPSL_BF16) return launch_wgrad_f32(a, s, label);
  // pixel blocks within one image row (im2col rows need no image-row
  // structure), or of any width; whole 16-byte channel vectors either way (an
  // image layer of other channel counts runs on im2col rows)
  if (a.Ci % 8 != 0 || a.Co > 64) return hipErrorInvalidValue;
  return (a.taps == 1 || a.W % 8 == 0) ? pick_wgrad<true>(a, s, label) : pick_wgrad<false>(a, s, label);
}
