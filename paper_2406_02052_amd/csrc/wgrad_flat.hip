// Weight gradient on flattened pixels (gfx950, MFMA, wave64):
//   part[split][o][tap*C_in + c] = sum over the split's pixels of dh[px][o] * x[px + tap][c]
// for 3x3 and 1x1 stride-1 convolutions of any image size, bf16 and fp32.
//
// As in the convolutions on flattened pixels, a tile is P consecutive pixels in
// memory order; a 3x3 conv's input rows are the P + 2 W + 2 consecutive ones around
// them, and a tap that leaves the image reads the patch's zero row (one bit per
// pixel and tap, worked out once per tile).  Both tiles stay in LDS as loaded,
// [pixel][channel].  bf16 operands need pixels along the reduction and come from
// transposing reads (lane 4 r + q of 16 addresses quarter q of a 16-channel run of
// pixel r and lane j receives channel j of 4 pixels); the fp32 MFMA takes one value
// per lane, 16 channels of 4 pixels.  A workgroup owns BO output x BC input channels
// and all taps over a strided set of tiles, the next one in flight in registers and
// parked in the other half of LDS (one barrier per tile).  Waves split the output
// channels (WO), the input channels (WC), the taps (WT) and, with their sums added
// in order at the end, the pixels (WP).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "prof.h"

namespace petra {

namespace wflat {

template <typename T> struct Pix;   // LDS pitch, 16-byte pieces
template <> struct Pix<bf16_t> {
  static constexpr int PV = 8;
  static constexpr int pitch(int c) { return c + 16; }
};
template <> struct Pix<float> {
  static constexpr int PV = 4;
  // four rows of 16 floats in distinct banks
  static constexpr int pitch(int c) { return c == 16 ? 16 : c + 16; }
};

// WO x WC x WT waves of one pixel group own OF x CF fragments of R R / WT taps.
template <typename T_, int R_, int WO_, int OF_, int WC_, int CF_, int WT_, int WP_, int P_>
struct Cfg {
  using T = T_;
  static constexpr int R = R_, WO = WO_, OF = OF_, WC = WC_, CF = CF_, WT = WT_, WP = WP_, P = P_;
  static constexpr int NW = WO * WC * WT, NT = 64 * NW * WP;
  static constexpr int BO = WO * OF * 16, BC = WC * CF * 16, TPW = R * R / WT;
  static constexpr int PV = Pix<T>::PV, PO = Pix<T>::pitch(BO), PC = Pix<T>::pitch(BC);
  static constexpr int DG = BO / PV, XG = BC / PV;   // 16-byte pieces per row
  static constexpr int KP = sizeof(T) == 2 ? 32 : 4; // pixels per MFMA
  // A third of the waves (at least one) load dh and the BN tensor beside it, the
  // others the input: a wave then holds one side's channel constants and pieces.
  static constexpr int ND = 64 * (NW * WP >= 3 ? NW * WP / 3 : 1), NX = NT - ND;
  static constexpr int D_PT = (P * DG + ND - 1) / ND;
  // pieces of the input patch per thread, rounded up: 3x3 plans take images up to 63
  // pixels wide (fp32: 95 with 16 channels; 61 with 64, by LDS).  One more piece would
  // be a register more for every width.
  static constexpr int X_PT = ((P + (R == 3 ? 122 : 0)) * XG + NX - 1) / NX;
  static constexpr int MAX_ROWS = X_PT * NX / XG;
  static_assert(TPW * WT == R * R && ND % DG == 0 && NX % XG == 0 && P % (KP * WP) == 0, "tile");
  // Workgroups of a launch, over all its layers: as many as fit on 256 CUs at once, and
  // two where more, smaller partials cost more.  Weight gradients and reduces of a
  // backward with 256 / 512 / 768: 64x28x28 64 -> 16 and back 45 / 41 / 47 us, 256 -> 64
  // (128x28x28) 270 (in 128-pixel tiles, 82 KB of LDS) / 229 / 188, im2col kernels 267;
  // fp32 64 -> 64 296 / 297 / 303.
  static constexpr int WGS = R == 3 || sizeof(T) == 4 ? 256 : BO * BC == 64 * 64 ? 768 : 512;
  static int rows(int w) { return P + (R == 3 ? 2 * (w + 1) : 0); }
  static size_t lds(int w) {
    const size_t tile = (static_cast<size_t>(P) * PO + static_cast<size_t>(rows(w) + 1) * PC) * sizeof(T);
    const size_t xch = WP > 1 ? static_cast<size_t>(NW) * OF * CF * TPW * 1024 : 0;
    return std::max(2 * (tile + P * sizeof(uint16_t)), xch);
  }
};

typedef short v4i16 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8_t tr_frag(const bf16_t* p0, const bf16_t* p1) {
  const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16*)(p0));
  const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16*)(p1));
  return __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <typename T> __device__ __forceinline__ void get16(u32x4_t v, float* o);
template <> __device__ __forceinline__ void get16<bf16_t>(u32x4_t v, float* o) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    o[2 * i] = __uint_as_float(v[i] << 16);
    o[2 * i + 1] = __uint_as_float(v[i] & 0xffff0000u);
  }
}
template <> __device__ __forceinline__ void get16<float>(u32x4_t v, float* o) {
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = __uint_as_float(v[i]);
}
template <typename T> __device__ __forceinline__ u32x4_t put16(const float* o);
template <> __device__ __forceinline__ u32x4_t put16<bf16_t>(const float* o) {
  return u32x4_t{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]), pack_bf16x2(o[4], o[5]),
                 pack_bf16x2(o[6], o[7])};
}
template <> __device__ __forceinline__ u32x4_t put16<float>(const float* o) {
  return u32x4_t{__float_as_uint(o[0]), __float_as_uint(o[1]), __float_as_uint(o[2]), __float_as_uint(o[3])};
}

template <typename C>
__device__ __forceinline__ void body(const WgradArgs& a, int bx, int by, int bz, int splits, int nbz) {
  using T = typename C::T;
  constexpr int R = C::R, ES = sizeof(T), PV = C::PV, P = C::P, NT = C::NT, NW = C::NW;
  constexpr int OF = C::OF, CF = C::CF, TPW = C::TPW, WP = C::WP, PO = C::PO, PC = C::PC;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const bool pro = a.pro_scale != nullptr;   // BN-apply + ReLU prologue of the conv input
  const int halo = R == 3 ? a.w + 1 : 0, rows = P + 2 * halo;
  // halves of LDS: dh tile, patch and its zero row, tap bits
  const int half_t = P * PO + (rows + 1) * PC;   // elements of T
  T* tiles = reinterpret_cast<T*>(lds);
  uint16_t* bits = reinterpret_cast<uint16_t*>(tiles + 2 * half_t);

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wo = wave % C::WO, wc = (wave / C::WO) % C::WC, wt = (wave / (C::WO * C::WC)) % C::WT;
  const int wp = wave / NW;
  const int li = lane & 15, kg = lane >> 4;
  const int o0 = by * C::BO, c0 = bz * C::BC;
  const int ntiles = (a.m + P - 1) / P;
  const __amdgpu_buffer_rsrc_t r_x = make_rsrc(a.src, static_cast<long>(a.m) * a.c_in * ES);
  const __amdgpu_buffer_rsrc_t r_d = make_rsrc(a.dh, static_cast<long>(a.m) * a.c_out * ES);
  const __amdgpu_buffer_rsrc_t r_h = make_rsrc(a.dh_h, static_cast<long>(a.m) * a.c_out * ES);

  // The wave's side, this thread's channels of it and their coefficients (dh: ca, cb,
  // cc, mean; input: scale, shift).
  const bool dside = wave < C::ND / 64;
  const int lt = dside ? tid : tid - C::ND;
  const int og = lt % C::DG, cg = lt % C::XG;
  float k[4][PV];
#pragma unroll
  for (int j = 0; j < PV; ++j) {
    const int o = o0 + og * PV + j, c = c0 + cg * PV + j;
    k[0][j] = dside ? a.dh_ca[o] : pro ? a.pro_scale[c] : 0.f;
    k[1][j] = dside ? a.dh_cb[o] : pro ? a.pro_shift[c] : 0.f;
    k[2][j] = dside ? a.dh_cc[o] : 0.f;
    k[3][j] = dside ? a.dh_mean[o] : 0.f;
  }
  constexpr int NR = 2 * C::D_PT > C::X_PT ? 2 * C::D_PT : C::X_PT;
  u32x4_t r[NR];   // dh and h in turn, or the input
  auto load_tile = [&](int t) {
    if (dside) {
#pragma unroll
      for (int i = 0; i < C::D_PT; ++i) {
        const int px = (lt + C::ND * i) / C::DG, m = t * P + px;
        const uint32_t off = px < P && m < a.m
                                 ? static_cast<uint32_t>((static_cast<long>(m) * a.c_out + o0 + og * PV) * ES)
                                 : BUF_OOB;
        r[2 * i] = buf_load16(r_d, off);
        r[2 * i + 1] = buf_load16(r_h, off);
      }
    } else {
#pragma unroll
      for (int i = 0; i < C::X_PT; ++i) {
        const int row = (lt + C::NX * i) / C::XG, m = t * P - halo + row;
        const uint32_t off = row < rows && m >= 0 && m < a.m
                                 ? static_cast<uint32_t>((static_cast<long>(m) * a.c_in + c0 + cg * PV) * ES)
                                 : BUF_OOB;
        r[i] = buf_load16(r_x, off);
      }
    }
  };
  auto park_tile = [&](int t, int buf) {
    T* sd = tiles + buf * half_t;
    T* sx = sd + P * PO;
    if (dside) {
#pragma unroll
      for (int i = 0; i < C::D_PT; ++i) {
        const int px = (lt + C::ND * i) / C::DG;
        if (px >= P) continue;
        float v[PV], h[PV];
        get16<T>(r[2 * i], v);
        get16<T>(r[2 * i + 1], h);
#pragma unroll
        for (int j = 0; j < PV; ++j) v[j] = fmaf(k[0][j], v[j], fmaf(k[1][j], h[j] - k[3][j], k[2][j]));
        u32x4_t w = put16<T>(v);
        if (t * P + px >= a.m) w = u32x4_t{0u, 0u, 0u, 0u};   // pixels past the end add nothing
        *reinterpret_cast<u32x4_t*>(sd + px * PO + og * PV) = w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < C::X_PT; ++i) {
        const int row = (lt + C::NX * i) / C::XG;
        if (row >= rows) continue;
        u32x4_t w = r[i];
        if (pro) {
          float v[PV];
          get16<T>(w, v);
#pragma unroll
          for (int j = 0; j < PV; ++j) v[j] = fmaxf(fmaf(k[0][j], v[j], k[1][j]), 0.f);
          w = put16<T>(v);
        }
        *reinterpret_cast<u32x4_t*>(sx + row * PC + cg * PV) = w;
      }
    }
    if constexpr (R == 3) {
      for (int i = tid; i < P; i += NT) {
        const int rem = min(t * P + i, a.m - 1) % (a.h * a.w);
        const int y = rem / a.w, x = rem - y * a.w;
        const uint32_t in_y = (y > 0 ? 0007u : 0u) | 0070u | (y < a.h - 1 ? 0700u : 0u);
        const uint32_t in_x = (x > 0 ? 0111u : 0u) | 0222u | (x < a.w - 1 ? 0444u : 0u);
        bits[buf * P + i] = static_cast<uint16_t>(in_y & in_x);
      }
    }
  };

  f32x4_t acc[OF][CF][TPW];
#pragma unroll
  for (int of = 0; of < OF; ++of)
#pragma unroll
    for (int cf = 0; cf < CF; ++cf)
#pragma unroll
      for (int u = 0; u < TPW; ++u) acc[of][cf][u] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int zero_row = rows * PC;
  for (int i = tid; i < 2 * C::XG; i += NT) {
    T* z = tiles + (i / C::XG) * half_t + P * PO + zero_row;
    *reinterpret_cast<u32x4_t*>(z + (i % C::XG) * PV) = u32x4_t{0u, 0u, 0u, 0u};
  }
  // patch row shift of this wave's taps, in elements
  int toff[TPW];
#pragma unroll
  for (int u = 0; u < TPW; ++u) {
    const int tap = wt * TPW + u;
    toff[u] = R == 3 ? (tap / 3 * a.w + tap % 3) * PC : 0;
  }

  // Loads are unconditional (the last tile again past the end), so their number in
  // flight does not depend on the path.
  int t = bx, buf = 0;
  load_tile(min(t, ntiles - 1));
  for (; t < ntiles; t += splits) {
    park_tile(t, buf);
    __syncthreads();
    load_tile(min(t + splits, ntiles - 1));
    const T* sd = tiles + buf * half_t + wo * OF * 16;
    const T* sx = tiles + buf * half_t + P * PO + wc * CF * 16;
    const uint16_t* bt = bits + buf * P;
    if constexpr (ES == 2) {
#pragma unroll
      for (int ks = 0; ks < P / 32 / WP; ++ks) {
        const int pa = (ks * WP + wp) * 32 + kg * 8 + (li >> 2), pb = pa + 4;
        const int qo = (li & 3) * 4;
        const uint32_t ma = R == 3 ? bt[pa] : 0u, mb = R == 3 ? bt[pb] : 0u;
        Frag<bf16_t> fa[OF];
#pragma unroll
        for (int of = 0; of < OF; ++of)
          fa[of].v = tr_frag(sd + pa * PO + qo + of * 16, sd + pb * PO + qo + of * 16);
#pragma unroll
        for (int u = 0; u < TPW; ++u) {
          const int tap = wt * TPW + u;
          const int xa = R == 1 || (ma >> tap & 1u) ? pa * PC + toff[u] : zero_row;
          const int xb = R == 1 || (mb >> tap & 1u) ? pb * PC + toff[u] : zero_row;
#pragma unroll
          for (int cf = 0; cf < CF; ++cf) {
            Frag<bf16_t> fb;
            fb.v = tr_frag(sx + xa + qo + cf * 16, sx + xb + qo + cf * 16);
#pragma unroll
            for (int of = 0; of < OF; ++of) acc[of][cf][u] = mfma(fa[of], fb, acc[of][cf][u]);
          }
        }
      }
    } else {
#pragma unroll 4
      for (int ks = 0; ks < P / 4 / WP; ++ks) {
        const int px = (ks * WP + wp) * 4 + kg;
        const uint32_t mk = R == 3 ? bt[px] : 0u;
        float fa[OF];
#pragma unroll
        for (int of = 0; of < OF; ++of) fa[of] = load1(sd + px * PO + of * 16 + li);
#pragma unroll
        for (int u = 0; u < TPW; ++u) {
          const int xo = R == 1 || (mk >> (wt * TPW + u) & 1u) ? px * PC + toff[u] : zero_row;
#pragma unroll
          for (int cf = 0; cf < CF; ++cf) {
            const float fb = load1(sx + xo + cf * 16 + li);
#pragma unroll
            for (int of = 0; of < OF; ++of)
              acc[of][cf][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[of], fb, acc[of][cf][u], 0, 0, 0);
          }
        }
      }
    }
    buf ^= 1;
  }

  // Pixel groups 1.. add their sums into group 0 through LDS, in order.
  constexpr int NFRAG = OF * CF * TPW;
  if constexpr (WP > 1) {
    f32x4_t* xch = reinterpret_cast<f32x4_t*>(lds);
#pragma unroll
    for (int g = 1; g < WP; ++g) {
      __syncthreads();   // the tiles, then the previous group's sums, have been read
      if (wp == g) {
#pragma unroll
        for (int f = 0; f < NFRAG; ++f)
          xch[((wave % NW) * NFRAG + f) * 64 + lane] = acc[f / TPW / CF][f / TPW % CF][f % TPW];
      }
      __syncthreads();
      if (wp == 0) {
#pragma unroll
        for (int f = 0; f < NFRAG; ++f)
          acc[f / TPW / CF][f / TPW % CF][f % TPW] += xch[(wave * NFRAG + f) * 64 + lane];
      }
    }
    if (wp > 0) return;
  }
  // Partials in fragment order (whole cache lines), as the split reduce expects.
  const long wg_base = (static_cast<long>(by) * nbz + bz) * NW + wave % NW;
  float* outp = a.partials + static_cast<long>(bx) * a.c_out * a.k_tot;
#pragma unroll
  for (int f = 0; f < NFRAG; ++f)
    *reinterpret_cast<f32x4_t*>(outp + (wg_base * NFRAG + f) * 256 + lane * 4) =
        acc[f / TPW / CF][f / TPW % CF][f % TPW];
}

template <typename C>
__global__ __launch_bounds__(C::NT) void wgrad_flat_kernel(WgradArgs a) {
  body<C>(a, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.x, gridDim.z);
}

// Several layers of one plan in one launch, as wgrad_tr_group_kernel.
template <typename C>
__global__ __launch_bounds__(C::NT) void wgrad_flat_group_kernel(WgGroupTable tab) {
  const long b = blockIdx.x;
  int i = 0;
  for (int e = 1; e < tab.n; ++e)
    if (tab.block_begin[e] <= b) i = e;
  const WgradArgs& a = tab.a[i];
  const long local = b - tab.block_begin[i];
  const int nby = a.c_out / C::BO, nbz = a.c_in / C::BC;
  const long r = local / a.splits;
  body<C>(a, static_cast<int>(local % a.splits), static_cast<int>(r % nby), static_cast<int>(r / nby),
          a.splits, nbz);
}

template <typename C>
void launch(const WgradArgs* args, int n, hipStream_t st) {
  if (n == 1) {
    const WgradArgs& a = args[0];
    PETRA_LAUNCH(wgrad_flat_kernel<C>, dim3(a.splits, a.c_out / C::BO, a.c_in / C::BC), dim3(C::NT),
                 C::lds(a.w), st, a);
    return;
  }
  for (int i0 = 0; i0 < n; i0 += MAX_WG_GROUP) {
    WgGroupTable tab{};
    tab.n = std::min(MAX_WG_GROUP, n - i0);
    long blocks = 0;
    size_t shm = 0;
    for (int i = 0; i < tab.n; ++i) {
      const WgradArgs& a = args[i0 + i];
      tab.a[i] = a;
      tab.block_begin[i] = blocks;
      blocks += static_cast<long>(a.splits) * (a.c_out / C::BO) * (a.c_in / C::BC);
      shm = std::max(shm, C::lds(a.w));
    }
    PETRA_LAUNCH(wgrad_flat_group_kernel<C>, dim3(static_cast<unsigned>(blocks)), dim3(C::NT), shm, st, tab);
  }
}

// Plans, by type, taps and channel blocks.  A workgroup takes 64, 32 or 16 output
// and input channels, whatever divides the layer's.  3x3: three waves of taps times
// four of channels (64 x 64), or of channels and pixels; 1x1: four waves of pixels.
// Four layers in one launch, one workgroup per CU: 64x28x28 64->64 33.7 us (im2col:
// 4 x 35 us and a reduce after each), 128x8x8 128->128 25.7 us (the kernel for 8x8
// tiles 30.2 us).  Register-bound: tiles of 128 pixels 51.2 and 37.2 us, all waves
// loading both sides (both sides' constants and pieces in every thread) 49.6 and
// 37.4 us, all nine taps in one wave 52.1 and 37.0 us.  bf16 1x1 of 64 x 64 channels:
// 2 x 2 waves of channels and 64 pixels, so that three workgroups fit on a CU.
template <typename T> struct Plans {
  static constexpr int P1 = sizeof(T) == 2 ? 128 : 64;
  using C64 = Cfg<T, 3, 2, 2, 2, 2, 3, 1, 64>;
  using C32 = std::conditional_t<sizeof(T) == 2, Cfg<T, 3, 1, 2, 2, 1, 3, 2, 128>,
                                 Cfg<T, 3, 1, 2, 1, 2, 3, 4, 64>>;
  using C16 = Cfg<T, 3, 1, 1, 1, 1, 3, 4, P1>;
  template <int OF, int CF> using One =
      std::conditional_t<sizeof(T) == 2 && OF == 4 && CF == 4, Cfg<T, 1, 2, 2, 2, 2, 1, 1, 64>,
                         Cfg<T, 1, 1, OF, 1, CF, 1, 4, P1>>;
};

// Calls f with the configuration of a plan (block sizes bo, bc in channels).
template <typename T, typename F>
bool with_cfg(int r, int bo, int bc, F&& f) {
  using P = Plans<T>;
  if (r == 3) {
    if (bo != bc) return false;
    if (bo == 64) { f(typename P::C64{}); return true; }
    if (bo == 32) { f(typename P::C32{}); return true; }
    if (bo == 16) { f(typename P::C16{}); return true; }
    return false;
  }
  switch (bo * 100 + bc) {
    case 6464: f(typename P::template One<4, 4>{}); return true;
    case 6432: f(typename P::template One<4, 2>{}); return true;
    case 6416: f(typename P::template One<4, 1>{}); return true;
    case 3264: f(typename P::template One<2, 4>{}); return true;
    case 3232: f(typename P::template One<2, 2>{}); return true;
    case 3216: f(typename P::template One<2, 1>{}); return true;
    case 1664: f(typename P::template One<1, 4>{}); return true;
    case 1632: f(typename P::template One<1, 2>{}); return true;
    case 1616: f(typename P::template One<1, 1>{}); return true;
    default: return false;
  }
}

int block_of(int c) { return c % 64 == 0 ? 64 : c == 32 || c == 16 ? c : 0; }

template <typename F>
bool with_plan(int dtype, const WgradArgs& a, F&& f) {
  const int bo = block_of(a.c_out), bc = block_of(a.c_in);
  return dtype == DT_BF16 ? with_cfg<bf16_t>(a.r, bo, bc, f) : with_cfg<float>(a.r, bo, bc, f);
}

constexpr size_t MAX_LDS = 160 * 1024 - 512;

}  // namespace wflat
using namespace wflat;

int wgrad_flat_plan(int dtype, const WgradArgs& a, int* splits) {
  if (!(a.src2 == nullptr && a.stride == 1 && a.r == a.s && (a.r == 3 || a.r == 1) && a.pad == a.r / 2 &&
        a.p == a.h && a.q == a.w && a.k_tot == a.r * a.r * a.c_in && a.dh_h != nullptr))
    return 0;
  const long esz = dtype == DT_BF16 ? 2 : 4;
  // byte offsets of the buffer loads are 32-bit
  if (static_cast<long>(a.m) * std::max(a.c_in, a.c_out) * esz >= static_cast<long>(BUF_OOB)) return 0;
  // By themselves the 1x1 layers of many pixels are no faster than the im2col kernel,
  // and slower beside other streams' work (16x64x64 256 -> 64 and back, 64 wide: 4k
  // pixels 77 against 117 us a backward, 64k 206 / 203, a step of two blocks 1416 / 1406)
  if (a.layers == 0 && a.r == 1 && a.m > 48 << 10) return 0;
  bool fits = false;
  int sp = 1;
  with_plan(dtype, a, [&](auto c) {
    using C = decltype(c);
    fits = C::rows(a.w) <= C::MAX_ROWS && C::lds(a.w) <= MAX_LDS;
    // one workgroup per CU of the 3x3 plans (four layers of 28x28 64->64: 33.7 us with
    // 64 each, 41.1 with 128; of fp32 32x32x32 32->32 34.9 and 39.4 us; backward of two
    // blocks of 64x28x28 as one launch with 64 each 549 us, with 32 531)
    const int per = (a.c_out / C::BO) * (a.c_in / C::BC);
    sp = std::max(1, std::min((a.m + C::P - 1) / C::P, wgrad_share(C::WGS, a) / per));
  });
  if (!fits) return 0;
  if (splits) *splits = sp;
  // one number per configuration: layers with the same one can share a launch
  return WGRAD_FLAT_PLAN + (a.r == 3 ? 0 : 1) + 2 * (block_of(a.c_out) + 128 * block_of(a.c_in));
}

bool wgrad_flat_map(int dtype, const WgradArgs& a, TrMap* out) {
  return with_plan(dtype, a, [&](auto c) {
    using C = decltype(c);
    *out = TrMap{C::WO, C::OF, C::WC, C::CF, C::WT, C::TPW, C::BO, C::BC, a.c_in / C::BC, a.c_in, a.k_tot};
  });
}

bool wgrad_flat(int dtype, const WgradArgs* args, int n, hipStream_t st) {
  return with_plan(dtype, args[0], [&](auto c) { launch<decltype(c)>(args, n, st); });
}

}  // namespace petra
