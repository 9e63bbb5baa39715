// 3x3 / 1x1 stride-1 convolutions on flattened pixels (gfx950, MFMA, wave64).
//
// Pixels are taken in memory order m = (n, h, w), whatever the image size: a
// workgroup owns BM consecutive pixels and BN output channels.  The input rows
// that the nine taps of those pixels can touch are the BM + 2 W + 2 consecutive
// rows from m0 - W - 1 on; per 32-channel chunk they are loaded into LDS once
// (prologue applied once per element) and tap (dy, dx) of pixel i is patch row
// i + dy W + dx.  Where that tap falls outside the image, the lane's address is
// the patch's zero row instead, so the taps need no masks and no image has to
// be a multiple of a tile.
//
// What bounds it: at the sizes it serves (a few GFLOP, tensors that stay in the
// caches) the time is latency, not rate, so every wave is given few, wide steps:
//  * WK waves split the input channels.  Each has a patch plane of its own, so
//    with one wave per plane nothing waits for another wave before the end, where
//    the partial sums are added in wave order through LDS and each wave finishes
//    FM / WK of the pixel fragments.
//  * the weights of all nine taps (bf16; three in fp32, whose MFMAs take eight
//    times as long) are in flight in registers while the patch is loaded.
//  * LDS rows of 96 bytes (bf16: 32 channels and a pad) let the 16 consecutive
//    rows of a fragment read fall in distinct banks at every tap offset, without a
//    permutation to work out per tap.
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "prof.h"

namespace petra {

namespace flatk {

constexpr int CK = 32;   // input channels per chunk (one bf16 MFMA's reduction)

template <typename T> struct Lay;
template <> struct Lay<bf16_t> {
  static constexpr int ROWB = 96, SUBS = 4, PV = 8, D = 9;
};
template <> struct Lay<float> {
  static constexpr int ROWB = 144, SUBS = 8, PV = 4, D = 3;
};

// 16 bytes of T as floats and back (rounded to T)
template <typename T> struct Piece;
template <> struct Piece<bf16_t> {
  static __device__ __forceinline__ void get(u32x4_t v, float* o) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = __uint_as_float(v[i] << 16);
      o[2 * i + 1] = __uint_as_float(v[i] & 0xffff0000u);
    }
  }
  static __device__ __forceinline__ u32x4_t put(const float* o) {
    return u32x4_t{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]), pack_bf16x2(o[4], o[5]),
                   pack_bf16x2(o[6], o[7])};
  }
};
template <> struct Piece<float> {
  static __device__ __forceinline__ void get(u32x4_t v, float* o) {
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = __uint_as_float(v[i]);
  }
  static __device__ __forceinline__ u32x4_t put(const float* o) {
    return u32x4_t{__float_as_uint(o[0]), __float_as_uint(o[1]), __float_as_uint(o[2]),
                   __float_as_uint(o[3])};
  }
};

// 4 consecutive channels of one pixel (8 bytes of bf16, 16 of fp32)
template <typename T> struct Quad;
template <> struct Quad<bf16_t> {
  u32x2_t w;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t off) { w = buf_load8(r, off); }
  __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t r, uint32_t off) const { buf_store8(w, r, off); }
  __device__ __forceinline__ void get(float* v) const {
    v[0] = __uint_as_float(w.x << 16); v[1] = __uint_as_float(w.x & 0xffff0000u);
    v[2] = __uint_as_float(w.y << 16); v[3] = __uint_as_float(w.y & 0xffff0000u);
  }
  __device__ __forceinline__ void put(const float* v) {
    w = u32x2_t{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
  }
};
template <> struct Quad<float> {
  u32x4_t w;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t off) { w = buf_load16(r, off); }
  __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t r, uint32_t off) const { buf_store16(w, r, off); }
  __device__ __forceinline__ void get(float* v) const {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = __uint_as_float(w[e]);
  }
  __device__ __forceinline__ void put(const float* v) {
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = __float_as_uint(v[e]);
  }
};

__device__ __forceinline__ void load_frag(Frag<bf16_t>& f, __amdgpu_buffer_rsrc_t r, uint32_t off) {
  f.v = __builtin_bit_cast(bf16x8_t, buf_load16(r, off));
}
__device__ __forceinline__ void load_frag(Frag<float>& f, __amdgpu_buffer_rsrc_t r, uint32_t off) {
  Piece<float>::get(buf_load16(r, off), f.v);
  Piece<float>::get(buf_load16(r, off + 16), f.v + 4);
}

template <typename T, int R, int FM, int FN, int WM, int WN, int WK, int EP, int PRO>
__global__ __launch_bounds__(64 * WM * WN * WK, 2) void conv_flat_kernel(ConvArgs a) {
  using L = Lay<T>;
  constexpr int ES = sizeof(T);
  constexpr int TAPS = R * R;
  constexpr int BM = WM * FM * 16, BN = WN * FN * 16;
  constexpr int GW = WM * WN, GT = 64 * GW;       // waves and threads per patch plane
  constexpr int D = TAPS == 1 ? 1 : L::D;         // taps whose weights are in flight
  constexpr bool BWD = PRO == PRO_BWD;
  constexpr bool STATS = EP == EP_STATS;
  constexpr bool GRAD = EP == EP_MASK || EP == EP_RESID_STATS;
  constexpr bool RES = EP == EP_RESID || EP == EP_RESID_STATS;
  constexpr int NB = BWD ? 4 : 8;                 // patch pieces in flight per thread
  constexpr int EM = FM / WK;                     // pixel fragments a wave finishes
  constexpr int EWM = WM * WK;                    // waves over pixels in the epilogue
  static_assert(FM % WK == 0, "the K waves share the pixel fragments");
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  __shared__ float red[EWM][3][BN];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wk = wave / GW, wg = wave - wk * GW;
  const int wm = wg % WM, wn = wg / WM;
  const int lr = lane & 15, lg = lane >> 4;
  const int gt = tid - wk * GT;                   // thread within its plane's group
  const int m0 = static_cast<int>(blockIdx.x) * BM, n0 = static_cast<int>(blockIdx.y) * BN;
  const int halo = R == 3 ? a.w + 1 : 0;
  const int rows = BM + 2 * halo;
  const int chunks = (a.c_in + CK - 1) / CK, cpw = chunks / WK;
  unsigned char* plane = lds + wk * (rows + 1) * L::ROWB;

  const long io_in = static_cast<long>(a.m) * a.c_in * ES;
  const __amdgpu_buffer_rsrc_t r_src = make_rsrc(a.src, io_in);
  const __amdgpu_buffer_rsrc_t r_proh = make_rsrc(BWD ? a.pro_h : a.src, io_in);
  const __amdgpu_buffer_rsrc_t r_wt = make_rsrc(a.wt, static_cast<long>(a.c_out) * a.k_tot * ES);
  const long io_out = static_cast<long>(a.m) * a.c_out * ES;
  const __amdgpu_buffer_rsrc_t r_out = make_rsrc(a.out, io_out);
  const __amdgpu_buffer_rsrc_t r_eph = make_rsrc(GRAD ? a.ep_h : a.out, GRAD ? io_out : 0);
  const __amdgpu_buffer_rsrc_t r_res = make_rsrc(RES && a.resid != nullptr ? a.resid : a.out,
                                                 RES && a.resid != nullptr ? io_out : 0);

  // Patch pieces of this thread: piece q = gt + GT i is 16 bytes of patch row
  // q / SUBS, always the same channels of a chunk.
  const int sub = gt & (L::SUBS - 1), row_t = gt / L::SUBS;
  constexpr int ROW_STEP = GT / L::SUBS;
  u32x4_t rp[NB], rh[BWD ? NB : 1];
  auto load_rows = [&](int c0, int row0) {
    const int c = c0 + sub * L::PV;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int row = row0 + row_t + ROW_STEP * i;
      const int pix = m0 - halo + row;
      const uint32_t off = row < rows && pix >= 0 && pix < a.m && c < a.c_in
                               ? static_cast<uint32_t>((static_cast<long>(pix) * a.c_in + c) * ES)
                               : BUF_OOB;
      rp[i] = buf_load16(r_src, off);
      if constexpr (BWD) rh[i] = buf_load16(r_proh, off);
    }
  };
  float pc[PRO == PRO_NONE ? 1 : BWD ? 4 : 2][L::PV];
  auto load_consts = [&](int c0) {   // zeros past c_in
    if constexpr (PRO != PRO_NONE) {
      const float* tab[4] = {BWD ? a.pro_ca : a.pro_scale, BWD ? a.pro_cb : a.pro_shift,
                             BWD ? a.pro_cc : a.pro_scale, BWD ? a.pro_mean : a.pro_scale};
#pragma unroll
      for (int t = 0; t < (BWD ? 4 : 2); ++t) {
        const __amdgpu_buffer_rsrc_t r = make_rsrc(tab[t], a.c_in * 4);
#pragma unroll
        for (int j = 0; j < L::PV; j += 4)
          Piece<float>::get(buf_load16(r, static_cast<uint32_t>(c0 + sub * L::PV + j) * 4u), &pc[t][j]);
      }
    }
  };
  auto park_rows = [&](int row0) {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int row = row0 + row_t + ROW_STEP * i;
      u32x4_t v = rp[i];
      if constexpr (PRO != PRO_NONE) {
        float x[L::PV];
        Piece<T>::get(v, x);
        if constexpr (BWD) {
          float h[L::PV];
          Piece<T>::get(rh[i], h);
#pragma unroll
          for (int j = 0; j < L::PV; ++j) x[j] = fmaf(pc[0][j], x[j], fmaf(pc[1][j], h[j] - pc[3][j], pc[2][j]));
        } else {
#pragma unroll
          for (int j = 0; j < L::PV; ++j) x[j] = fmaxf(fmaf(pc[0][j], x[j], pc[1][j]), 0.f);
        }
        v = Piece<T>::put(x);
      }
      if (row < rows) *reinterpret_cast<u32x4_t*>(plane + row * L::ROWB + sub * 16) = v;
    }
  };

  // Weight fragments: lane (lr, lg) of fragment fn holds output channel
  // n0 + wn FN 16 + fn 16 + lr, 8 input channels of one tap.
  Frag<T> wb[D][FN];
  uint32_t wrow[FN];
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) {
    const int col = n0 + (wn * FN + fn) * 16 + lr;
    wrow[fn] = col < a.c_out ? static_cast<uint32_t>(col * a.k_tot + lg * 8) * ES : BUF_OOB;
  }
  auto load_w = [&](int c0, int tap, int slot) {
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
      const bool ok = wrow[fn] != BUF_OOB && c0 + lg * 8 < a.c_in;
      load_frag(wb[slot][fn], r_wt,
                ok ? wrow[fn] + static_cast<uint32_t>(tap * a.c_in + c0) * ES : BUF_OOB);
    }
  };

  load_consts(wk * cpw * CK);
  load_rows(wk * cpw * CK, 0);
#pragma unroll
  for (int d = 0; d < D; ++d) load_w(wk * cpw * CK, d, d);

  // Epilogue operands of the fragments this wave finishes: lane (lr, lg) holds
  // channels n0 + (wn FN + fn) 16 + lg 4 .. + 3 of pixel m0 + i.
  const int ewm = wm * WK + wk;
  Quad<T> eh[GRAD ? EM : 1][FN], er[RES ? EM : 1][FN];
  uint32_t eoff[EM][FN];
#pragma unroll
  for (int f = 0; f < EM; ++f)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
      const int pix = m0 + (ewm * EM + f) * 16 + lr, c = n0 + (wn * FN + fn) * 16 + lg * 4;
      eoff[f][fn] = pix < a.m && c < a.c_out
                        ? static_cast<uint32_t>((static_cast<long>(pix) * a.c_out + c) * ES)
                        : BUF_OOB;
      if constexpr (GRAD) eh[f][fn].load(r_eph, eoff[f][fn]);
      if constexpr (RES) er[f][fn].load(r_res, eoff[f][fn]);
    }

  // LDS address of this lane's pixels and, per pixel, the taps inside the image
  // (bit 3 dy + dx): lane l works pixel l out, the lanes that hold it fetch it.
  static_assert(FM <= 4, "a lane per pixel");
  int arow[FM];
  uint32_t inside[FM];
  {
    uint32_t mask = ~0u;
    if constexpr (R == 3) {
      const int pix = min(m0 + wm * FM * 16 + lane, a.m - 1);
      const int rem = pix % (a.h * a.w);
      const int y = rem / a.w, x = rem - y * a.w;
      mask = (y > 0 ? 0007u : 0u) | 0070u | (y < a.h - 1 ? 0700u : 0u);
      mask &= (x > 0 ? 0111u : 0u) | 0222u | (x < a.w - 1 ? 0444u : 0u);
    }
#pragma unroll
    for (int fm = 0; fm < FM; ++fm) {
      arow[fm] = ((wm * FM + fm) * 16 + lr) * L::ROWB + lg * (L::SUBS / 4) * 16;
      inside[fm] = __shfl(mask, fm * 16 + lr, 64);
    }
  }
  const int zero_row = rows * L::ROWB;
  if (gt < L::SUBS) *reinterpret_cast<u32x4_t*>(plane + zero_row + gt * 16) = u32x4_t{0u, 0u, 0u, 0u};

  f32x4_t acc[FM][FN];
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  auto join = [&]() {   // the plane's writes are seen by its waves
    if constexpr (GW > 1) {
      __syncthreads();
    } else {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  };
  for (int ck = 0; ck < cpw; ++ck) {
    const int c0 = (wk * cpw + ck) * CK;
    if (ck > 0) {
      join();   // the previous chunk has been read
      load_consts(c0);
      load_rows(c0, 0);
    }
    park_rows(0);
    for (int row0 = ROW_STEP * NB; row0 < rows; row0 += ROW_STEP * NB) {
      load_rows(c0, row0);
      park_rows(row0);
    }
    join();
#pragma unroll
    for (int t = 0; t < TAPS; ++t) {
      Frag<T> af[FM];
      const int toff = R == 3 ? (t / 3 * a.w + t % 3) * L::ROWB : 0;
#pragma unroll
      for (int fm = 0; fm < FM; ++fm)
        af[fm].load(reinterpret_cast<const T*>(
            plane + (R == 1 || (inside[fm] >> t & 1u) ? arow[fm] + toff : zero_row)));
#pragma unroll
      for (int fm = 0; fm < FM; ++fm)
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = mfma(wb[t % D][fn], af[fm], acc[fm][fn]);
      // refill the slot: D taps ahead, over the chunk's end (wave-uniform branch)
      if (t + D < TAPS)
        load_w(c0, t + D, t % D);
      else if (ck + 1 < cpw)
        load_w(c0 + CK, t + D - TAPS, t % D);
    }
  }

  // Partial sums of the K waves, added in wave order; wave wk keeps fragments
  // wk EM .. wk EM + EM - 1.
  f32x4_t out[EM][FN];
  if constexpr (WK > 1) {
    __syncthreads();   // every plane has been read
    f32x4_t* xch = reinterpret_cast<f32x4_t*>(lds);
    auto slot = [&](int k, int fm, int fn) { return (((k * GW + wg) * FM + fm) * FN + fn) * 64 + lane; };
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
      if (fm / EM != wk) {
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) xch[slot(wk, fm, fn)] = acc[fm][fn];
      }
    __syncthreads();
#pragma unroll
    for (int f = 0; f < EM; ++f)
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) {
        f32x4_t own{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < WK; ++k)
          if (k == wk) own = acc[k * EM + f][fn];
        f32x4_t s{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < WK; ++k) s += k == wk ? own : xch[slot(k, wk * EM + f, fn)];
        out[f][fn] = s;
      }
  } else {
#pragma unroll
    for (int f = 0; f < EM; ++f)
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) out[f][fn] = acc[f][fn];
  }

  // Epilogue on D[cout][pixel]: each lane stores 4 channels of one pixel; BN sums
  // go over the wave's pixels with DPP and over the waves in LDS, and are written as
  // partial row blockIdx.x: the sum and, about the wave's mean, the squares.
  float es[FN][4], esh[FN][4], emu[FN][4], ers[FN][4];
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) {
    const int c0 = n0 + (wn * FN + fn) * 16 + lg * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool ok = GRAD && c0 < a.c_out;
      es[fn][e] = ok && EP == EP_MASK ? a.ep_scale[c0 + e] : 0.f;
      esh[fn][e] = ok && EP == EP_MASK ? a.ep_shift[c0 + e] : 0.f;
      emu[fn][e] = ok ? a.ep_mean[c0 + e] : 0.f;
      ers[fn][e] = ok ? a.ep_rstd[c0 + e] : 0.f;
    }
  }
  float sa[FN][4], sb[FN][4], nv = 0.f;
#pragma unroll
  for (int fn = 0; fn < FN; ++fn)
#pragma unroll
    for (int e = 0; e < 4; ++e) sa[fn][e] = sb[fn][e] = 0.f;
#pragma unroll
  for (int f = 0; f < EM; ++f) {
    const bool vm = m0 + (ewm * EM + f) * 16 + lr < a.m;
    nv += vm ? 1.f : 0.f;
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
      float v[4] = {out[f][fn][0], out[f][fn][1], out[f][fn][2], out[f][fn][3]};
      float hl[4] = {0.f, 0.f, 0.f, 0.f};
      if constexpr (GRAD) eh[f][fn].get(hl);
      if constexpr (RES) {
        float rv[4];
        er[f][fn].get(rv);   // a null residual reads zeros
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] += rv[e];
      }
      if constexpr (EP == EP_MASK) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = fmaf(es[fn][e], hl[e], esh[fn][e]) > 0.f ? v[e] : 0.f;
      }
      Quad<T> q;
      q.put(v);
      q.store(r_out, eoff[f][fn]);
      q.get(v);   // statistics of the stored values
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = vm ? v[e] : 0.f;
        if constexpr (STATS) out[f][fn][e] = v[e];
        sa[fn][e] += v[e];
        if constexpr (GRAD) sb[fn][e] += v[e] * ((hl[e] - emu[fn][e]) * ers[fn][e]);
      }
    }
  }
  if constexpr (STATS || GRAD) {
    const float n16 = sum16(nv);
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x = sum16(sa[fn][e]);
        if constexpr (STATS) {
          const float mean = n16 > 0.f ? x / n16 : 0.f;
#pragma unroll
          for (int f = 0; f < EM; ++f) {
            const float d = m0 + (ewm * EM + f) * 16 + lr < a.m ? out[f][fn][e] - mean : 0.f;
            sb[fn][e] = fmaf(d, d, sb[fn][e]);
          }
        }
        const float y = sum16(sb[fn][e]);
        if (lr == 0) {
          const int c = (wn * FN + fn) * 16 + lg * 4 + e;
          red[ewm][0][c] = n16;
          red[ewm][1][c] = x;
          red[ewm][2][c] = y;
        }
      }
    __syncthreads();
    for (int c = tid; c < BN; c += 64 * WM * WN * WK) {
      const int col = n0 + c;
      if (col >= a.c_out) continue;
      const long row = static_cast<long>(blockIdx.x);
      float n = 0.f, t1 = 0.f, t2 = 0.f;
#pragma unroll
      for (int w = 0; w < EWM; ++w) {
        n += red[w][0][c];
        t1 += red[w][1][c];
        t2 += red[w][2][c];
      }
      if constexpr (STATS) {
        // from the waves' means to the tile's (the first wave always has rows)
        if constexpr (EWM > 1) {
          const float mean = t1 / n;
#pragma unroll
          for (int w = 0; w < EWM; ++w) {
            const float nb = red[w][0][c], d = nb > 0.f ? red[w][1][c] / nb - mean : 0.f;
            t2 = fmaf(nb * d, d, t2);
          }
        }
        a.partials[(row * 3 + 0) * a.c_out + col] = n;
        a.partials[(row * 3 + 1) * a.c_out + col] = t1;
        a.partials[(row * 3 + 2) * a.c_out + col] = t2;
      } else {
        a.partials[(row * 2 + 0) * a.c_out + col] = t1;
        a.partials[(row * 2 + 1) * a.c_out + col] = t2;
      }
    }
  }
}

template <typename T, int R, int FM, int FN, int WM, int WN, int WK>
bool launch(const ConvArgs& a, int ep, hipStream_t st) {
  constexpr int BM = WM * FM * 16, BN = WN * FN * 16;
  const int rows = BM + (R == 3 ? 2 * (a.w + 1) : 0);
  const size_t planes = static_cast<size_t>(WK) * (rows + 1) * Lay<T>::ROWB;
  const size_t xch = WK > 1 ? static_cast<size_t>(WK) * WM * WN * FM * FN * 1024 : 0;
  const size_t shm = std::max(planes, xch);
  const dim3 grid((a.m + BM - 1) / BM, (a.c_out + BN - 1) / BN), block(64 * WM * WN * WK);
#define PETRA_FLAT(EP_, PRO_)                                                                   \
  PETRA_LAUNCH((conv_flat_kernel<T, R, FM, FN, WM, WN, WK, EP_, PRO_>), grid, block, shm, st, a)
  const bool bwd = a.pro_h != nullptr;
  if (ep == EP_STATS && !bwd) {
    if (a.pro_scale != nullptr)
      PETRA_FLAT(EP_STATS, PRO_RELU);
    else
      PETRA_FLAT(EP_STATS, PRO_NONE);
  } else if (ep == EP_MASK && bwd) {
    PETRA_FLAT(EP_MASK, PRO_BWD);
  } else if (ep == EP_RESID && bwd) {
    PETRA_FLAT(EP_RESID, PRO_BWD);
  } else if (ep == EP_RESID_STATS && bwd) {
    PETRA_FLAT(EP_RESID_STATS, PRO_BWD);
  } else {
    return false;
  }
#undef PETRA_FLAT
  return true;
}

// Tile shapes (FM, FN, WM, WN, WK).  Measured alone, us per launch with BN-apply
// / masked input-gradient prologue and epilogue, against the im2col kernels these
// shapes ran on before (conv_staged for bf16, conv_gemm for fp32):
//  * F_K4 64 x 32, four K waves: 128x4x4 256->256 11.0 / 11.6 (before: 52 / 58),
//    128x8x8 128->128 10.8 / 11.9 (36 / 42); fp32 16x14x14 128->128 17.3 / 16.4.
//  * F_K2 64 x 64, two K waves, two channel waves: the same 8x8 shape 10.8 / 11.8,
//    but 64x14x14 128->128 15.5 / 19.2 against 18.0 / 20.8 for F_K4, which needs
//    the patch, prologue included, once per 32 output channels: F_K4 where F_K2
//    would not give every CU a workgroup.  64x28x28 64->64 18.6 / 23.1 (23 / 29).
//  * F_M128 128 x 32, F_M64 64 x 32, four pixel waves: one chunk of channels.
//    37x23x23 32->32 6.2 / 6.0 and 7.0 / 7.2 (15.4 / 18.3); 8x32x32 6.1 / 5.8 and
//    5.8 / 5.3: the smaller one below one tile per CU.
//  * fp32, one chunk: F_N2 64 x 32 over 2 x 2 waves, 32x32x32 32->32 10.6 / 12.0
//    (19.9 / 27.5); F_N1 64 x 16, four pixel waves, for at most 16 output channels,
//    8x8x8 16->16 5.7 / 5.0 (9.2 / 12.1).
enum Shape { F_NO = 0, F_K4, F_K2, F_M128, F_M64, F_N2, F_N1 };

struct Tile { int bm, wk; };
constexpr Tile TILE[] = {{0, 0}, {64, 4}, {64, 2}, {128, 1}, {64, 1}, {64, 1}, {64, 1}};
constexpr long MAX_LDS = 60 << 10;   // dynamic LDS of a launch (patch planes)

// Whether the im2col kernels (bf16: conv_staged, fp32 and 16 channels: conv_gemm) take
// less time.  A workgroup here loads its patch, multiplies and stores once, without
// overlap, which a few of them per CU hide; with many, the im2col kernels' wider tiles
// win, which read each pixel for 128 output channels and each weight for 128 pixels.
// Lines from the time of each conv against theirs, widths 7 to 64, 4k to 400k pixels
// (64 x 64 tiles; below / above the line):
//  * 3x3, 64 to 512 channels: 1280 tiles.  64 channels 64k / 98k pixels 0.81 - 1.04 /
//    0.92 - 1.20, 128 channels 32k / 64k 0.76 - 0.96 / 1.04 - 1.27, 256 channels 16k /
//    32k below 0.91 / 0.95 - 1.21.  Wider images have more halo rows in a patch: 64
//    pixels wide, 128 channels, 24k / 32k pixels at most 0.8 / 1.14, hence the bound
//    on tiles times patch rows.
//  * 1x1: 960 tiles.  256 -> 64 channels 48k / 80k pixels 0.78 - 0.89 / 0.97 - 1.08.
//    Forwards to more channels stay: 64 -> 256, 98k pixels, 0.87.  Input gradients with
//    a residual read it beside the two prologue tensors: 768 tiles, and 512 with the
//    32-channel tiles.  64 -> 256 16k / 32k pixels 0.86 - 1.06 / 0.94 - 1.21, 128 -> 512
//    4k / 12k 0.90 / 1.04 - 1.17, 32 -> 64 24k / 64k 0.86 - 0.93 / 1.02 - 1.22.
//  * 16 input channels, 3x3 forwards, half of a chunk empty: bf16 48k / 98k pixels
//    0.85 - 0.95 / 1.09 - 1.16, fp32 32k / 64k 0.92 - 0.99 / 1.04 - 1.06.
//  * fp32 1x1 forwards to 16 channels, a quarter of a tile: 1.0 / 1.5 at 4k / 64k.
bool im2col_better(int dtype, const ConvArgs& a, int ep) {
  if (dtype == DT_FP32)
    return ep == EP_STATS && ((a.r == 1 && a.c_out <= 16) || (a.r == 3 && a.c_in == 16 && a.m > 48 << 10));
  if (a.c_in == 16) return ep == EP_STATS && a.r == 3 && a.m > 64 << 10;
  if (a.c_in % 32 != 0) return false;
  const long tiles = static_cast<long>((a.m + 63) / 64) * ((a.c_out + 63) / 64);
  if (a.r == 3) return a.c_in > 32 && (tiles > 1280 || tiles * (64 + 2 * (a.w + 1)) > 190000);
  if (ep == EP_RESID || ep == EP_RESID_STATS) return tiles > (a.c_in == 32 ? 512 : 768);
  return a.c_in > 32 && (ep != EP_STATS || a.c_out <= a.c_in) && tiles > 960;
}

Shape shape_of(int dtype, const ConvArgs& a, int ep) {
  const bool fp32 = dtype == DT_FP32;
  if (!(a.src2 == nullptr && (a.r == 3 || a.r == 1) && a.s == a.r && a.stride == 1 &&
        a.pad == a.r / 2 && a.p == a.h && a.q == a.w && a.k_tot == a.r * a.r * a.c_in &&
        a.c_in % 8 == 0 && a.c_out % 8 == 0 && a.c_in >= 16))
    return F_NO;
  // forward convs and input gradients with their BN backward (PRO_BWD)
  if (ep == EP_STATS ? a.pro_h != nullptr : a.pro_h == nullptr) return F_NO;
  const long esz = fp32 ? 4 : 2;
  // byte offsets of the buffer loads/stores are 32-bit
  if (static_cast<long>(a.m) * std::max(a.c_in, a.c_out) * esz >= static_cast<long>(BUF_OOB)) return F_NO;
  if (im2col_better(dtype, a, ep)) return F_NO;
  const int chunks = (a.c_in + CK - 1) / CK;
  const long rowb = fp32 ? Lay<float>::ROWB : Lay<bf16_t>::ROWB;
  auto fits = [&](Shape s) {
    const long rows = TILE[s].bm + (a.r == 3 ? 2 * (a.w + 1) : 0) + 1;
    return chunks % TILE[s].wk == 0 && TILE[s].wk * rows * rowb <= MAX_LDS;
  };
  const long k2_tiles = static_cast<long>((a.m + 63) / 64) * ((a.c_out + 63) / 64);
  if (fits(F_K4) && (fp32 || k2_tiles <= 256)) return F_K4;
  if (fits(F_K2)) return F_K2;
  if (fp32) {
    if (a.c_out <= 16 && fits(F_N1)) return F_N1;
    return fits(F_N2) ? F_N2 : F_NO;
  }
  // the pixel waves go over several chunks one after the other: 64 channels 160 x 160
  // 123 against the im2col kernel's 95 us a forward, 128 channels 128 x 128 191 / 160
  if (chunks > 1) return F_NO;
  if ((a.m + 127) / 128 < 256 && fits(F_M64)) return F_M64;
  return fits(F_M128) ? F_M128 : F_NO;
}

template <typename T, int R>
bool launch_shape(Shape s, const ConvArgs& a, int ep, hipStream_t st) {
  switch (s) {
    case F_K4: return launch<T, R, 4, 2, 1, 1, 4>(a, ep, st);
    case F_K2: return launch<T, R, 4, 2, 1, 2, 2>(a, ep, st);
    default: break;
  }
  if constexpr (sizeof(T) == 2) {
    if (s == F_M128) return launch<T, R, 2, 2, 4, 1, 1>(a, ep, st);
    if (s == F_M64) return launch<T, R, 1, 2, 4, 1, 1>(a, ep, st);
  } else {
    if (s == F_N2) return launch<T, R, 2, 1, 2, 2, 1>(a, ep, st);
    if (s == F_N1) return launch<T, R, 1, 1, 4, 1, 1>(a, ep, st);
  }
  return false;
}

}  // namespace flatk
using namespace flatk;

int conv_flat_tiles(int dtype, const ConvArgs& a, int ep) {
  const Shape s = shape_of(dtype, a, ep);
  return s == F_NO ? 0 : (a.m + TILE[s].bm - 1) / TILE[s].bm;
}

bool conv_flat(int dtype, const ConvArgs& a, int ep, hipStream_t st) {
  const Shape s = shape_of(dtype, a, ep);
  if (s == F_NO) return false;
  if (dtype == DT_BF16)
    return a.r == 3 ? launch_shape<bf16_t, 3>(s, a, ep, st) : launch_shape<bf16_t, 1>(s, a, ep, st);
  return a.r == 3 ? launch_shape<float, 3>(s, a, ep, st) : launch_shape<float, 1>(s, a, ep, st);
}

}  // namespace petra
