// FP64 3x3 stride-2 convolutions on v_mfma_f64_16x16x4: the building blocks of the FP64 tier
// (f64.hip) and of the crop predicates (crop.hip).
//
// One MFMA tile is 16 output channels (A, weights) x 16 output positions (B, activations) and four
// products deep.  Both operands are read straight from memory in the layout they already have:
// a lane's four consecutive input channels of one tap are 16 bytes of fp32 weights ([co][tap][ci])
// and 32 bytes of FP64 activations (NHWC), one element for each of four MFMAs (lane group g of 16
// holds channels 4g..4g+3 of a 16-channel block, the same on both sides, so the order in which the
// MFMAs take them does not matter).  An MFMA holds its SIMD for 64 cycles, four of them 256, so
// the 48 bytes per lane that feed them come from L1 / L2 with nothing staged in LDS.
//
// The result's row of register r, lane group g is 4r + g (read back from a lane-layout probe);
// the weight rows are permuted so that it holds channel 4g + r, and each lane stores four
// consecutive channels of its position.
#pragma once

#include "common.h"

namespace hydro {

typedef double doublex4 __attribute__((ext_vector_type(4)));

// The raw frame that layer 1 reads: pixel (y, x) of the image is pixel (y0 + y, x0 + x) of a frame
// of row_px pixels per row.
struct Image64 {
  const void* base;      // first element of the frame
  int dtype;
  int row_px;
  int y0, x0;
};

__device__ inline Image64 image64(const FrameSrc& fr, uint32_t idx, int row_px, int y0, int x0) {
  const size_t item = fr.dtype == HYDRO_DTYPE_F32 ? 4 : fr.dtype == HYDRO_DTYPE_BF16 ? 2 : 1;
  return Image64{static_cast<const char*>(fr.base) + (size_t)idx * (size_t)fr.elems * item, fr.dtype, row_px, y0, x0};
}

// Normalised value of one element (the frame exactly as the definition has it, in FP64).
__device__ inline double image64_at(const Image64& im, int y, int x, int c) {
  const int o = ((im.y0 + y) * im.row_px + im.x0 + x) * 3 + c;
  double v;
  if (im.dtype == HYDRO_DTYPE_BF16) v = (double)(float)static_cast<const __bf16*>(im.base)[o];
  else if (im.dtype == HYDRO_DTYPE_U8) v = (double)static_cast<const uint8_t*>(im.base)[o] / 255.0;
  else v = (double)static_cast<const float*>(im.base)[o];
  return (v - 0.5) * 4.0;
}

// One layer: weights [cout][9][cin] fp32 (cin = 3 for the first layer, else a multiple of 16; cout a
// multiple of 16), bias [cout], input hin x win, output ho x wo = ceil(hin / 2) x ceil(win / 2).
struct Conv64 {
  const float* w;
  const float* bias;
  int cin, cout, hin, win, ho, wo;
};

// 16-channel blocks of the sum (all nine taps); the first layer's 27 products are one block.
__device__ inline int conv64_blocks(const Conv64& L, bool first) { return first ? 1 : 9 * (L.cin >> 4); }

// acc[c] += the products of blocks [b0, b1) for channels o0 + 16 c .. + 15 and positions p0 .. p0 + 15
// (positions past the image contribute zeros).
template <bool FIRST, int CT>
__device__ inline void conv64_acc(const Conv64& L, const Image64& im, const double* in, int p0, int o0, int b0, int b1,
                                  doublex4 (&acc)[CT]) {
  const int lane = lane_id(), g = lane >> 4, l16 = lane & 15;
  const int p = p0 + l16, i = p / L.wo, j = p - i * L.wo;
  const bool pok = i < L.ho;
  const int co = o0 + 4 * (l16 & 3) + (l16 >> 2);          // this lane's weight row (permuted, see above)
  if constexpr (FIRST) {
    // k = 4q + g = tap * 3 + channel, 27 of 28 used
    const float* w = L.w + (size_t)co * 27;
    double xv[7];
#pragma unroll
    for (int q = 0; q < 7; ++q) {
      const int k = 4 * q + g, t = k / 3, c = k - 3 * t;
      const int y = 2 * i + t / 3 - 1, x = 2 * j + t % 3 - 1;
      xv[q] = pok && k < 27 && y >= 0 && x >= 0 && y < L.hin && x < L.win ? image64_at(im, y, x, c) : 0.0;
    }
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int q = 0; q < 7; ++q) {
        const int k = 4 * q + g;
        const double wv = k < 27 ? (double)w[c * 16 * 27 + k] : 0.0;
        acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(wv, xv[q], acc[c], 0, 0, 0);
      }
  } else {
    const int nc = L.cin >> 4;
    const size_t row = (size_t)9 * L.cin;
    const float* w = L.w + (size_t)co * row + 4 * g;
    int t = b0 / nc, c0 = b0 - t * nc;
    for (int b = b0; b < b1; ++t, c0 = 0) {
      const int y = 2 * i + t / 3 - 1, x = 2 * j + t % 3 - 1;
      const bool ok = pok && y >= 0 && x >= 0 && y < L.hin && x < L.win;
      const double* xp = in + ((size_t)(ok ? y : 0) * L.win + (ok ? x : 0)) * L.cin + 4 * g;
      const int be = min(b1, b + nc - c0);
#pragma unroll 4
      for (int bb = b; bb < be; ++bb) {
        doublex4 xv = *reinterpret_cast<const doublex4*>(xp + (size_t)(c0 + bb - b) * 16);
        floatx4 wv[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) wv[c] = *reinterpret_cast<const floatx4*>(w + c * 16 * row + (size_t)bb * 16);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const double xq = ok ? xv[q] : 0.0;
#pragma unroll
          for (int c = 0; c < CT; ++c) acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)wv[c][q], xq, acc[c], 0, 0, 0);
        }
      }
      b = be;
    }
  }
}

// Bias, ReLU and store of one tile (out: [position][cout]).
template <int CT>
__device__ inline void conv64_store(const Conv64& L, const doublex4 (&acc)[CT], double* out, int p0, int o0) {
  const int lane = lane_id(), g = lane >> 4, l16 = lane & 15;
  if (p0 + l16 >= L.ho * L.wo) return;
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int ch = o0 + 16 * c + 4 * g;
    doublex4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double s = acc[c][r] + (double)L.bias[ch + r];
      v[r] = s > 0.0 ? s : 0.0;
    }
    *reinterpret_cast<doublex4*>(out + (size_t)(p0 + l16) * L.cout + ch) = v;
  }
}

template <bool FIRST, int CT>
__device__ inline void conv64_wg_tiles(const Conv64& L, const Image64& im, const double* in, double* out, int wave,
                                       int waves) {
  const int pt = (L.ho * L.wo + 15) >> 4, tiles = pt * (L.cout / (16 * CT));
  for (int t = wave; t < tiles; t += waves) {
    const int p0 = (t % pt) * 16, o0 = (t / pt) * 16 * CT;
    doublex4 acc[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[c] = (doublex4){0.0, 0.0, 0.0, 0.0};
    conv64_acc<FIRST, CT>(L, im, in, p0, o0, 0, conv64_blocks(L, FIRST), acc);
    conv64_store<CT>(L, acc, out, p0, o0);
  }
}

// One layer of one image by a whole workgroup, one tile per wave at a time.  A wave takes four (two)
// channel tiles at once where that still leaves every wave a tile: each activation it reads then
// feeds four (two) times the MFMAs.
template <bool FIRST>
__device__ inline void conv64_wg(const Conv64& L, const Image64& im, const double* in, double* out, int wave, int waves) {
  const int ct = L.cout >> 4, pt = (L.ho * L.wo + 15) >> 4;
  if ((ct & 3) == 0 && pt * (ct >> 2) >= waves) conv64_wg_tiles<FIRST, 4>(L, im, in, out, wave, waves);
  else if ((ct & 1) == 0 && pt * (ct >> 1) >= waves) conv64_wg_tiles<FIRST, 2>(L, im, in, out, wave, waves);
  else conv64_wg_tiles<FIRST, 1>(L, im, in, out, wave, waves);
}

// Mean pool over P positions of [P][ld] activations (the first C of ld channels, ld a multiple of
// 16), FC and the ten logits, by a workgroup of THREADS threads (a power of two, at least 64).
// part: THREADS doubles of LDS, g: C doubles, z: kClasses doubles; z is readable by every thread on
// return.
template <int THREADS>
__device__ inline void head64_wg(const double* act, int P, int C, int ld, const float* fc_w, const float* fc_b,
                                 double* part, double* g, double* z) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int parts = ld < THREADS ? THREADS / ld : 1;
  for (int c0 = 0; c0 < ld; c0 += THREADS) {
    const int q = ld < THREADS ? tid / ld : 0, ch = ld < THREADS ? tid % ld : c0 + tid;
    double s = 0.0;
    if (q < parts && ch < C)
      for (int p = q; p < P; p += parts) s += act[(size_t)p * ld + ch];
    part[tid] = s;
    __syncthreads();
    if (q == 0 && ch < C) {
      for (int u = 1; u < parts; ++u) s += part[u * ld + ch];
      g[ch] = s / (double)P;
    }
    __syncthreads();
  }
  for (int c = wave; c < kClasses; c += THREADS / 64) {
    double s = 0.0;
    for (int ch = lane; ch < C; ch += 64) s = fma(g[ch], (double)fc_w[ch * kClasses + c], s);
    for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) z[c] = s + (double)fc_b[c];
  }
  __syncthreads();
}

}  // namespace hydro
