// FP64 3x3 stride-2 convolutions on v_mfma_f64_16x16x4: the building blocks of the FP64 tier
// (f64.hip) and of the crop predicates (crop.hip).
//
// One MFMA tile is 16 output channels (A, weights) x 16 output positions (B, activations) and four
// products deep.  A lane's four channels of a 16-channel block (lane group g of 16 holds channels
// 4g..4g+3, the same on both sides, so the order in which the MFMAs take them does not matter) are one
// element each for four MFMAs.  An MFMA holds its SIMD for 64 cycles, four of them 256, so the 48 bytes
// per lane that feed them come from L1 / L2 with nothing staged in LDS - if neighbouring lanes read
// neighbouring bytes: a wave's 16-byte load takes the CU's address unit 16 cycles then, and 64 with a
// row per lane (weights [co][tap][ci] and activations NHWC kept it busy for three times the MFMAs'
// time).  Weights are packed in the order the lanes take them (conv64_pack); activations between
// layers are planes of two channels, a row's even columns before its odd ones, so that the positions of
// a tile, which read every second column, read one run.
//
// Fewer than 16 input channels would leave most of such a block empty: there the products (tap, channel) are
// packed one after the other, as the first layer's are, and gathered one by one (3,000 crops of 64x64 frames,
// widths 1-1: 511 us padded, 349 so; 4-8-16 at 32x32 in the allocation-free array, where the padding also
// cost workgroups: 390, 314).
//
// The result's row of register r, lane group g is 4r + g (read back from a lane-layout probe);
// the weight rows are permuted so that it holds channel 4g + r, and each lane stores four
// consecutive channels of its position.
#pragma once

#include "engine.h"

namespace hydro {

typedef double doublex4 __attribute__((ext_vector_type(4)));
typedef double doublex2 __attribute__((ext_vector_type(2)));

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

// Normalised value of one element (the frame exactly as the definition has it, in FP64: 4 (v - 1/2) is
// one rounding either way).
__device__ inline double image64_norm(double v) { return fma(v, 4.0, -2.0); }
__device__ inline double image64_value(float v) { return image64_norm((double)v); }
__device__ inline double image64_value(__bf16 v) { return image64_norm((double)(float)v); }
__device__ inline double image64_value(uint8_t b) {
  // b / 255 correctly rounded: the product with 1 / 255, corrected once (equal for all 256 bytes)
  constexpr double r = 1.0 / 255.0;
  const double q = (double)b * r;
  return image64_norm(fma(fma(-255.0, q, (double)b), r, q));
}

// One layer: weights fp32 as conv64_pack leaves them (cin = 3 for the first layer, else below 16 or a
// multiple of 16; cout a multiple of 16, of which the first cstore are stored), bias [cout], input hin x win,
// output ho x wo = ceil(hin / 2) x ceil(win / 2).  last: the output is [position][cstore], for the head.
struct Conv64 {
  const float* w;
  const float* bias;
  int cin, cout, cstore, hin, win, ho, wo;
  bool last;
};
enum { CONV64_WIDE, CONV64_FIRST, CONV64_NARROW };     // kinds of input: whole blocks, the frame, below 16 channels

// Index of channel ch at position (i, j) in a layer's output.
__device__ inline int conv64_at(const Conv64& L, int i, int j, int ch) {
  if (L.last) return (i * L.wo + j) * L.cstore + ch;
  const int wh = (L.wo + 1) >> 1;
  return ((((ch >> 1) * L.ho + i) * 2 + (j & 1)) * wh + (j >> 1)) * 2 + (ch & 1);
}

// 16-channel blocks of the sum (all nine taps); other kinds' products are one block.
__device__ inline int conv64_blocks(const Conv64& L, int kind) { return kind == CONV64_WIDE ? 9 * (L.cin >> 4) : 1; }

// acc[c] += the products of blocks [b0, b1) for channels o0 + 16 c .. + 15 and positions p0 .. p0 + 15
// (positions past the image contribute zeros).
template <int KIND, int CT>
__device__ inline void conv64_acc(const Conv64& L, const Image64& im, const double* in, int p0, int o0, int b0, int b1,
                                  doublex4 (&acc)[CT]) {
  const int lane = lane_id(), g = lane >> 4, l16 = lane & 15;
  const int p = p0 + l16, i = p / L.wo, j = p - i * L.wo;
  // taps inside the image, bit 3 u + v
  const uint32_t cols = (j > 0 ? 1u : 0u) | 2u | (2 * j + 1 < L.win ? 4u : 0u);
  const uint32_t inside = i < L.ho ? (i > 0 ? cols : 0u) | cols << 3 | (2 * i + 1 < L.hin ? cols << 6 : 0u) : 0u;
  if constexpr (KIND == CONV64_FIRST) {
    // k = 4q + g = tap * 3 + channel, 27 of 28 used (tap 9 is never inside)
    const floatx4* w = reinterpret_cast<const floatx4*>(L.w) + ((size_t)(o0 >> 4) * 64 + lane) * 2;
    const int at = i < L.ho ? ((im.y0 + 2 * i) * im.row_px + im.x0 + 2 * j) * 3 : 0;   // element of tap (1, 1)
    double xv[7];
    auto gather = [&](auto* src) {
#pragma unroll
      for (int q = 0; q < 7; ++q) {
        const int k = 4 * q + g, t = k / 3, u = t / 3;
        const int o = ((u - 1) * im.row_px + t - 3 * u - 1) * 3 + k - 3 * t;
        const bool ok = (inside >> t) & 1u;
        const double v = image64_value(src[ok ? at + o : 0]);
        xv[q] = ok ? v : 0.0;
      }
    };
    if (im.dtype == HYDRO_DTYPE_BF16) gather(static_cast<const __bf16*>(im.base));
    else if (im.dtype == HYDRO_DTYPE_U8) gather(static_cast<const uint8_t*>(im.base));
    else gather(static_cast<const float*>(im.base));
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      const floatx4 wl = w[c * 128], wh = w[c * 128 + 1];
#pragma unroll
      for (int q = 0; q < 7; ++q)
        acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)(q < 4 ? wl[q & 3] : wh[q & 3]), xv[q], acc[c], 0, 0, 0);
    }
  } else if constexpr (KIND == CONV64_NARROW) {
    // k = 4q + g = tap * cin + channel, below 9 cin (taps from 9 on are never inside); four steps per load
    const int n4 = conv64_narrow_steps(L.cin) / 4, wh = (L.win + 1) >> 1;
    const uint32_t inv = 65536u / L.cin + 1;             // k / cin = k inv >> 16 (k < 144, cin < 16)
    const floatx4* w = reinterpret_cast<const floatx4*>(L.w) + ((size_t)(o0 >> 4) * 64 + lane) * n4;
    for (int b = 0; b < n4; ++b) {
      double xv[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = 16 * b + 4 * q + g, t = (int)((uint32_t)k * inv >> 16), ch = k - t * L.cin;
        const int u = (t * 11) >> 5, v = t - 3 * u;      // t / 3 (t < 16)
        const bool ok = (inside >> t) & 1u;
        const int at = ((((ch >> 1) * L.hin + 2 * i + u - 1) * 2 + (v == 1 ? 0 : 1)) * wh + j - (v == 0 ? 1 : 0)) * 2 + (ch & 1);
        const double x = in[ok ? at : 0];
        xv[q] = ok ? x : 0.0;
      }
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        const floatx4 wv = w[(size_t)c * 64 * n4 + b];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)wv[q], xv[q], acc[c], 0, 0, 0);
      }
    }
  } else {
    const int nc = L.cin >> 4, wh = (L.win + 1) >> 1, plane = L.hin * wh * 2;
    const floatx4* w = reinterpret_cast<const floatx4*>(L.w) + (size_t)(o0 >> 4) * 9 * nc * 64 + lane;
    // tap (1, 1), in the even columns; tap columns 0 and 2 are odd columns j - 1 and j
    const doublex2* xg = reinterpret_cast<const doublex2*>(in) + 2 * g * plane + 4 * i * wh + j;
    int t = b0 / nc, c0 = b0 - t * nc;
    for (int b = b0; b < b1; ++t, c0 = 0) {
      const int u = t / 3, v = t - 3 * u;
      const bool ok = (inside >> t) & 1u;
      const doublex2* xp = ok ? xg + (u - 1) * 2 * wh + (v == 1 ? 0 : v == 0 ? wh - 1 : wh)
                              : reinterpret_cast<const doublex2*>(in);
      const int be = min(b1, b + nc - c0);
#pragma unroll 4
      for (int bb = b; bb < be; ++bb) {
        const doublex2 x01 = xp[(c0 + bb - b) * 8 * plane], x23 = xp[((c0 + bb - b) * 8 + 1) * plane];
        const double xv[4] = {x01[0], x01[1], x23[0], x23[1]};
        floatx4 wv[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) wv[c] = w[((size_t)c * 9 * nc + bb) * 64];
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

// Bias, ReLU and store of one tile.
template <int CT>
__device__ inline void conv64_store(const Conv64& L, const doublex4 (&acc)[CT], double* out, int p0, int o0) {
  const int lane = lane_id(), g = lane >> 4, l16 = lane & 15;
  const int p = p0 + l16, i = p / L.wo, j = p - i * L.wo;
  if (i >= L.ho) return;
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int ch = o0 + 16 * c + 4 * g;
    doublex4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double s = acc[c][r] + (double)L.bias[ch + r];
      v[r] = s > 0.0 ? s : 0.0;
    }
    if (ch < L.cstore) *reinterpret_cast<doublex2*>(out + conv64_at(L, i, j, ch)) = (doublex2){v[0], v[1]};
    if (ch + 2 < L.cstore) *reinterpret_cast<doublex2*>(out + conv64_at(L, i, j, ch + 2)) = (doublex2){v[2], v[3]};
  }
}

template <int KIND, int CT>
__device__ inline void conv64_wg_tiles(const Conv64& L, const Image64& im, const double* in, double* out, int wave,
                                       int waves) {
  const int pt = (L.ho * L.wo + 15) >> 4, tiles = pt * (L.cout / (16 * CT));
  for (int t = wave; t < tiles; t += waves) {
    const int p0 = (t % pt) * 16, o0 = (t / pt) * 16 * CT;
    doublex4 acc[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[c] = (doublex4){0.0, 0.0, 0.0, 0.0};
    conv64_acc<KIND, CT>(L, im, in, p0, o0, 0, conv64_blocks(L, KIND), acc);
    conv64_store<CT>(L, acc, out, p0, o0);
  }
}

// One layer of one image by a whole workgroup, one tile per wave at a time.  A wave takes four (two)
// channel tiles at once where that still leaves every wave a tile: each activation it reads then
// feeds four (two) times the MFMAs.
template <int KIND>
__device__ inline void conv64_wg(const Conv64& L, const Image64& im, const double* in, double* out, int wave, int waves) {
  const int ct = L.cout >> 4, pt = (L.ho * L.wo + 15) >> 4;
  if (KIND != CONV64_NARROW && (ct & 3) == 0 && pt * (ct >> 2) >= waves) conv64_wg_tiles<KIND, 4>(L, im, in, out, wave, waves);
  else if ((ct & 1) == 0 && pt * (ct >> 1) >= waves) conv64_wg_tiles<KIND, 2>(L, im, in, out, wave, waves);
  else conv64_wg_tiles<KIND, 1>(L, im, in, out, wave, waves);
}

// Mean pool over P positions of [P][ld] activations (the first C of ld channels), FC and the ten logits, by a workgroup of THREADS threads (a power of two, at least 64).
// part: THREADS doubles of LDS, g: C doubles, z: kClasses doubles; z is readable by every thread on
// return.
template <int THREADS>
__device__ inline void head64_wg(const double* act, int P, int C, int ld, const float* fc_w, const float* fc_b,
                                 double* part, double* g, double* z) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int parts = ld < THREADS ? min(THREADS / ld, 64) : 1;
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
