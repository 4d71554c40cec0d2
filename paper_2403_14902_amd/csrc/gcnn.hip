// Generic CNN predicates on gfx950 (any square input divisible by 2^L, up to 4 conv3x3/s2
// layers with widths that are multiples of 16): used when a model's activations do not fit the
// fused per-frame kernel (e.g. 128x128 frames with 4 layers).
//
// Each layer is one implicit-GEMM launch over every queued frame of the tier: rows = output
// positions of all frames (a tile of 128 or 256 rows may span frames), columns = output channels, K = (tap, input channel).  Activations live in a
// per-tier scratch (bf16 or fp32, NHWC per frame).  Layer 1 reads the raw frame (bf16 or uint8,
// exact in bf16) with the normalisation folded into its weights and border taps set to the raw
// value that normalises to zero.  A head launch pools, applies FC and decides.  The FP64 tier
// is in f64.hip.
#include <algorithm>
#include <type_traits>

#include "engine.h"

namespace hydro {

// K of a layer: layer 1 uses 27 of 32 slots in g_first_k's order; later layers k = (u*3 + v)*Cin + c,
// padded to whole MFMA steps of 32.
__host__ __device__ inline int g_ksteps(int layer, int cin) { return layer == 0 ? 1 : (9 * cin + 31) / 32; }

// What K slot k (0..31) of the first layer holds: value r (0..8: three pixels of three channels)
// of input row u.  Slots 8u..8u+7 are the first eight values of row u, 24..26 the ninth value of
// rows 0..2: a lane (which holds eight consecutive slots) then reads one staged row, or three words.
__host__ __device__ inline bool g_first_k(int k, int* u, int* r) {
  *u = k < 24 ? k / 8 : k - 24 < 3 ? k - 24 : 0;
  *r = k < 24 ? k % 8 : 8;
  return k < 27;
}

// Output channel of row r of a layer's channel tile ct.  Of two tiles, lane group g of 16 holds rows
// 4g .. 4g + 3 each: channels 8g .. 8g + 7 of the pair's 32, so that a lane stores 16 bytes of bf16, not
// 8 a tile (a store takes the address unit a cycle per 64 bytes that it touches).
__host__ __device__ inline int g_channel(int cout, int ct, int r) {
  return cout % 32 == 0 ? (ct >> 1) * 32 + 8 * (r >> 2) + 4 * (ct & 1) + (r & 3) : ct * 16 + r;
}

// Bias, ReLU and store of channels ch .. ch + 3 (o and b: theirs); returns the largest ...
template <typename T>
__device__ inline float store_relu4(T* o, floatx4 v, float4 b) {
  const float v0 = fmaxf(v[0] + b.x, 0.f), v1 = fmaxf(v[1] + b.y, 0.f);
  const float v2 = fmaxf(v[2] + b.z, 0.f), v3 = fmaxf(v[3] + b.w, 0.f);
  if constexpr (sizeof(T) == 2) {
    alignas(8) __bf16 h[4] = {static_cast<__bf16>(v0), static_cast<__bf16>(v1), static_cast<__bf16>(v2), static_cast<__bf16>(v3)};
    *reinterpret_cast<uint2*>(o) = *reinterpret_cast<const uint2*>(h);
  } else {
    *reinterpret_cast<float4*>(o) = make_float4(v0, v1, v2, v3);
  }
  return fmaxf(fmaxf(v0, v1), fmaxf(v2, v3));
}
// ... or ch .. ch + 7, from the two tiles of a pair.
template <typename T>
__device__ inline float store_relu8(T* o, floatx4 v, floatx4 w, const float* b) {
  const float4 b0 = *reinterpret_cast<const float4*>(b), b1 = *reinterpret_cast<const float4*>(b + 4);
  if constexpr (sizeof(T) == 2) {
    alignas(16) __bf16 h[8];
    const float m0 = store_relu4(h, v, b0), m1 = store_relu4(h + 4, w, b1);
    *reinterpret_cast<uint4*>(o) = *reinterpret_cast<const uint4*>(h);
    return fmaxf(m0, m1);
  } else {
    const float m0 = store_relu4(o, v, b0), m1 = store_relu4(o + 4, w, b1);
    return fmaxf(m0, m1);
  }
}

// FP32 arithmetic from bf16 terms holds for finite values: of an infinity the split leaves inf - inf, and
// products of its terms have either sign.  Values from 2^96 on (raw ones of a frame; an activation leaves a
// mark with its frame, byte l of act_wide for layer l's output, which the head clears) and layers
// with a weight from 2^30 on (wide_w) are multiplied in fp32 instead, on the same operands: the weight is the
// sum of its terms, and fp32 step j takes value j of every lane.
constexpr float G_WIDE = 7.9228162514264338e28f;      // 2^96
constexpr uint32_t G_WIDE_BF = 0x6F80;                // its bf16 bits
__device__ inline bool wide_bf16(bf16x8 x) {
  u32x4 u;
  __builtin_memcpy(&u, &x, sizeof(u));
  uint32_t m = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) m = max(m, max(u[w] >> 16 & 0x7FFFu, u[w] & 0x7FFFu));
  return m >= G_WIDE_BF;
}
__device__ inline float wide_weight(const __bf16* hi, const __bf16* mid, const __bf16* lo) {
  return ((float)*hi + (float)*mid) + (float)*lo;
}
// One channel tile of the first layer in FP32, from the lane's fragments of the weights' terms: every product
// of a frame value and a term is exact.
__device__ inline floatx4 mfma_first(const __bf16* hi, const __bf16* mid, const __bf16* lo, bf16x8 x, bool wide) {
  floatx4 c = (floatx4){0.f, 0.f, 0.f, 0.f};
  if (wide) {
    u32x4 u;
    __builtin_memcpy(&u, &x, sizeof(u));
#pragma unroll 1
    for (int j = 0; j < 8; ++j) {       // (rolled: a rare path, which is to cost the others no registers)
      const uint32_t d = j < 4 ? j < 2 ? u[0] : u[1] : j < 6 ? u[2] : u[3];
      const float xv = __uint_as_float(j & 1 ? d & 0xFFFF0000u : d << 16);
      c = __builtin_amdgcn_mfma_f32_16x16x4f32(wide_weight(hi + j, mid + j, lo + j), xv, c, 0, 0, 0);
    }
    return c;
  }
  auto frag = [](const __bf16* p) { return *reinterpret_cast<const bf16x8*>(p); };
  return mfma_bf16(frag(hi), x, mfma_bf16(frag(mid), x, mfma_bf16(frag(lo), x, c)));
}
__device__ inline void mark_wide(const GcnnArgs& a, int64_t frame, int layer) {
  reinterpret_cast<uint8_t*>(a.act_wide)[frame * 4 + layer] = 1;
}

constexpr int GT_M = 64;     // positions per tile
constexpr int GT_N = 64;     // channels per tile

// One channel tile of the first layer, weights from memory.
template <typename T>
__device__ inline floatx4 first_mfma(const GcnnArgs& a, int slot, int tile, int lane, bf16x8 x, bool wide) {
  const __bf16* hi = a.w_bf[slot][0] + tile * 512 + lane * 8;
  if constexpr (sizeof(T) == 4) {
    const int64_t n = (int64_t)(a.widths[slot][0] / 16) * 512;       // elements of a term's image
    const __bf16* mid = a.w_ml[slot][0] + tile * 512 + lane * 8;
    return mfma_first(hi, mid, mid + n, x, wide);
  }
  return mfma_bf16(*reinterpret_cast<const bf16x8*>(hi), x, (floatx4){0.f, 0.f, 0.f, 0.f});
}

// First layer of shapes that gconv_first_kernel does not take, one wave per 16 positions, its gather
// straight from the frame (any in_hw, any Cout).
template <typename T>
__global__ __launch_bounds__(256) void gconv_first_any_kernel(GcnnArgs a) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, l16 = lane & 15;
  // tiles per predicate slot: ceil(count * P / 64) position tiles x ceil(Cout / 64) channel tiles
  auto tiles_of = [&](int i) {
    const int hout = a.in_hw[i] >> 1;
    const int64_t rows = (int64_t)a.q.counts[a.pred[i]] * hout * hout;
    return (int)((rows + GT_M - 1) / GT_M) * ((a.widths[i][0] + GT_N - 1) / GT_N);
  };
  int total = 0;
  for (int i = 0; i < a.n_preds; ++i) total += tiles_of(i);
  for (int t = blockIdx.x; t < total; t += gridDim.x) {
    int slot = 0, off = t, ebase = 0;
    for (int i = 0; i < a.n_preds; ++i) {
      const int c = tiles_of(i);
      if (off < c) { slot = i; break; }
      off -= c;
      ebase += a.q.counts[a.pred[i]];
    }
    const int k = a.pred[slot];
    const int cnt = a.q.counts[k];
    const int hin = a.in_hw[slot], hout = hin >> 1, P = hout * hout;
    const int cout = a.widths[slot][0];
    const int nct = (cout + GT_N - 1) / GT_N;
    const int mt = off / nct, ct = off % nct;
    const int ncw = min(4, cout / 16 - ct * 4);         // channel tiles of 16 in this tile
    // this wave's 16 positions
    const int64_t row = (int64_t)mt * GT_M + wave * 16 + l16;
    const bool rvalid = row < (int64_t)cnt * P;
    const int e = rvalid ? (int)(row / P) : 0;
    const int p = rvalid ? (int)(row % P) : 0;
    const int oi = p / hout, oj = p % hout;
    const uint32_t idx = entry_idx(a.q.entries[(int64_t)k * a.q.cap + e]);
    floatx4 acc[4];
    auto raw_at = [&](int u, int v, int c) {
      const int y = 2 * oi + u - 1, x = 2 * oj + v - 1;
      if (y < 0 || x < 0 || y >= hin || x >= hin) return a.pad_raw;
      const int64_t o = (int64_t)idx * a.fr.elems + ((int64_t)y * hin + x) * 3 + c;
      return a.fr.dtype == HYDRO_DTYPE_BF16 ? (float)static_cast<const __bf16*>(a.fr.base)[o]
                                            : (float)static_cast<const uint8_t*>(a.fr.base)[o];
    };
    alignas(16) __bf16 t8[8];            // exact: frame values fit bf16
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      int u, r;
      const bool used = g_first_k(8 * g + q, &u, &r);
      t8[q] = static_cast<__bf16>(used && rvalid ? raw_at(u, r / 3, r % 3) : 0.f);
    }
    const bf16x8 av = *reinterpret_cast<const bf16x8*>(t8);
    const bool wide = sizeof(T) == 4 && ((a.wide_w[slot] & 1u) || __any(wide_bf16(av)));
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (j < ncw) acc[j] = first_mfma<T>(a, slot, ct * 4 + j, lane, av, wide);
    // bias + ReLU -> activations (rows = channels 4g.., column = this lane's position)
    if (rvalid) {
      const float* bias = a.bias[slot][0];
      T* out = reinterpret_cast<T*>(a.act[0]) + ((int64_t)ebase + e) * a.act_stride + (int64_t)p * cout;
      float top = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (j >= ncw) continue;
        const int ch = g_channel(cout, ct * 4 + j, 4 * g);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v = fmaxf(acc[j][r] + bias[ch + r], 0.f);
          out[ch + r] = static_cast<T>(v);
          top = fmaxf(top, v);
        }
      }
      if (sizeof(T) == 4 && top >= G_WIDE) mark_wide(a, (int64_t)ebase + e, 0);
    }
  }
}

// Layers after the first: implicit GEMM on tiles of GD::BM output positions (any frames of one slot) x
// BN output channels, the widest of 128, 64, 32 and 16 that divides the slot's Cout (one launch per
// width present, over its slots).  A k-block is 128 bytes of (tap, input channel) values per
// position, 64 bf16 or 32 fp32: its eight 16-byte chunks lie within a tap each (Cin is a multiple of
// 16) and are copied global -> LDS by global_load_lds_dwordx4, chunk c of row r at slot c ^ (r mod 8),
// padding taps from zeros; the packed weight fragments are copied as they are.  Two stages, two
// workgroups per CU (one waits while the other multiplies); each wave holds 64 positions.
// fp32 arithmetic: the weights as three bf16 terms, the activations split on the fly (split3); a k-step's six
// products are summed by themselves and then added, so that the running sum is rounded once a k-step, not
// six times (16x16 frames through 1024-1024: rms error 4.2e-7 with fp32 MFMAs, 5.6e-7 with six
// roundings, 1.9e-7; FP32 logits of 600 128x128 frames 511 -> 527 us).
// Bound by the copies: at 64 bf16 channels a block brings 40 KB for 2.1 MFLOP.  16-32-64 and 32-64-128
// CNNs on 8,192 128x128 frames (12,288 evaluations): layers 2 and 3 take 1.5 ms in bf16 (8-byte
// stores: 1.7); register-staged 128-position tiles, and one wave per 16 positions where Cin is 16, took
// 3.6.  The FP32 band of the same query: 0.66 ms (0.63 with six roundings a k-step; on fp32 MFMAs nearly
// twice that).
template <typename T, int BN> struct GD {
  static constexpr bool F32 = sizeof(T) == 4;
  static constexpr int KB = 128 / (int)sizeof(T), CE = 16 / (int)sizeof(T);   // values per block, per chunk
  static constexpr int NCT = BN / 16;                          // 16-channel MFMA tiles
  static constexpr int WC = BN > 64 || (F32 && BN > 32) ? 2 : 1, WP = 4 / WC;  // waves over channels, positions
  static constexpr int CT = NCT / WC;                          // channel tiles per wave
  static constexpr int BM = WP * 64;
  static constexpr int NU = (F32 ? 3 : 2) * NCT;               // 1 KB weight units: two k-steps, or one of three terms
  static constexpr int NIX = BM * 8 / 256;                     // 16-byte loads per lane and stage: positions
  static constexpr int NIW = (NU + 3) / 4;                     // ... weights
  static constexpr int STAGE = BM * 128 + NU * 1024;
};

static int gconv_tile_bn(int cout) { return cout % 128 == 0 ? 128 : cout % 64 == 0 ? 64 : cout % 32 == 0 ? 32 : 16; }

// slots: bit i set if slot i takes part (every slot's queue counts towards the activations' places).
template <typename T, int BN>
__global__ __launch_bounds__(256, 2) void gconv_dma_kernel(GcnnArgs a, int layer, uint32_t slots) {
  typedef GD<T, BN> G;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * G::STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, l16 = lane & 15;
  const int wp = wave % G::WP, wc = wave / G::WP;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds);
  // this lane's chunk of every row it copies (its rows are equal mod 8)
  const int chunk = (lane & 7) ^ (lane >> 3);
  int total = 0;
  for (int i = 0; i < a.n_preds; ++i) {
    if (!((slots >> i) & 1u)) continue;
    const int hout = a.in_hw[i] >> (layer + 1);
    const int64_t rows = (int64_t)a.q.counts[a.pred[i]] * hout * hout;
    total += (int)((rows + G::BM - 1) / G::BM) * (a.widths[i][layer] / BN);
  }
  for (int t = blockIdx.x; t < total; t += gridDim.x) {
    int slot = 0, off = t, ebase = 0;
    for (int i = 0; i < a.n_preds; ++i) {
      const int q = a.q.counts[a.pred[i]];
      if ((slots >> i) & 1u) {
        const int hout = a.in_hw[i] >> (layer + 1);
        const int c = (int)(((int64_t)q * hout * hout + G::BM - 1) / G::BM) * (a.widths[i][layer] / BN);
        if (off < c) { slot = i; break; }
        off -= c;
      }
      ebase += q;
    }
    const int cnt = a.q.counts[a.pred[slot]];
    const int hin = a.in_hw[slot] >> layer, hout = hin >> 1, P = hout * hout;
    const int cin = a.widths[slot][layer - 1], cout = a.widths[slot][layer];
    const int nct = cout / BN, cb = off % nct;
    const int64_t R0 = (int64_t)(off / nct) * G::BM;
    const int e0 = (int)(R0 / P), r0 = (int)(R0 % P);
    const int KS = g_ksteps(layer, cin), nkb = G::F32 ? KS : (KS + 1) / 2;
    const T* act_in = static_cast<const T*>(a.act[(layer - 1) & 1]);
    // the positions this lane copies a chunk of: address of tap (0, 0), and which taps are padding
    const T* src[G::NIX];
    uint32_t edge = 0;                 // bits 2i, 2i + 1: position i is in output row 0, column 0
#pragma unroll
    for (int i = 0; i < G::NIX; ++i) {
      const int r = r0 + (wave + 4 * i) * 8 + (lane >> 3);
      const int e = e0 + r / P, p = r % P, oi = p / hout, oj = p % hout;
      // rows past the queue re-read its last entry; their results are never stored
      src[i] = act_in + ((int64_t)ebase + min(e, cnt - 1)) * a.act_stride + ((int64_t)(2 * oi - 1) * hin + 2 * oj - 1) * cin;
      edge |= (oi == 0 ? 1u : 0u) << (2 * i) | (oj == 0 ? 2u : 0u) << (2 * i);
    }
    const int dtap = G::KB / cin, dch = G::KB % cin;
    int tap = chunk * G::CE / cin, ch = chunk * G::CE % cin;  // (tap, channel) of this lane's chunk of the next block
    const T* zero = static_cast<const T*>(a.zero_page);
    const int64_t wks = (int64_t)(cout / 16) * 512;         // weight elements per k-step
    const __bf16* wsrc = a.w_bf[slot][layer] + (int64_t)cb * G::NCT * 512 + lane * 8;
    const __bf16* wml = G::F32 ? a.w_ml[slot][layer] + (int64_t)cb * G::NCT * 512 + lane * 8 : nullptr;
    auto issue = [&](int kb, int buf) {
      const uint32_t base = lds0 + buf * G::STAGE;
      const int u = tap / 3, v = tap - 3 * u;
      const uint32_t hit = tap < 9 ? (u == 0 ? 1u : 0u) | (v == 0 ? 2u : 0u) : 0u;
      const int o = (u * hin + v) * cin + ch;
#pragma unroll
      for (int i = 0; i < G::NIX; ++i) {
        const bool pad = tap >= 9 || ((edge >> (2 * i)) & hit) != 0;
        lds_dma16(pad ? zero : src[i] + o, __builtin_amdgcn_readfirstlane(base + (wave + 4 * i) * 1024));
      }
#pragma unroll
      for (int i = 0; i < G::NIW; ++i) {
        // unit: k-step (or term) s, channel tile c
        const int unit = (wave + 4 * i) % G::NU, s = unit / G::NCT, c = unit % G::NCT;
        const __bf16* w = !G::F32 ? wsrc + min(2 * kb + s, KS - 1) * wks
                          : s == 0 ? wsrc + kb * wks : wml + ((s - 1) * KS + kb) * wks;
        lds_dma16(w + c * 512, __builtin_amdgcn_readfirstlane(base + G::BM * 128 + unit * 1024));
      }
      tap += dtap;
      ch += dch;
      if (ch >= cin) {
        ch -= cin;
        ++tap;
      }
    };
    floatx4 acc[G::CT][4];
#pragma unroll
    for (int c = 0; c < G::CT; ++c)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[c][q] = (floatx4){0.f, 0.f, 0.f, 0.f};
    issue(0, 0);
    // fp32: whether the tile's frames or the layer hold values beyond the split (the same for every wave; read
    // behind the first block's copies, which are waited for next anyway)
    bool wide = false;
    if constexpr (G::F32) {
#pragma unroll
      for (int i = 0; i < G::BM / 64; ++i) {
        const int e = min(e0 + (r0 + i * 64 + lane) / P, cnt - 1);
        wide = wide || reinterpret_cast<const uint8_t*>(a.act_wide)[((int64_t)ebase + e) * 4 + layer - 1] != 0;
      }
      wide = __any(wide) || ((a.wide_w[slot] >> layer) & 1u);
    }
    auto k_loop = [&](auto wide_tag) {
      constexpr bool WIDE = decltype(wide_tag)::value;
#pragma unroll 1
      for (int kb = 0; kb < nkb; ++kb) {
        wait_vmcnt<0>();
        __syncthreads();                 // block kb has landed; every wave is done with the other buffer
        if (kb + 1 < nkb) issue(kb + 1, (kb + 1) & 1);
        const unsigned char* X = lds + (kb & 1) * G::STAGE;
        const unsigned char* W = X + G::BM * 128;
        if constexpr (WIDE) {
#pragma unroll 1
          for (int j = 0; j < 8; ++j) {
            float xv[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int r = wp * 64 + q * 16 + l16;
              xv[q] = *reinterpret_cast<const float*>(X + r * 128 + ((2 * g + (j >> 2)) ^ (r & 7)) * 16 + (j & 3) * 4);
            }
#pragma unroll
            for (int c = 0; c < G::CT; ++c) {
              const __bf16* w = reinterpret_cast<const __bf16*>(W + (wc * G::CT + c) * 1024 + lane * 16) + j;
              const float wv = wide_weight(w, w + G::NCT * 512, w + 2 * G::NCT * 512);
#pragma unroll
              for (int q = 0; q < 4; ++q) acc[c][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv, xv[q], acc[c][q], 0, 0, 0);
            }
          }
        } else if constexpr (G::F32) {
          bf16x8 wf[G::CT][3];
#pragma unroll
          for (int c = 0; c < G::CT; ++c)
#pragma unroll
            for (int u = 0; u < 3; ++u)
              wf[c][u] = *reinterpret_cast<const bf16x8*>(W + (u * G::NCT + wc * G::CT + c) * 1024 + lane * 16);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int r = wp * 64 + q * 16 + l16;
            bf16x8 x[3];
            split3(*reinterpret_cast<const float4*>(X + r * 128 + ((2 * g) ^ (r & 7)) * 16),
                   *reinterpret_cast<const float4*>(X + r * 128 + ((2 * g + 1) ^ (r & 7)) * 16), x);
#pragma unroll
            for (int c = 0; c < G::CT; ++c) acc[c][q] += mfma_s3(wf[c], x, (floatx4){0.f, 0.f, 0.f, 0.f});
          }
        } else {
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            if (2 * kb + s >= KS) break;   // an odd number of k-steps: the last block holds one
            bf16x8 xf[4], wf[G::CT];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int r = wp * 64 + q * 16 + l16;
              xf[q] = *reinterpret_cast<const bf16x8*>(X + r * 128 + ((4 * s + g) ^ (r & 7)) * 16);
            }
#pragma unroll
            for (int c = 0; c < G::CT; ++c)
              wf[c] = *reinterpret_cast<const bf16x8*>(W + (s * G::NCT + wc * G::CT + c) * 1024 + lane * 16);
#pragma unroll
            for (int c = 0; c < G::CT; ++c)
#pragma unroll
              for (int q = 0; q < 4; ++q) acc[c][q] = mfma_bf16(wf[c], xf[q], acc[c][q]);
          }
        }
      }
    };
    if (G::F32 && wide) k_loop(std::true_type{});
    else k_loop(std::false_type{});
    // bias + ReLU; lane holds channels g_channel(4g .. 4g + 3) of tile c for position 16q + l16 of its wave
    // (BN 16: channels that do not come in pairs of tiles)
    constexpr int PER = BN > 16 ? 8 : 4;
    const int ch0 = cb * BN + wc * G::CT * 16 + PER * g;
    const float* bias = a.bias[slot][layer] + ch0;
    T* out = static_cast<T*>(a.act[layer & 1]);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = r0 + wp * 64 + q * 16 + l16, e = e0 + r / P, p = r % P;
      if (e >= cnt) continue;
      T* o = out + ((int64_t)ebase + e) * a.act_stride + (int64_t)p * cout + ch0;
      float top = 0.f;
      if constexpr (BN > 16) {
        static_assert(G::CT % 2 == 0, "pairs of tiles");
#pragma unroll
        for (int c = 0; c < G::CT; c += 2)
          top = fmaxf(top, store_relu8(o + c * 16, acc[c][q], acc[c + 1][q], bias + c * 16));
      } else {
        top = store_relu4(o, acc[0][q], *reinterpret_cast<const float4*>(bias));
      }
      if (G::F32 && top >= G_WIDE) mark_wide(a, (int64_t)ebase + e, layer);
    }
    __syncthreads();   // the next tile's first block overwrites buffer 0
  }
}

// First layer (Cin = 3, K = 27) of frames of 32, 64, 128 or 256 pixels a side and at most 64 channels:
// a tile is GF_P output positions, whole output rows of one frame.  The input rows it reads are
// staged in LDS as bf16 (exact for bf16 and uint8 values) by 16-byte loads, pixel 0 of a row at element
// GF_X0 with the border pixel before it, rows above the frame holding the pad value.  A position's nine
// values of one row start at an odd element: five aligned words hold them, and a lane's eight K
// slots (g_first_k) are four funnel shifts of one row's words.  HBM-bound: 12,288 evaluations of
// 128x128 uint8 frames into 16 or 32 channels read and write 2.7 GB in 0.64 ms: the rows of the next tile
// are requested while this one is computed, weights and biases stay in LDS (both loaded where they were
// used, and 8-byte stores: 0.87 ms; one load and one fp32 LDS word per value, eight LDS reads per
// fragment: 3.26 ms).
constexpr int GF_P = 512, GF_X0 = 8;
__host__ __device__ inline bool gconv_first_ok(int hout, int cout) {
  return hout >= 16 && 128 % hout == 0 && cout % 16 == 0 && cout <= 64;
}
__host__ __device__ inline int gf_rows(int hout) { return hout * hout < GF_P ? hout : GF_P / hout; }   // output rows per tile
__host__ __device__ inline int gf_stride(int hin) { return GF_X0 + 3 * hin + 8; }                     // elements per staged row

// 16 bytes at any address (frames may start anywhere)
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));

template <typename T>
__global__ __launch_bounds__(256) void gconv_first_kernel(GcnnArgs a) {
  constexpr int MAXE = 9 * (GF_X0 + 3 * 256 + 8);        // the largest of the four sizes (256-pixel frames)
  static_assert(MAXE >= 17 * (GF_X0 + 3 * 128 + 8) && MAXE >= 33 * (GF_X0 + 3 * 64 + 8) && MAXE >= 33 * (GF_X0 + 3 * 32 + 8),
                "staged rows");
  __shared__ __attribute__((aligned(16))) uint16_t xin[MAXE];
  constexpr int TERMS = sizeof(T) == 4 ? 3 : 1;
  __shared__ __attribute__((aligned(16))) __bf16 w_s[TERMS * 4 * 512];   // the predicate's weights [term][tile]
  __shared__ __attribute__((aligned(16))) float bias_s[64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, l16 = lane & 15;
  const uint16_t pad = a.fr.dtype == HYDRO_DTYPE_BF16 ? 0x3F00 : 0x42FF;     // 0.5, 127.5 in bf16
  const bool u8 = a.fr.dtype != HYDRO_DTYPE_BF16;
  int total = 0;
  for (int i = 0; i < a.n_preds; ++i) {
    const int hout = a.in_hw[i] >> 1;
    total += a.q.counts[a.pred[i]] * (hout / gf_rows(hout));
  }
  struct Tile { int slot, e, ebase, oi0, lg; };        // lg: log2 of the frame side (a power of two)
  auto decode = [&](int t) {
    Tile r{};
    int off = t;
    for (int i = 0; i < a.n_preds; ++i) {
      const int hout = a.in_hw[i] >> 1, n = a.q.counts[a.pred[i]];
      const int c = n * (hout / gf_rows(hout));
      if (off < c) { r.slot = i; break; }
      off -= c;
      r.ebase += n;
    }
    const int hout = a.in_hw[r.slot] >> 1, ro = gf_rows(hout), tpf = hout / ro;
    r.e = off / tpf;
    r.oi0 = (off - r.e * tpf) * ro;
    r.lg = 31 - __builtin_clz(a.in_hw[r.slot]);
    return r;
  };
  auto entry = [&](const Tile& r) { return a.q.entries[(int64_t)a.pred[r.slot] * a.q.cap + r.e]; };
  // Staged row r of a tile is input row y = 2 oi0 - 1 + r (y < 0 only for r = 0 of a frame's first tile), as
  // 16-byte chunks: at most 864 of bf16 values, 432 of bytes.  A tile's chunks are requested while the
  // previous tile is computed, its queue entry a tile earlier.
  u32x4 v[4];
  auto request = [&](const Tile& r, uint32_t e) {
    const int hin = 1 << r.lg, lc = u8 ? r.lg - 4 : r.lg - 3, cpr = 3 << lc;
    const int n = (2 * gf_rows(hin >> 1) + 1) * cpr, first = r.oi0 == 0 ? cpr : 0;
    const unsigned char* src = static_cast<const unsigned char*>(a.fr.base) +
                               ((int64_t)entry_idx(e) * a.fr.elems + (int64_t)(2 * r.oi0 - 1) * hin * 3) * (u8 ? 1 : 2);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i >= 2 && u8) break;
      const int q = min(max(tid + 256 * i, first), n - 1);      // (chunks of no use are read again)
      v[i] = *reinterpret_cast<const u32x4_any*>(src + (int64_t)q * 16);
    }
  };
  auto stage = [&](const Tile& r) {
    const int hin = 1 << r.lg, lc = u8 ? r.lg - 4 : r.lg - 3, cpr = 3 << lc, RS = gf_stride(hin);
    const int rows = 2 * gf_rows(hin >> 1) + 1;
    const uint32_t padw = pad | (uint32_t)pad << 16;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int q = tid + 256 * i, y = (q >> lc) / 3, c = q - y * cpr;
      if ((i >= 2 && u8) || q >= rows * cpr) break;
      const bool in = y > 0 || r.oi0 > 0;
      if (u8) {
        u32x4 lo, hi;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          // bf16 of a byte: the upper half of its float
          const uint32_t b = v[i][w];
          const uint32_t f0 = __float_as_uint((float)(b & 255u)), f1 = __float_as_uint((float)(b >> 8 & 255u));
          const uint32_t f2 = __float_as_uint((float)(b >> 16 & 255u)), f3 = __float_as_uint((float)(b >> 24));
          const uint32_t p0 = in ? f0 >> 16 | (f1 & 0xFFFF0000u) : padw, p1 = in ? f2 >> 16 | (f3 & 0xFFFF0000u) : padw;
          if (w < 2) { lo[2 * w] = p0; lo[2 * w + 1] = p1; }
          else { hi[2 * w - 4] = p0; hi[2 * w - 3] = p1; }
        }
        u32x4* dst = reinterpret_cast<u32x4*>(xin + y * RS + GF_X0 + c * 16);
        dst[0] = lo;
        dst[1] = hi;
      } else {
        u32x4 x = v[i];
        if (!in) x = (u32x4){padw, padw, padw, padw};
        *reinterpret_cast<u32x4*>(xin + y * RS + GF_X0 + c * 8) = x;
      }
    }
    if (tid < rows)
#pragma unroll
      for (int c = 1; c <= 3; ++c) xin[tid * RS + GF_X0 - c] = pad;
  };
  int t = blockIdx.x, loaded = -1;
  if (t >= total) return;
  const int last = total - 1;
  Tile cur = decode(t), nx = decode(min(t + (int)gridDim.x, last));
  request(cur, entry(cur));
  uint32_t e_nx = entry(nx);
  for (; t < total; t += gridDim.x) {
    const int slot = cur.slot, cout = a.widths[slot][0], nct = cout / 16;
    if (slot != loaded) {
      for (int q = tid; q < TERMS * nct * 64; q += 256) {
        const int term = q / (nct * 64), o = q - term * nct * 64;
        const __bf16* src = term == 0 ? a.w_bf[slot][0] : a.w_ml[slot][0] + (int64_t)(term - 1) * nct * 512;
        reinterpret_cast<u32x4*>(w_s)[term * 256 + o] = reinterpret_cast<const u32x4*>(src)[o];
      }
      if (tid < cout) bias_s[tid] = a.bias[slot][0][tid];
      loaded = slot;
    }
    stage(cur);
    __syncthreads();
    const Tile at = cur;
    if (t + (int)gridDim.x < total) {
      cur = nx;
      request(cur, e_nx);
      nx = decode(min(t + 2 * (int)gridDim.x, last));
      e_nx = entry(nx);
    }
    const int hout = 1 << (at.lg - 1), RS = gf_stride(2 << (at.lg - 1));
    T* o0 = reinterpret_cast<T*>(a.act[0]) + ((int64_t)at.ebase + at.e) * a.act_stride + (int64_t)at.oi0 * hout * cout;
    const int np = gf_rows(hout) * hout;            // a multiple of 64
    bool wide = false;
    auto tile_mfma = [&](int c, bf16x8 x) {
      const __bf16* w = w_s + (c * 64 + lane) * 8;
      if constexpr (TERMS == 3) return mfma_first(w, w + 2048, w + 4096, x, wide);
      return mfma_bf16(*reinterpret_cast<const bf16x8*>(w), x, (floatx4){0.f, 0.f, 0.f, 0.f});
    };
    float top = 0.f;
    for (int pt = wave * 32; pt < np; pt += 128) {
      const uint16_t* base[2];                      // element before the position's first value
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int pl = pt + q * 16 + l16;
        base[q] = xin + 2 * (pl >> (at.lg - 1)) * RS + GF_X0 - 4 + 6 * (pl & (hout - 1));
      }
      bf16x8 xf[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        uint32_t d[5];
#pragma unroll
        for (int w = 0; w < 5; ++w)
          d[w] = *reinterpret_cast<const uint32_t*>(base[q] + (g < 3 ? g * RS + 2 * w : min(w, 2) * RS + 8));
        u32x4 f;
#pragma unroll
        for (int w = 0; w < 4; ++w) f[w] = __builtin_amdgcn_alignbit(d[w + 1], d[w], 16);
        if (g == 3) f = (u32x4){(d[0] >> 16) | (d[1] & 0xFFFF0000u), d[2] >> 16, 0u, 0u};
        xf[q] = *reinterpret_cast<const bf16x8*>(&f);
      }
      if constexpr (TERMS == 3) wide = (a.wide_w[slot] & 1u) || (!u8 && __any(wide_bf16(xf[0]) || wide_bf16(xf[1])));
      T* o = o0 + (int64_t)(pt + l16) * cout;
      if (cout % 32 == 0) {
#pragma unroll
        for (int c = 0; c < 4; c += 2) {
          if (c >= nct) break;
#pragma unroll
          for (int q = 0; q < 2; ++q)
            top = fmaxf(top, store_relu8(o + q * 16 * cout + c * 16 + 8 * g, tile_mfma(c, xf[q]), tile_mfma(c + 1, xf[q]),
                                         bias_s + c * 16 + 8 * g));
        }
      } else {
        // an odd number of tiles: the lane groups of the two position tiles trade places, so that each lane
        // holds eight channels of one position
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          if (c >= nct) break;
          const float4 b = *reinterpret_cast<const float4*>(bias_s + c * 16 + 4 * g);
          if constexpr (sizeof(T) == 2) {
            alignas(8) T h[2][4];
#pragma unroll
            for (int q = 0; q < 2; ++q) store_relu4(h[q], tile_mfma(c, xf[q]), b);
            const uint2 v0 = *reinterpret_cast<const uint2*>(h[0]), v1 = *reinterpret_cast<const uint2*>(h[1]);
            const auto lo = __builtin_amdgcn_permlane16_swap(v0.x, v1.x, false, false);
            const auto hi = __builtin_amdgcn_permlane16_swap(v0.y, v1.y, false, false);
            *reinterpret_cast<uint4*>(o + (g & 1) * 16 * cout + c * 16 + (g >> 1) * 8) =
                make_uint4(lo[0], hi[0], lo[1], hi[1]);
          } else {
#pragma unroll
            for (int q = 0; q < 2; ++q)
              top = fmaxf(top, store_relu4(o + q * 16 * cout + c * 16 + 4 * g, tile_mfma(c, xf[q]), b));
          }
        }
      }
    }
    if (TERMS == 3 && top >= G_WIDE) mark_wide(a, (int64_t)at.ebase + at.e, 0);
    __syncthreads();   // the next tile restages xin
  }
}

// Pool + FC + margin + decision: one wave per frame, 16-byte loads (12,288 frames of 16x16x64 or
// 16x16x128 bf16: 290 us; one channel per lane and load: 489); a workgroup's decisions forwarded
// together: 160 us.
template <typename T>
__global__ __launch_bounds__(256) void gcnn_head_kernel(GcnnArgs a, Forward f) {
  int total = 0;
  for (int i = 0; i < a.n_preds; ++i) total += a.q.counts[a.pred[i]];
  __shared__ DecisionBuf dec;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // a wave's frames between two flushes: what one pass over the grid leaves it, at most a buffer's share
  const int fpw = min(DBUF / 4, max(1, (total + (int)gridDim.x * 4 - 1) / ((int)gridDim.x * 4)));
  for (int base = blockIdx.x * 4 * fpw; base < total; base += gridDim.x * 4 * fpw) {
    for (int it = 0; it < fpw; ++it) {
      const int t = base + it * 4 + wave;
      const bool active = t < total;
      int slot = 0, off = t;
      for (int i = 0; i < a.n_preds; ++i) {
        const int c = a.q.counts[a.pred[i]];
        if (off < c) { slot = i; break; }
        off -= c;
      }
      if (!active) { slot = 0; off = 0; }
      const int k = a.pred[slot];
      const uint32_t e = active ? a.q.entries[(int64_t)k * a.q.cap + off] : 0u;
      const int L = a.n_layers[slot];
      const int hl = a.in_hw[slot] >> L, P = hl * hl;
      const int cl = a.widths[slot][L - 1];
      float zp[kClasses];
#pragma unroll
      for (int c = 0; c < kClasses; ++c) zp[c] = 0.f;
      int64_t act_frame = off;
      if (active) {
        for (int i = 0; i < slot; ++i) act_frame += a.q.counts[a.pred[i]];
        const T* act = reinterpret_cast<const T*>(a.act[(L - 1) & 1]) + act_frame * a.act_stride;
        const float* fw = a.fc_w[slot];
        constexpr int VE = 16 / (int)sizeof(T);      // channels per 16-byte load
        const int vpp = cl / VE;                     // loads per position
        if (vpp <= 64 && 64 % vpp == 0) {
          // a lane keeps the same VE channels and takes every (64 / vpp)-th position; the lanes of one
          // channel group add up across the wave
          float s[VE];
#pragma unroll
          for (int u = 0; u < VE; ++u) s[u] = 0.f;
          const uint4* av = reinterpret_cast<const uint4*>(act);
#pragma unroll 8
          for (int q = lane; q < P * vpp; q += 64) {
            const uint4 v = av[q];
            const T* tv = reinterpret_cast<const T*>(&v);
#pragma unroll
            for (int u = 0; u < VE; ++u) s[u] += (float)tv[u];
          }
          for (int o = vpp; o < 64; o <<= 1)
#pragma unroll
            for (int u = 0; u < VE; ++u) s[u] += __shfl_xor(s[u], o);
          // every lane holds its group's sums: the group's lanes share its channels in the FC
          const int copies = 64 / vpp, cpy = lane / vpp;
          for (int u0 = 0; u0 < VE; u0 += copies) {
            const int u = u0 + cpy;
            float sv = 0.f;
#pragma unroll
            for (int w = 0; w < VE; ++w) sv = w == u ? s[w] : sv;
            if (u < VE) {
              const float* fr = fw + ((lane % vpp) * VE + u) * kClasses;
#pragma unroll
              for (int c = 0; c < kClasses; ++c) zp[c] += sv / (float)P * fr[c];
            }
          }
        } else {
          for (int ch = lane; ch < cl; ch += 64) {
            float s = 0.f;
#pragma unroll 8
            for (int p = 0; p < P; ++p) s += (float)act[(int64_t)p * cl + ch];
            const float gch = s / (float)P;
#pragma unroll
            for (int c = 0; c < kClasses; ++c) zp[c] += gch * fw[ch * kClasses + c];
          }
        }
      }
      wave_sum_n(zp);
      bool pass = false, defer = false;
      if (active) {
        float z[kClasses];
        for (int c = 0; c < kClasses; ++c) z[c] = zp[c] + a.fc_b[slot][c];
        const uint32_t idx = entry_idx(e);
        if (f.logits != nullptr && lane == 0)
          for (int c = 0; c < kClasses; ++c) f.logits[(int64_t)idx * kClasses + c] = (double)z[c];
        const float d = class_margin(z, a.class_mask[slot]);
        const float th = theta_of(f, k, idx);
        pass = d > th;
        defer = f.defer.entries != nullptr && fabsf(d - th) < f.tau[k];
      }
      if (active && lane == 0) {
        decision_set(dec, it * 4 + wave, k, e, defer, pass);
        if (sizeof(T) == 4) a.act_wide[act_frame] = 0u;         // for the next launch
      }
    }
    if (f.logits == nullptr) {
      if (threadIdx.x == 0) dec.n = min(4 * fpw, total - base);
      decision_flush(f, dec, a.n_preds, a.pred);
    }
  }
}

void launch_gcnn_layerwise(const GcnnArgs& a, const Forward& f, int tier, int grid, hipStream_t s);

// ---------------------------------------------------------------- host side
size_t gcnn_packed_elems(int layer, int cin, int cout) { return (size_t)g_ksteps(layer, cin) * (cout / 16) * 512; }

// [kstep][channel tile of 16][64 lanes][8]; lane l: row l % 16 of the tile (g_channel), k = 32 kstep + 8 (l/16) + e.
// Weights are read eight channels of a tap at a time, 16 rows beside each other (element by element, with the
// indices divided out of each place, a 1,024-channel layer took twice as long).
void gcnn_pack_layer(int layer, int cin, int cout, const float* w, float scale, float* out) {
  std::fill(out, out + gcnn_packed_elems(layer, cin, cout), 0.f);
  const int nct = cout / 16;
  for (int ct = 0; ct < nct; ++ct) {
    const float* rows[16];                                     // [ic][tap]
    for (int r = 0; r < 16; ++r) rows[r] = w + (size_t)g_channel(cout, ct, r) * cin * 9;
    float* dst = out + (size_t)ct * 512;
    if (layer == 0) {
      for (int k = 0; k < 32; ++k) {
        int u, v;
        if (!g_first_k(k, &u, &v)) continue;
        for (int r = 0; r < 16; ++r) dst[((k >> 3) * 16 + r) * 8 + (k & 7)] = scale * rows[r][v % 3 * 9 + u * 3 + v / 3];
      }
      continue;
    }
    for (int tap = 0, k = 0; tap < 9; ++tap)
      for (int ic = 0; ic < cin; ic += 8, k += 8) {
        float* d = dst + (size_t)(k >> 5) * nct * 512 + (k >> 3 & 3) * 128;
        for (int r = 0; r < 16; ++r, d += 8)
          for (int e = 0; e < 8; ++e) d[e] = scale * rows[r][(ic + e) * 9 + tap];
      }
  }
}

// Slot i of src becomes slot j of dst.
void gcnn_copy_slot(GcnnArgs& dst, int j, const GcnnArgs& src, int i) {
  dst.pred[j] = src.pred[i]; dst.n_layers[j] = src.n_layers[i]; dst.in_hw[j] = src.in_hw[i];
  dst.class_mask[j] = src.class_mask[i]; dst.fc_w[j] = src.fc_w[i]; dst.fc_b[j] = src.fc_b[i];
  dst.esc_act[j] = src.esc_act[i]; dst.c4[j] = src.c4[i];
  dst.c4_w1b[j] = src.c4_w1b[i]; dst.c4_w1f[j] = src.c4_w1f[i]; dst.wide_w[j] = src.wide_w[i];
  for (int l = 0; l < HYDRO_MAX_LAYERS; ++l) {
    dst.widths[j][l] = src.widths[i][l]; dst.w_bf[j][l] = src.w_bf[i][l]; dst.w_ml[j][l] = src.w_ml[i][l];
    dst.bias[j][l] = src.bias[i][l]; dst.wt_canon[j][l] = src.wt_canon[i][l]; dst.b_canon[j][l] = src.b_canon[i][l];
  }
  // (array extents, so that a new entry is never left behind)
  for (size_t p = 0; p < sizeof(src.c4_w2[0]) / sizeof(src.c4_w2[0][0]); ++p) dst.c4_w2[j][p] = src.c4_w2[i][p];
  for (size_t p = 0; p < sizeof(src.c4_wscale[0]) / sizeof(src.c4_wscale[0][0]); ++p) dst.c4_wscale[j][p] = src.c4_wscale[i][p];
  for (size_t p = 0; p < sizeof(src.c4_ascale[0]) / sizeof(src.c4_ascale[0][0]); ++p) dst.c4_ascale[j][p] = src.c4_ascale[i][p];
  for (int l = 0; l < 2; ++l)
    for (size_t p = 0; p < sizeof(src.c4_img[0][0]) / sizeof(src.c4_img[0][0][0]); ++p) dst.c4_img[j][l][p] = src.c4_img[i][l][p];
}

void launch_gcnn_pass(const GcnnArgs& a0, const Forward& f, int tier, int grid, hipStream_t s) {
  if (a0.n_preds == 0) return;
  if (tier != TIER_F64) {
    // slots of the 4-layer 128x128 shape take the dedicated kernels; the rest the layer-wise ones
    GcnnArgs c4a = a0, gen = a0;
    c4a.n_preds = gen.n_preds = 0;
    for (int i = 0; i < a0.n_preds; ++i) {
      if (a0.c4[i]) gcnn_copy_slot(c4a, c4a.n_preds++, a0, i);
      else gcnn_copy_slot(gen, gen.n_preds++, a0, i);
    }
    if (c4a.n_preds > 0) {
      const int p = tier == TIER_MID ? (a0.prec == HYDRO_PREC_FP8 ? C4_BF16 : C4_X3)
                    : tier != TIER_FIRST ? C4_F32
                    : a0.prec == HYDRO_PREC_FP8 ? C4_FP8 : a0.prec == HYDRO_PREC_BF16 ? C4_BF16 : C4_F32;
      launch_c4_pass(c4a, f, p, grid, s);
    }
    if (gen.n_preds == 0) return;
    launch_gcnn_layerwise(gen, f, tier, grid, s);
    return;
  }
  launch_gcnn_layerwise(a0, f, tier, grid, s);
}

template <int BN>
static void launch_gconv(bool bf, const GcnnArgs& a, int l, uint32_t slots, int grid, hipStream_t s) {
  if (bf) hipLaunchKernelGGL((gconv_dma_kernel<__bf16, BN>), dim3(grid * 8), dim3(256), 0, s, a, l, slots);
  else hipLaunchKernelGGL((gconv_dma_kernel<float, BN>), dim3(grid * 8), dim3(256), 0, s, a, l, slots);
}

void launch_gcnn_layerwise(const GcnnArgs& a, const Forward& f, int tier, int grid, hipStream_t s) {
  int maxl = 0;
  for (int i = 0; i < a.n_preds; ++i) maxl = a.n_layers[i] > maxl ? a.n_layers[i] : maxl;
  if (tier == TIER_F64) {
    F64Args b{};
    b.n_preds = a.n_preds;
    for (int i = 0; i < a.n_preds; ++i) {
      b.pred[i] = a.pred[i]; b.class_mask[i] = a.class_mask[i]; b.n_layers[i] = a.n_layers[i]; b.in_hw[i] = a.in_hw[i];
      for (int l = 0; l < a.n_layers[i]; ++l) {
        b.widths[i][l] = a.widths[i][l];
        b.wt[i][l] = a.wt_canon[i][l]; b.bias[i][l] = a.b_canon[i][l];
      }
      b.fc_w[i] = a.fc_w[i]; b.fc_b[i] = a.fc_b[i]; b.esc_act[i] = a.esc_act[i];
    }
    b.esc_stride = a.esc_stride; b.esc_off = a.esc_half; b.esc_cap = a.esc_cap;
    b.scratch = a.rest_scratch; b.per_block = a.rest_per_block; b.scratch_off = a.rest_per_block / 2;
    b.rest_grid = a.rest_grid; b.q = a.q; b.fr = a.fr;
    launch_f64_cnn(b, f, grid, s);
    return;
  }
  const bool bf = a.prec == HYDRO_PREC_BF16 && tier == TIER_FIRST;
  for (int l = 0; l < maxl; ++l) {
    if (l == 0) {
      bool first_ok = true;
      for (int i = 0; i < a.n_preds; ++i) first_ok = first_ok && gconv_first_ok(a.in_hw[i] >> 1, a.widths[i][0]);
      if (first_ok) {                  // (as many workgroups as the registers let in: their tiles are a stream)
        if (bf) hipLaunchKernelGGL(gconv_first_kernel<__bf16>, dim3(grid * 5), dim3(256), 0, s, a);
        else hipLaunchKernelGGL(gconv_first_kernel<float>, dim3(grid * 4), dim3(256), 0, s, a);
      } else {
        if (bf) hipLaunchKernelGGL(gconv_first_any_kernel<__bf16>, dim3(grid * 4), dim3(256), 0, s, a);
        else hipLaunchKernelGGL(gconv_first_any_kernel<float>, dim3(grid * 4), dim3(256), 0, s, a);
      }
      continue;
    }
    for (int bn = 128; bn >= 16; bn >>= 1) {
      uint32_t slots = 0;
      for (int i = 0; i < a.n_preds; ++i)
        if (l < a.n_layers[i] && gconv_tile_bn(a.widths[i][l]) == bn) slots |= 1u << i;
      if (!slots) continue;
      if (bn == 128) launch_gconv<128>(bf, a, l, slots, grid, s);
      else if (bn == 64) launch_gconv<64>(bf, a, l, slots, grid, s);
      else if (bn == 32) launch_gconv<32>(bf, a, l, slots, grid, s);
      else launch_gconv<16>(bf, a, l, slots, grid, s);
    }
  }
  if (bf) hipLaunchKernelGGL(gcnn_head_kernel<__bf16>, dim3(grid * 4), dim3(256), 0, s, a, f);
  else hipLaunchKernelGGL(gcnn_head_kernel<float>, dim3(grid * 4), dim3(256), 0, s, a, f);
}

}  // namespace hydro
