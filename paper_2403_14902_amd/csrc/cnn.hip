// CNN predicates on gfx950: one fused kernel evaluates conv3x3/s2 x3 + ReLU, global average
// pooling, FC and the class-subset decision for a frame entirely in LDS and registers.
//
// Model (synthetic UDF): 64x64x3 frame -> conv(16m) -> conv(32m) -> conv(64m) -> mean over 8x8 ->
// FC 10, m in {1, 2, 4}; every conv has stride 2, zero padding 1 (in normalised space), ReLU.
//
// Per frame, one workgroup (8 wave64s for the widest class; 4 for the two narrower ones in the
// bf16 first pass, two workgroups per CU with the LDS of their own width, so that one frame's barriers
// and per-frame work overlap another frame's MFMAs):
//   FR   the raw frame in LDS as bf16 (exact for bf16 and uint8 inputs): rows of 64 pixels x 3
//        channels (row stride 200 elements), with a one-pixel top/left border holding the raw
//        value that normalises to zero.
//        Layer 1 uses the folded form sW * raw + (b - 2 sum W), so no normalisation pass runs.
//   S1   one 16-channel slab of layer-1 output (all 32x32 positions);
//   ACC2 layer-2 accumulators for all 16x16 positions and all 32m channels stay in registers while
//        the m slabs of layer 1 stream through S1 (layer 2's K loop runs slab by slab), so
//        layer 1's full output never needs to fit in LDS and every layer-2 weight is read once
//        per frame;
//   L2   layer-2 output (bias + ReLU) written over FR/S1 once all slabs are consumed;
//   ACC3 layer-3 accumulators (64 positions x 64m channels) in registers; their ReLU is summed
//        straight into the pooled vector, then FC, margin and decision.
// Convolutions are implicit GEMMs on MFMA: M = output positions, N = output channels,
// K = (tap, input channel).  Weights are pre-packed in MFMA-fragment order so each lane reads
// one contiguous run per fragment.
#include "engine.h"

namespace hydro {

// k-steps of the 16x16x32 MFMA (the FP32 tier's too: bf16 terms), operands per lane
constexpr int KSTEP = 32, KPL = 8;

// geometry
constexpr int H0 = 64, H1 = 32, H2 = 16, H3 = 8;
constexpr int NTHR = 512;           // 8 wave64s per workgroup (the narrowest class: 4, two per CU)
constexpr int FRS = 200;            // FR row stride (bf16 elements): 5 unused, border pixel, 64 pixels
constexpr int FR_X0 = 8;            // element offset of pixel 0 in an FR row (16-byte aligned)
constexpr int S1_W = H1 + 1;        // layer-1 slab row stride in pixels (top/left border)
constexpr int L2_W = H2 + 1;
constexpr int CB1 = 16;             // layer-1 channels per slab

// A 16-byte LDS read of a wave takes lanes 0 .. 7 and 16 .. 23 together (8 .. 15 and 24 .. 31, and so on):
// eight pixels two columns apart, two neighbouring 16-byte units of each, which must be sixteen
// different units of LDS's 256 bytes.  So a row holds its even columns before its odd ones, and a pixel
// pitch is twice an odd number of units; the odd columns start a unit later, so that the 8-byte stores
// of consecutive columns differ too.  (With columns in order at padded pitches every read took two passes.
// Cycles lost to bank conflicts, share of a CU's: bf16 width 128 0.305 -> 0.15, width 64 0.287 -> 0.19; 16,384 frames:
// 1494 -> 1450, 541 -> 510 and, width 32, 256 -> 246 us; FP32, three terms: 0.126 -> 0.117, width 32 808 -> 755 us.)
template <typename T> struct Pad {
  // bytes of a layer-1 slab pixel (fp32: three bf16 planes of 16 channels), and of a row
  static constexpr int S1PB = CB1 * (sizeof(T) == 4 ? 6 : 2), S1RB = S1_W * S1PB + 16;
  static_assert(S1PB / 16 % 4 == 2, "pitch");
  // byte b of pixel (y, x), borders included
  __host__ __device__ static constexpr int at(int y, int x, int b) {
    return y * S1RB + (x & 1) * ((S1_W + 1) / 2 * S1PB + 16) + (x >> 1) * S1PB + b;
  }
};
// Layer-2 pixel of width class m: bf16, or for the FP32 tier three bf16 planes (the widest class: fp32, its
// planes do not fit LDS, nor does a pitch that suits its 32-byte reads)
template <typename T, int M> struct PadL2 {
  static constexpr bool PLANES = sizeof(T) == 4 && M < 4;
  static constexpr int D = 32 * M * (PLANES ? 6 : (int)sizeof(T));
  static constexpr int PB = D + (sizeof(T) == 4 && !PLANES ? 16 : 32), RB = L2_W * PB + 16;
  static_assert((sizeof(T) == 4 && !PLANES) || PB / 16 % 4 == 2, "pitch");
  __host__ __device__ static constexpr int at(int y, int x, int b) {
    return y * RB + (x & 1) * ((L2_W + 1) / 2 * PB + 16) + (x >> 1) * PB + b;
  }
};

template <typename T, int MMAX = 4> struct CnnLds {
  static constexpr int FR_BYTES = (H0 + 1) * FRS * 2;
  static constexpr int S1_OFF = (FR_BYTES + 15) / 16 * 16;
  static constexpr int S1_BYTES = S1_W * Pad<T>::S1RB;
  static constexpr int L2_BYTES_MAX = L2_W * PadL2<T, MMAX>::RB;
  static constexpr int REGION = (S1_OFF + S1_BYTES) > L2_BYTES_MAX ? (S1_OFF + S1_BYTES) : L2_BYTES_MAX;
};

// packed-layer geometry: [slab][kstep][ntile][64][KPL]
// layer 1: K = 27 and the bias in conv1_k's slots
__host__ __device__ constexpr int cnn_ksteps(int layer, int m) {
  return layer == 0 ? 1 : layer == 1 ? (9 * CB1 + KSTEP - 1) / KSTEP : 9 * 32 * m / KSTEP;
}
__host__ __device__ constexpr int cnn_slabs(int layer, int m) { return layer == 2 ? 1 : m; }
__host__ __device__ constexpr int cnn_ntiles(int layer, int m) { return layer == 0 ? 1 : layer == 1 ? 2 * m : 4 * m; }

// Per-slot constants staged in LDS when a workgroup's slot changes: biases of layers 2 and 3
// (layer 1's is among its weights) and, in the bf16 kernels, the FC weights and bias.
constexpr int CB_L2 = 0, CB_L3 = 128, CB_N = 384;
constexpr int FCW_MAX = 256 * kClasses;

struct CnnShared {
  float cb[CB_N];
  float fcb[kClasses];
  float gpart[2][256];
  float z[kClasses];
  DecisionBuf dec;
  unsigned long long ticks[kMaxK];
  __attribute__((aligned(16))) __bf16 feat[192];   // router features of the current frame
};

// Raw frame bytes held in registers between the issue of their loads and their LDS store
// (the next frame is fetched while the current one is in layer 3).
template <int NT>
struct FramePrefetch {
  uint4 v[1536 / NT];
};

// bf16 frames: 1536 chunks of 8 elements; uint8 frames: 768 chunks of 16 elements.  One
// unconditional load sequence serves both (uint8 chunk indices past the frame are clamped to its
// last chunk and the values ignored), so the loads are never skipped and no register is the
// target of two alternative loads: the compiler can count outstanding loads exactly.
template <int NT>
__device__ inline void frame_issue(const CnnArgs& a, uint32_t idx, FramePrefetch<NT>& pf) {
  const int tid = threadIdx.x;
  const bool bf = a.fr.dtype == HYDRO_DTYPE_BF16;
  const int last = bf ? 1535 : 767;
  const uint4* src = reinterpret_cast<const uint4*>(static_cast<const unsigned char*>(a.fr.base) +
                                                    (int64_t)idx * a.fr.elems * (bf ? 2 : 1));
#pragma unroll
  for (int r = 0; r < 1536 / NT; ++r) pf.v[r] = src[min(tid + r * NT, last)];
}

// The loaded registers pass through an empty asm statement at the point of use, so no
// computation on them (the uint8 unpacking, which the compiler otherwise evaluates speculatively
// for every frame type) can be scheduled next to the loads: the wave does not wait for the frame
// until it stores it.
__device__ inline uint4 frame_regs_ready(uint4 v) {
  asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
  return v;
}

// Store a prefetched frame into FR and (re)write the borders of FR and the layer-1 slab.
template <typename T, int NT>
__device__ inline void frame_store(const CnnArgs& a, const FramePrefetch<NT>& pf, unsigned char* region) {
  const int tid = threadIdx.x;
  __bf16* FR = reinterpret_cast<__bf16*>(region);
  if (a.fr.dtype == HYDRO_DTYPE_BF16) {
#pragma unroll
    for (int r = 0; r < 1536 / NT; ++r) {
      const int q = tid + r * NT, y = q / 24, c = q % 24;
      *reinterpret_cast<uint4*>(FR + (y + 1) * FRS + FR_X0 + c * 8) = frame_regs_ready(pf.v[r]);
    }
  } else {
#pragma unroll
    for (int r = 0; r < (768 + NT - 1) / NT; ++r) {
      const int q = tid + r * NT;
      if (q < 768) {
        const int y = q / 12, c = q % 12;
        const uint4 raw = frame_regs_ready(pf.v[r]);
        const uint8_t* b = reinterpret_cast<const uint8_t*>(&raw);
        alignas(16) __bf16 o[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) o[j] = static_cast<__bf16>((float)b[j]);
        uint4* d = reinterpret_cast<uint4*>(FR + (y + 1) * FRS + FR_X0 + c * 16);
        d[0] = reinterpret_cast<const uint4*>(o)[0];
        d[1] = reinterpret_cast<const uint4*>(o)[1];
      }
    }
  }
  const __bf16 padv = static_cast<__bf16>(a.pad_raw);
  for (int e = tid; e < FRS; e += NT) FR[e] = padv;                                // top border row
  for (int e = tid; e < H0 * 3; e += NT) FR[(e / 3 + 1) * FRS + FR_X0 - 3 + e % 3] = padv;  // left border
  constexpr int WP = Pad<T>::S1PB / 4;            // words per pixel
  for (int p = tid; p < (2 * S1_W - 1) * WP; p += NT) {
    const int q = p / WP, c = p % WP;
    const int y = q < S1_W ? 0 : q - S1_W + 1, x = q < S1_W ? q : 0;
    *reinterpret_cast<uint32_t*>(region + CnnLds<T>::S1_OFF + Pad<T>::at(y, x, 4 * c)) = 0u;
  }
}

// 4 consecutive channels of one position, stored with one LDS write.
template <typename T>
__device__ inline void store4(T* dst, float v0, float v1, float v2, float v3) {
  if constexpr (sizeof(T) == 2) {
    alignas(8) __bf16 h[4] = {static_cast<__bf16>(v0), static_cast<__bf16>(v1), static_cast<__bf16>(v2),
                              static_cast<__bf16>(v3)};
    *reinterpret_cast<uint2*>(dst) = *reinterpret_cast<const uint2*>(h);
  } else {
    *reinterpret_cast<float4*>(dst) = make_float4(v0, v1, v2, v3);
  }
}

// One frame through the network (FR already holds it).  The MFMAs compute the transposed
// products (rows = output channels from the packed weights, columns = positions from LDS), so
// each lane ends with 4 consecutive channels of one position.  Wave 0 finishes with FC, margin
// and the decision record; if next_valid, the next frame is stored into FR meanwhile.  Returns
// the logits in z (wave 0, lane 0 holds all 10).
// Router features of the frame in FR: the 8x8-pixel cell means per channel (8 x 8 cells x 3),
// normalised as the predicates normalise their input.  Each (cell, row) segment is 8 pixels x 3
// channels = 24 contiguous elements (three aligned 16-byte reads); lanes 8m..8m+7 hold the eight
// rows of one cell and add them with three DPP steps.  Pass it (0 .. 512/NT - 1) covers segments
// tid + it * NT; lanes with row 0 hold their cell's three values.
template <int NT>
struct FrameFeat {
  float v[512 / NT][3];
};
template <int NT>
__device__ inline void frame_features(const __bf16* FR, float scale, FrameFeat<NT>& ff) {
#pragma unroll
  for (int it = 0; it < 512 / NT; ++it) {
    const int sg = threadIdx.x + it * NT;
    const int cell = sg >> 3, r = sg & 7, by = cell >> 3, bx = cell & 7;
    const uint4* p = reinterpret_cast<const uint4*>(FR + (8 * by + r + 1) * FRS + FR_X0 + 24 * bx);
    float c3[3] = {0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const uint4 u = p[q];
      const __bf16* h = reinterpret_cast<const __bf16*>(&u);
#pragma unroll
      for (int e = 0; e < 8; ++e) c3[(8 * q + e) % 3] += (float)h[e];
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      c3[c] += dpp_mov<0xB1>(c3[c]);    // quad_perm [1,0,3,2]
      c3[c] += dpp_mov<0x4E>(c3[c]);    // quad_perm [2,3,0,1]
      c3[c] += dpp_mov<0x141>(c3[c]);   // row_half_mirror: the other quad of the 8 lanes
      ff.v[it][c] = (c3[c] * scale - 0.5f) * 4.0f;
    }
  }
}
// Each thread with row 0 writes its cells' values (to HBM, or to sh.feat).
template <int NT>
__device__ inline void frame_features_put(const FrameFeat<NT>& ff, __bf16* dst) {
#pragma unroll
  for (int it = 0; it < 512 / NT; ++it) {
    const int sg = threadIdx.x + it * NT;
    if ((sg & 7) == 0) {
#pragma unroll
      for (int c = 0; c < 3; ++c) dst[(sg >> 3) * 3 + c] = static_cast<__bf16>(ff.v[it][c]);
    }
  }
}

template <typename T, int M, int NWV>
__device__ void cnn_frame(const CnnArgs& a, int slot, unsigned char* region, CnnShared& sh, const float* fcw,
                          bool next_valid, uint32_t next_idx, __bf16* feat_dst, float* z_out) {
  constexpr int NT = NWV * 64;                       // threads
  constexpr int C2 = 32 * M, C3 = 64 * M;
  typedef Pad<T> P1;
  typedef PadL2<T, M> P2;
  // FP32 tier (T = float): bf16 MFMAs on three-term operands, in the bf16 fragment layout (k-steps
  // of 32, 8 per lane); activations held in LDS as their three terms, or in fp32 and split at
  // every read where the terms do not fit (layer 2 of the widest class).  A layer-1 output is read
  // 2.25 times by each of one to four channel groups, a layer-2 output by all eight waves, so
  // splitting where they are written saves most of the vector work: FP32 kernel 861 -> 680 us a
  // launch on the 10,007-frame query, with layer 1's gather in five words instead of eight elements
  constexpr bool S3 = sizeof(T) == 4;
  typedef bf16x8 frag;
  // term t of the FP32 tier's packed layer l: fragments [slab][k-step][n-tile][lane]
  auto s3w = [&](int l, int t) {
    const size_t per_term = (size_t)cnn_slabs(l, M) * cnn_ksteps(l, M) * cnn_ntiles(l, M) * 64;
    return reinterpret_cast<const bf16x8*>(a.w_s3[slot][l]) + t * per_term;
  };
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, l16 = lane & 15;

  const __bf16* FR = reinterpret_cast<const __bf16*>(region);
  unsigned char* S1 = region + CnnLds<T>::S1_OFF;
  unsigned char* L2 = region;

  const __bf16* const* wpk = a.w_bf[slot];   // (bf16 tier)
  const float* b2 = sh.cb + CB_L2;
  const float* b3 = sh.cb + CB_L3;
  // The narrow classes fetch the next frame now: their layer 3 is too short to cover the HBM
  // latency before the frame is stored (not the four-wave m = 2 form: no registers to spare).
  constexpr bool kEarlyFetch = M == 1 || (M == 2 && NWV == 8);
  constexpr int KS1 = cnn_ksteps(0, M), KS2 = cnn_ksteps(1, M);
  constexpr int NT2 = 2 * M;
  // layer-2 wave tile: MT2 position tiles x NW2 channel tiles (the waves cover 16 x NT2)
  constexpr int MT2 = (M == 1 && NWV == 8) ? 2 : (M == 4 && sizeof(T) == 2) ? 8 : 4, NW2 = NT2 * (16 / MT2) / NWV;
  constexpr int NG2 = NT2 / NW2;                       // channel groups
  // weight prefetch depth (k-steps); the widest bf16 class has no registers to spare in layer 2
  constexpr int PD2 = S3 ? 1 : ((M == 4 || (M == 2 && NWV == 4)) ? 2 : 3);
  const int mg2 = wave / NG2, ng2 = wave % NG2;
  static_assert((16 / MT2) * NG2 == NWV, "layer-2 wave tiling must cover the waves");
  // With the early fetch, slab 0's layer-1 weights and its first PD2 layer-2 weight k-steps are
  // requested before the frame: a wave's vector loads complete in issue order, so a weight load
  // issued after the frame's would wait for the frame's HBM latency.  (Not in the FP32 kernel:
  // it has no registers to spare.)
  constexpr bool kPreW = kEarlyFetch && sizeof(T) == 2;
  frag w1_0[kPreW ? KS1 : 1];
  frag bw2_0[kPreW ? PD2 : 1][NW2];
  if constexpr (kPreW) {
    const frag* w1p0 = reinterpret_cast<const frag*>(wpk[0]);
#pragma unroll
    for (int ks = 0; ks < KS1; ++ks) w1_0[ks] = w1p0[ks * 64 + lane];
    const frag* w2p0 = reinterpret_cast<const frag*>(wpk[1]) + ng2 * NW2 * 64 + lane;
#pragma unroll
    for (int d = 0; d < PD2; ++d)
#pragma unroll
      for (int n = 0; n < NW2; ++n)
        if (d < KS2) bw2_0[d][n] = w2p0[(d * NT2 + n) * 64];
  }
  // First evaluation of a tuple in the first pass: its router features, from the frame in LDS.
  // Early fetch: computed now and stored by every wave right after the frame loads are issued
  // (everything waited on later already waits for those loads, which complete in issue order).
  // Late fetch: staged in LDS at slab 0 and stored by wave 0 after the late frame issue.
  const float fscale = (a.fr.dtype == HYDRO_DTYPE_U8 ? 1.0f / 255.0f : 1.0f) * (1.0f / 64.0f);
  FrameFeat<NT> ff;
  if (kEarlyFetch && feat_dst != nullptr) frame_features<NT>(FR, fscale, ff);
  // The frame loads are issued whether or not a next frame exists (next_idx is then the current
  // frame and nothing is stored): a conditional issue would leave the compiler unsure how many
  // loads are outstanding, and every later weight wait would then also wait for the frame.
  FramePrefetch<NT> pf;
  if (kEarlyFetch) frame_issue<NT>(a, next_idx, pf);
  if (kEarlyFetch && feat_dst != nullptr) frame_features_put<NT>(ff, feat_dst);

  // ---- layer-1 im2col fragments of this wave's MPW m-tiles (cached when several slabs reuse them)
  constexpr int MPW = 64 / NWV;                      // layer-1 m-tiles per wave
  constexpr bool kCacheA1 = sizeof(T) == 2 && M > 1 && NWV == 8;
  bf16x8 a1[kCacheA1 ? MPW : 1];
  static_assert(KS1 == 1 && MPW % 2 == 0, "layer 1: one k-step, whole rows of tiles");
  // (position j of row i: values from element 5 + 6 j of FR rows 2 i .. 2 i + 2; the wave's tiles are at
  // fixed distances from its first)
  constexpr int RP = FRS / 2;
  const uint32_t* gp[5];
#pragma unroll
  for (int i = 0; i < 5; ++i)
    gp[i] = reinterpret_cast<const uint32_t*>(FR) + wave * MPW * RP + (g < 3 ? g * RP + i : min(i, 2) * RP + 4) + 3 * l16 + 2;
  const uint32_t sel0 = conv1_sel(g);
  auto gather1 = [&](int q) -> bf16x8 {               // tile wave * MPW + q (MPW is even)
    uint32_t d[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) d[i] = gp[i][(q >> 1) * 2 * RP + (q & 1) * 48];
    return conv1_frag(d, g == 3, sel0);
  };
  if constexpr (kCacheA1) {
#pragma unroll
    for (int q = 0; q < MPW; ++q) a1[q] = gather1(q);
  }

  floatx4 acc2[MT2][NW2];
#pragma unroll
  for (int q = 0; q < MT2; ++q)
#pragma unroll
    for (int j = 0; j < NW2; ++j) acc2[q][j] = (floatx4){0.f, 0.f, 0.f, 0.f};

  // bf16, several slabs: layer 2's weights are one stream of k-steps over the slabs, two ahead of the
  // MFMAs, and layer 1's are requested a slab ahead, so that no slab starts by waiting for L2 (16,384
  // frames of the widest class 1,586 -> 1,494 us; six k-steps ahead in layer 3 changed nothing)
  constexpr bool kStream = sizeof(T) == 2 && M > 1;
  frag w1_next, bw2s[2][kStream ? NW2 : 1];
  const frag* w2s = reinterpret_cast<const frag*>(wpk[1]) + ng2 * NW2 * 64 + lane;
  if constexpr (kStream) {
    static_assert(PD2 == 2 && KS2 % 2 == 1, "pairs of k-steps and one");
    w1_next = reinterpret_cast<const frag*>(wpk[0])[lane];
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int n = 0; n < NW2; ++n) bw2s[d][n] = w2s[(d * NT2 + n) * 64];
  }
  (void)w1_next;
  (void)w2s;
  auto slab_pass = [&](int slab) {
    // layer 1: 64 m-tiles (16 positions each) x 16 channels; wave w owns m-tiles 8w..8w+7
    const frag* w1p = reinterpret_cast<const frag*>(wpk[0]) + (size_t)slab * KS1 * 64;
    frag w1f[S3 ? 1 : KS1];
    bf16x8 w1t[3];
    if constexpr (S3) {
#pragma unroll
      for (int t = 0; t < 3; ++t) w1t[t] = s3w(0, t)[slab * 64 + lane];
    } else if constexpr (kStream) {
      w1f[0] = w1_next;
    } else if (kPreW && slab == 0) {
#pragma unroll
      for (int ks = 0; ks < KS1; ++ks) w1f[ks] = w1_0[ks];
    } else {
#pragma unroll
      for (int ks = 0; ks < KS1; ++ks) w1f[ks] = w1p[ks * 64 + lane];
    }
    (void)w1t;
    if (!kEarlyFetch && slab == 0 && feat_dst != nullptr) {
      frame_features<NT>(FR, fscale, ff);
      frame_features_put<NT>(ff, sh.feat);
    }
    auto l1_store = [&](int q, const floatx4& acc) {
      unsigned char* dst = S1 + P1::at(wave * MPW / 2 + 1, l16 + 1, 8 * g) + (q >> 1) * P1::S1RB + (q & 1) * 8 * P1::S1PB;
      const float v[4] = {fmaxf(acc[0], 0.f), fmaxf(acc[1], 0.f), fmaxf(acc[2], 0.f), fmaxf(acc[3], 0.f)};
      if constexpr (S3) store_planes<3>(dst, 2 * CB1, v);
      else store4<__bf16>(reinterpret_cast<__bf16*>(dst), v[0], v[1], v[2], v[3]);
    };
    const floatx4 zero = (floatx4){0.f, 0.f, 0.f, 0.f};
    // tiles in pairs: both gathers, both MFMAs, then both epilogues, so one tile's LDS and MFMA
    // latencies overlap the other's.  FP32 tier: the raw frame values are exact in bf16, so the
    // three weight terms give every product exactly (smallest term first)
#pragma unroll (S3 ? 2 : 4)
    for (int q = 0; q < MPW; q += 2) {
      bf16x8 av0, av1;
      if constexpr (kCacheA1) {
        av0 = a1[q];
        av1 = a1[q + 1];
      } else {
        av0 = gather1(q);
        av1 = gather1(q + 1);
      }
      floatx4 acc0 = zero, acc1 = zero;
      if constexpr (S3) {
#pragma unroll
        for (int t = 2; t >= 0; --t) {
          acc0 = mfma_bf16(w1t[t], av0, acc0);
          acc1 = mfma_bf16(w1t[t], av1, acc1);
        }
      } else {
        acc0 = mfma_bf16(w1f[0], av0, zero);
        acc1 = mfma_bf16(w1f[0], av1, zero);
      }
      l1_store(q, acc0);
      l1_store(q + 1, acc1);
    }
    __syncthreads();
    if constexpr (S3) {
      // FP32 tier, layer 2 partial of this slab: K = 9 taps x 16 channels in k-steps of 32 (lane
      // group g: tap (32 ks + 8 g) / 16, channels from 8 (g % 2)); the weights run a k-step ahead
      const bf16x8* w2t[3] = {s3w(1, 0), s3w(1, 1), s3w(1, 2)};
      auto l2w = [&](int ks, bf16x8 (&w)[NW2][3]) {
#pragma unroll
        for (int n = 0; n < NW2; ++n)
#pragma unroll
          for (int t = 0; t < 3; ++t) w[n][t] = w2t[t][((slab * KS2 + ks) * NT2 + ng2 * NW2 + n) * 64 + lane];
      };
      auto l2_step = [&](int ks, const bf16x8 (&w)[NW2][3]) {
        const int k0 = ks * 32 + 8 * g;
        const int tp = min(k0 / CB1, 8);        // padded k (zero weights) reads a valid tap
        const int c0 = k0 % CB1;
        const int u = tp / 3, v = tp % 3;
        const unsigned char* src0 = S1 + P1::at(2 * mg2 * MT2 + u, 2 * l16 + v, c0 * 2);
#pragma unroll
        for (int q = 0; q < MT2; ++q) {
          const unsigned char* src = src0 + q * 2 * P1::S1RB;
          bf16x8 x[3];
#pragma unroll
          for (int t = 0; t < 3; ++t) x[t] = *reinterpret_cast<const bf16x8*>(src + t * 2 * CB1);
#pragma unroll
          for (int n = 0; n < NW2; ++n) acc2[q][n] = mfma_s3(w[n], x, acc2[q][n]);
          if (M == 4) __builtin_amdgcn_sched_barrier(0);    // one position tile's operands live at a time
        }
      };
      if constexpr (M == 4) {          // (no registers for two sets; a k-step's 96 MFMAs cover the latency)
        bf16x8 w[NW2][3];
#pragma unroll 1
        for (int ks = 0; ks < KS2; ++ks) {
          l2w(ks, w);
          l2_step(ks, w);
        }
      } else {
        bf16x8 wa[NW2][3], wb[NW2][3];
        l2w(0, wa);
#pragma unroll
        for (int ks = 0; ks < KS2; ++ks) {
          if (ks + 1 < KS2) l2w(ks + 1, ks & 1 ? wa : wb);
          __builtin_amdgcn_sched_barrier(0);
          l2_step(ks, ks & 1 ? wb : wa);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    } else if constexpr (kStream) {
      // layer 2 partial: K = 9 taps x 16 channels of this slab
      w1_next = reinterpret_cast<const frag*>(wpk[0])[min(slab + 1, M - 1) * 64 + lane];
      auto step = [&](int ks, frag (&w)[kStream ? NW2 : 1]) {
        const int k0 = ks * KSTEP + KPL * g, t = min(k0 / CB1, 8), c0 = k0 % CB1;   // (padded k: a valid tap, zero weights)
        const int u = t / 3, v = t - 3 * u;
        frag av[MT2];
        const unsigned char* src = S1 + P1::at(2 * mg2 * MT2 + u, 2 * l16 + v, c0 * (int)sizeof(T));
#pragma unroll
        for (int q = 0; q < MT2; ++q) av[q] = *reinterpret_cast<const frag*>(src + q * 2 * P1::S1RB);
#pragma unroll
        for (int n = 0; n < NW2; ++n)
#pragma unroll
          for (int q = 0; q < MT2; ++q) acc2[q][n] = mfma_bf16(w[n], av[q], acc2[q][n]);
        // (behind the last k-step the last fragment again, for nobody; the barrier keeps the loads here)
#pragma unroll
        for (int n = 0; n < NW2; ++n) w[n] = w2s[(min(slab * KS2 + ks + 2, M * KS2 - 1) * NT2 + n) * 64];
        __builtin_amdgcn_sched_barrier(0);
      };
#pragma unroll 1
      for (int ks = 0; ks + 1 < KS2; ks += 2) {
        step(ks, bw2s[0]);
        step(ks + 1, bw2s[1]);
      }
      step(KS2 - 1, bw2s[0]);
      // the next slab's first k-step is in the second set
#pragma unroll
      for (int n = 0; n < NW2; ++n) {
        const frag w = bw2s[0][n];
        bw2s[0][n] = bw2s[1][n];
        bw2s[1][n] = w;
      }
    } else {
      // layer 2 partial: K = 9 taps x 16 channels of this slab.  The weight fragments run PD2
      // k-steps ahead of the MFMAs (they come from L2 cache; one k-step of MFMAs is far shorter
      // than that latency).
      const frag* w2p = reinterpret_cast<const frag*>(wpk[1]) + (size_t)slab * KS2 * NT2 * 64 + ng2 * NW2 * 64 + lane;
      frag bw2[PD2][NW2];
      if (kPreW && slab == 0) {
  #pragma unroll
        for (int d = 0; d < PD2; ++d)
  #pragma unroll
          for (int n = 0; n < NW2; ++n)
            if (d < KS2) bw2[d][n] = bw2_0[d][n];
      } else {
  #pragma unroll
        for (int d = 0; d < PD2; ++d)
  #pragma unroll
          for (int n = 0; n < NW2; ++n)
            if (d < KS2) bw2[d][n] = w2p[(d * NT2 + n) * 64];
      }
  #pragma unroll (kPreW && M == 1 ? 4 : 1)
      for (int ks0 = 0; ks0 < KS2; ks0 += PD2) {
  #pragma unroll
        for (int d = 0; d < PD2; ++d) {
          const int ks = ks0 + d;
          // (when PD2 divides KS2 the guard folds away and the loop body has no branches)
          if (KS2 % PD2 == 0 || ks < KS2) {
            const int k0 = ks * KSTEP + KPL * g;
            int t = k0 / CB1;
            const int c0 = k0 % CB1;
            if (t > 8) t = 8;                       // padded k (zero weights) reads a valid tap
            const int u = t / 3, v = t % 3;
            frag av[MT2];
            const unsigned char* src = S1 + P1::at(2 * mg2 * MT2 + u, 2 * l16 + v, c0 * (int)sizeof(T));
  #pragma unroll
            for (int q = 0; q < MT2; ++q) av[q] = *reinterpret_cast<const frag*>(src + q * 2 * P1::S1RB);
  #pragma unroll
            for (int n = 0; n < NW2; ++n)
  #pragma unroll
              for (int q = 0; q < MT2; ++q) acc2[q][n] = mfma_bf16(bw2[d][n], av[q], acc2[q][n]);
            if constexpr (KS2 % PD2 == 0) {
              // unconditional refill; the last PD2 k-steps re-read the last fragment (unused).  The
              // scheduling barrier keeps the loads here: sunk to the end of the iteration (to
              // shorten register lifetimes) they would be waited on right after being issued.
  #pragma unroll
              for (int n = 0; n < NW2; ++n) bw2[d][n] = w2p[(min(ks + PD2, KS2 - 1) * NT2 + n) * 64];
              __builtin_amdgcn_sched_barrier(0);
            } else if (ks + PD2 < KS2) {
  #pragma unroll
              for (int n = 0; n < NW2; ++n) bw2[d][n] = w2p[((ks + PD2) * NT2 + n) * 64];
            }
          }
        }
      }
    }
    __syncthreads();
  };
#pragma unroll 1
  for (int slab = 0; slab < M; ++slab) slab_pass(slab);

  // ---- layer-2 epilogue into L2 (overwrites FR / S1)
#pragma unroll
  for (int n = 0; n < NW2; ++n) {
    const int ch = (ng2 * NW2 + n) * 16 + 4 * g;
    const float bb0 = b2[ch], bb1v = b2[ch + 1], bb2 = b2[ch + 2], bb3 = b2[ch + 3];
#pragma unroll
    for (int q = 0; q < MT2; ++q) {
      unsigned char* dst = L2 + P2::at(mg2 * MT2 + q + 1, l16 + 1, 0);
      const float v[4] = {fmaxf(acc2[q][n][0] + bb0, 0.f), fmaxf(acc2[q][n][1] + bb1v, 0.f),
                          fmaxf(acc2[q][n][2] + bb2, 0.f), fmaxf(acc2[q][n][3] + bb3, 0.f)};
      if constexpr (PadL2<T, M>::PLANES) store_planes<3>(dst + 2 * ch, 2 * C2, v);
      else store4<T>(reinterpret_cast<T*>(dst) + ch, v[0], v[1], v[2], v[3]);
    }
  }
  constexpr int WP2 = PadL2<T, M>::D / 16;               // 16-byte chunks per pixel
  for (int p = tid; p < (2 * L2_W - 1) * WP2; p += NT) {
    const int qq = p / WP2, c = p % WP2;
    const int y = qq < L2_W ? 0 : qq - L2_W + 1, x = qq < L2_W ? qq : 0;
    reinterpret_cast<uint4*>(L2 + P2::at(y, x, 0))[c] = make_uint4(0u, 0u, 0u, 0u);
  }
  __syncthreads();

  // ---- layer 3: 4 position tiles (64 positions) x 4M channel tiles; wave tile MT3 x NW3
  constexpr int KS3 = cnn_ksteps(2, M), NT3 = 4 * M;
  constexpr int MT3 = (M == 1 && NWV == 8) ? 2 : 4, NW3 = NT3 * (4 / MT3) / NWV;
  constexpr int MG3 = 4 / MT3;                         // position groups (1 or 2)
  constexpr int PD3 = S3 ? 1 : ((M == 2 && NWV == 4) ? 2 : 3);
  static_assert(MG3 * (NT3 / NW3) == NWV, "layer-3 wave tiling must cover the waves");
  const int mh = wave % MG3, ng = wave / MG3;
  floatx4 acc3[MT3][NW3];
#pragma unroll
  for (int q = 0; q < MT3; ++q)
#pragma unroll
    for (int j = 0; j < NW3; ++j) acc3[q][j] = (floatx4){0.f, 0.f, 0.f, 0.f};
  const frag* w3p = reinterpret_cast<const frag*>(wpk[2]) + (size_t)(ng * NW3) * 64 + lane;
  static_assert(KS3 % PD3 == 0, "layer-3 k-steps must be a multiple of the prefetch depth");
  frag bw3[PD3][NW3];
  if constexpr (!S3) {
#pragma unroll
    for (int d = 0; d < PD3; ++d)
#pragma unroll
      for (int n = 0; n < NW3; ++n) bw3[d][n] = w3p[(d * NT3 + n) * 64];
  }
  auto l3_step = [&](int ks, const frag (&b)[NW3]) {
    const int k0 = ks * KSTEP + KPL * g;
    const int t = k0 / C2, c0 = k0 % C2;
    const int u = t / 3, v = t % 3;
    frag av[MT3];
    const unsigned char* src = L2 + P2::at(4 * mh * MT3 + 2 * (l16 >> 3) + u, 2 * (l16 & 7) + v, c0 * (int)sizeof(T));
#pragma unroll
    for (int q = 0; q < MT3; ++q) av[q] = *reinterpret_cast<const frag*>(src + q * 4 * P2::RB);
#pragma unroll
    for (int n = 0; n < NW3; ++n)
#pragma unroll
      for (int q = 0; q < MT3; ++q) acc3[q][n] = mfma_bf16(b[n], av[q], acc3[q][n]);
  };
  if constexpr (sizeof(T) == 2) {
    // every k-step but the last PD3 refills its buffer PD3 k-steps ahead
#pragma unroll 1
    for (int ks0 = 0; ks0 < KS3 - PD3; ks0 += PD3) {
#pragma unroll
      for (int d = 0; d < PD3; ++d) {
        const int ks = ks0 + d;
        l3_step(ks, bw3[d]);
#pragma unroll
        for (int n = 0; n < NW3; ++n) bw3[d][n] = w3p[((ks + PD3) * NT3 + n) * 64];
      }
    }
    // The late fetch goes after the last weight request: loads complete in issue order, so any
    // weight requested after the frame would wait for it.
    if (!kEarlyFetch) frame_issue<NT>(a, next_idx, pf);
    if (!kEarlyFetch && feat_dst != nullptr && wave == 0 && lane < 24)
      reinterpret_cast<uint4*>(feat_dst)[lane] = reinterpret_cast<const uint4*>(sh.feat)[lane];
#pragma unroll
    for (int d = 0; d < PD3; ++d) l3_step(KS3 - PD3 + d, bw3[d]);
  } else {
    // FP32 tier: the frame is requested before layer 3 (its wait falls on the first k-step only);
    // the weight terms run a k-step ahead
    if (!kEarlyFetch) frame_issue<NT>(a, next_idx, pf);
    if (!kEarlyFetch && feat_dst != nullptr && wave == 0 && lane < 24)
      reinterpret_cast<uint4*>(feat_dst)[lane] = reinterpret_cast<const uint4*>(sh.feat)[lane];
    (void)bw3;
    const bf16x8* w3t[3] = {s3w(2, 0), s3w(2, 1), s3w(2, 2)};
    auto l3w = [&](int ks, bf16x8 (&w)[NW3][3]) {
#pragma unroll
      for (int n = 0; n < NW3; ++n)
#pragma unroll
        for (int t = 0; t < 3; ++t) w[n][t] = w3t[t][(ks * NT3 + ng * NW3 + n) * 64 + lane];
    };
    auto l3_s3step = [&](int ks, const bf16x8 (&w)[NW3][3]) {
      const int k0 = ks * 32 + 8 * g;
      const int tp = k0 / C2, c0 = k0 % C2;
      const int u = tp / 3, v = tp % 3;
      const unsigned char* src0 = L2 + P2::at(4 * mh * MT3 + 2 * (l16 >> 3) + u, 2 * (l16 & 7) + v, 0);
#pragma unroll
      for (int q = 0; q < MT3; ++q) {
        const unsigned char* src = src0 + q * 4 * P2::RB;
        bf16x8 x[3];
        if constexpr (PadL2<T, M>::PLANES) {
#pragma unroll
          for (int t = 0; t < 3; ++t) x[t] = *reinterpret_cast<const bf16x8*>(src + 2 * c0 + t * 2 * C2);
        } else {
          const float4* p = reinterpret_cast<const float4*>(src + 4 * c0);
          split3(p[0], p[1], x);
        }
#pragma unroll
        for (int n = 0; n < NW3; ++n) acc3[q][n] = mfma_s3(w[n], x, acc3[q][n]);
        if (!PadL2<T, M>::PLANES) __builtin_amdgcn_sched_barrier(0);   // one tile's operands live at a time
      }
    };
    bf16x8 wa[NW3][3], wb[NW3][3];
    l3w(0, wa);
#pragma unroll 1
    for (int ks = 0; ks + 1 < KS3; ks += 2) {
      l3w(ks + 1, wb);
      __builtin_amdgcn_sched_barrier(0);
      l3_s3step(ks, wa);
      l3w(min(ks + 2, KS3 - 1), wa);
      __builtin_amdgcn_sched_barrier(0);
      l3_s3step(ks + 1, wb);
    }
    if constexpr (KS3 % 2 == 1) l3_s3step(KS3 - 1, wa);
  }
  // ReLU + pooled partial sums over this wave's positions
#pragma unroll
  for (int n = 0; n < NW3; ++n) {
    const int ch0 = (ng * NW3 + n) * 16 + 4 * g;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float bb = b3[ch0 + r];
      float s = 0.f;
#pragma unroll
      for (int q = 0; q < MT3; ++q) s += fmaxf(acc3[q][n][r] + bb, 0.f);
      s = row_sum16(s);
      if (l16 == 0) sh.gpart[mh][ch0 + r] = s;
    }
  }
  __syncthreads();
  // wave 0: FC (lanes over channels) -> z; the other waves store the next frame meanwhile
  if (wave == 0) {
    const float* fw = fcw;
    float zp[kClasses];
#pragma unroll
    for (int c = 0; c < kClasses; ++c) zp[c] = 0.f;
#pragma unroll
    for (int q = 0; q < M; ++q) {
      const int ch = lane + 64 * q;
      float gs = sh.gpart[0][ch];
      if constexpr (MG3 == 2) gs += sh.gpart[1][ch];
      const float gch = gs * (1.0f / 64.0f);
#pragma unroll
      for (int c = 0; c < kClasses; ++c) zp[c] += gch * fw[ch * kClasses + c];
    }
    wave_sum_n(zp);
#pragma unroll
    for (int c = 0; c < kClasses; ++c) z_out[c] = zp[c] + sh.fcb[c];
  }
  if (next_valid) frame_store<T, NT>(a, pf, region);
}

// Persistent over every queue of the launch: entry t of the concatenated queues goes to workgroup
// t mod grid; slots are ordered by cost, so the widest frames come first.  VSET is the set of width
// classes the instantiation holds code for (bit m for width multiplier m); one register
// allocation covers them all, so classes whose union would spill get launches of their own.
template <typename T, int VSET, int NWV = 8>
__global__ __launch_bounds__(NWV * 64) __attribute__((amdgpu_waves_per_eu(NWV == 4 ? 2 : 1)))
void cnn_fused_kernel(CnnArgs a, Forward f) {
  constexpr int NT = NWV * 64;
  constexpr int MMAX = (VSET & 4) ? 4 : (VSET & 2) ? 2 : 1;   // widest class of the launch
  __shared__ __attribute__((aligned(16))) unsigned char region[CnnLds<T, MMAX>::REGION];
  __shared__ CnnShared sh;
  // FC weights of the current slot (the FP32 kernel of the widest class has no LDS left and reads them
  // from global memory)
  constexpr bool FCL = sizeof(T) == 2 || MMAX < 4;
  __shared__ float fcw_s[FCL ? 64 * MMAX * kClasses : 1];
  const int tid = threadIdx.x;
  if (tid == 0) sh.dec.n = 0;
  if (tid < kMaxK) sh.ticks[tid] = 0;
  // queue prefix offsets, kept in LDS (read when entries are staged)
  __shared__ int cum_s[kMaxK + 1];
  if (tid == 0) {
    int c = 0;
    cum_s[0] = 0;
    for (int i = 0; i < kMaxK; ++i) {
      c += i < a.n_preds ? a.q.counts[a.pred[i]] : 0;
      cum_s[i + 1] = c;
    }
  }
  __syncthreads();
  const int total = cum_s[kMaxK];
  const int G = gridDim.x;
  // This workgroup's queue entries, their slots and decision thresholds are staged in LDS, ECH
  // frames per chunk, double-buffered: wave 0 requests chunk c + 1 when chunk c starts.  The
  // per-frame path then issues no dependent global load (a wave's vector loads complete in issue
  // order, so a per-frame entry or threshold load would hold up the next weight wait).
  constexpr int ECH = 64;
  __shared__ uint32_t ring_e[2 * ECH];
  __shared__ float ring_th[2 * ECH];
  __shared__ uint8_t ring_s[2 * ECH];
  auto fill = [&](int c, int lo) {
    const int i = tid - lo;
    if (i >= 0 && i < ECH) {
      const int t = (int)blockIdx.x + (c * ECH + i) * G;
      if (t < total) {
        int slot = 0, base = 0;
        for (int j = 1; j < a.n_preds; ++j)
          if (t >= cum_s[j]) { slot = j; base = cum_s[j]; }
        const uint32_t e = a.q.entries[(int64_t)a.pred[slot] * a.q.cap + (t - base)];
        ring_e[(c & 1) * ECH + i] = e;
        ring_s[(c & 1) * ECH + i] = (uint8_t)slot;
        ring_th[(c & 1) * ECH + i] = f.logits == nullptr ? theta_of(f, a.pred[slot], entry_idx(e)) : 0.f;
      }
    }
  };
  fill(0, 0);
  fill(1, 64);
  __syncthreads();
  if ((int)blockIdx.x < total) {
    FramePrefetch<NT> pf;
    frame_issue<NT>(a, entry_idx(ring_e[0]), pf);
    frame_store<T, NT>(a, pf, region);
  }
  __syncthreads();
  int loaded = -1;
  int nf = 0;   // frames of this workgroup so far
  for (int t = blockIdx.x; t < total; t += G, ++nf) {
    if (nf % ECH == 0 && nf > 0) fill(nf / ECH + 1, 0);   // read after this frame's barriers
    const int slot = ring_s[nf % (2 * ECH)];
    const int k = a.pred[slot];
    const int v = a.variant[slot];
    if (slot != loaded) {
      const int m = v == CNN_W4 ? 4 : v == CNN_W2 ? 2 : 1;
      for (int q = tid; q < 32 * m; q += NT) sh.cb[CB_L2 + q] = a.bias[slot][1][q];
      for (int q = tid; q < 64 * m; q += NT) sh.cb[CB_L3 + q] = a.bias[slot][2][q];
      if (tid < kClasses) sh.fcb[tid] = a.fc_b[slot][tid];
      if constexpr (FCL) {
        for (int q = tid; q < 64 * m * kClasses; q += NT) fcw_s[q] = a.fc_w[slot][q];
      }
      __syncthreads();
      loaded = slot;
    }
    const float* fcw = FCL ? fcw_s : a.fc_w[slot];
    const uint32_t e = ring_e[nf % (2 * ECH)];
    const uint32_t idx = entry_idx(e);
    const float th = ring_th[nf % (2 * ECH)];
    const bool next_valid = t + G < total;
    // with no next frame, the loads re-read this one (cached) unused
    const uint32_t next_idx = next_valid ? entry_idx(ring_e[(nf + 1) % (2 * ECH)]) : idx;
    __bf16* feat_dst = a.feats != nullptr && f.logits == nullptr && entry_mask(e) == 0
                           ? a.feats + (int64_t)idx * 192 : nullptr;
    unsigned long long t0 = wall_clock64();
    float z[kClasses];
    if constexpr ((VSET & 4) != 0) {
      if (v == CNN_W4) cnn_frame<T, 4, NWV>(a, slot, region, sh, fcw, next_valid, next_idx, feat_dst, z);
    }
    if constexpr ((VSET & 2) != 0) {
      if (v == CNN_W2) cnn_frame<T, 2, NWV>(a, slot, region, sh, fcw, next_valid, next_idx, feat_dst, z);
    }
    if constexpr ((VSET & 1) != 0) {
      if (v == CNN_W1) cnn_frame<T, 1, NWV>(a, slot, region, sh, fcw, next_valid, next_idx, feat_dst, z);
    }
    if (tid == 0) {
      if (f.logits != nullptr) {
        for (int c = 0; c < kClasses; ++c) f.logits[(int64_t)idx * kClasses + c] = (double)z[c];
      } else {
        float d = class_margin(z, a.class_mask[slot]);
        bool defer = f.defer.entries != nullptr && fabsf(d - th) < f.tau[k];
        decision_set(sh.dec, sh.dec.n++, k, e, defer, d > th);
      }
      sh.ticks[k] += wall_clock64() - t0;
    }
    __syncthreads();
    if (sh.dec.n == DBUF) decision_flush(f, sh.dec, a.n_preds, a.pred);
  }
  if (f.logits == nullptr) decision_flush(f, sh.dec, a.n_preds, a.pred);
  __syncthreads();
  if (tid < kMaxK && sh.ticks[tid] && a.count_ticks) atomicAdd(&a.st->r_ticks[tid], sh.ticks[tid]);
}

// ---------------------------------------------------------------- host helpers
int cnn_variant_of(int in_hw, int n_layers, const int* widths) {
  if (in_hw != 64 || n_layers != 3) return CNN_NONE;
  for (int v = 0, m = 1; v < 3; ++v, m *= 2)
    if (widths[0] == 16 * m && widths[1] == 32 * m && widths[2] == 64 * m) return v;
  return CNN_NONE;
}

static int mult_of(int variant) { return variant == CNN_W1 ? 1 : variant == CNN_W2 ? 2 : 4; }

size_t cnn_packed_elems(int variant, int layer) {
  const int m = mult_of(variant);
  return (size_t)cnn_slabs(layer, m) * cnn_ksteps(layer, m) * cnn_ntiles(layer, m) * 64 * KPL;
}

// Term t (0, 1, 2) of v as a sum of three bf16 values.
static float bf16_term(float v, int t) {
  for (;; --t) {
    const float h = static_cast<float>(static_cast<__bf16>(v));
    if (t == 0) return h;
    v -= h;
  }
}

// Pack one conv layer ([co][ci][3][3] fp32, scaled by `scale`) into fragment order; bias: layer 1's.
void cnn_pack_layer(int variant, int layer, const float* w, float scale, const float* bias, float* out) {
  const int m = mult_of(variant);
  const int slabs = cnn_slabs(layer, m), ks_n = cnn_ksteps(layer, m), nt_n = cnn_ntiles(layer, m);
  const int C2 = 32 * m;
  const int cin = layer == 0 ? 3 : layer == 1 ? 16 * m : C2;
  size_t o = 0;
  for (int sl = 0; sl < slabs; ++sl)
    for (int ks = 0; ks < ks_n; ++ks)
      for (int nt = 0; nt < nt_n; ++nt)
        for (int lane = 0; lane < 64; ++lane)
          for (int e = 0; e < KPL; ++e) {
            const int k = ks * KSTEP + KPL * (lane >> 4) + e;
            const int n = nt * 16 + (lane & 15);
            int oc, ic, tap;
            bool valid;
            if (layer == 0) {
              // k = 9u + 3v + c in conv1_k's slots, then the bias in three bf16 terms
              const int kk = conv1_k(lane >> 4, e);
              tap = (kk / 9) * 3 + (kk % 9) / 3;
              ic = kk % 3;
              oc = sl * CB1 + n;
              valid = kk < 27;
              if (kk >= 27) {
                out[o++] = kk < 30 ? bf16_term(bias[oc], kk - 27) : 0.f;
                continue;
              }
            } else if (layer == 1) {
              tap = k / CB1;
              ic = sl * CB1 + k % CB1;
              oc = n;
              valid = tap < 9;
            } else {
              tap = k / C2;
              ic = k % C2;
              oc = n;
              valid = tap < 9;
            }
            out[o++] = valid ? scale * w[((size_t)(oc * cin + ic) * 3 + tap / 3) * 3 + tap % 3] : 0.f;
          }
}

void launch_cnn_pass(const CnnArgs& a, const Forward& f, int tier, int grid, hipStream_t s) {
  if (a.n_preds == 0) return;
  if (tier == TIER_F64) {
    F64Args b{};
    b.n_preds = a.n_preds;
    for (int i = 0; i < a.n_preds; ++i) {
      const int m = mult_of(a.variant[i]);
      b.pred[i] = a.pred[i]; b.class_mask[i] = a.class_mask[i]; b.n_layers[i] = 3; b.in_hw[i] = H0;
      for (int l = 0; l < 3; ++l) {
        b.widths[i][l] = (16 << l) * m;
        b.wt[i][l] = a.wt_canon[i][l]; b.bias[i][l] = a.b_canon[i][l];
      }
      b.fc_w[i] = a.fc_w[i]; b.fc_b[i] = a.fc_b[i]; b.esc_act[i] = a.esc_act[i];
    }
    b.esc_stride = a.esc_stride; b.esc_off = a.esc_off; b.esc_cap = a.esc_cap;
    b.scratch = a.scratch64; b.per_block = a.scratch64_per_block; b.scratch_off = a.scratch64_per_block / 2;
    b.rest_grid = a.rest_grid; b.q = a.q; b.fr = a.fr;
    launch_f64_cnn(b, f, grid, s);
    return;
  }
  // The FP32 re-score tier: one persistent launch over every queue of the pass (its queues are a band
  // of a few hundred frames; a launch per class has a tail per class).  A first pass, whose queues
  // are long: one launch per width class (a shared launch would give the narrow classes the
  // widest one's register allocation and code footprint).  BF16: the widest class
  // runs 8-wave workgroups, one per CU; the two narrower classes 4-wave workgroups, two per CU, so
  // one workgroup's LDS phases overlap the other's matrix phases.  FP32: the layer-1 slab leaves room
  // for one workgroup per CU, of 8 waves (10,007 frames through the classes in turn: 440 / 550 / 1040 us;
  // one launch for all: 490 / 575 / 1080; 16 waves for the narrower two: 465 / 550, with spills).  Up to 16
  // frames a workgroup the classes' tails outweigh that, since a shared launch runs them beside each other
  // (queries over three classes, FP32, shared against per class: 200 frames 305 / 376 us, 1,024 391 / 460,
  // 4,096 721 / 773 or 747 / 745 in written order, 8,192 1,146 / 1,195 or 1,297 / 1,276).
  const bool bf = a.prec == HYDRO_PREC_BF16;
  bool mixed = false;
  for (int i = 1; i < a.n_preds; ++i) mixed = mixed || a.variant[i] != a.variant[0];
  if (tier != TIER_FIRST || (!bf && mixed && a.most <= (int64_t)16 * grid)) {
    hipLaunchKernelGGL((cnn_fused_kernel<float, 7>), dim3(grid), dim3(NTHR), 0, s, a, f);
    return;
  }
  for (int v = CNN_W4; v >= CNN_W1; --v) {
    CnnArgs b = a;
    b.n_preds = 0;
    for (int i = 0; i < a.n_preds; ++i) {
      if (a.variant[i] != v) continue;
      const int j = b.n_preds++;
      b.pred[j] = a.pred[i]; b.variant[j] = a.variant[i]; b.class_mask[j] = a.class_mask[i];
      for (int l = 0; l < 3; ++l) {
        b.w_bf[j][l] = a.w_bf[i][l]; b.w_s3[j][l] = a.w_s3[i][l]; b.bias[j][l] = a.bias[i][l];
        b.b_canon[j][l] = a.b_canon[i][l]; b.wt_canon[j][l] = a.wt_canon[i][l];
      }
      b.fc_w[j] = a.fc_w[i]; b.fc_b[j] = a.fc_b[i]; b.esc_act[j] = a.esc_act[i];
    }
    if (b.n_preds == 0) continue;
    if (!bf) {
      if (v == CNN_W4) hipLaunchKernelGGL((cnn_fused_kernel<float, 4>), dim3(grid), dim3(NTHR), 0, s, b, f);
      else if (v == CNN_W2) hipLaunchKernelGGL((cnn_fused_kernel<float, 2, 8>), dim3(grid), dim3(512), 0, s, b, f);
      else hipLaunchKernelGGL((cnn_fused_kernel<float, 1, 8>), dim3(grid), dim3(512), 0, s, b, f);
    } else if (v == CNN_W4) hipLaunchKernelGGL((cnn_fused_kernel<__bf16, 4>), dim3(grid), dim3(NTHR), 0, s, b, f);
    else if (v == CNN_W2) hipLaunchKernelGGL((cnn_fused_kernel<__bf16, 2, 4>), dim3(grid * 2), dim3(256), 0, s, b, f);
    else hipLaunchKernelGGL((cnn_fused_kernel<__bf16, 1, 4>), dim3(grid * 2), dim3(256), 0, s, b, f);
  }
}

}  // namespace hydro
