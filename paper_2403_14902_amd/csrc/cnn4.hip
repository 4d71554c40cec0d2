// Four-layer CNN predicates on 128x128x3 frames (conv3x3/s2/p1 widths 32-64-128-256, ReLU, mean
// pool, FC 10) on gfx950, in three launches per tier and round:
//
//   front   one frame per workgroup pass: layer 1 (K = 27 on one bf16 MFMA k-step) and layer 2,
//           streamed in eight bands of four layer-2 output rows.  Layer 1's output never leaves
//           LDS: a ring of nine layer-1 rows (the eight of the band plus the one above it) feeds
//           layer 2, whose weights stay in registers for the whole launch.  Layer 2's output
//           (32x32x64) goes to an activation buffer.
//   gemm3   layer 3 as an implicit GEMM over every queued frame of the launch: rows = output
//           positions, columns = the 128 output channels, K = (tap, input channel) = 576.
//   gemm4   layer 4 the same way (K = 1152, 256 channels), with the epilogue pooling each
//           frame's 64 positions, applying FC, the class-subset margin and the decision.
//
// Arithmetic tiers (template P): FP32 and the three-product tier (bf16 MFMAs on operands split into
// bf16 terms; layer 1 and 2's activations as planes of terms in LDS, layers 3 and 4's split where they are
// read, or stored as two planes), BF16 (16x16x32 and 32x32x16 MFMAs) and FP8 (OCP e4m3 operands on
// the scaled 16x16x128 MFMA with unit block scales; per-output-channel weight scales and per-layer
// activation scales applied in fp32 in the epilogues).  Layer 1 runs bf16 in the BF16 and FP8 tiers:
// raw uint8 / bf16 frame values are exact in bf16, and the normalisation is folded into its weights.
// Accumulation is fp32 throughout.
//
// The GEMM tiles copy A (weights, pre-packed per k-block in the LDS image order) and B (the im2col rows
// of the activations, gathered per 16-byte chunk) straight from global memory into a ring of two to
// five LDS stages.  LDS rows are XOR-swizzled by 16-byte chunk so that the sixteen rows an MFMA
// fragment reads fall on distinct banks.
#include <cmath>
#include <cstring>
#include <vector>

#include "engine.h"

namespace hydro {

template <int P> struct C4T;
template <> struct C4T<C4_F32> { typedef float T; static constexpr int ES = 4; };
template <> struct C4T<C4_BF16> { typedef __bf16 T; static constexpr int ES = 2; };
template <> struct C4T<C4_FP8> { typedef uint8_t T; static constexpr int ES = 1; };
template <> struct C4T<C4_S3> { typedef float T; static constexpr int ES = 4; };

typedef int i32x8 __attribute__((ext_vector_type(8)));

__device__ inline floatx4 c4_mfma(bf16x8 a, bf16x8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// BF16 contractions use the 32x32x16 MFMA, which keeps the matrix pipe busy with few independent
// accumulators.  Lane l supplies A[l % 32][8 (l / 32) + e] and B[8 (l / 32) + e][l % 32]; output
// element (i, j) sits in lane j + 32 ((i / 4) % 2), value (i % 4) + 4 (i / 8).
typedef float floatx16 __attribute__((ext_vector_type(16)));
__device__ inline floatx16 c4_mfma32(bf16x8 a, bf16x8 b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// e4m3 x e4m3, K = 128, block scales 2^0 (E8M0 127)
__device__ inline floatx4 c4_mfma(i32x8 a, i32x8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 0, 0, 0, 127, 0, 127);
}

// Round to e4m3 (RNE) with saturation at the largest finite value (the conversion itself does
// not saturate: values above 448 would become NaN).
__device__ inline uint32_t c4_pack_fp8x4(float v0, float v1, float v2, float v3) {
  v0 = fminf(v0, 448.f); v1 = fminf(v1, 448.f); v2 = fminf(v2, 448.f); v3 = fminf(v3, 448.f);
  int w = __builtin_amdgcn_cvt_pk_fp8_f32(v0, v1, 0, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(v2, v3, w, true);
  return (uint32_t)w;
}

// Stores 4 consecutive activations (already >= 0) in the tier's element type.
template <int P>
__device__ inline void c4_store4(void* dst, float v0, float v1, float v2, float v3) {
  if constexpr (P == C4_F32 || P == C4_S3) {
    *reinterpret_cast<float4*>(dst) = make_float4(v0, v1, v2, v3);
  } else if constexpr (P == C4_BF16) {
    alignas(8) __bf16 h[4] = {static_cast<__bf16>(v0), static_cast<__bf16>(v1), static_cast<__bf16>(v2),
                              static_cast<__bf16>(v3)};
    *reinterpret_cast<uint2*>(dst) = *reinterpret_cast<const uint2*>(h);
  } else {
    *reinterpret_cast<uint32_t*>(dst) = c4_pack_fp8x4(v0, v1, v2, v3);
  }
}

// Calibration (FP32 tier): running maximum of a layer's activations, as float bits (values >= 0
// order like their bit patterns).
__device__ inline void c4_track_max(unsigned* slot, float v) {
  if (slot == nullptr) return;
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  if (lane_id() == 0 && v > 0.f) atomicMax(slot, __float_as_uint(v));
}

// ---------------------------------------------------------------- front: layers 1 and 2
constexpr int F_NB = 8;            // bands per frame (four layer-2 rows each)
constexpr int F_RING = 9;          // layer-1 rows held: the band's eight and the one above
constexpr int F_SLOTS = 65;        // layer-1 columns of a row: even 0..62, then odd -1..63
constexpr int F_FROWS = 17;        // frame rows a band reads
constexpr int F_FX0 = 8;           // element of column 0 in a staged frame row (16-byte aligned); the
                                   // left pad column is the three elements before it
constexpr int F_FPITCH = F_FX0 + 128 * 3;
// Per tier: waves per workgroup, bytes per layer-1 column slot (32 channels, FP32 arithmetic in bf16
// planes of 64 bytes, + padding: the slot pitch in 16-byte units is odd so that eight consecutive
// slots fall on distinct bank groups), output channels per wave of layer 2
template <int P, bool X3> struct FrontCfg;
template <bool X3> struct FrontCfg<C4_F32, X3> { static constexpr int NW = 8, PLANES = X3 ? 2 : 3, PITCH = X3 ? 144 : 208, CW = 32; };
template <> struct FrontCfg<C4_BF16, false> { static constexpr int NW = 4, PLANES = 1, PITCH = 80, CW = 64; };
template <> struct FrontCfg<C4_FP8, false> { static constexpr int NW = 4, PLANES = 1, PITCH = 48, CW = 64; };

// bytes per position row of a wave's layer-2 output staging (its channels + 16 bytes of padding)
template <int P> constexpr int F_TPITCH = FrontCfg<P, false>::CW * C4T<P>::ES + 16;
// the frame band area, which also stages the layer-2 output (32 positions a wave) after layer 1 has
// read the band
constexpr int c4_max(int x, int y) { return x < y ? y : x; }
template <int P> constexpr int front_waves() { typedef FrontCfg<P, false> C; return C::NW; }
template <int P> constexpr int F_FRAME_B = c4_max(F_FROWS * F_FPITCH * 2, front_waves<P>() * 32 * F_TPITCH<P>);
// A ring row: even columns j at j / 2 slots, odd ones (from -1) at ODD + (j + 1) / 2 slots.  The gap
// before the odd ones makes sixteen consecutive columns, which one store writes, fall on distinct
// 16-byte bank groups: with a slot of p (odd) groups, even column 2m starts at group p m, odd column 2m + 1
// at p m + 8.
template <int PITCH> struct RingRow {
  static constexpr int GAP = ((8 - PITCH / 16) % 16 + 16) % 16 * 16;
  static constexpr int ODD = 32 * PITCH + GAP, BYTES = F_SLOTS * PITCH + GAP;
};
template <int P, bool X3> constexpr int front_ring_bytes() { typedef FrontCfg<P, X3> C; return F_RING * RingRow<C::PITCH>::BYTES; }
template <int P, bool X3> constexpr int front_lds_bytes() { return F_FRAME_B<P> + front_ring_bytes<P, X3>(); }

// Where channel ch (a multiple of 4) of a position stored as two planes starts: [32-channel group][hi, mid][32].
__device__ inline unsigned char* c4_plane_ptr(void* pos, int ch) {
  return static_cast<unsigned char*>(pos) + (ch >> 5) * 128 + (ch & 31) * 2;
}

// What bounds it: vector instructions and latency, not the matrix cores (25 % busy in BF16 before).
// Hence the layer-1 gather as five loads at addresses fixed for the launch, two permutes and two
// shifts, the biases inside the MFMAs (layer 1 in spare K slots, layer 2 as the accumulators' start),
// and for the FP32 arithmetic the split of layer 1's outputs into bf16 terms once, where they are
// written to the ring, with eight waves (four, splitting at every read: 113 us a frame in the
// three-product tier, now 66).  8,192 uint8 frames in BF16: 603 -> 565 us; eight waves of half the channels
// each took the same time there, what they gained in latency spent on twice the ring reads.
// X3 (with P = C4_F32 only): the three-product arithmetic of the C4_X3 tier; its layer-2 outputs are
// stored as two bf16 planes, [position][32-channel group][hi, mid][32], in the bytes of the fp32 values.
template <int P, bool U8, bool X3 = false>
__global__ __launch_bounds__((FrontCfg<P, X3>::NW * 64)) __attribute__((amdgpu_waves_per_eu(2)))
void c4_front_kernel(GcnnArgs a) {
  typedef typename C4T<P>::T T;
  typedef FrontCfg<P, X3> C;
  constexpr int ES = C4T<P>::ES;
  constexpr int PITCH = C::PITCH, PLANES = C::PLANES, NTHR = C::NW * 64;
  constexpr bool F32 = P == C4_F32;
  __shared__ __attribute__((aligned(16))) unsigned char lds[front_lds_bytes<P, X3>()];
  __shared__ unsigned long long ticks_s[kMaxK];
  // per-slot epilogue constants: layer-2 bias [64], FP8 layer-2 scales [64]
  __shared__ __attribute__((aligned(16))) float consts_s[128];
  // layer-1 fragments: [channel tile]; X3: [term][channel tile] (three terms stay in registers, LDS is full)
  constexpr int W1N = X3 ? 4 : F32 ? 1 : 2;
  __shared__ __attribute__((aligned(16))) bf16x8 w1_s[W1N][64];
  __bf16* fb = reinterpret_cast<__bf16*>(lds);          // staged frame band (raw values, bf16)
  unsigned char* ring = lds + F_FRAME_B<P>;                // layer-1 output rows
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, l16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (tid < kMaxK) ticks_s[tid] = 0;
  // the left pad column (the first odd one) of every ring row is a zero activation
  typedef RingRow<PITCH> RR;
  for (int q = tid; q < F_RING * (PITCH / 4); q += NTHR)
    reinterpret_cast<uint32_t*>(ring + (q / (PITCH / 4)) * RR::BYTES + RR::ODD)[q % (PITCH / 4)] = 0u;

  int total = 0;
  for (int i = 0; i < a.n_preds; ++i) total += a.c4[i] ? a.q.counts[a.pred[i]] : 0;
  // frame staging: chunk q (16 bytes) of band row r; uint8 frames: 24 chunks a row, bf16: 48.
  // The next band's chunks are loaded into registers while the current band's layer 2 runs (the
  // next frame's first band during the last band), and converted into LDS after it.
  constexpr int CPR = U8 ? 24 : 48;
  constexpr int NCHUNK = F_FROWS * CPR;
  constexpr int NPF = (NCHUNK + NTHR - 1) / NTHR;
  constexpr int FROWB = 128 * 3 * (U8 ? 1 : 2);
  u32x4 pf[NPF];
  // the loads are unconditional (indices clamped; a clamped chunk is never committed), so that the
  // registers are not merged across branches and the wait for them falls at the commit
#define C4_FISSUE(frm_, band_)                                                                     \
  do {                                                                                             \
    _Pragma("unroll") for (int c = 0; c < NPF; ++c) {                                              \
      const int q = min(tid + NTHR * c, NCHUNK - 1);                                               \
      const int y = max(16 * (band_) - 1 + q / CPR, 0);                                            \
      pf[c] = reinterpret_cast<const u32x4*>((frm_) + (int64_t)y * FROWB)[q % CPR];                \
    }                                                                                              \
  } while (0)
  const uint32_t pad2 = __builtin_amdgcn_perm(__float_as_uint(a.pad_raw), __float_as_uint(a.pad_raw), 0x07060302u);
#define C4_FCOMMIT(band_)                                                                          \
  do {                                                                                             \
    /* the pad column (the three elements before column 0; the area also stages layer-2 output) */ \
    if (tid < F_FROWS * 2)                                                                         \
      reinterpret_cast<uint32_t*>(fb + (tid >> 1) * F_FPITCH)[2 + (tid & 1)] = pad2;               \
    _Pragma("unroll") for (int c = 0; c < NPF; ++c) {                                              \
      const int q = tid + NTHR * c;                                                                \
      if (q < NCHUNK) {                                                                            \
        const int r = q / CPR, j = q % CPR;                                                        \
        u32x4* dst = reinterpret_cast<u32x4*>(fb + r * F_FPITCH + F_FX0 + (U8 ? 16 : 8) * j);      \
        const bool above = (band_) == 0 && r == 0;     /* the row above the frame */               \
        if (U8) {                                                                                  \
          u32x4 h[2];                                                                              \
          _Pragma("unroll") for (int w = 0; w < 8; ++w) {                                          \
            /* bf16 of a byte: the upper half of its float (exact) */                              \
            const uint32_t b = pf[c][w >> 1] >> (16 * (w & 1));                                    \
            const uint32_t f0 = __float_as_uint((float)(b & 255u)), f1 = __float_as_uint((float)(b >> 8 & 255u)); \
            h[w >> 2][w & 3] = above ? pad2 : __builtin_amdgcn_perm(f1, f0, 0x07060302u);          \
          }                                                                                        \
          dst[0] = h[0];                                                                           \
          dst[1] = h[1];                                                                           \
        } else {                                                                                   \
          dst[0] = above ? (u32x4){pad2, pad2, pad2, pad2} : pf[c];                                \
        }                                                                                          \
      }                                                                                            \
    }                                                                                              \
  } while (0)
  bool pf_valid = false;      // pf holds band pf_band of frame pf_idx
  uint32_t pf_idx = 0;
  int pf_band = 0;
  // Few frames (a re-score band, a small query): a frame's bands are shared among up to eight
  // workgroups, as many as leave every workgroup one item at most.  A segment that does not start at
  // band 0 first runs layer 1 alone of the band before it (its last row is the one above the
  // segment).  Some 20 frames in FP32: 90 -> 22 us, 16 with the eight waves.
  int segs = 1;
  while (segs < F_NB && total * segs * 2 <= (int)gridDim.x) segs *= 2;
  const int seg_nb = F_NB / segs;
  total *= segs;

  // Layer 1's gather.  The 9 values of input row u for output column j (pixels 2j-1 .. 2j+1) are
  // elements 6j + 5 .. 6j + 13 of the staged row: dwords from element 6j + 4 hold them in pairs.
  // Lane groups 0..2 read dwords 0..4 of row g, group 3 dword 4 of rows 0..2.
  constexpr int RP = F_FPITCH / 2;            // dwords per staged row
  constexpr int L1R = 8 / C::NW;              // layer-1 rows per wave
  const uint32_t* gp[5];
#pragma unroll
  for (int i = 0; i < 5; ++i)
    gp[i] = reinterpret_cast<const uint32_t*>(fb) + 2 * L1R * wave * RP + (g < 3 ? g * RP + i : min(i, 2) * RP + 4) + 3 * l16 + 2;
  // group 3: word 0 = ninths of rows 0 and 1, word 1 = ninth of row 2 and 1.0, word 2 = 1.0, 1.0, word 3 = 0
  const uint32_t sel0 = g < 3 ? 0x05040302u : 0x07060302u, sel1 = g < 3 ? 0x05040302u : 0x03020706u;
  const uint32_t m1 = g < 3 ? ~0u : 0xFFFFu, c1 = g < 3 ? 0u : 0x3F800000u, m2 = g < 3 ? ~0u : 0u, c2 = g < 3 ? 0u : 0x3F803F80u;

  // per-slot state (reloaded when the slot changes)
  int cur = -1;
  bf16x8 w1t[F32 && !X3 ? 3 : 1][2];                 // layer-1 weights, FP32 arithmetic: [term][channel tile]
  bf16x8 w2b[P == C4_BF16 ? 9 : 1][2][2];            // [tap][channel half of the tap][32-channel tile]
  bf16x8 w2x[X3 ? 9 : 1][2][2];                      // three-product tier: [tap][term][the wave's channel tile]
  i32x8 w2q[P == C4_FP8 ? 3 : 1][P == C4_FP8 ? 4 : 1];
  float inv_s1 = 1.f, inv_s2 = 1.f;
  // layer 2: this wave's output row of the band and first channel
  const int lrow = wave & 3, lch = (wave >> 2) * C::CW;

  for (int t = blockIdx.x; t < total; t += gridDim.x) {
    int slot = 0, off = t / segs, ebase = 0;
    const int b0 = (t % segs) * seg_nb, bs = max(b0 - 1, 0);     // first band, first band run
    for (int i = 0; i < a.n_preds; ++i) {
      const int c = a.c4[i] ? a.q.counts[a.pred[i]] : 0;
      if (off < c) { slot = i; break; }
      off -= c;
      ebase += a.q.counts[a.pred[i]];
    }
    const int k = a.pred[slot];
    const int64_t ent = (int64_t)ebase + off;
    if (ent >= a.act_cap) {   // cannot happen: a round holds at most act_cap evaluations
      if (tid == 0) atomicOr(&a.st->overflow, 1);
      continue;
    }
    const uint32_t idx = entry_idx(a.q.entries[(int64_t)k * a.q.cap + off]);
    if (slot != cur) {
      cur = slot;
      // (the previous frame's last barrier ordered every read of the previous slot's constants)
      if (tid < 64) consts_s[tid] = a.bias[slot][1][tid];
      else if (tid < 128)
        consts_s[tid] = P == C4_FP8 ? a.c4_wscale[slot][0][tid - 64] * a.c4_ascale[slot][0] : 1.f;
      if constexpr (F32 && !X3) {
        const bf16x8* w1 = static_cast<const bf16x8*>(a.c4_w1f[slot]);
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
          for (int ct = 0; ct < 2; ++ct) w1t[t][ct] = w1[(t * 2 + ct) * 64 + lane];
      } else {
        if (tid < W1N * 64) w1_s[tid >> 6][tid & 63] = static_cast<const bf16x8*>(X3 ? a.c4_w1f[slot] : a.c4_w1b[slot])[tid];
      }
      if constexpr (P == C4_BF16) {
        const bf16x8* w2 = static_cast<const bf16x8*>(a.c4_w2[slot][C4_BF16]);
#pragma unroll
        for (int tp = 0; tp < 9; ++tp)
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int c2 = 0; c2 < 2; ++c2) w2b[tp][h][c2] = w2[((tp * 2 + h) * 2 + c2) * 64 + lane];
      }
      if constexpr (X3) {
        const bf16x8* w2 = static_cast<const bf16x8*>(a.c4_w2[slot][C4_S3]);
#pragma unroll
        for (int tp = 0; tp < 9; ++tp)
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int c = 0; c < 2; ++c) w2x[tp][u][c] = w2[((tp * 4 + lch / 16 + c) * 3 + u) * 64 + lane];
      }
      if constexpr (P == C4_FP8) {
        const i32x8* w2 = static_cast<const i32x8*>(a.c4_w2[slot][C4_FP8]);
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
          for (int ct = 0; ct < 4; ++ct) w2q[s][ct] = w2[(s * 4 + ct) * 64 + lane];
        inv_s1 = 1.f / a.c4_ascale[slot][0];
        inv_s2 = 1.f / a.c4_ascale[slot][1];
      }
    }
    const unsigned long long t0 = wall_clock64();
    const unsigned char* frame = static_cast<const unsigned char*>(a.fr.base) + (int64_t)idx * a.fr.elems * (U8 ? 1 : 2);
    // the work item after this one (its first band is prefetched during this frame's last band)
    const unsigned char* next_frame = nullptr;
    uint32_t nidx = 0;
    int nbs = 0;
    {
      const int t2 = t + gridDim.x;
      if (t2 < total) {
        int off2 = t2 / segs, eb2 = 0, s2 = -1;
        nbs = max((t2 % segs) * seg_nb - 1, 0);
        for (int i = 0; i < a.n_preds; ++i) {
          const int c = a.c4[i] ? a.q.counts[a.pred[i]] : 0;
          if (off2 < c) { s2 = i; break; }
          off2 -= c;
          eb2 += a.q.counts[a.pred[i]];
        }
        if (s2 >= 0 && (int64_t)eb2 + off2 < a.act_cap) {
          nidx = entry_idx(a.q.entries[(int64_t)a.pred[s2] * a.q.cap + off2]);
          next_frame = static_cast<const unsigned char*>(a.fr.base) + (int64_t)nidx * a.fr.elems * (U8 ? 1 : 2);
        }
      }
    }
    if (!(pf_valid && pf_idx == idx && pf_band == bs)) C4_FISSUE(frame, bs);
    C4_FCOMMIT(bs);
    pf_valid = false;
    unsigned char* out2 = static_cast<unsigned char*>(a.c4_act2) + ent * (32 * 32 * 64 * ES);
    unsigned* amax1 = a.c4_act_max ? a.c4_act_max + k * 4 + 0 : nullptr;
    unsigned* amax2 = a.c4_act_max ? a.c4_act_max + k * 4 + 1 : nullptr;

    const int be = b0 + seg_nb;
    for (int b = bs; b < be; ++b) {
      {
        // next band of this frame, or the first band of the next work item (this frame again when
        // there is none: a load whose data is not used); in flight over this band's layers 1 and 2
        const unsigned char* src = b + 1 < be ? frame : next_frame != nullptr ? next_frame : frame;
        C4_FISSUE(src, b + 1 < be ? b + 1 : nbs);
        if (b + 1 == be && next_frame != nullptr) {
          pf_valid = true;
          pf_idx = nidx;
          pf_band = nbs;
        }
      }
      // the ring slot of layer-1 row -1 is zero for the first band
      const int base_slot = (8 * b) % F_RING;   // ring index of layer-1 row 8b - 1
      if (b == 0)
        for (int q = tid; q < RR::BYTES / 4; q += NTHR) reinterpret_cast<uint32_t*>(ring)[q] = 0u;
      __syncthreads();

      // ---- layer 1: the wave's rows (local i = L1R w ..), four tiles of 16 columns each
#pragma unroll
      for (int ir = 0; ir < L1R; ++ir) {
        const int ridx = (base_slot + 1 + L1R * wave + ir) % F_RING;
        unsigned char* drow = ring + ridx * RR::BYTES + ((l16 & 1) ? RR::ODD + ((l16 + 1) >> 1) * PITCH : (l16 >> 1) * PITCH) +
                              4 * g * (F32 ? 2 : ES);
        bf16x8 wf[W1N];
        if constexpr (!F32 || X3)
#pragma unroll
          for (int i = 0; i < W1N; ++i) wf[i] = w1_s[i][lane];
        float m = 0.f;
#pragma unroll
        for (int jt = 0; jt < 4; ++jt) {
          uint32_t d[5];
#pragma unroll
          for (int i = 0; i < 5; ++i) d[i] = gp[i][2 * ir * RP + 48 * jt];
          uint32_t xw[4];
          xw[0] = __builtin_amdgcn_perm(d[1], d[0], sel0);
          xw[1] = (__builtin_amdgcn_perm(d[2], d[1], sel1) & m1) | c1;
          xw[2] = (__builtin_amdgcn_alignbit(d[3], d[2], 16) & m2) | c2;
          xw[3] = __builtin_amdgcn_alignbit(d[4], d[3], 16) & m2;
          bf16x8 xb;
          __builtin_memcpy(&xb, xw, sizeof(xb));
#pragma unroll
          for (int ct = 0; ct < 2; ++ct) {
            floatx4 acc = {0.f, 0.f, 0.f, 0.f};
            // FP32 arithmetic: raw frame values are exact in bf16 and the weights are the sum of their
            // three terms: every product exact, fp32 sums (smallest term first); X3 drops the lowest
            if constexpr (X3) {
              acc = c4_mfma(wf[2 + ct], xb, acc);
              acc = c4_mfma(wf[ct], xb, acc);
            } else if constexpr (F32) {
              acc = c4_mfma(w1t[2][ct], xb, acc);
              acc = c4_mfma(w1t[1][ct], xb, acc);
              acc = c4_mfma(w1t[0][ct], xb, acc);
            } else {
              acc = c4_mfma(wf[ct], xb, acc);
            }
            float v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = fmaxf(acc[r], 0.f);
            unsigned char* dst = drow + 8 * jt * PITCH + ct * 16 * (F32 ? 2 : ES);
            if constexpr (F32) {
              if (!X3 && amax1 != nullptr) m = fmaxf(m, fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])));
              store_planes<PLANES>(dst, 64, v);
            } else {
              if constexpr (P == C4_FP8)
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] *= inv_s1;
              c4_store4<P>(dst, v[0], v[1], v[2], v[3]);
            }
          }
        }
        if constexpr (F32 && !X3) c4_track_max(amax1, m);
      }
      __syncthreads();
      if (b >= b0) {             // (the band before a segment: layer 1 only)
      // ---- layer 2: output row 4b + lrow, columns 0..31 (two position tiles), channels lch ..; the sums
      // start from the bias
      floatx4 acc[F32 ? 2 : P == C4_FP8 ? 4 : 1][2];
      floatx16 acc32[P == C4_BF16 ? 2 : 1];
      if constexpr (P == C4_BF16) {
#pragma unroll
        for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
          for (int vq = 0; vq < 4; ++vq) {
            const float4 bb = *reinterpret_cast<const float4*>(consts_s + c2 * 32 + 8 * vq + 4 * (lane >> 5));
            acc32[c2][4 * vq] = bb.x; acc32[c2][4 * vq + 1] = bb.y; acc32[c2][4 * vq + 2] = bb.z; acc32[c2][4 * vq + 3] = bb.w;
          }
      } else if constexpr (F32) {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int mt = 0; mt < 2; ++mt) acc[c][mt] = *reinterpret_cast<const floatx4*>(consts_s + lch + 16 * c + 4 * g);
      } else {
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
          for (int mt = 0; mt < 2; ++mt) acc[ct][mt] = (floatx4){0.f, 0.f, 0.f, 0.f};
      }
      // ring row of layer-1 row 8b + 2w + u - 1 is (base_slot + 2w + u) mod 9
      if constexpr (P == C4_FP8) {
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          int tp = 4 * s + g;
          tp = tp > 8 ? 8 : tp;       // taps 9..11: zero weights
          const int u = tp / 3, v = tp % 3;
          const int rr = (base_slot + 2 * lrow + u) % F_RING;
          i32x8 xb[2];
#pragma unroll
          for (int mt = 0; mt < 2; ++mt) {
            const int j = mt * 16 + l16;
            const uint4* src = reinterpret_cast<const uint4*>(ring + rr * RR::BYTES + j * PITCH + (v == 1 ? 0 : RR::ODD + (v >> 1) * PITCH));
            const uint4 lo = src[0], hi = src[1];
            xb[mt] = (i32x8){(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
          }
#pragma unroll
          for (int ct = 0; ct < 4; ++ct)
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) acc[ct][mt] = c4_mfma(w2q[s][ct], xb[mt], acc[ct][mt]);
        }
      } else if constexpr (P == C4_BF16) {
        // the wave's 32 positions (lane % 32) x two 32-channel tiles; k-step (tap, h): channels
        // 16h .. 16h + 15 of the tap, lane half lane / 32 taking 8 of them
        const int j = lane & 31, hg = lane >> 5;
#pragma unroll
        for (int tp = 0; tp < 9; ++tp) {
          const int u = tp / 3, v = tp % 3;
          const int rr = (base_slot + 2 * lrow + u) % F_RING;
          const unsigned char* src = ring + rr * RR::BYTES + j * PITCH + (v == 1 ? 0 : RR::ODD + (v >> 1) * PITCH) + 16 * hg;
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const bf16x8 xb = *reinterpret_cast<const bf16x8*>(src + 32 * h);
            acc32[0] = c4_mfma32(w2b[tp][h][0], xb, acc32[0]);
            acc32[1] = c4_mfma32(w2b[tp][h][1], xb, acc32[1]);
          }
          // keep each tap's fragment reads next to its MFMAs (hoisting them all spills registers)
          if (tp & 1) __builtin_amdgcn_sched_barrier(0);
        }
      } else {
        // FP32 arithmetic from bf16 MFMAs: per tap, lane group g takes input channels 8g..8g+7
        // (one 16x16x32 k-step) of the ring's planes, multiplied with the three-term weights
        // ([tap][ct][term][lane]; X3 holds its two terms in registers, the three terms are read from
        // L2); the six products down to 2^-24 relative (X3: the three leading ones) are summed,
        // smallest first
        const bf16x8* w2 = static_cast<const bf16x8*>(a.c4_w2[slot][C4_S3]);
#pragma unroll
        for (int tp = 0; tp < 9; ++tp) {
          const int u = tp / 3, v = tp % 3;
          const int rr = (base_slot + 2 * lrow + u) % F_RING;
          bf16x8 xs[2][3];
#pragma unroll
          for (int mt = 0; mt < 2; ++mt) {
            const int j = mt * 16 + l16;
            const unsigned char* src = ring + rr * RR::BYTES + j * PITCH + (v == 1 ? 0 : RR::ODD + (v >> 1) * PITCH) + 16 * g;
#pragma unroll
            for (int pl = 0; pl < PLANES; ++pl) xs[mt][pl] = *reinterpret_cast<const bf16x8*>(src + 64 * pl);
          }
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            if constexpr (X3) {
#pragma unroll
              for (int mt = 0; mt < 2; ++mt) {
                acc[c][mt] = c4_mfma(w2x[tp][0][c], xs[mt][1], acc[c][mt]);
                acc[c][mt] = c4_mfma(w2x[tp][1][c], xs[mt][0], acc[c][mt]);
                acc[c][mt] = c4_mfma(w2x[tp][0][c], xs[mt][0], acc[c][mt]);
              }
            } else {
              const int ct = lch / 16 + c;
              const bf16x8 w[3] = {w2[((tp * 4 + ct) * 3 + 0) * 64 + lane], w2[((tp * 4 + ct) * 3 + 1) * 64 + lane],
                                   w2[((tp * 4 + ct) * 3 + 2) * 64 + lane]};
#pragma unroll
              for (int mt = 0; mt < 2; ++mt) acc[c][mt] = mfma_s3(w, xs[mt], acc[c][mt]);
            }
          }
          if (X3 && (tp & 1)) __builtin_amdgcn_sched_barrier(0);   // (as above)
        }
      }
      // ReLU -> layer-2 activations of row 4b + lrow, staged through this wave's slice of the
      // (now free) frame band area so that the global stores are whole contiguous lines
      {
        const int orow = 4 * b + lrow;
        constexpr int TP = F_TPITCH<P>;
        unsigned char* tw = lds + wave * 32 * TP;
        float m = 0.f;
        // quads of 4 consecutive channels per lane: (position j, first channel c0 of the wave's, values)
#pragma unroll
        for (int qd = 0; qd < (F32 ? 4 : 8); ++qd) {
          int j, c0;
          float v[4];
          if constexpr (P == C4_BF16) {
            const int c2 = qd >> 2, vq = qd & 3;
            j = lane & 31;
            c0 = c2 * 32 + 8 * vq + 4 * (lane >> 5);
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = fmaxf(acc32[c2][4 * vq + r], 0.f);
          } else if constexpr (F32) {
            const int mt = qd >> 1, c = qd & 1;
            j = mt * 16 + l16;
            c0 = c * 16 + 4 * g;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = fmaxf(acc[c][mt][r], 0.f);
            if (!X3 && amax2 != nullptr) m = fmaxf(m, fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])));
          } else {
            const int mt = qd >> 2, ct = qd & 3;
            j = mt * 16 + l16;
            c0 = ct * 16 + 4 * g;
            const float4 bb = *reinterpret_cast<const float4*>(consts_s + c0);
            const float4 ss = *reinterpret_cast<const float4*>(consts_s + 64 + c0);
            const float bv[4] = {bb.x, bb.y, bb.z, bb.w}, sv[4] = {ss.x, ss.y, ss.z, ss.w};
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = fmaxf(acc[ct][mt][r] * sv[r] + bv[r], 0.f) * inv_s2;
          }
          if constexpr (X3) store_planes<2>(tw + j * TP + c0 * 2, 64, v);
          else c4_store4<P>(tw + j * TP + c0 * ES, v[0], v[1], v[2], v[3]);
        }
        if constexpr (F32 && !X3) c4_track_max(amax2, m);
        // the wave's 32 positions x its channels: whole runs of RB bytes, 16 bytes a lane
        constexpr int RB = C::CW * ES;
        unsigned char* dst = out2 + (int64_t)orow * 32 * (64 * ES) + lch * ES;
#pragma unroll
        for (int i = 0; i < RB / 32; ++i) {
          const int o = i * 1024 + lane * 16;
          *reinterpret_cast<u32x4*>(dst + (o / RB) * (64 * ES) + o % RB) =
              *reinterpret_cast<const u32x4*>(tw + (o / RB) * TP + o % RB);
        }
      }
      }
      __syncthreads();   // the next band restages the frame rows and overwrites ring rows
      if (b + 1 < be) C4_FCOMMIT(b + 1);
    }
    if (tid == 0) ticks_s[k] += wall_clock64() - t0;
  }
  __syncthreads();
  if (tid < kMaxK && ticks_s[tid] && a.count_ticks) atomicAdd(&a.st->r_ticks[tid], ticks_s[tid]);
#undef C4_FISSUE
#undef C4_FCOMMIT
}

// ---------------------------------------------------------------- layers 3 and 4: implicit GEMM
// ROWB: bytes of one LDS tile row per k-block; UPR: 16-byte units per row; CE: elements per unit
template <int P> struct GemmCfg;
template <> struct GemmCfg<C4_FP8> { static constexpr int ROWB = 128, UPR = 8, CE = 16; };
// S3: B rows (fp32 activations) as FP32; A rows are three 64-byte bf16 rows (hi, mid, lo)
template <> struct GemmCfg<C4_S3> { static constexpr int ROWB = 128, UPR = 8, CE = 4; };

// chunk swizzle of tile row r: rows of 4 units xor (r/2) mod 4, rows of 8 units xor r mod 8
template <int UPR>
__host__ __device__ inline int c4_swz(int r) { return UPR == 4 ? ((r >> 1) & 3) : (r & 7); }

template <int P, int LAYER> struct GemmShape;
// LAYER 2 = the third conv (32x32x64 -> 16x16x128), LAYER 3 = the fourth (16x16x128 -> 8x8x256).
// Eight waves, each a 64 x 64 tile (4 x 4 MFMA tiles): layer 3 tiles one frame (256 positions) x
// all 128 channels, layer 4 two frames (128 positions) x all 256 channels (the head needs every
// channel of a frame in one workgroup).
template <int P> struct GemmShape<P, 2> {
  static constexpr int CIN = 64, COUT = 128, HIN = 32, HOUT = 16, BM = 256, BN = 128;
};
template <int P> struct GemmShape<P, 3> {
  static constexpr int CIN = 128, COUT = 256, HIN = 16, HOUT = 8, BM = 128, BN = 256;
};

// Output channel held by row R of the BF16 third-convolution weight image.  In a 16x16 MFMA
// tile, lane group g holds rows 4 g .. 4 g + 3 of the tile; with this order the four tiles of a
// wave's 64 channels give lane group g channels 8 g .. 8 g + 7 (tiles 0, 1) and 32 + 8 g .. + 7
// (tiles 2, 3), so each lane stores 16 contiguous bytes and a position's 64 channels are two
// 64-byte runs per store instruction.
__host__ __device__ inline int c4_l3_channel(int row) {
  const int blk = row / 64, w = row % 64, nt = w / 16, i = w % 16;
  return 64 * blk + (nt / 2) * 32 + 8 * (i / 4) + (nt % 2) * 4 + i % 4;
}

__host__ __device__ inline int c4_nkb(int prec, int layer) {
  const int cin = layer == 2 ? 64 : 128;
  const int bke = prec == C4_FP8 ? 128 : prec == C4_BF16 ? 64 : 32;   // S3: 32
  return (9 * cin + bke - 1) / bke;
}


// The k-block worked on as number i, of those that PER_TAP make up a tap.  The taps come by the parity
// of the pixels they read - (0,0) (0,2) (2,0) (2,2), (0,1) (2,1), (1,0) (1,2), (1,1) - so that a pixel's
// up to four reads follow each other and hit L2: in row order the 32 workgroups of an XCD come back to
// it a whole frame each later (4 MB), and layer 4 read every activation twice from memory.
template <int PER_TAP>
__device__ inline int c4_kblock(int i) {
  const int n = i / PER_TAP;
  return (int)(0x453718620ull >> (4 * n) & 15) * PER_TAP + (i - n * PER_TAP);
}

// Epilogue of one GEMM tile (acc: the 64 x 64 block of wave (wm, wn) of the tile).  Layer 3: bias +
// ReLU, stored as the next layer's activations.  Layer 4: bias + ReLU, mean over each frame's 64
// positions, this wave's share of the FC, then the margin and decision (or the logits).
// PERM: the tile's channels follow c4_l3_channel (BF16 third convolution).  X3: stored as two bf16 planes.
template <int P, int LAYER, bool PERM = false, bool X3 = false>
__device__ inline void c4_gemm_epilogue(const GcnnArgs& a, const Forward& f, const floatx4 (&acc)[4][4], int slot,
                                        int k, int cb, int ebase, int64_t row0, int64_t rows, const float* ep_bias,
                                        const float* ep_scale, const float* fcw_s, float (*zpart)[kClasses]) {
  typedef typename C4T<P>::T T;
  typedef GemmShape<P, LAYER> S;
  constexpr int COUT = S::COUT, HOUT = S::HOUT, PP = HOUT * HOUT, BM = S::BM, BN = S::BN, WM = 64, WN = 64;
  constexpr int MT = WM / 16, NT = WN / 16, WGM = BM / WM;
  constexpr bool HEAD = LAYER == 3;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, l16 = lane & 15;
  const int wm = wave % WGM, wn = wave / WGM;
  if constexpr (PERM) {
    static_assert(P == C4_BF16 && !HEAD, "permuted channels: BF16 third convolution");
    __bf16* out = reinterpret_cast<__bf16*>(a.c4_act3);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int64_t row = row0 + wm * WM + mt * 16 + l16;
      const bool valid = row < rows && ebase + row / PP < a.act_cap;
      const int64_t e = valid ? row / PP : 0;
      const int p = (int)(row % PP);
      __bf16* o = out + ((int64_t)ebase + e) * (PP * COUT) + (int64_t)p * COUT + cb * BN;
#pragma unroll
      for (int h = 0; h < 2; ++h) {              // tiles 2h, 2h + 1: channels 32 h + 8 g .. + 7
        const int cl = wn * WN + 32 * h + 8 * g;
        const floatx4 b0 = *reinterpret_cast<const floatx4*>(ep_bias + cl);
        const floatx4 b1 = *reinterpret_cast<const floatx4*>(ep_bias + cl + 4);
        alignas(16) __bf16 v[8];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          v[r] = static_cast<__bf16>(fmaxf(acc[2 * h][mt][r] + b0[r], 0.f));
          v[4 + r] = static_cast<__bf16>(fmaxf(acc[2 * h + 1][mt][r] + b1[r], 0.f));
        }
        if (valid) *reinterpret_cast<uint4*>(o + cl) = *reinterpret_cast<const uint4*>(v);
      }
    }
  } else if constexpr (!HEAD) {
    T* out = reinterpret_cast<T*>(a.c4_act3);
    const float inv_out = P == C4_FP8 ? 1.f / a.c4_ascale[slot][2] : 1.f;
    unsigned* amax = a.c4_act_max ? a.c4_act_max + k * 4 + 2 : nullptr;
    float m = 0.f;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int64_t row = row0 + wm * WM + mt * 16 + l16;
      const bool valid = row < rows && ebase + row / PP < a.act_cap;
      const int64_t e = valid ? row / PP : 0;
      const int p = (int)(row % PP);
      T* o = out + ((int64_t)ebase + e) * (PP * COUT) + (int64_t)p * COUT;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const int cl = wn * WN + nt * 16 + 4 * g;    // channel within the tile
        const int ch = cb * BN + cl;
        const floatx4 bb = *reinterpret_cast<const floatx4*>(ep_bias + cl);
        floatx4 sc = {1.f, 1.f, 1.f, 1.f};
        if constexpr (P == C4_FP8) sc = *reinterpret_cast<const floatx4*>(ep_scale + cl);
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float x = acc[nt][mt][r];
          if constexpr (P == C4_FP8) x *= sc[r];
          v[r] = fmaxf(x + bb[r], 0.f);
          m = fmaxf(m, valid ? v[r] : 0.f);
          v[r] *= inv_out;
        }
        if (valid) {
          if constexpr (X3) store_planes<2>(c4_plane_ptr(o, ch), 64, v);
          else c4_store4<P>(o + ch, v[0], v[1], v[2], v[3]);
        }
      }
    }
    if constexpr (P == C4_F32 || P == C4_S3) c4_track_max(amax, m);
  } else {
    // wave (wm, wn): frame wm of the tile, channels wn*WN .. +WN-1.  Pool over the frame's 64
    // positions, then this wave's share of FC.
    const int64_t frow = row0 + wm * WM;             // first row of the frame
    const bool fvalid = frow < rows;
    float zc = 0.f;                                   // lane l16 < 10: class l16
    const int cls = l16 < kClasses ? l16 : 0;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int chb = wn * WN + nt * 16 + 4 * g;
      const floatx4 bb = *reinterpret_cast<const floatx4*>(ep_bias + chb);
      floatx4 sc = {1.f, 1.f, 1.f, 1.f};
      if constexpr (P == C4_FP8) sc = *reinterpret_cast<const floatx4*>(ep_scale + chb);
      float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float x = acc[nt][mt][r];
          if constexpr (P == C4_FP8) x *= sc[r];
          s[r] += fmaxf(x + bb[r], 0.f);
        }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float gch = row_sum16(s[r]) * (1.f / PP);
        zc += gch * fcw_s[(chb + r) * kClasses + cls];
      }
    }
    if (l16 >= kClasses) zc = 0.f;
    // rows g = 0..3 hold different channel groups: add them
    zc = (__shfl(zc, l16) + __shfl(zc, 16 + l16)) + (__shfl(zc, 32 + l16) + __shfl(zc, 48 + l16));
    if (lane < kClasses) zpart[wave][lane] = zc;
    __syncthreads();
    if (wn == 0) {
      bool pass = false, defer = false, active = false;
      uint32_t e = 0;
      if (fvalid) {
        const int64_t ei = frow / PP;
        e = a.q.entries[(int64_t)k * a.q.cap + ei];
        if (lane == 0) {
          active = true;
          float z[kClasses];
#pragma unroll
          for (int c = 0; c < kClasses; ++c) {
            float sum = 0.f;
            for (int w2 = 0; w2 < BN / WN; ++w2) sum += zpart[wm + WGM * w2][c];
            z[c] = sum + a.fc_b[slot][c];
          }
          const uint32_t idx = entry_idx(e);
          if (f.logits != nullptr)
            for (int c = 0; c < kClasses; ++c) f.logits[(int64_t)idx * kClasses + c] = (double)z[c];
          const float d = class_margin(z, a.class_mask[slot]);
          const float th = theta_of(f, k, idx);
          pass = d > th;
          defer = f.defer.entries != nullptr && fabsf(d - th) < f.tau[k];
        }
      }
      if (f.logits == nullptr) forward_decision(f, k, e, active, defer, pass);
    }
  }
}

// Layers 3 and 4 of a launch that holds few frames (a re-score band, a late round, a small query),
// where the tiles above leave most CUs idle and one tile's time is the launch's: tiles of 64
// positions x 128 channels (layer 3 four per frame, layer 4 two), eight waves of 16 positions x 64
// channels, in a ring of four or five stages.  The products and the order in which they are added
// are the large tiles', and so is the pooling's and the head's, so a frame's logits do not depend on
// which tiles it took.  Layer 4: the two workgroups of a frame leave its pooled channels in the
// (now free) layer-2 activations with device-scope exchanges, each complete before its workgroup
// counts itself, and the second to arrive finishes the frame.
// A re-score band of some 20 frames through layers 3 + 4 in FP32: 50 + 86 -> 18 + 36 us.  A launch takes
// these tiles while its items fill the GPU at most C4_FEW times (layer 3 up to 128 frames, layer 4
// up to 256); beyond, the large tiles, which read each weight once per two or four frames, are ahead.
constexpr int C4_FEW = 2;
template <int P, int LAYER>
__device__ inline bool c4_is_few(const GcnnArgs& a) {
  typedef GemmShape<P, LAYER> S;
  int frames = 0;
  for (int i = 0; i < a.n_preds; ++i) frames += a.c4[i] ? a.q.counts[a.pred[i]] : 0;
  return (int64_t)frames * (S::HOUT * S::HOUT / 64) * (S::COUT / 128) <= (int64_t)C4_FEW * gridDim.x;
}

template <int P, int LAYER, bool X3, int LDS_BYTES>
__device__ inline void c4_few(const GcnnArgs& a, const Forward& f, unsigned char* lds, uint32_t lds0) {
  typedef typename C4T<P>::T T;
  typedef GemmShape<P, LAYER> S;
  constexpr bool S3 = P == C4_S3, HEAD = LAYER == 3;
  static_assert(S3 || P == C4_BF16, "tiers with few-frame tiles");
  constexpr int CIN = S::CIN, COUT = S::COUT, HIN = S::HIN, HOUT = S::HOUT, PP = HOUT * HOUT;
  constexpr int BM = 64, BN = 128, PT = PP / BM, CTL = COUT / BN;
  constexpr int TERMS = S3 ? (X3 ? 2 : 3) : 1, ROWA = S3 ? 64 : 128, UA = ROWA / 16;
  constexpr int CE = 16 / (int)sizeof(T), BKE = 128 / (int)sizeof(T), NKB = 9 * CIN / BKE;
  constexpr int AUNITS = TERMS * BN * UA, UNITS = AUNITS + BM * 8, NI = UNITS / 512, NIA = AUNITS / 512;
  constexpr int STAGE = UNITS * 16, NS = LDS_BYTES / STAGE < 5 ? LDS_BYTES / STAGE : 5;
  static_assert(UNITS % 512 == 0 && AUNITS % 512 == 0 && NI - NIA == 1, "eight waves fill a stage");
  static_assert(NS >= 3 && NKB >= NS && 2 * 4 * 16 * 64 * 4 <= LDS_BYTES, "ring");
  __shared__ float pool_s[256], zw_s[4][kClasses];
  __shared__ int last_s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, l16 = lane & 15;
  const int pg = wave & 3, cg = wave >> 2;
  int frames = 0;
  for (int i = 0; i < a.n_preds; ++i) frames += a.c4[i] ? a.q.counts[a.pred[i]] : 0;
  const T* act_in = reinterpret_cast<const T*>(LAYER == 2 ? a.c4_act2 : a.c4_act3);
  for (int t = blockIdx.x; t < frames * PT * CTL; t += gridDim.x) {
    const int fi = t / (PT * CTL), pt = t / CTL % PT, cb = t % CTL;
    int slot = 0, off = fi, ebase = 0;
    for (int i = 0; i < a.n_preds; ++i) {
      const int c = a.c4[i] ? a.q.counts[a.pred[i]] : 0;
      if (off < c) { slot = i; break; }
      off -= c;
      ebase += a.q.counts[a.pred[i]];
    }
    const int k = a.pred[slot];
    const int64_t ent = (int64_t)ebase + off;
    if (ent >= a.act_cap) continue;         // cannot happen (the front kernel reports it)
    const unsigned long long t0 = wall_clock64();
    const unsigned char* img = static_cast<const unsigned char*>(a.c4_img[slot][LAYER - 2][P]) + (size_t)cb * BN * ROWA;
    // the position row and chunk this lane gathers
    const int r = wave * 8 + (lane >> 3), p = pt * BM + r, oi = p / HOUT, oj = p % HOUT;
    const int chunk = ((lane & 7) ^ c4_swz<8>(r)) * CE;
    const T* bsrc = act_in + ent * (HIN * HIN * CIN);
    auto issue = [&](int n) {
      const uint32_t base = lds0 + (n % NS) * STAGE;
      const int kb = c4_kblock<NKB / 9>(n);
#pragma unroll
      for (int i = 0; i < NIA; ++i) {
        const int U = (wave + 8 * i) * 64 + lane;
        const unsigned char* src;
        if constexpr (S3) {
          const int term = U / (BN * 4), rr = U / 4 % BN;
          src = img + (size_t)kb * 3 * COUT * 64 + ((size_t)term * COUT + rr) * 64 + (U % 4) * 16;
        } else {
          src = img + (size_t)kb * COUT * 128 + (size_t)U * 16;
        }
        lds_dma16(src, __builtin_amdgcn_readfirstlane(base + (wave + 8 * i) * 1024));
      }
      const int ke = kb * BKE + chunk, tap = ke / CIN, ch = ke % CIN;
      const int y = 2 * oi + tap / 3 - 1, x = 2 * oj + tap % 3 - 1;
      const bool ok = y >= 0 && x >= 0;
      lds_dma16(ok ? static_cast<const void*>(bsrc + (y * HIN + x) * CIN + ch) : a.zero_page,
                __builtin_amdgcn_readfirstlane(base + (wave + 8 * NIA) * 1024));
    };
    floatx4 acc[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) acc[nt] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s0 = 0; s0 < NS - 1; ++s0) issue(s0);
#pragma unroll 1
    for (int kb = 0; kb < NKB; ++kb) {
      // this wave's copies of block kb have landed; those of later blocks may be in flight
      const int ahead = min(NS - 2, NKB - 1 - kb);
      if (NS >= 5 && ahead >= 3) wait_vmcnt<3 * NI>();
      else if (NS >= 4 && ahead >= 2) wait_vmcnt<2 * NI>();
      else if (ahead >= 1) wait_vmcnt<NI>();
      else wait_vmcnt<0>();
      __syncthreads();
      if (kb + NS - 1 < NKB) issue(kb + NS - 1);
      const unsigned char* A = lds + (kb % NS) * STAGE;
      const unsigned char* Bm = A + AUNITS * 16;
      const int rb = pg * 16 + l16;
      if constexpr (S3) {
        bf16x8 x[3];
        if constexpr (X3) {
          x[0] = *reinterpret_cast<const bf16x8*>(Bm + (rb * 8 + (g ^ c4_swz<8>(rb))) * 16);
          x[1] = *reinterpret_cast<const bf16x8*>(Bm + (rb * 8 + ((4 + g) ^ c4_swz<8>(rb))) * 16);
        } else {
          split3(*reinterpret_cast<const float4*>(Bm + (rb * 8 + ((2 * g) ^ c4_swz<8>(rb))) * 16),
                 *reinterpret_cast<const float4*>(Bm + (rb * 8 + ((2 * g + 1) ^ c4_swz<8>(rb))) * 16), x);
        }
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
          const int ra = cg * 64 + nt * 16 + l16;
          bf16x8 w[3];
#pragma unroll
          for (int u = 0; u < TERMS; ++u)
            w[u] = *reinterpret_cast<const bf16x8*>(A + ((u * BN + ra) * 4 + (g ^ c4_swz<4>(ra))) * 16);
          if constexpr (X3) {
            floatx4 c = c4_mfma(w[0], x[1], acc[nt]);
            c = c4_mfma(w[1], x[0], c);
            acc[nt] = c4_mfma(w[0], x[0], c);
          } else {
            acc[nt] += mfma_s3(w, x, (floatx4){0.f, 0.f, 0.f, 0.f});
          }
        }
      } else {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          const bf16x8 x = *reinterpret_cast<const bf16x8*>(Bm + (rb * 8 + ((4 * ks + g) ^ c4_swz<8>(rb))) * 16);
#pragma unroll
          for (int nt = 0; nt < 4; ++nt) {
            const int ra = cg * 64 + nt * 16 + l16;
            acc[nt] = c4_mfma(*reinterpret_cast<const bf16x8*>(A + (ra * 8 + ((4 * ks + g) ^ c4_swz<8>(ra))) * 16), x, acc[nt]);
          }
        }
      }
    }
    const float* bias = a.bias[slot][LAYER];
    if constexpr (!HEAD) {
      T* o = reinterpret_cast<T*>(a.c4_act3) + ent * (PP * COUT) + (int64_t)(pt * BM + pg * 16 + l16) * COUT;
      unsigned* amax = a.c4_act_max ? a.c4_act_max + k * 4 + 2 : nullptr;
      float m = 0.f;
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) {
        // (BF16: image rows in c4_l3_channel's order, four consecutive channels all the same)
        const int row = cb * BN + cg * 64 + nt * 16 + 4 * g, ch = S3 ? row : c4_l3_channel(row);
        const float4 bb = *reinterpret_cast<const float4*>(bias + ch);
        const float v0 = fmaxf(acc[nt][0] + bb.x, 0.f), v1 = fmaxf(acc[nt][1] + bb.y, 0.f);
        const float v2 = fmaxf(acc[nt][2] + bb.z, 0.f), v3 = fmaxf(acc[nt][3] + bb.w, 0.f);
        m = fmaxf(m, fmaxf(fmaxf(v0, v1), fmaxf(v2, v3)));
        const float v[4] = {v0, v1, v2, v3};
        if constexpr (X3) store_planes<2>(c4_plane_ptr(o, ch), 64, v);
        else c4_store4<P>(o + ch, v0, v1, v2, v3);
      }
      if constexpr (S3) c4_track_max(amax, m);
      __syncthreads();                 // the next item's first stages overwrite the ring
    } else {
      // bias + ReLU of every position, then per channel the sum over the frame's positions in
      // the large tile's order: lane l16's four positions, then the sixteen lanes
      __syncthreads();
      float* hs = reinterpret_cast<float*>(lds);           // [cg][pg][nt][r][lane]
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) {
        const float4 bb = *reinterpret_cast<const float4*>(bias + cb * BN + cg * 64 + nt * 16 + 4 * g);
        const float bv[4] = {bb.x, bb.y, bb.z, bb.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) hs[((wave * 4 + nt) * 4 + q) * 64 + lane] = fmaxf(acc[nt][q] + bv[q], 0.f);
      }
      __syncthreads();
      float mine = 0.f;                                    // wave (cg, pg): channel tile nt = pg
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float sum = 0.f;
#pragma unroll
        for (int m4 = 0; m4 < 4; ++m4) sum += hs[(((cg * 4 + m4) * 4 + pg) * 4 + q) * 64 + lane];
        sum = row_sum16(sum) * (1.f / PP);
        mine = l16 == q ? sum : mine;
      }
      float* pool = static_cast<float*>(a.c4_act2) + (int64_t)fi * COUT;
      if (l16 < 4) {
        const unsigned old = atomicExch(reinterpret_cast<unsigned*>(pool + cb * BN + cg * 64 + pg * 16 + 4 * g + l16),
                                        __float_as_uint(mine));
        asm volatile("" : : "v"(old));                     // wait for the exchange to be done
      }
      __syncthreads();
      if (tid == 0) {
        const int n = atomicAdd(&a.c4_few_cnt[fi], 1);
        last_s = n == CTL - 1;
        if (last_s) atomicExch(&a.c4_few_cnt[fi], 0);      // ready for the next launch
      }
      __syncthreads();
      if (last_s) {
        if (tid < COUT)
          pool_s[tid] = __hip_atomic_load(pool + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (wave < 4) {                                    // channels 64 wave .. + 63, as one wave of the large tile
          const int cls = l16 < kClasses ? l16 : 0;
          float zc = 0.f;
#pragma unroll
          for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int ch = wave * 64 + nt * 16 + 4 * g + q;
              zc += pool_s[ch] * a.fc_w[slot][ch * kClasses + cls];
            }
          if (l16 >= kClasses) zc = 0.f;
          zc = (__shfl(zc, l16) + __shfl(zc, 16 + l16)) + (__shfl(zc, 32 + l16) + __shfl(zc, 48 + l16));
          if (lane < kClasses) zw_s[wave][lane] = zc;
        }
        __syncthreads();
        if (wave == 0) {
          const uint32_t e = a.q.entries[(int64_t)k * a.q.cap + off];
          bool pass = false, defer = false;
          if (lane == 0) {
            float z[kClasses];
#pragma unroll
            for (int c = 0; c < kClasses; ++c) {
              float sum = 0.f;
              for (int w2 = 0; w2 < 4; ++w2) sum += zw_s[w2][c];
              z[c] = sum + a.fc_b[slot][c];
            }
            const uint32_t idx = entry_idx(e);
            if (f.logits != nullptr)
              for (int c = 0; c < kClasses; ++c) f.logits[(int64_t)idx * kClasses + c] = (double)z[c];
            const float d = class_margin(z, a.class_mask[slot]);
            const float th = theta_of(f, k, idx);
            pass = d > th;
            defer = f.defer.entries != nullptr && fabsf(d - th) < f.tau[k];
          }
          if (f.logits == nullptr) forward_decision(f, k, e, lane == 0, defer, pass);
        }
      }
      __syncthreads();                 // the next item reuses LDS
    }
    if (tid == 0 && a.count_ticks) atomicAdd(&a.st->r_ticks[k], (unsigned long long)(wall_clock64() - t0));
  }
}

// X3 (with P = C4_S3 only): the three-product arithmetic of the C4_X3 tier
template <int P, int LAYER, bool X3 = false>
__global__ __launch_bounds__(512) void c4_gemm_kernel(GcnnArgs a, Forward f) {
  typedef typename C4T<P>::T T;
  typedef GemmCfg<P> G;
  typedef GemmShape<P, LAYER> S;
  constexpr int ES = C4T<P>::ES, UPR = G::UPR, CE = G::CE, BKE = G::ROWB / ES;
  constexpr int CIN = S::CIN, COUT = S::COUT, HIN = S::HIN, HOUT = S::HOUT, PP = HOUT * HOUT;
  constexpr int BM = S::BM, BN = S::BN, WM = 64, WN = 64;
  constexpr int MT = WM / 16, NT = WN / 16;
  constexpr int WGM = BM / WM;                        // waves along M (8 waves in all)
  constexpr int NKB = (9 * CIN + BKE - 1) / BKE;
  constexpr bool S3 = P == C4_S3;
  constexpr int ATERMS = X3 ? 2 : 3;                  // weight terms staged (X3 reads hi and mid)
  constexpr int AUNITS = S3 ? ATERMS * BN * 4 : BN * UPR;   // A: S3 holds a 64-byte row per channel and term
  constexpr int UNITS = AUNITS + BM * UPR;            // 16-byte units of one stage
  constexpr int NI = UNITS / 64 / 8;                  // load instructions per wave and stage
  constexpr int NIA = AUNITS / 64 / 8;                // ... of them for A (the rest gather B)
  constexpr int STAGE = UNITS * 16;
  constexpr int NS = S3 && !X3 ? 2 : 3;               // stages in flight (what LDS holds)
  constexpr bool HEAD = LAYER == 3;
  static_assert(UNITS % 512 == 0 && AUNITS % 512 == 0, "stage rows must fill the waves' load units");
  static_assert(WGM * (BN / WN) == 8, "eight waves per tile");
  static_assert(!HEAD || (BN == COUT && WM == PP), "the head needs whole frames per wave and all channels");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[NS * STAGE];
  __shared__ float zpart[8][kClasses];
  // epilogue constants of the tile, staged before its k loop: bias and (FP8) weight scale x input
  // activation scale of its channels, and (last layer) the FC weights
  __shared__ __attribute__((aligned(16))) float ep_bias[BN];
  __shared__ __attribute__((aligned(16))) float ep_scale[P == C4_FP8 ? BN : 1];
  __shared__ float fcw_s[HEAD ? COUT * kClasses : 1];
  __shared__ unsigned long long ticks_s[kMaxK];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, l16 = lane & 15;
  const int wm = wave % WGM, wn = wave / WGM;
  if (tid < kMaxK) ticks_s[tid] = 0;
  const T* act_in = reinterpret_cast<const T*>(LAYER == 2 ? a.c4_act2 : a.c4_act3);
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds);
  if constexpr (S3) {
    if (c4_is_few<P, LAYER>(a)) {
      c4_few<P, LAYER, X3, NS * STAGE>(a, f, lds, lds0);
      return;
    }
  }
  // tiles: per slot ceil(count * PP / BM) x COUT / BN
  int total = 0;
  for (int i = 0; i < a.n_preds; ++i)
    if (a.c4[i]) total += (int)(((int64_t)a.q.counts[a.pred[i]] * PP + BM - 1) / BM) * (COUT / BN);
  const int u_slot = lane % UPR;     // the LDS slot of every unit this lane loads

  for (int t = blockIdx.x; t < total; t += gridDim.x) {
    int slot = 0, off = t, ebase = 0;
    for (int i = 0; i < a.n_preds; ++i) {
      const int c = a.c4[i] ? (int)(((int64_t)a.q.counts[a.pred[i]] * PP + BM - 1) / BM) * (COUT / BN) : 0;
      if (off < c) { slot = i; break; }
      off -= c;
      ebase += a.q.counts[a.pred[i]];
    }
    const int k = a.pred[slot];
    const int cnt = a.q.counts[k];
    const int mt0 = off / (COUT / BN), cb = off % (COUT / BN);
    const int64_t row0 = (int64_t)mt0 * BM;           // first position row of the tile (slot-local)
    const int64_t rows = (int64_t)cnt * PP;
    const unsigned long long t0 = wall_clock64();
    const unsigned char* img = static_cast<const unsigned char*>(a.c4_img[slot][LAYER - 2][P]) +
                               (size_t)cb * BN * (S3 ? 64 : G::ROWB);
    // (the previous tile's closing barrier ordered every read of these)
    for (int i = tid; i < BN; i += 512) {
      ep_bias[i] = a.bias[slot][LAYER][cb * BN + i];
      if constexpr (P == C4_FP8) ep_scale[i] = a.c4_wscale[slot][LAYER - 1][cb * BN + i] * a.c4_ascale[slot][LAYER - 1];
    }
    if constexpr (HEAD)
      for (int i = tid; i < COUT * kClasses; i += 512) fcw_s[i] = a.fc_w[slot][i];

    // B rows this lane gathers: frame pointer, output position and chunk, per load instruction
    const T* bsrc[NI - NIA];
    int boi[NI - NIA], boj[NI - NIA], bch[NI - NIA];
#pragma unroll
    for (int i = NIA; i < NI; ++i) {
      const int U = (wave + 8 * i) * 64 + lane - AUNITS;
      const int rb = U / UPR;
      const int64_t row = row0 + rb;
      const bool valid = row < rows && ebase + row / PP < a.act_cap;
      const int64_t e = valid ? row / PP : 0;
      const int p = valid ? (int)(row % PP) : 0;
      bsrc[i - NIA] = act_in + ((int64_t)ebase + e) * (HIN * HIN * CIN);
      boi[i - NIA] = valid ? p / HOUT : -1000;        // invalid rows read the zero page
      boj[i - NIA] = p % HOUT;
      bch[i - NIA] = (u_slot ^ c4_swz<UPR>(rb)) * CE;  // element offset of the chunk in the k-block
    }
    // stage kb of A (packed image, a straight copy) and B (im2col gathers) into LDS buffer buf
    auto issue = [&](int n, int buf) {
      const uint32_t base = lds0 + buf * STAGE;
      const int kb = NKB % 9 == 0 ? c4_kblock<NKB % 9 == 0 ? NKB / 9 : 1>(n) : n;   // (FP8 layer 3: blocks of two taps)
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int q = wave + 8 * i;
        const void* src;
        if (i < NIA) {
          // S3 image: [kb][term][oc][64 bytes], the tile's channels of each term contiguous
          if constexpr (S3) {
            const int U = q * 64 + lane, term = U / (BN * 4), r = (U / 4) % BN;
            src = img + (size_t)kb * 3 * COUT * 64 + ((size_t)term * COUT + r) * 64 + (U % 4) * 16;
          } else {
            src = img + (size_t)kb * COUT * G::ROWB + (size_t)(q * 64 + lane) * 16;
          }
        } else {
          const int ke = kb * BKE + bch[i - NIA];
          const int tap = ke / CIN, ch = ke % CIN;
          const int y = 2 * boi[i - NIA] + tap / 3 - 1, x = 2 * boj[i - NIA] + tap % 3 - 1;
          const bool ok = tap < 9 && y >= 0 && x >= 0 && y < HIN && x < HIN;
          src = ok ? static_cast<const void*>(bsrc[i - NIA] + (y * HIN + x) * CIN + ch) : a.zero_page;
        }
        lds_dma16(src, __builtin_amdgcn_readfirstlane(base + q * 1024));
      }
    };

    floatx4 acc[NT][MT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = (floatx4){0.f, 0.f, 0.f, 0.f};

    auto compute = [&](int buf) {
      const unsigned char* A = lds + buf * STAGE;
      const unsigned char* B = A + AUNITS * 16;
      if constexpr (S3) {
        // one 32-deep k-step: lane group g takes k = 8 g .. 8 g + 7 (A chunk g of each 64-byte
        // row, B chunks 2 g and 2 g + 1 of each 128-byte fp32 row); the fp32 activations are
        // split a = hi + mid + lo in bf16 and the six products down to 2^-24 relative are summed,
        // smallest first, by themselves and then added, so that the running sum is rounded once a step
        // (rms error of four CNNs' logits 0.74 to 0.94 of six roundings', FP32 logits 2 to 4 % longer; X3:
        // the previous layer has stored hi and mid, three products)
        bf16x8 aw[3][NT];
#pragma unroll
        for (int term = 0; term < ATERMS; ++term)
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            const int r = wn * WN + nt * 16 + l16;
            aw[term][nt] = *reinterpret_cast<const bf16x8*>(A + ((term * BN + r) * 4 + (g ^ c4_swz<4>(r))) * 16);
          }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const int r = wm * WM + mt * 16 + l16;
          bf16x8 x[3];
          if constexpr (X3) {       // stored as planes: chunks 0..3 of the row hi, 4..7 mid
            x[0] = *reinterpret_cast<const bf16x8*>(B + (r * UPR + (g ^ c4_swz<UPR>(r))) * 16);
            x[1] = *reinterpret_cast<const bf16x8*>(B + (r * UPR + ((4 + g) ^ c4_swz<UPR>(r))) * 16);
          } else {
            split3(*reinterpret_cast<const float4*>(B + (r * UPR + ((2 * g) ^ c4_swz<UPR>(r))) * 16),
                   *reinterpret_cast<const float4*>(B + (r * UPR + ((2 * g + 1) ^ c4_swz<UPR>(r))) * 16), x);
          }
#pragma unroll
          for (int nt = 0; nt < NT; ++nt) {
            if constexpr (X3) {         // hi x hi + hi x mid + mid x hi (about 2^-16 relative)
              floatx4 c = c4_mfma(aw[0][nt], x[1], acc[nt][mt]);
              c = c4_mfma(aw[1][nt], x[0], c);
              acc[nt][mt] = c4_mfma(aw[0][nt], x[0], c);
            } else {
              const bf16x8 w[3] = {aw[0][nt], aw[1][nt], aw[2][nt]};
              acc[nt][mt] += mfma_s3(w, x, (floatx4){0.f, 0.f, 0.f, 0.f});
            }
          }
        }
      } else {
        static_assert(P == C4_FP8, "BF16 has a kernel of its own");
        i32x8 af[NT], bfr[MT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const int r = wn * WN + nt * 16 + l16;
          const uint4 lo = *reinterpret_cast<const uint4*>(A + (r * UPR + ((2 * g) ^ c4_swz<UPR>(r))) * 16);
          const uint4 hi = *reinterpret_cast<const uint4*>(A + (r * UPR + ((2 * g + 1) ^ c4_swz<UPR>(r))) * 16);
          af[nt] = (i32x8){(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const int r = wm * WM + mt * 16 + l16;
          const uint4 lo = *reinterpret_cast<const uint4*>(B + (r * UPR + ((2 * g) ^ c4_swz<UPR>(r))) * 16);
          const uint4 hi = *reinterpret_cast<const uint4*>(B + (r * UPR + ((2 * g + 1) ^ c4_swz<UPR>(r))) * 16);
          bfr[mt] = (i32x8){(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = c4_mfma(af[nt], bfr[mt], acc[nt][mt]);
      }
    };

    // NS-stage ring, one barrier per k-block: block kb + NS - 1 is loaded while block kb is read.
    // The wait before the barrier covers this wave's loads of block kb (the blocks issued after
    // it may stay in flight); the barrier then covers every wave's.
#pragma unroll
    for (int s0 = 0; s0 < NS - 1; ++s0)
      if (s0 < NKB) issue(s0, s0);
#pragma unroll 1
    for (int kb = 0; kb < NKB; ++kb) {
      const int ahead = min(NS - 2, NKB - 1 - kb);
      if (NS >= 4 && ahead >= 2) wait_vmcnt<2 * NI>();
      else if (NS >= 3 && ahead >= 1) wait_vmcnt<NI>();
      else wait_vmcnt<0>();
      __syncthreads();
      if (kb + NS - 1 < NKB) issue(kb + NS - 1, (kb + NS - 1) % NS);
      compute(kb % NS);
    }

    c4_gemm_epilogue<P, LAYER, false, X3>(a, f, acc, slot, k, cb, ebase, row0, rows, ep_bias, ep_scale, fcw_s, zpart);
    if (tid == 0) ticks_s[k] += wall_clock64() - t0;
    __syncthreads();   // the next tile's prologue rewrites LDS (stages, constants, zpart)
  }
  if (tid < kMaxK && ticks_s[tid] && a.count_ticks) atomicAdd(&a.st->r_ticks[tid], ticks_s[tid]);
}

// BF16 layers 3 and 4 (the first pass): the implicit GEMM of c4_gemm_kernel with its pipeline
// restructured so that the matrix cores are not left waiting on LDS or memory latency:
//  - one stream of k-blocks over all of a workgroup's tiles: the first stages of the next tile are
//    loaded during the current tile's last k-blocks and its epilogue, and nothing a tile does on its
//    way waits for a load (queue offsets are kept in LDS, biases and FC weights are reloaded when the
//    predicate changes; a wave's loads complete in issue order, so any such wait would drain the ring);
//  - both operands come in by buffer loads to LDS: a lane's offset within a tile is the same for every
//    tile and the tap is a scalar offset, so a load costs one or two vector instructions, and padding is
//    an offset past the end, which reads zero;
//  - each k-block's fragments are read into registers one MFMA step ahead (two register sets), and
//    the barrier that publishes the next k-block and frees the oldest buffer sits between two
//    MFMA steps; the reads of the next step and the loads are dealt out between the MFMAs, and a tile's
//    stores are not waited for before two k-blocks of the next.
// Layer 3 moves 196 KB per frame between memory and the CU and 442 KB from L2 into LDS, layer 4 65 and
// 295 KB: 8,192 frames 450 -> 384 us (805 TFLOP/s) and 300 -> 284 us (1,088); with every activation in
// L2 they take 312 and 263, with no loads at all 260 and 206 us: what is left is memory latency that
// LDS has no room to cover.
// The arithmetic (operands, products and the order in which they are added) is the generic
// kernel's.
// Epilogue of a four-frame layer-4 tile: wave (wm, wn) holds frames 2 wm and 2 wm + 1 of the tile
// (rows 64 h .. 64 h + 63 of its 128, h = 0, 1) x channels 64 wn .. 64 wn + 63.  Bias + ReLU, mean
// over each frame's 64 positions, this wave's share of the FC; then per frame the sum over the
// four channel quarters, margin and decision (or the logits).  Same arithmetic, in the same
// order, as the two-frame epilogue of c4_gemm_epilogue.
__device__ inline void c4_head4_epilogue(const GcnnArgs& a, const Forward& f, const floatx4 (&acc)[4][8], int slot,
                                         int k, int64_t row0, int64_t rows, const float* ep_bias, const float* fcw_s,
                                         float (*zp)[2][kClasses]) {
  constexpr int PP = 64, WN = 64, NT = 4, WGM = 2, NWN = 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, l16 = lane & 15;
  const int wm = wave % WGM, wn = wave / WGM;
  const int cls = l16 < kClasses ? l16 : 0;
  float zc[2] = {0.f, 0.f};                         // lane l16 < 10: class l16 of frame h
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int chb = wn * WN + nt * 16 + 4 * g;
    const floatx4 bb = *reinterpret_cast<const floatx4*>(ep_bias + chb);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float s4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int mt = 4 * h; mt < 4 * h + 4; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) s4[r] += fmaxf(acc[nt][mt][r] + bb[r], 0.f);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float gch = row_sum16(s4[r]) * (1.f / PP);
        zc[h] += gch * fcw_s[(chb + r) * kClasses + cls];
      }
    }
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    float z = l16 < kClasses ? zc[h] : 0.f;
    // rows g = 0..3 hold different channel groups: add them
    z = (__shfl(z, l16) + __shfl(z, 16 + l16)) + (__shfl(z, 32 + l16) + __shfl(z, 48 + l16));
    if (lane < kClasses) zp[wave][h][lane] = z;
  }
  __syncthreads();
  if (wn == 0) {
    // lane h < 2: frame 2 wm + h of the tile
    const int h = lane & 1;
    const int64_t frow = row0 + (int64_t)(2 * wm + h) * PP;
    bool pass = false, defer = false, active = false;
    uint32_t e = 0;
    if (lane < 2 && frow < rows) {
      e = a.q.entries[(int64_t)k * a.q.cap + frow / PP];
      active = true;
      float z[kClasses];
#pragma unroll
      for (int c = 0; c < kClasses; ++c) {
        float sum = 0.f;
        for (int w2 = 0; w2 < NWN; ++w2) sum += zp[wm + WGM * w2][h][c];
        z[c] = sum + a.fc_b[slot][c];
      }
      const uint32_t idx = entry_idx(e);
      if (f.logits != nullptr)
        for (int c = 0; c < kClasses; ++c) f.logits[(int64_t)idx * kClasses + c] = (double)z[c];
      const float d = class_margin(z, a.class_mask[slot]);
      const float th = theta_of(f, k, idx);
      pass = d > th;
      defer = f.defer.entries != nullptr && fabsf(d - th) < f.tau[k];
    }
    if (f.logits == nullptr) forward_decision(f, k, e, active, defer, pass);
  }
}

template <int LAYER>
__global__ __launch_bounds__(512) void c4_gemm_bf16_kernel(GcnnArgs a, Forward f) {
  constexpr int P = C4_BF16;
  typedef __bf16 T;
  typedef GemmCfg<P> G;
  typedef GemmShape<P, LAYER> S;
  constexpr int CIN = S::CIN, COUT = S::COUT, HIN = S::HIN, HOUT = S::HOUT, PP = HOUT * HOUT;
  // layer 3: one frame per tile (a wave: 64 positions x 64 channels), three 48 KB stages of 64 k;
  // layer 4: four frames per tile (a wave: two frames x 64 channels), so the weight image is read once
  // per four frames, in four 32 KB stages of 32 k (two of 64 k left the loads one k-block to arrive)
  constexpr bool HEAD = LAYER == 3;
  constexpr int BM = HEAD ? 4 * PP : S::BM, BN = S::BN, WM = HEAD ? 2 * PP : 64, WN = 64, FPT = BM / PP;
  constexpr int MT = WM / 16, NT = WN / 16, WGM = BM / WM;
  constexpr int ROWB = HEAD ? 64 : 128, UPR = ROWB / 16, KS = ROWB / 64;   // MFMA steps per k-block
  constexpr int NKB = 9 * CIN * 2 / ROWB;
  constexpr int AUNITS = BN * UPR, UNITS = AUNITS + BM * UPR, NI = UNITS / 512, NIA = AUNITS / 512, NB = NI - NIA;
  constexpr int STAGE = UNITS * 16, NS = HEAD ? 4 : 3;
  // layer 3: loads of a k-block issued in the following one's first step, stores of a tile's epilogue
  constexpr int LH = NI / 2, ST = MT * NT * 4 * 2 / 16;
  constexpr uint32_t SHIFT = (HIN + 1) * CIN * 2;        // bytes from a frame's position (-1, -1) to (0, 0)
  constexpr uint32_t FRAME_B = HIN * HIN * CIN * 2, OOB = 0x80000000u;
  static_assert(9 * CIN * 2 % ROWB == 0 && CIN * 2 % ROWB == 0 && NKB >= NS, "whole k-blocks of one tap each");
  static_assert(UNITS % 512 == 0 && AUNITS % 512 == 0 && WGM * (BN / WN) == 8 && BN == COUT, "tile layout");
  static_assert(!HEAD || (MT == 8 && NT == 4), "layer 4: whole frames");
  static_assert(FPT * FRAME_B + SHIFT < OOB, "a masked offset is past the end");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[NS * STAGE];
  __shared__ float zpart[8][2][kClasses];
  __shared__ __attribute__((aligned(16))) float ep_bias[BN];
  __shared__ float fcw_s[HEAD ? COUT * kClasses : 1];
  __shared__ unsigned long long ticks_s[kMaxK];
  __shared__ int tile_s[kMaxK + 1], base_s[kMaxK], cnt_s[kMaxK];   // per slot: first tile, first act frame, frames
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, l16 = lane & 15;
  const int wm = wave % WGM, wn = wave / WGM;
  if (tid < kMaxK) ticks_s[tid] = 0;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds);
  if (c4_is_few<P, LAYER>(a)) {
    c4_few<P, LAYER, false, NS * STAGE>(a, f, lds, lds0);
    return;
  }
  if (tid == 0) {
    int tiles = 0, frames = 0;
    for (int i = 0; i < a.n_preds; ++i) {
      const int c = a.q.counts[a.pred[i]];
      tile_s[i] = tiles;
      base_s[i] = frames;
      cnt_s[i] = c;
      if (a.c4[i]) tiles += (c + FPT - 1) / FPT;
      frames += c;
    }
    tile_s[a.n_preds] = tiles;
  }
  __syncthreads();
  const int n_slots = a.n_preds;
  const int total = __builtin_amdgcn_readfirstlane(tile_s[n_slots]);
  // slot of tile t, searched from an earlier tile's
  auto slot_of = [&](int t, int slot) {
    while (t >= tile_s[slot + 1]) ++slot;
    return __builtin_amdgcn_readfirstlane(slot);
  };

  // ---- issue side
  // weights: the packed image is the LDS image of rows of 128 bytes (chunk u of row r at slot
  // u ^ (r % 8)); rows of 64 bytes take half a row, chunk j at slot j ^ (r / 2 % 4)
  const int arow = tid / UPR, aslot = tid % UPR;
  const uint32_t va = ROWB == 128 ? tid * 16
                                  : arow * 128 + ((aslot ^ ((arow >> 1) & 3)) ^ (arow & 7)) * 16;
  // activations: row (output position) rb of the tile, chunk of the slot, at tap (0, 0), from the
  // tile's first position less SHIFT; flag bits per load: output row 0 (tap row 0 reads padding),
  // output column 0 (tap column 0 does).  A stride-2 3x3 convolution with HIN = 2 HOUT reads padding
  // nowhere else.
  uint32_t vb0[NB], flags = 0;
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int rb = (tid + 512 * i) / UPR, p = rb % PP, oi = p / HOUT, oj = p % HOUT;
    vb0[i] = (uint32_t)(((rb / PP) * HIN * HIN + 2 * oi * HIN + 2 * oj) * CIN * 2 + (tid % UPR ^ c4_swz<UPR>(rb)) * 16);
    flags |= ((oi == 0 ? 1u : 0u) | (oj == 0 ? 2u : 0u)) << (2 * i);
  }
  const unsigned char* act_in = reinterpret_cast<const unsigned char*>(LAYER == 2 ? a.c4_act2 : a.c4_act3);
  i32x4 ra, rb;
  uint32_t vb[NB];
  int it = blockIdx.x, islot = 0, ikb = 0;
  // the issue side's tile: its image, its rows (past the last tile, or frames past the queue or the
  // activation buffer: zeros)
  auto set_tile = [&]() {
    int valid = 0, frame0 = 0;
    if (it < total) {
      islot = slot_of(it, islot);
      const int first = (it - tile_s[islot]) * FPT;
      frame0 = __builtin_amdgcn_readfirstlane(base_s[islot] + first);
      valid = __builtin_amdgcn_readfirstlane(min(cnt_s[islot] - first, (int)a.act_cap - frame0));
    }
    ra = buffer_rsrc(a.c4_img[islot][LAYER - 2][P], 9 * CIN * 2 * COUT);
    rb = buffer_rsrc(act_in + (int64_t)frame0 * FRAME_B - SHIFT, FPT * FRAME_B + SHIFT);
#pragma unroll
    for (int i = 0; i < NB; ++i) vb[i] = (tid + 512 * i) / UPR / PP < valid ? vb0[i] : OOB;
  };
  // load i of the issue side's k-block into buffer buf
  auto issue = [&](int i, int buf) {
    const uint32_t dst = lds0 + buf * STAGE + wave * 1024 + i * 8192;
    const int kb = c4_kblock<NKB / 9>(ikb);
    if (i < NIA) {
      const uint32_t off = (ROWB == 128 ? kb : kb >> 1) * COUT * 128 + i * (512 / UPR) * 128;
      buf_lds_dma16(ra, ROWB == 128 ? va : va ^ ((kb & 1) * 64), off, dst);
    } else {
      const int tap = kb * (ROWB / 2) / CIN, dy = tap / 3, dx = tap - 3 * dy;
      const uint32_t bad = (dy == 0 ? 1u : 0u) | (dx == 0 ? 2u : 0u);
      buf_lds_dma16(rb, (flags >> (2 * (i - NIA))) & bad ? OOB : vb[i - NIA],
                    (uint32_t)((dy * HIN + dx) * CIN * 2 + kb * ROWB % (CIN * 2)), dst);
    }
  };
  auto advance = [&]() {
    if (++ikb == NKB) {
      ikb = 0;
      it += gridDim.x;
      set_tile();
    }
  };

  // ---- compute side
  struct Frag { bf16x8 v[NT + MT]; };              // channel tiles, position tiles
  // fragment i of MFMA step ks (k = 32 ks .. 32 ks + 31 of the k-block) of buffer buf: lane group g
  // reads chunk 4 ks + g of each row
  auto frag = [&](int buf, int ks, int i) {
    const unsigned char* A = lds + buf * STAGE + l16 * ROWB + ((4 * ks + g) ^ c4_swz<UPR>(l16)) * 16;
    return *reinterpret_cast<const bf16x8*>(i < NT ? A + (wn * WN + i * 16) * ROWB
                                                   : A + AUNITS * 16 + (wm * WM + (i - NT) * 16) * ROWB);
  };
  floatx4 acc[NT][MT];
  // One step: the MFMAs of F, the reads of the next step's fragments and the loads [l0, l1) of the
  // issue side's k-block, dealt out between them.  (Issued in front, they held every wave's MFMAs back
  // until the memory pipeline had taken the loads of all eight: half of the step.)
  auto step = [&](const Frag& F, Frag& N, int nbuf, int nks, int l0, int l1, int lbuf) {
    constexpr int MM = NT * MT, R = NT + MT, LEFT = MM - R;
    static_assert(LEFT > 0 && MM >= R, "a read behind each of the first MFMAs");
#pragma unroll
    for (int n = 0; n < MM; ++n) {
      acc[n / MT][n % MT] = c4_mfma(F.v[n / MT], F.v[NT + n % MT], acc[n / MT][n % MT]);
      if (n < R) N.v[n] = frag(nbuf, nks, n);
      else
#pragma unroll
        for (int l = l0; l < l1; ++l)
          if (n - R == (l - l0) * LEFT / (l1 - l0)) issue(l, lbuf);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  int t = blockIdx.x;
  if (t < total) {
    // past the last tile the weights of the last slot seen are loaded (nothing uses them)
    islot = slot_of(t, 0);
    set_tile();
    // prologue: the stream's first NS k-blocks
#pragma unroll
    for (int s0 = 0; s0 < NS; ++s0) {
#pragma unroll
      for (int l = 0; l < NI; ++l) issue(l, s0);
      advance();
    }
    wait_vmcnt<(NS - 1) * NI>();
    __syncthreads();
    Frag F[2];
#pragma unroll
    for (int i = 0; i < NT + MT; ++i) F[0].v[i] = frag(0, 0, i);
    int buf = 0, slot = islot, loaded = -1;        // buffer of the current k-block
    bool stored = false;                           // the previous tile's epilogue has stored its results
    (void)stored;
    unsigned long long t0 = wall_clock64();
    for (;;) {
      slot = slot_of(t, loaded < 0 ? 0 : slot);
      const int k = a.pred[slot];
      if (slot != loaded) {
        // epilogue constants of this predicate (the previous tile's closing barrier ordered every read)
        if (loaded >= 0) {
          const unsigned long long now = wall_clock64();
          if (tid == 0) ticks_s[a.pred[loaded]] += now - t0;
          t0 = now;
        }
        for (int i = tid; i < BN; i += 512) ep_bias[i] = a.bias[slot][LAYER][i];
        if constexpr (HEAD)
          for (int i = tid; i < COUT * kClasses; i += 512) fcw_s[i] = a.fc_w[slot][i];
        loaded = slot;
      }
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[nt][mt] = (floatx4){0.f, 0.f, 0.f, 0.f};
      // the step in front of which the next k-block is published (it was issued NS - 1 k-blocks ago,
      // the NS - 2 after it may stay in flight) and this one's buffer freed, whose fragments every wave
      // has read; nl loads of a k-block start to fill it.  extra: stores issued after that k-block's
      // loads, which a wait that let only loads through would wait for too.
      auto turn = [&](const Frag& G0, Frag& G1, int nl, bool extra) {
        __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): this step's fragments
        if (extra) wait_vmcnt<(NS - 2) * NI + (HEAD ? 0 : ST)>();
        else wait_vmcnt<(NS - 2) * NI>();
        __syncthreads();
        const int nbuf = buf + 1 == NS ? 0 : buf + 1;
        step(G0, G1, nbuf, 0, 0, nl, buf);             // (reads unused after the last tile)
        buf = nbuf;
      };
      if constexpr (KS == 1) {
        static_assert(KS == 2 || NKB % 2 == 0, "two k-blocks per trip: the register sets alternate");
#pragma unroll 1
        for (int kb = 0; kb < NKB; kb += 2) {
          turn(F[0], F[1], NI, false);
          advance();
          turn(F[1], F[0], NI, false);
          advance();
        }
      } else {
        // a k-block's loads are issued half in its turn and half in the next k-block's first step, but
        // all before the epilogue's stores
        step(F[0], F[1], buf, 1, 0, 0, 0);
        turn(F[1], F[0], NI - LH, stored);
#pragma unroll 1
        for (int kb = 1; kb < NKB; ++kb) {
          __builtin_amdgcn_s_waitcnt(0xC07F);
          step(F[0], F[1], buf, 1, NI - LH, NI, buf == 0 ? NS - 1 : buf - 1);
          advance();
          turn(F[1], F[0], NI - LH, stored && kb == 1);
        }
#pragma unroll
        for (int l = NI - LH; l < NI; ++l) issue(l, buf == 0 ? NS - 1 : buf - 1);
        advance();
        stored = base_s[slot] + (t - tile_s[slot]) < a.act_cap;
      }
      const int64_t row0 = (int64_t)(t - tile_s[slot]) * BM, rows = (int64_t)cnt_s[slot] * PP;
      if constexpr (HEAD)
        c4_head4_epilogue(a, f, acc, slot, k, row0, rows, ep_bias, fcw_s, zpart);
      else
        c4_gemm_epilogue<P, LAYER, true>(a, f, acc, slot, k, 0, base_s[slot], row0, rows, ep_bias, nullptr, fcw_s,
                                         zpart[0]);
      __syncthreads();                // epilogue constants and zpart are rewritten next
      t += gridDim.x;
      if (t >= total) break;
    }
    if (tid == 0) ticks_s[a.pred[slot]] += wall_clock64() - t0;
    wait_vmcnt<0>();                  // the loads issued past the last tile
  }
  __syncthreads();
  if (tid < kMaxK && ticks_s[tid] && a.count_ticks) atomicAdd(&a.st->r_ticks[tid], ticks_s[tid]);
}

// ---------------------------------------------------------------- launch
template <int P, bool X3 = false>
static void launch_front(const GcnnArgs& a, int grid, hipStream_t s) {
  constexpr int nthr = FrontCfg<P, X3>::NW * 64;
  if (a.fr.dtype == HYDRO_DTYPE_U8) hipLaunchKernelGGL((c4_front_kernel<P, true, X3>), dim3(grid), dim3(nthr), 0, s, a);
  else hipLaunchKernelGGL((c4_front_kernel<P, false, X3>), dim3(grid), dim3(nthr), 0, s, a);
}

void launch_c4_pass(const GcnnArgs& a, const Forward& f, int prec, int grid, hipStream_t s) {
  const int g1 = grid * (prec == C4_F32 || prec == C4_X3 ? 1 : 2);
  if (prec == C4_FP8) {
    launch_front<C4_FP8>(a, g1, s);
    hipLaunchKernelGGL((c4_gemm_kernel<C4_FP8, 2>), dim3(grid), dim3(512), 0, s, a, f);
    hipLaunchKernelGGL((c4_gemm_kernel<C4_FP8, 3>), dim3(grid), dim3(512), 0, s, a, f);
  } else if (prec == C4_BF16) {
    launch_front<C4_BF16>(a, g1, s);
    hipLaunchKernelGGL((c4_gemm_bf16_kernel<2>), dim3(grid), dim3(512), 0, s, a, f);
    hipLaunchKernelGGL((c4_gemm_bf16_kernel<3>), dim3(grid), dim3(512), 0, s, a, f);
  } else if (prec == C4_X3) {
    // the FP32 tier's kernels and images with the three leading products only
    launch_front<C4_F32, true>(a, g1, s);
    hipLaunchKernelGGL((c4_gemm_kernel<C4_S3, 2, true>), dim3(grid), dim3(512), 0, s, a, f);
    hipLaunchKernelGGL((c4_gemm_kernel<C4_S3, 3, true>), dim3(grid), dim3(512), 0, s, a, f);
  } else {
    // FP32 arithmetic: the front in fp32, layers 3 and 4 as three-term bf16 products
    launch_front<C4_F32>(a, g1, s);
    hipLaunchKernelGGL((c4_gemm_kernel<C4_S3, 2>), dim3(grid), dim3(512), 0, s, a, f);
    hipLaunchKernelGGL((c4_gemm_kernel<C4_S3, 3>), dim3(grid), dim3(512), 0, s, a, f);
  }
}

// ---------------------------------------------------------------- host-side packing
bool c4_shape_ok(int in_hw, int n_layers, const int* widths) {
  return in_hw == 128 && n_layers == 4 && widths[0] == 32 && widths[1] == 64 && widths[2] == 128 && widths[3] == 256;
}

// OCP e4m3 (bias 7, largest finite 448, no infinities), round to nearest even, saturating.
uint8_t c4_fp8_e4m3(float x) {
  const uint8_t sign = std::signbit(x) ? 0x80 : 0x00;
  float a = std::fabs(x);
  if (!(a == a)) return 0x7F;
  if (a >= 448.f) return sign | 0x7E;
  if (a < std::ldexp(1.f, -10)) return sign;            // below half the smallest subnormal
  int e;
  std::frexp(a, &e);                                     // a = m * 2^e, m in [0.5, 1)
  int ex = e - 1;                                        // a in [2^ex, 2^(ex+1))
  if (ex < -6) ex = -6;                                  // subnormal range: spacing 2^-9
  const float q = std::ldexp(1.f, ex - 3);               // spacing of the binade
  float r = std::nearbyint(a / q);                       // round half even (default mode)
  float v = r * q;
  if (v >= 448.f) return sign | 0x7E;
  // encode v
  if (v < std::ldexp(1.f, -6)) return sign | (uint8_t)(int)std::nearbyint(v / std::ldexp(1.f, -9));
  int ev;
  const float mv = std::frexp(v, &ev);                   // v = mv * 2^ev
  const int E = ev - 1 + 7;
  const int M = (int)std::nearbyint((mv * 2.f - 1.f) * 8.f);
  return sign | (uint8_t)((E << 3) | M);
}

float c4_fp8_value(uint8_t b) {
  const int s = b >> 7, E = (b >> 3) & 15, M = b & 7;
  float v = E == 0 ? std::ldexp((float)M, -9) : std::ldexp(1.f + M / 8.f, E - 7);
  if (E == 15 && M == 7) v = NAN;
  return s ? -v : v;
}

static uint16_t c4_bf16_bits(float v) {
  uint32_t u;
  memcpy(&u, &v, 4);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
static float c4_bf16_value(uint16_t h) {
  const uint32_t u = (uint32_t)h << 16;
  float v;
  memcpy(&v, &u, 4);
  return v;
}

// conv weights w: [cout][cin][3][3] canonical fp32.  Element (oc, k) of the GEMM with
// k = tap * cin + ch, tap = 3u + v.
static inline float c4_w(const float* w, int cin, int oc, int k) {
  const int tap = k / cin, ch = k % cin;
  return w[((size_t)(oc * cin + ch) * 3 + tap / 3) * 3 + tap % 3];
}

void c4_pack_front(const float* w1, float scale1, const float* b1, const float* w2, const float* s2, C4FrontPack* out) {
  // layer 1: k = 9u + 3v + c (27 real), then the bias (its activation is 1) in three bf16 terms that
  // add up to it exactly; K slots per conv1_k
  auto w1k = [&](int oc, int kk) -> float {
    if (kk >= 30) return 0.f;
    if (kk >= 27) {
      float v = b1[oc];
      for (int t = 27; t < kk; ++t) v -= c4_bf16_value(c4_bf16_bits(v));
      return c4_bf16_value(c4_bf16_bits(v));
    }
    const int u = kk / 9, t = kk % 9, v = t / 3, c = t % 3;
    return scale1 * w1[((size_t)(oc * 3 + c) * 3 + u) * 3 + v];
  };
  out->w1b.assign(2 * 64 * 8, 0.f);
  for (int ct = 0; ct < 2; ++ct)
    for (int l = 0; l < 64; ++l)
      for (int e = 0; e < 8; ++e) out->w1b[(ct * 64 + l) * 8 + e] = w1k(ct * 16 + (l & 15), conv1_k(l >> 4, e));
  // FP32 arithmetic: the bf16 fragments' values split into three bf16 terms [term][ct][lane][8]
  out->w1s3.assign(3 * 2 * 64 * 8, 0);
  for (int ct = 0; ct < 2; ++ct)
    for (int l = 0; l < 64; ++l)
      for (int e = 0; e < 8; ++e) {
        float v = w1k(ct * 16 + (l & 15), conv1_k(l >> 4, e));
        for (int t = 0; t < 3; ++t) {
          const uint16_t h = c4_bf16_bits(v);
          out->w1s3[(((size_t)t * 2 + ct) * 64 + l) * 8 + e] = h;
          v -= c4_bf16_value(h);
        }
      }
  // layer 2 (cin 32), bf16 32x32x16 fragments [tap][h][c2][lane][8]: output channel
  // 32 c2 + lane % 32, input channel 16 h + 8 (lane / 32) + e
  out->w2b.assign(9 * 2 * 2 * 64 * 8, 0.f);
  for (int tp = 0; tp < 9; ++tp)
    for (int h = 0; h < 2; ++h)
      for (int c2 = 0; c2 < 2; ++c2)
        for (int l = 0; l < 64; ++l)
          for (int e = 0; e < 8; ++e)
            out->w2b[(((tp * 2 + h) * 2 + c2) * 64 + l) * 8 + e] =
                c4_w(w2, 32, c2 * 32 + (l & 31), tp * 32 + 16 * h + 8 * (l >> 5) + e);
  // FP32 arithmetic from bf16 terms, [tap][ct][term][lane][8]: the fp32 fragment's eight values
  // (output channel 16 ct + lane % 16, input channels 8 (lane / 16) + e) split hi, mid, lo
  out->w2s3.assign(9 * 4 * 3 * 64 * 8, 0);
  for (int tp = 0; tp < 9; ++tp)
    for (int ct = 0; ct < 4; ++ct)
      for (int l = 0; l < 64; ++l)
        for (int e = 0; e < 8; ++e) {
          float v = c4_w(w2, 32, ct * 16 + (l & 15), tp * 32 + 8 * (l >> 4) + e);
          for (int t = 0; t < 3; ++t) {
            const uint16_t h = c4_bf16_bits(v);
            out->w2s3[((((size_t)tp * 4 + ct) * 3 + t) * 64 + l) * 8 + e] = h;
            v -= c4_bf16_value(h);
          }
        }
  // fp8 [s][ct][lane][32 bytes]: tap 4s + g, channels 0..31
  out->w2q.assign(3 * 4 * 64 * 32, 0);
  for (int s = 0; s < 3; ++s)
    for (int ct = 0; ct < 4; ++ct)
      for (int l = 0; l < 64; ++l) {
        const int tp = 4 * s + (l >> 4), oc = ct * 16 + (l & 15);
        for (int c = 0; c < 32; ++c)
          out->w2q[((s * 4 + ct) * 64 + l) * 32 + c] = tp < 9 ? c4_fp8_e4m3(c4_w(w2, 32, oc, tp * 32 + c) / s2[oc]) : 0;
      }
}

size_t c4_img_bytes(int prec, int layer) {
  const int cout = layer == 2 ? 128 : 256;
  return (size_t)c4_nkb(prec, layer) * cout * (prec == C4_S3 ? 3 * 64 : 128);
}


// A image of a GEMM layer: [kb][oc][UPR units of 16 bytes], unit s holding chunk s ^ swz(oc);
// chunk c of k-block kb holds k = kb * BKE + c * CE + e.
void c4_pack_img(int prec, int layer, const float* w, const float* scale, unsigned char* out) {
  const int cin = layer == 2 ? 64 : 128, cout = layer == 2 ? 128 : 256;
  if (prec == C4_S3) {
    // [kb][term][oc][4 units]: unit s of a row holds chunk s ^ swz4(oc), chunk c holds
    // k = 32 kb + 8 c + e; term t of w is the bf16 rounding of w minus the earlier terms
    const int nkb = c4_nkb(prec, layer);
    for (int kb = 0; kb < nkb; ++kb)
      for (int oc = 0; oc < cout; ++oc)
        for (int s = 0; s < 4; ++s) {
          const int c = s ^ c4_swz<4>(oc);
          for (int e = 0; e < 8; ++e) {
            const int kk = kb * 32 + c * 8 + e;
            float v = kk < 9 * cin ? c4_w(w, cin, oc, kk) : 0.f;
            for (int t = 0; t < 3; ++t) {
              const uint16_t h = c4_bf16_bits(v);
              memcpy(out + ((((size_t)kb * 3 + t) * cout + oc) * 4 + s) * 16 + 2 * e, &h, 2);
              v -= c4_bf16_value(h);
            }
          }
        }
    return;
  }
  const int es = prec == C4_FP8 ? 1 : 2;
  const int rowb = 128, upr = rowb / 16, ce = 16 / es, bke = rowb / es;
  const int nkb = c4_nkb(prec, layer);
  for (int kb = 0; kb < nkb; ++kb)
    for (int row = 0; row < cout; ++row)
      for (int s = 0; s < upr; ++s) {
        // BF16 layer 3 (the third convolution): image row R holds channel c4_l3_channel(R)
        const int oc = prec == C4_BF16 && layer == 2 ? c4_l3_channel(row) : row;
        const int c = s ^ (upr == 4 ? c4_swz<4>(row) : c4_swz<8>(row));
        unsigned char* dst = out + (((size_t)kb * cout + row) * upr + s) * 16;
        for (int e = 0; e < ce; ++e) {
          const int kk = kb * bke + c * ce + e;
          const float v = kk < 9 * cin ? c4_w(w, cin, oc, kk) : 0.f;
          if (prec == C4_FP8) {
            dst[e] = c4_fp8_e4m3(v / scale[oc]);
          } else {
            const uint16_t h = c4_bf16_bits(v);
            memcpy(dst + 2 * e, &h, 2);
          }
        }
      }
}

}  // namespace hydro
