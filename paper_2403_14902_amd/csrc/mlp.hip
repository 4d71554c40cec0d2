// MLP predicates on gfx950: gathered-row GEMM1 on MFMA (bf16 or fp32 operands, fp32
// accumulation) with ReLU and a partial GEMM2 in the epilogue; a head kernel that finishes the
// logits, takes the class-subset margin and forwards the decision; and an FP64 tier.
//
// The model (one synthetic UDF predicate): h = ReLU(x' W1 + b1), z = h W2 + b2 with
// x' = (x - 0.5) * 4 flattened NHWC.  The first two passes use the folded form
// h = ReLU((s W1)^T raw + (b1 - 2 colsum(W1))) with s = 4 (or 4/255 for uint8 frames), which is
// the same function of the stored frame without a separate normalisation step.
#include "engine.h"

namespace hydro {

template <typename T> struct MlpTile;
template <> struct MlpTile<__bf16> { static constexpr int BK = 32, LD = 40; };   // LDS row stride (elements)
template <> struct MlpTile<float> { static constexpr int BK = 16, LD = 20; };

// Load `N` consecutive frame elements of type In starting at element `off` of frame `idx`,
// converted to T.  The element type is a template parameter, so the loads are straight-line code
// and the compiler can count the ones in flight precisely.
template <typename T, typename In, int N>
__device__ inline void load_frame_run(const FrameSrc& fr, uint32_t idx, int64_t off, T* out) {
  constexpr int BYTES = N * (int)sizeof(In);
  static_assert(BYTES == 4 || BYTES == 8 || BYTES % 16 == 0, "frame run size");
  const In* p = static_cast<const In*>(fr.base) + (int64_t)idx * fr.elems + off;
  alignas(16) In buf[N];
  if constexpr (BYTES % 16 == 0) {
#pragma unroll
    for (int v = 0; v < BYTES / 16; ++v) reinterpret_cast<uint4*>(buf)[v] = reinterpret_cast<const uint4*>(p)[v];
  } else if constexpr (BYTES == 8) {
    *reinterpret_cast<uint2*>(buf) = *reinterpret_cast<const uint2*>(p);
  } else {
    *reinterpret_cast<uint32_t*>(buf) = *reinterpret_cast<const uint32_t*>(p);
  }
#pragma unroll
  for (int j = 0; j < N; ++j) out[j] = static_cast<T>((float)buf[j]);
}

// How a GEMM launch is cut into work units.  Its (rows x hidden) tiles fill the GPU's resident
// workgroups (MlpArgs::units of them) a whole number of times; the tiles that are left over, or
// all of them in a short launch (a re-score band, a late round), are split along K into S parts
// each, so that they fill the GPU once more.  A whole tile ends in partial logits; a part stores its
// raw sums in the workspace, and the head kernel, which runs next on the stream, adds a tile's parts
// in order (so the result does not depend on which part finished first, and no part waits for or
// signals another).  S is a power of two and a function of the queue counts alone.
// Against splitting only launches of less than half a CU's tile each, by parts that counted
// themselves and left the sum to the last one to arrive (a device-scope fence per part): the FP32
// band of a 3,072-input query 84 + 7 (head) -> 28 + 18 us a round; the six-MLP query (131,072 x 12,288
// bf16) 9.7 -> 6.5 ms together with the XCD order below.
constexpr int SPLIT_MAX = 16;
constexpr int SPLIT_MIN_K = 4;       // k-blocks per part, at least
struct MlpPlan { int full, rest, S, units; };
__device__ inline MlpPlan mlp_plan(const MlpArgs& a) {
  int tiles = 0, nk = 1 << 30;
  for (int i = 0; i < a.n_preds; ++i) {
    tiles += ((a.q.counts[a.pred[i]] + a.bm - 1) / a.bm) * (a.hidden[i] / a.bn);
    nk = min(nk, a.d_in[i] / a.bk);
  }
  MlpPlan p{tiles, 0, 1, tiles};
  const bool may = a.split_below < 0 || tiles < a.split_below;
  const int full = tiles / a.units * a.units, rest = tiles - full;
  if (may && a.splitk_ws != nullptr && rest > 0) {
    const int most = min(min(a.units / rest, SPLIT_MAX), min(a.split_slots / rest, nk / SPLIT_MIN_K));
    int S = 1;
    while (2 * S <= most) S *= 2;
    if (S > 1) p = MlpPlan{full, rest, S, full + rest * S};
  }
  return p;
}

// Work unit u: its tile, K range and workspace tile (ws < 0: a whole tile).  Consecutive workgroups
// go to the eight XCDs in turn, each with an L2 of its own; units are dealt so that every XCD gets
// consecutive tiles, whose hidden-unit tiles (the fastest index) read the same frame rows: each
// row then comes from HBM once, not once per XCD (8,192 x 12,288 bf16 rows x 2,048 units: 1,105 TFLOP/s;
// tiles dealt in turn averaged 494 over the six-MLP query's launches, now 780 with its short ones).
struct MlpUnit { int slot, mt, nt, kb0, kb1, ws; };
__device__ inline MlpUnit mlp_unit(const MlpArgs& a, const MlpPlan& p, int u) {
  const int base = u < p.full ? u / a.units * a.units : p.full;
  const int n = min(a.units, (u < p.full ? p.full : p.units) - base), v = u - base;
  const int x = v & 7, each = n >> 3, more = n & 7;
  const int w = base + x * each + min(x, more) + (v >> 3);
  int t = w, part = 0;
  MlpUnit m;
  m.ws = -1;
  if (w >= p.full && p.S > 1) {
    t = p.full + (w - p.full) % p.rest;
    part = (w - p.full) / p.rest;
    m.ws = (t - p.full) * p.S + part;
  }
  m.slot = m.mt = m.nt = 0;
  for (int i = 0; i < a.n_preds; ++i) {
    const int n_nt = a.hidden[i] / a.bn;
    const int tiles = ((a.q.counts[a.pred[i]] + a.bm - 1) / a.bm) * n_nt;
    if (t < tiles) {
      m.slot = i;
      m.mt = t / n_nt;
      m.nt = t % n_nt;
      break;
    }
    t -= tiles;
  }
  const int nk = a.d_in[m.slot] / a.bk;
  m.kb0 = m.ws < 0 ? 0 : (int)((int64_t)nk * part / p.S);
  m.kb1 = m.ws < 0 ? nk : (int)((int64_t)nk * (part + 1) / p.S);
  return m;
}

// End of a unit for one wave, which holds rows row0 + 16 i + 4 g + r and hidden units col0 + 16 j + l16
// of the tile in acc[i][j][r].  A part: raw sums to the workspace, [column][row], four consecutive rows
// per store.  A whole tile: H = ReLU(acc + b1'), partial logits over the wave's hidden units, lane
// l16 storing class l16 of each row.
template <int BM, int BN, int MT, int NT>
__device__ inline void mlp_finish(const MlpArgs& a, const MlpUnit& m, floatx4 (&acc)[MT][NT], int row0, int col0) {
  const int lane = lane_id(), g = lane >> 4, l16 = lane & 15;
  if (m.ws >= 0) {
    float* wt = a.splitk_ws + (int64_t)m.ws * (BM * BN);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
        *reinterpret_cast<float4*>(&wt[(col0 + j * 16 + l16) * BM + row0 + i * 16 + 4 * g]) =
            make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
    return;
  }
  const float* b1 = a.b1_fold[m.slot];
  const float* w2 = a.w2[m.slot];
  const int cnt = a.q.counts[a.pred[m.slot]];
  const int c0 = m.nt * BN + col0 + l16;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const float bb = b1[c0 + j * 16];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = fmaxf(acc[i][j][r] + bb, 0.f);
  }
  float zv[MT][4];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) zv[i][r] = 0.f;
#pragma unroll 1
  for (int c = 0; c < kClasses; ++c) {
    float w2v[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) w2v[j] = w2[(c0 + j * 16) * kClasses + c];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float s = 0.f;
#pragma unroll
        for (int j = 0; j < NT; ++j) s += acc[i][j][r] * w2v[j];
        s = row_sum16(s);
        zv[i][r] = l16 == c ? s : zv[i][r];
      }
  }
  float* part = a.partial[m.slot] + (int64_t)((m.nt * BN + col0) / (16 * NT)) * a.part_cap * kClasses;
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int rr = m.mt * BM + row0 + i * 16 + 4 * g + r;
      if (l16 < kClasses && rr < cnt) part[(int64_t)rr * kClasses + l16] = zv[i][r];
    }
}

// Tile shapes (rows of queued tuples x hidden units) an autotuner may pick per predicate.
// Every launch covers the predicates of one tile shape.  The bound on the registers keeps two 128x128
// workgroups on a CU (left alone, the compiler takes 258 with uint8 frames, which lets in one: 6,000 rows
// of 12,288 inputs x 2,048 units 1,310 us, so 880), three 128x64 and five 64x64 ones.
template <typename T, typename In, int BM, int BN>
__global__ __launch_bounds__(256, BM * BN == 16384 ? 2 : BM * BN == 8192 ? 3 : 5) void mlp_gemm_kernel(MlpArgs a) {
  constexpr int BK = MlpTile<T>::BK, LD = MlpTile<T>::LD;
  // every thread loads one run of each k-tile: 256 / BM threads per gathered frame row (PA
  // elements each) and 256 / BN per weight row (PB elements each)
  constexpr int TPA = 256 / BM, PA = BK / TPA, TPB = 256 / BN, PB = BK / TPB;
  constexpr int WM = BM / 2, WN = BN / 2;         // 2 x 2 waves
  constexpr int FM = WM / 16, FN = WN / 16;       // MFMA tiles per wave
  __shared__ __attribute__((aligned(16))) T As[2][BM * LD];
  __shared__ __attribute__((aligned(16))) T Bs[2][BN * LD];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int ar = tid / TPA, ak = (tid % TPA) * PA;   // this thread's frame row in the tile, k offset
  const int br = tid / TPB, bk = (tid % TPB) * PB;   // this thread's weight row in the tile, k offset

  const MlpPlan plan = mlp_plan(a);
  for (int u = blockIdx.x; u < plan.units; u += gridDim.x) {
    const MlpUnit m = mlp_unit(a, plan, u);
    const int slot = m.slot, mt = m.mt, nt = m.nt;
    const int k = a.pred[slot];
    const int cnt = a.q.counts[k];
    const int D = a.d_in[slot];
    const uint32_t* qe = a.q.entries + (int64_t)k * a.q.cap;
    unsigned long long t0 = wall_clock64();

    const int row = mt * BM + ar;
    const uint32_t idx = entry_idx(qe[row < cnt ? row : cnt - 1]);
    const T* wrow;
    if constexpr (sizeof(T) == 2) wrow = reinterpret_cast<const T*>(a.w1_bf[slot]) + (int64_t)(nt * BN + br) * D;
    else wrow = reinterpret_cast<const T*>(a.w1_f32[slot]) + (int64_t)(nt * BN + br) * D;

    floatx4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = (floatx4){0.f, 0.f, 0.f, 0.f};

    // NS register stages: the global loads of k-tile kt + NS - 1 are issued while tile kt is
    // computed (two stages measured fastest: deeper staging costs more than it hides here).
    constexpr int NS = 2;
    alignas(16) T ra[NS][PA];
    alignas(16) T rb[NS][PB];
    auto gload = [&](int kt, int st) {
      load_frame_run<T, In, PA>(a.fr, idx, (int64_t)kt * BK + ak, ra[st]);
      const uint4* pb = reinterpret_cast<const uint4*>(wrow + (int64_t)kt * BK + bk);
#pragma unroll
      for (int v = 0; v < PB * (int)sizeof(T) / 16; ++v) reinterpret_cast<uint4*>(rb[st])[v] = pb[v];
    };
    auto lstore = [&](int st, int buf) {
#pragma unroll
      for (int v = 0; v < PA * (int)sizeof(T) / 16; ++v)
        reinterpret_cast<uint4*>(&As[buf][ar * LD + ak])[v] = reinterpret_cast<uint4*>(ra[st])[v];
#pragma unroll
      for (int v = 0; v < PB * (int)sizeof(T) / 16; ++v)
        reinterpret_cast<uint4*>(&Bs[buf][br * LD + bk])[v] = reinterpret_cast<uint4*>(rb[st])[v];
    };
    auto compute = [&](int buf) {
      if constexpr (sizeof(T) == 2) {
        bf16x8 af[FM], bfr[FN];
#pragma unroll
        for (int i = 0; i < FM; ++i)
          af[i] = *reinterpret_cast<const bf16x8*>(&As[buf][(wm * WM + i * 16 + (lane & 15)) * LD + 8 * (lane >> 4)]);
#pragma unroll
        for (int j = 0; j < FN; ++j)
          bfr[j] = *reinterpret_cast<const bf16x8*>(&Bs[buf][(wn * WN + j * 16 + (lane & 15)) * LD + 8 * (lane >> 4)]);
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
      } else {
        // a k-tile's products are summed by themselves and then added, so that the running sum is rounded once a
        // k-tile (5,000 rows of 3,072 fp32 inputs in four parts: rms error 1.6e-6 with one sum, 0.5e-6 so; in seven
        // parts 1.2e-6)
        float af[FM][BK / 4];
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int ks = 0; ks < BK / 4; ++ks)
            af[i][ks] = As[buf][(wm * WM + i * 16 + (lane & 15)) * LD + ks * 4 + (lane >> 4)];
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          float bfr[BK / 4];
#pragma unroll
          for (int ks = 0; ks < BK / 4; ++ks)
            bfr[ks] = Bs[buf][(wn * WN + j * 16 + (lane & 15)) * LD + ks * 4 + (lane >> 4)];
          floatx4 t[FM];
#pragma unroll
          for (int i = 0; i < FM; ++i) t[i] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < BK / 4; ++ks)
#pragma unroll
            for (int i = 0; i < FM; ++i) t[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[i][ks], bfr[ks], t[i], 0, 0, 0);
#pragma unroll
          for (int i = 0; i < FM; ++i) acc[i][j] += t[i];
        }
      }
    };

    const int kt0 = m.kb0, nk = m.kb1;
#pragma unroll
    for (int u = 0; u < NS - 1; ++u)
      if (kt0 + u < nk) gload(kt0 + u, u);
    lstore(0, kt0 & 1);
    __syncthreads();
    // k-tile kt = kb + u lives in register stage u (kb - kt0 is a multiple of NS)
    for (int kb = kt0; kb < nk; kb += NS) {
#pragma unroll
      for (int u = 0; u < NS; ++u) {
        const int kt = kb + u;
        if (kt < nk) {
          const int buf = kt & 1;
          if (kt + NS - 1 < nk) gload(kt + NS - 1, (u + NS - 1) % NS);
          compute(buf);
          if (kt + 1 < nk) {
            __syncthreads();
            lstore((u + 1) % NS, buf ^ 1);
            __syncthreads();
          }
        }
      }
    }

    mlp_finish<BM, BN, FM, FN>(a, m, acc, wm * WM, wn * WN);
    __syncthreads();
    if (tid == 0 && a.count_ticks) atomicAdd(&a.st->r_ticks[k], (unsigned long long)(wall_clock64() - t0));
  }
}

// GEMM2 of one row's hidden units c = cg, cg + ng, ... of a split tile.  Every part of a column, and
// four columns at a time, are requested before the first is used: the parts come from other
// XCDs' writes, past the L2, and their latency is all that this costs.
template <int S>
__device__ inline void mlp_split_cols(const float* wt, int64_t tsz, int bm, int bn, int cg, int ng, const float* b1,
                                      const float* w2, float (&z)[kClasses]) {
  constexpr int CU = S >= 16 ? 2 : 4;
  for (int c0 = cg; c0 < bn; c0 += CU * ng) {        // bn is a multiple of CU * ng
    float v[CU][S];
#pragma unroll
    for (int u = 0; u < CU; ++u)
#pragma unroll
      for (int p = 0; p < S; ++p) v[u][p] = wt[(int64_t)p * tsz + (int64_t)(c0 + u * ng) * bm];
#pragma unroll
    for (int u = 0; u < CU; ++u) {
      const int c = c0 + u * ng;
      float h = 0.f;
#pragma unroll
      for (int p = 0; p < S; ++p) h += v[u][p];
      h = fmaxf(h + b1[c], 0.f);
      const float2* w = reinterpret_cast<const float2*>(w2 + (int64_t)c * kClasses);
#pragma unroll
      for (int cc = 0; cc < kClasses / 2; ++cc) {
        const float2 x = w[cc];
        z[2 * cc] = fmaf(h, x.x, z[2 * cc]);
        z[2 * cc + 1] = fmaf(h, x.y, z[2 * cc + 1]);
      }
    }
  }
}

// Head: z = b2 + the partial logits of the whole tiles + GEMM2 of the split ones (their parts added in
// order, then bias and ReLU); margin; decision / deferral; forwarding.  One workgroup per RG rows of
// one predicate: 64, or 16 when those would leave CUs idle (a re-score band), since a split tile's
// parts are most of what it reads.  Thread (row, group): the groups share a row's hidden units.
__global__ __launch_bounds__(256) void mlp_head_kernel(MlpArgs a, Forward f) {
  __shared__ float zs[256 * kClasses];
  const int tid = threadIdx.x;
  const MlpPlan plan = mlp_plan(a);
  int groups64 = 0;
  for (int i = 0; i < a.n_preds; ++i) groups64 += (a.q.counts[a.pred[i]] + 63) / 64;
  const int RG = groups64 < a.n_cu ? 16 : 64, ng = 256 / RG;
  const int row = tid & (RG - 1), cg = tid / RG;
  int total = 0;
  for (int i = 0; i < a.n_preds; ++i) total += (a.q.counts[a.pred[i]] + RG - 1) / RG;
  for (int t = blockIdx.x; t < total; t += gridDim.x) {
    int slot = 0, off = t, tile0 = 0;         // tile0: the slot's first tile in the launch's order
    for (int i = 0; i < a.n_preds; ++i) {
      const int cnt = a.q.counts[a.pred[i]], c = (cnt + RG - 1) / RG;
      slot = i;
      if (off < c) break;
      off -= c;
      tile0 += ((cnt + a.bm - 1) / a.bm) * (a.hidden[i] / a.bn);
    }
    const int k = a.pred[slot], cnt = a.q.counts[k];
    const int rr = off * RG + row, rc = min(rr, cnt - 1);
    const int n_nt = a.hidden[slot] / a.bn, mt = off * RG / a.bm;
    const int first = tile0 + mt * n_nt;      // this row group's tiles: first .. first + n_nt - 1
    float z[kClasses];
#pragma unroll
    for (int c = 0; c < kClasses; ++c) z[c] = 0.f;
    const int whole = plan.S > 1 ? max(0, min(n_nt, plan.full - first)) : n_nt;
    const int ppt = a.bn / a.part_w[slot];    // partial-logit parts per tile
    for (int p = cg; p < whole * ppt; p += ng) {
      const float2* pp = reinterpret_cast<const float2*>(a.partial[slot] + ((int64_t)p * a.part_cap + rc) * kClasses);
#pragma unroll
      for (int c = 0; c < kClasses / 2; ++c) {
        const float2 v = pp[c];
        z[2 * c] += v.x;
        z[2 * c + 1] += v.y;
      }
    }
    const float* b1 = a.b1_fold[slot];
    const float* w2 = a.w2[slot];
    const int64_t tsz = (int64_t)a.bm * a.bn;
    for (int nt = whole; nt < n_nt; ++nt) {
      const float* wt = a.splitk_ws + (int64_t)(first + nt - plan.full) * plan.S * tsz + (rc - mt * a.bm);
      const float *tb1 = b1 + nt * a.bn, *tw2 = w2 + (int64_t)nt * a.bn * kClasses;
      if (plan.S == 2) mlp_split_cols<2>(wt, tsz, a.bm, a.bn, cg, ng, tb1, tw2, z);
      else if (plan.S == 4) mlp_split_cols<4>(wt, tsz, a.bm, a.bn, cg, ng, tb1, tw2, z);
      else if (plan.S == 8) mlp_split_cols<8>(wt, tsz, a.bm, a.bn, cg, ng, tb1, tw2, z);
      else mlp_split_cols<16>(wt, tsz, a.bm, a.bn, cg, ng, tb1, tw2, z);
    }
#pragma unroll
    for (int c = 0; c < kClasses; ++c) zs[c * 256 + tid] = z[c];
    __syncthreads();
    if (tid < kWave) {
      const bool active = tid < RG && rr < cnt;
      const uint32_t e = active ? a.q.entries[(int64_t)k * a.q.cap + rr] : 0u;
      bool pass = false, defer = false;
      if (active) {
        const float* b2 = a.b2[slot];
#pragma unroll
        for (int c = 0; c < kClasses; ++c) {
          float s = b2[c];
          for (int g = 0; g < ng; ++g) s += zs[c * 256 + g * RG + row];
          z[c] = s;
        }
        if (f.logits != nullptr) {
          for (int c = 0; c < kClasses; ++c) f.logits[(int64_t)entry_idx(e) * kClasses + c] = (double)z[c];
        } else {
          const float d = class_margin(z, a.class_mask[slot]), th = theta_of(f, k, entry_idx(e));
          defer = f.defer.entries != nullptr && fabsf(d - th) < f.tau[k];
          pass = d > th;
        }
      }
      if (f.logits == nullptr) forward_decision(f, k, e, active, defer, pass);
    }
    __syncthreads();           // zs is reused by the next group
  }
}

// FP64 tier: frames normalised in fp64 exactly as defined; canonical fp32 weights widened to
// fp64.  Escalated entries of each predicate are evaluated across many workgroups: work item =
// (predicate, group of 8 entries, 256 hidden units, chunk of the input) -> partial hidden sums; a
// second launch adds the chunks (one workgroup per entry: with one wave, H / 64 x D / 256 dependent
// loads took up to 0.3 ms of a round), applies ReLU, GEMM2, the margin and the decision.  The partial
// sums have room for esc_cap entries of 256-long chunks: more entries get longer chunks, down to one
// chunk an entry; what is still beyond runs in the second launch, one group per block.  1,024 entries
// of 12,288 inputs and 2,048 hidden units: 50 ms with all but 128 of them in the second launch, 4.4 ms
// so (11.6 TFLOP/s, LDS reads of the inputs).  Tiles of 16 entries on FP64 matrix instructions take
// 3.4 ms there but 52 us instead of 35 in a query's rounds of a few entries.
constexpr int F64_B = 8;
constexpr int F64_DCH = 256;
int mlp_f64_chunks(int d_in) { return (d_in + F64_DCH - 1) / F64_DCH; }

// A predicate's share of the layer-parallel part: entries, 256-long units of input a chunk, chunks
struct F64Split { int ne, len, nch; };
__device__ inline F64Split mlp_f64_split(int count, int cap, int D) {
  const int units = (D + F64_DCH - 1) / F64_DCH;
  if (count <= cap) return {count, 1, units};
  const int all = cap * units, ne = min(count, all);      // (far below 2^31: 8 H `all` bytes are allocated)
  const int room = min(all / ne, units);
  const int len = (units + room - 1) / room;
  return {ne, len, (units + len - 1) / len};
}

__device__ inline double frame_norm64_flat(const FrameSrc& fr, uint32_t idx, int64_t d) {
  const int64_t o = (int64_t)idx * fr.elems + d;
  double x;
  if (fr.dtype == HYDRO_DTYPE_BF16) x = (double)(float)static_cast<const __bf16*>(fr.base)[o];
  else if (fr.dtype == HYDRO_DTYPE_U8) x = (double)static_cast<const uint8_t*>(fr.base)[o] / 255.0;
  else x = (double)static_cast<const float*>(fr.base)[o];
  return (x - 0.5) * 4.0;
}

__global__ __launch_bounds__(256) void mlp_f64_hidden_kernel(MlpArgs a) {
  __shared__ double xs[F64_B][F64_DCH];
  __shared__ uint32_t ents[F64_B];
  const int tid = threadIdx.x;
  auto items = [&](int i, const F64Split& sp) { return (sp.ne + F64_B - 1) / F64_B * ((a.hidden[i] + 255) / 256) * sp.nch; };
  int total = 0;
  for (int i = 0; i < a.n_preds; ++i) total += items(i, mlp_f64_split(a.q.counts[a.pred[i]], a.esc_cap, a.d_in[i]));
  for (int t = blockIdx.x; t < total; t += gridDim.x) {
    int slot = 0, off = t;
    F64Split sp = {0, 1, 1};
    for (int i = 0; i < a.n_preds; ++i) {
      sp = mlp_f64_split(a.q.counts[a.pred[i]], a.esc_cap, a.d_in[i]);
      const int c = items(i, sp);
      slot = i;
      if (off < c) break;
      off -= c;
    }
    const int k = a.pred[slot];
    const int D = a.d_in[slot], H = a.hidden[slot];
    const int nhb = (H + 255) / 256;
    const int ch = off % sp.nch;
    const int hb = (off / sp.nch) % nhb;
    const int grp = off / (sp.nch * nhb);
    const int nb = min(F64_B, sp.ne - grp * F64_B);
    if (tid < F64_B) ents[tid] = tid < nb ? a.q.entries[(int64_t)k * a.q.cap + grp * F64_B + tid] : 0u;
    __syncthreads();
    const int j = hb * 256 + tid;
    double s[F64_B];
#pragma unroll
    for (int b = 0; b < F64_B; ++b) s[b] = 0.0;
    const float* W1 = a.w1_canon[slot];
    const int d_lo = ch * sp.len * F64_DCH, d_hi = min(D, d_lo + sp.len * F64_DCH);
    for (int d0 = d_lo; d0 < d_hi; d0 += F64_DCH) {
      const int dl = min(F64_DCH, d_hi - d0);
      for (int q = tid; q < F64_B * F64_DCH; q += 256) {
        const int b = q / F64_DCH, dd = q % F64_DCH;
        xs[b][dd] = (b < nb && dd < dl) ? frame_norm64_flat(a.fr, entry_idx(ents[b]), d0 + dd) : 0.0;
      }
      __syncthreads();
      if (j < H) {
#pragma unroll 16
        for (int dd = 0; dd < dl; ++dd) {
          const double w = (double)W1[(int64_t)(d0 + dd) * H + j];
#pragma unroll
          for (int b = 0; b < F64_B; ++b) s[b] = fma(w, xs[b][dd], s[b]);
        }
      }
      __syncthreads();
    }
    if (j < H) {
      double* hp = a.esc_h[slot] + (int64_t)ch * sp.ne * H;
      for (int b = 0; b < nb; ++b) hp[(int64_t)(grp * F64_B + b) * H + j] = s[b];
    }
    __syncthreads();
  }
}

// Decisions of the layer-parallel entries; the entries beyond them: groups of 4 per block, the whole
// input and hidden width in one block, 256 hidden units at a time (all of them at once, a thread's
// eight units behind eight branches, waited for every weight by itself).
constexpr int R64_B = 4;
constexpr int R64_DCH = 256;

__global__ __launch_bounds__(256) void mlp_f64_entry_kernel(MlpArgs a, Forward f) {
  __shared__ double xs[R64_B][R64_DCH];
  __shared__ double zred[4][R64_B][kClasses];
  __shared__ uint32_t ents[R64_B];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // the layer-parallel entries: their hidden units' chunk sums added, ReLU, GEMM2, decision
  int heads = 0;
  for (int i = 0; i < a.n_preds; ++i) heads += mlp_f64_split(a.q.counts[a.pred[i]], a.esc_cap, a.d_in[i]).ne;
  for (int t = blockIdx.x; t < heads; t += gridDim.x) {
    int slot = 0, off = t;
    F64Split sp = {0, 1, 1};
    for (int i = 0; i < a.n_preds; ++i) {
      sp = mlp_f64_split(a.q.counts[a.pred[i]], a.esc_cap, a.d_in[i]);
      slot = i;
      if (off < sp.ne) break;
      off -= sp.ne;
    }
    const int k = a.pred[slot], H = a.hidden[slot];
    double zp[kClasses];
#pragma unroll
    for (int c = 0; c < kClasses; ++c) zp[c] = 0.0;
    for (int j = tid; j < H; j += 256) {
      double h = (double)a.b1_canon[slot][j];
      const double* hp = a.esc_h[slot] + (int64_t)off * H + j;
#pragma unroll 16
      for (int c = 0; c < sp.nch; ++c) h += hp[(int64_t)c * sp.ne * H];
      h = h > 0.0 ? h : 0.0;
#pragma unroll
      for (int c = 0; c < kClasses; ++c) zp[c] = fma(h, (double)a.w2[slot][j * kClasses + c], zp[c]);
    }
#pragma unroll
    for (int c = 0; c < kClasses; ++c) {
      for (int o = 32; o >= 1; o >>= 1) zp[c] += __shfl_xor(zp[c], o);
      if (lane == 0) zred[wave][0][c] = zp[c];
    }
    __syncthreads();
    if (wave == 0) {
      const uint32_t e = a.q.entries[(int64_t)k * a.q.cap + off];
      const uint32_t idx = entry_idx(e);
      bool pass = false;
      if (lane == 0) {
        double z[kClasses];
        for (int c = 0; c < kClasses; ++c)
          z[c] = (double)a.b2[slot][c] + ((zred[0][0][c] + zred[1][0][c]) + (zred[2][0][c] + zred[3][0][c]));
        if (f.logits != nullptr)
          for (int c = 0; c < kClasses; ++c) f.logits[(int64_t)idx * kClasses + c] = z[c];
        pass = class_margin(z, a.class_mask[slot]) > (double)theta_of(f, k, idx);
      }
      if (f.logits == nullptr) forward_decision(f, k, e, lane == 0, false, pass);
    }
    __syncthreads();
  }
  auto rest_of = [&](int i) {
    const int n = a.q.counts[a.pred[i]];
    return n - mlp_f64_split(n, a.esc_cap, a.d_in[i]).ne;
  };
  int total = 0;
  for (int i = 0; i < a.n_preds; ++i) total += (rest_of(i) + R64_B - 1) / R64_B;
  for (int t = blockIdx.x; t < total; t += gridDim.x) {
    int slot = 0, off = t;
    for (int i = 0; i < a.n_preds; ++i) {
      const int c = (rest_of(i) + R64_B - 1) / R64_B;
      if (off < c) { slot = i; break; }
      off -= c;
    }
    const int k = a.pred[slot];
    const int rest = rest_of(slot);
    const int D = a.d_in[slot], H = a.hidden[slot];
    const int nb = min(R64_B, rest - off * R64_B);
    if (tid < R64_B)
      ents[tid] = tid < nb ? a.q.entries[(int64_t)k * a.q.cap + a.q.counts[k] - rest + off * R64_B + tid] : 0u;
    __syncthreads();
    double zp[R64_B][kClasses];
#pragma unroll
    for (int b = 0; b < R64_B; ++b)
#pragma unroll
      for (int c = 0; c < kClasses; ++c) zp[b][c] = 0.0;
    const float* w2 = a.w2[slot];
    for (int j0 = 0; j0 < H; j0 += 256) {
      const int col = j0 + tid;
      double s[R64_B];
#pragma unroll
      for (int b = 0; b < R64_B; ++b) s[b] = 0.0;
      for (int d0 = 0; d0 < D; d0 += R64_DCH) {
        for (int q = tid; q < R64_B * R64_DCH; q += blockDim.x) {
          const int b = q / R64_DCH, dd = q % R64_DCH;
          xs[b][dd] = (b < nb && d0 + dd < D) ? frame_norm64_flat(a.fr, entry_idx(ents[b]), d0 + dd) : 0.0;
        }
        __syncthreads();
        if (col < H) {
          const int dlim = min(R64_DCH, D - d0);
          const float* wr = a.w1_canon[slot] + (int64_t)d0 * H + col;
#pragma unroll 16
          for (int dd = 0; dd < dlim; ++dd) {
            const double w = (double)wr[(int64_t)dd * H];
#pragma unroll
            for (int b = 0; b < R64_B; ++b) s[b] = fma(w, xs[b][dd], s[b]);
          }
        }
        __syncthreads();
      }
      if (col < H) {
        const double bb = (double)a.b1_canon[slot][col];
#pragma unroll
        for (int b = 0; b < R64_B; ++b) {
          double h = s[b] + bb;
          h = h > 0.0 ? h : 0.0;
#pragma unroll
          for (int c = 0; c < kClasses; ++c) zp[b][c] = fma(h, (double)w2[col * kClasses + c], zp[b][c]);
        }
      }
    }
#pragma unroll
    for (int b = 0; b < R64_B; ++b)
#pragma unroll
      for (int c = 0; c < kClasses; ++c) {
        double v = zp[b][c];
        for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
        if (lane == 0) zred[wave][b][c] = v;
      }
    __syncthreads();
    if (wave == 0) {
      const bool active = lane < nb;
      bool pass = false;
      const uint32_t e = active ? ents[lane] : 0u;
      if (active) {
        double z[kClasses];
        const float* b2 = a.b2[slot];
        for (int c = 0; c < kClasses; ++c)
          z[c] = (double)b2[c] + ((zred[0][lane][c] + zred[1][lane][c]) + (zred[2][lane][c] + zred[3][lane][c]));
        if (f.logits != nullptr)
          for (int c = 0; c < kClasses; ++c) f.logits[(int64_t)entry_idx(e) * kClasses + c] = z[c];
        pass = class_margin(z, a.class_mask[slot]) > (double)theta_of(f, k, entry_idx(e));
      }
      if (f.logits == nullptr) forward_decision(f, k, e, active, false, pass);
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------- weights
// Folded weights [hidden][d_in] from the canonical [d_in][hidden]: w * scale rounded to fp32, that
// rounded to bf16 and, where the FP32 tier multiplies bf16 terms, split in three: hi = bf16(w),
// mid = bf16(w - hi), lo = bf16(w - hi - mid), each difference exact in fp32.  A transpose by tiles
// of 32 inputs x 64 hidden units; once a session.  (A host loop reads a cache line per weight and sends each
// form up by itself: the first call on a wide MLP 95 ms, so 3.0; a one-shot query of two MLPs of 3,072 inputs
// 5.7, so 3.1.)
__device__ inline uint16_t bf16_nearest(float v) {
  uint32_t u = __float_as_uint(v);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
constexpr int PK_D = 32, PK_H = 64;      // d_in is a multiple of 32, hidden of 128
__global__ __launch_bounds__(256) void mlp_pack_kernel(const float* w1, int D, int H, double scale, float* wt, uint16_t* wb, uint16_t* w3) {
  __shared__ float tile[PK_D][PK_H + 1];
  const int d0 = blockIdx.x * PK_D, j0 = blockIdx.y * PK_H;
  for (int q = threadIdx.x; q < PK_D * PK_H; q += 256)
    tile[q / PK_H][q % PK_H] = (float)((double)w1[(int64_t)(d0 + q / PK_H) * H + j0 + q % PK_H] * scale);
  __syncthreads();
  for (int q = threadIdx.x; q < PK_D * PK_H; q += 256) {
    const int j = q / PK_D, d = q % PK_D;
    const int64_t o = (int64_t)(j0 + j) * D + d0 + d;
    const float v = tile[d][j];
    const uint16_t hi = bf16_nearest(v);
    wt[o] = v;
    wb[o] = hi;
    if (w3 != nullptr) {
      const int64_t plane = (int64_t)H * D;
      const float r1 = v - __uint_as_float((uint32_t)hi << 16);
      const uint16_t mid = bf16_nearest(r1);
      w3[o] = hi;
      w3[plane + o] = mid;
      w3[2 * plane + o] = bf16_nearest(r1 - __uint_as_float((uint32_t)mid << 16));
    }
  }
}
// b - 2 * (sum of the unit's weights), in fp64 and in the inputs' order: one thread a hidden unit
__global__ __launch_bounds__(64) void mlp_pack_bias_kernel(const float* w1, const float* b1, int D, int H, float* out) {
  const int j = blockIdx.x * 64 + threadIdx.x;
  double sum = 0.0;
#pragma unroll 32
  for (int d = 0; d < D; ++d) sum += (double)w1[(int64_t)d * H + j];
  out[j] = (float)((double)b1[j] - 2.0 * sum);
}

// ---------------------------------------------------------------- launchers
void launch_mlp_pack(const MlpArgs& a, int i, double scale, hipStream_t s) {
  const int D = a.d_in[i], H = a.hidden[i];
  hipLaunchKernelGGL(mlp_pack_kernel, dim3(D / PK_D, H / PK_H), dim3(256), 0, s, a.w1_canon[i], D, H, scale,
                     const_cast<float*>(a.w1_f32[i]), (uint16_t*)a.w1_bf[i], (uint16_t*)a.w1_s3[i]);
  hipLaunchKernelGGL(mlp_pack_bias_kernel, dim3(H / 64), dim3(64), 0, s, a.w1_canon[i], a.b1_canon[i], D, H,
                     const_cast<float*>(a.b1_fold[i]));
}

// Tile configurations: 0 = 128x128, 1 = 64x128, 2 = 128x64, 3 = 64x64 (rows x hidden units).
int mlp_tile_bn(int cfg) { return cfg == 0 || cfg == 1 ? 128 : 64; }

// BF16 first pass on bf16 frames (d_in a multiple of 64): 256 queued rows x 128 hidden units per
// tile, eight waves of 64 x 64.  Each k-block (64 elements: 128 bytes of every frame row and
// weight row) is copied global -> LDS with global_load_lds_dwordx4 into a three-stage ring, one
// barrier per k-block; the 16-byte chunks of row r sit at slot chunk ^ (r mod 8), so the MFMA
// operand reads of 16 rows spread over the banks.
constexpr int MD_BM = 256, MD_BN = 128, MD_NS = 3;
__global__ __launch_bounds__(512) void mlp_gemm_dma_kernel(MlpArgs a) {
  constexpr int UPR = 8, ROWB = 128, BKE = 64;             // 16-byte units per row, bytes, elements
  constexpr int UNITS = (MD_BM + MD_BN) * UPR;
  constexpr int NI = UNITS / 512, NIF = MD_BM * UPR / 512; // loads per wave and stage (frames first)
  constexpr int STAGE = UNITS * 16;
  constexpr int WM = 64, WN = 64, MT = WM / 16, NT = WN / 16;
  static_assert(UNITS % 512 == 0 && (MD_BM * UPR) % 512 == 0, "stage rows fill the waves' loads");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[MD_NS * STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, l16 = lane & 15;
  const int wm = wave & 3, wn = wave >> 2;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds);
  const int u_slot = lane % UPR;

  const MlpPlan plan = mlp_plan(a);
  for (int u = blockIdx.x; u < plan.units; u += gridDim.x) {
    const MlpUnit m = mlp_unit(a, plan, u);
    const int slot = m.slot, mt = m.mt, nt = m.nt;
    const int k = a.pred[slot];
    const int cnt = a.q.counts[k];
    const int D = a.d_in[slot];
    const uint32_t* qe = a.q.entries + (int64_t)k * a.q.cap;
    const unsigned long long t0 = wall_clock64();

    // the rows this lane copies: gathered frame rows (rows past the queue re-read its last entry;
    // their results are never stored), then weight rows; element offset of the lane's chunk
    const __bf16* src[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int U = (wave + 8 * i) * 64 + lane;
      if (i < NIF) {
        const int r = U / UPR;
        const int row = mt * MD_BM + r;
        const uint32_t idx = entry_idx(qe[row < cnt ? row : cnt - 1]);
        src[i] = static_cast<const __bf16*>(a.fr.base) + (int64_t)idx * a.fr.elems + (u_slot ^ (r & 7)) * 8;
      } else {
        const int r = U / UPR - MD_BM;
        src[i] = a.w1_bf[slot] + (int64_t)(nt * MD_BN + r) * D + (u_slot ^ (r & 7)) * 8;
      }
    }
    auto issue = [&](int kb, int buf) {
      const uint32_t base = lds0 + buf * STAGE;
#pragma unroll
      for (int i = 0; i < NI; ++i)
        lds_dma16(src[i] + (int64_t)kb * BKE, __builtin_amdgcn_readfirstlane(base + (wave + 8 * i) * 1024));
    };

    floatx4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = (floatx4){0.f, 0.f, 0.f, 0.f};
    // k-step ks (chunk 4 ks + g of each row) of buffer buf, read into registers
    struct Frag { bf16x8 a[MT], b[NT]; };
    auto frags = [&](int buf, int ks, Frag& fr) {
      const unsigned char* F = lds + buf * STAGE;
      const unsigned char* W = F + MD_BM * ROWB;
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int r = wm * WM + i * 16 + l16;
        fr.a[i] = *reinterpret_cast<const bf16x8*>(F + (r * UPR + ((4 * ks + g) ^ (r & 7))) * 16);
      }
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const int r = wn * WN + j * 16 + l16;
        fr.b[j] = *reinterpret_cast<const bf16x8*>(W + (r * UPR + ((4 * ks + g) ^ (r & 7))) * 16);
      }
    };
    auto mma = [&](const Frag& fr) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr.a[i], fr.b[j], acc[i][j], 0, 0, 0);
    };

    const int kt0 = m.kb0, kt1 = m.kb1;
    const int nkb = kt1 - kt0;
    // Ring of MD_NS k-blocks (k-block kb in buffer kb % MD_NS).  Fragments are read one MFMA step
    // ahead, and the barrier that publishes k-block kb + 1 and frees buffer kb sits between a
    // k-block's two steps: every wave reaches it with MFMAs in its pipe.  (The previous tile's last
    // barrier ordered every read of the ring.)
#pragma unroll
    for (int s0 = 0; s0 < MD_NS; ++s0)
      if (s0 < nkb) issue(kt0 + s0, s0);
    if (nkb >= 3) wait_vmcnt<2 * NI>();
    else if (nkb == 2) wait_vmcnt<NI>();
    else wait_vmcnt<0>();
    __syncthreads();
    Frag F0, F1;
    frags(0, 0, F0);
    int buf = 0;
#pragma unroll 1
    for (int kb = 0; kb < nkb; ++kb) {
      frags(buf, 1, F1);
      mma(F0);
      if (kb + 2 < nkb) wait_vmcnt<NI>();   // k-block kb + 1 landed; kb + 2 may stay in flight
      else wait_vmcnt<0>();
      __syncthreads();
      if (kb + MD_NS < nkb) issue(kt0 + kb + MD_NS, buf);
      buf = buf + 1 == MD_NS ? 0 : buf + 1;
      frags(buf, 0, F0);                     // the next k-block's first step (unused after the last)
      mma(F1);
    }

    mlp_finish<MD_BM, MD_BN, MT, NT>(a, m, acc, wm * WM, wn * WN);
    __syncthreads();
    if (tid == 0 && a.count_ticks) atomicAdd(&a.st->r_ticks[k], (unsigned long long)(wall_clock64() - t0));
  }
}

// FP32 arithmetic on bf16 frames (the FP32 tier, and an FP32 first pass): every fp32 weight w is
// split into three bf16 terms w = hi + mid + lo (each the bf16 rounding of what is left; three
// terms carry all 24 bits of the fp32 significand), so x * w = x * hi + x * mid + x * lo with
// every product exact (a bf16 x bf16 product fits fp32) and fp32 accumulation: the fp32 GEMM's
// result up to summation order, from three bf16 MFMAs instead of eight fp32 ones (16x16x32 bf16
// against 16x16x4 fp32).  The hi products are summed apart from the others,
// which are 2^-8 of them and less, and in runs of M3_RUN k-blocks: few roundings fall on the whole sum, and
// the error does not hang on how many parts a tile is split in (2,048 rows of 12,288 inputs x 512 units:
// rms 1.7e-6 with one running sum in four parts, 0.33e-6 so; 0.55e-6 with runs of all three terms).
// 128 x 128 tiles, four waves of 64 x 64, k-blocks of 64 elements (the
// frame rows, then the hi, mid and lo weight rows) in a two-stage direct-to-LDS ring.
constexpr int M3_BM = 128, M3_BN = 128, M3_NS = 2, M3_RUN = 4;
__global__ __launch_bounds__(256) void mlp_gemm_s3_kernel(MlpArgs a) {
  constexpr int UPR = 8, ROWB = 128, BKE = 64;
  constexpr int UNITS = (M3_BM + 3 * M3_BN) * UPR;
  constexpr int NI = UNITS / 256, NIF = M3_BM * UPR / 256;   // loads per wave and stage (frames first)
  constexpr int STAGE = UNITS * 16;
  constexpr int WM = 64, WN = 64, MT = WM / 16, NT = WN / 16;
  static_assert(UNITS % 256 == 0 && (M3_BM * UPR) % 256 == 0, "stage rows fill the waves' loads");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[M3_NS * STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, l16 = lane & 15;
  const int wm = wave >> 1, wn = wave & 1;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds);
  const int u_slot = lane % UPR;

  const MlpPlan plan = mlp_plan(a);
  for (int u = blockIdx.x; u < plan.units; u += gridDim.x) {
    const MlpUnit m = mlp_unit(a, plan, u);
    const int slot = m.slot, mt = m.mt, nt = m.nt;
    const int k = a.pred[slot];
    const int cnt = a.q.counts[k];
    const int D = a.d_in[slot], H = a.hidden[slot];
    const uint32_t* qe = a.q.entries + (int64_t)k * a.q.cap;
    const unsigned long long t0 = wall_clock64();

    const __bf16* src[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int U = (wave + 4 * i) * 64 + lane;
      if (i < NIF) {
        const int r = U / UPR;
        const int row = mt * M3_BM + r;
        const uint32_t idx = entry_idx(qe[row < cnt ? row : cnt - 1]);
        src[i] = static_cast<const __bf16*>(a.fr.base) + (int64_t)idx * a.fr.elems + (u_slot ^ (r & 7)) * 8;
      } else {
        const int r = U / UPR - M3_BM;                   // 0 .. 3 * BN - 1: term r / BN, row r % BN
        const int term = r / M3_BN, rr = r % M3_BN;
        src[i] = a.w1_s3[slot] + ((int64_t)term * H + nt * M3_BN + rr) * D + (u_slot ^ (rr & 7)) * 8;
      }
    }
    auto issue = [&](int kb, int buf) {
      const uint32_t base = lds0 + buf * STAGE;
#pragma unroll
      for (int i = 0; i < NI; ++i)
        lds_dma16(src[i] + (int64_t)kb * BKE, __builtin_amdgcn_readfirstlane(base + (wave + 4 * i) * 1024));
    };

    // sum: of the hi products of the runs so far; acc: of the current run's; low: of all mid and lo products
    floatx4 acc[MT][NT], sum[MT][NT], low[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) sum[i][j] = low[i][j] = (floatx4){0.f, 0.f, 0.f, 0.f};
    auto compute = [&](int buf) {
      const unsigned char* F = lds + buf * STAGE;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        bf16x8 af[MT];
#pragma unroll
        for (int i = 0; i < MT; ++i) {
          const int r = wm * WM + i * 16 + l16;
          af[i] = *reinterpret_cast<const bf16x8*>(F + (r * UPR + ((4 * ks + g) ^ (r & 7))) * 16);
        }
        // smallest terms first: the three partial products enter each sum in the order lo, mid, hi
#pragma unroll
        for (int term = 2; term >= 0; --term) {
          const unsigned char* W = F + (M3_BM + term * M3_BN) * ROWB;
          bf16x8 bfr[NT];
#pragma unroll
          for (int j = 0; j < NT; ++j) {
            const int r = wn * WN + j * 16 + l16;
            bfr[j] = *reinterpret_cast<const bf16x8*>(W + (r * UPR + ((4 * ks + g) ^ (r & 7))) * 16);
          }
#pragma unroll
          for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) {
              floatx4& c = term == 0 ? acc[i][j] : low[i][j];
              c = mfma_bf16(af[i], bfr[j], c);
            }
        }
      }
    };

    const int kt0 = m.kb0, kt1 = m.kb1;
    const int nkb = kt1 - kt0;
    // two stages: block kb + 1 is copied while block kb is read; the barrier at the top of each
    // iteration also retires every wave's reads of the buffer the next copy overwrites
    if (nkb > 0) issue(kt0, 0);
#pragma unroll 1
    for (int k0 = 0; k0 < nkb; k0 += M3_RUN) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = (floatx4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < M3_RUN; ++u) {
        const int kb = k0 + u;
        if (u > 0 && kb >= nkb) break;
        wait_vmcnt<0>();
        __syncthreads();
        if (kb + 1 < nkb) issue(kt0 + kb + 1, (kb + 1) & 1);
        compute(kb & 1);
      }
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) sum[i][j] += acc[i][j];
    }

#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) sum[i][j] += low[i][j];
    mlp_finish<M3_BM, M3_BN, MT, NT>(a, m, sum, wm * WM, wn * WN);
    __syncthreads();
    if (tid == 0 && a.count_ticks) atomicAdd(&a.st->r_ticks[k], (unsigned long long)(wall_clock64() - t0));
  }
}

template <typename T, int BM, int BN>
static void launch_gemm_t(MlpArgs& b, hipStream_t s) {
  b.bm = BM;
  b.bn = BN;
  b.bk = MlpTile<T>::BK;
  b.units = 2 * b.n_cu;          // workgroups that the kernel's registers let in: two or three per CU
  const dim3 grid(b.units * 4);
  if (b.fr.dtype == HYDRO_DTYPE_BF16)
    hipLaunchKernelGGL((mlp_gemm_kernel<T, __bf16, BM, BN>), grid, dim3(256), 0, s, b);
  else if (b.fr.dtype == HYDRO_DTYPE_U8)
    hipLaunchKernelGGL((mlp_gemm_kernel<T, uint8_t, BM, BN>), grid, dim3(256), 0, s, b);
  else
    hipLaunchKernelGGL((mlp_gemm_kernel<T, float, BM, BN>), grid, dim3(256), 0, s, b);
}

// Picks and launches the GEMM; the tile shape it used is left in b for the head.
void launch_mlp_gemm(MlpArgs& b, int cfg, bool bf, hipStream_t s) {
  bool dma = bf && b.fr.dtype == HYDRO_DTYPE_BF16 && (cfg == 0 || cfg == 1);
  for (int i = 0; i < b.n_preds && dma; ++i) dma = b.d_in[i] % 64 == 0 && b.hidden[i] % MD_BN == 0;
  bool s3 = !bf && b.fr.dtype == HYDRO_DTYPE_BF16 && (cfg == 0 || cfg == 1);
  for (int i = 0; i < b.n_preds && s3; ++i) s3 = b.w1_s3[i] != nullptr;
  if (s3 || dma) {
    b.bm = s3 ? M3_BM : MD_BM;
    b.bn = s3 ? M3_BN : MD_BN;
    b.bk = 64;
    b.units = b.n_cu;            // the ring takes a CU's LDS
    b.split_slots = (int)((int64_t)b.split_slots * 128 * 128 / (b.bm * b.bn));
    if (s3) hipLaunchKernelGGL(mlp_gemm_s3_kernel, dim3(b.units * 4), dim3(256), 0, s, b);
    else hipLaunchKernelGGL(mlp_gemm_dma_kernel, dim3(b.units * 4), dim3(512), 0, s, b);
  } else if (bf) {
    if (cfg == 0) launch_gemm_t<__bf16, 128, 128>(b, s);
    else if (cfg == 1) launch_gemm_t<__bf16, 64, 128>(b, s);
    else if (cfg == 2) launch_gemm_t<__bf16, 128, 64>(b, s);
    else launch_gemm_t<__bf16, 64, 64>(b, s);
  } else {
    if (cfg == 0) launch_gemm_t<float, 128, 128>(b, s);
    else if (cfg == 1) launch_gemm_t<float, 64, 128>(b, s);
    else if (cfg == 2) launch_gemm_t<float, 128, 64>(b, s);
    else launch_gemm_t<float, 64, 64>(b, s);
  }
}

void mlp_copy_slot(MlpArgs& dst, int j, const MlpArgs& src, int i) {
  dst.pred[j] = src.pred[i];
  dst.d_in[j] = src.d_in[i];
  dst.hidden[j] = src.hidden[i];
  dst.class_mask[j] = src.class_mask[i];
  dst.w1_bf[j] = src.w1_bf[i];
  dst.w1_f32[j] = src.w1_f32[i];
  dst.w1_s3[j] = src.w1_s3[i];
  dst.b1_fold[j] = src.b1_fold[i];
  dst.w2[j] = src.w2[i];
  dst.b2[j] = src.b2[i];
  dst.w1_canon[j] = src.w1_canon[i];
  dst.b1_canon[j] = src.b1_canon[i];
  dst.partial[j] = src.partial[i];
  dst.part_w[j] = src.part_w[i];
  dst.tile_cfg[j] = src.tile_cfg[i];
  dst.esc_h[j] = src.esc_h[i];
}

void launch_mlp_pass(const MlpArgs& a, const Forward& f, int tier, int grid, hipStream_t s) {
  if (a.n_preds == 0) return;
  if (tier == TIER_F64) {
    hipLaunchKernelGGL(mlp_f64_hidden_kernel, dim3(grid * 2), dim3(256), 0, s, a);
    hipLaunchKernelGGL(mlp_f64_entry_kernel, dim3(grid), dim3(256), 0, s, a, f);
    return;
  }
  // one GEMM and head launch per tile shape present among the predicates
  const bool bf = a.prec == HYDRO_PREC_BF16 && tier == TIER_FIRST;
  for (int cfg = 0; cfg < MLP_TILE_CONFIGS; ++cfg) {
    MlpArgs b = a;
    b.n_preds = 0;
    for (int i = 0; i < a.n_preds; ++i) {
      if (a.tile_cfg[i] != cfg) continue;
      mlp_copy_slot(b, b.n_preds++, a, i);
    }
    if (b.n_preds == 0) continue;
    launch_mlp_gemm(b, cfg, bf, s);
    hipLaunchKernelGGL(mlp_head_kernel, dim3(grid), dim3(256), 0, s, b, f);
  }
}

}  // namespace hydro
