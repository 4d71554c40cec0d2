// FP64 tier of the CNN predicates (the fused 64x64 shapes, the 4-layer 128x128 shape and the layer-wise
// ones alike): the frame normalised in FP64 exactly as defined, the canonical (unfolded) fp32
// weights widened to FP64, FP64 accumulation on matrix instructions (conv64.h).  Decisions made
// here are final.
//
// The first esc_cap escalated entries of each predicate are spread over the whole GPU, one launch
// per layer (a round escalates a handful at most, so latency is what counts: one tile of 16
// positions x 16 channels per workgroup, whose four waves split the sum); any entries beyond
// that (band calibration runs every sample frame here) take one 16-wave workgroup each, all
// layers in one launch.
//
// Bound by the FP64 matrix rate (76 TFLOP/s measured with registers alone) and by the waits between the
// layers of a frame: 1,024 frames through the 64-128-256 CNN (81 GFLOP) take 1.69 + 0.17 ms (entries
// beyond esc_cap, layers of the others), 44 TFLOP/s; 1.99 + 0.22 ms with weights [co][tap][ci] and NHWC
// activations, whose loads took the address units longer than the MFMAs.  Calibrating three CNNs this
// way is 3.0 ms of a one-shot query of 2,048 frames; with one scalar product chain per thread it was
// 118 of 139 ms.
#include <algorithm>

#include "conv64.h"

namespace hydro {

constexpr int F64_LAYER_THREADS = 256;
constexpr int F64_WG_THREADS = 1024;

__device__ inline Conv64 f64_layer(const F64Args& a, int slot, int l) {
  Conv64 L;
  L.w = a.wt[slot][l];
  L.bias = a.bias[slot][l];
  L.cin = l == 0 ? 3 : a.widths[slot][l - 1];
  L.cout = L.cstore = a.widths[slot][l];
  L.hin = L.win = a.in_hw[slot] >> l;
  L.ho = L.wo = L.hin >> 1;
  L.last = l == a.n_layers[slot] - 1;
  return L;
}

// Work units of one entry's layer: 16 channels x 64 positions (layer 1, a 16-position tile per wave)
// or x 16 positions (later layers, the waves split the sum).
__device__ inline int f64_units(const Conv64& L, int layer) {
  const int pt = (L.ho * L.wo + 15) >> 4;
  return (layer == 0 ? (pt + 3) >> 2 : pt) * (L.cout >> 4);
}

__global__ __launch_bounds__(F64_LAYER_THREADS) void f64_layer_kernel(F64Args a, int layer) {
  __shared__ double red[4][4][64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int64_t total = 0;
  for (int i = 0; i < a.n_preds; ++i) {
    if (layer >= a.n_layers[i]) continue;
    total += (int64_t)min(a.q.counts[a.pred[i]], a.esc_cap) * f64_units(f64_layer(a, i, layer), layer);
  }
  for (int64_t u = blockIdx.x; u < total; u += gridDim.x) {
    int slot = 0, units = 1;
    int64_t rem = u;
    for (int i = 0; i < a.n_preds; ++i) {
      if (layer >= a.n_layers[i]) continue;
      units = f64_units(f64_layer(a, i, layer), layer);
      const int64_t c = (int64_t)min(a.q.counts[a.pred[i]], a.esc_cap) * units;
      if (rem < c) { slot = i; break; }
      rem -= c;
    }
    const Conv64 L = f64_layer(a, slot, layer);
    const int e = (int)(rem / units), un = (int)(rem % units);
    const int ct = L.cout >> 4, o0 = (un % ct) * 16, pu = un / ct;
    double* act = a.esc_act[slot] + (int64_t)e * a.esc_stride;
    double* out = act + ((layer & 1) ? a.esc_off : 0);
    doublex4 acc[1] = {(doublex4){0.0, 0.0, 0.0, 0.0}};
    if (layer == 0) {
      const uint32_t idx = entry_idx(a.q.entries[(int64_t)a.pred[slot] * a.q.cap + e]);
      const int p0 = (pu * 4 + wave) * 16;
      conv64_acc<CONV64_FIRST, 1>(L, image64(a.fr, idx, L.win, 0, 0), nullptr, p0, o0, 0, 1, acc);
      conv64_store<1>(L, acc, out, p0, o0);
      continue;
    }
    const double* in = act + ((layer & 1) ? 0 : a.esc_off);
    const int nb = conv64_blocks(L, CONV64_WIDE), p0 = pu * 16;
    conv64_acc<CONV64_WIDE, 1>(L, Image64{}, in, p0, o0, nb * wave / 4, nb * (wave + 1) / 4, acc);
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][r][lane] = acc[0][r];
    __syncthreads();
    // wave w finishes register w of every lane: channel 4 (lane / 16) + w
    const int ch = o0 + 4 * (lane >> 4) + wave, p = p0 + (lane & 15);
    const double s = ((red[0][wave][lane] + red[1][wave][lane]) + (red[2][wave][lane] + red[3][wave][lane])) +
                     (double)L.bias[ch];
    if (p < L.ho * L.wo) out[conv64_at(L, p / L.wo, p % L.wo, ch)] = s > 0.0 ? s : 0.0;
    __syncthreads();           // red is rewritten by the next unit
  }
}

// Pool, FC, margin and decision of every escalated entry, one workgroup per entry; entries beyond
// esc_cap run their layers here first, in this block's scratch.
__global__ __launch_bounds__(F64_WG_THREADS) void f64_entry_kernel(F64Args a, Forward f) {
  __shared__ double part[F64_WG_THREADS], g[F64_WG_THREADS], z[kClasses];
  const int wave = threadIdx.x >> 6;
  int total = 0;
  for (int i = 0; i < a.n_preds; ++i) total += a.q.counts[a.pred[i]];
  for (int t = blockIdx.x; t < total; t += gridDim.x) {
    int slot = 0, off = t;
    for (int i = 0; i < a.n_preds; ++i) {
      const int c = a.q.counts[a.pred[i]];
      if (off < c) { slot = i; break; }
      off -= c;
    }
    const int k = a.pred[slot], nl = a.n_layers[slot];
    const uint32_t e = a.q.entries[(int64_t)k * a.q.cap + off];
    const uint32_t idx = entry_idx(e);
    const double* act;
    if (off < a.esc_cap) {
      act = a.esc_act[slot] + (int64_t)off * a.esc_stride + (((nl - 1) & 1) ? a.esc_off : 0);
    } else {
      double* buf = a.scratch + (int64_t)blockIdx.x * a.per_block;
      for (int l = 0; l < nl; ++l) {
        const Conv64 L = f64_layer(a, slot, l);
        double* out = buf + ((l & 1) ? a.scratch_off : 0);
        const double* in = buf + ((l & 1) ? 0 : a.scratch_off);
        if (l == 0) conv64_wg<CONV64_FIRST>(L, image64(a.fr, idx, L.win, 0, 0), nullptr, out, wave, F64_WG_THREADS / 64);
        else conv64_wg<CONV64_WIDE>(L, Image64{}, in, out, wave, F64_WG_THREADS / 64);
        __syncthreads();
      }
      act = buf + (((nl - 1) & 1) ? a.scratch_off : 0);
    }
    const int hl = a.in_hw[slot] >> nl, C = a.widths[slot][nl - 1];
    head64_wg<F64_WG_THREADS>(act, hl * hl, C, C, a.fc_w[slot], a.fc_b[slot], part, g, z);
    if (wave == 0) {
      const bool lead = threadIdx.x == 0;
      bool pass = false;
      if (lead) {
        if (f.logits != nullptr)
          for (int c = 0; c < kClasses; ++c) f.logits[(int64_t)idx * kClasses + c] = z[c];
        pass = class_margin(z, a.class_mask[slot]) > (double)theta_of(f, k, idx);
      }
      if (f.logits == nullptr) forward_decision(f, k, e, lead, false, pass);
    }
    __syncthreads();           // z and the scratch are reused by the next entry
  }
}

// Per 16 output channels, 16-channel block of the sum (tap outermost) and lane (g, l16): channels
// 4g..4g+3 of weight row 4 (l16 % 4) + l16 / 4.  First layer, and layers of fewer than 16 input channels, per 16
// output channels and lane: products 4q + g of the (tap, channel)s, q = 0, 1, ....
std::vector<float> conv64_pack(const float* w, int cin, int cout, bool first) {
  const bool dense = first || cin < 16;
  const int ct = crop_pad(cout) / 16, nc = crop_pad(cin) / 16;
  const int nb = dense ? 1 : 9 * nc, per = dense ? conv64_narrow_steps(cin) : 4;
  std::vector<float> out((size_t)ct * nb * 64 * per, 0.f);
  // weight row of lane l16 in channel tile c: [channel][tap] (nullptr: a padded one)
  auto row = [&](int c, int l16) {
    const int o = c * 16 + 4 * (l16 & 3) + (l16 >> 2);
    return o < cout ? w + (size_t)o * cin * 9 : nullptr;
  };
  for (int c = 0; c < ct; ++c) {
    float* d = out.data() + (size_t)c * nb * 64 * per;
    if (dense) {
      for (int l16 = 0; l16 < 16; ++l16)
        if (const float* r = row(c, l16))
          for (int t = 0, k = 0; t < 9; ++t)
            for (int ch = 0; ch < cin; ++ch, ++k) d[((k & 3) * 16 + l16) * per + (k >> 2)] = r[ch * 9 + t];
      continue;
    }
    const float* rows[16];
    for (int l16 = 0; l16 < 16; ++l16) rows[l16] = row(c, l16);
    for (int t = 0; t < 9; ++t)
      for (int c0 = 0; c0 < cin; c0 += 4) {
        float* e = d + ((size_t)(t * nc + (c0 >> 4)) * 64 + (c0 >> 2 & 3) * 16) * 4;
        if (c0 + 4 <= cin && rows[15] != nullptr) {          // (the rows of a tile that is not full end with the last)
          for (int l16 = 0; l16 < 16; ++l16, e += 4)
            for (int q = 0; q < 4; ++q) e[q] = rows[l16][(c0 + q) * 9 + t];
          continue;
        }
        for (int l16 = 0; l16 < 16; ++l16, e += 4)
          for (int q = 0; rows[l16] != nullptr && q < std::min(4, cin - c0); ++q) e[q] = rows[l16][(c0 + q) * 9 + t];
      }
  }
  return out;
}

void launch_f64_cnn(const F64Args& a, const Forward& f, int grid, hipStream_t s) {
  int nl = 0;
  for (int i = 0; i < a.n_preds; ++i) nl = a.n_layers[i] > nl ? a.n_layers[i] : nl;
  for (int l = 0; l < nl; ++l) hipLaunchKernelGGL(f64_layer_kernel, dim3(grid * 4), dim3(F64_LAYER_THREADS), 0, s, a, l);
  hipLaunchKernelGGL(f64_entry_kernel, dim3(a.rest_grid), dim3(F64_WG_THREADS), 0, s, a, f);
}

}  // namespace hydro
