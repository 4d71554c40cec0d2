// CNN predicates on variable-size inputs: each tuple's crop (y0, x0, h, w) of its frame (the UDF
// composition of section 5.3, a classifier applied to Crop(frame, bbox)).  Evaluated in FP64 (the
// decisions are final), one workgroup per tuple, so the work of a tuple follows its crop's area.
// How a round's tuples are dealt to the workgroups is the data-aware load balancing of section
// 5.3: in queue order (each workgroup takes every gridDim-th tuple), or largest estimated work
// first (the crop's area, the paper's input-size heuristic) from a shared counter, so that no
// workgroup is left with a long tail of large crops.
//
// The convolutions run on FP64 matrix instructions (conv64.h).  65,536 crops of 64x64 frames, sides
// log-uniform 2..64, 16-32-64 CNN, largest first: 2.40 ms of kernel time (36 GFLOP; about twice that
// with the last tile of each layer filled up, most crops being smaller than a tile in layers 2 and
// 3; matrix cores busy 41 % of it, the rest is the chain of short layers), against 12.9 ms with one
// output per thread.  Query 13.85 -> 2.84 ms.  (Looking the next item up during the current one,
// forwarding decisions in batches, or requesting blocks ahead of their MFMAs changed nothing.)
#include "conv64.h"

namespace hydro {

constexpr int kCropThreads = 256;
constexpr int kOrderThreads = 1024;
constexpr int kCropBuckets = 256;
// Activations of a crop that fit this many doubles (both ping-pong buffers: square crops up to 24 x 24
// with the 16-32-64 widths, four in five of a log-uniform side distribution) stay in LDS; 32 KB
// each leaves room for four workgroups per CU.
constexpr int kCropLds = 4096;

// One workgroup per crop predicate slot: queue positions in decreasing order of crop area
// (bucketed: area * 255 / frame area), and the work counter of the following launch reset.  Bound
// by the latency of its gathers (entry, then crop): 16 waves and unrolled loops keep them in flight.
__global__ __launch_bounds__(kOrderThreads) void k_crop_order(CropArgs a) {
  __shared__ int hist[kCropBuckets];
  const int slot = blockIdx.x;
  const int k = a.pred[slot];
  const int c = a.q.counts[k];
  const int full = a.fh * a.fw;
  const uint32_t* ent = a.q.entries + (int64_t)k * a.q.cap;
  const int2* crops = reinterpret_cast<const int2*>(a.crops);
  if (threadIdx.x < kCropBuckets) hist[threadIdx.x] = 0;
  if (slot == 0 && threadIdx.x == 0) *a.next = 0;
  __syncthreads();
  auto bucket = [&](int i) {
    const int2 hw = crops[(int64_t)entry_idx(ent[i]) * 2 + 1];
    return (kCropBuckets - 1) - (int)((int64_t)hw.x * hw.y * (kCropBuckets - 1) / full);   // larger area, smaller bucket
  };
#pragma unroll 4
  for (int i = threadIdx.x; i < c; i += kOrderThreads) atomicAdd(&hist[bucket(i)], 1);
  __syncthreads();
  if (threadIdx.x < kWave) {            // exclusive scan of the 256 counts, four per lane
    const int lane = threadIdx.x;
    int v[4], sum = 0;
    for (int u = 0; u < 4; ++u) {
      v[u] = sum;
      sum += hist[4 * lane + u];
    }
    int inc = sum;
    for (int o = 1; o < kWave; o <<= 1) {
      const int up = __shfl_up(inc, o);
      if (lane >= o) inc += up;
    }
    for (int u = 0; u < 4; ++u) hist[4 * lane + u] = inc - sum + v[u];
  }
  __syncthreads();
  uint32_t* ord = a.order + (int64_t)slot * a.q.cap;
#pragma unroll 4
  for (int i = threadIdx.x; i < c; i += kOrderThreads) ord[atomicAdd(&hist[bucket(i)], 1)] = (uint32_t)i;
}

// All layers of one crop; the activations ping-pong between buf and buf + off.  Returns the last
// layer's output.
__device__ inline const double* crop_layers(const CropArgs& a, int slot, const Image64& im, int h, int w, double* buf,
                                            int64_t off, int wave) {
  Conv64 L;
  L.cin = 3;
  L.hin = h;
  L.win = w;
  const int nl = a.n_layers[slot];
  for (int l = 0; l < nl; ++l) {
    L.w = a.wt[slot][l];
    L.bias = a.bias[slot][l];
    const int width = a.widths[slot][l];
    L.cout = crop_pad(width);
    L.cstore = crop_store(width);
    L.ho = (L.hin + 1) / 2;
    L.wo = (L.win + 1) / 2;
    L.last = l == nl - 1;
    double* out = buf + ((l & 1) ? off : 0);
    const double* in = buf + ((l & 1) ? 0 : off);
    if (l == 0) conv64_wg<CONV64_FIRST>(L, im, nullptr, out, wave, kCropThreads / 64);
    else if (L.cin < 16) conv64_wg<CONV64_NARROW>(L, im, in, out, wave, kCropThreads / 64);
    else conv64_wg<CONV64_WIDE>(L, im, in, out, wave, kCropThreads / 64);
    __syncthreads();
    L.hin = L.ho;
    L.win = L.wo;
    L.cin = width < 16 ? width : L.cout;
  }
  return buf + (((nl - 1) & 1) ? off : 0);
}

// Four workgroups per CU: 122 VGPRs; left to itself the compiler takes 132, which lets in three
// (query 3.47 against 3.09 ms, before weights and activations were laid out for coalesced loads).
__global__ __launch_bounds__(kCropThreads, 4) void k_crop_cnn(CropArgs a, Forward f) {
  __shared__ __attribute__((aligned(32))) double act_s[kCropLds];
  __shared__ double part[kCropThreads], g_s[256], z_s[kClasses];
  __shared__ int item_s;
  const int tid = threadIdx.x, wave = tid >> 6;
  int total = 0;
  for (int i = 0; i < a.n_preds; ++i) total += a.q.counts[a.pred[i]];
  double* buf = a.scratch + (int64_t)blockIdx.x * 2 * a.act_doubles;
  for (int t0 = blockIdx.x;; t0 += gridDim.x) {
    // the next work item: the queue's t0-th (queue order) or the counter's (largest first)
    if (a.balance) {
      if (tid == 0) item_s = atomicAdd(a.next, 1);
      __syncthreads();
    }
    const int t = a.balance ? item_s : t0;
    if (t >= total) break;
    int slot = 0, off = t;
    for (int i = 0; i < a.n_preds; ++i) {
      const int c = a.q.counts[a.pred[i]];
      if (off < c) { slot = i; break; }
      off -= c;
    }
    const int k = a.pred[slot];
    const int pos = a.balance ? (int)a.order[(int64_t)slot * a.q.cap + off] : off;
    const uint32_t e = a.q.entries[(int64_t)k * a.q.cap + pos];
    const uint32_t idx = entry_idx(e);
    const unsigned long long c0 = wall_clock64();
    const int4 box = reinterpret_cast<const int4*>(a.crops)[idx];     // y0, x0, h, w
    const Image64 im = image64(a.fr, idx, a.fw, box.x, box.y);
    // doubles that the even and the odd layers' outputs take
    int need0 = 0, need1 = 0, hl = box.z, wl = box.w;
    for (int l = 0; l < a.n_layers[slot]; ++l) {
      hl = (hl + 1) / 2;
      wl = (wl + 1) / 2;
      const int n = (int)conv64_doubles(hl, wl, crop_store(a.widths[slot][l]), l == a.n_layers[slot] - 1);
      if (l & 1) need1 = max(need1, n);
      else need0 = max(need0, n);
    }
    const int C = a.widths[slot][a.n_layers[slot] - 1];
    if (need0 + need1 <= kCropLds) {
      const double* act = crop_layers(a, slot, im, box.z, box.w, act_s, need0, wave);
      head64_wg<kCropThreads>(act, hl * wl, C, crop_store(C), a.fc_w[slot], a.fc_b[slot], part, g_s, z_s);
    } else {
      const double* act = crop_layers(a, slot, im, box.z, box.w, buf, a.act_doubles, wave);
      head64_wg<kCropThreads>(act, hl * wl, C, crop_store(C), a.fc_w[slot], a.fc_b[slot], part, g_s, z_s);
    }
    if (tid < kWave) {
      const double d = class_margin(z_s, a.class_mask[slot]);
      const bool pass = d > (double)theta_of(f, k, idx);
      forward_decision(f, k, e, tid == 0, false, pass);
      if (tid == 0 && f.count_eval) atomicAdd(&a.st->r_ticks[k], (unsigned long long)(wall_clock64() - c0));
    }
    __syncthreads();          // item_s, z_s and the buffers are reused by the next item
  }
}

void launch_crop_pass(const CropArgs& a, const Forward& f, int grid, hipStream_t s) {
  if (a.n_preds == 0) return;
  if (a.balance) hipLaunchKernelGGL(k_crop_order, dim3(a.n_preds), dim3(kOrderThreads), 0, s, a);
  hipLaunchKernelGGL(k_crop_cnn, dim3(grid), dim3(kCropThreads), 0, s, a, f);
}

}  // namespace hydro
