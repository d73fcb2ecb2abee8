// Fused LM head + confidence for gfx950.
//
// For each scored hidden row n the kernels form z[v] = <H[row_idx[n]], W[v]>
// on bf16 MFMA with fp32 accumulation and reduce every vocabulary tile to a
// (max m, sum s = sum exp(z - m), first argmax) triple in registers, so the
// logits never reach memory (paper Section 3.2: confidence-based transfer
// uses the max-probability token of each masked position; refine lanes
// suppress EOS).
//
// lmhead_tile_kernel (lmhead_tile.h) writes one partial (m, s, argmax) per
// column and vocabulary tile; lmhead_merge_kernel combines them in a fixed
// order, so results are bitwise reproducible.  (A single-kernel merge by the
// last workgroup to arrive needs agent-scope fences, which on gfx950 write
// back and invalidate the L2 in every workgroup; the separate launch is
// cheaper.)
#include <math.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <mutex>

#include "../../include/asynclane.h"
#include "common.h"
#include "launch.h"
#include "lmhead.h"

namespace al {

// One 256-thread workgroup per scored row.  Thread t merges vocab-tile
// partials t, t+256, ... in ascending order (loads issued four at a time so
// they overlap), then a fixed xor butterfly combines the lanes of each
// wavefront and wavefront 0 combines the four wavefront results in order.
constexpr int LM_MERGE_THREADS = 256;
__global__ __launch_bounds__(LM_MERGE_THREADS) void lmhead_merge_kernel(
    const LmPartial* part, int N, int n_vt, int nt_cols, float* conf, int32_t* argmax, float* lse) {
  __shared__ float sm[LM_MERGE_THREADS / kWave], ss[LM_MERGE_THREADS / kWave];
  __shared__ int si[LM_MERGE_THREADS / kWave];
  const int n = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = tid >> 6;
  const int nt = n / nt_cols;
  const int col = n - nt * nt_cols;
  const LmPartial* base = part + ((size_t)nt * nt_cols + col) * n_vt;
  float m = -INFINITY, s = 0.f;
  int idx = 0x7fffffff;
  for (int v0 = tid; v0 < n_vt; v0 += 4 * LM_MERGE_THREADS) {
    LmPartial q[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int v = v0 + j * LM_MERGE_THREADS;
      q[j] = base[min(v, n_vt - 1)];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (v0 + j * LM_MERGE_THREADS < n_vt) merge_state(m, s, idx, q[j].m, q[j].s, q[j].idx);
  }
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1)
    merge_state(m, s, idx, __shfl_xor(m, o, kWave), __shfl_xor(s, o, kWave), __shfl_xor(idx, o, kWave));
  if (lane == 0) {
    sm[w] = m;
    ss[w] = s;
    si[w] = idx;
  }
  __syncthreads();
  if (tid == 0) {
    for (int ww = 1; ww < LM_MERGE_THREADS / kWave; ++ww) merge_state(m, s, idx, sm[ww], ss[ww], si[ww]);
    conf[n] = 1.0f / s;
    argmax[n] = idx;
    if (lse) lse[n] = m + logf(s);
  }
}

// ------------------------------------------------------------------ host
// Compute units of the current device (cached per device).
static int lm_cu_count() {
  static int cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cached[dev] <= 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}


// One layout: tiles of 64 ra vocabulary rows x 16 cbt columns.
struct LmLayout {
  int ra, cbt, n_vt, n_nt;
  LmVariant var;
  size_t bytes() const { return sizeof(LmPartial) * (size_t)n_nt * n_vt * 16 * cbt; }
};

constexpr struct {
  int ra, cbt;
} kLmInstances[] = {
#define AL_LM_X(RA, CBT) {RA, CBT},
    AL_LM_INSTANCES(AL_LM_X)
#undef AL_LM_X
};

// Workspace bytes.  The bound is a tiling by 256 or 512 vocabulary rows x nf <= 7
// fragments of 32 columns, with the tiles rounded up to a multiple of the CU
// count: callers keep workspaces of these sizes, and they decide which calls
// the fixed array of lmhead_confidence_noalloc takes.  Smaller tiles for small
// vocabularies may take more, up to that array's size.  Both grow with N, so
// a workspace made for N rows serves every smaller call.  Some layout always
// fits: the instance of that tiling's own rows and columns, for each nf.
constexpr bool lm_bound_is_built() {
  for (int nf = 1; nf <= 7; ++nf) {
    bool found = false;
    for (const auto& in : kLmInstances) found |= in.ra == (nf <= 3 ? 8 : 4) && in.cbt == 2 * nf;
    if (!found) return false;
  }
  return true;
}
static_assert(lm_bound_is_built(), "an instance for every column count of the workspace bound");
static size_t lm_tile_bound(int N, int V, bool packed, int cus) {
  const int frags = (N + 31) / 32;
  const bool multi = packed && frags > 7;
  const int n_nt = (frags + (multi ? 4 : 7) - 1) / (multi ? 4 : 7);
  const int nf = (frags + n_nt - 1) / n_nt;
  const int rows = multi || nf <= 3 ? 512 : 256;
  const int base = (int)(((long long)V + rows - 1) / rows);
  int n_vt = base <= cus ? base : cus * ((base + cus - 1) / cus);
  if (packed && n_vt > base) {
    const long long n_hg = (V + 31) / 32, slots = (long long)n_vt * (rows / 32);
    if (8 * n_hg < 7 * slots) n_vt = base;
  }
  return sizeof(LmPartial) * (size_t)n_nt * n_vt * 32 * nf;
}

size_t lmhead_workspace_bytes(int N, int d, int V) {
  (void)d;
  if (N <= 0 || V <= 0) return 0;
  const int cus = lm_cu_count();
  const size_t big = std::max(lm_tile_bound(N, V, false, cus), lm_tile_bound(N, V, true, cus));
  const int units = (V + 31) / 32;
  const size_t tiles = (size_t)std::max(std::min((units + 1) / 2, 2 * cus), (units + 7) / 8);
  const size_t small = sizeof(LmPartial) * tiles * 32 * (size_t)((N + 31) / 32);
  return std::max(big, std::min(small, (size_t)AL_NOALLOC_SCRATCH_BYTES));
}

// The layout of a call: the cheapest under a cost model of the tile kernel,
// among those whose partials fit the workspace.  The model's constants are
// fitted to times of one instance each (MI355X, d = 4096):
// * a 64-element K stage takes 91 + 36 RA + 13 CBT + 8.8 RA CBT ns (V = 2048,
//   one tile per CU: RA, CBT = 1, 2 21 us per call; 1, 13 37; 4, 2 32; 4, 8
//   48; 4, 13 66; 5, 8 57), 1.25 times that when only two stages of W fit
//   the LDS, and up to 1.45 times with every CU busy (V = 126464, N = 614: 4,
//   13 511 us, 4, 16 599, 4, 10 548, 5, 8 566; the clock drops under the
//   power limit), plus ~3 us per tile;
// * W cannot stream faster than ~7 TB/s;
// * the shorter of the two hides under the longer but for ~15%.
// So few columns take the widest vocabulary tiles that fill whole rounds of
// workgroups (V = 152064: RA = 5 at 128 columns 178 us, RA = 4 202; V =
// 126464: RA = 4 170, RA = 5 192), and small vocabularies the smallest tiles
// (V = 16384, N = 32: RA = 1 28 us, 2 36, 4 50).
static LmLayout lm_layout(int N, int d, int V, bool packed) {
  const int cus = lm_cu_count();
  const int units = (V + 31) / 32, frags = (N + 15) / 16;
  const double stages = (d + 63) / 64;
  const double w_bytes = 2.0 * V * d, hbm = w_bytes / 7.0e6;   // us
  const size_t limit = lmhead_workspace_bytes(N, d, V);
  LmLayout best{};
  double best_t = 1e30;
  for (const auto& in : kLmInstances) {
    const LmLayout c{in.ra, in.cbt, (units + 2 * in.ra - 1) / (2 * in.ra), (frags + in.cbt - 1) / in.cbt, {}};
    if (c.bytes() > limit) continue;
    const long long tiles = (long long)c.n_vt * c.n_nt;
    const double rounds = (double)((tiles + cus - 1) / cus);
    // 320 rows x 32 columns: up to two rounds (V = 140000 198 -> 169 us, 81900 109 ->
    // 105, 1 row packed); past them 512-row tiles read better (V = 330000 446 us, 407).
    if (c.ra == 5 && c.cbt == 2 && rounds > 2) continue;
    const double busy = std::min(1.0, (double)tiles / cus);
    const bool two = 3 * c.ra * 8192 + 2 * c.cbt * 2048 > 160 * 1024;
    const double stage = 1e-3 * (91 + 36 * c.ra + 13 * c.cbt + 8.8 * c.ra * c.cbt) *
                         (1 + 0.45 * busy * busy) * (two ? 1.25 : 1.0);
    const double comp = rounds * (stages * stage + 3.0);
    const double t = std::max(comp, hbm) + 0.15 * std::min(comp, hbm);
    if (t < best_t) {
      best_t = t;
      best = c;
    }
  }
  best.var.packed = packed;
  best.var.ragged = d % 64 != 0 || (!packed && V % 8 != 0);
  // Non-temporal loads where every element of W is read once and W exceeds
  // the 256 MB memory-side cache anyway (packed weight only: pieces of 1 KB.
  // V = 65536: 92 us against 122 us for W as given; below, caching wins: V =
  // 16384 34 us non-temporal, 29 us cached; ragged K too: V = 126464, d = 4072,
  // N = 96 191 us cached, 156 us non-temporal).
  best.var.nt = packed && best.n_nt == 1 && w_bytes > 384.0e6;
  // Two barriers per K stage (tiles of 512 rows, at most 64 columns) keep loads
  // in flight across stages.  That wins where the grid leaves compute units
  // idle, so that each one's own stream counts, and loses a little where the
  // memory is busy anyway.  MI355X, d = 4096, us per call, one barrier -> two:
  // packed V = 85000 (167 tiles) 1 row 127 -> 102, 64 rows 136 -> 113; 118000
  // (231) 145 -> 143, 151 -> 144; 126464 (247) 150 -> 154, 154 -> 155; 200000
  // (391, two rounds) 270 -> 249; as given 85000 133 -> 122, 142 -> 126; 112000
  // (219) 1 row 156 -> 158, 32 rows 157 -> 157; 200000 303 -> 284; d = 8192, V =
  // 128256 (251) 8 rows 352 -> 357, 32 rows 363 -> 356.
  const double full = (double)best.n_vt * best.n_nt / cus;
  const double fill = full / std::ceil(full);
  best.var.split = fill < (packed ? 0.93 : 0.82) || (!packed && N > 16);
  return best;
}

int al_internal_lmhead_plan(int N, int d, int V, int packed, int32_t* out) {
  const LmLayout L = lm_layout(N, d, V, packed != 0);
  const int form = lm_stage_form(L.ra, L.cbt);
  const int32_t v[8] = {L.ra, L.cbt, L.n_vt, L.n_nt, L.var.ragged, L.var.nt, form == 1 || (form == 2 && L.var.split),
                        L.ra != 0 && L.bytes() <= lmhead_workspace_bytes(N, d, V)};
  std::copy(v, v + 8, out);
  return 0;
}

int al_internal_lmhead_instances(int32_t* out, int most) {
  int n = 0;
  for (const auto& in : kLmInstances)
    if (n < most) {
      out[2 * n] = in.ra;
      out[2 * n++ + 1] = in.cbt;
    }
  return n;
}

// Partials of lmhead_confidence_noalloc.  In host code `scratch` names a
// host-side stand-in, not device memory: kernels get the device address
// that hipGetSymbolAddress returns for the current device (each GPU holds
// its own copy of the array).
static __device__ __align__(256) unsigned char scratch[AL_NOALLOC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
static std::atomic<void*> g_scratch_addr[kMaxDevices];
static std::mutex g_scratch_mu;

size_t lmhead_scratch_bytes() { return sizeof(scratch); }

hipError_t lmhead_scratch(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  void* p = g_scratch_addr[dev].load(std::memory_order_acquire);
  if (!p) {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    p = g_scratch_addr[dev].load(std::memory_order_relaxed);
    if (!p) {
      e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
      if (e != hipSuccess) return e;
      if (!p) return hipErrorInvalidSymbol;
      g_scratch_addr[dev].store(p, std::memory_order_release);
    }
  }
  *out = p;
  return hipSuccess;
}

size_t lmhead_packed_bytes(int d, int V) {
  return (size_t)((d + 63) / 64) * 64 * (size_t)((V + 31) / 32) * 32 * sizeof(uint16_t);
}

// One 16-byte segment per thread and step: segment o of the packed buffer
// is lane l = o % 64, step s = (o / 64) % 4 of block (c, u) = o / 256.
__global__ __launch_bounds__(256) void lmhead_pack_kernel(const uint16_t* W, int d, int V,
                                                          int n_hg, long long n_seg, uint16_t* Wp) {
  for (long long o = (long long)blockIdx.x * 256 + threadIdx.x; o < n_seg;
       o += (long long)gridDim.x * 256) {
    const int l = (int)(o & 63);
    const int st = (int)((o >> 6) & 3);
    const long long blk = o >> 8;
    const int u = (int)(blk % n_hg);
    const int c = (int)(blk / n_hg);
    const int v = u * 32 + (l & 31);
    const int k = c * 64 + st * 16 + (l >> 5) * 8;
    i32x4 val = {0, 0, 0, 0};
    if (v < V && k < d) val = *reinterpret_cast<const i32x4*>(W + (size_t)v * d + k);
    reinterpret_cast<i32x4*>(Wp)[o] = val;
  }
}

hipError_t launch_lmhead_pack(const uint16_t* W, int d, int V, uint16_t* Wp, hipStream_t stream) {
  const int n_hg = (V + 31) / 32;
  const long long n_seg = (long long)((d + 63) / 64) * n_hg * 256;
  hipLaunchKernelGGL(lmhead_pack_kernel, dim3(8192), dim3(256), 0, stream, W, d, V, n_hg, n_seg, Wp);
  return hipGetLastError();
}

hipError_t launch_lmhead(const uint16_t* hidden, const int32_t* row_idx, int N,
                         const uint16_t* W, int d, int V, const uint8_t* sup, int eos_id,
                         float* conf, int32_t* argmax, float* lse, void* ws,
                         hipStream_t stream, bool packed) {
  if (N <= 0) return hipSuccess;
  const LmLayout L = lm_layout(N, d, V, packed);
  LmTileParams p{};
  p.hidden = hidden;
  p.row_idx = row_idx;
  p.W = W;
  p.sup = sup;
  p.part = static_cast<LmPartial*>(ws);
  p.N = N;
  p.d = d;
  p.V = V;
  p.eos_id = eos_id;
  p.n_vt = L.n_vt;
  p.n_nt = L.n_nt;
  p.n_hg = (V + 31) / 32;
  p.tiles_total = L.n_vt * L.n_nt;
  p.tiles_per_xcd = (p.tiles_total + 7) / 8;
  // At most one workgroup per CU, dealt to the 8 XCDs in contiguous runs of
  // tiles (the column tiles of a vocabulary tile share that XCD's L2).
  const dim3 grid(8 * std::min(p.tiles_per_xcd, std::max(1, lm_cu_count() / 8)));
  switch (L.ra * 32 + L.cbt) {
#define AL_LM_X(RA, CBT) \
  case RA * 32 + CBT: launch_lmhead_tile<RA, CBT>(p, L.var, grid, stream); break;
    AL_LM_INSTANCES(AL_LM_X)
#undef AL_LM_X
    default: return hipErrorInvalidValue;
  }
  hipLaunchKernelGGL(lmhead_merge_kernel, dim3(N), dim3(LM_MERGE_THREADS), 0, stream, p.part, N,
                     L.n_vt, 16 * L.cbt, conf, argmax, lse);
  return hipGetLastError();
}

}  // namespace al
