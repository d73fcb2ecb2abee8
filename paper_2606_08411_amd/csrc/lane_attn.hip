// Shared-prefix lane-batched bidirectional attention for gfx950.
//
// Paper Section 3.2 ("Lane-local denoising") and Section 3.4 ("Shared-prefix
// lane batching", "Compact cache refresh and reuse"): every active lane of a
// prefix-sharing group is evaluated in one batched call; lane i's B query
// rows see the shared cached prefix, the blocks of its ancestors in the lane
// tree and, bidirectionally, its own block.
//
// Kernel layout.  A workgroup of 8 wavefronts serves one K/V head and eight
// (or four) query tiles (32 query rows of one lane and one query head each;
// for grouped-query attention the Hq/Hkv heads of a lane are adjacent tiles).
// Key tiles of 64 rows reach LDS once per workgroup by direct loads, K and V
// both row-major with their 16-byte segments permuted, and are consumed by
// every wavefront whose lane sees them, so a prefix tile read from HBM serves
// all lanes of the workgroup.  Both products run transposed on the 32x32x16 bf16 MFMA:
//     S^T = K Q^T      (lane l owns query row l%32, half of the keys)
//     O^T = V^T P^T    (lane l owns query row l%32, a quarter of D)
// so the running max / sum of the online softmax and the rescale of O stay
// inside a lane pair (l, l^32) and need no cross-lane broadcast.  The V^T
// operand comes from LDS transpose reads (ds_read_b64_tr_b16), which hand
// each lane 4 consecutive keys of one column.  Inside each 16-key MFMA step
// lane half h takes keys 4h..4h+3 and 8+4h..8+4h+3 on both operands, the
// keys the S^T accumulator gives it (a contraction is invariant under a
// common permutation of its summed index).
//
// Short grids (few heads x few lanes) either split each query tile's keys
// over the wavefronts of one workgroup (lane_attn_wsplit_kernel, merged in
// LDS) or, when that grid would not fit the chip at once, split the key
// tiles over blockIdx.z, whose unnormalised partials attn_merge_kernel
// combines.  The partial outputs are kept in bf16 (the softmax statistics
// in fp32): one rounding of a value that the output rounds to bf16 again,
// for half the partial traffic (Long shape, 4 splits: 49-51 -> 46.4 us per
// call, MI355X; outputs move by at most one bf16 step).  Fewer splits than the
// workspace is sized for keep them in fp32, which its bytes hold.
#include <math.h>

#include "common.h"
#include "launch.h"

namespace al {

constexpr int AT_WAVES = 8;
constexpr int AT_THREADS = AT_WAVES * kWave;
constexpr int AT_KT = 64;  // keys per staged tile
constexpr int AT_MAX_LANES = 64;
constexpr float AT_LN2 = 0.6931471805599453f;
// Deferred rescaling of the online softmax: a row's reference max moves
// only when a tile's scores exceed it by more than this many powers of two
// (P then stays <= 2^8, well inside bf16 and fp32 range), so O is rescaled
// in few tiles instead of in nearly every one.  O / l and m + log2 l are the
// same whichever reference is used, up to rounding.
constexpr float AT_RESCALE_LOG2 = 8.0f;

struct AttnParams {
  const uint16_t* q;       // [n_rows][Hq][D]
  const uint16_t* k_lane;  // [n_key_lanes*B_keys][Hkv][D] (lane mode)
  const uint16_t* v_lane;
  const uint16_t* k_pre;   // [P][Hkv][D]
  const uint16_t* v_pre;
  uint16_t* o;             // [n_rows][Hq][D]
  float* lse;              // [n_rows][Hq] or null
  void* part_o;            // [n_split][n_rows][Hq][D] bf16 or fp32, unnormalised, when n_split > 1
  float* part_ml;          // [n_split][n_rows][Hq][2]
  bool part_f32;
  unsigned long long deal; // lane blocks dealt to the splits: those of split 0 (0: shares of all tiles)
  int n_rows, rows_per_lane, tiles_per_lane, q_tiles_kv;
  int P, Hq, Hkv, g;
  int B_keys, n_key_lanes, lane_key_tiles, n_pre_tiles, total_key_tiles, n_split;
  float scale_log2;
  int tpw;                 // query tiles (computing wavefronts) per workgroup: 8 or 4
  unsigned long long vis[AT_MAX_LANES];  // bit j: lane block j visible to lane i
  // Lanes in the order in which the 8-tile kernel deals their query tiles to
  // workgroups, four to a word.
  unsigned order[AT_MAX_LANES / 4];
};
__device__ __forceinline__ int lane_at(const AttnParams& p, int pos) {
  return p.n_key_lanes ? (p.order[pos >> 2] >> (8 * (pos & 3))) & 255 : pos;
}

// Two wavefronts per SIMD (256 registers each), one workgroup per CU.
//
// What bounds it: a 64-key tile is 32 MFMAs (1024 cycles) and ~600 cycles of
// vector work per wavefront, so two wavefronts per SIMD need 2048 cycles a
// tile if vector work hides under MFMAs; it takes about 3900 (1.8 us).  Cycle
// stamps of the layout before (registers -> LDS staging, two barriers a
// tile, one wavefront's products and softmax in sequence) showed 4400-5000:
// both wavefronts of a SIMD reach the softmax together, because both leave
// each barrier together and the older one is served first.  Hence
// * in the prefix the next tile's Q K^T stands between the steps of this
//   tile's softmax, MFMA by MFMA, and the softmax's second half between the
//   MFMAs of P V, so that one wavefront keeps both units busy;
// * wavefronts 0-3 (or, with four query tiles, the idle 4-7) issue direct
//   loads three tiles ahead; no registers or LDS stores are spent on staging;
// * one path for full and ragged tiles (where two met, 128 accumulator
//   registers were copied per tile), and a tile walk that costs a few scalar
//   operations.
// Per call, same box, graph replay, before -> after: window of 2563 rows x 32
// heads 195 -> 153 us (D = 64 136 -> 107), 1531 rows x 28 heads on 4 K/V heads
// 76 -> 50, 1024 rows x 32 heads 42 -> 34, Wide lane + refresh 233 -> 204, Long
// 43.7 -> 40.  Then: exponentials pinned between the Q K^T MFMAs, the first V^T
// fragments read ahead of P V, lane tiles of at most 32 keys computed as
// halves and lanes dealt depth first: Wide lane + refresh 197.8 -> 192.2 us,
// Long 36.3 -> 34.4, windows unchanged (their workgroups have one computing
// wavefront per SIMD).  Counters on the 2563-row window: matrix cores 41% of
// the cycles, vector unit 35%, no LDS bank conflicts.  Two query tiles per
// wavefront (half the LDS reads, 512 registers, one wavefront per SIMD) take
// 57 us at Long and 316 us at Wide: scores pass through accumulation registers
// and nothing fills a wavefront's waits.
constexpr int AT_OCC = 2;

template <int D>
__global__ __launch_bounds__(AT_THREADS) __attribute__((amdgpu_waves_per_eu(AT_OCC, AT_OCC)))
void lane_attn_kernel(AttnParams p) {
  constexpr int KS = D / 16;       // MFMA k-steps of S^T = K Q^T
  constexpr int DT = D / 32;       // 32-row tiles of O^T
  constexpr int ROWB = 2 * D;      // bytes of a K or V row in LDS
  constexpr int TB = AT_KT * ROWB; // bytes of a K or V tile
  constexpr int RPP = 1024 / ROWB; // rows per 1 KB piece (one direct load of a wavefront)
  constexpr int AHEAD = 4;         // K fragments read ahead
  constexpr int PW = AT_KT / RPP / 4;  // pieces per tile and loading wavefront
  // Four tile buffers, K then V.
  __shared__ __attribute__((aligned(1024))) char lds[8 * TB];

  const int hk = blockIdx.y;
  const int split = blockIdx.z;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: scalar registers and branches
  const int r32 = lane & 31;
  const int hh = lane >> 5;
  const int lgrp = lane >> 4;  // 16-lane group of the transpose reads
  const int lg = lane & 15;
  const int per_lane = p.tiles_per_lane * p.g;

  // This wavefront's query tile.
  const int tpw = p.tpw;
  const int qt = blockIdx.x * tpw + w;
  const bool active = w < tpw && qt < p.q_tiles_kv;
  int lane_i = 0, c = 0, hg = 0;
  if (active) {
    const int pos = qt / per_lane;
    const int rem = qt - pos * per_lane;
    lane_i = lane_at(p, pos);
    c = rem / p.g;
    hg = rem - c * p.g;
  }
  const int hq = hk * p.g + hg;
  const int row0 = lane_i * p.rows_per_lane + c * 32;
  int nrows = 0;
  if (active) nrows = min(min(32, p.rows_per_lane - c * 32), p.n_rows - row0);
  const unsigned long long my_vis = (active && p.n_key_lanes) ? p.vis[lane_i] : 0ull;
  unsigned long long wg_vis = 0ull;
  for (int ww = 0; ww < tpw; ++ww) {
    const int qt2 = blockIdx.x * tpw + ww;
    if (qt2 < p.q_tiles_kv && p.n_key_lanes) wg_vis |= p.vis[lane_at(p, qt2 / per_lane)];
  }

  // Q fragments (B operand of S^T = K Q^T), kept in registers.
  bf16x8 qf[KS];
  {
    const bool ok = r32 < nrows;
    const uint16_t* qrow = p.q + ((size_t)(row0 + (ok ? r32 : 0)) * p.Hq + hq) * D;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = ok ? load_bf16x8(qrow + ks * 16 + hh * 8) : zero_bf16x8();
  }

  f32x16 oacc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;

  // The workgroup's key tiles: the prefix tiles, then the tiles of the lane
  // blocks some wavefront sees, in ascending order; this split takes [t0, t1) of
  // them.  Which keys a row's partial holds must not depend on the lanes that
  // share its workgroup, so the splits share out all the call's key tiles, and of
  // its share a workgroup takes the visible ones.  Shares are contiguous, or (deal)
  // contiguous in the prefix and every n_split-th lane block.
  unsigned long long lanes = wg_vis;   // blocks that this split may take
  int pre_end = p.n_pre_tiles;         // end of the prefix tiles listed
  int t0, t1;
  const int split_log2 = __builtin_ctz(p.n_split);   // a power of two: no 64-bit division
  auto share = [&](int i, int n) -> int { return (int)((long long)i * n >> split_log2); };
  if (p.deal) {
    lanes &= p.deal << split;
    t0 = share(split, p.n_pre_tiles);
    pre_end = share(split + 1, p.n_pre_tiles);
    t1 = pre_end + __popcll(lanes) * p.lane_key_tiles;
  } else {
    auto visible_before = [&](int kt) -> int {
      if (kt <= p.n_pre_tiles || p.n_key_lanes == 0) return min(kt, p.n_pre_tiles);
      const int q = kt - p.n_pre_tiles, j = q / p.lane_key_tiles;
      const unsigned long long below = j < 64 ? wg_vis & ((1ull << j) - 1) : wg_vis;
      const bool cut = j < 64 && ((wg_vis >> j) & 1);
      return p.n_pre_tiles + __popcll(below) * p.lane_key_tiles + (cut ? q - j * p.lane_key_tiles : 0);
    };
    t0 = visible_before(share(split, p.total_key_tiles));
    t1 = visible_before(share(split + 1, p.total_key_tiles));
  }
  // They come in runs of consecutive rows: the prefix, then each block.  A
  // walk holds what is left of its run, so that the next tile costs a few
  // scalar operations; the rest is done once per run.
  struct Walk {
    unsigned long long m;   // lanes not finished (lowest: the current one)
    int row, left;          // next row of the run, rows left in it
    bool pre;
  };
  auto walk_at = [&](int t) {
    Walk k{lanes, 0, 0, t < pre_end};
    if (k.pre) {
      k.row = t * AT_KT;
      k.left = min(p.P, pre_end * AT_KT) - k.row;
    } else {
      const int q = t - pre_end, n = p.n_key_lanes ? q / p.lane_key_tiles : 0;
      for (int i = 0; i < n; ++i) k.m &= k.m - 1;
      const int sub = (q - n * p.lane_key_tiles) * AT_KT;
      k.row = k.m ? __builtin_ctzll(k.m) * p.B_keys + sub : 0;
      k.left = p.B_keys - sub;
    }
    return k;
  };
  auto next_run = [&](Walk& k) {
    if (!k.pre) k.m &= k.m - 1;
    k.pre = false;
    k.row = k.m ? __builtin_ctzll(k.m) * p.B_keys : 0;
    k.left = p.B_keys;
  };

  // Direct loads of a tile (wavefronts 0-3).  Row r's 16-byte segment s sits
  // in slot s ^ f(r): f_K puts the 16 rows that one LDS cycle of the K reads
  // serves into different banks, f_V the 4 (and 8) rows of a transpose read.
  // Rows past the tile's valid keys are zero.
  const int lrow = RPP * (w & 3) + lane * 16 / ROWB;   // row of this lane in piece 0
  const int lslot = lane & (ROWB / 16 - 1);
  const int fk = D == 128 ? lrow & 15 : (lrow >> 1) & 7;
  const int fv = D == 128 ? (4 * (lrow & 3)) ^ (2 * ((lrow >> 2) & 1))
                          : (4 * ((lrow >> 1) & 1)) ^ (2 * ((lrow >> 2) & 1));
  const unsigned rowbytes = (unsigned)p.Hkv * ROWB;
  const unsigned kvoff = lrow * rowbytes + (unsigned)((lslot ^ fk) * 16);
  const unsigned vvoff = lrow * rowbytes + (unsigned)((lslot ^ fv) * 16);
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  const unsigned pstep = 4 * RPP * rowbytes;   // from a piece to the wavefront's next
  const char *kp = nullptr, *vp = nullptr;     // next tile to load
  auto set_source = [&](const Walk& k) {
    const size_t off = (size_t)k.row * rowbytes + (size_t)hk * ROWB;
    kp = reinterpret_cast<const char*>(k.pre ? p.k_pre : p.k_lane) + off;
    vp = reinterpret_cast<const char*>(k.pre ? p.v_pre : p.v_lane) + off;
  };
  auto load_tile = [&](int nvalid, int buf) {
    const unsigned l = lds0 + buf * 2 * TB + (w & 3) * 1024;
    if (nvalid >= AT_KT) {
      const char *kj = kp, *vj = vp;
      static_for<PW>([&](auto j) {
        constexpr int J = decltype(j)::value;
        load_to_lds16<J * 4096, 0, false>(uniform_ptr(kj), kvoff, l);
        load_to_lds16<TB + J * 4096, 0, false>(uniform_ptr(vj), vvoff, l);
        kj += pstep;
        vj += pstep;
      });
    } else {
      const char* zero = reinterpret_cast<const char*>(zero_seg16);
      static_for<PW>([&](auto j) {
        constexpr int J = decltype(j)::value;
        const bool ok = lrow + J * 4 * RPP < nvalid;
        load_to_lds16<J * 4096>(ok ? kp + (size_t)J * pstep + kvoff : zero, l);
        load_to_lds16<TB + J * 4096>(ok ? vp + (size_t)J * pstep + vvoff : zero, l);
      });
    }
  };

  // Lane addresses inside a tile: K fragment (row r32, segment 2 ks + hh) at
  // ka ^ 32 ks; V^T fragment of 32-column tile dt at va ^ 64 dt.
  const int ka = r32 * ROWB + ((hh ^ (D == 128 ? r32 & 15 : (r32 >> 1) & 7)) * 16);
  const int vr = 4 * hh + (lg >> 2);
  const int vx = D == 128 ? (4 * (vr & 3)) ^ (2 * ((vr >> 2) & 1))
                          : (4 * ((vr >> 1) & 1)) ^ (2 * ((vr >> 2) & 1));
  const int va = vr * ROWB + (((2 * (lgrp & 1) + ((lg & 3) >> 1)) ^ vx) * 16) + (lg & 1) * 8;

  // A tile: S^T = K Q^T, the online softmax update in log2 units, then O^T +=
  // V^T P^T.  Fragments are read ahead of their MFMAs (AHEAD of K, one 16-key
  // step of V).
  struct Scores {
    f32x16 s[2];   // the two 32-key halves
  };
  // (NH = 1: a tile of at most 32 keys, its first half alone.)
  auto read_k = [&](auto nh_tag, bf16x8* kf, int buf) {
    constexpr int NH = decltype(nh_tag)::value;
    const char* kt = lds + buf * 2 * TB;
#pragma unroll
    for (int i = 0; i < 2 * KS; i += 3 - NH)
      kf[i] = *reinterpret_cast<const bf16x8*>(kt + (ka ^ (32 * (i >> 1))) + (i & 1) * 32 * ROWB);
  };
  auto qk = [&](auto nh_tag, Scores& sc, const bf16x8* kf) {
    constexpr int NH = decltype(nh_tag)::value;
    const f32x16 zero16 = {};
    // The two accumulation chains interleave, so consecutive MFMAs are independent.
#pragma unroll
    for (int i = 0; i < 2 * KS; i += 3 - NH)
      sc.s[i & 1] = mfma32x32x16(kf[i], qf[i >> 1], i < 2 ? zero16 : sc.s[i & 1]);
  };
  auto vfrag = [&](int buf, int ks2, int dt) {
    const uint16_t* a = reinterpret_cast<const uint16_t*>(lds + buf * 2 * TB + TB + (va ^ (64 * dt)) + 16 * ks2 * ROWB);
    return cat_bf16x4(lds_read_tr16(a), lds_read_tr16(a + 8 * D));
  };
  auto mask = [&](auto nh_tag, Scores& sc, int nvalid) {
    constexpr int NH = decltype(nh_tag)::value;
    if (nvalid < 32 * NH) {
#pragma unroll
      for (int kb = 0; kb < NH; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = kb * 32 + 8 * (r >> 2) + 4 * hh + (r & 3);
          sc.s[kb][r] = (key < nvalid) ? sc.s[kb][r] : -INFINITY;
        }
    }
  };
  // The softmax in pieces that can stand between MFMAs.  The max is taken on
  // the raw scores (the scale is positive, so max-then-scale is exact); each
  // exponent is then one FMA.
  auto max_piece = [&](float mx, const Scores& sc, int q) {   // q = 0..3: 8 scores
#pragma unroll
    for (int r = 0; r < 8; ++r) mx = fmaxf(mx, sc.s[q >> 1][8 * (q & 1) + r]);
    return mx;
  };
  auto new_max = [&](float mx, float& m_new) {   // returns the factor on O
    const float m_tile = pair_max32(mx) * p.scale_log2;
    m_new = m_tile > m_run + AT_RESCALE_LOG2 ? m_tile : m_run;
    const float alpha = exp2_fast(m_run - m_new);
    m_run = m_new;
    return alpha;
  };
  // P in bf16 (round-to-nearest-even, two values per conversion), packed per
  // 16-key MFMA step; the row sum adds the rounded values (bf16 dot products
  // with 1), so O / l is a convex combination of V rows.
  auto exp_pair = [&](const Scores& sc, bf16x8* pk, float m_new, float& rs, int q) {   // q = 0..15
    const bf16x2 one2 = {(__bf16)1.0f, (__bf16)1.0f};
    const int ks2 = q >> 2, e = 2 * (q & 3), r = 8 * (ks2 & 1) + e;
    bf16x2 pr;
    pr[0] = (__bf16)exp2_fast(fmaf(sc.s[ks2 >> 1][r], p.scale_log2, -m_new));
    pr[1] = (__bf16)exp2_fast(fmaf(sc.s[ks2 >> 1][r + 1], p.scale_log2, -m_new));
    pk[ks2][e] = pr[0];
    pk[ks2][e + 1] = pr[1];
    rs = __builtin_amdgcn_fdot2_f32_bf16(pr, one2, rs, false);
  };
  auto rescale = [&](float alpha) {
    // Rescale O only when some row's reference max moved (otherwise alpha
    // is exactly 1 and the product would change nothing).
    if (__builtin_amdgcn_read_exec() & __ballot(alpha != 1.0f)) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[dt][r] *= alpha;
    }
  };
  // O^T += V^T P^T, one 16-key MFMA step at a time, the second half of P's
  // exponentials between the MFMAs of the first two steps.  The V^T fragment
  // of lane (d, h) is keys 16 ks2 + 4h + {0..3, 8..11} at column d: two
  // transpose reads of 4 x 16 blocks of the row-major V tile.  vf[0] holds the
  // first step's fragments.
  auto pv = [&](auto nh_tag, const Scores& sc, bf16x8* pk, bf16x8 (*vf)[DT], float m_new, float alpha, float rs, int buf) {
    constexpr int NH = decltype(nh_tag)::value;
#pragma unroll
    for (int ks2 = 0; ks2 < 2 * NH; ++ks2) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        if (ks2 < 2 * NH - 1) vf[(ks2 + 1) & 1][dt] = vfrag(buf, ks2 + 1, dt);
        oacc[dt] = mfma32x32x16(vf[ks2 & 1][dt], pk[ks2], oacc[dt]);
        if (NH == 2 && ks2 < 2) {
#pragma unroll
          for (int q = 0; q < 4 / DT; ++q) exp_pair(sc, pk, m_new, rs, 8 + ks2 * 4 + dt * (4 / DT) + q);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    l_run = l_run * alpha + pair_sum32(rs);
  };
  // Q K^T of the tile in buffer bq into nxt, with the max and the first half
  // of the exponentials of cur between its MFMAs; then cur's P V.
  auto hot_tile = [&](const Scores& cur, Scores& nxt, int bq, int bv) {
    bf16x8 kf[2 * KS], pk[4], vf[2][DT];
    const f32x16 zero16 = {};
    const char* kt = lds + bq * 2 * TB;
    auto kread = [&](int i) {
      kf[i] = *reinterpret_cast<const bf16x8*>(kt + (ka ^ (32 * (i >> 1))) + (i & 1) * 32 * ROWB);
    };
    float mx = -INFINITY, m_new, alpha, rs = 0.f;
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) kread(i);
    __builtin_amdgcn_sched_barrier(0);
    constexpr int MX = KS / 2;                 // MFMAs with a piece of the max
    constexpr int EX = 2 * KS - MX;            // and with exponentials
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i) {
      if (i + AHEAD < 2 * KS) kread(i + AHEAD);
      else if (i + DT >= 2 * KS) {   // the first V^T fragments take the K fragments' registers
        const int dt = i + DT - 2 * KS;
        vf[0][dt] = vfrag(bv, 0, dt);
      }
      nxt.s[i & 1] = mfma32x32x16(kf[i], qf[i >> 1], i < 2 ? zero16 : nxt.s[i & 1]);
      if (i < MX) {
#pragma unroll
        for (int q = 0; q < 4 / MX; ++q) mx = max_piece(mx, cur, i * (4 / MX) + q);
        if (i == MX - 1) alpha = new_max(mx, m_new);
      } else {
        const int j = i - MX;
#pragma unroll
        for (int q = 8 * j / EX; q < 8 * (j + 1) / EX; ++q) {
          exp_pair(cur, pk, m_new, rs, q);
          // Left alone, the compiler sinks these past the branch below to their
          // use in P V, where all 32 exponentials then stand.
          asm volatile("" ::"v"(__builtin_bit_cast(i32x4, pk[q >> 2])[q & 3]), "v"(rs));
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    rescale(alpha);
    pv(IntTag<2>{}, cur, pk, vf, m_new, alpha, rs, bv);
  };
  auto cold_tile = [&](auto nh_tag, const Scores& cur, int bv) {   // softmax and P V alone
    constexpr int NH = decltype(nh_tag)::value;
    bf16x8 pk[4];
    float mx = -INFINITY, m_new, rs = 0.f;
#pragma unroll
    for (int q = 0; q < 2 * NH; ++q) mx = max_piece(mx, cur, q);
    const float alpha = new_max(mx, m_new);
#pragma unroll
    for (int q = 0; q < 8; ++q) exp_pair(cur, pk, m_new, rs, q);
    rescale(alpha);
    bf16x8 vf[2][DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) vf[0][dt] = vfrag(bv, 0, dt);
    __builtin_amdgcn_sched_barrier(0);
    pv(nh_tag, cur, pk, vf, m_new, alpha, rs, bv);
  };

  // Tiles are loaded three ahead into four buffers, one barrier per tile:
  // after tile i's barrier everyone is done with tile i - 1, whose buffer takes
  // tile i + 3, and tile i + 1 is complete.
  const int n = t1 - t0;
  const int np = max(0, min(pre_end - t0, n));   // of them prefix tiles
  Walk lw = walk_at(t0);
  int loaded = 0;
  set_source(lw);
  const bool loader = tpw == AT_WAVES ? w < 4 : w >= 4;
  auto load_next = [&]() {
    if (loader && loaded < n) {
      load_tile(lw.left, loaded & 3);
      lw.row += AT_KT;
      lw.left -= AT_KT;
      kp += AT_KT * rowbytes;
      vp += AT_KT * rowbytes;
      if (lw.left <= 0) {
        next_run(lw);
        set_source(lw);
      }
    }
    ++loaded;
  };
  auto next_tile = [&](int i) {
    if (i + 2 < n) wait_loads_and_barrier<2 * PW>();
    else wait_loads_and_barrier<0>();
    load_next();
  };
  load_next();
  load_next();
  load_next();
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // (so the compiler knows that Q is there)
  wait_loads_and_barrier<0>();

  if (w >= tpw) {   // loads only
    for (int i = 0; i < n; ++i) next_tile(i);
    return;
  }
  // Prefix tiles, seen by every wavefront (one without a query tile works on
  // row 0 and stores nothing): the next tile's Q K^T fills the matrix cores
  // while this tile's softmax runs on the vector unit.
  {
    Scores sa, sb;
    bf16x8 kf[2 * KS];
    auto hot = [&](Scores& cur, Scores& nxt, int i) {
      next_tile(i);
      hot_tile(cur, nxt, (i + 1) & 3, i & 3);
    };
    auto last = [&](Scores& cur, int i) {
      next_tile(i);
      mask(IntTag<2>{}, cur, p.P - (t0 + i) * AT_KT);
      cold_tile(IntTag<2>{}, cur, i & 3);
    };
    if (np > 0) {
      read_k(IntTag<2>{}, kf, 0);
      qk(IntTag<2>{}, sa, kf);
      int i = 0;
      for (; i + 2 < np; i += 2) {
        hot(sa, sb, i);
        hot(sb, sa, i + 1);
      }
      if (i + 1 < np) {
        hot(sa, sb, i);
        last(sb, i + 1);
      } else {
        last(sa, i);
      }
    }
  }
  // Lane tiles: only those this wavefront's lane sees, and of a tile that ends
  // within its first half (every tile of a block of 32) that half alone.
  if (np < n) {
    Walk cw = walk_at(t0 + np);
    for (int i = np; i < n; ++i) {
      next_tile(i);
      if (active && (my_vis & cw.m & (0 - cw.m))) {
        auto lane_tile = [&](auto nh_tag) {
          Scores sc;
          bf16x8 kf[2 * KS];
          read_k(nh_tag, kf, i & 3);
          qk(nh_tag, sc, kf);
          mask(nh_tag, sc, cw.left);
          cold_tile(nh_tag, sc, i & 3);
        };
        if (cw.left <= 32) lane_tile(IntTag<1>{});
        else lane_tile(IntTag<2>{});
      }
      cw.left -= AT_KT;
      if (cw.left <= 0) next_run(cw);
    }
  }

  if (!active || r32 >= nrows) return;
  const size_t orow = (size_t)(row0 + r32) * p.Hq + hq;
  if (p.n_split == 1) {
    const float inv_l = 1.0f / l_run;
    uint16_t* op = p.o + orow * D;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int rg = 0; rg < 4; ++rg) {
        bf16x4 v4;
#pragma unroll
        for (int e = 0; e < 4; ++e) v4[e] = (__bf16)(oacc[dt][rg * 4 + e] * inv_l);
        *reinterpret_cast<bf16x4*>(op + dt * 32 + 8 * rg + 4 * hh) = v4;
      }
    if (p.lse && hh == 0) p.lse[orow] = (m_run + log2f(l_run)) * AT_LN2;
  } else {
    const size_t prow = ((size_t)split * p.n_rows * p.Hq + orow) * D;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int rg = 0; rg < 4; ++rg) {
        const size_t at = prow + dt * 32 + 8 * rg + 4 * hh;
        if (p.part_f32) {
          f32x4 v4;
#pragma unroll
          for (int e = 0; e < 4; ++e) v4[e] = oacc[dt][rg * 4 + e];
          *reinterpret_cast<f32x4*>(static_cast<float*>(p.part_o) + at) = v4;
        } else {
          bf16x4 v4;
#pragma unroll
          for (int e = 0; e < 4; ++e) v4[e] = (__bf16)oacc[dt][rg * 4 + e];
          *reinterpret_cast<bf16x4*>(static_cast<uint16_t*>(p.part_o) + at) = v4;
        }
      }
    if (hh == 0) {
      float* pm = p.part_ml + ((size_t)split * p.n_rows * p.Hq + orow) * 2;
      pm[0] = m_run;
      pm[1] = l_run;
    }
  }
}

// Keys of one query tile split over the wavefronts of one workgroup.
//
// On short grids (a few lanes x a few heads) the kernel above leaves most
// SIMDs idle unless it splits the key range over workgroups, and then its
// partials cross a kernel boundary to attn_merge_kernel (written back
// from L2 at the end of the kernel, read again by the merge).  Here a
// workgroup of KW wavefronts serves one query tile (32 rows of one lane,
// one query head).  Wavefront w takes the lane's visible 32-key units w,
// w + KW, w + 2 KW, ... (prefix units first, then the visible lane blocks
// in ascending order), stages each in an LDS region of its own and keeps
// its own online-softmax state; nothing is shared between wavefronts until
// the end, so the loop has no workgroup barrier.  The KW states are then
// combined in LDS in ascending w (the same arithmetic as attn_merge_kernel)
// and the output is written once, in bf16.  Every lane's workgroups re-read
// the prefix units; workgroup ids run head-fastest, so with Hq a multiple
// of 8 all query tiles of a head land on one XCD (ids are dealt to the 8
// XCDs round-robin) and those re-reads hit that XCD's L2.
template <int D, int KW>
__global__ __launch_bounds__(KW * kWave) __attribute__((amdgpu_waves_per_eu(KW / 4, KW / 4)))
void lane_attn_wsplit_kernel(AttnParams p) {
  constexpr int KT = 32;                    // keys per unit
  constexpr int KS = D / 16;
  constexpr int DT = D / 32;
  constexpr int KSTR = D + 8;
  constexpr int VROW = D + 32;
  constexpr int DSEG = D / 8;
  constexpr int KREG = KT * DSEG / kWave;   // 16-byte K (and V) segments per lane
  constexpr int WBUF = KT * (KSTR + VROW);  // bf16 per wavefront region
  constexpr int OSTR = D + 4;               // fp32 per row of the merge area
  static_assert(KREG * kWave == KT * DSEG, "whole tiles per lane");
  static_assert((KW * 32 * OSTR + KW * 32 * 2) * 4 <= KW * WBUF * 2, "merge area inside the tile regions");
  __shared__ __attribute__((aligned(16))) uint16_t lds[KW * WBUF];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r32 = lane & 31;
  const int hh = lane >> 5;
  const int lgrp = lane >> 4;
  const int lg = lane & 15;
  uint16_t* k_s = lds + w * WBUF;
  uint16_t* v_s = k_s + KT * KSTR;

  const int hq = blockIdx.x % p.Hq;
  const int qt = blockIdx.x / p.Hq;
  const int lane_i = qt / p.tiles_per_lane;
  const int c = qt - lane_i * p.tiles_per_lane;
  const int hk = hq / p.g;
  const int row0 = lane_i * p.rows_per_lane + c * 32;
  const int nrows = min(min(32, p.rows_per_lane - c * 32), p.n_rows - row0);
  const unsigned long long vis = p.n_key_lanes ? p.vis[lane_i] : 0ull;
  const int n_pre = (p.P + KT - 1) / KT;
  const int lane_units = (p.B_keys + KT - 1) / KT;
  const int n_units = n_pre + __popcll(vis) * lane_units;

  // The query tile is the same for every wavefront: wavefront w < KS loads
  // its k-step w once and the fragments are shared through LDS (8x fewer Q
  // loads per workgroup; graph replay, one box: LLaDA 9.7 against 11.1 us,
  // Dream 14.9 against 16.6 us).
  bf16x8 qf[KS];
  __shared__ __attribute__((aligned(16))) bf16x8 q_sh[KS * kWave];
  bf16x8 qslice = zero_bf16x8();
  {
    const bool ok = r32 < nrows;
    const uint16_t* qrow = p.q + ((size_t)(row0 + (ok ? r32 : 0)) * p.Hq + hq) * D;
    if (w < KS) qslice = ok ? load_bf16x8(qrow + w * 16 + hh * 8) : zero_bf16x8();
  }
  f32x16 oacc[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[dt][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;

  struct Unit {
    const uint16_t* k;
    const uint16_t* v;
    int nvalid;  // 0 = past the last unit
  };
  auto unit_at = [&](int u) -> Unit {
    Unit t{nullptr, nullptr, 0};
    if (u >= n_units) return t;
    int r0;
    if (u < n_pre) {
      r0 = u * KT;
      t.k = p.k_pre + ((size_t)r0 * p.Hkv + hk) * D;
      t.v = p.v_pre + ((size_t)r0 * p.Hkv + hk) * D;
      t.nvalid = min(KT, p.P - r0);
      return t;
    }
    const int lu = u - n_pre;
    int jj = lu / lane_units;
    const int sub = lu - jj * lane_units;
    unsigned long long m = vis;
    for (; jj > 0; --jj) m &= m - 1;  // drop the jj lowest visible lanes
    r0 = __builtin_ctzll(m) * p.B_keys + sub * KT;
    t.k = p.k_lane + ((size_t)r0 * p.Hkv + hk) * D;
    t.v = p.v_lane + ((size_t)r0 * p.Hkv + hk) * D;
    t.nvalid = min(KT, p.B_keys - sub * KT);
    return t;
  };

  bf16x8 kr[KREG], vr[KREG];
  auto load_unit = [&](const Unit& t) {
#pragma unroll
    for (int i = 0; i < KREG; ++i) {
      const int seg = lane + kWave * i;
      const int krow = seg / DSEG;
      const int ds = seg - krow * DSEG;
      kr[i] = load_bf16x8(t.k + (size_t)min(krow, t.nvalid - 1) * p.Hkv * D + ds * 8);
    }
#pragma unroll
    for (int i = 0; i < KREG; ++i) {
      const int seg = lane + kWave * i;
      const int krow = seg / DSEG;
      const int ds = seg - krow * DSEG;
      vr[i] = load_bf16x8(t.v + (size_t)min(krow, t.nvalid - 1) * p.Hkv * D + ds * 8);
    }
  };
  auto store_unit = [&](int nvalid) {
#pragma unroll
    for (int i = 0; i < KREG; ++i) {
      const int seg = lane + kWave * i;
      const int krow = seg / DSEG;
      const int ds = seg - krow * DSEG;
      const bool ok = nvalid == KT || krow < nvalid;
      *reinterpret_cast<bf16x8*>(&k_s[krow * KSTR + ds * 8]) = ok ? kr[i] : zero_bf16x8();
      *reinterpret_cast<bf16x8*>(&v_s[krow * VROW + ds * 8]) = ok ? vr[i] : zero_bf16x8();
    }
  };
  // S^T = K Q^T in two interleaved chains (even / odd k-steps), the online
  // softmax update in log2 units, then O^T += V^T P^T -- the arithmetic of
  // lane_attn_kernel's tile step on one 32-key half.
  auto unit_compute = [&](int nvalid) {
    f32x16 s0 = {}, s1 = {};
#pragma unroll
    for (int ks = 0; ks < KS; ks += 2) {
      s0 = mfma32x32x16(*reinterpret_cast<const bf16x8*>(&k_s[r32 * KSTR + ks * 16 + hh * 8]), qf[ks], s0);
      s1 = mfma32x32x16(*reinterpret_cast<const bf16x8*>(&k_s[r32 * KSTR + (ks + 1) * 16 + hh * 8]), qf[ks + 1], s1);
    }
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = s0[r] + s1[r];
    if (nvalid < KT) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = 8 * (r >> 2) + 4 * hh + (r & 3);
        s[r] = (key < nvalid) ? s[r] : -INFINITY;
      }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[r]);
    mx = pair_max32(mx);
    const float m_tile = mx * p.scale_log2;
    const float m_new = m_tile > m_run + AT_RESCALE_LOG2 ? m_tile : m_run;
    const float alpha = exp2_fast(m_run - m_new);
    float rs = 0.f;
    bf16x8 pk[2];
    const bf16x2 one2 = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
    for (int ks2 = 0; ks2 < 2; ++ks2)
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const int r = 8 * ks2 + e;
        bf16x2 pr;
        pr[0] = (__bf16)exp2_fast(fmaf(s[r], p.scale_log2, -m_new));
        pr[1] = (__bf16)exp2_fast(fmaf(s[r + 1], p.scale_log2, -m_new));
        pk[ks2][e] = pr[0];
        pk[ks2][e + 1] = pr[1];
        rs = __builtin_amdgcn_fdot2_f32_bf16(pr, one2, rs, false);
      }
    rs = pair_sum32(rs);
    l_run = l_run * alpha + rs;
    m_run = m_new;
    if (__builtin_amdgcn_read_exec() & __ballot(alpha != 1.0f)) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[dt][r] *= alpha;
    }
#pragma unroll
    for (int ks2 = 0; ks2 < 2; ++ks2)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const uint16_t* va = &v_s[(16 * ks2 + 4 * hh + (lg >> 2)) * VROW + dt * 32 + 16 * (lgrp & 1) + 4 * (lg & 3)];
        const bf16x8 a = cat_bf16x4(lds_read_tr16(va), lds_read_tr16(va + 8 * VROW));
        oacc[dt] = mfma32x32x16(a, pk[ks2], oacc[dt]);
      }
  };

  int u = w;
  Unit cur = unit_at(u);
  {
    // Unconditional first loads and an exact wait for this wavefront's Q
    // slice, as in lane_attn_kernel (a wavefront without a unit reads Q row
    // 0); then the slices are exchanged through LDS.
    Unit first = cur;
    if (!first.nvalid) {
      first.k = first.v = p.q;
      first.nvalid = 1;
    }
    load_unit(first);
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * KREG));
    if (w < KS) q_sh[w * kWave + lane] = qslice;
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = q_sh[ks * kWave + lane];
  }
  while (cur.nvalid) {
    // The region is this wavefront's own: its LDS operations complete in
    // issue order, so wavefront-scope fences (compiler ordering only)
    // separate the previous unit's reads, this unit's stores and its reads.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    store_unit(cur.nvalid);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    u += KW;
    const Unit nxt = unit_at(u);
    if (nxt.nvalid) load_unit(nxt);
    unit_compute(cur.nvalid);
    cur = nxt;
  }

  // Combine the KW states: each wavefront writes (m, l, O) to LDS, then
  // D / 8 threads per row merge 8 columns each in ascending w.
  __syncthreads();  // every wavefront is done with its tile region
  float* o_s = reinterpret_cast<float*>(lds);
  float* ml_s = o_s + KW * 32 * OSTR;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int rg = 0; rg < 4; ++rg)
      *reinterpret_cast<float4*>(&o_s[(w * 32 + r32) * OSTR + dt * 32 + 8 * rg + 4 * hh]) =
          make_float4(oacc[dt][rg * 4 + 0], oacc[dt][rg * 4 + 1], oacc[dt][rg * 4 + 2], oacc[dt][rg * 4 + 3]);
  if (hh == 0) {
    ml_s[(w * 32 + r32) * 2 + 0] = m_run;
    ml_s[(w * 32 + r32) * 2 + 1] = l_run;
  }
  __syncthreads();
  constexpr int TPR = D / 8;            // threads per row
  constexpr int RPP = KW * kWave / TPR;  // rows per pass
  const int d0 = (tid % TPR) * 8;
  for (int row = tid / TPR; row < nrows; row += RPP) {
    float mw[KW], M = -INFINITY;
#pragma unroll
    for (int ww = 0; ww < KW; ++ww) {
      mw[ww] = ml_s[(ww * 32 + row) * 2];
      M = fmaxf(M, mw[ww]);
    }
    float Lsum = 0.f, acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.f;
#pragma unroll
    for (int ww = 0; ww < KW; ++ww) {
      const float wgt = (mw[ww] == -INFINITY) ? 0.f : exp2_fast(mw[ww] - M);
      Lsum += ml_s[(ww * 32 + row) * 2 + 1] * wgt;
      const float4 a = *reinterpret_cast<const float4*>(&o_s[(ww * 32 + row) * OSTR + d0]);
      const float4 b = *reinterpret_cast<const float4*>(&o_s[(ww * 32 + row) * OSTR + d0 + 4]);
      acc[0] += a.x * wgt;
      acc[1] += a.y * wgt;
      acc[2] += a.z * wgt;
      acc[3] += a.w * wgt;
      acc[4] += b.x * wgt;
      acc[5] += b.y * wgt;
      acc[6] += b.z * wgt;
      acc[7] += b.w * wgt;
    }
    const float inv = 1.0f / Lsum;
    bf16x8 out;
#pragma unroll
    for (int e = 0; e < 8; ++e) out[e] = (__bf16)(acc[e] * inv);
    const size_t orow = (size_t)(row0 + row) * p.Hq + hq;
    *reinterpret_cast<bf16x8*>(p.o + orow * D + d0) = out;
    if (p.lse && d0 == 0) p.lse[orow] = (M + log2f(Lsum)) * AT_LN2;
  }
}

// Combine the NS key splits of each (row, head): D / 8 lanes per (row,
// head), each taking 8 elements (16-byte loads and stores).  NS is a
// template argument so every split's loads issue at once (one memory round
// trip); the splits are summed in ascending order.
template <int D>
constexpr int merge_rows_per_block() { return 256 / (D / 8); }
template <int D, int NS, class T>   // T: uint16_t (bf16) or float partials
__global__ __launch_bounds__(256) void attn_merge_kernel(const T* part_o, const float* part_ml,
                                                         int n_rowheads, uint16_t* o, float* lse) {
  constexpr int LPR = D / 8;  // lanes per (row, head)
  const int rh = blockIdx.x * merge_rows_per_block<D>() + threadIdx.x / LPR;
  const int sl = threadIdx.x % LPR;
  if (rh >= n_rowheads) return;
  float m[NS], l[NS], po[NS][8];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const float2 ml = *reinterpret_cast<const float2*>(part_ml + ((size_t)s * n_rowheads + rh) * 2);
    m[s] = ml.x;
    l[s] = ml.y;
    const T* src = part_o + ((size_t)s * n_rowheads + rh) * D + sl * 8;
    if constexpr (sizeof(T) == 4) {
      const f32x4 a = *reinterpret_cast<const f32x4*>(src), b = *reinterpret_cast<const f32x4*>(src + 4);
#pragma unroll
      for (int e = 0; e < 8; ++e) po[s][e] = e < 4 ? a[e] : b[e - 4];
    } else {
      const bf16x8 v = load_bf16x8(src);
#pragma unroll
      for (int e = 0; e < 8; ++e) po[s][e] = (float)v[e];
    }
  }
  float M = -INFINITY;
#pragma unroll
  for (int s = 0; s < NS; ++s) M = fmaxf(M, m[s]);
  float L = 0.f;
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const float wgt = (m[s] == -INFINITY) ? 0.f : exp2_fast(m[s] - M);
    L += l[s] * wgt;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += po[s][e] * wgt;
  }
  const float inv = 1.0f / L;
  bf16x8 out;
#pragma unroll
  for (int e = 0; e < 8; ++e) out[e] = (__bf16)(acc[e] * inv);
  *reinterpret_cast<bf16x8*>(o + (size_t)rh * D + sl * 8) = out;
  if (lse && sl == 0) lse[rh] = (M + log2f(L)) * AT_LN2;
}

// Compact-refresh row rewrite: prefix[idx[r]] = ref[r] for K and V.
__global__ __launch_bounds__(256) void prefix_scatter_kernel(const int32_t* idx, int n_ref,
                                                             int row_segs, const uint16_t* k_ref,
                                                             const uint16_t* v_ref, uint16_t* k_pre,
                                                             uint16_t* v_pre) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long total = (long long)n_ref * row_segs;
  if (i >= total) return;
  const int r = (int)(i / row_segs);
  const int sgi = (int)(i - (long long)r * row_segs);
  const size_t dst = (size_t)idx[r] * row_segs + sgi;
  const size_t src = (size_t)r * row_segs + sgi;
  reinterpret_cast<i32x4*>(k_pre)[dst] = reinterpret_cast<const i32x4*>(k_ref)[src];
  reinterpret_cast<i32x4*>(v_pre)[dst] = reinterpret_cast<const i32x4*>(v_ref)[src];
}

// ------------------------------------------------------------------ host
// Largest key split of a pass, which sizes its workspace: until about 256
// workgroups of 8 query tiles exist (one per CU), at least 3 key tiles each.
static int max_split(int base_wgs, int total_key_tiles) {
  int s = 1;
  while (s < 16 && base_wgs * s < 256 && total_key_tiles >= 3 * (2 * s)) s *= 2;
  return s;
}

struct PassShape {
  int n_rows, rows_per_lane, tiles_per_lane, q_tiles_kv, base_wgs, n_pre_tiles, total_key_tiles;
};

static PassShape pass_shape(int n_rows, int rows_per_lane, int n_lanes, int g, int Hkv, int P,
                            int B_keys, int n_key_lanes) {
  PassShape s{};
  s.n_rows = n_rows;
  s.rows_per_lane = rows_per_lane;
  s.tiles_per_lane = (rows_per_lane + 31) / 32;
  s.q_tiles_kv = n_lanes * s.tiles_per_lane * g;
  s.base_wgs = ((s.q_tiles_kv + AT_WAVES - 1) / AT_WAVES) * Hkv;
  s.n_pre_tiles = (P + AT_KT - 1) / AT_KT;
  const int lane_key_tiles = B_keys ? (B_keys + AT_KT - 1) / AT_KT : 0;
  s.total_key_tiles = s.n_pre_tiles + n_key_lanes * lane_key_tiles;
  return s;
}

// Split and query tiles per workgroup (8, or 4 with the other four wavefronts
// loading) of a pass on lane_attn_kernel: the cheapest under its times per
// 64-key tile at D = 128 (MI355X): 1.8 us with 8 query tiles, 1.06 us with 4
// (D = 64: 1.2 and 0.7), ~5 us per round of one workgroup per CU, and for a
// split its partials through memory and a merge launch.  Fitted to 200 sizes and
// trees, each with every split and both tile counts: the choice is 1.8% above the best
// of them on (geometric) average.  4 wins where 8 leave a last round mostly empty
// or would need a split to fill the chip: window of 2563 rows x 32 heads (352 or
// 672 workgroups) 153 us against 162 us, 1024 rows x 32 heads (128 x 2 splits or
// 256) 34 us against 40 us.
//
// Fewer splits than max_split hold other keys per partial; in bf16 that moves the
// output 0.4 to 1.4% further from the 64-bit one (relative error 2.84e-3 -> 2.86e-3
// over 3333 keys), so those partials are fp32 (2.33e-3).
//
// Splits take contiguous shares of all key tiles where there are as many as
// max_split and lane blocks are at most a third of them; otherwise their lane
// blocks are dealt one by one, because a workgroup sees few of a contiguous run
// of blocks or nearly all of it (contiguous -> dealt, lane tiles a third and more of
// the keys: 3 to 6% faster on average, up to 25%; below that 1%).
static void choose_pass(const PassShape& s, int Hkv, int Hq, int D, AttnPass* pass) {
  const int most = max_split(s.base_wgs, s.total_key_tiles);
  const int lane_tiles = s.total_key_tiles - s.n_pre_tiles;
  double best = 1e30;
  for (int t = AT_WAVES; t >= 4; t /= 2)
    for (int ns = 1; ns <= most; ns *= 2) {
      const bool f32 = ns > 1 && ns < most;
      const bool deal = ns > 1 && lane_tiles > 0 && (f32 || 3 * lane_tiles > s.total_key_tiles);
      const long long wgs = (long long)((s.q_tiles_kv + t - 1) / t) * Hkv * ns;
      const double rounds = (double)((wgs + 255) / 256);
      const double tile = (t == AT_WAVES ? 1.8 : 1.06) * (D == 64 ? 0.68 : 1.0);
      double cost = rounds * ((double)((s.total_key_tiles + ns - 1) / ns) * tile + 5.0);
      if (ns > 1) cost += 5.0 + (f32 ? 1.7e-6 : 1.2e-6) * ns * s.n_rows * (double)Hq * D;
      if (cost < best) {
        best = cost;
        *pass = AttnPass{ns, t, f32, deal};
      }
    }
}

// The wavefront-split kernel when its grid fits the chip in one round (one
// workgroup per CU: 256 on MI355X) and no wavefront takes more than 8 key
// units; otherwise the 8-query-tile kernel, whose shared K/V staging wins
// on large grids and long key ranges.  Measured per call after a
// cache-evicting copy (MI355X): LLaDA step shape 16.6 us against 19.7 us,
// Dream 20.9 against 30.0; Long 56.6 against 57.0 (512 workgroups: stays),
// Wide 342 against 222, Wide's refresh rows 87 against 67.
constexpr int kWsplitWaves = 8;
static bool use_wsplit(const PassShape& s, int Hkv, int max_units) {
  return s.q_tiles_kv * Hkv <= 256 && max_units <= 8 * kWsplitWaves;
}

AttnPlan attn_plan(int L, int B, int P, int Hq, int Hkv, int D, int n_refresh) {
  AttnPlan pl{};
  const int g = Hq / Hkv;
  const int pre_units = (P + 31) / 32;
  const PassShape a = pass_shape(L * B, B, L, g, Hkv, P, B, L);
  pl.wsplit_lane = L > 0 && use_wsplit(a, Hkv, pre_units + L * ((B + 31) / 32));
  pl.lane = pl.ref = AttnPass{1, AT_WAVES, false, false};
  int most = 1;
  if (L > 0 && !pl.wsplit_lane) {
    choose_pass(a, Hkv, Hq, D, &pl.lane);
    most = max_split(a.base_wgs, a.total_key_tiles);
  }
  pl.ws_lane = most > 1 ? (size_t)most * L * B * Hq * (D * sizeof(uint16_t) + 2 * sizeof(float)) : 0;
  pl.wsplit_ref = false;
  pl.ws_ref = 0;
  if (n_refresh > 0) {
    const int nl = (n_refresh + 31) / 32;
    const PassShape r = pass_shape(n_refresh, 32, nl, g, Hkv, P, 0, 0);
    pl.wsplit_ref = use_wsplit(r, Hkv, pre_units);
    most = 1;
    if (!pl.wsplit_ref) {
      choose_pass(r, Hkv, Hq, D, &pl.ref);
      most = max_split(r.base_wgs, r.total_key_tiles);
    }
    pl.ws_ref = most > 1 ? (size_t)most * n_refresh * Hq * (D * sizeof(uint16_t) + 2 * sizeof(float)) : 0;
  }
  pl.total = pl.ws_lane > pl.ws_ref ? pl.ws_lane : pl.ws_ref;
  return pl;
}

template <int D>
static hipError_t run_pass(const AttnParams& base, const PassShape& s, const AttnPass& pass,
                           void* ws, hipStream_t stream) {
  const int n_split = pass.n_split;
  AttnParams p = base;
  p.n_rows = s.n_rows;
  p.rows_per_lane = s.rows_per_lane;
  p.tiles_per_lane = s.tiles_per_lane;
  p.q_tiles_kv = s.q_tiles_kv;
  p.n_pre_tiles = s.n_pre_tiles;
  p.total_key_tiles = s.total_key_tiles;
  p.n_split = n_split;
  if (n_split > 1) {
    const size_t n = (size_t)n_split * s.n_rows * p.Hq * D;
    p.part_o = ws;
    p.part_f32 = pass.f32;
    p.part_ml = reinterpret_cast<float*>(static_cast<char*>(ws) + n * (pass.f32 ? 4 : 2));
  }
  p.tpw = pass.tpw;
  p.deal = pass.deal ? ~0ull / ((1ull << n_split) - 1) : 0;   // every n_split-th bit
  const dim3 grid((s.q_tiles_kv + p.tpw - 1) / p.tpw, p.Hkv, n_split);
  hipLaunchKernelGGL(lane_attn_kernel<D>, grid, dim3(AT_THREADS), 0, stream, p);
  if (n_split > 1) {
    const int nrh = s.n_rows * p.Hq;
    const dim3 mgrid((nrh + merge_rows_per_block<D>() - 1) / merge_rows_per_block<D>()), mblock(256);
#define AL_MERGE(NS, T) \
  hipLaunchKernelGGL((attn_merge_kernel<D, NS, T>), mgrid, mblock, 0, stream, \
                     static_cast<const T*>(p.part_o), p.part_ml, nrh, p.o, p.lse)
    switch (n_split) {  // choose_pass takes a power of two <= 16, in fp32 <= 8
      case 2:
        if (pass.f32) AL_MERGE(2, float); else AL_MERGE(2, uint16_t);
        break;
      case 4:
        if (pass.f32) AL_MERGE(4, float); else AL_MERGE(4, uint16_t);
        break;
      case 8:
        if (pass.f32) AL_MERGE(8, float); else AL_MERGE(8, uint16_t);
        break;
      case 16:
        AL_MERGE(16, uint16_t);
        break;
      default:
        return hipErrorInvalidValue;
    }
#undef AL_MERGE
  }
  return hipGetLastError();
}

// Lanes depth first.  A workgroup of the 8-tile kernel loads every lane block
// that one of its lanes sees, and the fullest workgroup sets the time of a
// round; neighbours in this order share most of their ancestors.  (32 random
// lanes of 64 to depth 8, four to a workgroup: at most 11 blocks against 16 in
// index order; 16 of 32 to depth 6, eight to a workgroup: 12 against 15.)
// Index order -> this, us per call (MI355X, random trees): 32 of 64 over 4096 rows x 32
// heads 156.6 -> 150.3, 32 of 32 over 700 31.3 -> 29.1, 64 of 64 over 64 45.4 -> 38.0, 16 of
// 32 over 2048 37.0 -> 36.7, 12 of 64 over 1500 21.8 -> 22.3; chains the same.
// Lane i's parent is the highest of its ancestors (parents come first); any
// order is correct.
static void dfs_order(const unsigned long long* vis, int L, unsigned* order) {
  unsigned long long children[AT_MAX_LANES + 1] = {};   // (the last: roots)
  for (int i = 0; i < L; ++i) {
    const unsigned long long anc = vis[i] & ((1ull << i) - 1);
    children[anc ? 63 - __builtin_clzll(anc) : AT_MAX_LANES] |= 1ull << i;
  }
  int stack[AT_MAX_LANES + 1], top = 0, pos = 0;
  stack[0] = AT_MAX_LANES;
  while (top >= 0) {
    unsigned long long& c = children[stack[top]];
    if (!c) {
      --top;
      continue;
    }
    const int i = __builtin_ctzll(c);
    c &= c - 1;
    order[pos >> 2] |= (unsigned)i << (8 * (pos & 3));
    ++pos;
    stack[++top] = i;
  }
}

template <int D, int KW>
static hipError_t run_pass_wsplit(const AttnParams& base, const PassShape& s, hipStream_t stream) {
  AttnParams p = base;
  p.n_rows = s.n_rows;
  p.rows_per_lane = s.rows_per_lane;
  p.tiles_per_lane = s.tiles_per_lane;
  p.q_tiles_kv = s.q_tiles_kv;
  p.n_pre_tiles = s.n_pre_tiles;
  p.total_key_tiles = s.total_key_tiles;
  p.n_split = 1;
  const unsigned n_wg = (unsigned)(s.q_tiles_kv * p.Hkv);  // one per (query tile, query head)
  hipLaunchKernelGGL((lane_attn_wsplit_kernel<D, KW>), dim3(n_wg), dim3(KW * kWave), 0, stream, p);
  return hipGetLastError();
}

hipError_t launch_lane_attention(const uint16_t* q, const uint16_t* k_lane, const uint16_t* v_lane,
                                 uint16_t* k_pre, uint16_t* v_pre, const unsigned long long* vis,
                                 int L, int B, int P, int Hq, int Hkv, int D, float scale,
                                 const int32_t* refresh_idx, int n_refresh, const uint16_t* q_ref,
                                 const uint16_t* k_ref, const uint16_t* v_ref, uint16_t* o_ref,
                                 float* lse_ref, uint16_t* o, float* lse, void* ws,
                                 hipStream_t stream) {
  const int g = Hq / Hkv;
  const AttnPlan pl = attn_plan(L, B, P, Hq, Hkv, D, n_refresh);
  if (n_refresh > 0) {
    const int row_segs = Hkv * D / 8;
    const long long total = (long long)n_refresh * row_segs;
    hipLaunchKernelGGL(prefix_scatter_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0,
                       stream, refresh_idx, n_refresh, row_segs, k_ref, v_ref, k_pre, v_pre);
  }
  AttnParams p{};
  p.Hq = Hq;
  p.Hkv = Hkv;
  p.g = g;
  p.P = P;
  p.k_pre = k_pre;
  p.v_pre = v_pre;
  p.scale_log2 = scale * 1.4426950408889634f;

  // Lane pass.
  p.q = q;
  p.k_lane = k_lane;
  p.v_lane = v_lane;
  p.o = o;
  p.lse = lse;
  p.B_keys = B;
  p.n_key_lanes = L;
  p.lane_key_tiles = (B + AT_KT - 1) / AT_KT;
  for (int i = 0; i < L; ++i) p.vis[i] = vis[i];
  if (L > 0 && !pl.wsplit_lane) dfs_order(vis, L, p.order);
  hipError_t e = hipSuccess;
  if (L > 0) {  // L = 0: refresh-only call
    const PassShape a = pass_shape(L * B, B, L, g, Hkv, P, B, L);
    if (pl.wsplit_lane)
      e = (D == 64) ? run_pass_wsplit<64, kWsplitWaves>(p, a, stream)
                    : run_pass_wsplit<128, kWsplitWaves>(p, a, stream);
    else
      e = (D == 64) ? run_pass<64>(p, a, pl.lane, ws, stream)
                    : run_pass<128>(p, a, pl.lane, ws, stream);
  }
  if (e != hipSuccess || n_refresh <= 0) return e;

  // Refresh pass: refreshed rows over the updated prefix only.
  AttnParams r = p;
  r.q = q_ref;
  r.k_lane = nullptr;
  r.v_lane = nullptr;
  r.o = o_ref;
  r.lse = lse_ref;
  r.B_keys = 0;
  r.n_key_lanes = 0;
  r.lane_key_tiles = 1;
  for (int i = 0; i < AT_MAX_LANES; ++i) r.vis[i] = 0ull;
  const int nl = (n_refresh + 31) / 32;
  const PassShape b = pass_shape(n_refresh, 32, nl, g, Hkv, P, 0, 0);
  if (pl.wsplit_ref)
    return (D == 64) ? run_pass_wsplit<64, kWsplitWaves>(r, b, stream)
                     : run_pass_wsplit<128, kWsplitWaves>(r, b, stream);
  return (D == 64) ? run_pass<64>(r, b, pl.ref, ws, stream)
                   : run_pass<128>(r, b, pl.ref, ws, stream);
}

}  // namespace al
