// LM head: partial (max, sum exp, first argmax) of one vocabulary tile x
// column tile, both operands staged through an LDS ring by direct global->LDS
// loads and multiplied by the 16x16x32 bf16 MFMA.
//
// A workgroup of 8 wavefronts (4 wavefront rows x 2 wavefront columns) covers
// 64 RA vocabulary rows (A operand; 2 RA units of 32) x 16 CBT scored rows (B
// operand, "columns"); a wavefront multiplies 16 RA rows x half the columns.
// Workgroups are persistent: at most one per CU, each walking its tiles with
// the loads running ahead over tile boundaries.
//
// What bounds it and why it looks like this (MI355X; cycles per wavefront
// stamped with s_memtime, one box each):
// * With W from HBM and few columns, the W stream; with many, the matrix
//   cores at the clock the power limit leaves (about 1.9 GHz of 2.4 with
//   both busy).  Everything else must hide under those two.
// * Loading W straight into registers, with the hidden rows copied to LDS
//   through registers (the layout before this one), left the matrix cores 40%
//   busy at 614 columns: two wavefronts per SIMD wait for the copies and for
//   a barrier per hidden block.
// * One barrier per 64 K elements.  A barrier costs ~250 cycles whatever lies
//   between (832 cycles of MFMA per 32 elements at 13 fragments took 1390
//   cycles with a barrier per 32 elements, 68% busy with one per 64).
// * Tiles of 384 and 512 rows (RA = 6, 8; at most 96 columns) leave LDS for two
//   stages only.  With one barrier a stage every load has to arrive before
//   the next is issued; a second barrier (SPLIT) keeps the loads in flight.  At
//   96 columns it always wins (LLaDA weight packed, N = 77 160 -> 156 us); with
//   fewer lmhead.hip has the rule and its figures.  RA = 6 fills the chip where RA
//   = 8 would leave a third of it idle (V = 85000, N = 96: 122 -> 107 us).
// * Fragments are read one half-stage (32 elements) ahead into a second
//   register set, so no MFMA waits for an LDS read of its own half-stage.
// * Wavefronts 0-3 issue all loads.  The SIMD serves its older wavefront
//   first, so these finish their MFMAs early and waited for wavefronts 4-7
//   anyway; issue stalls of the loads (each blocks its wavefront, ~40 cycles)
//   fall into that time.
// * The compiler waits for all outstanding loads before any LDS read that
//   follows a direct load of its own; the loads are inline asm (no register
//   is written) and the waits explicit.
// Per call, same box, before -> after: LLaDA weight packed N = 128
// 181 -> 170 us, 205 255 -> 196, 614 622 -> 511; as given N = 77 196 -> 180,
// 205 271 -> 225, 614 713 -> 517; Dream weight packed N = 77 225 -> 169, 128
// 236 -> 178; V = 2048 .. 16384, d = 4096, N = 32: 71 .. 84 -> 22 .. 28 us.
#pragma once
#include "common.h"
#include "lmhead.h"

namespace al {

constexpr int tile_stages(int wb, int hb) {
  int s = 2;
  while (s < 6 && (s + 2) * wb + (s + 1) * hb <= 160 * 1024) ++s;
  return s;
}

template <int RA, int CBT, bool RAGGED, bool PACKED, bool NT, bool SPLIT>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void lmhead_tile_kernel(LmTileParams p) {
  constexpr int CB0 = (CBT + 1) / 2;         // column fragments of wavefronts 0-3
  constexpr int CB1 = CBT - CB0;             // and of wavefronts 4-7
  constexpr int TU = 2 * RA;                 // 32-row units per tile
  constexpr int WB = TU * 4096;              // bytes of W per 64-element K stage
  constexpr int HB = CBT * 2048;             // bytes of hidden rows per stage
  // Stages in LDS: SH of the hidden rows and one more of W, as many as fit
  // (at least two of each).
  constexpr int SH = tile_stages(WB, HB);
  constexpr int SW = (SH + 1) * WB + SH * HB <= 160 * 1024 ? SH + 1 : SH;
  constexpr bool TWO = SH == 2 && SW == 2;
  static_assert(!SPLIT || TWO, "waits of the two-barrier stage");
  constexpr int COLS = 16 * CBT;
  // Wavefronts 0-3 load: LW pieces (1 KB) of W and LH of the hidden rows
  // each per stage (the last hidden pieces may be loaded twice).
  constexpr int LW = TU, NH = 2 * CBT, LH = (NH + 3) / 4, L = LW + LH;
  static_assert(4 * COLS * 12 <= HB, "reduction scratch inside a hidden buffer");
  __shared__ __attribute__((aligned(1024))) char ring[SW * WB + SH * HB];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wr = w & 3, wc = w >> 2;
  const int l16 = lane & 15, k8 = lane >> 4;
  const int d = p.d;
  const int nst = (d + 63) >> 6;
  const int slots = gridDim.x >> 3;
  const int t0 = (int)(blockIdx.x & 7) * p.tiles_per_xcd + (int)(blockIdx.x >> 3);
  const int tend = min(((int)(blockIdx.x & 7) + 1) * p.tiles_per_xcd, p.tiles_total);
  if (t0 >= tend) return;
  auto unit0 = [&](int vt) { return (int)((long long)vt * p.n_hg / p.n_vt); };

  // ---- loads (wavefronts 0-3).  Rows of 128 bytes (64 K elements) sit in
  // LDS as eight 16-byte segments, segment s of row r in slot s ^ f(r) with
  // f(r) = (r & 2) | (r & 8) / 2: the 16 lanes that one LDS cycle serves
  // (0-3, 12-15, 20-23, 24-27 and so on) then touch every bank once.
  auto swz = [](int r) { return (r & 2) | ((r & 8) >> 1); };
  const unsigned ring0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)ring;
  const char* const zero = reinterpret_cast<const char*>(zero_seg16);
  const char* wp = nullptr;               // W: next stage of its tile (uniform)
  int wk = 0, hk = 0;                     // K stage of the next W / hidden load
  unsigned woff = 0;                      // lane offset in a piece
  int wt = t0, wleft = 0, wnv = 0;        // tile, stages left, valid rows (packed: units)
  const char* hp = nullptr;
  unsigned hoff[LH];
  int ht = t0, hleft = 0;
  int todo = TWO ? (tend - t0 + slots - 1) / slots * nst - SH : 1;
  // W as given is walked in a rotated K order, one start per group of eight
  // neighbouring tiles: workgroups in step would otherwise all read one
  // column offset of W at a time, and how those requests spread over the HBM
  // channels depends on where W happens to sit.
  auto rot = [&](int t) { return (int)((long long)(t >> 3) * 13 % nst); };
  auto w_tile = [&](int t) {
    const int vt = t / p.n_nt;
    const int ub = unit0(vt), ue = unit0(vt + 1);
    wleft = nst;
    if constexpr (PACKED) {   // a short tile repeats its last unit
      wp = reinterpret_cast<const char*>(p.W) + (size_t)ub * 4096;
      wnv = ue - ub;
      woff = (unsigned)(wr * 1024 + lane * 16);
    } else {
      const int vb = ub * 32;
      wnv = min(p.V, ue * 32) - vb;
      wp = reinterpret_cast<const char*>(p.W) + (size_t)vb * d * 2;
      woff = (unsigned)((lane >> 3) * 2 * d) + (unsigned)(((lane & 7) ^ swz(8 * wr + (lane >> 3))) * 16);
      wk = rot(t);
      wp += (size_t)wk * 128;
    }
  };
  auto h_tile = [&](int t, bool first) {
    const int nt = t - t / p.n_nt * p.n_nt;
    hleft = nst;
    hk = PACKED ? 0 : rot(t);
    hp = reinterpret_cast<const char*>(p.hidden) + (size_t)hk * 128;
    if (!first && p.n_nt == 1) return;
#pragma unroll
    for (int j = 0; j < LH; ++j) {
      const int r = 8 * min(wr + 4 * j, NH - 1) + (lane >> 3);
      const int n = min(nt * COLS + r, p.N - 1);
      hoff[j] = (unsigned)(p.row_idx ? p.row_idx[n] : n) * (unsigned)(2 * d) +
                (unsigned)(((lane & 7) ^ swz(r)) * 16);
    }
  };
  // Piece J of W's next stage into the W buffer at byte wb of the ring:
  // packed, 16 K elements (k-step wr) of unit J; plain, 8 rows.
  auto load_w = [&](auto j_tag, int wb) {
    constexpr int J = decltype(j_tag)::value;
    const unsigned lds = ring0 + wb + wr * 1024;
    if constexpr (PACKED) {   // (zero past d in memory)
      load_to_lds16<J * 4096, 0, NT>(uniform_ptr(wp + min(J, wnv - 1) * 4096), woff, lds);
    } else if constexpr (RAGGED) {
      const int row = 8 * (4 * J + wr) + (lane >> 3);
      const int sg = (lane & 7) ^ swz(row);
      const char* g = wp + (size_t)min(row, wnv - 1) * (2 * d) + sg * 16;
      load_to_lds16<J * 4096>(wk * 64 + sg * 8 < d ? g : zero, lds);
    } else {
      const int rb = min(8 * (4 * J + wr), wnv - 8);   // whole 8-row pieces (V % 8 == 0)
      load_to_lds16<J * 4096, 0, NT>(uniform_ptr(wp + (size_t)rb * (2 * d)), woff, lds);
    }
  };
  auto load_h = [&](auto j_tag, int hb) {
    constexpr int J = decltype(j_tag)::value;
    const unsigned lds = ring0 + SW * WB + hb + min(wr + 4 * J, NH - 1) * 1024;
    if (RAGGED) {
      const int sg = (lane & 7) ^ swz(8 * min(wr + 4 * J, NH - 1) + (lane >> 3));
      load_to_lds16<0>(hk * 64 + sg * 8 < d ? hp + hoff[J] : zero, lds);
    } else {
      load_to_lds16<0, 0, false>(uniform_ptr(hp), hoff[J], lds);
    }
  };
  // To the next stage.  Past the last tile the loads go on with a tile whose
  // data nobody reads, so that the number in flight stays what the waits say.
  // With two stages in LDS (TWO) every wait but one is for all loads, and they end:
  // todo counts the stages still to load.  (LLaDA weight packed, N = 77: 1.050
  // GB fetched per call -> 1.042.)
  auto w_advance = [&]() {
    wp += PACKED ? (size_t)p.n_hg * 4096 : (size_t)128;
    if (!PACKED && ++wk == nst) {
      wk = 0;
      wp -= (size_t)nst * 128;
    }
    if (--wleft == 0) {
      wt = wt + slots < tend ? wt + slots : wt;
      w_tile(wt);
    }
  };
  auto h_advance = [&]() {
    hp += 128;
    if (++hk == nst) {
      hk = 0;
      hp -= (size_t)nst * 128;
    }
    if (--hleft == 0) {
      ht = ht + slots < tend ? ht + slots : ht;
      h_tile(ht, false);
    }
  };

  // ---- fragments.  Half KK (32 K elements) of a stage.
  // (Packed, fragment i is 16-row half (wr RA + i) % 2 of unit (wr RA + i) / 2:
  // even and odd i have an address of their own.)
  const int g0 = wr * RA;
  const int apk = (k8 >> 1) * 1024 + (k8 & 1) * 512 + l16 * 16;
  const int abase = PACKED ? (g0 >> 1) * 4096 + (g0 & 1) * 256 + apk : g0 * 2048 + l16 * 128;
  const int abase_odd = PACKED ? ((g0 + 1) >> 1) * 4096 + ((g0 + 1) & 1) * 256 + apk : abase + 2048;
  const int bbase = SW * WB + wc * CB0 * 2048 + l16 * 128;
  const int sl0 = (k8 ^ swz(l16)) * 16;       // slot of half 0 (half 1: the other bit 2)

  auto body = [&](auto nc_tag, auto load_tag) {
    constexpr int NC = decltype(nc_tag)::value;
    constexpr bool LOADER = decltype(load_tag)::value;
    bf16x8 a0[RA], b0[NC], a1[RA], b1[NC];
    f32x4 acc[RA][NC];
    auto read1 = [&](bf16x8* a, bf16x8* b, const char* as, const char* bs, auto kk_tag, int i) {
      constexpr int KK = decltype(kk_tag)::value;
      if (i < RA)
        a[i] = *reinterpret_cast<const bf16x8*>(
            as + (i & 1 ? abase_odd - abase : 0) + (PACKED ? KK * 2048 : 0) + (i >> 1) * 4096);
      else
        b[i - RA] = *reinterpret_cast<const bf16x8*>(bs + (i - RA) * 2048);
    };
    int wb = 0, hb = 0;   // ring offsets of the current stage
    if (LOADER) {
      w_tile(t0);
      h_tile(t0, true);
      static_for<SH>([&](auto i) {
        static_for<LW>([&](auto j) { load_w(j, decltype(i)::value * WB); });
        w_advance();
        static_for<LH>([&](auto j) { load_h(j, decltype(i)::value * HB); });
        h_advance();
      });
      if (SW > SH) {
        static_for<LW>([&](auto j) { load_w(j, SH * WB); });
        w_advance();
      }
      wait_loads_and_barrier<(SW - SH) * LW + (SH - 1) * L>();
    } else {
      wait_loads_and_barrier<0>();
    }
    const char* ar = ring + abase + (PACKED ? 0 : sl0);
    const char* ar1 = ring + abase + (PACKED ? 0 : (sl0 ^ 64));
    const char* br = ring + bbase + sl0;
    const char* br1 = ring + bbase + (sl0 ^ 64);
#pragma unroll
    for (int i = 0; i < RA + NC; ++i) read1(a0, b0, ar, br, IntTag<0>{}, i);

    constexpr int C0 = NC > 1 ? 1 : 0;                   // column after which loads start
    constexpr int RPC = (RA + NC + NC - C0 - 1) / (NC - C0);  // reads per column of MFMAs
    constexpr int PPC = (L + NC - C0 - 1) / (NC - C0);        // loads per column
    // One stage.  First half: its fragments are in (a0, b0); the second
    // half's are read meanwhile.  After the barrier everyone has read the
    // stage and the next one is complete: its first half's fragments are
    // read during the second half, and the loads that take the freed
    // buffers are issued (not in a tile's last stage: the epilogue uses the
    // hidden buffer first).  SPLIT: with two stages in LDS that order lets
    // every load arrive before the next is issued; here the next stage need not
    // be complete at the barrier, so that the freed buffers are refilled while
    // it is still arriving, and a second barrier follows its wait.
    auto stage = [&](bool refill) {
      const bool load = LOADER && refill && (!TWO || todo > 0);
      static_for<NC>([&](auto jt) {
        constexpr int j = decltype(jt)::value;
#pragma unroll
        for (int i = 0; i < RPC; ++i)
          if (j * RPC + i < RA + NC) read1(a1, b1, ar1 + wb, br1 + hb, IntTag<1>{}, j * RPC + i);
#pragma unroll
        for (int i = 0; i < RA; ++i) acc[i][j] = mfma16x16x32(a0[i], b0[j], acc[i][j]);
        __builtin_amdgcn_sched_barrier(0);
      });
      if (SPLIT) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      else if (LOADER) wait_loads_and_barrier<(SW - SH) * LW + (SH - 2) * L>();
      else wait_loads_and_barrier<0>();
      const int wn = wb + WB == SW * WB ? 0 : wb + WB, hn = hb + HB == SH * HB ? 0 : hb + HB;
      static_for<NC>([&](auto jt) {
        constexpr int j = decltype(jt)::value;
#pragma unroll
        for (int i = 0; i < RPC; ++i)
          if (!SPLIT && j * RPC + i < RA + NC) read1(a0, b0, ar + wn, br + hn, IntTag<0>{}, j * RPC + i);
#pragma unroll
        for (int i = 0; i < RA; ++i) acc[i][j] = mfma16x16x32(a1[i], b1[j], acc[i][j]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (LOADER && j >= C0) {
          if (load)
            static_for<PPC>([&](auto q) {
              constexpr int x = (j - C0) * PPC + decltype(q)::value;
              if constexpr (x < LH) load_h(IntTag<x>{}, hb);
              else if constexpr (x < L) load_w(IntTag<x - LH>{}, wb);
            });
        }
      });
      if (load) {
        h_advance();
        w_advance();
        if (TWO) --todo;
      }
      if (SPLIT) {
        if (load) wait_loads_and_barrier<L>();
        else wait_loads_and_barrier<0>();
#pragma unroll
        for (int i = 0; i < RA + NC; ++i) read1(a0, b0, ar + wn, br + hn, IntTag<0>{}, i);
      }
      if (refill) {
        wb = wn;
        hb = hn;
      }
    };
    for (int t = t0; t < tend; t += slots) {
#pragma unroll
      for (int i = 0; i < RA; ++i)
#pragma unroll
        for (int j = 0; j < NC; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int k = nst; k > 0; --k) stage(k > 1);
      // Epilogue: lane (l16, k8) holds vocab rows v0 + 16 i + 4 k8 + r of
      // columns 16 j + l16.
      const int vt = t / p.n_nt, nt = t - vt * p.n_nt;
      const int ub = unit0(vt), ue = unit0(vt + 1);
      const int ve = min(p.V, ue * 32);
      const int v0 = ub * 32 + wr * RA * 16 + 4 * k8;
      const int c0 = wc * CB0 * 16 + l16;
      // The stage's hidden buffer was read by everyone before the last barrier
      // and is refilled after the reduction over the four wavefronts of a column.
      float(*red_m)[COLS] = reinterpret_cast<float(*)[COLS]>(ring + SW * WB + hb);
      float(*red_s)[COLS] = red_m + 4;
      int(*red_i)[COLS] = reinterpret_cast<int(*)[COLS]>(red_s + 4);
      const bool eos_here = p.sup && p.eos_id >= ub * 32 && p.eos_id < ve;
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        int excl = -1;
        if (eos_here) {
          const int n = nt * COLS + c0 + 16 * j;
          excl = (n < p.N && p.sup[n]) ? p.eos_id : -1;
        }
        float m = -INFINITY;
        int idx = 0x7fffffff;
#pragma unroll
        for (int i = 0; i < RA; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int v = v0 + 16 * i + r;
            const float z = (v < ve && v != excl) ? acc[i][j][r] : -INFINITY;
            acc[i][j][r] = z;
            const bool gt = z > m;
            m = gt ? z : m;
            idx = gt ? v : idx;
          }
        const float m0 = (m == -INFINITY) ? 0.f : m;
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < RA; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) s += exp2_fast((acc[i][j][r] - m0) * LM_LOG2E);
        merge_state(m, s, idx, __shfl_xor(m, 16, kWave), __shfl_xor(s, 16, kWave), __shfl_xor(idx, 16, kWave));
        merge_state(m, s, idx, __shfl_xor(m, 32, kWave), __shfl_xor(s, 32, kWave), __shfl_xor(idx, 32, kWave));
        if (k8 == 0) {
          red_m[wr][c0 + 16 * j] = m;
          red_s[wr][c0 + 16 * j] = s;
          red_i[wr][c0 + 16 * j] = idx;
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      for (int col = tid; col < COLS; col += 512) {
        float m = red_m[0][col], s = red_s[0][col];
        int idx = red_i[0][col];
#pragma unroll
        for (int ww = 1; ww < 4; ++ww) merge_state(m, s, idx, red_m[ww][col], red_s[ww][col], red_i[ww][col]);
        LmPartial q;
        q.m = m;
        q.s = s;
        q.idx = idx;
        q.pad = 0;
        p.part[((size_t)nt * COLS + col) * p.n_vt + vt] = q;
      }
      // The stores drain here so that the loop's load counts hold.
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      if (t + slots < tend) {
        if (LOADER && (!TWO || todo > 0)) {
          static_for<LH>([&](auto j) { load_h(j, hb); });
          static_for<LW>([&](auto j) { load_w(j, wb); });
          h_advance();
          w_advance();
          if (TWO) --todo;
        }
        wb = wb + WB == SW * WB ? 0 : wb + WB;
        hb = hb + HB == SH * HB ? 0 : hb + HB;
      }
    }
  };
  if (wc == 0) body(IntTag<CB0>{}, IntTag<1>{});
  else body(IntTag<CB1>{}, IntTag<0>{});
  // (Every wavefront has waited for its loads: none lands after the end.)
}
// ------------------------------------------------------------------ host
template <int RA, int CBT, bool SPLIT>
void launch_form(const LmTileParams& p, LmVariant v, dim3 grid, hipStream_t stream) {
#define AL_LM_TILE(RG, PK, NTL) \
  hipLaunchKernelGGL((lmhead_tile_kernel<RA, CBT, RG, PK, NTL, SPLIT>), grid, dim3(512), 0, stream, p)
  if (!v.packed) {
    if (v.ragged) AL_LM_TILE(true, false, false);
    else AL_LM_TILE(false, false, false);
  } else if (v.nt) {
    if (v.ragged) AL_LM_TILE(true, true, true);
    else AL_LM_TILE(false, true, true);
  } else {
    if (v.ragged) AL_LM_TILE(true, true, false);
    else AL_LM_TILE(false, true, false);
  }
#undef AL_LM_TILE
}
template <int RA, int CBT>
void launch_lmhead_tile(const LmTileParams& p, LmVariant v, dim3 grid, hipStream_t stream) {
  constexpr int form = lm_stage_form(RA, CBT);
  if constexpr (form != 0)
    if (form == 1 || v.split) return launch_form<RA, CBT, true>(p, v, grid, stream);
  if constexpr (form != 1) launch_form<RA, CBT, false>(p, v, grid, stream);
}

#define AL_LM_INSTANCE(RA, CBT) \
  template void launch_lmhead_tile<RA, CBT>(const LmTileParams&, LmVariant, dim3, hipStream_t);

}  // namespace al
