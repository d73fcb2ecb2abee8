// Shared by the LM-head kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stddef.h>
#include <stdint.h>

#include "common.h"

namespace al {

constexpr float LM_LOG2E = 1.4426950408889634f;

struct LmPartial {
  float m;
  float s;
  int idx;
  int pad;
};

// Merge (m2, s2, i2) into (m, s, i): max, rescaled sum, lowest index on ties.
// Commutative, so lanes that exchange states obtain identical bits.
__device__ __forceinline__ void merge_state(float& m, float& s, int& idx, float m2, float s2,
                                            int idx2) {
  if (m2 == -INFINITY) return;
  if (m == -INFINITY) {
    m = m2;
    s = s2;
    idx = idx2;
    return;
  }
  const float M = fmaxf(m, m2);
  s = s * exp2_fast((m - M) * LM_LOG2E) + s2 * exp2_fast((m2 - M) * LM_LOG2E);
  if (m2 > m || (m2 == m && idx2 < idx)) idx = idx2;
  m = M;
}

struct LmTileParams {
  const uint16_t* hidden;
  const int32_t* row_idx;
  const uint16_t* W;
  const uint8_t* sup;
  LmPartial* part;  // [n_nt][COLS][n_vt]
  int N, d, V, eos_id;
  int n_hg, n_vt, n_nt, tiles_total, tiles_per_xcd;
};

// The instances built, X(RA, CBT): 64 RA vocabulary rows x 16 CBT columns.
// Their products must fit a wavefront's 256 registers at two wavefronts per
// SIMD (RA CBT <= 65 beside the two sets of fragments).  RA = 6 and 8 serve at
// most 96 columns on large vocabularies, where the W stream is the bound.  The
// sources lmhead_tile_*.hip hold a few each.
#define AL_LM_INSTANCES(X)                                                                  \
  X(1, 2) X(1, 4) X(1, 6) X(1, 10)                                                         \
  X(2, 2) X(2, 4) X(2, 6) X(2, 8) X(2, 10) X(2, 13)                                         \
  X(4, 2) X(4, 4) X(4, 6) X(4, 8) X(4, 9) X(4, 10) X(4, 11) X(4, 12) X(4, 13) X(4, 14)      \
  X(4, 15) X(4, 16)                                                                         \
  X(5, 2) X(5, 4) X(5, 6) X(5, 8) X(5, 9) X(5, 10) X(5, 11) X(5, 12) X(5, 13)               \
  X(6, 6) X(8, 2) X(8, 4) X(8, 6)

// Stage forms of an instance: 0 one barrier per K stage, 1 two (SPLIT), 2 both
// are built and LmVariant::split chooses.
constexpr int lm_stage_form(int ra, int cbt) { return ra < 6 ? 0 : cbt == 6 ? 1 : 2; }

// Which variant of an instance a call takes.
struct LmVariant {
  bool packed;
  bool ragged;   // loads with per-lane addresses: K past d, W rows past V in an 8-row piece
  bool nt;       // W loaded non-temporally
  bool split;    // of stage form 2: two barriers per K stage
};
template <int RA, int CBT>
void launch_lmhead_tile(const LmTileParams& p, LmVariant v, dim3 grid, hipStream_t stream);

}  // namespace al
