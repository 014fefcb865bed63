// Host-side state object shared by the runtime sources of libthor.
#pragma once

#include <hip/hip_runtime.h>

#include <map>
#include <string>
#include <vector>

#include "kernels.h"

struct TimedLaunch {
  std::string family;
  hipEvent_t start, stop;
};

// Kernel families with a tuned workgroup size (wavefronts per workgroup).
enum { FAM_LARGE = 0, FAM_SLOW, FAM_HMOM, FAM_VERT, FAM_COUNT };
static const char *const kFamily[FAM_COUNT] = {"large", "slow", "hmom", "vert"};

// Default wavefronts per workgroup for `waves` gather-mapping wavefronts in a
// launch (the tuner may choose others).  The card holds 3072 wavefronts of phase
// V at a time (3 per SIMD) and 2048 of phase M, the slow terms and k_large1
// (FP64).  Up to a few rounds of them, single wavefronts fill the compute units
// most evenly: a large step takes 160 us with 1 and 184 with 4 at g4 L20 (214
// wavefronts), 1025 and 1079 at g6 L32 (5121); at 10241 it makes little
// difference (g7 L16 2253 / 2249, mixed 1423 / 1422; g6 L64 2072 / 2033, mixed
// 1220 / 1229).  With more rounds the rows that neighbouring wavefronts share in
// L1 count, with 1 / 4 / 8:
//   g7 L20  13654  2899 / 2819 / 2810, mixed 1870 / 1831 / 1890
//   g7 L24  16385  3456 / 3335 / 3374, mixed 2213 / 2167 / 2248
//   g7 L32  20481  4370 / 4260 / 4279, mixed 2796 / 2787 / 2859
//   g7 L40  27307  5659 / 5394 / 5342, mixed 3656 / 3549 / 3617
// and by kernel (g7 L40) V 209 / 202.5 / 193, mixed 137 / 134 / 144, M 133 / 125
// / 131, slow terms 216 / 202 / 203, large step 546 / 515 / 499.  The line lies
// between 10241 and 13654.  An ensemble's launch holds planets of several sizes:
// 9 planets 3925 us per large step with 4 throughout, 3960 with the 8s, 3983
// with 1.  The tuner finds a little more (2 for the slow terms at g6, 8 for an
// ensemble's).
inline void default_wpb(long waves, bool mixed, bool ensemble, int wpb[FAM_COUNT]) {
  const bool many = waves > 12288;
  wpb[FAM_LARGE] = many ? (ensemble ? 4 : 8) : 1;
  wpb[FAM_SLOW] = many ? 4 : 1;
  wpb[FAM_HMOM] = many ? 4 : 1;
  wpb[FAM_VERT] = many ? (mixed || ensemble ? 4 : 8) : 1;
}

struct thor_state {
  int precision = THOR_FP64;
  thor::Consts c{};
  // f[0] and f[1] are the same buffers with the state set and the Phi[t] set
  // exchanged; between large steps the state is in the *_t buffers of
  // f[parity], and every large step flips the parity.
  thor::Fields<double> f64[2]{};
  thor::Fields<float> f32[2]{};
  int parity = 0;
  int wpb[FAM_COUNT] = {1, 1, 1, 1};   // set by default_wpb
  hipStream_t stream = nullptr;
  hipStream_t cap_stream = nullptr;
  std::map<int, hipGraphExec_t> graphs;   // key: n_acoustic * 2 + parity
  bool timing = false;
  std::vector<TimedLaunch> timed;
  std::vector<hipEvent_t> event_pool;
  size_t next_event = 0;
  int64_t n_col = 0;
  int n_lev = 0;
  bool in_batch = false;   // members of an ensemble are stepped by thor_batch_step
};

