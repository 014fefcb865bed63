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
// launch (the tuner may choose others).  Up to about four rounds of the
// card's 3072 slots, single wavefronts fill the compute units most evenly: a
// large step takes 160 us with 1 and 184 with 4 at g4 L20 (214 wavefronts),
// 1025 and 1079 at g6 L32 (5121; V 35.5 / 37.5 us, M 23.7 / 25.4), no
// difference at g6 L64 (10241: V 76.4 / 77.1, M 53.7 / 53.5).  With more
// rounds the rows that neighbouring wavefronts share in L1 count: g7 L48
// (32769) V 249 us with 1, 239 with 4, 234 with 8 (in the mixed form 4 is
// the better: g7 L40 135 against 147), M 170, 166, 187, slow terms 261, 247,
// 254, large step 685, 662, 644.  An ensemble's launch holds planets of
// several sizes: 9 planets 3925 us per large step with 4 throughout, 3960
// with the 8s, 3983 with 1.
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

