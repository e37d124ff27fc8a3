// Internal launch interface of the small-model kernels: a whole decode level, and the chunker with the STEP behind it, of an
// fp32 model in one launch each (paper Section 2.3.3 steps (i) and (ii)-(iii)), one workgroup per chunk or sequence.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/photon.h"

namespace photon {

// All C sub-steps of a local decoder on n_chunks chunks: converter, blocks, final norm; with E != nullptr (token level) logits,
// token choice and the decoder-side embedding fed back, else the item itself fed back.
struct SmallLevel {
  const photon_module_weights* mod = nullptr;     // host struct, fp32 matrices
  const void *conv_w = nullptr, *W_lm = nullptr, *E = nullptr;
  const float *conv_b = nullptr, *cond = nullptr; // cond: row ch conditions chunk ch
  float* units = nullptr;                         // item j of chunk ch at row ch * C + j (nullptr: not wanted, token level only)
  float* logits = nullptr;                        // token level: row ch * ld_logits + j * ld_item
  int64_t ld_logits = 0, ld_item = 0;
  const int32_t* forced = nullptr;                // [n_chunks * C] or nullptr
  int32_t* tokens = nullptr;
  int64_t n_chunks = 0;
  int n_layers = 0, D = 0, F = 0, H = 0, C = 0, R = 0, vocab = 0;
  float eps = 0.f, theta = 0.f;
};
bool small_level_pays(const SmallLevel& a);
int32_t launch_small_level(const SmallLevel& a, hipStream_t st);

// Top chunker on the C_L new units of every sequence and the STEP of the top-level encoder behind it.
struct SmallStep {
  const photon_module_weights* mod = nullptr;
  const void* chunker_w = nullptr;
  const float *chunker_b = nullptr, *bottleneck = nullptr;   // chunker_b may be nullptr; bottleneck: [Bt, C_L * D]
  float *a_hat = nullptr, *x_top = nullptr;                  // [Bt, D] each
  float *k_cache = nullptr, *v_cache = nullptr;
  const int32_t* seq_len = nullptr;                          // counts the new unit already
  int64_t S_max = 0;
  int Bt = 0, n_layers = 0, D = 0, F = 0, H = 0, CL = 0;
  float eps = 0.f, theta = 0.f;
};
bool small_step_pays(const SmallStep& a);
int32_t launch_small_step(const SmallStep& a, hipStream_t st);

}  // namespace photon
