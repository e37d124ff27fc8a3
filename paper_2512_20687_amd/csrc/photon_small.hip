// Small fp32 models: one launch per decode level and one for chunker + STEP, instead of five or more launches per block.
//
// What bounds a step of a small model is its launches: 64 of them, 3.4 us each with next to nothing to do, and as many trips
// through the host's queue.  The chunks of a level are independent of each other (paper Section 2.1.2), so one workgroup
// takes a chunk through everything the level does: activations, window and rotary angles stay in LDS, phases meet at
// workgroup barriers, and the matrices (a few hundred KB) stream from the caches.  Sixteen lanes hold a matrix row, the 32
// groups of a workgroup take 32 rows a pass; the first rows of a phase's matrix are requested a phase ahead.  A compute unit
// takes in 60 to 75 bytes per ns, which is what limits the sizes this pays for (SmallTimes).  A step of the tiny
// configuration (D = 64, one block): 297 us enqueued launch by launch, 100 us so (levels 34 and 43, chunker and STEP 14).
// Eight waves with 8 pieces each in flight: 44 us for the token level alone; four with 16 52 us, sixteen with 4 60 us.
#include "photon_small.h"

#include <type_traits>

#include "photon_attn.h"
#include "photon_device.h"
#include "photon_host.h"

namespace photon {

namespace {

constexpr int SM_THREADS = 512, SM_WAVES = SM_THREADS / 64, SM_GROUPS = SM_THREADS / 16;
constexpr int CHOOSE_WAVES = CHOOSE_THREADS / 64;
constexpr int SM_MAX_LAYERS = 8, SM_MAX_D = 128, SM_MAX_CACHE = 2048;
constexpr int SM_AHEAD = 8;                              // float4 per lane requested a phase ahead
constexpr size_t SM_LDS_LIMIT = 64 * 1024;

struct SmallLayer { const float *g1, *wqkv, *wo, *g2, *wgu, *wd; };
struct SmallModule { SmallLayer layer[SM_MAX_LAYERS]; const float* g_final; };

__host__ __device__ constexpr int pad64(int n) { return n <= 64 ? 64 : (n + 127) / 128 * 128; }   // whole k steps: 1 or 2, as the kernels are built
__host__ __device__ constexpr int pad256(int n) { return (n + 255) / 256 * 256; }

// N outputs of K-long rows; pair: N gate rows, then N up rows, taken in turn (pass 2 q: gate rows of 32 outputs, 2 q + 1: up).
struct Matrix { const float* w; int N, K; bool pair; };

struct Batch { float4_t w[SM_AHEAD]; };

// The thread's number, formed anew: addresses derived from it are not kept over the loops, where they would take most of the
// registers (kept: 256 registers and 125 to 195 spilled).
__device__ __forceinline__ int fresh_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Rows of a batch and k steps of 64 that a batch covers: with KS > 0 the rows are KS steps long (K <= 64 KS), else any length
// is walked in batches of four steps.
template <int KS> struct Deal {
  static constexpr int STEPS = KS > 0 ? KS : 4, PASSES = SM_AHEAD / STEPS;
  static_assert(STEPS * PASSES == SM_AHEAD, "a batch is whole");
};

// Bounds-checked view of a matrix: what lies outside reads as zero, with no branch or mask in front of the load.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t matrix_view(const Matrix& m) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(m.w), 0, (m.pair ? 2 : 1) * m.N * m.K * 4, 0x00020000);
}

// This lane's pieces of the passes from pass0 on and the k steps from ks0 on.
template <int KS> __device__ __forceinline__ void request(const Matrix& m, int pass0, int ks0, Batch& b) {
  const int tid = fresh_tid(), grp = tid >> 4, l16 = tid & 15;
  const __amdgpu_buffer_rsrc_t view = matrix_view(m);
  int at[Deal<KS>::STEPS];
#pragma unroll
  for (int t = 0; t < Deal<KS>::STEPS; ++t) {
    const int k = (ks0 + t) * 64 + l16 * 4;
    at[t] = k < m.K ? (grp * m.K + k) * 4 : 0x40000000;             // past the row's end: past the matrix (which is below 1 GiB)
  }
#pragma unroll
  for (int p = 0; p < Deal<KS>::PASSES; ++p) {
    const int pass = pass0 + p, row_at = ((m.pair ? pass >> 1 : pass) * SM_GROUPS + (m.pair && (pass & 1) ? m.N : 0)) * m.K * 4;
#pragma unroll
    for (int t = 0; t < Deal<KS>::STEPS; ++t)
      b.w[p * Deal<KS>::STEPS + t] = __builtin_bit_cast(float4_t, __builtin_amdgcn_raw_buffer_load_b128(view, at[t] + row_at, 0, 0));
  }
}

// Sums of P values over the 16 lanes of a group; lane l is left with the sum of value l % P.  Every exchange is made by all
// lanes, the choice behind it.
template <int P> __device__ __forceinline__ float sums_to_lanes(float (&v)[P], int l16) {
  static_assert((P & (P - 1)) == 0 && P <= 16, "");
  // lanes 4 (8) apart: a lane below takes from above, a lane above from below
  constexpr int SHL4 = 0x104, SHR4 = 0x114, SHL8 = 0x108, SHR8 = 0x118, ROR4 = 0x124, ROR8 = 0x128;
  auto halve = [&](int i, int bit, auto below, auto above) {
    const float lo = v[2 * i] + dpp<decltype(below)::value>(v[2 * i]), hi = v[2 * i + 1] + dpp<decltype(above)::value>(v[2 * i + 1]);
    v[i] = (l16 & bit) ? hi : lo;
  };
  using X1 = std::integral_constant<int, DPP_XOR1>;
  using X2 = std::integral_constant<int, DPP_XOR2>;
#pragma unroll
  for (int i = 0; i < P / 2; ++i) halve(i, 1, X1{}, X1{});
#pragma unroll
  for (int i = 0; i < P / 4; ++i) halve(i, 2, X2{}, X2{});
#pragma unroll
  for (int i = 0; i < P / 8; ++i) halve(i, 4, std::integral_constant<int, SHL4>{}, std::integral_constant<int, SHR4>{});
#pragma unroll
  for (int i = 0; i < P / 16; ++i) halve(i, 8, std::integral_constant<int, SHL8>{}, std::integral_constant<int, SHR8>{});
  float y = v[0];
  if constexpr (P < 2) y += dpp<DPP_XOR1>(y);
  if constexpr (P < 4) y += dpp<DPP_XOR2>(y);
  if constexpr (P < 8) y += dpp<ROR4>(y);
  if constexpr (P < 16) y += dpp<ROR8>(y);
  return y;
}

__device__ __forceinline__ float wave_max(float x) {
  x = fmaxf(x, dpp<DPP_XOR1>(x));
  x = fmaxf(x, dpp<DPP_XOR2>(x));
  x = fmaxf(x, dpp<DPP_HALF_MIRROR>(x));
  x = fmaxf(x, dpp<DPP_MIRROR>(x));
  typedef uint32_t uint2_native __attribute__((ext_vector_type(2)));
  const uint2_native r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  const uint2_native h = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(h[0]), __uint_as_float(h[1]));
}
__device__ __forceinline__ uint32_t wave_min(uint32_t x) {
  auto lane = [](uint32_t v, auto ctrl) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, 0xf, 0xf, false); };
  x = min(x, lane(x, std::integral_constant<int, DPP_XOR1>{}));
  x = min(x, lane(x, std::integral_constant<int, DPP_XOR2>{}));
  x = min(x, lane(x, std::integral_constant<int, DPP_HALF_MIRROR>{}));
  x = min(x, lane(x, std::integral_constant<int, DPP_MIRROR>{}));
  typedef uint32_t uint2_native __attribute__((ext_vector_type(2)));
  const uint2_native r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  x = min(r[0], r[1]);
  const uint2_native h = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return min(h[0], h[1]);
}

// y[row, n] = W[n] . x[row] for `rows` rows of x in LDS (pitch xp, zero beyond K up to whole batches of k steps).  done(n, row, y)
// is called once per output (pair: with the up and the gate row's sum), by a lane per pass of a batch, which all hold the sums.
// `cur` holds the first batch on entry; `next_first` requests the next matrix's, under the last batch's arithmetic.
template <int KS, int MR, class Done, class Next>
__device__ __forceinline__ void contract_rows(const Matrix& m, const float* x, int xp, int rows, Batch& cur, Next next_first, Done done) {
  constexpr int STEPS = Deal<KS>::STEPS, PASSES = Deal<KS>::PASSES;
  const int tid = fresh_tid(), grp = tid >> 4, l16 = tid & 15;
  const int passes = (m.N + SM_GROUPS - 1) / SM_GROUPS * (m.pair ? 2 : 1), k_batches = KS > 0 ? 1 : (m.K + 255) / 256;
  float4_t xv[MR][STEPS];
  auto read_x = [&](int ks0) {
#pragma unroll
    for (int r = 0; r < MR; ++r)
#pragma unroll
      for (int t = 0; t < STEPS; ++t)
        xv[r][t] = r < rows ? *reinterpret_cast<const float4_t*>(x + r * xp + (ks0 + t) * 64 + l16 * 4) : float4_t{0.f, 0.f, 0.f, 0.f};
  };
  if (KS > 0) read_x(0);
  for (int p0 = 0; p0 < passes; p0 += PASSES) {
    float acc[MR][PASSES];
#pragma unroll
    for (int r = 0; r < MR; ++r)
#pragma unroll
      for (int p = 0; p < PASSES; ++p) acc[r][p] = 0.f;
    for (int kb = 0; kb < k_batches; ++kb) {
      Batch nxt;
      const bool wraps = kb + 1 == k_batches, more = !wraps || p0 + PASSES < passes;
      if (more) request<KS>(m, wraps ? p0 + PASSES : p0, wraps ? 0 : (kb + 1) * STEPS, nxt);
      else next_first();
      if (KS <= 0) read_x(kb * STEPS);
#pragma unroll
      for (int p = 0; p < PASSES; ++p) {
        if (p0 + p >= passes) continue;
#pragma unroll
        for (int t = 0; t < STEPS; ++t)
#pragma unroll
          for (int r = 0; r < MR; ++r) {
            const float4_t w = cur.w[p * STEPS + t], v = xv[r][t];
            acc[r][p] = fmaf(w.x, v.x, fmaf(w.y, v.y, fmaf(w.z, v.z, fmaf(w.w, v.w, acc[r][p]))));
          }
      }
      if (more) cur = nxt;
    }
#pragma unroll
    for (int r = 0; r < MR; ++r) {
      const float y = sums_to_lanes<PASSES>(acc[r], l16);
      const float gate = m.pair ? dpp<DPP_XOR1>(y) : 0.f;             // of the lane below, which holds the pass before
      const int pass = p0 + l16, n = (m.pair ? pass >> 1 : pass) * SM_GROUPS + grp;
      if (r < rows && l16 < PASSES && n < m.N && (!m.pair || (l16 & 1))) done(n, r, y, gate);
    }
  }
}

// Barrier between phases that exchange LDS only: what is requested from memory stays in flight (__syncthreads waits for it: the
// tiny model's token level 64 us instead of 52, with four waves).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// 1 / rms of a row in LDS (every wave forms it for itself: no barrier).
__device__ __forceinline__ float row_scale(const float* x, int D, float eps) {
  float ss = 0.f;
  for (int d = fresh_tid() & 63; d < D; d += 64) ss = fmaf(x[d], x[d], ss);
  return 1.0f / sqrtf(wave_sum(ss) / (float)D + eps);
}

// LDS of both kernels, in floats: rows padded to the k steps that are walked (the padding stays zero), window rows to a pitch
// that spreads the positions over the banks.
struct SmallLds {
  int DP, FP, WP, gains, h, mid, xn, attn, act, qkv, kc, vc, rot, red, extra, total;
};
__host__ __device__ inline SmallLds small_lds(int rows, int D, int F, int layers, int window, int angles, int extra_floats) {
  SmallLds s;
  s.DP = pad64(D); s.FP = pad256(F > 0 ? F : 1); s.WP = s.DP + 4;
  int at = 0;
  auto take = [&](int n) { const int p = at; at += (n + 3) / 4 * 4; return p; };
  s.gains = take((2 * layers + 1) * s.DP);
  s.h = take(rows * s.DP); s.mid = take(rows * s.DP); s.xn = take(rows * s.DP); s.attn = take(rows * s.DP);
  s.act = take(rows * s.FP); s.qkv = take(rows * 3 * s.DP);
  s.kc = take(layers * window * s.WP); s.vc = take(layers * window * s.WP);
  s.rot = take(2 * angles);
  s.red = take(2 * CHOOSE_WAVES + 4);
  s.extra = take(extra_floats);
  s.total = at;
  return s;
}

__device__ __forceinline__ void load_gains(const SmallModule& mod, int n_layers, int D, int DP, float* gains) {
  for (int i = 0; i <= 2 * n_layers; ++i) {
    const float* g = i == 2 * n_layers ? mod.g_final : i & 1 ? mod.layer[i >> 1].g2 : mod.layer[i >> 1].g1;
    if (g == nullptr) continue;                          // no feed-forward
    for (int d = threadIdx.x; d < D; d += SM_THREADS) gains[i * DP + d] = g[d];
  }
}

// Everything of a block behind its attention, whose rows are in `attn`; leaves the residual stream in h and, times the next
// norm's gain (`g_next`), in xn.  `b`: the O projection's first batch; next_first() requests what comes behind the block, into `a`.
template <int KS, int MR, class Next>
__device__ __forceinline__ void small_block_tail(const SmallLayer& w, float* lds, const SmallLds& s, int D, int F, int rows, float eps,
                                                 const float* g2, const float* g_next, Batch& a, Batch& b, Next next_first) {
  float *h = lds + s.h, *mid = lds + s.mid, *xn = lds + s.xn, *act = lds + s.act;
  const Matrix wo{w.wo, D, D, false}, wgu{w.wgu, F, D, true}, wd{w.wd, D, F, false};
  if (F == 0) {
    contract_rows<KS, MR>(wo, lds + s.attn, s.DP, rows, b, next_first, [&](int n, int r, float y, float) {
      const float v = h[r * s.DP + n] + y;
      h[r * s.DP + n] = v;
      xn[r * s.DP + n] = v * g_next[n];
    });
    lds_barrier();
    return;
  }
  contract_rows<KS, MR>(wo, lds + s.attn, s.DP, rows, b, [&] { request<KS>(wgu, 0, 0, a); }, [&](int n, int r, float y, float) {
    const float v = h[r * s.DP + n] + y;
    mid[r * s.DP + n] = v;
    xn[r * s.DP + n] = v * g2[n];
  });
  lds_barrier();
  float rs[MR];
#pragma unroll
  for (int r = 0; r < MR; ++r) rs[r] = r < rows ? row_scale(mid + r * s.DP, D, eps) : 0.f;
  contract_rows<KS, MR>(wgu, xn, s.DP, rows, a, [&] { request<0>(wd, 0, 0, b); },
                        [&](int n, int r, float up, float gate) { act[r * s.FP + n] = silu(gate * rs[r]) * (up * rs[r]); });
  lds_barrier();
  contract_rows<0, MR>(wd, act, s.FP, rows, b, next_first, [&](int n, int r, float y, float) {
    const float v = mid[r * s.DP + n] + y;
    h[r * s.DP + n] = v;
    xn[r * s.DP + n] = v * g_next[n];
  });
  lds_barrier();
}

struct SmallLevelArgs {
  SmallModule mod;
  const float *conv_w, *conv_b, *W_lm, *E, *cond;
  float *units, *logits;
  const int32_t* forced;
  int32_t* tokens;
  int64_t ld_logits, ld_item;
  int n_layers, D, F, H, C, R, vocab;
  float eps, scale_log2e;
  double freq_ratio;                                     // theta^(-2 / d_h); 0: no rotation
};

static_assert(PHOTON_MAX_WINDOW * 4 <= 64, "four lanes of a wave hold a window position");

// KS: 64-wide k steps of a row of D.  MR: rows of the first sub-step (converter length R <= MR); further sub-steps have one row.
template <int KS, int MR>
__global__ __launch_bounds__(SM_THREADS) void small_level_kernel(const SmallLevelArgs p) {
  extern __shared__ __align__(16) float lds[];
  const int D = p.D, F = p.F, W = p.R + p.C - 1, d_h = D / p.H, half = d_h / 2;
  const SmallLds s = small_lds(MR, D, F, p.n_layers, W, W * half, 0);
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int64_t chunk = blockIdx.x;
  float *h = lds + s.h, *xn = lds + s.xn, *qkv = lds + s.qkv, *attn = lds + s.attn, *gains = lds + s.gains;
  float *cosv = lds + s.rot, *sinv = cosv + W * half;
  const bool token_level = p.E != nullptr;

  Batch a, b;
  const Matrix conv{p.conv_w, p.R * D, D, false}, head{p.W_lm, p.vocab, D, false};
  auto wqkv = [&](int layer) { return Matrix{p.mod.layer[layer].wqkv, 3 * D, D, false}; };
  request<KS>(conv, 0, 0, b);
  for (int i = tid; i < s.total; i += SM_THREADS) lds[i] = 0.f;   // the padding has to be zero
  lds_barrier();
  load_gains(p.mod, p.n_layers, D, s.DP, gains);
  for (int d = tid; d < D; d += SM_THREADS) lds[s.mid + d] = p.cond[chunk * D + d];
  // angles of the window's positions (below 16: single precision is exact enough for sine and cosine; the frequencies are powers
  // in double)
  for (int i = tid; i < W * half; i += SM_THREADS) {
    double base = p.freq_ratio, f = p.freq_ratio == 0.0 ? 0.0 : 1.0;
    for (int e = i % half; e != 0; e >>= 1) {
      if (e & 1) f *= base;
      base *= base;
    }
    sincosf((float)(i / half) * (float)f, &sinv[i], &cosv[i]);
  }
  lds_barrier();
  contract_rows<KS, 1>(conv, lds + s.mid, s.DP, 1, b, [&] { request<KS>(wqkv(0), 0, 0, a); }, [&](int n, int, float y, float) {
    const int r = n / D, d = n - r * D;
    const float v = y + p.conv_b[n];
    h[r * s.DP + d] = v;
    xn[r * s.DP + d] = v * gains[d];
  });
  lds_barrier();

  for (int j = 0; j < p.C; ++j) {
    const int q_len = j == 0 ? p.R : 1, q_pos = j == 0 ? 0 : p.R + j - 1;
    for (int i = 0; i < p.n_layers; ++i) {
      float rs[MR];
#pragma unroll
      for (int r = 0; r < MR; ++r) rs[r] = r < q_len ? row_scale(h + r * s.DP, D, p.eps) : 0.f;
      contract_rows<KS, MR>(wqkv(i), xn, s.DP, q_len, a, [&] { request<KS>(Matrix{p.mod.layer[i].wo, D, D, false}, 0, 0, b); },
                            [&](int n, int r, float y, float) { qkv[r * 3 * s.DP + n] = y * rs[r]; });
      lds_barrier();
      // A wave takes a head: rotation, append to the window and attention of its rows in turn (what a row attends to was written
      // by the same wave).  Four lanes share a window position.
      for (int hd = wave; hd < p.H; hd += SM_WAVES) {
        float *kc = lds + s.kc + i * W * s.WP + hd * d_h, *vc = lds + s.vc + i * W * s.WP + hd * d_h;
        for (int r = 0; r < q_len; ++r) {
          const int pos = q_pos + r;
          float* q = qkv + r * 3 * s.DP + hd * d_h;
          for (int d = lane; d < half; d += 64) {
            const float c = cosv[pos * half + d], sn = sinv[pos * half + d];
            const float q0 = q[d], q1 = q[d + half], k0 = q[D + d], k1 = q[D + d + half];
            q[d] = q0 * c - q1 * sn;
            q[d + half] = q1 * c + q0 * sn;
            kc[pos * s.WP + d] = k0 * c - k1 * sn;
            kc[pos * s.WP + d + half] = k1 * c + k0 * sn;
            vc[pos * s.WP + d] = q[2 * D + d];
            vc[pos * s.WP + d + half] = q[2 * D + d + half];
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
          const int t = lane >> 2;
          float score = 0.f;
          if (t <= pos) {
#pragma unroll 4
            for (int d = lane & 3; d < d_h; d += 4) score = fmaf(q[d], kc[t * s.WP + d], score);
          }
          score = group_sum<4>(score) * p.scale_log2e;
          const float mx = wave_max(t <= pos ? score : NEG_BIG);
          const float weight = t <= pos ? fast_exp2(score - mx) : 0.f;
          const float inv = 4.f / wave_sum(weight);                  // (four lanes hold each weight)
          for (int d = lane; d < d_h; d += 64) {
            float o = 0.f;
#pragma unroll 4
            for (int u = 0; u <= pos; ++u)
              o = fmaf(__uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(weight), u * 4)), vc[u * s.WP + d], o);
            attn[r * s.DP + hd * d_h + d] = o * inv;
          }
        }
      }
      lds_barrier();
      const bool last = i + 1 == p.n_layers;
      const float* g_next = gains + (last ? 2 * p.n_layers : 2 * (i + 1)) * s.DP;
      small_block_tail<KS, MR>(p.mod.layer[i], lds, s, D, F, q_len, p.eps, gains + (2 * i + 1) * s.DP, g_next, a, b,
                               [&] { request<KS>(!last ? wqkv(i + 1) : token_level ? head : wqkv(0), 0, 0, a); });
    }
    // item j: final norm of the chunk's last row
    const int at = q_len - 1;
    const float rf = row_scale(h + at * s.DP, D, p.eps);
    if (p.units != nullptr)
      for (int d = tid; d < D; d += SM_THREADS) p.units[(chunk * p.C + j) * D + d] = h[at * s.DP + d] * rf * gains[2 * p.n_layers * s.DP + d];
    if (token_level) {
      float best = -INFINITY;
      int column = NO_COLUMN;
      float* lg = p.logits + chunk * p.ld_logits + j * p.ld_item;
      contract_rows<KS, 1>(head, xn + at * s.DP, s.DP, 1, a, [&] { request<KS>(wqkv(0), 0, 0, b); }, [&](int n, int, float y, float) {
        const float v = y * rf;
        lg[n] = v;
        if (v > best || v != v || column == NO_COLUMN) { best = v; column = n; }   // columns come in increasing order; a NaN stays
      });
      auto meet = [&] {                                  // the wave's best value, and the first column that has it
        const float top = wave_max(best);
        column = (int)wave_min(best == top ? (uint32_t)column : (uint32_t)NO_COLUMN);
        best = top;
      };
      const bool nan_here = __any(best != best);
      meet();
      float* bv = lds + s.red;
      int *bc = reinterpret_cast<int*>(bv + CHOOSE_WAVES), *chosen = bc + CHOOSE_WAVES;
      if (lane == 0) { bv[wave] = nan_here ? NAN : best; bc[wave] = column; }
      lds_barrier();
      best = bv[lane & (SM_WAVES - 1)];
      const bool nan_row = __any(best != best);
      if (nan_row) {                                     // a NaN among the logits: read them again, in the order that decides then
        __syncthreads();
#pragma unroll 1
        for (int w = wave; w < CHOOSE_WAVES; w += SM_WAVES) {
          best_of_share(lg, p.ld_logits, p.vocab, w * 64 + lane, best, column);
          best_of_wave(best, column);
          if (lane == 0) { bv[w] = best; bc[w] = column; }
        }
        lds_barrier();
      }
      if (wave == 0) {
        if (nan_row) {
          best = bv[0]; column = bc[0];
          for (int w = 1; w < CHOOSE_WAVES; ++w) take_better(bv[w], bc[w], best, column);
        } else {
          column = bc[lane & (SM_WAVES - 1)];
          meet();
        }
        if (lane == 0) {
          const int64_t flat = chunk * p.C + j;
          if (p.forced != nullptr) column = p.forced[flat];
          column = column < 0 ? 0 : column >= p.vocab ? p.vocab - 1 : column;
          p.tokens[flat] = column;
          *chosen = column;
        }
      }
      lds_barrier();
      if (j + 1 < p.C) {
        for (int d = tid; d < D; d += SM_THREADS) {
          const float v = p.E[(int64_t)*chosen * D + d];
          h[d] = v;
          xn[d] = v * gains[d];
        }
        a = b;
        lds_barrier();
      }
    } else if (j + 1 < p.C) {
      lds_barrier();                                   // every wave has its statistic of the row that is replaced (and of row 0)
      for (int d = tid; d < D; d += SM_THREADS) {
        const float v = h[at * s.DP + d] * rf * gains[2 * p.n_layers * s.DP + d];
        h[d] = v;                                        // at > 0: row 0 is replaced by the same thread's element of row `at`
        xn[d] = v * gains[d];
      }
      lds_barrier();
    }
  }
}

struct SmallStepArgs {
  SmallModule mod;
  const float *chunker_w, *chunker_b, *bottleneck;
  float *a_hat, *x_top, *kc, *vc;
  const int32_t* seq_len;
  int64_t S_max;
  int Bt, n_layers, D, F, H, CL, pitch;
  float eps, theta, scale_log2e;
};

template <int KS>
__global__ __launch_bounds__(SM_THREADS) void small_step_kernel(const SmallStepArgs p) {
  extern __shared__ __align__(16) float lds[];
  const int D = p.D, F = p.F, H = p.H, d_h = D / H, half = d_h / 2, KC = p.CL * D;
  // beyond the common areas: scores of every head, weighted values of every wave, the chunker's input row
  const int S = (int)p.S_max, o_part = (H * S + 3) / 4 * 4, o_in = o_part + SM_WAVES * p.pitch;
  const SmallLds s = small_lds(1, D, F, p.n_layers, 0, half, o_in + pad256(KC));
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int seq = blockIdx.x;
  float *h = lds + s.h, *xn = lds + s.xn, *qkv = lds + s.qkv, *attn = lds + s.attn, *gains = lds + s.gains;
  float *score = lds + s.extra, *part = score + o_part, *in = score + o_in;

  Batch a, b;
  const Matrix chunker{p.chunker_w, D, KC, false};
  auto wqkv = [&](int layer) { return Matrix{p.mod.layer[layer].wqkv, 3 * D, D, false}; };
  request<0>(chunker, 0, 0, b);
  for (int i = tid; i < s.total; i += SM_THREADS) lds[i] = 0.f;
  lds_barrier();
  load_gains(p.mod, p.n_layers, D, s.DP, gains);
  for (int k = tid; k < KC; k += SM_THREADS) in[k] = p.bottleneck[(int64_t)seq * KC + k];
  const int32_t count = p.seq_len[seq];
  const int pos = count - 1;                             // of the new unit; outside the cache: not written
  const int n = count < 0 ? 0 : count > S ? S : count;
  for (int i = tid; i < half; i += SM_THREADS) {
    float c, sn;
    rope_angle(pos, i, d_h, p.theta, c, sn);
    lds[s.rot + i] = c;
    lds[s.rot + half + i] = sn;
  }
  lds_barrier();
  contract_rows<0, 1>(chunker, in, pad256(KC), 1, b, [&] { request<KS>(wqkv(0), 0, 0, a); }, [&](int d, int, float y, float) {
    const float v = y + (p.chunker_b != nullptr ? p.chunker_b[d] : 0.f);
    p.a_hat[(int64_t)seq * D + d] = v;
    h[d] = v;
    xn[d] = v * gains[d];
  });
  lds_barrier();

  const int LPR = p.pitch / 4, rpw = 64 / LPR, row = lane / LPR, col = lane % LPR * 4;   // lanes of a cache row, rows of a wave
  // waves of a head; with more heads than waves a wave takes several
  const int per_head = H < SM_WAVES ? SM_WAVES / H : 1, head0 = wave / per_head, sub = wave - head0 * per_head;
  const int stride = per_head * rpw;
  for (int i = 0; i < p.n_layers; ++i) {
    const float rs = row_scale(h, D, p.eps);
    contract_rows<KS, 1>(wqkv(i), xn, s.DP, 1, a, [&] { request<KS>(Matrix{p.mod.layer[i].wo, D, D, false}, 0, 0, b); },
                         [&](int c, int, float y, float) { qkv[c] = y * rs; });
    lds_barrier();
    const int64_t stream = ((int64_t)i * p.Bt + seq) * H;
    for (int e = tid; e < H * half; e += SM_THREADS) {
      const int hd = e / half, d = e - hd * half, lo = hd * d_h + d, hi = lo + half;
      const float c = lds[s.rot + d], sn = lds[s.rot + half + d];
      const float q0 = qkv[lo], q1 = qkv[hi], k0 = qkv[D + lo], k1 = qkv[D + hi];
      qkv[lo] = fmaf(q0, c, -(q1 * sn));
      qkv[hi] = fmaf(q0, sn, q1 * c);
      if (pos < 0 || pos >= S) continue;
      float *k = p.kc + ((stream + hd) * p.S_max + pos) * p.pitch, *v = p.vc + ((stream + hd) * p.S_max + pos) * p.pitch;
      k[d] = fmaf(k0, c, -(k1 * sn));
      k[d + half] = fmaf(k0, sn, k1 * c);
      v[d] = qkv[2 * D + lo];
      v[d + half] = qkv[2 * D + hi];
      for (int t = d_h + d; t < p.pitch; t += half) k[t] = v[t] = 0.f;
    }
    __syncthreads();                                     // the new entry is read back from the cache below, by this workgroup alone
    const int head_step = H < SM_WAVES ? H : SM_WAVES;   // a wave whose first head lies past the last has nothing to do
    for (int hd = head0; hd < H; hd += head_step) {
      const float* kc = p.kc + (stream + hd) * p.S_max * p.pitch;
      float4_t q = float4_t{0.f, 0.f, 0.f, 0.f};
      if (col < d_h) q = float4_t{qkv[hd * d_h + col], qkv[hd * d_h + col + 1], qkv[hd * d_h + col + 2], qkv[hd * d_h + col + 3]};
      for (int t0 = sub * rpw; t0 < n; t0 += 4 * stride) {
        float4_t k[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int t = t0 + u * stride + row;
          k[u] = t < n ? *reinterpret_cast<const float4_t*>(kc + (int64_t)t * p.pitch + col) : float4_t{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int t = t0 + u * stride + row;
          float v = fmaf(q.x, k[u].x, fmaf(q.y, k[u].y, fmaf(q.z, k[u].z, q.w * k[u].w)));
          v = LPR == 8 ? group_sum<8>(v) : LPR == 16 ? group_sum<16>(v) : group_sum<32>(v);
          if (t < n && col == 0) score[hd * S + t] = v * p.scale_log2e;
        }
      }
    }
    lds_barrier();
    for (int hd = head0; hd < H; hd += head_step) {
      const float* vc = p.vc + (stream + hd) * p.S_max * p.pitch;
      float mx = NEG_BIG, l = 0.f;                       // (every wave of the head forms them for itself)
      for (int t = lane; t < n; t += 64) mx = fmaxf(mx, score[hd * S + t]);
#pragma unroll
      for (int mask = 1; mask < 64; mask <<= 1) mx = fmaxf(mx, __shfl_xor(mx, mask));
      for (int t = lane; t < n; t += 64) l += fast_exp2(score[hd * S + t] - mx);
      l = wave_sum(l);
      float4_t o = float4_t{0.f, 0.f, 0.f, 0.f};
      for (int t0 = sub * rpw; t0 < n; t0 += 4 * stride) {
        float4_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int t = t0 + u * stride + row;
          v[u] = t < n ? *reinterpret_cast<const float4_t*>(vc + (int64_t)t * p.pitch + col) : float4_t{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int t = t0 + u * stride + row;
          if (t < n) o += fast_exp2(score[hd * S + t] - mx) * v[u];
        }
      }
      for (int mask = LPR; mask < 64; mask <<= 1)
#pragma unroll
        for (int u = 0; u < 4; ++u) o[u] += __shfl_xor(o[u], mask);
      const float inv = l > 0.f ? 1.f / l : 0.f;
      if (per_head == 1) {
        if (lane < LPR && col < d_h)
          for (int u = 0; u < 4; ++u) attn[hd * d_h + col + u] = o[u] * inv;
      } else if (lane < LPR) {
        *reinterpret_cast<float4_t*>(part + wave * p.pitch + col) = o * inv;
      }
    }
    lds_barrier();
    if (per_head > 1) {
      for (int d = tid; d < D; d += SM_THREADS) {
        const int hd = d / d_h;
        float v = 0.f;
        for (int w = 0; w < per_head; ++w) v += part[(hd * per_head + w) * p.pitch + d - hd * d_h];
        attn[d] = v;
      }
      lds_barrier();
    }
    const bool last = i + 1 == p.n_layers;
    small_block_tail<KS, 1>(p.mod.layer[i], lds, s, D, F, 1, p.eps, gains + (2 * i + 1) * s.DP, gains + (last ? 2 * p.n_layers : 2 * (i + 1)) * s.DP,
                            a, b, [&] { request<KS>(wqkv(last ? 0 : i + 1), 0, 0, a); });
  }
  const float rf = row_scale(h, D, p.eps);
  for (int d = tid; d < D; d += SM_THREADS) p.x_top[(int64_t)seq * D + d] = h[d] * rf * gains[2 * p.n_layers * s.DP + d];
}

bool fill_module(const photon_module_weights& m, int n_layers, SmallModule* out) {
  if (n_layers > SM_MAX_LAYERS) return false;
  *out = SmallModule{};
  for (int i = 0; i < n_layers; ++i) {
    const photon_layer_weights& w = m.layers[i];
    out->layer[i] = SmallLayer{w.g1, (const float*)w.wqkv, (const float*)w.wo, w.g2, (const float*)w.wgu, (const float*)w.wd};
  }
  out->g_final = m.g_final;
  return true;
}

bool small_shape(int n_layers, int D, int H, int64_t workgroups) {
  return n_layers <= SM_MAX_LAYERS && D <= SM_MAX_D && D % 4 == 0 && D / H % 4 == 0 && workgroups <= 256;
}

// Batches that a workgroup takes in one after the other: of rows padded to whole k steps (ks of 64), and of rows of any length.
int row_batches(int N, int ks, bool pair = false) {
  const int passes = (N + SM_GROUPS - 1) / SM_GROUPS * (pair ? 2 : 1), per = SM_AHEAD / ks;
  return (passes + per - 1) / per;
}
int long_batches(int N, int K) { return row_batches(N, 4) * ((K + 255) / 256); }

// Time of the one launch and of the launches it replaces, in us.  Fitted to steps of 838 models replayed from a graph, with either
// part in either form (widths 8 - 128, 1 - 8 blocks, 100 - 32000 columns, 1 - 256 chunks, caches of 32 - 2048 entries; 9.6 % rms): what
// a workgroup takes is its batches (64 KB each, padding included, at 75 bytes per ns), barriers and heads in turn; a separate launch
// takes 2.4 us and more with every doubling of its rows.  A level is one launch where that is faster by a twentieth, STEP where it is
// slower by a tenth at most: enqueued call by call, separate launches take an eighth more.  Of the 838 steps four are then slower than
// separate launches (by 2 to 10 %), and the geometric mean is 0.5 % above the best choice for every model.  (By true bytes and 4 us a
// launch 51 were slower: four blocks 32 wide, 8 items, 32000 columns, one sequence 1299 us instead of 558; one block 72 wide, 4000 columns,
// 512 entries 78 instead of 44.)  Whole steps, one launch / separate, enqueued: D = 64, one block, 1 and 8 sequences 100 / 232 and 101 / 442 us;
// D = 128, two blocks, 8 sequences 266 / 802.  Rows beyond 128 wide have 1.7 MB a block and more, which the launches deal over the chip.
struct SmallTimes { double one, separate; };

double layer_megabytes(int D, int F) { return 4e-6 * (4.0 * D * D + 3.0 * D * F); }
int layer_batches(int D, int F) {
  const int ks = D <= 64 ? 1 : 2;
  return row_batches(3 * D, ks) + row_batches(D, ks) + (F > 0 ? row_batches(F, ks, true) + long_batches(D, F) : 0);
}
int head_rounds(int H) { return (H + SM_WAVES - 1) / SM_WAVES; }

SmallTimes level_times(const SmallLevel& a) {
  const int ks = a.D <= 64 ? 1 : 2, vocab = a.E != nullptr ? a.vocab : 0;
  const double rows = (double)a.n_chunks, phases = a.C * ((a.F > 0 ? 5 : 3) * a.n_layers + (vocab > 0 ? 2 : 1));
  const double batches = a.C * (a.n_layers * layer_batches(a.D, a.F) + row_batches(vocab, ks)) + row_batches(a.R * a.D, ks);
  const double head_mb = 4e-6 * vocab * a.D;
  return {2.5 + 0.16 * phases + 0.84 * batches + 1.34 * a.n_layers * head_rounds(a.H) * (a.C + a.R - 1),
          phases * (2.4 + 1.17 * log2(rows)) +
              a.C * (0.043 * rows * (a.n_layers * layer_megabytes(a.D, a.F) + head_mb) + 0.35 * head_mb + 38e-6 * rows * vocab)};
}

SmallTimes step_times(const SmallStep& a) {
  const int pitch = kv_row_elems(a.D / a.H), per_head = a.H < SM_WAVES ? SM_WAVES / a.H : 1, entries = 4 * per_head * (256 / pitch);
  const int block = a.F > 0 ? 5 : 3;
  const double rows = (double)a.Bt, launches = (block + 1) * a.n_layers + 2;
  const double kv_rounds = (double)head_rounds(a.H) * (double)((a.S_max + entries - 1) / entries);
  const double score_rounds = (double)head_rounds(a.H) * (double)((a.S_max + 63) / 64);
  return {6.3 + 0.65 * ((block + 2) * a.n_layers + 2) + 0.55 * (a.n_layers * layer_batches(a.D, a.F) + long_batches(a.D, a.CL * a.D)) +
              a.n_layers * (1.66 * kv_rounds + 0.12 * score_rounds),
          launches * (2.2 + 0.96 * log2(rows)) + a.n_layers * (0.061 * rows * layer_megabytes(a.D, a.F) + 0.29 * (double)a.S_max / 64 +
                                                               0.12 * rows * 8e-6 * (double)a.S_max * a.H * pitch)};
}

size_t level_lds(const SmallLevel& a) {
  return sizeof(float) * small_lds(a.R <= 1 ? 1 : 2, a.D, a.F, a.n_layers, a.R + a.C - 1, (a.R + a.C - 1) * (a.D / a.H / 2), 0).total;
}
size_t step_lds(const SmallStep& a) {
  const int64_t extra = ((int64_t)a.H * a.S_max + 3) / 4 * 4 + SM_WAVES * kv_row_elems(a.D / a.H) + pad256(a.CL * a.D);
  if (extra > (int64_t)(SM_LDS_LIMIT / sizeof(float))) return SM_LDS_LIMIT + 1;
  return sizeof(float) * small_lds(1, a.D, a.F, a.n_layers, 0, a.D / a.H / 2, (int)extra).total;
}

}  // namespace

bool small_level_pays(const SmallLevel& a) {
  if (!small_shape(a.n_layers, a.D, a.H, a.n_chunks) || a.R > 2) return false;
  if ((int64_t)a.vocab * a.D > ((int64_t)1 << 27)) return false;   // a matrix view takes offsets below 1 GiB
  const SmallTimes t = level_times(a);
  return level_lds(a) <= SM_LDS_LIMIT && 1.05 * t.one < t.separate;
}

int32_t launch_small_level(const SmallLevel& a, hipStream_t st) {
  SmallLevelArgs p{};
  if (!small_level_pays(a) || !fill_module(*a.mod, a.n_layers, &p.mod)) return fail(PHOTON_ERR_UNSUPPORTED, "small decode level: sizes out of range");
  p.conv_w = (const float*)a.conv_w; p.conv_b = a.conv_b; p.W_lm = (const float*)a.W_lm; p.E = (const float*)a.E; p.cond = a.cond;
  p.units = a.units; p.logits = a.logits; p.forced = a.forced; p.tokens = a.tokens; p.ld_logits = a.ld_logits; p.ld_item = a.ld_item;
  p.n_layers = a.n_layers; p.D = a.D; p.F = a.F; p.H = a.H; p.C = a.C; p.R = a.R; p.vocab = a.vocab; p.eps = a.eps;
  const int d_h = a.D / a.H;
  p.scale_log2e = LOG2E / sqrtf((float)d_h);
  p.freq_ratio = a.theta == 0.f ? 0.0 : pow((double)a.theta, -2.0 / (double)d_h);
  const size_t lds = level_lds(a);
#define PHOTON_SMALL(KS, MR) PHOTON_LAUNCH(KC_SMALL, st, (small_level_kernel<KS, MR>), dim3((unsigned)a.n_chunks), dim3(SM_THREADS), lds, st, p)
  if (a.D <= 64) { if (a.R == 1) PHOTON_SMALL(1, 1); else PHOTON_SMALL(1, 2); }
  else { if (a.R == 1) PHOTON_SMALL(2, 1); else PHOTON_SMALL(2, 2); }
#undef PHOTON_SMALL
  return check_launch("small_level_kernel");
}

bool small_step_pays(const SmallStep& a) {
  // Longer caches are beyond the times' fit, and a workgroup walks alone what the separate kernel deals over the chip: of 100 models with
  // full caches of 2049 - 16384 entries that the times had in one launch, 37 were slower so by a twentieth and more (2049 - 4096 entries:
  // geometric mean 1.05, 14 of 54; 4097 - 8192: 0.96, 17 of 38; above: 0.82, 6 of 8; worst 528 us instead of 361), of 60 up to 2048 one (1.44).
  if (!small_shape(a.n_layers, a.D, a.H, a.Bt) || a.S_max > SM_MAX_CACHE) return false;
  const SmallTimes t = step_times(a);
  return step_lds(a) <= SM_LDS_LIMIT && 0.9 * t.one < t.separate;
}

int32_t launch_small_step(const SmallStep& a, hipStream_t st) {
  SmallStepArgs p{};
  if (!small_step_pays(a) || !fill_module(*a.mod, a.n_layers, &p.mod)) return fail(PHOTON_ERR_UNSUPPORTED, "small STEP: sizes out of range");
  p.chunker_w = (const float*)a.chunker_w; p.chunker_b = a.chunker_b; p.bottleneck = a.bottleneck; p.a_hat = a.a_hat; p.x_top = a.x_top;
  p.kc = a.k_cache; p.vc = a.v_cache; p.seq_len = a.seq_len; p.S_max = a.S_max; p.Bt = a.Bt; p.n_layers = a.n_layers;
  p.D = a.D; p.F = a.F; p.H = a.H; p.CL = a.CL; p.pitch = kv_row_elems(a.D / a.H); p.eps = a.eps; p.theta = a.theta;
  p.scale_log2e = LOG2E / sqrtf((float)(a.D / a.H));
  if (a.D <= 64) PHOTON_LAUNCH(KC_SMALL, st, small_step_kernel<1>, dim3((unsigned)a.Bt), dim3(SM_THREADS), step_lds(a), st, p);
  else PHOTON_LAUNCH(KC_SMALL, st, small_step_kernel<2>, dim3((unsigned)a.Bt), dim3(SM_THREADS), step_lds(a), st, p);
  return check_launch("small_step_kernel");
}

}  // namespace photon
