// Dense bf16 contractions on the matrix cores: out[M,N] = x[M,K] * W[N,K]^T (+ bias, + residual).
//   * the context-chunker projection (paper Eq. 4) at many-row shapes: bf16 in, bf16 out;
//   * the block projections of the prefill, and of a decode step once a level carries many rows (large
//     batches, deep hierarchies): a row kernel normalises the fp32 activations and rounds them to bf16, the
//     matrix cores' operand type (the few-row kernels keep a bf16 remainder as well; at many rows that second
//     pass over the matrix cores costs a fifth of the prefill and of a large-batch step, for accuracy far
//     beyond what bf16 matrices and a bf16 cache leave).
//
// K is walked in slabs of 64: rows of x and W move global -> LDS directly (no staging registers), several slabs ahead
// of the one that the matrix cores contract, and MFMA 16x16x32 tiles accumulate in registers.  Two kernels: one group of
// waves with three or more slab buffers (tiles of 32 x 32 to 128 x 160), and two groups in counter-phase (128 x 256 and
// 256 x 256).  A contraction of fewer than 128 rows is too small to fill the chip and is split over K as well: the fp32
// partial products go to a scratch area and are added, in a fixed order, by the kernel that reads the result anyway (the row
// kernel in front of the next contraction, the attention kernels).  The gate/up projection forms SwiGLU in the accumulators.
#include <type_traits>

#include "photon_device.h"
#include "photon_host.h"
#include "photon_linear.h"

namespace photon {

constexpr int G_BK = 64;                                         // K must be a multiple of this
// Order of a sum over K.  From ORDERED_ROWS rows on the products are added up along K.  Below, in the order of the few-row
// kernels: K in chunks of 128, chunk c in class c % 8, each class added up along K, then the classes' sums in order.  A row's
// result then depends neither on the other rows of the pass nor on the tile and the split that plan_gemm finds fastest.
constexpr int ORDERED_ROWS = 128, K_CLASSES = 8, CHUNK_SLABS = 2;

// 16 bytes per lane from global memory straight into LDS: lane l lands at lds_base + 16 l (lds_base: byte offset in
// LDS, wave-uniform).  Written as an instruction rather than through the compiler's builtin: the compiler treats
// the builtin as an access to both memories that may complete out of order, and while one is in flight it makes
// every wait for an LDS read a wait for ALL LDS reads, which serialises the operand prefetch below.  Completion is
// tracked by hand (s_waitcnt vmcnt) at the one place per slab where it matters.
// m0 (the LDS base of the load) is named as clobbered so that the compiler keeps no value of its own in it across the
// statement; it notes that m0 is a reserved register, which is the point here.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load16_to_lds(const void* gsrc, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(gsrc), "s"(lds_base) : "memory", "m0");
}
__device__ __forceinline__ void load4_to_lds(const void* gsrc, uint32_t lds_base) {   // 4 bytes per lane
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(gsrc), "s"(lds_base) : "memory", "m0");
}
#pragma clang diagnostic pop

typedef __attribute__((address_space(3))) void* lptr_t;

enum GemmOut { GEMM_OUT_BF16 = 0, GEMM_OUT_F32 = 1, GEMM_OUT_SWIGLU = 2, GEMM_OUT_QKV = 3, GEMM_OUT_LOGITS = 4 };

// ---- shared by the tile kernels ------------------------------------------------------------------------------------------

// One contraction as the kernels take it: out[m, n] (bf16, fp32 or the SwiGLU product as bf16) = x[m, :] . W[n, :]
// (+ bias[n] + res[m, n]).  fp32 output in classes may be split over K: split s contracts classes s * split_classes ..
// + split_classes; the first writes their sum, the others each class's sum, to the partial products out + part *
// part_stride (no bias or residual then).  group_m: row tiles that are walked together.
struct GemmArgs {
  const bf16_t* x; const bf16_t* W; const float* bias; const float* res; void* out;
  int64_t ldres, ldo, part_stride;
  int M, N, K, tiles_m, tiles_n, group_m, split_classes, tiles;  // tiles: of all splits
  bool cold;                                                     // W comes from HBM: see ContractArgs
  RowBest* best; int stretches;                                  // GEMM_OUT_LOGITS (fp32 output): see ContractArgs
  QkvOperands qkv;                                               // GEMM_OUT_QKV: where the columns go instead of `out`
};

// Workgroups that share W rows on an XCD, from which on touching their lines pays.  Geometric means over 11 projections, weights in the
// memory-side cache / in HBM, by 64 x 32, 64 x 64 and 128 x 64: of 2 row tiles 1.01 / 1.07, 0.90 / 0.99 and 0.98 / 1.05 times as fast as without, of
// 3 1.01 / 1.12, 0.96 / 1.08 and 0.99 / 1.13, of 4 and more 1.02 / 1.10, 0.96 / 1.08 and 1.00 / 1.10.
constexpr int TOUCH_SHARERS = 3;
// Slabs whose lines are requested ahead of the barrier at hand: 8, 16, 32 and all 1.08, 1.09, 1.09 and 1.10 times as fast from HBM, 0.96, 0.96, 0.95 and
// 0.95 from the memory-side cache (64 x 64 tiles); by 128 x 64 1.10 each, and 1.00, 0.99, 0.99 and 0.99.
constexpr int TOUCH_AHEAD = 8;

// Workgroup ids are dealt round-robin to the 8 XCDs.  Each XCD takes a contiguous run of tiles (also when the count is
// not a multiple of 8), walked as bands of group_m row tiles, row tiles fastest: the 32 tiles resident on an XCD form a
// patch of about group_m x 32 / group_m whose x rows and W rows that XCD's L2 holds once.
struct TilePos { int tm, tn, split; };
__device__ __forceinline__ TilePos tile_position(const GemmArgs& p, int id, int total) {
  const int xcd = id & 7, base = total >> 3, rem = total & 7;
  const int logical = xcd * base + (xcd < rem ? xcd : rem) + (id >> 3);
  const int per_split = p.tiles_m * p.tiles_n;
  const int split = logical / per_split, t = logical - split * per_split;
  const int band = p.group_m * p.tiles_n;
  const int b = t / band, in_band = t - b * band;
  const int gm = min(p.group_m, p.tiles_m - b * p.group_m);
  return TilePos{b * p.group_m + in_band % gm, in_band / gm, split};
}

// 16-byte column c of staged row r (128 bytes per row) lies at column c ^ ((r >> 1) & 7): the 16 rows that a
// quarter-wave reads together fall on distinct 16-byte slots of the 256-byte bank line.
__device__ __forceinline__ int swizzled_column(int r, int c) { return c ^ ((r >> 1) & 7); }
__device__ __forceinline__ bf16x8_t fragment(const char* slab, int r, int c16) {
  return as_bf16x8(*reinterpret_cast<const uint4_t*>(slab + r * 128 + (swizzled_column(r, c16) << 4)));
}

// Row of W behind staged W row r of a tile whose output columns start at n0 (clamped into the matrix).  SwiGLU: 16 gate
// rows, then the 16 up rows of the same columns, so that both products of a column meet in one lane; IN8 (a wave holds an odd
// number of MFMA tiles): 8 gate rows, then the 8 up rows of the same columns, which meet in lanes l and l + 32.
template <bool GU, bool IN8 = false> __device__ __forceinline__ int weight_row(int r, int n0, int N) {
  if (!GU) return n0 + r < N ? n0 + r : N - 1;
  const int c = IN8 ? n0 + (r >> 4) * 8 + (r & 7) : n0 + (r >> 5) * 16 + (r & 15);
  return (c < N ? c : N - 1) + ((r >> (IN8 ? 3 : 4)) & 1) * N;
}

template <int VM> __device__ __forceinline__ void wait_loads_and_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(VM) : "memory");
}

// One row of a wave's accumulators: the MFMAs take W as their row operand, so a lane holds 4 consecutive columns of
// output row m: acc[j] is columns wave_col + j * 16 + 4 fk .. +3 of the tile's staged W rows.
template <int OUT, int TJ>
__device__ __forceinline__ void store_row(const GemmArgs& p, const float4_t (&acc)[TJ], int m, int n0, int wave_col, int fk, int part) {
  if (m >= p.M) return;
  if constexpr (OUT == GEMM_OUT_SWIGLU) {
    static_assert(TJ % 2 == 0, "gate and up tiles in turn");
#pragma unroll
    for (int j = 0; j < TJ; j += 2) {
      const int n = n0 + (wave_col + j * 16) / 2 + fk * 4;
      if (n >= p.N) continue;
      const float4_t g = acc[j], u = acc[j + 1];
      *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(p.out) + (int64_t)m * p.ldo + n) =
          uint2{pack_bf16x2(silu(g.x) * u.x, silu(g.y) * u.y), pack_bf16x2(silu(g.z) * u.z, silu(g.w) * u.w)};
    }
  } else {
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      const int n = n0 + wave_col + j * 16 + fk * 4;
      if (n >= p.N) continue;                                    // N is a multiple of 16
      float4_t y = acc[j];
      if (p.bias != nullptr) y += float4_t{p.bias[n], p.bias[n + 1], p.bias[n + 2], p.bias[n + 3]};
      if constexpr (OUT == GEMM_OUT_F32 || OUT == GEMM_OUT_LOGITS) {
        if (p.res != nullptr) y += *reinterpret_cast<const float4_t*>(p.res + (int64_t)m * p.ldres + n);
        *reinterpret_cast<float4_t*>(reinterpret_cast<float*>(p.out) + part * p.part_stride + (int64_t)m * p.ldo + n) = y;
      } else {
        *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(p.out) + (int64_t)m * p.ldo + n) = uint2{pack_bf16x2(y.x, y.y), pack_bf16x2(y.z, y.w)};
      }
    }
  }
}

// SwiGLU of two MFMA rows m and m + 16 in the IN8 order: the halves of the wave trade accumulators, after which the lower lanes
// hold gate and up of row m, the upper lanes of row m + 16.
template <int TJ>
__device__ __forceinline__ void store_swiglu_rows(const GemmArgs& p, const float4_t (&lo)[TJ], const float4_t (&hi)[TJ], int m, int n0, int wave_col, int fk) {
  typedef uint32_t uint2_native __attribute__((ext_vector_type(2)));
  const int row = m + (fk >> 1) * 16;
#pragma unroll
  for (int j = 0; j < TJ; ++j) {
    float4_t g, u;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint2_native r = __builtin_amdgcn_permlane32_swap(__float_as_uint(lo[j][t]), __float_as_uint(hi[j][t]), false, false);
      g[t] = __uint_as_float(r[0]); u[t] = __uint_as_float(r[1]);
    }
    const int n = n0 + (wave_col + j * 16) / 2 + (fk & 1) * 4;
    if (row < p.M && n < p.N)
      *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(p.out) + (int64_t)row * p.ldo + n) =
          uint2{pack_bf16x2(silu(g.x) * u.x, silu(g.y) * u.y), pack_bf16x2(silu(g.z) * u.z, silu(g.w) * u.w)};
  }
}

// Best column of a wave's 16 * TJ columns of row m, for the token choice: the choice then reads a pair per stretch instead
// of all logits (1024 rows of 32000: 32 -> 7 us).  The four lanes that share a row are 16 and 32 apart.
template <int TJ>
__device__ __forceinline__ void store_best(const GemmArgs& p, const float4_t (&acc)[TJ], int m, int col0, int fk) {
  if (m >= p.M || col0 >= p.N) return;
  float best = -INFINITY;
  int column = 0x7fffffff;
#pragma unroll
  for (int j = 0; j < TJ; ++j) {
    const int n = col0 + j * 16 + fk * 4;
    if (n >= p.N) continue;
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (acc[j][t] > best || column == 0x7fffffff) { best = acc[j][t]; column = n + t; }
  }
#pragma unroll
  for (int mask = 16; mask < 64; mask <<= 1) {
    const float v = __shfl_xor(best, mask);
    const int c = __shfl_xor(column, mask);
    if (v > best || (v == best && c < column)) { best = v; column = c; }
  }
  if (fk == 0) p.best[(int64_t)m * p.stretches + col0 / (16 * TJ)] = RowBest{best, column};
}

// Four consecutive cache entries.
__device__ __forceinline__ void store_cache4(void* cache, int64_t at, const float4_t& y, bool fp8) {
  if (fp8) *reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(cache) + at) = pack_fp8x2(y.x, y.y) | (pack_fp8x2(y.z, y.w) << 16);
  else *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(cache) + at) = uint2{pack_bf16x2(y.x, y.y), pack_bf16x2(y.z, y.w)};
}

// One row of a wave's 64 columns of a QKV projection, which are one head of q, k or v: q and k are rotated (element i and
// i + 32 sit in accumulators j and j + 2 of the same lane), q scaled, everything rounded to fp16 and stored as the attention
// kernel reads it; k and v also go to the cache.  Called by whole groups of four lanes (rows m .. m + 3) when positions come
// in fours: they then exchange their v values and each stores four positions of one element instead of four single values.
// 32768 x 3072 x 1024: 225 us, against 218 us for the fp32 projection and 135 us for the pass over it that this replaces.
template <int TJ>
__device__ __forceinline__ void store_qkv(const GemmArgs& p, const float4_t (&acc)[TJ], int m, int col0, int fk) {
  static_assert(TJ == 4, "a wave holds one head");
  if (m >= p.M || col0 >= p.N) return;
  const QkvOperands& o = p.qkv;
  const int D = o.H * 64, section = col0 / D, h = (col0 - section * D) >> 6;
  const int b = (int)((unsigned)m / (unsigned)o.M), pos = m - b * o.M;
  const int64_t bh = (int64_t)b * o.H + h;
  const bool cached = o.kc != nullptr && pos < o.S_max;
  const int64_t slot = (bh * o.S_max + pos) * 64;
  if (section < 2) {
    uint16_t* dst = (section == 0 ? o.qh : o.kh) + (bh * o.Mp + pos) * 64;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int i = j * 16 + fk * 4;
      const float4_t c = *reinterpret_cast<const float4_t*>(o.table + (int64_t)pos * 64 + i);
      const float4_t s = *reinterpret_cast<const float4_t*>(o.table + (int64_t)pos * 64 + 32 + i);
      float4_t y0, y1;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        float lower, upper;
        rotate_pair(acc[j][t], acc[j + 2][t], c[t], s[t], lower, upper);
        y0[t] = lower; y1[t] = upper;
      }
      if (section == 0) {
        y0 *= o.qscale; y1 *= o.qscale;
      } else if (cached) {
        store_cache4(o.kc, slot + i, y0, o.cache_fp8);
        store_cache4(o.kc, slot + 32 + i, y1, o.cache_fp8);
      }
      *reinterpret_cast<uint2*>(dst + i) = uint2{pack_f16x2(y0.x, y0.y), pack_f16x2(y0.z, y0.w)};
      *reinterpret_cast<uint2*>(dst + 32 + i) = uint2{pack_f16x2(y1.x, y1.y), pack_f16x2(y1.z, y1.w)};
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int d = j * 16 + fk * 4;
    if (cached) store_cache4(o.vc, slot + d, acc[j], o.cache_fp8);
    const uint32_t lo = pack_f16x2(acc[j].x, acc[j].y), hi = pack_f16x2(acc[j].z, acc[j].w);
    uint16_t* dst = o.vt + (bh * 64 + d) * o.Mp;
    if (o.M % 4 == 0) {
      // a 4 x 4 transpose over the lanes q = 0..3 of the group: lane q ends up with element d + q of positions pos - q .. +3
      const int q = threadIdx.x & 3;
      const uint32_t lo1 = __builtin_amdgcn_update_dpp(0, lo, DPP_XOR1, 0xf, 0xf, false), hi1 = __builtin_amdgcn_update_dpp(0, hi, DPP_XOR1, 0xf, 0xf, false);
      const uint32_t a = (q & 1) ? (lo1 >> 16) | (lo & 0xffff0000u) : (lo & 0xffffu) | (lo1 << 16);
      const uint32_t c = (q & 1) ? (hi1 >> 16) | (hi & 0xffff0000u) : (hi & 0xffffu) | (hi1 << 16);
      const uint32_t a2 = __builtin_amdgcn_update_dpp(0, a, DPP_XOR2, 0xf, 0xf, false), c2 = __builtin_amdgcn_update_dpp(0, c, DPP_XOR2, 0xf, 0xf, false);
      *reinterpret_cast<uint2*>(dst + (int64_t)q * o.Mp + pos - q) = (q & 2) ? uint2{c2, c} : uint2{a, a2};
    } else {
      dst[pos] = (uint16_t)lo; dst[o.Mp + pos] = (uint16_t)(lo >> 16);
      dst[2 * (int64_t)o.Mp + pos] = (uint16_t)hi; dst[3 * (int64_t)o.Mp + pos] = (uint16_t)(hi >> 16);
    }
  }
}

// ---- small and middle contractions: one group of waves, NB slab buffers ------------------------------------------------
//
// WM x WN waves share a BM x BN tile.  A compute unit is fed at 40 to 100 bytes per ns here, depending on how many
// workgroups share it, so what a small contraction costs is the bytes its busiest unit has to take in (its x rows and
// its W rows, 128 bytes per row and slab) plus about 2.5 us of launch, first slab and stores: the tile and the split
// over K are chosen together so that every unit has work (plan_gemm).
// Measured against the kernels it replaces (MI355X): 64 rows, 2048 x 5120: 28 -> 8.7 us (8 splits); 64 rows, 6144 x 2048:
// 16.4 -> 11.6 us; 64 rows, SwiGLU 2 x 2560 x 1024: 12.3 -> 8.7 us; 512 rows, 2048 x 5120: 32 -> 28 us.
// Sums along K: within a slab the operand reads of one half go out among the MFMAs of the other half, one read at a time: reads issued together
// in front of the MFMAs keep the matrix cores waiting, as all waves leave the barrier together.  The one barrier per slab lies
// between the halves: everybody then holds the rest of slab kt in registers, slab kt + 1 has landed, and the buffer takes slab
// kt + NB.  Against reads, then MFMAs behind the barrier (512 rows, weights in the memory-side cache / in HBM): 64 x 64 tiles
// 2048 x 2048 10.7 / 11.8 -> 9.4 / 11.6 us, 2048 x 5120 22.2 / 26.7 -> 19.0 / 25.8 us; 128 x 160, 10240 x 2048 29.2 / 33.7 -> 27.4 / 31.9 us.
// Small wave tiles help for the same reason: 32 x 32 by four waves.
// TOUCH: one more wave, which requests four bytes of every line of W some slabs ahead of the others: its workgroup's share of what the
// workgroups with the same columns read together on an XCD.  A unit holds about 64 KB of requests in flight and returns them in order, so
// x rows that lie in L2 wait behind W lines that come from HBM, and every sharer waits for itself; a line that is touched once is in L2
// when they ask.  Weights in the memory-side cache / in HBM, without and with it: 256 rows, 1664 x 4096 by 64 x 32 12.5 / 17.4 and 12.5 / 14.3 us,
// 1664 x 1664 6.9 / 8.9 and 6.7 / 7.8; 512 rows, 2048 x 5120 by 64 x 64 19.4 / 26.8 and 21.0 / 22.4; 1024 rows, 1664 x 4096 by 128 x 64 24.6 / 30.9 and
// 25.4 / 25.8.  (A wave that met no barrier held the others at their first one until it had touched all its lines: from HBM 14.9, 8.3, 24.9 and
// 27.3 us.)  128 x 96 and 128 x 160 gain less and stay without it (34 and 32 projections: 0.99 / 1.04 and 0.99 / 1.03).
// The launch bounds name two waves per SIMD also where four make a workgroup: with all 512 registers to deal the compiler keeps
// accumulators in the accumulation registers and moves them about in every slab, behind the MFMAs (64 x 32 tiles of the chunker: 64 rows,
// 8192 x 2048 24.7 us instead of 19.5; 512 rows, 2048 x 512 8.2 instead of 6.7; tiles of eight waves are the same).
// CLASSES: the sum in classes (see ORDERED_ROWS).  A second set of accumulators takes the classes' sums; the slabs are loaded
// in the classes' order, which costs a few scalar instructions per slab.
template <int BM, int BN, int WM, int WN, int NB, int OUT, bool CLASSES, bool TOUCH = false>
__global__ __launch_bounds__((WM * WN + TOUCH) * 64, 2) void gemm_tile_kernel(const GemmArgs p) {
  constexpr bool GU = (OUT == GEMM_OUT_SWIGLU);
  constexpr int WAVES = WM * WN, STAGE = (BM + BN) * 128;
  constexpr int PIECES = (BM + BN) / 8, LPS = (PIECES + WAVES - 1) / WAVES;   // load instructions of a slab, and per wave
  constexpr int TI = BM / WM / 16, TJ = BN / WN / 16;            // MFMA tiles of a wave
  constexpr bool IN8 = GU && TJ % 2 != 0;
  // 128 x 64 and 128 x 128 tiles gain little by the reads ahead (1024 rows, 1664 x 4096 by 128 x 64 27.5 / 26.7 us; 2048 rows, 1664 x 1664 by
  // 128 x 128 19.9 / 19.7), and the one slab more that is requested past the end costs where K is short (1200 rows, 768 x 1600 by
  // 128 x 64 8.1 / 8.3 us; a prefill at the width 384 3280 / 3319 us).
  constexpr bool READS_AHEAD = !CLASSES && !(BM == 128 && (BN == 64 || BN == 128));
  static_assert(!IN8 || TI % 2 == 0, "a wave trades rows in pairs");
  static_assert(BM % 8 == 0 && NB >= 2, "");
  extern __shared__ __align__(16) char lds[];                    // [NB buffers][BM x rows | BN W rows], TOUCH: 256 bytes nobody reads
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const TilePos at = tile_position(p, blockIdx.x, gridDim.x);
  const int m0 = at.tm * BM, n0 = at.tn * (GU ? BN / 2 : BN);
  if constexpr (TOUCH) {
    static_assert(!GU && !CLASSES, "plain columns, summed along K");
    if (wave == WAVES) {                                         // (a wave that has ended takes no part in the barriers)
      const int band = at.tm / p.group_m, sharers = min(p.group_m, p.tiles_m - band * p.group_m);
      const int share = (BN + sharers - 1) / sharers, first = n0 + (at.tm - band * p.group_m) * share, lines = sharers < TOUCH_SHARERS ? 0 : share * (p.K / G_BK);
      const uint32_t sink = (uint32_t)(uintptr_t)(lptr_t)lds + NB * STAGE;
      // The workgroup's barriers wait for this wave too: it meets each of them.
      int l0 = 0;
      for (int met = 0; met < p.K / G_BK + (READS_AHEAD ? 1 : 0); ++met) {
        for (const int until = min(lines, (met + TOUCH_AHEAD) * share); l0 < until; l0 += 64) {
          const int l = l0 + lane < lines ? l0 + lane : lines - 1, r = first + l % share;
          load4_to_lds(reinterpret_cast<const char*>(p.W + (int64_t)(r < p.N ? r : p.N - 1) * p.K) + (l / share) * (G_BK * 2), sink);
        }
        asm volatile("s_barrier" ::: "memory");
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      return;
    }
  }
  const int KT = p.K / G_BK, chunks = (KT + CHUNK_SLABS - 1) / CHUNK_SLABS;
  const int classes = chunks < K_CLASSES ? chunks : K_CLASSES;
  const int class0 = CLASSES ? at.split * p.split_classes : 0;
  const int class1 = CLASSES ? min(class0 + p.split_classes, classes) : 1;

  // Piece of load instruction i: 8 rows.  Where the pieces do not divide, surplus instructions repeat the last piece (the same
  // bytes to the same place), so that every wave has the same number of loads in flight.
  auto piece = [&](int i) { const int q = i * WAVES + wave; return PIECES % WAVES == 0 || q < PIECES ? q : PIECES - 1; };
  const char* src[LPS];
#pragma unroll
  for (int i = 0; i < LPS; ++i) {
    const int r = piece(i) * 8 + (lane >> 3);
    const bf16_t* row;
    if (piece(i) * 8 < BM) row = p.x + (int64_t)(m0 + r < p.M ? m0 + r : p.M - 1) * p.K;   // past the end: never stored
    else row = p.W + (int64_t)weight_row<GU, IN8>(r - BM, n0, p.N) * p.K;
    src[i] = reinterpret_cast<const char*>(row + swizzled_column(r, lane & 7) * 8);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)lds;
  // Slab that is loaded next, and its class.  Past the end: the last slab again, into a buffer nobody reads (every wait then names a
  // constant; waits chosen by what is left, without those loads: 64 rows, SwiGLU 2 x 2560 x 1024 8.4 -> 9.5 us).
  int ahead = CLASSES ? class0 * CHUNK_SLABS : 0, ahead_class = class0;
  auto load = [&](int buf) {
    const int64_t ko = (int64_t)ahead * (G_BK * 2);
#pragma unroll
    for (int i = 0; i < LPS; ++i) load16_to_lds(src[i] + ko, lds0 + buf * STAGE + piece(i) * 1024);
    if constexpr (!CLASSES) {
      if (ahead + 1 < KT) ++ahead;
    } else {
      const int next_chunk = ahead / CHUNK_SLABS + K_CLASSES;
      if (ahead % CHUNK_SLABS + 1 < CHUNK_SLABS && ahead + 1 < KT) ++ahead;
      else if (next_chunk < chunks) ahead = next_chunk * CHUNK_SLABS;
      else if (ahead_class + 1 < class1) ahead = ++ahead_class * CHUNK_SLABS;
    }
  };
  // slabs of class c: whole chunks, but for the last one of K
  auto class_slabs = [&](int c) {
    if (!CLASSES) return KT;
    const int n = (chunks - c + K_CLASSES - 1) / K_CLASSES;
    return n * CHUNK_SLABS - ((chunks - 1) % K_CLASSES == c ? chunks * CHUNK_SLABS - KT : 0);
  };
  float4_t acc[TI][TJ], sum[CLASSES ? TI : 1][CLASSES ? TJ : 1];
  const int wm = (wave / WN) * (BM / WM), wn = (wave % WN) * (BN / WN);
  const int fr = lane & 15, fk = lane >> 4;                      // operand fragment: row, 8-wide k group
  auto store = [&](const float4_t (&y)[TI][TJ], int part) {
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      if constexpr (IN8) {
        if (i % 2 == 0) store_swiglu_rows<TJ>(p, y[i], y[i + 1], m0 + wm + i * 16 + fr, n0, wn, fk);
      } else if constexpr (OUT == GEMM_OUT_QKV) {
        store_qkv<TJ>(p, y[i], m0 + wm + i * 16 + fr, n0 + wn, fk);
      } else {
        store_row<OUT, TJ>(p, y[i], m0 + wm + i * 16 + fr, n0, wn, fk, part);
      }
      if constexpr (OUT == GEMM_OUT_LOGITS) store_best<TJ>(p, y[i], m0 + wm + i * 16 + fr, n0 + wn, fk);
    }
  };

  bf16x8_t xf[2][TI], wf[2][TJ];                                 // [half of the slab]
  auto read_one = [&](int buf, int ks, int t) {
    const char* s = lds + buf * STAGE;
    if (t < TJ) wf[ks][t] = fragment(s, BM + wn + t * 16 + fr, ks * 4 + fk);
    else xf[ks][t - TJ] = fragment(s, wm + (t - TJ) * 16 + fr, ks * 4 + fk);
    __builtin_amdgcn_sched_barrier(0);
  };
  // MFMAs of half 1 - KS of the slab at hand; under the first three quarters of them the operands of half KS of buffer `buf` (in front
  // of them where there are one or two: a read between them would come late; 6 rows, 3072 x 1664 9.0 / 10.7 us)
  auto half = [&](int buf, auto KS) {
    constexpr int ks = decltype(KS)::value, READS = TI + TJ, MFMAS = TI * TJ, SPAN = MFMAS <= 2 ? 1 : (MFMAS * 3 + 3) / 4;
#pragma unroll
    for (int q = 0; q < MFMAS; ++q) {
#pragma unroll
      for (int t = 0; t < READS; ++t)
        if (t * SPAN / READS == q) read_one(buf, ks, t);
      const int i = q % TI, j = q / TI;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[1 - ks][j], xf[1 - ks][i], acc[i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto clear = [&] {
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j) acc[i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
  };
  int buf = 0;
  if constexpr (READS_AHEAD) {
#pragma unroll
    for (int s = 0; s < NB; ++s) load(s);
    clear();
    wait_loads_and_barrier<(NB - 1) * LPS>();                    // the first slab
#pragma unroll
    for (int t = 0; t < TI + TJ; ++t) read_one(0, 0, t);
    for (int kt = 0; kt < KT; ++kt) {
      half(buf, std::integral_constant<int, 1>{});
      wait_loads_and_barrier<(NB - 2) * LPS>();
      load(buf);
      buf = buf + 1 < NB ? buf + 1 : 0;
      half(buf, std::integral_constant<int, 0>{});               // (behind the last slab: not used)
    }
  } else {
    // Classes: a class is two slabs where K is 1024: with its sum to be closed every other slab, reads ahead only get in the way (64 rows, K = 1024:
    // SwiGLU 2 x 2560 8.0 us, with reads ahead 9.5; 3072 columns 6.8 and 7.3).
#pragma unroll
    for (int s = 0; s < NB - 1; ++s) load(s);
    int next = NB - 1;
    for (int c = class0; c < class1; ++c) {
      clear();
      for (int left = class_slabs(c); left > 0; --left) {
        wait_loads_and_barrier<(NB - 2) * LPS>();                // (behind a class's stores, which count as well, longer than it has to be)
        load(next);
        const char* s = lds + buf * STAGE;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
          for (int i = 0; i < TI; ++i) xf[ks][i] = fragment(s, wm + i * 16 + fr, ks * 4 + fk);
#pragma unroll
          for (int j = 0; j < TJ; ++j) wf[ks][j] = fragment(s, BM + wn + j * 16 + fr, ks * 4 + fk);
#pragma unroll
          for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[ks][j], xf[ks][i], acc[i][j], 0, 0, 0);
        }
        buf = buf + 1 < NB ? buf + 1 : 0;
        next = next + 1 < NB ? next + 1 : 0;
      }
      if constexpr (CLASSES) {
        if (class0 == 0) {
#pragma unroll
          for (int i = 0; i < TI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) sum[i][j] = c == 0 ? acc[i][j] : sum[i][j] + acc[i][j];
        } else if (OUT == GEMM_OUT_F32 && c + 1 < class1) {
          store(acc, c + 1 - p.split_classes);
        }
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");               // the surplus loads of the tail land before the workgroup ends
  if constexpr (CLASSES) {
    if (class0 == 0) store(sum, 0);
    else store(acc, class1 - p.split_classes);
  } else {
    store(acc, 0);
  }
}

// ---- large contractions: two groups of waves in counter-phase, 256 x 256 (TI = 4) or 128 x 256 (TI = 2) tile ------------
//
// What bounds a large contraction here is how much of the time the matrix cores have an instruction to run: with one
// group of waves that reads operands, meets at a barrier and multiplies, the cores idle through every read phase (58 %
// busy at 32768 x 2048 x 16384 on all-zero operands, where the clock does not drop).  So 8 waves work as two groups of
// four, one wave of each group on every SIMD, half a phase apart: while one group issues a half-slab of MFMAs the
// other fetches its next operands from LDS, and every phase ends at a barrier.  Per 64-wide K slab and wave:
//   read 0: W fragments (64 columns) and x fragments of the wave's upper 64 rows    | barrier
//   mma  0: 32 MFMAs 16x16x32                                                       | barrier
//   read 1: x fragments of the lower 64 rows (the W fragments stay in registers)    | barrier
//   mma  1: 32 MFMAs                                                                | barrier
// The rows a slab buffer holds are ordered by when they are last read: [W rows | upper x rows of both groups] (part X,
// 48 KB) is free after read 0, [lower x rows] (part Y) after read 1, so the direct global -> LDS loads of slab kt + 2
// go out part by part, X in read 1 and Y in the next read 0, with four phases (about 1 us) to land before the wait for
// them; two 64 KB buffers suffice.  Every wait names the number of younger loads (XI + YI, a constant).
// MFMA 16x16x32 rather than 32x32x16: at the same schedule 10-15 % faster on real data, where power limits the clock.
// Measured (MI355X, data spread like N(0,1)): 32768 x 2048 x 16384, timed in turn with the single group of waves on two cards,
// 1975 -> 1538 and 2007 -> 1597 us (1.43 and 1.38 PFLOP/s); 8192 x 2048 x 5120
// 122 us (1.41 PFLOP/s) where a 16-wave kernel without the counter-phase takes 134 us.
constexpr int PP_BN = 256, PP_THREADS = 512;

// WALK: a workgroup walks several tiles (launch_gemm says when), its loads running over the end of one into the next; else
// one tile, whose slab addresses need no state of their own.
template <int TI, int OUT, bool WALK = false>
__global__ __launch_bounds__(PP_THREADS) void gemm_pingpong_kernel(const GemmArgs p) {
  constexpr bool GU = (OUT == GEMM_OUT_SWIGLU);
  constexpr int TJ = 4;                                          // MFMA tiles of a wave's half: TI x 16 rows, 64 columns
  constexpr int PP_BM = 64 * TI, HALF = 16 * TI;                 // rows of the tile, rows of a wave's half
  constexpr int PP_STAGE = (PP_BM + PP_BN) * 128;                // one slab
  constexpr int PP_XI = (PP_BN + PP_BM / 2) / 64;                // load instructions per wave and slab, part X
  constexpr int PP_YI = PP_BM / 2 / 64;                          // part Y
  extern __shared__ __align__(16) char lds[];                    // [2 buffers][256 W rows | upper x rows | lower x rows]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = wave >> 2, wcol = wave & 3;                  // group 0: upper half of the tile's rows, group 1: lower half
  const int fr = lane & 15, fk = lane >> 4;                      // operand fragment: row, 8-wide k group
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)lds;

  // one load instruction moves 64 lanes x 16 B = 8 staged rows; instruction i of wave w covers rows (i * 8 + w) * 8 .. +8
  auto source = [&](const TilePos& at, int i) {
    const int r = (i * 8 + wave) * 8 + (lane >> 3);
    const bf16_t* row;
    if ((i * 8 + wave) * 8 < PP_BN) {
      row = p.W + (int64_t)weight_row<GU>(r, at.tn * (GU ? PP_BN / 2 : PP_BN), p.N) * p.K;
    } else {
      const int a = r - PP_BN, half = a / (2 * HALF), w = a % (2 * HALF);   // staged x row -> row of the tile
      const int m = at.tm * PP_BM + (w / HALF) * (2 * HALF) + half * HALF + w % HALF;
      row = p.x + (int64_t)(m < p.M ? m : p.M - 1) * p.K;        // rows past the end repeat the last one: never stored
    }
    return reinterpret_cast<const char*>(row + swizzled_column(r, lane & 7) * 8);
  };
  const int KT = p.K / G_BK;
  // Loads run ahead of the slab that is contracted; each part has a place of its own in the sequence of all slabs.  After the
  // last tile the last slab is loaded again, into rows nobody reads any more (the number of loads in flight stays constant).
  struct Ahead { int id, left, slab; };                          // tile, slabs left in it, count of all slabs so far
  Ahead ax{(int)blockIdx.x, 0, 0}, ay = ax;
  const char* src[PP_XI + PP_YI];
  auto enter = [&](Ahead& a, auto first, auto last) {
    const TilePos to = tile_position(p, a.id, p.tiles);
    a.left = KT;
#pragma unroll
    for (int i = decltype(first)::value; i < decltype(last)::value; ++i) src[i] = source(to, i);
  };
  auto load = [&](Ahead& a, auto first, auto last) {
    const uint32_t to = lds0 + (a.slab & 1) * PP_STAGE;
    const int64_t ko = WALK ? 0 : (int64_t)(a.slab < a.left ? a.slab : a.left - 1) * (G_BK * 2);
    ++a.slab;
#pragma unroll
    for (int i = decltype(first)::value; i < decltype(last)::value; ++i) load16_to_lds(src[i] + ko, to + (i * 8 + wave) * 1024);
    if constexpr (WALK) {
      if (--a.left > 0) {
#pragma unroll
        for (int i = decltype(first)::value; i < decltype(last)::value; ++i) src[i] += G_BK * 2;
      } else if (a.left == 0 && a.id + (int)gridDim.x < p.tiles) {
        a.id += gridDim.x;
        enter(a, first, last);
      }
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using IX = std::integral_constant<int, PP_XI>;
  using IE = std::integral_constant<int, PP_XI + PP_YI>;

  float4_t acc[2][TI][TJ];
  bf16x8_t xf[2][TI], wf[2][TJ];
  auto read_w = [&](int slab) {
    const char* s = lds + (slab & 1) * PP_STAGE;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int j = 0; j < TJ; ++j) wf[ks][j] = fragment(s, wcol * 64 + j * 16 + fr, ks * 4 + fk);
  };
  auto read_x = [&](int slab, int half) {
    const char* s = lds + (slab & 1) * PP_STAGE;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < TI; ++i) xf[ks][i] = fragment(s, PP_BN + (half * 2 + group) * HALF + i * 16 + fr, ks * 4 + fk);
  };
  auto mma = [&](int half) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
          acc[half][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[ks][j], xf[ks][i], acc[half][i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // End of a read phase: own fragments in registers (part of the buffer may be overwritten from here on), own share of
  // what the next read phase needs landed; after the barrier both hold for every wave.  (Behind a tile's stores, which
  // count as well, the wait is longer than it has to be, never shorter.)
  auto read_done = [&] {
    __builtin_amdgcn_sched_barrier(0);
    wait_loads_and_barrier<PP_XI + PP_YI>();
  };

  enter(ax, I0{}, IX{});
  enter(ay, IX{}, IE{});
  load(ax, I0{}, IX{});
  load(ay, IX{}, IE{});
  load(ax, I0{}, IX{});
  wait_loads_and_barrier<PP_XI + PP_YI>();                       // part X of slab 0
  if (group == 1) asm volatile("s_barrier" ::: "memory");        // half a phase behind group 0 from here on
  int slab = 0, id = blockIdx.x;
  do {
    const TilePos at = tile_position(p, id, p.tiles);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) acc[h][i][j] = float4_t{0.f, 0.f, 0.f, 0.f};
    for (int kt = 0; kt < KT; ++kt, ++slab) {
      read_w(slab);
      read_x(slab, 0);
      load(ay, IX{}, IE{});                                      // part Y of the other buffer: last read one slab ago
      read_done();
      mma(0);
      read_x(slab, 1);
      load(ax, I0{}, IX{});                                      // part X of this buffer: both groups are past read 0
      read_done();
      mma(1);
    }
    if constexpr (!WALK) {
      if (group == 0) asm volatile("s_barrier" ::: "memory");
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // the surplus loads of the tail land before the workgroup ends
    }
    const int m0 = at.tm * PP_BM, n0 = at.tn * (GU ? PP_BN / 2 : PP_BN);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < TI; ++i) {
        const int m = m0 + (group * 2 + h) * HALF + i * 16 + fr;
        if constexpr (OUT == GEMM_OUT_QKV) store_qkv<TJ>(p, acc[h][i], m, n0 + wcol * 64, fk);
        else store_row<OUT, TJ>(p, acc[h][i], m, n0, wcol * 64, fk, 0);
        if constexpr (OUT == GEMM_OUT_LOGITS) store_best<TJ>(p, acc[h][i], m, n0 + wcol * 64, fk);
      }
  } while (WALK && (id += gridDim.x) < p.tiles);
  if constexpr (WALK) {
    if (group == 0) asm volatile("s_barrier" ::: "memory");
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
}

// ---- row kernel between contractions --------------------------------------------------------------------------------------
//
// Per row: add up what the value consists of (the partial products of a split contraction, bias, residual row, in this
// order, as a contraction in one piece does), write the sum if asked, normalise (RMS with gain) and write it as bf16 (the
// next contraction's operand, rounded to nearest even) or fp32.  TPR threads hold a row in registers, NV float4 each (one
// read of the row; loads of all sources in flight together); NV == 0: rows longer than the registers hold, read again for
// the second pass.  The squares are added up as by 256 threads at every TPR, so that a row's result does not depend on how
// many rows there are.
template <int TPR, int NV>
__global__ __launch_bounds__(256) void rows_kernel(const RowsArgs p) {
  const int row = blockIdx.x * (256 / TPR) + threadIdx.x / TPR, t = threadIdx.x % TPR;
  if (row >= p.M) return;                                        // TPR == 256: never; TPR == 64: whole waves, which share nothing
  const int K = p.K;
  const float* x = p.in.x != nullptr ? p.in.x + (int64_t)row * p.in.ld : nullptr;
  const float* parts = p.in.parts + (int64_t)row * p.in.part_ld;
  auto value = [&](int k) {
    float4_t v = float4_t{0.f, 0.f, 0.f, 0.f};
    for (int s = 0; s < p.in.n_parts; ++s) v += *reinterpret_cast<const float4_t*>(parts + s * p.in.part_stride + k);
    if (p.bias != nullptr) v += float4_t{p.bias[k], p.bias[k + 1], p.bias[k + 2], p.bias[k + 3]};
    if (x != nullptr) v += *reinterpret_cast<const float4_t*>(x + k);
    return v;
  };
  // with fp32 rows asked for as well, the bf16 rows are those rounded
  auto emit = [&](int k, const float4_t& v, const float4_t& g, float r) {
    float4_t w = p.gain != nullptr ? v * g * r : v;
    if (p.y != nullptr) {
      w = v * r * g;
      *reinterpret_cast<float4_t*>(p.y + (int64_t)row * p.ldy + k) = w;
    }
    if (p.xb != nullptr)
      *reinterpret_cast<uint2*>(p.xb + (int64_t)row * K + k) = uint2{pack_bf16x2(w.x, w.y), pack_bf16x2(w.z, w.w)};
  };
  auto inv_rms = [&](const float (&of)[4]) {
    float ss;
    if constexpr (TPR == 64) {
      ss = (wave_sum(of[0]) + wave_sum(of[1])) + (wave_sum(of[2]) + wave_sum(of[3]));
    } else {
      ss = wave_sum(of[0]);
      __shared__ float partsum[4];
      if ((threadIdx.x & 63) == 0) partsum[threadIdx.x >> 6] = ss;
      __syncthreads();
      ss = (partsum[0] + partsum[1]) + (partsum[2] + partsum[3]);
    }
    return 1.0f / sqrtf(ss / (float)K + p.eps);
  };
  float ss[4] = {0.f, 0.f, 0.f, 0.f}, r = 1.f;                   // TPR == 64: of the four waves that 256 threads would be
  if constexpr (NV > 0) {
    float4_t v[NV], g[NV], whole[NV];
    // the gain is requested with the rows, not after the reduction
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int k = (i * TPR + t) * 4;
      g[i] = p.gain != nullptr && k < K ? *reinterpret_cast<const float4_t*>(p.gain + k) : float4_t{1.f, 1.f, 1.f, 1.f};
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int k = (i * TPR + t) * 4;
      whole[i] = k < K && x != nullptr ? *reinterpret_cast<const float4_t*>(x + k) : float4_t{0.f, 0.f, 0.f, 0.f};
      v[i] = float4_t{0.f, 0.f, 0.f, 0.f};
    }
    // several partial products in flight: taken in one after the other, each costs a trip to memory
    constexpr int PB = NV <= 2 ? K_CLASSES : NV <= 4 ? 4 : 2;
    for (int s0 = 0; s0 < p.in.n_parts; s0 += PB) {
      float4_t w[PB][NV];
#pragma unroll
      for (int u = 0; u < PB; ++u) {
#pragma unroll
        for (int i = 0; i < NV; ++i) w[u][i] = float4_t{0.f, 0.f, 0.f, 0.f};
        if (s0 + u >= p.in.n_parts) continue;
        const float* ps = parts + (s0 + u) * p.in.part_stride;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
          const int k = (i * TPR + t) * 4;
          if (k < K) w[u][i] = *reinterpret_cast<const float4_t*>(ps + k);
        }
      }
#pragma unroll
      for (int u = 0; u < PB; ++u) {
        if (s0 + u >= p.in.n_parts) continue;
#pragma unroll
        for (int i = 0; i < NV; ++i) v[i] += w[u][i];
      }
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int k = (i * TPR + t) * 4;
      if (k >= K) continue;
      if (p.bias != nullptr) v[i] += float4_t{p.bias[k], p.bias[k + 1], p.bias[k + 2], p.bias[k + 3]};
      v[i] += whole[i];
      if (p.sum != nullptr) *reinterpret_cast<float4_t*>(p.sum + (int64_t)row * p.ld_sum + k) = v[i];
      float& to = ss[TPR == 64 ? i & 3 : 0];
      to = fmaf(v[i].x, v[i].x, fmaf(v[i].y, v[i].y, fmaf(v[i].z, v[i].z, fmaf(v[i].w, v[i].w, to))));
    }
    if (p.gain != nullptr) r = inv_rms(ss);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int k = (i * TPR + t) * 4;
      if (k < K) emit(k, v[i], g[i], r);
    }
  } else {
    if (p.gain != nullptr) {
      for (int k = t * 4; k < K; k += TPR * 4) {
        const float4_t v = value(k);
        ss[0] = fmaf(v.x, v.x, fmaf(v.y, v.y, fmaf(v.z, v.z, fmaf(v.w, v.w, ss[0]))));
      }
      r = inv_rms(ss);
    }
    for (int k = t * 4; k < K; k += TPR * 4) {
      const float4_t v = value(k);
      if (p.sum != nullptr) *reinterpret_cast<float4_t*>(p.sum + (int64_t)row * p.ld_sum + k) = v;
      emit(k, v, p.gain != nullptr ? *reinterpret_cast<const float4_t*>(p.gain + k) : float4_t{1.f, 1.f, 1.f, 1.f}, r);
    }
  }
}

int32_t launch_rows(const RowsArgs& p, hipStream_t st) {
  if (p.M <= 0) return PHOTON_OK;
  if (p.K % 4 != 0 || p.in.ld % 4 != 0 || p.in.part_ld % 4 != 0 || p.in.part_stride % 4 != 0 || p.ld_sum % 4 != 0 || p.ldy % 4 != 0 ||
      (p.y != nullptr && p.gain == nullptr))
    return fail(PHOTON_ERR_UNSUPPORTED, "row kernel: K=%d and the row pitches must be multiples of 4, fp32 rows come normalised", p.K);
#define PHOTON_ROWS(TPR, NV) PHOTON_LAUNCH(KC_NORM, st, (rows_kernel<TPR, NV>), dim3((unsigned)((p.M + 256 / TPR - 1) / (256 / TPR))), dim3(256), 0, st, p)
  // Few rows: a whole workgroup per row, for the latency of one row.  From 4096 rows on (16 workgroups per compute unit
  // in flight either way) a wave per row, which saves the barrier.
  if (p.M >= 4096 && p.K <= 2048) {
    if (p.K <= 1024) PHOTON_ROWS(64, 4); else PHOTON_ROWS(64, 8);
  } else if (p.K <= 1024) PHOTON_ROWS(256, 1);
  else if (p.K <= 2048) PHOTON_ROWS(256, 2);
  else if (p.K <= 4096) PHOTON_ROWS(256, 4);
  else if (p.K <= 8192) PHOTON_ROWS(256, 8);
  else PHOTON_ROWS(256, 0);
#undef PHOTON_ROWS
  return check_launch("rows_kernel");
}

__global__ __launch_bounds__(256) void copy_bytes16_kernel(const uint4_t* __restrict__ src, uint4_t* __restrict__ dst, int64_t n16) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx < n16) dst[idx] = src[idx];
}

// ---- which tile, how many splits ------------------------------------------------------------------------------------------

enum TileKind { T_64x32 = 0, T_64x64, T_128x64, T_128x128, T_CLASS_KINDS, T_128x256 = T_CLASS_KINDS, T_256x256, T_32x32, T_128x96, T_128x160, T_KINDS };
struct TileShape { int bm, bn, wave_columns; };
constexpr TileShape TILES[T_KINDS] = {{64, 32, 32}, {64, 64, 32}, {128, 64, 32}, {128, 128, 64}, {128, 256, 64}, {256, 256, 64}, {32, 32, 16}, {128, 96, 48}, {128, 160, 80}};
// Time model behind the choice, in us: fixed + slabs per split * (slab1 if every compute unit has one workgroup at most,
// slabn * workgroups per unit otherwise) + `round` for every workgroup of a unit behind its first + what the output bytes cost.  It
// ranks the choices rather than predicting a time; 256 x 256 with its long first slab and store pays off once the other tiles need
// several rounds.
// PASS: fp32 and SwiGLU results summed along K, workgroups per unit counted as ROUNDED of the whole number that its busiest unit has and
// the rest of the mean.  Fitted to a sweep of all tiles over 1000 projections of 128 - 4096 rows, widths 64 to 5120, weights half of
// the time in the memory-side cache and half in HBM (6-8 % rms, 256 x 256 11): its choice is within 1.3 % of the best tile (geometric mean), and
// 7 % faster than the tiles and kernels before the present ones.  Of 1200 times of 600 other projections 32 are more than 3 % longer than
// with those, most of them of launches of 3 - 5 us.  (Fitted over the widths 448 to 2048 only, with neither `round` nor means: 59, 576 columns
// of 2679 rows at K = 192 5.8 us instead of 4.8, 9216 columns of 2025 rows at K = 3072 from HBM 145 instead of 126.)
// CLASSED: sums in classes, the chunker's own entry point and passes of more than PASS_ROWS rows (where the fit above does not reach:
// a prefill of 24 x 5696 tokens at the width 384 3482 us with these, 3526 with those) and more than PASS_SLABS slabs of K (up to three, by PASS
// instead: 47 projections of 4097 - 32768 rows 1.10 times as fast), over 128 - 2048 rows at the widths 1024, 1664 and 2048 (5-11 % rms).
struct TileTime { float fixed, slab1, slabn, round = 0.f; };
constexpr int PASS_ROWS = 4096, PASS_SLABS = 3;
constexpr TileTime CLASSED[] = {{1.6f, 0.21f, 0.17f}, {2.3f, 0.24f, 0.22f}, {2.8f, 0.34f, 0.34f}, {3.5f, 0.50f, 0.59f}, {6.2f, 0.74f, 0.94f}, {8.6f, 1.00f, 1.36f}};
constexpr TileTime PASS[T_KINDS] = {{2.9f, 0.150f, 0.143f, 0.3f}, {3.2f, 0.192f, 0.201f, 0.5f},  {3.4f, 0.312f, 0.311f, 0.4f},
                                    {4.2f, 0.462f, 0.513f, 1.3f}, {6.4f, 0.784f, 0.859f, 2.0f},  {10.1f, 1.033f, 1.272f, 2.5f},
                                    {2.7f, 0.132f, 0.096f, 0.1f}, {4.2f, 0.407f, 0.438f, 1.7f},  {5.2f, 0.553f, 0.612f, 2.3f}};
constexpr float ROUNDED = 0.7f;
constexpr float US_PER_MB_OUT = 0.18f, US_PER_MB_PARTS = 0.17f;      // writing the output; reading partial products back

// parts: partial products (1: none); split_classes: classes of K per split (0: the sum runs along K, unsplit)
struct GemmPlan { int kind, splits, parts, split_classes; };

enum PlanOutput { PLAN_F32, PLAN_SWIGLU, PLAN_LOGITS, PLAN_CHUNKER, PLAN_QKV };
// Which tiles an output takes.  A wave of the 32 x 32 tile holds 16 columns: half a gate/up pair, less than a stretch of logits.
// (By 32 x 32, 64 - 512 columns: 505 shapes of 128 - 4096 rows, medians 5.2 -> 4.2 us at K = 1024, 11.3 -> 8.7 at K = 4096.)
// 128 x 96 and 128 x 160 fill the units where the other tiles leave a part of them idle or need a second
// round: 512 rows, SwiGLU 2 x 5120 x 2048, 160 tiles of 128 x 256 32.8 us, 256 tiles of 128 x 160 25.7 us.
static bool tile_takes(int kind, PlanOutput output, bool classes, bool pass) {
  if (classes) return kind < T_CLASS_KINDS;
  if (output == PLAN_QKV) return kind == T_128x128 || kind == T_128x256 || kind == T_256x256;   // a wave holds a head
  if (!pass) return kind <= T_256x256;
  return kind != T_32x32 || output == PLAN_F32;
}

// classes: the sum is formed in classes of K (then not by the counter-phase kernels), and may be split between them.
// part_cap: floats the scratch area for partial products holds (0: no splitting).  join_us: what reading the partial
// products back costs beyond the bytes (a launch of its own, or nothing where the next kernel reads the result anyway).
static GemmPlan plan_gemm(int64_t M, int N, int K, PlanOutput output, bool classes, int64_t part_cap, float join_us, float* model_us = nullptr) {
  const bool gate_up = output == PLAN_SWIGLU, out_f32 = output == PLAN_F32 || output == PLAN_LOGITS;
  const int KT = K / G_BK, chunks = (KT + CHUNK_SLABS - 1) / CHUNK_SLABS, n_classes = chunks < K_CLASSES ? chunks : K_CLASSES;
  const bool pass = !classes && output != PLAN_CHUNKER && (M <= PASS_ROWS || KT <= PASS_SLABS);
  GemmPlan best{T_64x64, 1, 1, classes ? K_CLASSES : 0};
  float best_us = 1e30f;
  const float out_mb = (float)M * N * (out_f32 ? 4e-6f : 2e-6f);
  for (int k = 0; k < T_KINDS; ++k) {
    if (!tile_takes(k, output, classes, pass)) continue;
    const TileTime& cost = pass ? PASS[k] : CLASSED[k];
    const int bn = gate_up ? TILES[k].bn / 2 : TILES[k].bn;
    const int64_t tiles = (M + TILES[k].bm - 1) / TILES[k].bm * ((N + bn - 1) / bn);
    for (int per = K_CLASSES; per >= 1; per /= 2) {               // classes per split: the first split's come in one part, every other class is one
      const int splits = (n_classes + per - 1) / per, parts = splits > 1 ? 1 + n_classes - per : 1;
      if (per < K_CLASSES && (splits == 1 || !classes)) continue;
      if (parts > 1 && parts * M * N > part_cap) break;
      const int slabs = splits == 1 ? KT : per * ((chunks + K_CLASSES - 1) / K_CLASSES) * CHUNK_SLABS;
      float rounds = (float)((tiles * splits + 255) / 256);
      if (pass && rounds > 1.f) rounds = ROUNDED * rounds + (1.f - ROUNDED) / 256.f * (float)tiles;
      const float us = cost.fixed + cost.round * (rounds - 1.f) + slabs * (rounds <= 1.f ? cost.slab1 : cost.slabn * rounds) +
                       out_mb * parts * US_PER_MB_OUT + (parts > 1 ? out_mb * parts * US_PER_MB_PARTS + join_us : 0.f);
      if (us < best_us) { best_us = us; best = GemmPlan{k, splits, parts, classes ? per : 0}; }
      if (tiles * splits >= 512) break;                           // more splits only add bytes
    }
  }
  if (model_us != nullptr) *model_us = best_us;
  return best;
}

static int32_t launch_kernel(void (*kern)(GemmArgs), bool* attr_set, unsigned grid, int threads, size_t lds_bytes, const GemmArgs& p, hipStream_t st) {
  if (!*attr_set) {                                              // more than 64 KiB of dynamic LDS has to be allowed once
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (e != hipSuccess) return fail(PHOTON_ERR_HIP, "gemm: cannot reserve %zu bytes of LDS: %s", lds_bytes, hipGetErrorString(e));
    *attr_set = true;
  }
  PHOTON_LAUNCH(KC_CHUNKER_GEMM, st, kern, dim3(grid), dim3(threads), lds_bytes, st, p);
  return check_launch("gemm kernel");
}

// Gate/up over several rounds of short 256 x 256 tiles: one workgroup per compute unit walks its tiles and loads the next
// one's first slabs under the last one's contraction, SiLU and stores.  Measured in prefills, dealt out / walked: 16 x 8192
// tokens at K = 1024, four layers of two levels 1567 / 1469 us; 131072 tokens at K = 2048, eight layers of two levels
// 10.30 / 9.87 ms.  128 x 256 tiles gain nothing by it (eight layers, 627 to 710 tiles at K = 256 to 1536: 2097 / 2108,
// 2456 / 2438, 1349 / 1345, 1397 / 1399, 1624 / 1622 us).  The other outputs lose (their stores and residual loads queue with
// the next tile's loads: 1024 columns of 32768 rows 147 / 166 us, QKV 228 / 264 us), and so do two rounds or long tiles,
// which have little to hide.
static bool walks(const GemmPlan& plan, int64_t M, int N, int K) {
  const int bn = TILES[T_256x256].bn / 2;
  return plan.kind == T_256x256 && (M + 255) / 256 * ((N + bn - 1) / bn) > 2 * 256 && K <= 2048;
}

template <int OUT>
static int32_t launch_gemm(GemmArgs p, const GemmPlan& plan, hipStream_t st) {
  const TileShape& t = TILES[plan.kind];
  const int bn = OUT == GEMM_OUT_SWIGLU ? t.bn / 2 : t.bn;
  p.tiles_m = (p.M + t.bm - 1) / t.bm;
  p.tiles_n = (p.N + bn - 1) / bn;
  p.group_m = p.tiles_m < 8 ? p.tiles_m : 8;
  p.split_classes = plan.split_classes;
  const int64_t grid = (int64_t)p.tiles_m * p.tiles_n * plan.splits;
  if (grid > 0x7fffffffLL) return fail(PHOTON_ERR_UNSUPPORTED, "gemm: %lld workgroups are too many for one launch", (long long)grid);
  p.tiles = (int)grid;
#define PHOTON_GEMM_CASE(KIND, KERN, THREADS, BUFS)                                                            \
  case KIND: {                                                                                                 \
    static bool attr_set = false;                                                                              \
    return launch_kernel(KERN, &attr_set, (unsigned)grid, THREADS, (size_t)(BUFS) * (t.bm + t.bn) * 128, p, st); \
  }
#define PHOTON_GEMM_TOUCH(KIND, KERN, THREADS, BUFS)                                                           \
  case KIND: {                                                                                                 \
    static bool attr_set = false;                                                                              \
    return launch_kernel(KERN, &attr_set, (unsigned)grid, THREADS + 64, (size_t)(BUFS) * (t.bm + t.bn) * 128 + 256, p, st); \
  }
  if constexpr (OUT != GEMM_OUT_QKV) {                           // a wave of these tiles does not hold a head
    if constexpr (OUT != GEMM_OUT_BF16) {                        // (the chunker's sum always runs along K)
      if (plan.split_classes != 0) {
        switch (plan.kind) {
          PHOTON_GEMM_CASE(T_64x32, (gemm_tile_kernel<64, 32, 4, 1, 4, OUT, true>), 256, 4)
          PHOTON_GEMM_CASE(T_64x64, (gemm_tile_kernel<64, 64, 4, 2, 4, OUT, true>), 512, 4)
          PHOTON_GEMM_CASE(T_128x64, (gemm_tile_kernel<128, 64, 4, 2, 3, OUT, true>), 512, 3)
          default:
          PHOTON_GEMM_CASE(T_128x128, (gemm_tile_kernel<128, 128, 4, 2, 3, OUT, true>), 512, 3)
        }
      }
      switch (plan.kind) {
        PHOTON_GEMM_CASE(T_128x96, (gemm_tile_kernel<128, 96, 4, 2, 3, OUT, false>), 512, 3)
        PHOTON_GEMM_CASE(T_128x160, (gemm_tile_kernel<128, 160, 4, 2, 3, OUT, false>), 512, 3)
        default: break;
      }
    }
    if constexpr (OUT == GEMM_OUT_F32) {
      if (plan.kind == T_32x32) {
        static bool attr_set = false;
        return launch_kernel(gemm_tile_kernel<32, 32, 2, 2, 4, OUT, false>, &attr_set, (unsigned)grid, 256, (size_t)4 * 64 * 128, p, st);
      }
      // W lines touched ahead: tiles that share their columns with others, one round of them, and the wide ones only where W comes from
      // HBM.  354 projections of 192 - 4096 rows, widths 384 - 2048, by the tiles they take: up to 256 tiles 1.02 / 1.13, 0.97 / 1.08 and 1.00 / 1.09 times
      // as fast with it (memory-side cache / HBM; 64 x 32, 64 x 64 and 128 x 64); the 29 of more tiles, none of them 64 x 32, 0.93 to 1.00 and
      // 0.99 to 1.06 (0.96 to 1.18 one by one): too few that gain to tell which.
      if (p.tiles_m >= TOUCH_SHARERS && grid <= 256) {
        switch (plan.kind == T_64x32 || p.cold ? plan.kind : T_KINDS) {
          PHOTON_GEMM_TOUCH(T_64x32, (gemm_tile_kernel<64, 32, 4, 1, 4, OUT, false, true>), 256, 4)
          PHOTON_GEMM_TOUCH(T_64x64, (gemm_tile_kernel<64, 64, 4, 2, 4, OUT, false, true>), 512, 4)
          PHOTON_GEMM_TOUCH(T_128x64, (gemm_tile_kernel<128, 64, 4, 2, 3, OUT, false, true>), 512, 3)
          default: break;
        }
      }
    }
    // 64 x 32 tiles of the chunker, whose sums are long, with a compute unit each: six slabs in flight
    if constexpr (OUT == GEMM_OUT_BF16) {
      if (grid <= 256) {
        switch (plan.kind) {
          PHOTON_GEMM_CASE(T_64x32, (gemm_tile_kernel<64, 32, 4, 1, 6, OUT, false>), 256, 6)
          default: break;
        }
      }
    }
    switch (plan.kind) {
      PHOTON_GEMM_CASE(T_64x32, (gemm_tile_kernel<64, 32, 4, 1, 4, OUT, false>), 256, 4)
      PHOTON_GEMM_CASE(T_64x64, (gemm_tile_kernel<64, 64, 4, 2, 4, OUT, false>), 512, 4)
      PHOTON_GEMM_CASE(T_128x64, (gemm_tile_kernel<128, 64, 4, 2, 3, OUT, false>), 512, 3)
      default: break;
    }
  }
  if constexpr (OUT == GEMM_OUT_SWIGLU) {
    if (walks(plan, p.M, p.N, p.K)) {
      static bool attr_set = false;
      return launch_kernel(gemm_pingpong_kernel<4, OUT, true>, &attr_set, 256, PP_THREADS, (size_t)2 * (t.bm + t.bn) * 128, p, st);
    }
  }
  switch (plan.kind) {
    PHOTON_GEMM_CASE(T_128x128, (gemm_tile_kernel<128, 128, 4, 2, 3, OUT, false>), 512, 3)
    PHOTON_GEMM_CASE(T_128x256, (gemm_pingpong_kernel<2, OUT>), PP_THREADS, 2)
    default:
    PHOTON_GEMM_CASE(T_256x256, (gemm_pingpong_kernel<4, OUT>), PP_THREADS, 2)
  }
#undef PHOTON_GEMM_CASE
#undef PHOTON_GEMM_TOUCH
}

int64_t contract_part_floats(int64_t rows, int D) {
  // 8 parts of a D-wide result, 5 of a 3D-wide one, at up to 512 rows (more rows have enough tiles)
  return (rows < 512 ? rows : 512) * 15 * (int64_t)D;
}

int32_t launch_contract(const ContractArgs& a, RowSource* result, hipStream_t st, int* best_stretches) {
  if (a.K % G_BK != 0 || a.N % 16 != 0 || a.ldo % 4 != 0) return fail(PHOTON_ERR_UNSUPPORTED, "contraction: K=%d must be a multiple of 64, N=%d of 16", a.K, a.N);
  GemmArgs p{};
  p.x = reinterpret_cast<const bf16_t*>(a.x); p.W = reinterpret_cast<const bf16_t*>(a.W); p.M = a.M; p.N = a.N; p.K = a.K;
  p.bias = a.bias; p.out = a.out; p.ldo = a.ldo; p.cold = a.cold;
  const bool classes = (a.order_rows > 0 ? a.order_rows : a.M) < ORDERED_ROWS;
  if (a.epilogue == EPI_SWIGLU) return launch_gemm<GEMM_OUT_SWIGLU>(p, plan_gemm(a.M, a.N, a.K, PLAN_SWIGLU, classes, 0, 0.f), st);
  // a plain result that the caller needs in one piece is joined by a launch of the row kernel
  const bool join = a.epilogue == EPI_PLAIN && !a.split_ok;
  const GemmPlan plan = plan_gemm(a.M, a.N, a.K, a.best != nullptr ? PLAN_LOGITS : PLAN_F32, classes, a.part_cap, join ? 3.5f : 0.f);
  const RowSource whole{reinterpret_cast<const float*>(a.out), a.ldo, nullptr, 0, 0, 0};
  if (a.best != nullptr && plan.splits == 1) {
    if (a.epilogue != EPI_PLAIN || a.bias != nullptr || best_stretches == nullptr)
      return fail(PHOTON_ERR_INVALID_ARG, "contraction: the rows' best columns come with plain logits only");
    const int wave_columns = TILES[plan.kind].wave_columns;
    p.best = a.best; p.stretches = *best_stretches = (a.N + wave_columns - 1) / wave_columns;
    *result = whole;
    return launch_gemm<GEMM_OUT_LOGITS>(p, plan, st);
  }
  if (plan.splits == 1) {
    if (a.epilogue == EPI_RESID) {
      if (a.res.n_parts != 0) return fail(PHOTON_ERR_INVALID_ARG, "contraction: the residual rows must be in one piece");
      const char *r0 = reinterpret_cast<const char*>(a.res.x), *o0 = reinterpret_cast<const char*>(a.out);
      const char *r1 = r0 + ((int64_t)(a.M - 1) * a.res.ld + a.N) * 4, *o1 = o0 + ((int64_t)(a.M - 1) * a.ldo + a.N) * 4;
      if (r0 < o1 && o0 < r1) return fail(PHOTON_ERR_INVALID_ARG, "contraction: the residual rows must not overlap the output");
      p.res = a.res.x; p.ldres = a.res.ld;
    }
    *result = whole;
    return launch_gemm<GEMM_OUT_F32>(p, plan, st);
  }
  p.bias = nullptr; p.out = a.parts; p.ldo = a.N; p.part_stride = (int64_t)a.M * a.N;
  PHOTON_TRY(launch_gemm<GEMM_OUT_F32>(p, plan, st));
  RowSource r{nullptr, 0, a.parts, plan.parts, a.N, p.part_stride};
  if (a.epilogue == EPI_RESID) { r.x = a.res.x; r.ld = a.res.ld; }
  if (!join) { *result = r; return PHOTON_OK; }
  RowsArgs rows{};
  rows.in = r; rows.bias = a.bias; rows.sum = reinterpret_cast<float*>(a.out); rows.ld_sum = a.ldo; rows.M = a.M; rows.K = a.N;
  *result = whole;
  return launch_rows(rows, st);
}

// The projection with the operands written by it (one of the wide tiles, K unsplit) against the best tile and the pass over
// its fp32 result, which costs a launch and reads and writes 1.5 times that result at 4.5 bytes per ns (135 us at 32768 rows
// of 3072).  Measured: 8192 rows of 3072 82 against 73 + 37 us; the model's margin matters below some hundred rows only.
bool qkv_rope_pays(int64_t rows, int D, int d_h) {
  if (d_h != 64 || rows < ORDERED_ROWS) return false;
  float fused = 0.f, best = 0.f;
  plan_gemm(rows, 3 * D, D, PLAN_QKV, false, 0, 0.f, &fused);
  plan_gemm(rows, 3 * D, D, PLAN_F32, false, 0, 0.f, &best);
  return fused <= best + 4.f + 0.33f * (float)rows * 3 * D * 4e-6f;
}

int32_t launch_qkv_rope(const void* x, const void* W, int rows, int D, const QkvOperands& o, hipStream_t st) {
  if (o.H * 64 != D || o.M <= 0 || rows % o.M != 0 || o.Mp % 64 != 0 || o.Mp < o.M)
    return fail(PHOTON_ERR_UNSUPPORTED, "QKV projection: rows=%d D=%d do not match %d heads of 64 and %d positions", rows, D, o.H, o.M);
  GemmArgs p{};
  p.x = reinterpret_cast<const bf16_t*>(x); p.W = reinterpret_cast<const bf16_t*>(W); p.M = rows; p.N = 3 * D; p.K = D; p.qkv = o;
  return launch_gemm<GEMM_OUT_QKV>(p, plan_gemm(rows, 3 * D, D, PLAN_QKV, false, 0, 0.f), st);
}

static int32_t launch_chunker_gemm(const void* x, const void* w, const float* bias, void* out, int64_t M, int N, int K, hipStream_t st) {
  GemmArgs p{};
  p.x = (const bf16_t*)x; p.W = (const bf16_t*)w; p.bias = bias; p.out = out; p.ldo = N; p.M = (int)M; p.N = N; p.K = K;
  return launch_gemm<GEMM_OUT_BF16>(p, plan_gemm(M, N, K, PLAN_CHUNKER, false, 0, 0.f), st);
}

}  // namespace photon

using namespace photon;

extern "C" int32_t photon_contract_tile(int64_t rows, int32_t N, int32_t K, int32_t output, int32_t* tile_rows, int32_t* tile_columns,
                                        int32_t* splits, int32_t* walked) {
  clear_error();
  PHOTON_REQUIRE(rows >= 1 && rows <= (1LL << 24) && N >= 16 && N % 16 == 0 && K >= G_BK && K % G_BK == 0 && K <= (1 << 24), PHOTON_ERR_INVALID_ARG,
                 "%s: rows=%lld N=%d K=%d invalid", __func__, (long long)rows, N, K);
  PHOTON_REQUIRE(output >= PHOTON_CONTRACT_F32 && output <= PHOTON_CONTRACT_SWIGLU, PHOTON_ERR_INVALID_ARG, "%s: unknown output %d", __func__, output);
  PHOTON_REQUIRE(tile_rows && tile_columns && splits && walked, PHOTON_ERR_INVALID_ARG, "%s: null result", __func__);
  const bool gate_up = output == PHOTON_CONTRACT_SWIGLU, f32 = output == PHOTON_CONTRACT_F32;
  const GemmPlan plan = plan_gemm(rows, N, K, gate_up ? PLAN_SWIGLU : f32 ? PLAN_F32 : PLAN_CHUNKER, output != PHOTON_CONTRACT_CHUNKER && rows < ORDERED_ROWS,
                                  f32 ? contract_part_floats(rows, N) : 0, 0.f);
  *tile_rows = TILES[plan.kind].bm;
  *tile_columns = TILES[plan.kind].bn / (gate_up ? 2 : 1);
  *splits = plan.splits;
  *walked = gate_up && walks(plan, rows, N, K) ? 1 : 0;
  return PHOTON_OK;
}

extern "C" int32_t photon_chunker_project(const void* x, const void* w, const float* bias, void* out, int64_t rows,
                                          int32_t C, int32_t d_in, int32_t d_out, photon_dtype dt, void* stream) {
  clear_error();
  PHOTON_REQUIRE(valid_dtype(dt), PHOTON_ERR_UNSUPPORTED, "%s: unknown dtype %d", __func__, (int)dt);
  PHOTON_REQUIRE(rows >= 0 && C >= 1 && d_in >= 1 && d_out >= 1, PHOTON_ERR_INVALID_ARG,
                 "%s: rows=%lld C=%d d_in=%d d_out=%d invalid", __func__, (long long)rows, C, d_in, d_out);
  const int64_t K64 = (int64_t)C * d_in;
  PHOTON_REQUIRE(K64 <= (1 << 24) && rows <= (1LL << 24), PHOTON_ERR_UNSUPPORTED, "%s: problem too large for one launch", __func__);
  const int K = (int)K64;
  if (rows == 0) return PHOTON_OK;
  PHOTON_REQUIRE_PTR(x);
  PHOTON_REQUIRE_PTR(out);
  hipStream_t st = (hipStream_t)stream;
  if (w == nullptr) {
    PHOTON_REQUIRE(d_out == K, PHOTON_ERR_INVALID_ARG, "%s: concatenation without projection needs d_out == C*d_in (%d != %d)",
                   __func__, d_out, K);
    PHOTON_REQUIRE(bias == nullptr, PHOTON_ERR_INVALID_ARG, "%s: bias without a projection matrix", __func__);
    const int64_t bytes = rows * K * (int64_t)dtype_size(dt);
    PHOTON_REQUIRE(bytes % 16 == 0, PHOTON_ERR_UNSUPPORTED, "%s: rows*C*d_in*elem must be a multiple of 16 bytes", __func__);
    PHOTON_LAUNCH(KC_MISC, st, copy_bytes16_kernel, dim3((unsigned)((bytes / 16 + 255) / 256)), dim3(256), 0, st, (const uint4_t*)x,
                       (uint4_t*)out, bytes / 16);
    return check_launch("copy_bytes16_kernel");
  }
  PHOTON_REQUIRE_PTR(w);
  if (dt == PHOTON_F32) {
    PHOTON_REQUIRE(K % 4 == 0, PHOTON_ERR_UNSUPPORTED, "%s: fp32 path needs C*d_in (%d) to be a multiple of 4", __func__, K);
    LinearArgs a;
    a.x = (const float*)x; a.ldx = K; a.W = w; a.bias = bias; a.out = (float*)out; a.ldo = d_out; a.M = (int)rows; a.N = d_out; a.K = K;
    return launch_linear(a, st);
  }
  PHOTON_REQUIRE(K % 64 == 0 && d_out % 16 == 0, PHOTON_ERR_UNSUPPORTED,
                 "%s: bf16 path needs C*d_in (%d) to be a multiple of 64 and d_out (%d) of 16", __func__, K, d_out);
  return launch_chunker_gemm(x, w, bias, out, rows, d_out, K, st);
}
