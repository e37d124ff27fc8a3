// Internal launch interface of the few-row linear maps.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace photon {

enum LinearEpilogue { EPI_PLAIN = 0, EPI_RESID = 1, EPI_SWIGLU = 2 };

// y = rmsnorm(x; gain, eps) * W^T (gain == nullptr: y = x * W^T), then
//   EPI_PLAIN : out = y + bias
//   EPI_RESID : out = res + y + bias            (out may alias res)
//   EPI_SWIGLU: out = silu(y[:, :N]) * y[:, N:] (W has 2N rows: gate rows, then up rows)
struct LinearArgs {
  const float* x = nullptr;    // fp32 [M, K], row pitch ldx elements (x_bf16: bf16 values behind the pointer)
  int64_t ldx = 0;
  bool x_bf16 = false;         // bf16 weights only, no norm, plain or residual epilogue: x is the MFMA operand as it stands
  const void* W = nullptr;     // [N, K] (2N for EPI_SWIGLU) row-major, bf16 when w_bf16 else fp32
  bool w_bf16 = false;
  const float* gain = nullptr; // [K] or nullptr
  float eps = 0.f;
  const float* bias = nullptr; // [N] or nullptr
  const float* res = nullptr;  // [M, N], row pitch ldres
  int64_t ldres = 0;
  float* out = nullptr;        // [M, N], row pitch ldo
  int64_t ldo = 0;
  bool out_bf16 = false;       // bf16 weights only: out holds bf16 values (rounded to nearest even), ldo in elements
  int M = 0, N = 0, K = 0;
  int epilogue = EPI_PLAIN;
};

int32_t launch_linear(const LinearArgs& a, hipStream_t st);

// bf16 weights, activations small enough to stay in LDS: issues the launch and returns true, else returns false
// (the caller then takes the streaming kernel).  Arguments must have passed launch_linear's checks.
bool launch_linear_resident(const LinearArgs& a, hipStream_t st);

// bf16 weights, fp32 activations of 17-32 rows, plain or SwiGLU epilogue, contraction length at most 2048: two row tiles of
// 16 per workgroup at the accuracy (and with the per-row arithmetic) of the 16-row kernel; the matrix is streamed once.
// Returns true when the launch was issued.
bool launch_linear_resident_x2(const LinearArgs& a, hipStream_t st);

// ---- 17 rows and up with bf16 weights: row kernel (norm, rounding to bf16) + tiled MFMA contraction ----

// Rows as a sum: n_parts partial products of a contraction split over K, parts[s * part_stride + row * part_ld ..], added
// in order, plus x[row * ld ..] (nullptr: nothing).
struct RowSource {
  const float* x = nullptr;
  int64_t ld = 0;
  const float* parts = nullptr;
  int n_parts = 0;
  int64_t part_ld = 0, part_stride = 0;
  // rows off, off + mul, off + 2 mul, ..
  RowSource pick(int64_t mul, int64_t off) const {
    RowSource r = *this;
    if (x != nullptr) r.x += off * ld;
    if (parts != nullptr) r.parts += off * part_ld;
    r.ld *= mul;
    r.part_ld *= mul;
    return r;
  }
};

// v = in + bias (nullptr: none); sum = v; xb [M, K] (dense bf16) = rmsnorm(v; gain, eps) rounded to nearest even
// (gain == nullptr: v rounded); y = rmsnorm(v; gain, eps) in fp32.  Each output may be nullptr; sum may be in.x itself.
struct RowsArgs {
  RowSource in;
  const float* bias = nullptr;
  const float* gain = nullptr;
  float eps = 0.f;
  float* sum = nullptr;
  int64_t ld_sum = 0;
  uint16_t* xb = nullptr;
  float* y = nullptr;
  int64_t ldy = 0;
  int M = 0, K = 0;
};
int32_t launch_rows(const RowsArgs& a, hipStream_t st);

// The largest of a stretch of columns of one row and the column it sits in (the first, where several are equal).
struct RowBest {
  float value;
  int column;
};

// x [M, K] dense bf16, W [N, K] (2N rows for EPI_SWIGLU) bf16; out fp32 [M, ldo], or for EPI_SWIGLU bf16 [M, ldo].
// EPI_RESID: out = res + x W^T, where out and res must not overlap.  parts: scratch of part_cap floats for the partial
// products of a contraction split over K.  `result` says where the fp32 result lies: in out, or still in pieces
// (EPI_RESID: the residual rows and the partial products; EPI_PLAIN with split_ok: the partial products, without the
// bias), for the next kernel to add.  order_rows: the row count whose order of the sum over K is kept (0: M); passes that take
// the rows of several smaller passes together give a row the result it has there.
struct ContractArgs {
  const void* x = nullptr;
  const void* W = nullptr;
  const float* bias = nullptr;   // EPI_PLAIN
  RowSource res;                 // EPI_RESID, in one piece
  void* out = nullptr;
  int64_t ldo = 0;
  float* parts = nullptr;
  int64_t part_cap = 0;
  int M = 0, N = 0, K = 0;
  int epilogue = EPI_PLAIN, order_rows = 0;
  bool split_ok = false;
  bool cold = false;             // W is not in the memory-side cache: the matrices in use between two reads of it exceed that
  // EPI_PLAIN without bias: row m's best of every stretch of columns goes to best[m * stretches + stretch], where `best`
  // holds M * best_stretches_max(N); launch_contract sets *best_stretches, and leaves it where K is split (nothing is written)
  RowBest* best = nullptr;
};
inline int best_stretches_max(int N) { return (N + 31) / 32; }
int64_t contract_part_floats(int64_t rows, int D);     // scratch that lets every contraction of a D-wide module split as it would
int32_t launch_contract(const ContractArgs& a, RowSource* result, hipStream_t st, int* best_stretches = nullptr);

// ---- QKV projection of an encoder (heads of 64) that writes the attention's operands itself ----

// fp16 operands of the encoders' attention, per stream bh = sequence * H + head: qh, kh [bh][Mp][64] (rotated, q scaled),
// vt [bh][64][Mp]; M positions per sequence, Mp: rounded up to 64.  kc, vc (both or neither): cache of S_max rows of 64 per
// stream that receives the rotated keys and the values as bf16 or E4M3 bytes.  table: per position 32 cosines, 32 sines.
struct QkvOperands {
  uint16_t *qh = nullptr, *kh = nullptr, *vt = nullptr;
  void *kc = nullptr, *vc = nullptr;
  const float* table = nullptr;
  int64_t S_max = 0;
  int M = 0, Mp = 0, H = 0;
  float qscale = 0.f;
  bool cache_fp8 = false;
};
bool qkv_rope_pays(int64_t rows, int D, int d_h);
// x [rows, D] dense bf16, rows = sequences * M; W [3D, D].
int32_t launch_qkv_rope(const void* x, const void* W, int rows, int D, const QkvOperands& o, hipStream_t st);

}  // namespace photon
