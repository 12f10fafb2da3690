// Internal interface of the decode GEMV kernels (not part of the public ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace pda {

constexpr int kTileRows = 16;                   // rows of W per MFMA tile
constexpr int kTileK = 32;                      // k per MFMA tile
constexpr int kPairK = 2 * kTileK;              // k per step of a wave: one 128-byte line of an activation row
constexpr int kMaxGemvBatch = 256;              // sequences: sixteen 16-column tiles
// Batches above this need the output rows in groups of 128 (a limit of the
// public interface; the kernels themselves need groups of 16).
constexpr int kMaxGemvBatchAnyRows = 64;
constexpr int kPackThreads = 256;

// How rows_kernel splits y = x W^T: a workgroup takes `rt` row tiles x `bt`
// column tiles over the whole k range, or one of `splits` parts of it, its
// waves dealing the 64-k pairs among them.  row_groups x col_groups
// workgroups a split; with several column groups the workgroups of a row
// group share an XCD.
struct RowsPlan {
  int rt, bt, waves;
  int kb;          // steps per block of weights
  bool wide;       // 32 x 32 x 16 matrix-core tiles instead of 16 x 16 x 32
  bool fused;      // the prelude epilogue runs in rows_kernel
  int row_groups, col_groups;
  int splits;      // of k (1 unless the epilogue is a kernel of its own)
  int split_grid;  // workgroups of one split
  int grid;
  int ss_parts;    // partial sums of z^2 per row tile and sequence (o_proj)
};
constexpr int kMaxRowsSplits = 4;

// Partial sums of z^2 that rows_kernel leaves per row tile and sequence: one
// per lane group of an item (see its epilogue items).
constexpr int rows_ss_parts(int rt, int bt, int waves, bool wide) {
  return (wide ? 2 : 1) * (rt * bt < waves ? 2 : 1);
}

constexpr int kMaxSsParts = 4;

// fusable: the prelude epilogue may run in the kernel (the plan says whether
// it is to).  max_splits: at most kMaxRowsSplits.
RowsPlan plan_rows(int batch, int n, int k, int num_cus, bool fusable, int max_splits);
// Most floats of y, all splits together, that the plan of any k and any batch
// up to `batch` has: never less for a larger batch.
int64_t rows_most_floats(int batch, int n, int num_cus, int max_splits);

// What a prelude's epilogue does with the projection, in rows_kernel or in
// prelude_epilogue.
struct PreludeArgs {
  const float* y;            // fp32 [splits, batch, (hq + 2 hkv) * d], prelude_epilogue only
  int splits;
  const uint16_t* bias;      // bf16 [(hq + 2 hkv) * d] or null
  const uint16_t* q_norm;    // bf16 [d] or null
  const uint16_t* k_norm;    // bf16 [d] or null
  const int32_t* lens;       // [batch]
  uint16_t* q_out;           // bf16 [batch, hq, d]
  uint16_t* k_out;           // bf16 [batch, hkv, d] or null
  uint16_t* v_out;
  uint16_t* k_cache;         // bf16 [num_pages, page, hkv, d] or null (no append)
  uint16_t* v_cache;
  const int32_t* bt;         // [batch, maxp]
  int page_shift, num_pages, maxp;
  int batch, hq, hkv, d, rotary_dim, interleaved;
  // theta^(-2 * 2^k / rotary_dim) for k = 0..7, in fp64 from the host: the
  // frequency theta^(-2i/rotary_dim) of pair i (i < 128) is the product of
  // those for the set bits of i
  double freq_pow2[8];
  float eps;
};

// The prelude epilogues that rows_kernel can run itself: no norm over the
// head (a workgroup holds two of its tiles), and rotation partners in the
// two tiles of a pair (or in one, interleaved).
inline bool prelude_fusable(bool qk_norm, bool interleaved, int rotary_dim) {
  return !qk_norm && (interleaved || rotary_dim % 32 == 0);
}

constexpr int kMaxOProjHidden = 32768;
constexpr int kSumThreads = 1024;
constexpr int kSumFeatures = 8192;   // hidden size oproj_sum_kernel holds
constexpr int kNormThreads = 256;
constexpr int kNormFeatures = 4 * kNormThreads;  // features per workgroup of oproj_norm_kernel

struct OProjArgs {
  const uint16_t* residual;   // bf16 [batch, hidden]
  const uint16_t* norm_w;     // bf16 [hidden]
  uint16_t* residual_out;     // bf16 [batch, hidden] (may be residual itself)
  uint16_t* normed_out;       // bf16 [batch, hidden]
  float* z;                   // fp32 [splits, batch, hidden] scratch
  int splits;
  float* ss;                  // fp32 [batch, ss_count] scratch: partial sums of z^2
  int ss_count;
  int batch, hidden;
  float eps;
};

struct RowsArgs {
  const uint16_t* x;   // bf16 [batch, k]
  const uint16_t* wp;  // packed bf16 [n, k]
  float* y;            // fp32 [batch, n] (no epilogue in the kernel)
  int batch, n, k;
  int row_groups, col_groups;
  int splits, split_grid;
};

hipError_t launch_pack(const uint16_t* w, uint16_t* wp, int n, int k, hipStream_t st);
// y only
hipError_t launch_rows(const RowsArgs& a, const RowsPlan& p, hipStream_t st);
// with the whole prelude epilogue (prelude_fusable, a plan made with pairs)
hipError_t launch_rows_prelude(const RowsArgs& a, const RowsPlan& p, const PreludeArgs& e, hipStream_t st);
// z = y + residual and the partial sums of z^2
hipError_t launch_rows_residual(const RowsArgs& a, const RowsPlan& p, const OProjArgs& o, hipStream_t st);
hipError_t launch_prelude_epilogue(const PreludeArgs& a, hipStream_t st);
hipError_t launch_oproj_sum(const OProjArgs& a, hipStream_t st);
hipError_t launch_oproj_norm(const OProjArgs& a, hipStream_t st);

}  // namespace pda
