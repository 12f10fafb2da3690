// Decode GEMV, the attention prelude and the output projection for MI355X
// (gfx950, CDNA4, wave64).
//
// What is computed: the paper's kernel family (i), the attention prelude
// (Method, "Principle-Driven LLM Kernel Generator"): the QKV projection of
// the new token's hidden state, then per-head RMSNorm of q and k (when the
// model has it) and the rotary position embedding of q and k.  Its template
// GEMV (Method, "CUDA Code Generator") reads [N, K] weight rows with 128-bit
// loads and reduces across lanes; on CDNA4 the same bandwidth-bound
// product is laid out differently:
//
//  * Weights are packed once into the matrix cores' operand order: a tile of
//    16 rows x 32 k is 1 KB, and lane l of a wave holds row l % 16, k
//    8 (l / 16) .. +7 of it.  Every weight load of the GEMV is then one
//    contiguous 1 KB wave access that feeds v_mfma_f32_16x16x32_bf16
//    directly, with no LDS staging and no lane shuffles.
//  * The batch forms the MFMA's B columns in tiles of 16 sequences; x rows
//    past the batch read as zeros through the buffer descriptor's size.
//  * A workgroup computes its output rows over the whole k range (or one of
//    a few splits), see rows_kernel, so most preludes end in the same kernel:
//    bias, rotation, bf16 rounding and the KV append into the page slot.
//    With a per-head RMSNorm, which needs all rows of a head, and in a few
//    large shapes the epilogue is a kernel of its own.
//
// The output projection after attention (kernel family (v): o_proj GEMV +
// residual add + the RMSNorm that follows) runs on the same kernel, which
// adds the residual and leaves z in fp32 with partial sums of z^2; the norm
// spans all features of a sequence and is a second, small kernel.
#include "pda_gemv.h"

#include <atomic>
#include <cmath>
#include <type_traits>
#include <utility>

namespace pda {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kBufferDword3 = 0x00020000;  // raw 32-bit buffer format
constexpr int kCachePolicyNT = 2;          // non-temporal: weights are read once

__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a >> 32));
  void* ub = reinterpret_cast<void*>((static_cast<uint64_t>(hi) << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(ub, 0, static_cast<int>(__builtin_amdgcn_readfirstlane(bytes)),
                                           kBufferDword3);
}

// Packed layout: tile (t, kt) of rows 16t .. 16t+15 and k 32kt .. 32kt+31 is
// stored at element (t * (k / 32) + kt) * 512; inside it, 16-byte chunk l
// holds W[16t + l % 16][32kt + 8 (l / 16) .. +7].  One thread per chunk.
__global__ __launch_bounds__(kPackThreads) void pack_kernel(const uint16_t* __restrict__ w,
                                                            uint16_t* __restrict__ wp, int n, int k) {
  const int64_t chunk = static_cast<int64_t>(blockIdx.x) * kPackThreads + threadIdx.x;
  const int64_t chunks = static_cast<int64_t>(n) * k / 8;
  if (chunk >= chunks) return;
  const int kt_count = k / kTileK;
  const int64_t tile = chunk / 64;
  const int l = static_cast<int>(chunk % 64);
  const int64_t t = tile / kt_count;
  const int kt = static_cast<int>(tile % kt_count);
  const int64_t row = t * kTileRows + (l & 15);
  const int64_t col = static_cast<int64_t>(kt) * kTileK + 8 * (l >> 4);
  *reinterpret_cast<u32x4*>(wp + chunk * 8) = *reinterpret_cast<const u32x4*>(w + row * k + col);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t h) {
  return __builtin_bit_cast(float, static_cast<uint32_t>(h) << 16);
}

__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f));
}

// y[b, n] = sum_k x[b, k] W[n, k] over a packed W.  A workgroup takes RT row
// tiles (16 rows each) x BT column tiles (16 sequences each) over the whole k
// range, or one of a.splits parts of it.  Its W waves deal the 64-k pairs of
// k tiles among themselves (wave w takes pairs w, w + W, ...), each with
// accumulators for all RT x BT tiles, and add them in LDS at the end.
//
// What bounds it is what a CU can take in: RT x 16 weight rows from memory
// and BT x 16 activation rows from L2, (16 RT + 16 BT) x k x 2 bytes a
// workgroup.  Measured on this GPU: 26 bytes/ns and CU from memory with every
// CU reading (6.7 TB/s), 50 with a quarter of them, whatever the depth; 104
// from L2; and since a CU's loads return in order, 45-60 for a mix of the two
// in small pieces.  Hence:
//  * Activations go straight into LDS, 8 rows x 128 bytes per wave load
//    (whole cache lines, consecutive lanes along a row): 104 bytes/ns, where
//    loads in operand order (16 rows x 64 bytes, consecutive lanes in
//    different rows) reach 38.  Lane l fetches the 16-byte piece
//    (l % 8) ^ (l / 8) of row l / 8, so that the operand reads (16 or 32
//    rows, one piece each) are free of bank conflicts.
//  * Weights come in bursts of KB steps ahead of the block that uses them,
//    not one step at a time: the L2 hits between two bursts then flow
//    together (64 x 4096 -> 6144: 19.8 -> 17.1 us a call).
//  * Every wave has a ring of DX steps of its own in LDS and two blocks of
//    weights in registers: no barrier before the final sum.
//  * The planner (plan_rows) picks the tile shape and the splits for the
//    least of those bytes that still fills the CUs.
// A stream-K split over workgroups of 8 row tiles, which this replaces, read
// its activations in operand order or behind a barrier per chunk and passed
// 9 MB of fp32 partials at 64 sequences, 38 MB at 256, to the epilogue.
// Whole calls replayed from a graph, cold weights, before -> now: prelude
// 64 x 4096 -> 6144 19.9 -> 17.1 us, 256 x 5120 -> 7168 48 -> 39, 16 x 3072
// -> 5120 13.4 -> 9.8, 4 x 8192 -> 10240 32.1 -> 31.2; o_proj 100 x 5120 ->
// 5120 28.3 -> 24.4, 4 x 8192 -> 8192 29.0 -> 26.5, 200 x 3072 -> 3072
// 26.8 -> 17.7.
//
// Columns at or past the batch and k at or past the end read as zeros
// (outside the descriptors), as do steps past a wave's last pair: every wave
// of the workgroup takes the same number of blocks with fixed wait counts.
struct NoEpilogue {};

// waves per SIMD the register budget is set for
constexpr int rows_min_waves(int rt, int bt, int w, int kb) { return w > 4 ? (rt * bt * kb <= 4 ? 4 : 2) : 1; }
// s_waitcnt vmcnt(n) alone; vmcnt is split over bits 3:0 and 15:14
constexpr int kWaitLoads = 0x0F70;
constexpr int wait_loads(int n) { return kWaitLoads | (n & 15) | ((n >> 4) << 14); }
__host__ __device__ constexpr int rows_lds_bytes(int rt, int bt, int w, int dx) {
  const int ring = w * dx * bt * 2048, sum = w * rt * bt * 1024;
  return ring > sum ? ring : sum;
}

// N consecutive bf16 values, packed two to a register; p need only be 2-byte
// aligned (the memory pipeline takes any alignment).
template <int N>
__device__ __forceinline__ void load_bf16(const uint16_t* p, uint32_t* v) {
  __builtin_memcpy(v, p, 2 * N);
}
__device__ __forceinline__ float unpack_bf16(const uint32_t* v, int j) {
  return bf16_to_f32(static_cast<uint16_t>(v[j / 2] >> (16 * (j & 1))));
}
template <int N>
__device__ __forceinline__ void store_bf16(uint16_t* p, const float (&v)[N]) {
  uint32_t w[N / 2];
#pragma unroll
  for (int j = 0; j < N / 2; ++j)
    w[j] = f32_to_bf16(v[2 * j]) | (static_cast<uint32_t>(f32_to_bf16(v[2 * j + 1])) << 16);
  __builtin_memcpy(p, w, 2 * N);
}

// Sine and cosine of position pos at rotary pair i0 + j, j < N (i0 a multiple
// of N): the angle p * theta^(-2i/r), in turns, in fp64 (positions reach 10^5
// and more, where an fp32 angle would already be off by ~10^-2 rad); its
// fraction in [-1/2, 1/2] goes to the hardware sine and cosine, which take
// turns.  The frequency is the product of the host's theta^(-2 * 2^k / r)
// over the set bits k of i.
template <int N>
__device__ __forceinline__ void rope_angles(const PreludeArgs& a, int pos, int i0, float (&sn)[N], float (&cs)[N]) {
  constexpr double kInvTwoPi = 0.15915494309189535;
  constexpr int kLow = N == 4 ? 2 : (N == 2 ? 1 : 0);
  double base = static_cast<double>(pos) * kInvTwoPi;
#pragma unroll
  for (int k = kLow; k < 8; ++k) base = (i0 >> k) & 1 ? base * a.freq_pow2[k] : base;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    double t = base;
    if (j & 1) t *= a.freq_pow2[0];
    if (j & 2) t *= a.freq_pow2[1];
    const float frac = static_cast<float>(t - __builtin_rint(t));
    sn[j] = __builtin_amdgcn_sinf(frac);
    cs[j] = __builtin_amdgcn_cosf(frac);
  }
}

__device__ __forceinline__ int clamped(int x, int most) { return x < 0 ? 0 : (x > most ? most : x); }

template <int RT, int BT, int W, int DX, int KB, bool kWide, bool kShared, class Epilogue>
__global__ __launch_bounds__(W * 64, rows_min_waves(RT, BT, W, KB)) void rows_kernel(RowsArgs a, Epilogue e) {
  constexpr bool kPrelude = std::is_same<Epilogue, PreludeArgs>::value;
  constexpr bool kResidual = std::is_same<Epilogue, OProjArgs>::value;
  static_assert(KB % DX == 0, "a block of weights covers whole turns of the activation ring");
  static_assert(!kPrelude || RT % 2 == 0, "the prelude's row tiles go in pairs");
  static_assert(!kWide || (RT % 2 == 0 && BT % 2 == 0), "wide tiles take row and column tiles in pairs");
  constexpr int kSlot = BT * 2048;               // one step's activations of a wave
  constexpr int kLx = 2 * BT, kLw = 2 * RT;      // vector memory instructions of a step
  constexpr uint32_t kOutside = 0x80000000u;     // past any descriptor: reads zero
  // matrix-core tiles, kTR x kTC of 16 x 16 x 32 or, with kWide, of
  // 32 x 32 x 16 (two row tiles x two column tiles); kTM of them cover a
  // step's k, and an accumulator is kTG groups of four rows per lane
  constexpr int kTR = kWide ? RT / 2 : RT, kTC = kWide ? BT / 2 : BT;
  constexpr int kTM = kWide ? 4 : 2, kTG = kWide ? 4 : 1;
  using Acc = typename std::conditional<kWide, f32x16, f32x4>::type;
  // epilogue items: a group of one accumulator, or for the prelude the same
  // group of both row tiles of a pair; half the rows of each lane where
  // there are fewer groups than waves
  constexpr int kUnits = kTR * kTC * kTG / (kPrelude ? 2 : 1);
  constexpr int kSub = kUnits < W ? 2 : 1;
  constexpr int kRows = 4 / kSub;                // rows per lane of an item
  constexpr int kItems = kUnits * kSub;
  constexpr int kPer = (kItems + W - 1) / W;     // items per wave, at most
  extern __shared__ __align__(1024) unsigned char xs[];

  const int lane = threadIdx.x & 63;
  const int wv = uniform(threadIdx.x >> 6);
  const int col = kWide ? lane & 31 : lane & 15;   // of a tile: operand row or column, result column
  const int kblk = kWide ? lane >> 5 : lane >> 4;  // operand k block of 8, result row block of 4
  const int k = a.k;
  const int kt_count = k / kTileK;
  // k split `sp` of a.splits (NoEpilogue only): whole pairs [pair0, pair1)
  const int sp = a.splits > 1 ? static_cast<int>(blockIdx.x) / a.split_grid : 0;
  const int blk0 = static_cast<int>(blockIdx.x) - sp * a.split_grid;
  int rg = blk0, bg = 0;
  if constexpr (kShared) {
    // workgroups go to the XCDs round-robin: those of one row group take
    // consecutive places of one XCD, so that its weights come from memory
    // once and from that XCD's L2 after that
    const int i = blk0 >> 3;
    const int q = i / a.col_groups;
    rg = q * 8 + (blk0 & 7);
    bg = i - q * a.col_groups;
    if (rg >= a.row_groups) return;
  }
  const int tile0 = rg * RT;                     // first row tile (or first pair x 2)
  const int b0 = bg * BT * 16;                   // first sequence
  const int tiles = a.n / kTileRows;

  // Item `it`: accumulator column c; row tile r of the workgroup (with the
  // prelude, pair r) and the lane's first row in it.
  struct Item {
    int c, r, row0, acc_r, group, sub;
  };
  auto item_of = [&](int it) __attribute__((always_inline)) {
    Item m;
    const int u = it / kSub;
    m.sub = it % kSub;
    constexpr int kG = kWide ? (kPrelude ? 2 : 4) : 1;  // groups of an accumulator taken one by one
    m.group = u % kG;
    m.c = (u / kG) % kTC;
    const int x = u / kG / kTC;
    m.acc_r = x;
    m.r = kWide && !kPrelude ? 2 * x + (m.group >> 1) : x;
    m.row0 = (kWide ? 8 * (m.group & 1) : 0) + 4 * kblk + m.sub * kRows;
    return m;
  };

  // ---- what the epilogue reads beside the sums, requested first
  int item_b[kPer];
  bool item_on[kPer];
  float sn[kPer][kRows], cs[kPer][kRows];
  // residual, or bias of the pair's rows: kept as loaded and converted after
  // the loop, so that nothing waits for them here
  uint32_t raw[kPer][kPrelude ? kRows : kRows / 2];
  int pos[kPer];
#pragma unroll
  for (int t = 0; t < kPer; ++t) {
    const int it = wv + t * W;
    const Item m = item_of(it);
    item_b[t] = b0 + (kWide ? 32 : 16) * m.c + col;
    item_on[t] = it < kItems && item_b[t] < a.batch;
    if constexpr (kPrelude) pos[t] = item_on[t] ? e.lens[item_b[t]] : 0;
    if constexpr (kResidual) {
      const int n = 16 * (tile0 + m.r) + m.row0;
      item_on[t] = item_on[t] && n < a.n;
#pragma unroll
      for (int j = 0; j < kRows / 2; ++j) raw[t][j] = 0u;
      if (item_on[t]) load_bf16<kRows>(e.residual + static_cast<int64_t>(item_b[t]) * a.n + n, raw[t]);
    }
  }

  // ---- load streams
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(a.x, static_cast<uint32_t>(a.batch) * k * 2u);
  const int xrow = lane >> 3;
  const int xpiece = (lane & 7) ^ xrow;
  const uint32_t xlane = static_cast<uint32_t>(b0 + xrow) * k * 2u + xpiece * 16u;
  const uint32_t xstep8 = static_cast<uint32_t>(k) * 16u;  // bytes of 8 rows
  unsigned char* ring = xs + wv * (DX * kSlot);
  // row tile r of the workgroup; a prelude pair's second tile holds the
  // rotation partners of its first
  auto tile_of = [&](int r) __attribute__((always_inline)) {
    int t = tile0 + r;
    if constexpr (kPrelude) {
      // pair q of a head of d / 16 tiles, rotated in halves over r dims:
      // tiles (q, q + r / 32) for q < r / 32, then and otherwise (2q, 2q + 1)
      const int per_head = e.d / 32;
      const int pair = t >> 1;
      const int h = pair / per_head, q = pair - h * per_head;
      const int half = (!e.interleaved && h < e.hq + e.hkv) ? e.rotary_dim / 32 : 0;
      t = h * 2 * per_head + (q < half ? q + (r & 1) * half : 2 * q + (r & 1));
    }
    return uniform(t);
  };
  // one descriptor per row tile, or (wide) per two, the second `wdelta` on
  __amdgpu_buffer_rsrc_t rw[kTR];
  uint32_t wlane[kTR];
#pragma unroll
  for (int r = 0; r < kTR; ++r) {
    const int t = tile_of(kWide ? 2 * r : r);
    const int t2 = kWide ? tile_of(2 * r + 1) : t;
    const uint32_t delta = static_cast<uint32_t>(t2 - t) * kt_count * 1024u;
    // tiles past the last row are outside: both, or (wide) the second alone
    const uint32_t bytes = t2 < tiles ? delta + kt_count * 1024u : (t < tiles ? kt_count * 1024u : 0u);
    rw[r] = make_rsrc(a.wp + static_cast<int64_t>(t < tiles ? t : 0) * kt_count * (kTileRows * kTileK), bytes);
    wlane[r] = kWide ? (lane & 16 ? delta : 0u) + (16 * kblk + (lane & 15)) * 16u : lane * 16u;
  }
  const int pairs = (kt_count + 1) / 2;
  const int pair0 = a.splits > 1 ? sp * pairs / a.splits : 0;
  const int pair1 = a.splits > 1 ? (sp + 1) * pairs / a.splits : pairs;
  const int k_end = pair1 * kPairK < k ? pair1 * kPairK : k;
  const int kt_end = pair1 * 2 < kt_count ? pair1 * 2 : kt_count;
  const int steps = (pair1 - pair0 + W - 1) / W;

  auto issue_x = [&](int slot, int s) __attribute__((always_inline)) {
    const int k0 = (pair0 + wv + s * W) * kPairK;
    const uint32_t off = (k0 + 8 * xpiece < k_end ? xlane : kOutside) + k0 * 2u;
#pragma unroll
    for (int i = 0; i < kLx; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rx, (__attribute__((address_space(3))) void*)(ring + slot * kSlot + i * 1024), 16, off + i * xstep8, 0, 0, 0);
  };
  // the weights of block blk (KB steps); k tiles past the end are outside
  u32x4 wa[2][KB][kTR][kTM];
  auto issue_w = [&](int buf, int blk) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < KB; ++i) {
      const int kt = 2 * (pair0 + wv + (blk * KB + i) * W);
      uint32_t at[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) at[j] = kt + j < kt_end ? static_cast<uint32_t>(kt + j) * 1024u : kOutside;
#pragma unroll
      for (int r = 0; r < kTR; ++r)
#pragma unroll
        for (int m = 0; m < kTM; ++m)
          wa[buf][i][r][m] = __builtin_amdgcn_raw_buffer_load_b128(
              rw[r], wlane[r] + at[kWide ? m >> 1 : m] + (kWide ? (m & 1) * 512 : 0), 0, kShared ? 0 : kCachePolicyNT);
    }
  };

  Acc acc[kTR][kTC];
#pragma unroll
  for (int r = 0; r < kTR; ++r)
#pragma unroll
    for (int c = 0; c < kTC; ++c) acc[r][c] = Acc{};
  // operand m of accumulator column c: row `col`, piece (pieces per m) m + kblk
  const int frag0 = (col >> 3) * 1024 + (col & 7) * 128 + ((kblk ^ (col & 7)) * 16);
  u32x4 xb[kTC][kTM];
  auto operands = [&](int slot) __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
#pragma unroll
    for (int c = 0; c < kTC; ++c)
#pragma unroll
      for (int m = 0; m < kTM; ++m)
        xb[c][m] = *reinterpret_cast<const u32x4*>(ring + slot * kSlot + c * (kSlot / kTC) + (frag0 ^ (m * (128 / kTM))));
  };
  // the slot takes the activations DX steps on once its operands are in registers
  auto refill = [&](int slot, int s) __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    asm volatile("" ::: "memory");
    issue_x(slot, s + DX);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto multiply = [&](int buf, int i) __attribute__((always_inline)) {
#pragma unroll
    for (int m = 0; m < kTM; ++m)
#pragma unroll
      for (int c = 0; c < kTC; ++c)
#pragma unroll
        for (int r = 0; r < kTR; ++r) {
          const bf16x8 w = __builtin_bit_cast(bf16x8, wa[buf][i][r][m]), v = __builtin_bit_cast(bf16x8, xb[c][m]);
          if constexpr (kWide)
            acc[r][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, v, acc[r][c], 0, 0, 0);
          else
            acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, v, acc[r][c], 0, 0, 0);
        }
  };

  issue_w(0, 0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 0; s < DX; ++s) issue_x(s, s);
  __builtin_amdgcn_sched_barrier(0);

  // while the first loads are in flight: rotary angles, bias, page ids
  uint32_t page_id[kPer];  // block-table entry of the appended token
  if constexpr (kPrelude) {
    const int per_head = e.d / 32;
#pragma unroll
    for (int t = 0; t < kPer; ++t) {
      const Item m = item_of(wv + t * W);
      const int pair = (tile0 >> 1) + m.r;
      const int h = pair / per_head, q = pair - h * per_head;
      const int p = pos[t] > 0 ? pos[t] - 1 : 0;
      page_id[t] = 0u;
      item_on[t] = item_on[t] && h < e.hq + 2 * e.hkv;
      const bool turned = h < e.hq + e.hkv;
      int tA = 2 * q, tB = 2 * q + 1;
      if (!e.interleaved && turned && q < e.rotary_dim / 32) tA = q, tB = q + e.rotary_dim / 32;
      if (item_on[t] && turned) {
        if (e.interleaved) {
          float s2[kRows / 2], c2[kRows / 2], s3[kRows / 2], c3[kRows / 2];
          rope_angles<kRows / 2>(e, p, (16 * tA + m.row0) / 2, s2, c2);
          rope_angles<kRows / 2>(e, p, (16 * tB + m.row0) / 2, s3, c3);
#pragma unroll
          for (int j = 0; j < kRows / 2; ++j) {
            sn[t][j] = s2[j], cs[t][j] = c2[j];
            sn[t][kRows / 2 + j] = s3[j], cs[t][kRows / 2 + j] = c3[j];
          }
        } else {
          rope_angles<kRows>(e, p, 16 * tA + m.row0, sn[t], cs[t]);
        }
      }
#pragma unroll
      for (int j = 0; j < kRows; ++j) raw[t][j] = 0u;
      if (e.bias && item_on[t]) {
        load_bf16<kRows>(e.bias + h * e.d + 16 * tA + m.row0, raw[t]);
        load_bf16<kRows>(e.bias + h * e.d + 16 * tB + m.row0, raw[t] + kRows / 2);
      }
      if (e.k_cache && item_on[t] && h >= e.hq) {
        const int at = clamped(pos[t], e.maxp << e.page_shift) - 1;
        if (at >= 0) page_id[t] = static_cast<uint32_t>(e.bt[static_cast<int64_t>(item_b[t]) * e.maxp + (at >> e.page_shift)]);
      }
    }
  }

  // A block issues the next block's weights, then per step waits for the
  // step's activations (and so for every older load, its weights among
  // them), reads them, requests those of DX steps on and multiplies.  The
  // last block issues no weights, and what it waits for is all that is in
  // flight (a fixed count would not do there: the compiler drops loads whose
  // results no later step uses).
  auto block = [&](int buf, int blk, auto last) __attribute__((always_inline)) {
    constexpr bool kLast = decltype(last)::value;
    if constexpr (!kLast) {
      issue_w(buf ^ 1, blk + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = 0; j < KB; ++j) {
      if constexpr (kLast) {
        if (j == 0 || j >= DX) __builtin_amdgcn_s_waitcnt(kWaitLoads);
      } else {
        // younger than the step's activations: those of the DX - 1 steps
        // after it, and the block's weights where they were issued before
        constexpr int kEarly = (DX - 1) * kLx + KB * kLw, kLate = (DX - 1) * kLx;
        static_assert(kEarly < 64, "vmcnt holds at most 63");
        if (j < DX)
          __builtin_amdgcn_s_waitcnt(wait_loads(kEarly));
        else
          __builtin_amdgcn_s_waitcnt(wait_loads(kLate));
      }
      operands(j % DX);
      if (!kLast || j + DX < KB) refill(j % DX, blk * KB + j);
      multiply(buf, j);
    }
  };
  const int blocks = (steps + KB - 1) / KB;
  int blk = 0;
  for (; blk + 2 < blocks; blk += 2) {
    block(0, blk, std::false_type{});
    block(1, blk + 1, std::false_type{});
  }
  if (blk + 1 < blocks) {
    block(0, blk, std::false_type{});
    block(1, blk + 1, std::true_type{});
  } else {
    block(0, blk, std::true_type{});
  }

  // ---- the waves' sums meet in LDS
  __builtin_amdgcn_s_waitcnt(kWaitLoads);  // copies into the rings (zeros past the end) are done
  __syncthreads();
  f32x4* red = reinterpret_cast<f32x4*>(xs);  // [W][kTR][kTC][kTG][64 lanes]
#pragma unroll
  for (int r = 0; r < kTR; ++r)
#pragma unroll
    for (int c = 0; c < kTC; ++c)
#pragma unroll
      for (int g = 0; g < kTG; ++g)
        red[(((wv * kTR + r) * kTC + c) * kTG + g) * 64 + lane] =
            f32x4{acc[r][c][4 * g], acc[r][c][4 * g + 1], acc[r][c][4 * g + 2], acc[r][c][4 * g + 3]};
  __syncthreads();
  auto total = [&](int r, int c, int g, int sub, float (&v)[kRows]) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < kRows; ++j) v[j] = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const float* p = reinterpret_cast<const float*>(red + (((w * kTR + r) * kTC + c) * kTG + g) * 64 + lane) + sub * kRows;
#pragma unroll
      for (int j = 0; j < kRows; ++j) v[j] += p[j];
    }
  };
#pragma unroll
  for (int t = 0; t < kPer; ++t) {
    const int it = wv + t * W;
    if (kItems % W != 0 && it >= kItems) break;
    const Item m = item_of(it);
    const int64_t b = item_b[t];
    if constexpr (kPrelude) {
      // the pair's tiles: two accumulators, or two groups of one
      float v[2][kRows];
      total(kWide ? m.acc_r : 2 * m.acc_r, m.c, m.group, m.sub, v[0]);
      total(kWide ? m.acc_r : 2 * m.acc_r + 1, m.c, kWide ? m.group + 2 : 0, m.sub, v[1]);
      const int per_head = e.d / 32;
      const int pair = (tile0 >> 1) + m.r;
      const int h = pair / per_head, q = pair - h * per_head;
      const bool turned = h < e.hq + e.hkv;
      const bool halves = !e.interleaved && turned && q < e.rotary_dim / 32;
      const int eA = 16 * (halves ? q : 2 * q) + m.row0;
      const int eB = 16 * (halves ? q + e.rotary_dim / 32 : 2 * q + 1) + m.row0;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < kRows; ++j) v[i][j] += unpack_bf16(raw[t] + i * (kRows / 2), j);
      if (halves) {
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
          const float x0 = v[0][j], x1 = v[1][j];
          v[0][j] = x0 * cs[t][j] - x1 * sn[t][j];
          v[1][j] = x1 * cs[t][j] + x0 * sn[t][j];
        }
      } else if (e.interleaved && turned) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < kRows; j += 2) {
            const int ei = (i ? eB : eA) + j;
            const float c1 = cs[t][i * (kRows / 2) + j / 2], s1 = sn[t][i * (kRows / 2) + j / 2];
            const float x0 = v[i][j], x1 = v[i][j + 1];
            if (ei < e.rotary_dim) {
              v[i][j] = x0 * c1 - x1 * s1;
              v[i][j + 1] = x1 * c1 + x0 * s1;
            }
          }
      }
      if (!item_on[t]) continue;
      uint16_t* dst = nullptr;
      if (h < e.hq) {
        dst = e.q_out + (b * e.hq + h) * e.d;
      } else {
        const bool is_k = turned;
        const int g = is_k ? h - e.hq : h - e.hq - e.hkv;
        uint16_t* out = is_k ? e.k_out : e.v_out;
        if (out) dst = out + (b * e.hkv + g) * e.d;
        const int at = clamped(pos[t], e.maxp << e.page_shift) - 1;
        if (e.k_cache && at >= 0) {  // length 0: no token in this slot, nothing to append
          const int64_t page = page_id[t] < static_cast<uint32_t>(e.num_pages) ? page_id[t] : e.num_pages - 1;
          const int64_t row = (page << e.page_shift) + (at & ((1 << e.page_shift) - 1));
          uint16_t* cache = (is_k ? e.k_cache : e.v_cache) + (row * e.hkv + g) * e.d;
          store_bf16<kRows>(cache + eA, v[0]);
          store_bf16<kRows>(cache + eB, v[1]);
        }
      }
      if (dst) {
        store_bf16<kRows>(dst + eA, v[0]);
        store_bf16<kRows>(dst + eB, v[1]);
      }
    } else {
      const int tile = tile0 + m.r;
      const int n = 16 * tile + m.row0;
      float v[kRows];
      total(m.acc_r, m.c, m.group, m.sub, v);
      if constexpr (kResidual) {
        float ss = 0.f;
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
          v[j] += unpack_bf16(raw[t], j);
          ss += v[j] * v[j];
        }
        // over the lanes of one column: a row tile, or half of one (wide)
        if constexpr (!kWide) ss += __shfl_xor(ss, 16);
        ss += __shfl_xor(ss, 32);
        constexpr int kParts = rows_ss_parts(RT, BT, W, kWide);
        const int part = kWide ? (m.group & 1) * kSub + m.sub : m.sub;
        if (item_on[t] && kblk == 0) e.ss[b * e.ss_count + tile * kParts + part] = ss;
      }
      if (b < a.batch && n < a.n) {
        float* p = a.y + (static_cast<int64_t>(sp) * a.batch + b) * a.n + n;
        if constexpr (kRows == 4)
          *reinterpret_cast<f32x4*>(p) = f32x4{v[0], v[1], v[2], v[3]};
        else
          *reinterpret_cast<float2*>(p) = make_float2(v[0], v[1]);
      }
    }
  }
}

// Second kernel of o_proj: workgroup (sequence b, chunk of kNormFeatures
// features) adds the sequence's partial sums of z^2 (ss_count of them, in a
// fixed order) and writes residual_out = bf16(z) and
// normed_out = z / sqrt(mean + eps) * w for its chunk.  z and the weights
// are requested before the sums are used.
__global__ __launch_bounds__(kNormThreads) void oproj_norm_kernel(OProjArgs a) {
  __shared__ float wsum[kNormThreads / 64];
  const int chunks = (a.hidden + kNormFeatures - 1) / kNormFeatures;
  const int b = blockIdx.x / chunks;
  const int c = blockIdx.x - b * chunks;
  const int tid = threadIdx.x;
  const int n = c * kNormFeatures + 4 * tid;
  const bool in = n < a.hidden;
  const int64_t at = static_cast<int64_t>(b) * a.hidden + n;
  float z[4] = {0.f, 0.f, 0.f, 0.f};
  uint32_t w[2] = {0u, 0u};
  if (in) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(a.z + at);
#pragma unroll
    for (int j = 0; j < 4; ++j) z[j] = v[j];
    load_bf16<4>(a.norm_w + n, w);
  }
  const float* ss = a.ss + static_cast<int64_t>(b) * a.ss_count;
  float t = 0.f;
#pragma unroll 4
  for (int i = tid; i < a.ss_count; i += kNormThreads) t += ss[i];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off);
  if ((tid & 63) == 0) wsum[tid >> 6] = t;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int i = 0; i < kNormThreads / 64; ++i) tot += wsum[i];
  const float inv = rsqrtf(tot / a.hidden + a.eps);
  if (!in) return;
  float h[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) h[j] = z[j] * inv * unpack_bf16(w, j);
  store_bf16<4>(a.residual_out + at, z);
  store_bf16<4>(a.normed_out + at, h);
}

// Second kernel of o_proj where the projection was split along k: one
// workgroup per sequence b adds the splits' partials (in order) and the
// residual, kept in registers (hidden <= kSumFeatures), reduces the sum of
// z^2 in a fixed order and writes both outputs.
__global__ __launch_bounds__(kSumThreads) void oproj_sum_kernel(OProjArgs a) {
  constexpr int kGroups = kSumFeatures / (4 * kSumThreads);
  __shared__ float wsum[kSumThreads / 64];
  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const int64_t base = static_cast<int64_t>(b) * a.hidden;
  const int64_t stride = static_cast<int64_t>(a.batch) * a.hidden;
  float z[kGroups][4];
  uint32_t w[kGroups][2];
  float ss = 0.f;
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    const int n = 4 * (tid + kSumThreads * g);
#pragma unroll
    for (int j = 0; j < 4; ++j) z[g][j] = 0.f;
    w[g][0] = w[g][1] = 0u;
    if (n < a.hidden) {
      uint32_t r[2];
      load_bf16<4>(a.norm_w + n, w[g]);
      load_bf16<4>(a.residual + base + n, r);
      f32x4 part[kMaxRowsSplits];
#pragma unroll
      for (int s = 0; s < kMaxRowsSplits; ++s)
        part[s] = *reinterpret_cast<const f32x4*>(a.z + (s < a.splits ? s : a.splits - 1) * stride + base + n);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float y = part[0][j];
#pragma unroll
        for (int s = 1; s < kMaxRowsSplits; ++s) y += s < a.splits ? part[s][j] : 0.f;
        z[g][j] = y + unpack_bf16(r, j);
        ss += z[g][j] * z[g][j];
      }
      store_bf16<4>(a.residual_out + base + n, z[g]);
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) ss += __shfl_xor(ss, off);
  if ((tid & 63) == 0) wsum[tid >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int i = 0; i < kSumThreads / 64; ++i) tot += wsum[i];
  const float inv = rsqrtf(tot / a.hidden + a.eps);
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    const int n = 4 * (tid + kSumThreads * g);
    if (n < a.hidden) {
      float h[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) h[j] = z[g][j] * inv * unpack_bf16(w[g], j);
      store_bf16<4>(a.normed_out + base + n, h);
    }
  }
}

// One wave per (sequence b, head h) of the projection: h < hq is a q head,
// then hkv k heads, then hkv v heads.  Lane owns elements lane + 64 j.
template <int D>
__global__ __launch_bounds__(64) void prelude_epilogue(PreludeArgs a) {
  constexpr int E = D / 64;
  __shared__ float s[D];
  const int heads = a.hq + 2 * a.hkv;
  const int b = blockIdx.x / heads;
  const int h = blockIdx.x - b * heads;
  const int lane = threadIdx.x;
  const bool is_q = h < a.hq;
  const bool is_k = !is_q && h < a.hq + a.hkv;
  const uint16_t* nw = is_q ? a.q_norm : (is_k ? a.k_norm : nullptr);

  // Everything the wave reads is requested before any of it is used: the
  // length, then (for an append) the page id of the new token's slot, the
  // partials, the bias and the norm weights.
  const int L = a.lens[b];
  const int pos = L > 0 ? L - 1 : 0;
  const bool kv_head = !is_q;
  const int g = kv_head ? (is_k ? h - a.hq : h - a.hq - a.hkv) : 0;
  uint16_t* cache = kv_head ? (is_k ? a.k_cache : a.v_cache) : nullptr;
  int64_t row = 0;
  if (cache) {
    const int max_ctx = a.maxp << a.page_shift;
    const int Lc = L < 0 ? 0 : (L > max_ctx ? max_ctx : L);
    if (Lc == 0) {
      cache = nullptr;  // no token in this slot: nothing to append
    } else {
      const int t = Lc - 1;
      const unsigned raw = static_cast<unsigned>(a.bt[static_cast<int64_t>(b) * a.maxp + (t >> a.page_shift)]);
      const int64_t page = raw < static_cast<unsigned>(a.num_pages) ? raw : a.num_pages - 1;
      row = (((page << a.page_shift) + (t & ((1 << a.page_shift) - 1))) * a.hkv + g) * D;
    }
  }
  // bias and norm weights are loaded whether present or not (from the
  // partials, a valid address, when absent; dropped by a select), so that
  // no load waits behind a branch
  const float* y = a.y + (static_cast<int64_t>(b) * heads + h) * D;
  const int64_t split_stride = static_cast<int64_t>(a.batch) * heads * D;
  const uint16_t* bias_p = a.bias ? a.bias + h * D : reinterpret_cast<const uint16_t*>(a.y);
  const uint16_t* nw_p = nw ? nw : reinterpret_cast<const uint16_t*>(a.y);
  float v[E];
  uint16_t bias_h[E], wn_h[E];
#pragma unroll
  for (int j = 0; j < E; ++j) {
    // every split's partial is requested before any is added; splits past
    // the last re-read it and are dropped
    float part[kMaxRowsSplits];
#pragma unroll
    for (int s2 = 0; s2 < kMaxRowsSplits; ++s2)
      part[s2] = y[lane + 64 * j + (s2 < a.splits ? s2 : a.splits - 1) * split_stride];
    v[j] = part[0];
#pragma unroll
    for (int s2 = 1; s2 < kMaxRowsSplits; ++s2) v[j] += s2 < a.splits ? part[s2] : 0.f;
    bias_h[j] = bias_p[lane + 64 * j];
    wn_h[j] = nw_p[lane + 64 * j];
  }
#pragma unroll
  for (int j = 0; j < E; ++j) v[j] += a.bias ? bf16_to_f32(bias_h[j]) : 0.f;
  if (nw) {
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < E; ++j) ss += v[j] * v[j];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) ss += __shfl_xor(ss, off);
    const float inv = rsqrtf(ss / D + a.eps);
#pragma unroll
    for (int j = 0; j < E; ++j) v[j] = v[j] * inv * bf16_to_f32(wn_h[j]);
  }
  if ((is_q || is_k) && a.rotary_dim > 0) {
    const int r = a.rotary_dim;
    constexpr double kInvTwoPi = 0.15915494309189535;
    // the angle p * theta^(-2i/r), in turns, in fp64 (positions reach 10^5
    // and more, where an fp32 angle would already be off by ~10^-2 rad);
    // its fraction in [-1/2, 1/2] goes to the hardware sine and cosine,
    // which take turns.  The frequency is the product of the host's
    // theta^(-2 * 2^k / r) over the set bits k of i (at most seven fp64
    // products, ~1e-15 relative) instead of an fp64 exp2 and division per
    // element (0.6 us of the 256-sequence epilogue).
    auto angle = [&](int i, float& sn, float& c) __attribute__((always_inline)) {
      double freq = 1.0;
#pragma unroll
      for (int k = 0; k < 8; ++k) freq = (i >> k) & 1 ? freq * a.freq_pow2[k] : freq;
      const double turns = static_cast<double>(pos) * freq * kInvTwoPi;
      const float frac = static_cast<float>(turns - __builtin_rint(turns));
      sn = __builtin_amdgcn_sinf(frac);
      c = __builtin_amdgcn_cosf(frac);
    };
    if (E % 2 == 0 && !a.interleaved && r == D) {
      // rotation of the whole head in halves: the partner of element
      // lane + 64 j (j < E / 2) is lane + 64 (j + E / 2), in this lane, at
      // the same angle, so the pair turns in registers with one angle
      // (the same arithmetic as the exchange below)
#pragma unroll
      for (int j = 0; j < E / 2; ++j) {
        float sn, c;
        angle(lane + 64 * j, sn, c);
        const float x0 = v[j], x1 = v[j + E / 2];
        v[j] = x0 * c - x1 * sn;
        v[j + E / 2] = x1 * c + x0 * sn;
      }
    } else if (a.interleaved) {
      // interleaved pairs (e, e ^ 1): the partner is the neighbouring lane,
      // same register, fetched with a DPP swap of adjacent lanes (every
      // lane takes part, before the range test)
#pragma unroll
      for (int j = 0; j < E; ++j) {
        const float other = __builtin_bit_cast(
            float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v[j]), 0xB1, 0xF, 0xF, false));
        const int e = lane + 64 * j;
        if (e >= r) continue;
        float sn, c;
        angle(e >> 1, sn, c);
        v[j] = (e & 1) == 0 ? v[j] * c - other * sn : v[j] * c + other * sn;
      }
    } else {
#pragma unroll
      for (int j = 0; j < E; ++j) s[lane + 64 * j] = v[j];
      __syncthreads();
#pragma unroll
      for (int j = 0; j < E; ++j) {
        const int e = lane + 64 * j;
        if (e >= r) continue;
        // a partial rotation in halves: pairs (e, e + r / 2), across lanes
        const bool first = e < r / 2;
        const int i = first ? e : e - r / 2;
        const int partner = first ? e + r / 2 : e - r / 2;
        float sn, c;
        angle(i, sn, c);
        const float other = s[partner];
        v[j] = first ? v[j] * c - other * sn : v[j] * c + other * sn;
      }
    }
  }

  // outputs: q to q_out; k and v to k_out / v_out and, with a cache, to the page slot
  uint16_t* dst = nullptr;
  if (is_q) {
    dst = a.q_out + (static_cast<int64_t>(b) * a.hq + h) * D;
  } else {
    uint16_t* out = is_k ? a.k_out : a.v_out;
    if (out) dst = out + (static_cast<int64_t>(b) * a.hkv + g) * D;
  }
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const uint16_t o = f32_to_bf16(v[j]);
    if (dst) dst[lane + 64 * j] = o;
    if (cache) cache[row + lane + 64 * j] = o;
  }
}

}  // namespace

hipError_t launch_pack(const uint16_t* w, uint16_t* wp, int n, int k, hipStream_t st) {
  const int64_t chunks = static_cast<int64_t>(n) * k / 8;
  const dim3 grid(static_cast<unsigned>((chunks + kPackThreads - 1) / kPackThreads));
  hipLaunchKernelGGL(pack_kernel, grid, dim3(kPackThreads), 0, st, w, wp, n, k);
  return hipGetLastError();
}

// The instantiated forms of rows_kernel (launch_rows_any must list the same).
// Row tiles x column tiles are bounded by a wave's registers (its
// accumulators, two blocks of weights, a step's operands): 32 tiles with one
// wave per SIMD, 16 with two.
struct RowsForm {
  int rt, bt, waves, kb;
  bool wide;
};
static constexpr RowsForm kRowsForms[] = {
    {1, 1, 8, 2, false}, {2, 1, 8, 2, false}, {3, 1, 8, 2, false}, {4, 1, 8, 2, false},
    {1, 2, 8, 2, false}, {2, 2, 8, 2, false}, {3, 2, 8, 2, false}, {4, 2, 8, 2, false},
    {1, 4, 8, 4, false}, {2, 4, 8, 4, false}, {3, 4, 8, 2, false}, {4, 4, 8, 2, false},
    {6, 4, 4, 2, true},  {8, 4, 4, 1, false}, {4, 6, 4, 2, true}};

static constexpr int most_row_tiles() {
  int most = 0;
  for (const RowsForm& f : kRowsForms) most = f.rt > most ? f.rt : most;
  return most;
}

// The form, and the k splits, with the least estimated time (us).  Per round
// of workgroups the estimate joins, as the root of the squares, a
// workgroup's bytes at the rate a CU takes them in (62 KB/us: its loads
// return in order, so activations from L2 queue behind weights from memory)
// and the round's weights at 11.2 TB/s, and adds 1 us for its ramp and 0.087
// us a step for every eight tiles of matrix instructions, the steps past the
// end of k that fill up a block of weights among them (at 1024 x 1024 with
// three splits they are three quarters of 2 x 4's).  One-tile workgroups
// share a CU: their rounds run together with one ramp, their weights at 78
// KB/us.  A round is what the CUs hold, and where column groups share an XCD
// what the XCD with the most row groups holds (27 row groups x 3 x 3 splits
// are 243 workgroups, but 36 on an XCD of 32 CUs: two rounds).  The sum over
// the waves and the epilogue take 0.19 us per tile and wave, an epilogue in a
// kernel of its own 4 us and 1 us per MB of partials it reads.  Launch costs,
// the same for all, are left out.
//
// These constants are fitted to timed forms: nineteen preludes and
// twenty-two output projections, weights of 96 x 128 to 16384 x 18432, at up
// to 27 batches from 1 to 256 (13,500 forms of 834 shapes).
//
// Two rules hold where a workgroup has one column tile (up to 16 sequences):
//  * Row tiles a multiple of 128 KB apart (k a multiple of 4096) take 8% longer
//    where a workgroup reads several of them and nearly every CU has one
//    workgroup: two row tiles at 8 x 8192 -> 8192 (256 workgroups) 26.5 to 30.3
//    us by where the weights lie, 24.3 and 25.7 at k = 7936 and 8448; 3 us over
//    them with 248 workgroups, 1.7 with 224; 0 to 4% with 160 and 192, or in
//    several rounds (288 to 512).  With one row tile 25.2, 24.8 and 26.0.
//  * Four row tiles are not split along k: that was the fastest form on 4 of
//    190 shapes, and chosen by the estimate on 8 x 4096 -> 8192 (20.9 us, one
//    row tile 15.3) and 8 x 8192 -> 8192 (29.2, 25.4).
// Over output projections of 1 to 16 sequences, weights 2048 to 12288 wide
// with 2560 to 10240 rows (190 shapes, up to 16 forms each), the form chosen is
// on average 0.9% slower than the fastest and at most 8%; without the two
// rules 2.6% and 37%.
static RowsPlan search_rows(int batch, int n, int k, int num_cus, bool fusable, int max_splits) {
  const int nbt = (batch + 15) / 16;
  const int tiles = n / kTileRows;
  const int bt_small = nbt <= 2 ? nbt : 4;  // up to 64 sequences: one column group
  RowsPlan best{};
  double best_us = 0;
  for (const RowsForm& f : kRowsForms) {
    if (nbt <= 4 ? f.bt != bt_small : f.bt < 4) continue;
    const int cols = (nbt + f.bt - 1) / f.bt;
    if (nbt > 4 && cols < 2) continue;  // (the forms for one column group stop at four tiles)
    if (nbt > 4 && f.rt == 1) continue;
    const int rows = (tiles + f.rt - 1) / f.rt;
    for (int fused = 0; fused <= 1; ++fused) {
      if (fused && (!fusable || f.rt % 2)) continue;
      for (int splits = 1; splits <= (fused ? 1 : max_splits); ++splits) {
        const int64_t wgs = static_cast<int64_t>(cols > 1 ? (rows + 7) / 8 * 8 : rows) * cols * splits;
        // workgroups of one row tile and one column tile: several reside on a
        // CU and their loads overlap, so rounds run together
        const bool small = f.rt == 1 && f.bt == 1;
        // splitting only fills a round, or six of one-tile workgroups (more
        // were the fastest by at most 2.4%, and past ten were not timed)
        if (splits > 1 && wgs > (small ? 6 : 1) * static_cast<int64_t>(num_cus)) break;
        if (splits > 1 && f.bt == 1 && f.rt >= 4) break;
        const double wk = 2.0 * k / splits / 1e3;  // KB per row
        const double x_rows = batch < 16 * f.bt ? batch : 16 * f.bt;
        const bool all_cus = 8 * wgs >= 7 * static_cast<int64_t>(num_cus) && wgs <= num_cus;
        const double apart = f.bt == 1 && f.rt > 1 && k % 4096 == 0 && all_cus ? 1.08 : 1.0;
        const double in_us = (16.0 * f.rt / (small ? 78.0 : 62.0) + x_rows / 62.0) * wk * apart;
        const double w_us = 16.0 * f.rt * wk / cols / 11.2e3 * apart;  // per workgroup in the round
        const int steps = ((k + kPairK * splits - 1) / (kPairK * splits) + f.waves - 1) / f.waves;
        const double mul_us = (steps + f.kb - 1) / f.kb * f.kb * 0.0109 * f.rt * f.bt * f.waves;
        const int64_t full = wgs / num_cus, rest = wgs % num_cus;
        double us;
        if (small) {
          const double rounds = static_cast<double>(full + (rest ? 1 : 0)), w_all = static_cast<double>(wgs) * w_us;
          us = std::sqrt(rounds * in_us * rounds * in_us + w_all * w_all) + 1.0 + rounds * mul_us;
        } else {
          auto round_us = [&](double m) { return std::sqrt(in_us * in_us + m * w_us * m * w_us) + 1.0 + mul_us; };
          us = full * round_us(num_cus) + (rest ? round_us(static_cast<double>(rest)) : 0.0);
        }
        us += 0.19 * f.rt * f.bt / f.waves;
        if (!fused) us += 4.0 + 4e-6 * splits * batch * static_cast<double>(n);
        if (best.grid && us >= best_us) continue;
        best_us = us;
        best.rt = f.rt, best.bt = f.bt, best.waves = f.waves, best.kb = f.kb, best.wide = f.wide;
        best.fused = fused != 0;
        best.row_groups = rows;
        best.col_groups = cols;
        best.splits = splits;
        best.split_grid = cols > 1 ? (rows + 7) / 8 * 8 * cols : rows;
        best.grid = best.split_grid * splits;
        best.ss_parts = rows_ss_parts(f.rt, f.bt, f.waves, f.wide);
      }
    }
  }
  return best;
}

// The search takes about 1 us, a tenth of a small call; a decode loop asks for
// the same few sizes, so each thread keeps its last ones (a plan follows from
// the sizes alone).
RowsPlan plan_rows(int batch, int n, int k, int num_cus, bool fusable, int max_splits) {
  struct Entry {
    int batch, n, k, num_cus, max_splits;
    bool fusable;
    RowsPlan plan;
  };
  constexpr unsigned kEntries = 16;
  static thread_local Entry kept[kEntries];
  Entry& e = kept[(static_cast<unsigned>(batch) * 7u + static_cast<unsigned>(n) / 16u + static_cast<unsigned>(k) / 32u * 3u +
                   (fusable ? 5u : 0u)) % kEntries];
  if (e.batch != batch || e.n != n || e.k != k || e.num_cus != num_cus || e.max_splits != max_splits ||
      e.fusable != fusable || !e.plan.grid)
    e = Entry{batch, n, k, num_cus, max_splits, fusable, search_rows(batch, n, k, num_cus, fusable, max_splits)};
  return e.plan;
}

// By search_rows: up to 16 sequences any number of splits; above, splits only
// fill one round of workgroups.
int64_t rows_most_floats(int batch, int n, int num_cus, int max_splits) {
  constexpr int most = most_row_tiles();
  const int rows = (n / kTileRows + most - 1) / most;
  const int round = num_cus / rows < 1 ? 1 : num_cus / rows;
  const int64_t few = static_cast<int64_t>(batch < 16 ? batch : 16) * max_splits;
  const int64_t many = static_cast<int64_t>(batch) * (round < max_splits ? round : max_splits);
  return (few > many ? few : many) * n;
}

namespace {

template <int RT, int BT, int W, int DX, int KB, bool kWide, bool kShared, class Epilogue>
hipError_t launch_rows_as(const RowsArgs& a, const RowsPlan& p, const Epilogue& e, hipStream_t st) {
  constexpr int lds = rows_lds_bytes(RT, BT, W, DX);
  auto* fn = &rows_kernel<RT, BT, W, DX, KB, kWide, kShared, Epilogue>;
  if constexpr (lds > 64 * 1024) {
    // the dynamic-LDS limit is raised once per device (bit = device ordinal)
    static std::atomic<uint64_t> attr_set{0};
    int dev = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return err;
    const uint64_t bit = dev < 64 ? uint64_t{1} << dev : 0;
    if (!bit || !(attr_set.load() & bit)) {
      err = hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
      if (err != hipSuccess) return err;
      attr_set.fetch_or(bit);
    }
  }
  hipLaunchKernelGGL(fn, dim3(p.grid), dim3(W * 64), lds, st, a, e);
  return hipGetLastError();
}

template <class Epilogue>
hipError_t launch_rows_any(RowsArgs a, const RowsPlan& p, const Epilogue& e, hipStream_t st) {
  a.row_groups = p.row_groups;
  a.col_groups = p.col_groups;
  a.splits = p.splits;
  a.split_grid = p.split_grid;
  constexpr bool kPairs = std::is_same<Epilogue, PreludeArgs>::value;
#define PDA_ROWS(RT, BT, W, DX, KB, WD, SH) \
  if (p.rt == RT && p.bt == BT && p.waves == W && p.wide == WD && p.kb == KB && (p.col_groups > 1) == SH) \
    return launch_rows_as<RT, BT, W, DX, KB, WD, SH, Epilogue>(a, p, e, st);
  if constexpr (!kPairs) {
    PDA_ROWS(1, 1, 8, 2, 2, false, false)
    PDA_ROWS(3, 1, 8, 2, 2, false, false)
    PDA_ROWS(1, 2, 8, 2, 2, false, false)
    PDA_ROWS(3, 2, 8, 2, 2, false, false)
    PDA_ROWS(1, 4, 8, 2, 4, false, false)
    PDA_ROWS(3, 4, 8, 2, 2, false, false)
    PDA_ROWS(3, 4, 8, 2, 2, false, true)
  }
  PDA_ROWS(2, 1, 8, 2, 2, false, false)
  PDA_ROWS(4, 1, 8, 2, 2, false, false)
  PDA_ROWS(2, 2, 8, 2, 2, false, false)
  PDA_ROWS(4, 2, 8, 2, 2, false, false)
  PDA_ROWS(2, 4, 8, 2, 4, false, false)
  PDA_ROWS(4, 4, 8, 2, 2, false, false)
  PDA_ROWS(6, 4, 4, 2, 2, true, false)
  PDA_ROWS(8, 4, 4, 1, 1, false, false)
  PDA_ROWS(2, 4, 8, 2, 4, false, true)
  PDA_ROWS(4, 4, 8, 2, 2, false, true)
  PDA_ROWS(6, 4, 4, 2, 2, true, true)
  PDA_ROWS(4, 6, 4, 2, 2, true, true)
  PDA_ROWS(8, 4, 4, 1, 1, false, true)
#undef PDA_ROWS
  return hipErrorInvalidValue;
}

template <int D>
hipError_t launch_prelude(const PreludeArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((prelude_epilogue<D>), dim3(a.batch * (a.hq + 2 * a.hkv)), dim3(64), 0, st, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_rows(const RowsArgs& a, const RowsPlan& p, hipStream_t st) {
  return launch_rows_any(a, p, NoEpilogue{}, st);
}
hipError_t launch_rows_prelude(const RowsArgs& a, const RowsPlan& p, const PreludeArgs& e, hipStream_t st) {
  return launch_rows_any(a, p, e, st);
}
hipError_t launch_rows_residual(const RowsArgs& a, const RowsPlan& p, const OProjArgs& o, hipStream_t st) {
  return launch_rows_any(a, p, o, st);
}

hipError_t launch_prelude_epilogue(const PreludeArgs& a, hipStream_t st) {
  if (a.d == 64) return launch_prelude<64>(a, st);
  if (a.d == 128) return launch_prelude<128>(a, st);
  return launch_prelude<256>(a, st);
}

hipError_t launch_oproj_sum(const OProjArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(oproj_sum_kernel, dim3(a.batch), dim3(kSumThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_oproj_norm(const OProjArgs& a, hipStream_t st) {
  const int chunks = (a.hidden + kNormFeatures - 1) / kNormFeatures;
  hipLaunchKernelGGL(oproj_norm_kernel, dim3(a.batch * chunks), dim3(kNormThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace pda
