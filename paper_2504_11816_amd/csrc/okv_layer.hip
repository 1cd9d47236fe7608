// Linear layers and layer norm of a decoder layer in the decode stage, for gfx950.
//
// out[m][n] = sum_k x[m][k] W[n][k] for a batch of m rows (paper §IV-D: the
// 8 h1^2 + 4 h1 h2 flops per token of the four projections and the feed-forward block).
// With a decode batch's few rows every weight is read once and used `m` times: the product is bound by
// streaming W from HBM, so the kernel is built like the attention kernel -- long runs of
// 16-byte-per-lane loads kept many deep in flight -- with the matrix cores doing the
// arithmetic on the side (one fp16 instruction per KiB of weights and 16 rows of x: a few
// percent of the time the loads take).
//
//   * weights are stored pre-arranged (okv_pack_linear_weight) so that one load instruction
//     brings a wavefront the 1 KiB it feeds to one 16x16x32 matrix-core instruction per 16 rows:
//     16 output features x 32 inputs, lane l holding feature l % 16, inputs 8 (l / 16) .. + 7;
//   * beyond a few rows, the rows of x must NOT be fetched per lane in the layout the matrix core
//     wants: such a gather touches 16 half cache lines per instruction, every wavefront needs
//     its own, and the time grows with the rows although x sits in L2 (16384 x 4096, weights
//     from HBM: 25.4 us at 4 rows, 26.6 at 8, 34.3 at 16).  So in the fast kernel a workgroup of
//     4 (or 3) wavefronts takes 64 (48) output features, one 16-feature tile per wavefront, over
//     one stretch of the input dimension, and one more wavefront stages the rows of x for that
//     stretch chunk by chunk in LDS, from where the others read their operands.  The staging
//     wavefront fetches whole rows of a chunk (512 contiguous bytes each), keeps three chunks
//     ahead of the others and meets them at one barrier per 256 inputs; it is a wavefront of
//     its own because the vector memory counter retires loads in order: a wavefront that waited
//     for staged rows would also wait for the weight pieces it issued before them.  16384 x
//     4096 from HBM: 28.4 us at 32 rows, 31.0 at 64, 44.6 at 128; with the staging switched off
//     (timing only) 27.6 and 28.5, of which about 5 us do not depend on the size of the matrix;
//   * the input dimension is cut across workgroups so that the launch has one per compute
//     unit (longer-lived workgroups measured faster than more of them); each writes its fp32
//     share of the tile and a small second kernel adds the shares in a fixed order and applies
//     the epilogue (bias, ReLU, residual, rounding to fp16, scatter into up to three output
//     tensors).  A hand-over inside the kernel (last workgroup adds up) needs device-wide
//     fences, which on this GPU write back and invalidate the L2 caches: 75 us instead of 11.
//     Where three tiles per workgroup fill the compute units without a cut (12288 features on
//     256 units) the workgroups have three streaming wavefronts and there is no second kernel;
//   * up to 8 rows, up to 16 where a model of both is in its favour, and some shapes the fast kernel does
//     not take (input dimension not a multiple of 256), run the simple kernel: a workgroup per 16
//     features, its wavefronts split the inputs and add up through LDS, x by gather;
//   * with hundreds of rows the matrix cores and what feeds them bound the product: linear_tile_kernel, and
//     linear_wide_kernel for the largest tiles.
#include "okv_kernels.h"
#include "okv_lanes.h"
#include "okv_layer.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace okv {

namespace {

typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

#ifndef OKV_LIN_DEPTH
#define OKV_LIN_DEPTH 8
#endif
// Up to this many rows the simple kernel runs unless the staged one is clearly faster, and up to a fragment of rows where its model
// says so (see few_rows_simple).
#ifndef OKV_LIN_SIMPLE_ROWS
#define OKV_LIN_SIMPLE_ROWS 8
#endif
#ifndef OKV_LIN_WAVES
#define OKV_LIN_WAVES 4
#endif
constexpr int kLinWaves = OKV_LIN_WAVES;

template <int MF>
constexpr int lin_depth() {
  return MF <= 2 ? OKV_LIN_DEPTH : MF <= 4 ? OKV_LIN_DEPTH / 2 : OKV_LIN_DEPTH / 4;   // pieces in flight: bounded by the registers x needs beside them
}

struct LinearArgs {
  const uint4 *x;          // [m][n_in] fp16, as 16-byte pieces
  const uint4 *w;          // packed weights
  // (the next twelve, what Sink takes, in the order in which they come by eight and four words: a load of three words is
  // one of four, and the wavefront then waits for it before it uses the fourth register again)
  _Float16 *out[3];
  const _Float16 *residual;
  float *shares;                    // several cuts or a layer norm to follow: [splits][m][n_out] fp32
  int32_t n_out, to_shares;         // the kernel writes shares
  int32_t seg0_cols, seg_cols;      // width of the first output tensor, of the others (multiples of 16)
  int32_t relu, m;
  const _Float16 *bias;
  int32_t n_in, n_kb, n_tiles, splits;   // blocks of 32 inputs, 16-feature tiles, cuts of the input dimension
  const _Float16 *ln_gamma, *ln_beta;
  _Float16 *ln_out;                 // layer norm of the result, or NULL
  float ln_eps;
};

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// Where a product's results go and what is added to them: the part of the arguments that the end of a kernel needs.
//
// The end of a product kernel is a chain of waits that nothing hides: every workgroup is there at the same time and has
// nothing else to do.  So these arguments are read while the first weights are on their way (`arrive`, without which the
// compiler reads them where they are used, after the last barrier), the output tensor is chosen by comparisons (an indexed
// pointer becomes a load), and the bias and the residual of all of a thread's results are asked for together before the first is
// stored (a load behind a store waits for that store).  us before -> now: 1024 rows x 4096 x 4096 with a residual 50.3 -> 43.3, 192
// x 16384 x 4096 46.0 -> 44.5, 4 x 4096 x 4096 7.5 -> 7.0; the products of 8 layers 1056 wide at 64 rows 311 -> 281, 768 wide at 512
// rows 310 -> 283; the kernels that add the shares up, 1024 rows x 4096 in four cuts 15.9 -> 13.5.
struct Sink {
  uint64_t out0, out1, out2, residual, shares;
  int32_t n_out, to_shares, seg0_cols, seg_cols, relu, m;

  __device__ __forceinline__ explicit Sink(const LinearArgs &a)
      : out0((uint64_t)a.out[0]), out1((uint64_t)a.out[1]), out2((uint64_t)a.out[2]), residual((uint64_t)a.residual), shares((uint64_t)a.shares),
        n_out(a.n_out), to_shares(a.to_shares), seg0_cols(a.seg0_cols), seg_cols(a.seg_cols), relu(a.relu), m(a.m) {}
  __device__ __forceinline__ void arrive() const {
    asm volatile("" ::"s"(out0), "s"(out1), "s"(out2), "s"(residual), "s"(seg0_cols), "s"(seg_cols), "s"(relu), "s"(m));
  }
  __device__ __forceinline__ void shares_arrive() const { asm volatile("" ::"s"(shares), "s"(n_out), "s"(to_shares)); }
  // Feature n of row mrow lands in the output tensor at `out`, at byte `at` (the tensors are [m][their width]).
  __device__ __forceinline__ void place(int mrow, int n, uint64_t &out, uint64_t &at) const {
    const int r = n - seg0_cols;
    const bool first = r < 0, third = r >= seg_cols;
    out = first ? out0 : third ? out2 : out1;
    at = 2 * ((uint64_t)mrow * (uint32_t)(first ? seg0_cols : seg_cols) + (uint32_t)(first ? n : third ? r - seg_cols : r));
  }
};

template <class T>
__device__ __forceinline__ T load_at(uint64_t p) {
  return *(const __attribute__((address_space(1))) T *)p;
}
template <class T>
__device__ __forceinline__ void store_at(uint64_t p, T v) {
  *(__attribute__((address_space(1))) T *)p = v;
}

// Epilogue for eight neighbouring features n .. n + 7 of row mrow: bias, ReLU, residual, one rounding, one 16-byte store.
// (Feature counts and segment widths are multiples of 16, so a group of eight never straddles a segment.)  The residual is
// asked for by residual_eight, before.
__device__ __forceinline__ u32x4_t residual_eight(const Sink &sink, int mrow, int n) {
  if (!sink.residual) return u32x4_t{0u, 0u, 0u, 0u};
  uint64_t out, at;
  sink.place(mrow, n, out, at);
  return load_at<u32x4_t>(sink.residual + at);
}
__device__ __forceinline__ void store_eight(const Sink &sink, int mrow, int n, const floatx4 t0, const floatx4 t1, const half8 bias, const half8 residual) {
  const float v[8] = {t0[0], t0[1], t0[2], t0[3], t1[0], t1[1], t1[2], t1[3]};
  half8 yo;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    float y = v[e] + (float)bias[e];
    if (sink.relu) y = fmaxf(y, 0.f);
    y += (float)residual[e];
    yo[e] = (_Float16)y;
  }
  uint64_t out, at;
  sink.place(mrow, n, out, at);
  store_at(out + at, __builtin_bit_cast(u32x4_t, yo));
}

__device__ __forceinline__ floatx4 mfma16(const uint2 a, const uint2 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(half4, a), __builtin_bit_cast(half4, b), c, 0, 0, 0);
}

// 16 x 16 result tile += [16 rows][32 inputs] . [32 inputs][16 features]; a lane's 16 bytes of either operand are
// inputs 8 (lane / 16) .. + 7 of row (feature) lane % 16
__device__ __forceinline__ floatx4 mfma32(const uint4 a, const uint4 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
}

// 16 bytes of a weight matrix.  NT: a load that asks the caches not to keep the line.  A step reads every weight once
// and a model with matrices of this size does not fit the memory-side cache (256 MiB), so what is kept is gone before it
// is wanted again: from HBM, 16384 x 4096 takes 25.1 -> 22.6 us at 4 rows (5.9 TB/s), 27.0 -> 25.0 at 32, 33.8 -> 32.2 at 96;
// 4096 x 16384 24.5 -> 22.4, 28.9 -> 26.4, 35.9 -> 34.6.  (The same matrix again and again, which stays cached: 20.9 -> 21.1, 23.0 ->
// 23.8.)  Not for matrices below these sizes, which a small model may keep cached (2048 x 2048 at 4 rows: 3.8 us kept, 4.6
// not), nor beyond 128 rows, where row tiles share a weight or the time follows x (4096 x 16384 at 192 rows: 48.9 -> 50.9;
// 33 MB matrices lose from 64 rows on: 4096 x 4096 at 128 rows 15.9 -> 17.9).
template <bool NT>
__device__ __forceinline__ uint4 load_weight(const uint4 *p) {
  if constexpr (NT) return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p)));
  else return *p;
}
constexpr int64_t kStreamSimpleBytes = 32 << 20, kStreamStagedBytes = 64 << 20;

template <int MF, bool NT>
__global__ __launch_bounds__(kLinWaves * 64) void linear_kernel(const uint4 *w, const uint4 *x, const _Float16 *bias,
                                                                   const int32_t n_kb, const int32_t n_in, const int32_t m,
                                                                   const LinearArgs a) {
  // (leading parameters: in scalar registers when the wavefront starts, see linear_lds_kernel)
  constexpr int D = lin_depth<MF>();
  __shared__ floatx4 part[kLinWaves][MF][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);      // uniform: the loops below are scalar loops
  const int ntile = blockIdx.x;
  const int kb0 = (int)((int64_t)wave * n_kb / kLinWaves), kb1 = (int)((int64_t)(wave + 1) * n_kb / kLinWaves);
  const int nk = kb1 - kb0;
  const char *const wp = reinterpret_cast<const char *>(w + ((size_t)ntile * n_kb + kb0) * 64);
  // this lane's piece of x for k-block kb and row fragment f: row 16 f + lane % 16, inputs 32 kb + 8 (lane / 16) .. + 7
  const int row = lane & 15, kq = lane >> 4;
  const char *const xp = reinterpret_cast<const char *>(x + (size_t)kb0 * 4);
  // Rows past the batch read row 0 instead: a row of x only ever reaches the same row of the
  // result, and those rows are not stored.
  uint32_t xoff[MF];
#pragma unroll
  for (int f = 0; f < MF; ++f) xoff[f] = (uint32_t)(f * 16 + row < m ? f * 16 + row : 0) * (uint32_t)n_in * 2 + (uint32_t)kq * 16;
  floatx4 acc[MF];
#pragma unroll
  for (int f = 0; f < MF; ++f) acc[f] = floatx4{0.f, 0.f, 0.f, 0.f};

  uint4 wbuf[D], xbuf[D][MF];
  // Every wavefront walks its blocks from a different starting point (and wraps around).  All
  // ranges have the same length and all wavefronts advance at the same pace, so without the
  // shift every wavefront of the launch would be reading addresses that are equal modulo the
  // range length at any moment, i.e. from a few of the memory channels at a time (the same shift
  // in the staged kernel below is worth up to 10 % on weights that come from HBM).
  const int rot = nk > 0 ? (int)(((unsigned)ntile * 5u + (unsigned)wave * 11u) % (unsigned)nk) : 0;
  // Past the last block the last one is asked for again and not used (of x a single line, by every lane): every load is
  // unconditional, so the waits in front of the blocks are exact.  With the loads of the last round behind conditions each wait had
  // to cover the case that none of them was made, and waited for those that were: a round trip to HBM at the end of every walk that
  // is no multiple of D blocks.  us before -> now, weights from HBM: 1 row x 2560 x 2560 6.1 -> 4.2 (3.1 TB/s), 8 rows x 2560 x 2560 6.7 ->
  // 5.0, 8 x 4224 x 1056 4.9 -> 4.3, 28 x 1056 x 4224 12.2 -> 11.9 (12.8 where lanes ask for their own lines of x again), 4 x 5120 x 13824
  // 30.7 -> 29.5; whole rounds gain by the loads in fetch_rest, 8 x 4096 x 4096 7.4 -> 7.0.
  auto load = [&](int slot, int k) {                           // k: position in this wavefront's walk
    int kk = min(k, nk - 1) + rot;
    kk = kk >= nk ? kk - nk : kk;                              // block index relative to kb0
    wbuf[slot] = load_weight<NT>(reinterpret_cast<const uint4 *>(wp + (size_t)(uint32_t)kk * 1024 + lane * 16));
    const uint32_t own = k < nk ? ~0u : 0u;
#pragma unroll
    for (int f = 0; f < MF; ++f) xbuf[slot][f] = *reinterpret_cast<const uint4 *>(xp + (size_t)(uint32_t)kk * 64 + (xoff[f] & own));
  };
  auto use = [&](int slot) {
    const uint4 w = wbuf[slot];
#pragma unroll
    for (int f = 0; f < MF; ++f) {
      const uint4 x = xbuf[slot][f];
      acc[f] = mfma16(make_uint2(x.x, x.y), make_uint2(w.x, w.y), acc[f]);
      acc[f] = mfma16(make_uint2(x.z, x.w), make_uint2(w.z, w.w), acc[f]);
    }
  };
  // This thread's results are feature threadIdx.x % 16 of rows threadIdx.x / 16 + 16 f: what is added to them, asked for
  // behind the first weights.
  const Sink sink(a);
  _Float16 add_bias, add_residual[MF];
  const int out_row = (int)threadIdx.x >> 4, out_feature = ntile * 16 + ((int)threadIdx.x & 15);
  uint64_t out, at;
  auto fetch_rest = [&]() {
    // (without them, weights: a branch around a load waits for it, and for all loads before it, where the paths meet)
    sink.arrive();
    add_bias = load_at<_Float16>((uint64_t)(bias ? bias + out_feature : reinterpret_cast<const _Float16 *>(w)));
#pragma unroll
    for (int f = 0; f < MF; ++f) {
      sink.place(min(16 * f + out_row, m - 1), out_feature, out, at);
      add_residual[f] = load_at<_Float16>(sink.residual ? sink.residual + at : (uint64_t)w);
    }
  };
  if (nk > 0) {
#pragma unroll
    for (int i = 0; i < D; ++i) {
      load(i, i);
      __builtin_amdgcn_sched_barrier(0);    // oldest first: the loop waits for the loads in this order
    }
  }
  fetch_rest();
  __builtin_amdgcn_sched_barrier(0);
  int k = 0;
  for (; k + D < nk; k += D) {
#pragma unroll
    for (int i = 0; i < D; ++i) {
      use(i);
      __builtin_amdgcn_sched_barrier(0);
      load(i, k + D + i);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int i = 0; i < D; ++i)
    if (k + i < nk) use(i);

  // add the wavefronts' shares and finish: result element (row 16 f + 4 (lane / 16) + r, feature lane % 16)
  // sits in acc[f][r] of that lane
#pragma unroll
  for (int f = 0; f < MF; ++f) part[wave][f][lane] = acc[f];
  __syncthreads();
  static_assert(kLinWaves * 64 == 256, "a row fragment of results, 16 rows x 16 features, per pass of the workgroup");
#pragma unroll
  for (int f = 0; f < MF; ++f) {
    const int mrow = 16 * f + out_row;
    if (mrow >= m) break;
    const int src_lane = (threadIdx.x & 15) + 16 * (out_row >> 2), r = out_row & 3;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < kLinWaves; ++w) v += part[w][f][src_lane][r];
    if (bias) v += (float)add_bias;
    if (sink.relu) v = fmaxf(v, 0.f);
    if (sink.residual) v += (float)add_residual[f];
    sink.place(mrow, out_feature, out, at);
    store_at(out + at, (_Float16)v);
  }
}

// Fast path: NW wavefronts x 16 features, x staged in LDS by one or two more wavefronts, input
// dimension cut across workgroups.  NW = 4 or 3 and the number of cuts: whatever staged_plan's model of the
// launch prefers (3 and no cut for 12288 features on 256 compute units, which saves the kernel that adds up
// the shares).
// 32-input blocks per staged chunk of x: 8 (256 inputs), 4 from 112 rows on.  A chunk takes chunk x MF KiB of LDS
// and there are lead + 1 of them: 128 KiB at most up to 128 rows (4 x 32 at 64 and at 128 rows), 144 at 96 rows
// (3 x 48) and from 129 to 192 rows (9 to 12 fragments of 16 rows: 3 x 36 .. 3 x 48).
constexpr int lin_chunk(int mf) { return mf <= 6 ? 8 : 4; }
// How many chunks of x the staging wavefronts are ahead of the others (one LDS buffer more than that).  Bounded by
// LDS and by the counter of loads in flight, which stops at 63: the wait for a chunk leaves the loads of the
// lead - 1 chunks after it outstanding.
constexpr int lin_lead(int mf) { return mf == 5 || mf == 6 || mf > 8 ? 2 : 3; }
// Staging wavefronts per workgroup: two from 64 rows on, each taking every other instruction of a chunk.  (At 128
// rows the rows of x that the workgroups fetch from L2 are twice the bytes of the weights, and that traffic is
// what the time then follows: 16384 x 4096 takes 40 us, 31 with the staging switched off, whether one wavefront
// stages or two, whatever the lead; the second wavefront is worth 1 us.)
constexpr int lin_stagers(int mf) { return mf >= 4 ? 2 : 1; }
// chunks of weights a streaming wavefront has in flight: 8 KiB either way
constexpr int lin_weight_lead(int mf) { return 8 / lin_chunk(mf) > 1 ? 8 / lin_chunk(mf) : 1; }
// s_waitcnt operand that waits until at most n vector memory loads are outstanding and for nothing else
constexpr int vmcnt_only(int n) { return (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }

// waves_per_eu: a workgroup has one or two wavefronts per SIMD and a compute unit holds one workgroup (LDS), so
// up to 128 registers cost nothing (256 with more than 8 row fragments, whose accumulators and operand registers
// need them: a SIMD holds two of the workgroup's six wavefronts at most); without the hint the compiler aimed
// at the occupancy the launch bounds allow and capped the kernel at 64.
template <int MF, int NW, bool NT>
__global__ __launch_bounds__((NW + lin_stagers(MF)) * 64) __attribute__((amdgpu_waves_per_eu(1, MF > 8 ? 2 : 4))) void linear_lds_kernel(
    const uint4 *w, const uint4 *x, const _Float16 *bias, const int32_t n_kb, const int32_t splits, const int32_t n_in, const int32_t m,
    const int32_t n_tiles, const LinearArgs a) {
  // (the parameters in front of `a` are what the first loads need: the build has the leading kernel arguments
  // arrive in scalar registers with the wavefront, so the weight stream starts without a round trip to the
  // argument segment)
  constexpr int NS = lin_stagers(MF);
  constexpr int kFastThreads = (NW + NS) * 64, kTileCols = NW * 16;      // kTileCols: output features of a workgroup
  constexpr int C = lin_chunk(MF), LEAD = lin_lead(MF), NBUF = LEAD + 1, PER = C * MF, MINE = PER / NS;
  static_assert(PER % NS == 0 && (LEAD - 1) * MINE <= 63, "the wait for a staged chunk must fit the load counter");
  // A chunk of x, 16 MF rows of LPR 16-byte pieces (LPR x 8 inputs), as PER staging instructions' worth of 64
  // pieces each.  An operand read takes, for block i of the chunk, piece 4 i + q of row 16 f + rr in lane 16 q + rr.
  // The LDS serves a 16-byte-per-lane read in groups of 16 lanes that are not consecutive (lanes 0-3, 12-15, 20-23,
  // 24-27 and so on: measured, a layout that only spread 16 consecutive lanes over the banks had every read take
  // twice its cycles), so the bank (16-byte unit modulo 16) of a piece is (rr + 2 i + q / 2) mod 16: it does not
  // depend on the low bit of q, and within any such group all 16 rows rr occur once.  The two pieces that share
  // a bank (q even and odd) and the rows of an instruction take the unit's upper bits:
  //   unit = 64 * instruction + 16 * (2 * (rr & 1) + (q & 1)) + bank,
  //   instruction = 8 f + rr / 2 (8 blocks a chunk: rows 2 t and 2 t + 1, 512 bytes each), or
  //                 4 f + (rr % 8) / 2 (4 blocks: rows 2 t, 2 t + 1, 2 t + 8, 2 t + 9, 256 bytes each; of rr and
  //                 rr + 8 exactly one has (bank - rr) mod 16 below 8, which is where 2 i + q / 2 lives then).
  // After the last chunk the same memory holds the fp32 tile [16 MF rows][kTileCols features] for the epilogue.
  static_assert(C == 8 || C == 4, "the LDS layout of x is laid out for chunks of 8 or 4 blocks");
  constexpr int LPR = C * 4, IPF = C;                  // pieces per row; staging instructions per 16 rows
  __shared__ uint4 xs[NBUF][PER][64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = blockIdx.x, cut = blockIdx.y;
  const int nk = n_kb / splits, kb0 = cut * nk, n_chunks = nk / C;
  floatx4 acc[MF];
#pragma unroll
  for (int f = 0; f < MF; ++f) acc[f] = floatx4{0.f, 0.f, 0.f, 0.f};
  // Every workgroup walks its chunks from a different starting point (and wraps around): all stretches have
  // the same length and all workgroups advance at the same pace, so without the shift the whole launch would
  // be reading addresses that are equal modulo the stretch length at any moment, i.e. from a few of the
  // memory channels at a time (16384 x 4096 at 32 rows, weights from HBM: 31.7 us without, 28.8 with).
  const int rot = (int)(((unsigned)group * 5u + (unsigned)cut * 3u) % (unsigned)n_chunks);
  auto rotc = [&](int c) { int cc = c + rot; return cc >= n_chunks ? cc - n_chunks : cc; };
  const Sink sink(a);
  _Float16 add_bias;                                     // of this lane's feature (without a bias: anything)

  if (wave >= NW) {
    // The staging wavefront.  Its loads have a counter of their own, so waiting for them never
    // holds up the weight stream of the others.  A load instruction writes straight into LDS, 16 bytes per
    // lane, lane l landing in unit l of the instruction's 1 KiB; every lane fetches the piece that belongs
    // there.  An instruction brings whole rows of the chunk (2 x 512 or 4 x 256 contiguous bytes).  (Fetched in
    // the order the matrix core reads -- 16 rows x 64 bytes per instruction -- the same bytes took twice as
    // many half-used cache lines.)
    const int row_pieces = n_in >> 3;
    const int bank = lane & 15, ql = (lane >> 4) & 1, odd = lane >> 5;
    const int first = wave - NW;                   // this staging wavefront takes instructions first, first + NS, ...
    const uint4 *xg[MINE];
#pragma unroll
    for (int k = 0; k < MINE; ++k) {
      const int j = first + NS * k;
      const int f = j / IPF, t = j % IPF;
      int rr = 2 * t + odd;
      const int d = (bank - rr) & 15;
      if (C == 4 && d >= 8) rr += 8;
      const int v = C == 4 ? (d & 7) : d;                            // 2 i + q / 2
      const int piece = 4 * (v >> 1) + 2 * (v & 1) + ql;
      const int row = 16 * f + rr;                 // rows past the batch read row 0: they only reach result rows that are not stored
      xg[k] = x + (size_t)(row < m ? row : 0) * row_pieces + (size_t)kb0 * 4 + piece;
    }
    auto stage = [&](int chunk, int buf) {
#pragma unroll
      for (int k = 0; k < MINE; ++k)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(xg[k] + (size_t)chunk * LPR),
                                         (__attribute__((address_space(3))) void *)&xs[buf][first + NS * k][0], 16, 0, 0);
    };
    // LEAD chunks ahead of the others, so that a chunk has LEAD of their chunk times to arrive, not one (with one:
    // 3 us of 30 at 32 rows and 16 of 44 at 64 rows went into waiting for it, 16384 x 4096).  Before barrier c
    // chunk c must have landed: the loads of the chunks issued after it, LEAD - 1 of them except at the end, may
    // still be on their way.
    auto landed = [&](int c) {
      if (n_chunks - 1 - c >= LEAD - 1) __builtin_amdgcn_s_waitcnt(vmcnt_only((LEAD - 1) * MINE));
      else __builtin_amdgcn_s_waitcnt(vmcnt_only(0));
    };
#pragma unroll
    for (int j = 0; j < LEAD; ++j)
      if (j < n_chunks) stage(rotc(j), j);
    sink.arrive();
    sink.shares_arrive();
    landed(0);
    __builtin_amdgcn_s_barrier();
    int buf = LEAD;
    for (int c = 0; c < n_chunks; ++c) {
      // the buffer of chunk c - 1: the others finished with it before the barrier this wavefront just passed
      if (c + LEAD < n_chunks) stage(rotc(c + LEAD), buf);
      buf = buf + 1 == NBUF ? 0 : buf + 1;
      if (c + 1 < n_chunks) landed(c + 1);
      __builtin_amdgcn_s_barrier();
    }
  } else {
    const int ntile = group * NW + wave;
    // a wavefront past the last tile streams tile 0 (valid memory) and never stores
    const uint4 *wp = w + ((size_t)(ntile < n_tiles ? ntile : 0) * n_kb + kb0) * 64 + lane;
    // where this lane's operand pieces sit in a chunk (see the layout above): rr = lane % 16, q = lane / 16
    const int rr = lane & 15, q = lane >> 4;
    const int xbase = 64 * (C == 8 ? rr >> 1 : (rr & 7) >> 1) + 16 * (2 * (rr & 1) + (q & 1));
    const int xrq = rr + (q >> 1);
    auto xat = [&](int buf, int i, int f) -> uint4 {
      return (&xs[buf][0][0])[64 * IPF * f + xbase + ((xrq + 2 * i) & 15)];
    };
    // Weights are fetched WD chunks ahead: with more than 64 rows a chunk is only 4 blocks (LDS), and 4 KiB in
    // flight, each refill waiting behind eight matrix instructions, did not keep the stream going (16384 x 4096
    // at 128 rows: 43 us; without the staging and the LDS reads still 36).
    constexpr int WD = lin_weight_lead(MF);
    uint4 wbuf[WD][C];
    auto ahead = [&](int c) { return rotc(c < n_chunks ? c : n_chunks - 1); };   // past the end: the last chunk again
#pragma unroll
    for (int u = 0; u < WD; ++u)
#pragma unroll
      for (int i = 0; i < C; ++i) {                          // oldest first: the loop waits for them in this order
        wbuf[u][i] = load_weight<NT>(wp + ((size_t)ahead(u) * C + i) * 64);
        __builtin_amdgcn_sched_barrier(0);
      }
    add_bias = bias ? bias[(ntile < n_tiles ? ntile : 0) * 16 + rr] : *reinterpret_cast<const _Float16 *>(w);
    sink.arrive();
    sink.shares_arrive();
    __syncthreads();
    int buf = 0;
    for (int c0 = 0; c0 < n_chunks; c0 += WD) {
#pragma unroll
      for (int u = 0; u < WD; ++u) {
        const int c = c0 + u;                    // the host only cuts the inputs into stretches of a multiple of WD chunks
        // the chunk WD after this one (past the end the last chunk is fetched once more instead of branching:
        // loads in this loop stay unconditional, so the waits stay exact)
        const int cn = ahead(c + WD);
        // the rows of x for a block are asked from LDS before the matrix instructions of the block before it are
        // issued (two sets of registers), so that they arrive while those run and while this wavefront waits for
        // the block's weights
        uint4 xr[2][MF];
#pragma unroll
        for (int f = 0; f < MF; ++f) xr[0][f] = xat(buf, 0, f);
#pragma unroll
        for (int i = 0; i < C; ++i) {
          if (i + 1 < C) {
#pragma unroll
            for (int f = 0; f < MF; ++f) xr[(i + 1) & 1][f] = xat(buf, i + 1, f);
          }
          const uint4 w = wbuf[u][i];
#pragma unroll
          for (int f = 0; f < MF; ++f) acc[f] = mfma32(xr[i & 1][f], w, acc[f]);
          __builtin_amdgcn_sched_barrier(0);
          wbuf[u][i] = load_weight<NT>(wp + ((size_t)cn * C + i) * 64);
          __builtin_amdgcn_sched_barrier(0);
        }
        buf = buf + 1 == NBUF ? 0 : buf + 1;
        __syncthreads();
      }
    }
  }

  // this workgroup's share of the tile [16 MF][kTileCols] in LDS (all reads of xs are behind the barrier above), with the bias
  // where it is the whole sum: result element (row 16 f + 4 (lane / 16) + r, feature 16 wave + lane % 16) sits in acc[f][r]
  float *tile = reinterpret_cast<float *>(&xs[0][0][0]);
  if (wave < NW) {
    const float add = sink.to_shares || !bias ? 0.f : (float)add_bias;
#pragma unroll
    for (int f = 0; f < MF; ++f)
#pragma unroll
      for (int r = 0; r < 4; ++r) tile[(f * 16 + 4 * (lane >> 4) + r) * kTileCols + wave * 16 + (lane & 15)] = acc[f][r] + add;
  }
  // eight neighbouring features of a row per thread (feature counts and segment widths are multiples of 16, so
  // a group of eight never straddles a segment and every access below is one aligned 16-byte piece)
  const int n0 = group * kTileCols;
  constexpr int VPR = kTileCols / 8;
  if (sink.to_shares) {                              // this cut's share; a second kernel adds them up
    __syncthreads();
    const uint64_t mine = sink.shares + (uint64_t)cut * m * sink.n_out * 4;
    for (int o = tid; o < 2 * m * VPR; o += kFastThreads) {          // neighbouring threads, neighbouring 16 bytes
      const int mrow = o / (2 * VPR), n = n0 + 4 * (o % (2 * VPR));
      if (n < sink.n_out) store_at(mine + ((uint64_t)mrow * sink.n_out + n) * 4, *reinterpret_cast<const floatx4 *>(tile + 4 * o));
    }
    return;
  }
  constexpr int kPasses = (16 * MF * VPR + kFastThreads - 1) / kFastThreads;
  u32x4_t residual[kPasses];
#pragma unroll
  for (int k = 0; k < kPasses; ++k) {
    const int o = tid + k * kFastThreads, n = n0 + 8 * (o % VPR);
    residual[k] = residual_eight(sink, min(o / VPR, m - 1), n < sink.n_out ? n : 0);
  }
  __syncthreads();
  const half8 no_bias = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int k = 0; k < kPasses; ++k) {
    const int o = tid + k * kFastThreads, mrow = o / VPR, n = n0 + 8 * (o % VPR);
    if (mrow >= m || n >= sink.n_out) continue;
    const floatx4 *t = reinterpret_cast<const floatx4 *>(tile + mrow * kTileCols + 8 * (o % VPR));
    store_eight(sink, mrow, n, t[0], t[1], no_bias, __builtin_bit_cast(half8, residual[k]));
  }
}

// ---- many rows: tiles of rows x features -------------------------------------------------------
//
// With a few hundred rows and more the product is no longer a stream of weights with some arithmetic beside it:
// the staged kernel above has every streaming wavefront read every row of x from LDS for 16 features, and takes
// the weights once per 192 rows.  Here a workgroup owns a tile of 16 FM WM rows x 16 FN WN features and its WM x WN
// wavefronts a 16 FM x 16 FN piece each, so an operand read from LDS serves FN products and a weight FM.
//
//   * x goes through LDS, 64 inputs at a time (a stage), fetched by the load that writes LDS directly (16 bytes per
//     lane, no registers), whole 128-byte lines of 8 rows an instruction; the weights go from memory straight into
//     the registers of the wavefronts that use them: packed, one load is one operand of the matrix instruction;
//   * the direct loads are written as assembly because the compiler, which cannot tell the stage being
//     written from the one being read, waits for all of them in front of every LDS read otherwise.  It does not
//     count them either: its waits for the weights are at worst longer than they need to be;
//   * loads retire in order, so a stage of x needs no more lead than the weights have: WD stages of both are in
//     flight (WD + 1 LDS buffers).
//
// Measured (weights from HBM, warm clocks): 1024 rows x 4096 x 4096 42 us, 512 x 16384 x 4096 68, 192 x 16384 x 4096 41 (96 x
// 128).  What bounds the small tiles: a compute unit takes in 58 KB/us once weights from HBM are among its loads, whatever the
// mix, the depth or the wavefronts (a probe of nothing but loads: 54 from HBM alone, 130 to 150 from its L2 alone; the L1 answers
// in order).  Two or three teams of wavefronts along the inputs, or the next half stage read from LDS early, change nothing.
//
// LDS layout of a stage: row r has its 8 pieces of 16 bytes in units 8 r .. 8 r + 7, piece p in unit 8 r + (p ^ (r / 2) % 8).
// An instruction of 64 lanes brings eight whole rows, eight lanes a line, and an operand read (lane 16 q + rr takes piece
// 4 i + q of row rr) meets every bank once in each of the groups of 16 lanes that the LDS serves together (see
// linear_lds_kernel).  (With the lanes of a quad on two rows x alone came in at 65 KB/us a unit; now 115.  384 rows of a
// 4096-wide layer 226 -> 219 us, 1024 rows of a 2048-wide one 88 -> 86.)
template <int FM, int FN, int WM, int WN, int WD>
struct TileShape {
  static constexpr int kThreads = WM * WN * 64, kRows = 16 * FM * WM, kCols = 16 * FN * WN;
  static constexpr int kBuffers = WD + 1, kStageBytes = kRows * 128;
  static constexpr int kLoads = 2 * FM / WN;             // staging instructions of a wavefront per stage
  static constexpr int kOutStride = 16 * FN + 4;         // floats between two rows of a wavefront's results in LDS
  static constexpr int kOutBytes = WM * WN * 32 * kOutStride * 4;
  static constexpr int kLds = kBuffers * kStageBytes > kOutBytes ? kBuffers * kStageBytes : kOutBytes;
  static_assert(2 * FM % WN == 0 && FM % 2 == 0, "staging instructions and result chunks come out even");
  static_assert(kLds <= 160 * 1024, "LDS of a compute unit");
  static_assert(WD * 2 * FN + (WD - 1) * kLoads <= 63, "the wait for a stage must fit the load counter");
};

// One 16-byte-per-lane load from `base` + off straight into LDS: lane l's bytes land at lds + 16 l.  The place goes through m0,
// which an asm statement cannot be said to change (the compiler reserves it): it is left as it was found.
__device__ __forceinline__ void load_to_lds(const void *base, uint32_t off, uint32_t lds) {
  uint32_t found;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b32 m0, %0"
               : "=&s"(found)
               : "s"(lds), "v"(off), "s"(base)
               : "memory");
}

template <int FM, int FN, int WM, int WN, int WD>
__global__ __launch_bounds__(WM * WN * 64) __attribute__((amdgpu_waves_per_eu(1, 2))) void linear_tile_kernel(
    const uint4 *w, const uint4 *x, const _Float16 *bias, const int32_t n_kb, const int32_t splits, const int32_t n_in, const int32_t m,
    const int32_t n_tiles, const int32_t m_tiles, const int32_t n_groups, const LinearArgs a) {
  using S = TileShape<FM, FN, WM, WN, WD>;
  __shared__ __attribute__((aligned(1024))) char lds[S::kLds];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  // Workgroups are dealt to the 8 XCDs in rotation; tiles that share weights (all row tiles of a feature group)
  // and neighbouring groups are put on the same XCD, whose L2 then reads them from memory once.
  const int total = m_tiles * n_groups * splits, xcd = blockIdx.x & 7, per = total >> 3, rem = total & 7;
  const int tile = xcd * per + min(xcd, rem) + (blockIdx.x >> 3);
  const int mt = tile % m_tiles, group = (tile / m_tiles) % n_groups, cut = tile / (m_tiles * n_groups);
  // This workgroup's stages of 64 inputs.  Where the inputs are an odd number of blocks of 32, the very last stage is
  // half full: it is the last one walked by the cut that has it (no shift of the walk then).
  const int all_stages = (n_kb + 1) >> 1, stage0 = (int)((unsigned)(cut * all_stages) / (unsigned)splits);
  const int n_stages = (int)((unsigned)((cut + 1) * all_stages) / (unsigned)splits) - stage0;
  const int half_stage = n_kb & 1 ? all_stages - 1 : -1;
  const int full_stages = n_stages - (stage0 + n_stages - 1 == half_stage ? 1 : 0);
  const int rot = m_tiles == 1 && half_stage < 0 ? (int)(((unsigned)group * 5u + (unsigned)cut * 3u) % (unsigned)n_stages) : 0;
  auto stage_at = [&](int s) {                           // position in this workgroup's walk -> stage; past the end: the last again
    const int t = min(s, n_stages - 1) + rot;
    return stage0 + (t >= n_stages ? t - n_stages : t);
  };

  // staging: this wavefront's instructions are kLoads * wave + j, eight rows each
  const int row0 = mt * S::kRows, last_row = m - 1 - row0;
  const uint32_t row_bytes = (uint32_t)n_in * 2;
  uint32_t xoff[S::kLoads];
  uint32_t second[S::kLoads];
#pragma unroll
  for (int j = 0; j < S::kLoads; ++j) {
    const int r = (wave * S::kLoads + j) * 8 + (lane >> 3), piece = (lane & 7) ^ ((r >> 1) & 7);
    xoff[j] = (uint32_t)min(r, last_row) * row_bytes + (uint32_t)piece * 16;   // rows past the batch: the last again
    second[j] = piece & 4 ? 64 : 0;                      // this lane fetches of the stage's second 32 inputs
  }
  const char *xbase = reinterpret_cast<const char *>(x) + (size_t)row0 * row_bytes;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds);
  auto stage_x = [&](int s, int buf) {
    const int st = stage_at(s);
    const char *src = xbase + (size_t)st * 128;
    const uint32_t dst = lds0 + (uint32_t)buf * S::kStageBytes + (uint32_t)(wave * S::kLoads) * 1024;
#pragma unroll
    for (int j = 0; j < S::kLoads; ++j)                  // (a half-full stage: its first half twice, the second is never used)
      load_to_lds(src, xoff[j] - (st == half_stage ? second[j] : 0), dst + j * 1024);
  };
  // weights: FN runs of 1 KiB per 32 inputs (a tile past the last one streams the last one and is never stored)
  const int tile0 = (group * WN + wn) * FN;
  const uint4 *wp[FN];
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) wp[fn] = w + (size_t)min(tile0 + fn, n_tiles - 1) * n_kb * 64;
  uint4 wbuf[WD][2][FN];
  auto load_w = [&](uint4 (&dst)[FN], int s, int i) {
    const size_t at = (size_t)min(2 * stage_at(s) + i, n_kb - 1) * 64;
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) dst[fn] = wp[fn][at + lane];
  };
  const int rr = lane & 15, q = lane >> 4;
  int xunit[2];                                          // where this lane's piece of 32 inputs i of fragment 0 sits in a stage
#pragma unroll
  for (int i = 0; i < 2; ++i) xunit[i] = 8 * rr + ((4 * i + q) ^ ((rr >> 1) & 7));

  floatx4 acc[FM][FN];
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = floatx4{0.f, 0.f, 0.f, 0.f};

  auto read_half = [&](uint4 (&dst)[FM], int buf, int i) {
    const uint4 *xs = reinterpret_cast<const uint4 *>(lds + buf * S::kStageBytes) + wm * FM * 128 + xunit[i];
#pragma unroll
    for (int fm = 0; fm < FM; ++fm) dst[fm] = xs[fm * 128];
  };
  auto multiply = [&](const uint4 (&wf)[FN], const uint4 (&xf)[FM]) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = mfma32(wf[fn], xf[fm], acc[fm][fn]);
    __builtin_amdgcn_s_setprio(0);
  };
#pragma unroll
  for (int u = 0; u < WD; ++u) {
    stage_x(u, u);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 2; ++i) load_w(wbuf[u][i], u, i);
    __builtin_amdgcn_sched_barrier(0);
  }
  const Sink sink(a);
  sink.arrive();
  sink.shares_arrive();
  // a stage of x has landed once no more loads are outstanding than were issued after it
  constexpr int kInFlight = WD * 2 * FN + (WD - 1) * S::kLoads;
  __builtin_amdgcn_s_waitcnt(vmcnt_only(kInFlight));
  __syncthreads();
  int buf = 0, fill = WD, s0 = 0;
  for (; s0 + WD <= full_stages; s0 += WD) {
#pragma unroll
    for (int u = 0; u < WD; ++u) {
      stage_x(s0 + u + WD, fill);                        // into the buffer that the stage before this one was read from
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        uint4 xf[FM];
        read_half(xf, buf, i);
        multiply(wbuf[u][i], xf);
        __builtin_amdgcn_sched_barrier(0);
        load_w(wbuf[u][i], s0 + u + WD, i);
        __builtin_amdgcn_sched_barrier(0);
      }
      buf = buf + 1 == S::kBuffers ? 0 : buf + 1;
      fill = fill + 1 == S::kBuffers ? 0 : fill + 1;
      __builtin_amdgcn_s_waitcnt(vmcnt_only(kInFlight));   // the next stage has landed
      __syncthreads();
    }
  }
  // What does not fill a round of WD stages (at most WD of them, a half-full one last) is on its way or here already.  (A
  // way out in the middle of a round instead cost 15 % of the whole walk: the compiler's waits in front of the weights
  // then cover every path that may have led there.)
  __builtin_amdgcn_s_waitcnt(vmcnt_only(0));             // nothing may still be on its way into LDS afterwards
  __syncthreads();
#pragma unroll
  for (int u = 0; u < WD; ++u)
    if (s0 + u < n_stages) {
      uint4 xf[FM];
      read_half(xf, buf, 0);
      multiply(wbuf[u][0], xf);
      if (stage0 + s0 + u != half_stage) {
        read_half(xf, buf, 1);
        multiply(wbuf[u][1], xf);
      }
      buf = buf + 1 == S::kBuffers ? 0 : buf + 1;
    }
  __syncthreads();

  // Results: acc[fm][fn][r] is row 16 fm + lane % 16, feature 16 fn + 4 (lane / 16) + r of the wavefront's piece.  They pass
  // through LDS that belongs to the wavefront, 32 rows at a time, and leave as 16-byte pieces of whole rows.
  float *mine = reinterpret_cast<float *>(lds) + wave * 32 * S::kOutStride;
  const int out_row = row0 + wm * FM * 16, out_feature = tile0 * 16;
  auto turn = [&](int c) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
        *reinterpret_cast<floatx4 *>(mine + (16 * h + rr) * S::kOutStride + 16 * fn + 4 * q) = acc[2 * c + h][fn];
  };
  auto piece = [&](int c, int k, int &mrow, int &n, floatx4 &t0, floatx4 &t1) {
    const int o = k * 64 + lane, r = o / (2 * FN), pc = o % (2 * FN);
    mrow = out_row + 32 * c + r, n = out_feature + pc * 8;
    const floatx4 *t = reinterpret_cast<const floatx4 *>(mine + r * S::kOutStride + pc * 8);
    t0 = t[0], t1 = t[1];
    return mrow < m && n < sink.n_out;
  };
  int mrow, n;
  floatx4 t0, t1;
  if (sink.to_shares) {
#pragma unroll
    for (int c = 0; c < FM / 2; ++c) {
      turn(c);
#pragma unroll
      for (int k = 0; k < 2 * FN; ++k) {                 // neighbouring lanes, neighbouring 16 bytes
        const int o = k * 64 + lane, r = o / (4 * FN), pc = o % (4 * FN);
        const int mrow = out_row + 32 * c + r, n = out_feature + pc * 4;
        const floatx4 t = *reinterpret_cast<const floatx4 *>(mine + r * S::kOutStride + pc * 4);
        if (mrow < m && n < sink.n_out) store_at(sink.shares + (((uint64_t)cut * m + mrow) * sink.n_out + n) * 4, t);
      }
    }
    return;
  }
  u32x4_t add_bias[FN] = {}, residual[FM / 2][FN] = {};
#pragma unroll
  for (int k = 0; k < FN; ++k) {
    const int o = k * 64 + lane, r = o / (2 * FN), at = out_feature + o % (2 * FN) * 8, n = at < sink.n_out ? at : 0;
    if (bias) add_bias[k] = load_at<u32x4_t>((uint64_t)(bias + n));
#pragma unroll
    for (int c = 0; c < FM / 2; ++c) residual[c][k] = residual_eight(sink, min(out_row + 32 * c + r, m - 1), n);
  }
  turn(0);
#pragma unroll
  for (int k = 0; k < FN; ++k) {                         // one wait for all of them, here: behind a store it would be one for the store
    asm volatile("" : "+v"(add_bias[k]));
#pragma unroll
    for (int c = 0; c < FM / 2; ++c) asm volatile("" : "+v"(residual[c][k]));
  }
#pragma unroll
  for (int c = 0; c < FM / 2; ++c) {
    if (c > 0) turn(c);
#pragma unroll
    for (int k = 0; k < FN; ++k)
      if (piece(c, k, mrow, n, t0, t1))
        store_eight(sink, mrow, n, t0, t1, __builtin_bit_cast(half8, add_bias[k]), __builtin_bit_cast(half8, residual[c][k]));
  }
}

// ---- the largest tiles: weights through LDS as well ----------------------------------------------
//
// With two rows of wavefronts the kernel above loads every weight twice, which with 256 x 256 or 192 x 128 tiles is a third to two
// fifths of all a compute unit takes in.  Here the weights go through LDS like x, half a stage (32 inputs, one operand of the
// matrix instruction, 1 KiB a piece) at a time, and every byte comes in once.  Nothing in the walk loads into registers, so the
// waits written here are the only ones and are exact.  A wavefront reads FM / 2 fragments of x ahead of its matrix instructions
// and the next half stage's weights under them; one barrier per half stage, in its middle: behind it the next half stage is in
// LDS and the buffers of the one before are free, so the reads ahead go on across half stages.
//
// What bounds it: 256 x 256 the matrix cores, busy in 66 % of a compute unit's cycles (1024 rows x 16384 x 4096 1.2 PFLOP/s; with nothing
// loaded 1.45), LDS in 27 %, of which conflicts are 2 %; 192 x 128 what a compute unit takes in (matrix cores 41 to 48 %, LDS 30 to
// 34 %).  us, the kernel above with the same tiles -> this one: 256 x 256, 1024 x 16384 x 4096 119 -> 114.5 and 4096 x 16384 in four cuts
// 136 -> 129; 192 x 128, 384 x 12288 x 4096 54 -> 50 (96 x 128 above: 59), 192 x 4096 x 16384 in eight cuts, with the launch that
// adds the shares, 42 (96 x 128 above, four cuts: 45).  Not for the other forms: 128 x 256 is 4 % slower so, 128 x 128 9 %, the smallest 10 %,
// whose walk is the latency of a half stage (two barriers a stage); 256 x 192, whose pieces do not come out even, 2 %.  Four wavefronts of
// 128 x 128, whole stages of weights, nontemporal weights and more stages in flight change nothing.
template <int FM, int FN, int WM, int WN, int NX>
struct WideShape {
  static constexpr int kWaves = WM * WN, kThreads = kWaves * 64, kRows = 16 * FM * WM, kCols = 16 * FN * WN;
  static constexpr int kXBuffers = NX, kWBuffers = 2 * NX - 2;        // stages of x, half stages of weights
  static constexpr int kXBytes = kRows * 128, kWBytes = kCols * 64;
  static constexpr int kAhead = FM / 2;                  // fragments of x a wavefront reads ahead; the barrier is as far into a half stage
  // loads of a wavefront: LX per stage of x, LW of the half stage's FN WN pieces of weights
  static constexpr int LX = kRows / 8 / kWaves, LW = FN * WN / kWaves;
  // How many loads may be outstanding for the next half stage to have landed: those issued after its last one, which are
  // kWBuffers - 3 half stages of weights and the stages of x among them (one more in front of an odd half)
  static constexpr int outstanding(int odd) { return (kWBuffers - 3) * LW + (kWBuffers - (odd ? 2 : 4)) / 2 * LX; }
  static constexpr int first() { return (kWBuffers - 2) * LW + (kXBuffers - 2) * LX; }        // and in front of the first half stage
  static constexpr int kOutStride = 16 * FN + 4;         // floats between two rows of a wavefront's results in LDS
  static constexpr int kOutBytes = kWaves * 32 * kOutStride * 4;
  static constexpr int kStageBytes = kXBuffers * kXBytes + kWBuffers * kWBytes;
  static constexpr int kLds = kStageBytes > kOutBytes ? kStageBytes : kOutBytes;
  static_assert(FM % 2 == 0 && NX >= 3 && kRows % (8 * kWaves) == 0 && FN * WN % kWaves == 0, "fragments and staging instructions come out even");
  static_assert(kLds <= 160 * 1024, "LDS of a compute unit");
  static_assert(outstanding(1) <= 63 && first() <= 63, "the wait for a half stage must fit the load counter");
};

// A barrier that does not wait for this wavefront's reads from LDS (__syncthreads does): what they read is not overwritten behind it.
__device__ __forceinline__ void barrier_leaving_reads() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <int FM, int FN, int WM, int WN, int NX>
__global__ __launch_bounds__(WM * WN * 64) __attribute__((amdgpu_waves_per_eu(1, 2))) void linear_wide_kernel(
    const uint4 *w, const uint4 *x, const _Float16 *bias, const int32_t n_kb, const int32_t splits, const int32_t n_in, const int32_t m,
    const int32_t n_tiles, const int32_t m_tiles, const int32_t n_groups, const LinearArgs a) {
  using S = WideShape<FM, FN, WM, WN, NX>;
  constexpr int kXB = S::kXBuffers, kWB = S::kWBuffers, kAhead = S::kAhead;
  __shared__ __attribute__((aligned(1024))) char lds[S::kLds];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  // Workgroups are dealt to the 8 XCDs in rotation; tiles that share weights (all row tiles of a feature group)
  // and neighbouring groups are put on the same XCD, whose L2 then reads them from memory once.
  const int total = m_tiles * n_groups * splits, xcd = blockIdx.x & 7, per = total >> 3, rem = total & 7;
  const int tile = xcd * per + min(xcd, rem) + (blockIdx.x >> 3);
  const int mt = tile % m_tiles, group = (tile / m_tiles) % n_groups, cut = tile / (m_tiles * n_groups);
  // This workgroup's stages of 64 inputs.  Where the inputs are an odd number of blocks of 32, the very last stage is
  // half full: it is the last one walked by the cut that has it (no shift of the walk then).
  const int all_stages = (n_kb + 1) >> 1, stage0 = (int)((unsigned)(cut * all_stages) / (unsigned)splits);
  const int n_stages = (int)((unsigned)((cut + 1) * all_stages) / (unsigned)splits) - stage0;
  const int half_stage = n_kb & 1 ? all_stages - 1 : -1;
  const int full_stages = n_stages - (stage0 + n_stages - 1 == half_stage ? 1 : 0);
  const int rot = m_tiles == 1 && half_stage < 0 ? (int)(((unsigned)group * 5u + (unsigned)cut * 3u) % (unsigned)n_stages) : 0;
  auto stage_at = [&](int s) {                           // position in this workgroup's walk -> stage; past the end: the last again
    const int t = min(s, n_stages - 1) + rot;
    return stage0 + (t >= n_stages ? t - n_stages : t);
  };
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds);
  constexpr uint32_t kW0 = kXB * S::kXBytes;             // where the weights begin

  // x: this wavefront's instructions are LX * wave + j, eight rows each
  const int row0 = mt * S::kRows, last_row = m - 1 - row0;
  const uint32_t row_bytes = (uint32_t)n_in * 2;
  uint32_t xoff[S::LX], second[S::LX];
#pragma unroll
  for (int j = 0; j < S::LX; ++j) {
    const int r = (wave * S::LX + j) * 8 + (lane >> 3), piece = (lane & 7) ^ ((r >> 1) & 7);
    xoff[j] = (uint32_t)min(r, last_row) * row_bytes + (uint32_t)piece * 16;   // rows past the batch: the last again
    second[j] = piece & 4 ? 64 : 0;                      // this lane fetches of the stage's second 32 inputs
  }
  const char *xbase = reinterpret_cast<const char *>(x) + (size_t)row0 * row_bytes;
  auto stage_x = [&](int s, int buf) {
    const int st = stage_at(s);
    const char *src = xbase + (size_t)st * 128;
    const uint32_t dst = lds0 + (uint32_t)buf * S::kXBytes + (uint32_t)(wave * S::LX) * 1024;
#pragma unroll
    for (int j = 0; j < S::LX; ++j)                      // (a half-full stage: its first half twice, the second is never used)
      load_to_lds(src, xoff[j] - (st == half_stage ? second[j] : 0), dst + j * 1024);
  };
  // weights: instructions wave, wave + kWaves, ... of a half stage, a tile each (past the last one: the last again, never stored)
  const int tile0 = group * (FN * WN);
  uint32_t woff[S::LW];
#pragma unroll
  for (int j = 0; j < S::LW; ++j)
    woff[j] = (uint32_t)min(wave + j * S::kWaves, n_tiles - 1 - tile0) * (uint32_t)n_kb * 1024 + lane * 16;
  const char *wbase = reinterpret_cast<const char *>(w) + (size_t)tile0 * n_kb * 1024;
  auto stage_w = [&](int h, int buf) {
    const char *src = wbase + (size_t)min(2 * stage_at(h >> 1) + (h & 1), n_kb - 1) * 1024;
    const uint32_t dst = lds0 + kW0 + (uint32_t)buf * S::kWBytes + (uint32_t)wave * 1024;
#pragma unroll
    for (int j = 0; j < S::LW; ++j) load_to_lds(src, woff[j], dst + j * S::kWaves * 1024);
  };
  auto landed = [&](auto odd) {                          // the next half stage: this wavefront's share of it
    __builtin_amdgcn_s_waitcnt(vmcnt_only(S::outstanding(decltype(odd)::value)));
  };

  const int rr = lane & 15, q = lane >> 4;
  uint32_t xunit[2];                                     // where this lane's piece of 32 inputs i of fragment 0 sits in a stage
#pragma unroll
  for (int i = 0; i < 2; ++i) xunit[i] = 16 * (wm * FM * 128 + 8 * rr + ((4 * i + q) ^ ((rr >> 1) & 7)));
  const uint32_t wunit = kW0 + (uint32_t)(wn * FN) * 1024 + lane * 16;
  auto read_x = [&](int buf, int j) -> uint4 {           // fragment j % FM of half j / FM
    return *reinterpret_cast<const uint4 *>(lds + (uint32_t)buf * S::kXBytes + xunit[j / FM] + (j % FM) * 2048);
  };
  auto read_w = [&](int buf, int fn) -> uint4 {
    return *reinterpret_cast<const uint4 *>(lds + (uint32_t)buf * S::kWBytes + wunit + fn * 1024);
  };
  floatx4 acc[FM][FN];
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = floatx4{0.f, 0.f, 0.f, 0.f};
  uint4 xf[kAhead], wf[2][FN];                           // fragments of x read ahead (fragment j in j % kAhead), weights of two halves

#pragma unroll
  for (int h = 0; h < kWB - 1; ++h) {                    // (in the order the walk goes on in)
    if (h == 0) stage_x(0, 0);
    if (h % 2 == 1) stage_x((h + 1) / 2, (h + 1) / 2);
    stage_w(h, h);
  }
  const Sink sink(a);
  sink.arrive();
  sink.shares_arrive();
  __builtin_amdgcn_s_waitcnt(vmcnt_only(S::first()));
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kAhead; ++j) xf[j] = read_x(0, j);
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) wf[0][fn] = read_w(0, fn);
  int xb = 0, xfill = kXB - 1, wnext = 1, wfill = kWB - 1;     // buffers: this stage, to fill; the next half's weights, to fill
  for (int s = 0; s < full_stages; ++s) {
    const int xn = xb + 1 == kXB ? 0 : xb + 1;
    auto half = [&](auto i_) {
      constexpr int i = decltype(i_)::value;
#pragma unroll
      for (int j0 = 0; j0 < FM; ++j0) {
        if (j0 == kAhead) {
          __builtin_amdgcn_sched_barrier(0);
          landed(i_);
          barrier_leaving_reads();
          __builtin_amdgcn_sched_barrier(0);
          if (i == 0) {
            stage_x(s + kXB - 1, xfill);
            xfill = xfill + 1 == kXB ? 0 : xfill + 1;
          }
          stage_w(2 * s + i + kWB - 1, wfill);
          wfill = wfill + 1 == kWB ? 0 : wfill + 1;
          __builtin_amdgcn_sched_barrier(0);
        }
        const int j = i * FM + j0;
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) acc[j0][fn] = mfma32(wf[i][fn], xf[j % kAhead], acc[j0][fn]);
        xf[j % kAhead] = j + kAhead < 2 * FM ? read_x(xb, j + kAhead) : read_x(xn, j + kAhead - 2 * FM);
#pragma unroll
        for (int fn = 0; fn < FN; ++fn)
          if (j0 >= kAhead && fn * (FM - kAhead) / FN == j0 - kAhead) wf[i ^ 1][fn] = read_w(wnext, fn);
        __builtin_amdgcn_sched_barrier(0);
      }
      wnext = wnext + 1 == kWB ? 0 : wnext + 1;
    };
    half(std::integral_constant<int, 0>{});
    half(std::integral_constant<int, 1>{});
    xb = xn;
  }
  if (full_stages < n_stages) {                          // a half-full last stage: in LDS already, as its first fragments are in registers
#pragma unroll
    for (int j = 0; j < FM; ++j) {
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) acc[j][fn] = mfma32(wf[0][fn], xf[j % kAhead], acc[j][fn]);
      if (j + kAhead < FM) xf[j % kAhead] = read_x(xb, j + kAhead);
    }
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_only(0));             // nothing may still be on its way into LDS
  __syncthreads();

  // Results: as in linear_tile_kernel.  (The same lines a second time: as one function of both kernels the compiler orders them
  // differently after inlining, 500 rows x 5120 x 1056 11.1 -> 11.3 us, 384 x 12288 x 4096 50.1 -> 51.4.)
  float *mine = reinterpret_cast<float *>(lds) + wave * 32 * S::kOutStride;
  const int out_row = row0 + wm * FM * 16, out_feature = (tile0 + wn * FN) * 16;
  auto turn = [&](int c) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
        *reinterpret_cast<floatx4 *>(mine + (16 * h + rr) * S::kOutStride + 16 * fn + 4 * q) = acc[2 * c + h][fn];
  };
  auto piece = [&](int c, int k, int &mrow, int &n, floatx4 &t0, floatx4 &t1) {
    const int o = k * 64 + lane, r = o / (2 * FN), pc = o % (2 * FN);
    mrow = out_row + 32 * c + r, n = out_feature + pc * 8;
    const floatx4 *t = reinterpret_cast<const floatx4 *>(mine + r * S::kOutStride + pc * 8);
    t0 = t[0], t1 = t[1];
    return mrow < m && n < sink.n_out;
  };
  int mrow, n;
  floatx4 t0, t1;
  if (sink.to_shares) {
#pragma unroll
    for (int c = 0; c < FM / 2; ++c) {
      turn(c);
#pragma unroll
      for (int k = 0; k < 2 * FN; ++k) {                 // neighbouring lanes, neighbouring 16 bytes
        const int o = k * 64 + lane, r = o / (4 * FN), pc = o % (4 * FN);
        const int mrow = out_row + 32 * c + r, n = out_feature + pc * 4;
        const floatx4 t = *reinterpret_cast<const floatx4 *>(mine + r * S::kOutStride + pc * 4);
        if (mrow < m && n < sink.n_out) store_at(sink.shares + (((uint64_t)cut * m + mrow) * sink.n_out + n) * 4, t);
      }
    }
    return;
  }
  u32x4_t add_bias[FN] = {}, residual[FM / 2][FN] = {};
#pragma unroll
  for (int k = 0; k < FN; ++k) {
    const int o = k * 64 + lane, r = o / (2 * FN), at = out_feature + o % (2 * FN) * 8, n = at < sink.n_out ? at : 0;
    if (bias) add_bias[k] = load_at<u32x4_t>((uint64_t)(bias + n));
#pragma unroll
    for (int c = 0; c < FM / 2; ++c) residual[c][k] = residual_eight(sink, min(out_row + 32 * c + r, m - 1), n);
  }
  turn(0);
#pragma unroll
  for (int k = 0; k < FN; ++k) {                         // one wait for all of them, here: behind a store it would be one for the store
    asm volatile("" : "+v"(add_bias[k]));
#pragma unroll
    for (int c = 0; c < FM / 2; ++c) asm volatile("" : "+v"(residual[c][k]));
  }
#pragma unroll
  for (int c = 0; c < FM / 2; ++c) {
    if (c > 0) turn(c);
#pragma unroll
    for (int k = 0; k < FN; ++k)
      if (piece(c, k, mrow, n, t0, t1))
        store_eight(sink, mrow, n, t0, t1, __builtin_bit_cast(half8, add_bias[k]), __builtin_bit_cast(half8, residual[c][k]));
  }
}

// Adds the cuts' shares in a fixed order and applies the epilogue; one thread per output element, a
// workgroup per 256 consecutive features of a row.  A launch of its own rather than a hand-over inside
// the product kernel: a workgroup that reads what other workgroups wrote needs device-wide fences, and on
// this GPU those write back and invalidate the L2 caches (measured: 75 us instead of 11 for a 32 MiB matrix).
__global__ __launch_bounds__(256) void reduce_epilogue_kernel(const float *shares, const _Float16 *bias, const _Float16 *residual,
                                                                 const int32_t n_out, const int32_t splits, const int32_t m,
                                                                 const int32_t seg0_cols, const int32_t seg_cols, const LinearArgs a) {
  // four neighbouring features per thread; the shares are fetched four cuts at a time with loads that do not
  // depend on one another (past the last cut the last is read again and left out of the sum: not added with
  // weight 0, which would make a NaN of an infinity), so a thread waits for one round trip, not for one per cut
  const int n = (blockIdx.x * 256 + threadIdx.x) * 4, mrow = blockIdx.y;
  if (n >= n_out) return;
  const Sink sink(a);
  floatx4 v = {0.f, 0.f, 0.f, 0.f};
  half4 add_bias, add_residual;
  const int r = n - seg0_cols;                           // a segment is a multiple of 16 features wide
  const bool first = r < 0, third = r >= seg_cols;
  const uint64_t at = 2 * ((uint64_t)mrow * (uint32_t)(first ? seg0_cols : seg_cols) + (uint32_t)(first ? n : third ? r - seg_cols : r));
  for (int s2 = 0; s2 < splits; s2 += 4) {
    floatx4 part[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int sj = s2 + j < splits ? s2 + j : splits - 1;
      part[j] = *reinterpret_cast<const floatx4 *>(shares + ((size_t)sj * m + mrow) * n_out + n);
    }
    if (s2 == 0) {                                       // behind the first shares, not behind their sum
      __builtin_amdgcn_sched_barrier(0);
      // (without them, whatever else can be read: a branch around a load waits for it where the paths meet)
      add_bias = load_at<half4>(bias ? (uint64_t)(bias + n) : (uint64_t)shares);
      add_residual = load_at<half4>(residual ? (uint64_t)residual + at : (uint64_t)shares);
      sink.arrive();
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool in = s2 + j < splits;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += in ? part[j][e] : 0.f;
    }
  }
  half4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float y = v[e];
    if (bias) y += (float)add_bias[e];
    if (sink.relu) y = fmaxf(y, 0.f);
    if (residual) y += (float)add_residual[e];
    o[e] = (_Float16)y;
  }
  store_at((first ? sink.out0 : third ? sink.out2 : sink.out1) + at, o);
}

// dst piece (block (nt, kb), lane) = src[16 nt + lane % 16][32 kb + 8 (lane / 16) .. + 7]
__global__ __launch_bounds__(256) void pack_weight_kernel(uint4 *dst, const uint4 *src, int32_t n_out, int32_t n_in) {
  const int64_t total = (int64_t)n_out * n_in / 8;
  const int n_kb = n_in / 32, row_pieces = n_in / 8;
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < total; p += (int64_t)gridDim.x * blockDim.x) {
    const int lane = (int)(p & 63);
    const int64_t blk = p >> 6;
    const int kb = (int)(blk % n_kb), nt = (int)(blk / n_kb);
    dst[p] = src[(size_t)(nt * 16 + (lane & 15)) * row_pieces + kb * 4 + (lane >> 4)];
  }
}

// One workgroup per row; every thread keeps its (one or two) 16-byte pieces in registers, so the row
// is read once: mean, then variance around it, then the output.  As many threads as the row has pieces, up
// to 1024: with so few rows the kernel takes as long as its chain of dependent loads, and a thread with one
// piece has one round of them.
constexpr int kLnMaxThreads = 1024, kLnMaxPieces = 2;
constexpr int kLnMaxWidth = kLnMaxThreads * kLnMaxPieces * 8;
inline int ln_threads(int h) { return std::min(kLnMaxThreads, ((h >> 3) + 63) / 64 * 64); }

// The sum of a value per thread, in every thread: over the lanes of a wavefront, then wavefront by wavefront through `scratch` (a place per
// wavefront, read by nobody else since the last barrier).
__device__ __forceinline__ float block_sum(float v, float4 (&scratch)[kLnMaxThreads / 256]) {
  const int waves = (int)(blockDim.x >> 6);
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) reinterpret_cast<float *>(scratch)[threadIdx.x >> 6] = v;
  __syncthreads();
  float t = 0.f;
#pragma unroll
  for (int w = 0; w < kLnMaxThreads / 64; w += 4) {
    if (w >= waves) break;
    const float4 s = scratch[w / 4];                       // (past the last wavefront: whatever is there, left out)
    t += s.x;
    t += w + 1 < waves ? s.y : 0.f;
    t += w + 2 < waves ? s.z : 0.f;
    t += w + 3 < waves ? s.w : 0.f;
  }
  return t;
}

// Mean and 1 / sqrt(variance + eps) of a row of h numbers of which a thread holds PPT pieces of eight (piece threadIdx.x + i blockDim.x): the
// mean of the whole row, then the squares around it.  The kernels are a chain of waits, and the two sums are most of it.  us with lane
// shuffles and two barriers a sum -> now, with the product in front: 32 rows x 4096 x 4096 12.5 -> 12.1, 32 x 5120 x 5120 16.3 -> 15.8, 100 x
// 10240 x 2560 23.4 -> 23.2; the norm alone, 1024 rows of 16384 14.6 -> 13.8, 4096 of 4096 13.3 -> 12.4.  The sums' order is the same bit for bit:
// squares around every wavefront's own mean, joined in one trip through LDS, took 0.2 us less (11.9, 15.5, 22.9; alone 12.7 and 12.2) and
// changed the roundings of a few results in 10000, in whole decoder layers as much as half of a result's error.
template <int PPT>
__device__ __forceinline__ void row_stats(const float (&v)[PPT][8], const int h, const float eps, float4 (&scratch)[2][kLnMaxThreads / 256], float &mean,
                                          float &rstd) {
  const int pieces = h >> 3;
  float s = 0.f, q = 0.f;
#pragma unroll
  for (int i = 0; i < PPT; ++i)
    if ((int)(threadIdx.x + i * blockDim.x) < pieces) {
#pragma unroll
      for (int e = 0; e < 8; ++e) s += v[i][e];
    }
  mean = block_sum(s, scratch[0]) / (float)h;
#pragma unroll
  for (int i = 0; i < PPT; ++i)
    if ((int)(threadIdx.x + i * blockDim.x) < pieces) {
#pragma unroll
      for (int e = 0; e < 8; ++e) q += (v[i][e] - mean) * (v[i][e] - mean);
    }
  rstd = 1.0f / sqrtf(block_sum(q, scratch[1]) / (float)h + eps);
}

template <int PPT>
__global__ __launch_bounds__(kLnMaxThreads) void layernorm_kernel(const uint4 *x, const uint4 *gamma, const uint4 *beta, uint4 *out,
                                                                int32_t h, float eps) {
  __shared__ float4 scratch[2][kLnMaxThreads / 256];
  const int pieces = h >> 3;
  const uint4 *xr = x + (size_t)blockIdx.x * pieces;
  float v[PPT][8];
#pragma unroll
  for (int i = 0; i < PPT; ++i) {
    const int p = threadIdx.x + i * blockDim.x;
    if (p < pieces) {
      const uint4 u = xr[p];
      const _Float16 *hp = reinterpret_cast<const _Float16 *>(&u);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[i][e] = (float)hp[e];
    }
  }
  float mean, rstd;
  row_stats<PPT>(v, h, eps, scratch, mean, rstd);
  uint4 *orow = out + (size_t)blockIdx.x * pieces;
#pragma unroll
  for (int i = 0; i < PPT; ++i) {
    const int p = threadIdx.x + i * blockDim.x;
    if (p < pieces) {
      const uint4 g = gamma[p], b = beta[p];
      const _Float16 *gp = reinterpret_cast<const _Float16 *>(&g), *bp = reinterpret_cast<const _Float16 *>(&b);
      uint4 o;
      _Float16 *op = reinterpret_cast<_Float16 *>(&o);
#pragma unroll
      for (int e = 0; e < 8; ++e) op[e] = (_Float16)((v[i][e] - mean) * rstd * (float)gp[e] + (float)bp[e]);
      orow[p] = o;
    }
  }
}

// The share reduction and epilogue for whole rows, followed by the layer norm of the result: one
// workgroup per row, the row in registers as in layernorm_kernel.  Saves a launch and a pass over
// the row whenever a product feeds a layer norm (output projection -> second norm, feed-forward
// -> the next layer's first norm).
template <int PPT>
__global__ __launch_bounds__(kLnMaxThreads) void reduce_layernorm_kernel(const float *shares, const _Float16 *bias, const _Float16 *residual,
                                                                           const _Float16 *gamma, const _Float16 *beta, const int32_t n_out,
                                                                           const int32_t splits, const int32_t m, const LinearArgs a) {
  // (leading parameters: in scalar registers when the wavefront starts, so everything is asked for at once)
  __shared__ float4 scratch[2][kLnMaxThreads / 256];
  const int h = n_out, pieces = h >> 3, mrow = blockIdx.x;
  const Sink sink(a);
  float v[PPT][8];
  // the bias, the residual, gamma and beta are fetched behind the first shares: not behind the sums nor behind the reductions,
  // whose barriers would otherwise stand between these loads and what they do not depend on
  uint4 gam[PPT], bet[PPT];
#pragma unroll
  for (int i = 0; i < PPT; ++i) {
    const int p = threadIdx.x + i * blockDim.x;
    if (p < pieces) {
      float acc[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = 0.f;
      u32x4_t rb, bb;
      const uint64_t at = ((uint64_t)mrow * h + p * 8) * 2;
      for (int s2 = 0; s2 < splits; s2 += 4) {             // four cuts at a time, loads independent of one another
        float4 lo[4], hi[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int sj = s2 + j < splits ? s2 + j : splits - 1;      // past the last cut: the last again, left out below
          const float4 *sp = reinterpret_cast<const float4 *>(shares + ((size_t)sj * m + mrow) * h + p * 8);
          lo[j] = sp[0], hi[j] = sp[1];
        }
        if (s2 == 0) {
          __builtin_amdgcn_sched_barrier(0);
          // (without them, gamma: a branch around a load waits for it where the paths meet)
          bb = load_at<u32x4_t>((uint64_t)(bias ? bias : gamma) + p * 16);
          rb = load_at<u32x4_t>(residual ? (uint64_t)residual + at : (uint64_t)gamma + p * 16);
          gam[i] = reinterpret_cast<const uint4 *>(gamma)[p], bet[i] = reinterpret_cast<const uint4 *>(beta)[p];
          if (i == 0) sink.arrive();
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bool in = s2 + j < splits;
          acc[0] += in ? lo[j].x : 0.f, acc[1] += in ? lo[j].y : 0.f, acc[2] += in ? lo[j].z : 0.f, acc[3] += in ? lo[j].w : 0.f;
          acc[4] += in ? hi[j].x : 0.f, acc[5] += in ? hi[j].y : 0.f, acc[6] += in ? hi[j].z : 0.f, acc[7] += in ? hi[j].w : 0.f;
        }
      }
      const u32x4_t none = {0u, 0u, 0u, 0u};
      const half8 bp = __builtin_bit_cast(half8, bias ? bb : none), rp = __builtin_bit_cast(half8, residual ? rb : none);
      uint4 yo;
      _Float16 *yp = reinterpret_cast<_Float16 *>(&yo);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float y = acc[e] + (float)bp[e];
        if (sink.relu) y = fmaxf(y, 0.f);
        y += (float)rp[e];
        yp[e] = (_Float16)y;                               // the norm sees the row as it is stored
        v[i][e] = (float)yp[e];
      }
      store_at(sink.out0 + at, __builtin_bit_cast(u32x4_t, yo));
    }
  }
  float mean, rstd;
  row_stats<PPT>(v, h, a.ln_eps, scratch, mean, rstd);
#pragma unroll
  for (int i = 0; i < PPT; ++i) {
    const int p = threadIdx.x + i * blockDim.x;
    if (p < pieces) {
      const _Float16 *gp = reinterpret_cast<const _Float16 *>(&gam[i]), *bp = reinterpret_cast<const _Float16 *>(&bet[i]);
      uint4 o;
      _Float16 *op = reinterpret_cast<_Float16 *>(&o);
#pragma unroll
      for (int e = 0; e < 8; ++e) op[e] = (_Float16)((v[i][e] - mean) * rstd * (float)gp[e] + (float)bp[e]);
      reinterpret_cast<uint4 *>(a.ln_out + (size_t)mrow * h)[p] = o;
    }
  }
}

// The kernel that adds the cuts' shares up (and takes the layer norm of the sums, if asked to).
void launch_reduce(const LinearArgs &args, hipStream_t stream) {
  if (args.ln_out && (args.n_out >> 3) <= kLnMaxThreads)
    hipLaunchKernelGGL(reduce_layernorm_kernel<1>, dim3(args.m), dim3(ln_threads(args.n_out)), 0, stream, args.shares, args.bias,
                       args.residual, args.ln_gamma, args.ln_beta, args.n_out, args.splits, args.m, args);
  else if (args.ln_out)
    hipLaunchKernelGGL(reduce_layernorm_kernel<2>, dim3(args.m), dim3(ln_threads(args.n_out)), 0, stream, args.shares, args.bias,
                       args.residual, args.ln_gamma, args.ln_beta, args.n_out, args.splits, args.m, args);
  else
    hipLaunchKernelGGL(reduce_epilogue_kernel, dim3((args.n_out + 1023) / 1024, args.m), dim3(256), 0, stream, args.shares,
                       args.bias, args.residual, args.n_out, args.splits, args.m, args.seg0_cols, args.seg_cols, args);
}

template <int MF, int NW, bool NT>
void launch_staged_as(const LinearArgs &args, int n_tiles, hipStream_t stream) {
  hipLaunchKernelGGL((linear_lds_kernel<MF, NW, NT>), dim3((n_tiles + NW - 1) / NW, args.splits), dim3((NW + lin_stagers(MF)) * 64), 0, stream,
                     args.w, args.x, args.bias, args.n_kb, args.splits, args.n_in, args.m, args.n_tiles, args);
}

template <int MF, int NW>
void launch_staged(const LinearArgs &args, int n_tiles, hipStream_t stream) {
  if constexpr (MF <= OKV_LINEAR_MAX_ROWS / 16) {
    if ((int64_t)args.n_out * args.n_in * 2 >= kStreamStagedBytes) return launch_staged_as<MF, NW, true>(args, n_tiles, stream);
  }
  launch_staged_as<MF, NW, false>(args, n_tiles, stream);
}

template <int MF>
hipError_t launch_linear_mf(const LinearArgs &args, int n_tiles, bool fast, int fast_waves, hipStream_t stream) {
  if (fast) {
    fast_waves == 3 ? launch_staged<MF, 3>(args, n_tiles, stream) : launch_staged<MF, 4>(args, n_tiles, stream);
    if (args.to_shares) {
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      launch_reduce(args, stream);
    }
  } else if constexpr (MF <= OKV_LINEAR_MAX_ROWS / 16) {
    const bool stream_w = MF == 1 && (int64_t)args.n_out * args.n_in * 2 >= kStreamSimpleBytes;
    if (stream_w) hipLaunchKernelGGL((linear_kernel<1, true>), dim3(n_tiles), dim3(kLinWaves * 64), 0, stream, args.w, args.x, args.bias, args.n_kb,
                                     args.n_in, args.m, args);
    else hipLaunchKernelGGL((linear_kernel<MF, false>), dim3(n_tiles), dim3(kLinWaves * 64), 0, stream, args.w, args.x, args.bias, args.n_kb, args.n_in,
                            args.m, args);
  } else {
    return hipErrorInvalidValue;                       // more than OKV_LINEAR_MAX_ROWS rows: the staged or the tile kernel only
  }
  return hipGetLastError();
}

// The forms linear_tile_kernel and linear_wide_kernel (256 x 256, 192 x 128) are built in, with what a stage of 64 inputs takes a
// workgroup when every compute unit has one (us, MI355X, weights from HBM) and whether a compute unit has room for more.
// Fitted, with the constants of tile_plan, to 260 shapes of 129 to 1024 rows, 512 to 20480 features and inputs.  On others drawn since
// (256 to 20480, every form and cut timed) what they choose is slower than the fastest by 1.9 % on average at 193 to 1024 rows (400
// shapes; 25 % at worst) and by 1.4 % at 1025 to 4096 (310; 33 % at worst, the narrowest outputs).  Without 192 x 128 the latter were 2.2 %:
// 1100 x 16384 x 4096 170 us instead of 160, 1281 x 4096 x 5120 67.5 instead of 61, 2066 x 2304 x 2304 31.8 instead of 29.5.
// Wavefronts side by side in the rows (2 x 4) load every weight twice in linear_tile_kernel, which 256 x 192 needs to keep its
// accumulators in registers; at 128 rows and below one row of wavefronts measured faster (128 x 128 at 1024 x 4096 x 4096: 41 us as 1 x 4,
// 47 as 2 x 2).
struct TileForm {
  int rows, cols;
  double stage_us;
  bool shares_cu;
};
constexpr TileForm kTileForms[] = {{256, 256, 1.442, false}, {256, 192, 1.23, false}, {128, 256, 0.825, false}, {192, 128, 0.7245, false}, {128, 128, 0.5305, true},
                                   {96, 128, 0.416, true},   {64, 128, 0.374, true},  {64, 64, 0.2256, true},   {32, 64, 0.164, true}};
constexpr int kTileFormCount = sizeof(kTileForms) / sizeof(kTileForms[0]);

template <int F, int FM, int FN, int WM, int WN, int WD>
void launch_tile_as(const LinearArgs &a, hipStream_t stream) {
  using S = TileShape<FM, FN, WM, WN, WD>;
  static_assert(kTileForms[F].rows == S::kRows && kTileForms[F].cols == S::kCols, "the model's form is the kernel's");
  const int m_tiles = (a.m + S::kRows - 1) / S::kRows, groups = (a.n_out + S::kCols - 1) / S::kCols;
  hipLaunchKernelGGL((linear_tile_kernel<FM, FN, WM, WN, WD>), dim3(m_tiles * groups * a.splits), dim3(S::kThreads), 0, stream, a.w, a.x,
                     a.bias, a.n_kb, a.splits, a.n_in, a.m, a.n_tiles, m_tiles, groups, a);
}

template <int F, int FM, int FN, int WM, int WN, int NX>
void launch_wide_as(const LinearArgs &a, hipStream_t stream) {
  using S = WideShape<FM, FN, WM, WN, NX>;
  static_assert(kTileForms[F].rows == S::kRows && kTileForms[F].cols == S::kCols, "the model's form is the kernel's");
  const int m_tiles = (a.m + S::kRows - 1) / S::kRows, groups = (a.n_out + S::kCols - 1) / S::kCols;
  hipLaunchKernelGGL((linear_wide_kernel<FM, FN, WM, WN, NX>), dim3(m_tiles * groups * a.splits), dim3(S::kThreads), 0, stream, a.w, a.x,
                     a.bias, a.n_kb, a.splits, a.n_in, a.m, a.n_tiles, m_tiles, groups, a);
}

hipError_t launch_linear_tile(const LinearArgs &a, int form, hipStream_t stream) {
  switch (form) {
    case 0: launch_wide_as<0, 8, 4, 2, 4, 3>(a, stream); break;
    case 1: launch_tile_as<1, 8, 3, 2, 4, 2>(a, stream); break;
    case 2: launch_tile_as<2, 8, 2, 1, 8, 2>(a, stream); break;
    case 3: launch_wide_as<3, 6, 2, 2, 4, 4>(a, stream); break;
    case 4: launch_tile_as<4, 8, 2, 1, 4, 4>(a, stream); break;
    case 5: launch_tile_as<5, 6, 2, 1, 4, 4>(a, stream); break;
    case 6: launch_tile_as<6, 4, 2, 1, 4, 4>(a, stream); break;
    case 7: launch_tile_as<7, 4, 1, 1, 4, 4>(a, stream); break;
    case 8: launch_tile_as<8, 2, 1, 1, 4, 4>(a, stream); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.splits == 1) return e;
  launch_reduce(a, stream);
  return hipGetLastError();
}

// Which kernel a product runs and how its input dimension is cut, with the time a small model of the launch gives it.
struct LinearPlan {
  enum Kind { kSimple = 0, kStaged = 1, kTile = 2 } kind;
  int waves, cuts, form;
  double us;                             // tiles only
};

// Streaming wavefronts per workgroup (4 or 3) and cuts of the input dimension for the staged kernel, by a small
// model of the launch, in microseconds:
//   max(weights / 6.0 MB/us, (weights + rows of x fetched) / 10 MB/us) / fill + second kernel
// -- the weights come from HBM, they and the rows of x (every workgroup fetches the rows of its stretch:
// m x n_in x 2 bytes per group of 64 or 48 features) come through the L2s, `fill` is the share of
// workgroup slots in use when the workgroups are dealt to the compute units in rounds, and a cut costs the
// kernel that adds the shares up (a dependent launch and the shares written and read).  The rates are
// measured on MI355X (16384 x 4096: 27 us at 32 rows, 41 at 128).  Cuts divide the chunks evenly, leave every
// cut at least two chunks, and the kernel takes the chunks `pace` at a time.  A launch with more than two
// workgroups per compute unit is not considered (longer-lived workgroups measured faster than more of them).
// Examples on 256 compute units: 12288 x 4096 -> 3 wavefronts, no cut (256 workgroups); 6144 x 4096 -> 3
// wavefronts, 2 cuts; 4096 x 4096 and 4096 x 16384 -> 4 wavefronts, 4 cuts; 16384 x 4096 -> 4, none.
// Cuts 0: not a shape for the staged kernel.
LinearPlan staged_plan(int32_t m, int32_t n_out, int32_t n_in, int32_t n_cus) {
  LinearPlan plan = {LinearPlan::kStaged, 4, 0, 0, 0.0};
  if (m > OKV_LINEAR_MAX_ROWS_STAGED) return plan;
  const int chunk = lin_chunk((m + 15) / 16), pace = lin_weight_lead((m + 15) / 16);
  if (n_in % (32 * chunk * pace)) return plan;
  const int chunks = n_in / (32 * chunk);
  const double weight_mb = (double)n_out * n_in * 2 / 1e6;
  double best = 0;
  for (int w : {4, 3}) {
    const int groups = (n_out / 16 + w - 1) / w;
    const double x_mb = (double)groups * m * n_in * 2 / 1e6;
    for (int s = 1; s <= chunks; ++s) {
      if (chunks % (s * pace)) continue;
      if (s > 1 && chunks / s < 2) break;
      const int64_t wgs = (int64_t)groups * s;
      if (s > 1 && wgs > 2 * (int64_t)n_cus) break;
      const int64_t rounds = (wgs + n_cus - 1) / n_cus;
      const double fill = (double)wgs / (double)(rounds * n_cus);
      const double second = s > 1 ? 4.5 + 2.0 * s * m * n_out * 4 / 1e6 / 3.0 : 0.0;
      const double t = std::max(weight_mb / 6.0, (weight_mb + x_mb) / 10.0) / fill + second;
      if (plan.cuts == 0 || t < best * 0.98) {                  // on a near tie the first one found: 4 wavefronts, fewer cuts
        best = t;
        plan.waves = w;
        plan.cuts = s;
      }
    }
  }
  return plan;
}

// The staged plan's time where the tile kernel is the alternative, two estimates.  By the bytes, from 129 rows on: 3.9 us, the weights at 7.7 MB/us,
// the rows of x that a compute unit takes in at 71.5 KB/us (60 where they are 16384 inputs apart: rows at multiples of 32 KiB
// share the memory channels) and for a cut 2.5 us and the shares at 4.4 MB/us.  (60 shapes of 129 to 192 rows, 512 to 20480 features and
// inputs, weights from HBM, warm clocks: within 4.6 % rms.)
double staged_intake_kb(const LinearPlan &p, int32_t m, int32_t n_out, int32_t n_in, int32_t n_cus, double *weights_kb) {
  const int64_t wgs = (int64_t)((n_out / 16 + p.waves - 1) / p.waves) * p.cuts, rounds = (wgs + n_cus - 1) / n_cus;
  *weights_kb = (double)rounds * 16 * p.waves * (n_in / p.cuts) * 2 / 1e3;
  return (double)rounds * m * (n_in / p.cuts) * 2 / 1e3;
}
double staged_us_by_bytes(const LinearPlan &p, int32_t m, int32_t n_out, int32_t n_in, int32_t n_cus) {
  double weights_kb;
  const double intake_kb = staged_intake_kb(p, m, n_out, n_in, n_cus, &weights_kb), weight_mb = (double)n_out * n_in * 2 / 1e6;
  return 3.9 + weight_mb / 7.7 + intake_kb / (n_in % 16384 ? 71.5 : 60.0) + (p.cuts > 1 ? 2.5 + (double)p.cuts * m * n_out * 4 / 4.4e6 : 0.0);
}
// By what a compute unit takes in, from 65 rows on; better for many cuts and for several rounds (309 shapes of 129 to 192 rows, 256 to 20480: 7.4 %
// rms, by the bytes 10 %): 3.4 us, the root of the sum of squares of the weights at 4.85 MB/us and of the intake at 58 KB/us (of its
// weights a quarter), and for a cut 1.9 us, 0.14 for each and the shares at 4.15 MB/us.  (From 65 to 128 rows with constants of
// their own, 478 shapes: 6.4 % rms.)
double staged_us_by_intake(const LinearPlan &p, int32_t m, int32_t n_out, int32_t n_in, int32_t n_cus) {
  double weights_kb;
  const double intake_kb = staged_intake_kb(p, m, n_out, n_in, n_cus, &weights_kb), weight_mb = (double)n_out * n_in * 2 / 1e6;
  if (m > OKV_LINEAR_MAX_ROWS)
    return 3.41 + std::hypot(weight_mb / 4.85, (intake_kb + 0.24 * weights_kb) / 58.1) +
           (p.cuts > 1 ? 1.87 + 0.14 * p.cuts + (double)p.cuts * m * n_out * 4 / 4.15e6 : 0.0);
  return 3.07 + std::hypot(weight_mb / 6.06, intake_kb / 54.0) +
         (p.cuts > 1 ? 1.72 + 0.14 * p.cuts + (double)p.cuts * m * n_out * 4 / 3.51e6 : 0.0);
}

// The tile kernels' form and cuts: 4 us for the launch, the weights at 19.4 MB/us (the part of their way from HBM that
// the walk does not hide), the walk, and for a cut 2.8 us and the shares at 4.7 MB/us (written and read back); a launch that
// leaves compute units idle walks up to 8 % faster, and a cut has to be worth 1 %.  Forms of which a compute unit holds several
// workgroups are taken half way between whole and broken rounds.  With an odd number of blocks of 32 inputs every other row of x begins
// in the middle of a line and a 192 x 128 stage takes 12 to 15 % longer (4096 features x 4128 inputs: 1152 rows 47.2 -> 52.8 us,
// 2304 rows 95 -> 107), a 256 x 192 one 3 %.  In a single round that changes no choice (what is left then, 96 x 128, loses as much); beyond one it is
// counted: 4051 rows x 4112 x 4128 187 us so, 256 x 192 in two cuts 183.  At up to 192 rows shares take
// longer, 3.9 MB/us between tiles (`worth`) and, in the comparison with the staged kernel, 3.4 (`us`).  The 3.4 between tiles favoured few cuts: 192
// rows x 4096 x 16384 45.0 us in four cuts of 96 x 128 against 42.5 in eight of 192 x 128, 180 x 5120 x 11008 40.8 in three against 37.8 in
// six, 168 x 4224 x 4096 22.1 uncut against 18.4 in three.  With none dearer, 13824-wide products go from two cuts to seven and 8 % slower.
// Shares beyond 134 MB, which with the weights no longer stay in the memory-side cache until they are added, take 0.3 us a MB more: 3507 rows x 6144
// x 8192 370 us in three cuts (258 MB), 324 uncut, 1405 x 16384 x 12288 544 in two, 504 uncut.
// Every product from 65 rows on asks for this on its way to the GPU, so what does not depend on the form is worked out once per number of cuts, at
// up to 128 rows forms whose rows are not needed are passed over (one of fewer rows and a shorter stage has as few tiles), and a form is left
// where even full rounds without rounding up would make it no better.  The choice is that of the whole search (2 million shapes).
// Host ns of a choice beside an MI355X, the whole search with both staged estimates made for every candidate -> now: 96 rows x 4096 x 4096 287
// -> 178, 128 x 16384 x 4096 249 -> 73, 160 x 2048 x 2048 312 -> 247, 1024 x 4096 x 4096 243 -> 55; 16 x 4096 x 4096 (no tiles) 72 -> 49.
LinearPlan tile_plan(int32_t m, int32_t n_out, int32_t n_in, int32_t n_cus, int64_t workspace_bytes) {
  LinearPlan plan = {LinearPlan::kTile, 0, 0, 0, 0.0};
  const int stages = (n_in + 63) / 64;
  const double fixed_us = 4.0 + (double)n_out * n_in * 2 / 1e6 / 19.4;
  struct { double walk, shares_us, shares_mb, dearer; } cut[9];
  int most = 0;
  for (int s = 1; s <= 8; ++s) {
    if (s > 1 && (stages / s < 4 || (int64_t)s * m * n_out * 4 > workspace_bytes)) break;
    const double shares_mb = s > 1 ? (double)s * m * n_out * 4 / 1e6 : 0.0;
    cut[s].walk = (stages + s - 1) / s;
    cut[s].shares_mb = shares_mb;
    cut[s].shares_us = s > 1 ? 2.8 + shares_mb / 4.7 : 0.0;
    cut[s].dearer = 0.3 * std::max(0.0, shares_mb - 134.0) + (m <= OKV_LINEAR_MAX_ROWS_STAGED ? 0.045 * shares_mb : 0.0);
    most = s;
  }
  double best = 0;
  for (int f = 0; f < kTileFormCount; ++f) {
    const TileForm &form = kTileForms[f];
    if (m <= 128 && (form.rows > 128 || (m <= 96 && form.rows == 128 && form.cols == 128))) continue;
    const int64_t tiles = (int64_t)((m + form.rows - 1) / form.rows) * ((n_out + form.cols - 1) / form.cols);
    const double per_cu = 0.919 *                              // (0.92 below: less than that by more than sums are rounded)
                           (double)tiles * stages / n_cus * form.stage_us;
    for (int s = 1; s <= most; ++s) {
      if (plan.cuts && fixed_us + cut[s].shares_us + per_cu >= best) break;
      const double q = (double)(tiles * s) / n_cus;
      double whole = (double)(int64_t)q;                       // (std::ceil is a call)
      if (whole < q) whole += 1.0;
      const double stage_us = form.rows == 192 && n_in % 64 && q > 1.0 ? 1.12 * form.stage_us : form.stage_us;
      const double rounds = form.shares_cu ? 0.5 * (whole + std::max(1.0, q)) : whole;
      const double t = fixed_us + rounds * cut[s].walk * stage_us * (1.0 - 0.08 * (1.0 - std::min(1.0, q))) + cut[s].shares_us;
      const double worth = s > 1 ? 1.01 * t + cut[s].dearer : t;
      if (plan.cuts == 0 || worth < best) best = worth, plan.us = t + 0.084 * cut[s].shares_mb, plan.form = f, plan.cuts = s;
    }
  }
  return plan;
}

// Up to 16 rows (one fragment): the simple kernel rather than the staged one?  It needs no second launch and has more workgroups, the
// staged one reads x in whole lines and evens out products whose 16-feature tiles leave compute units idle or one round short.
// Models of both in us: 2.57 (2.91) for the launch, 0.56 where a wavefront's quarter of the inputs is no whole number of rounds of
// the walk, 3.39 for cuts, and the root of the sum of squares of the weights at 9.3 (8.1) MB/us and of what a compute unit takes in at
// 72 (58) KB/us, of which a row of x counts 2 of a feature's bytes (0.42), workgroups beyond whole rounds for 1 / 1.29 of one.  (414
// shapes of 1 to 24 rows, 256 to 24576 features, 256 to 20480 inputs, weights from HBM: 8 and 9 % rms.)  Up to 8 rows the staged
// one has to be 14 % better, which the models are not always good for (8 rows x 16384 x 4096 22 us simple, 25 staged).  Beyond, the simple
// one has to be 2 us better, since a layer norm of the result is a launch more behind it and not behind the staged kernel's shares (16
// x 768 x 3072 6.2 / 6.9 us simple / staged, with a norm 8.4 / 7.2; of 255 shapes of 9 to 16 rows, with and without a norm, 46 change and none is
// slower; at 1 us 63 change and 12 x 768 x 3072 with a norm loses 4 %).  us, the rule by rows alone -> this one: 8 rows x 5120 x 20480 48.4 ->
// 36.7, 3 x 512 x 20480 with a norm 18.1 -> 10.5, 8 x 1632 x 17920 19.9 -> 14.0; 12 x 4096 x 4096 10.6 -> 7.3, with a norm 12.2 -> 10.1, 12 x
// 2048 x 2048 7.8 -> 4.7, 9 x 3840 x 2560 8.3 -> 5.3, 9 x 2560 x 2560 7.4 -> 5.2, with a norm 8.6 -> 7.6, 12 x 2400 x 13568 (whose 53 chunks cannot
// be cut) 32.2 -> 18.9.
double few_rows_simple_us(int32_t m, int32_t n_out, int32_t n_in, int32_t n_cus) {
  const double q = n_out / 16.0 / n_cus, rounds = q <= 1.0 ? 1.0 : 1.29 * std::ceil(q) - 0.29 * q;
  const double intake_us = rounds * n_in * 2 / 1e3 * (16.0 + 2.0 * m) / 72.0, weights_us = (double)n_out * n_in * 2 / 1e6 / 9.3;
  return 2.57 + (n_in % 1024 ? 0.56 : 0.0) + std::sqrt(intake_us * intake_us + weights_us * weights_us);
}
bool few_rows_simple(int32_t m, int32_t n_out, int32_t n_in, int32_t n_cus, const LinearPlan &staged) {
  const double weight_mb = (double)n_out * n_in * 2 / 1e6, row_kb = (double)n_in * 2 / 1e3;
  const double simple_us = few_rows_simple_us(m, n_out, n_in, n_cus);
  const int64_t wgs = (int64_t)((n_out / 16 + staged.waves - 1) / staged.waves) * staged.cuts;
  const double intake_kb = (double)((wgs + n_cus - 1) / n_cus) * (16.0 * staged.waves + 0.42 * m) * row_kb / staged.cuts;
  const double staged_us = 2.91 + (staged.cuts > 1 ? 3.39 : 0.0) + std::sqrt(intake_kb / 58.0 * (intake_kb / 58.0) + weight_mb / 8.1 * (weight_mb / 8.1));
  if (m <= OKV_LIN_SIMPLE_ROWS) return simple_us < 1.14 * staged_us;
  return simple_us + 2.0 < staged_us;
}

// The kernel for a product.  Up to 16 rows the simple or the staged one (few_rows_simple), up to 64 the staged one where it takes the
// shape (86 shapes of 17 to 32 rows: 0.5 % slower on average than the faster of it and tiles, 95 of 33 to 64: 1.6 %).  From there to
// OKV_LINEAR_MAX_ROWS rows tiles where their model is 7 % below the staged kernel's by intake: us staged / tiles 128 rows x 5120 x 20480 65.5 /
// 49.0, 128 x 20480 x 5120 66 / 52, 128 x 28672 x 4096 62.3 / 48.8, 128 x 2304 x 768 6.2 / 4.9, 96 x 5120 x 20480 56.8 / 44.7, 97 x 272 x 8192
// 11.4 / 8.2; 128 x 12288 x 4096 28 / 31, 128 x 16384 x 4096 35 / 38 (478 shapes of 288 to 20480 features: 55 change, 14 % faster, the worst
// 0.5 % slower; at 5 % 74 change and the worst, 80 x 4096 x 16384 with a norm, is 3 % slower; 27 of 16 to 272: 4 change, 27 % faster).  Beyond
// 20480 features with less than 4096 inputs 12 % below (at 7 % 86 x 36256 x 3328 61.9 / 65.4, 84 x 29232 x 1024 17.3 / 18.2; of 120 shapes of
// 20608 to 51664 features 67 change, 14 % faster, the worst 0.5 % slower).  From there to the staged kernel's 192 rows whichever the models
// favour by more than they are good for (at 192 rows 4096 x 16384 42 us against 53 and 16384 x 4096 40 against 43, tiles; 2304 x 4096 17.7 against 15.2 and 6144 x 2048
// 20.2 against 17.0, staged), or whichever the second estimate of the staged one favours by 4 % (129 rows x 496 x 6400, 25 cuts, 13.1 against
// 8.9, 136 x 608 x 12032, 47 cuts, 20.2 against 12.8, 160 x 272 x 8192, 32 cuts, 13.0 against 8.5, 192 x 20480 x 5120 uncut in two rounds 85
// against 72, tiles; none of 309 shapes slower; of 27 of 16 to 272 features 26 are tiles, 22 % faster, the worst, 160 x 64 x 2048, 2 % slower),
// beyond always a tile kernel.  Where the staged kernel does not take the shape (inputs not a multiple of its chunks, or a cut without a
// workspace) the simple kernel's time follows the row fragments and the blocks of a wavefront, in rounds of a workgroup per compute unit
// (which overlap a little) and somewhat faster where units are idle; the tile model is 1.2 us high for such short walks, and 2 for
// cut ones.  simple / tile us: 9 rows x 4096 x 10240 16.6 / 37.3, 12 x 4096 x 5120 10.0 / 19.8, 16 x 4224 x 4096 14.1 / 16.1, 19 x 3072 x
// 2304 6.1 / 8.7, 52 x 5120 x 4224 35.6 / 17.4, 110 x 5120 x 2400 32.9 / 14.4, 17 x 192 x 20480 29 / 58 uncut, 11.5 in eight cuts.  (1200
// shapes of 9 to 128 rows, 96 to 20480 features and inputs, weights from HBM: the choice is 0.6 % slower than the faster of the two
// on average.  The simple kernel's time scatters by 10 % around its model: in doubt the line favours tiles, whose model is the better one.)
LinearPlan choose_linear(int32_t m, int32_t n_out, int32_t n_in, int32_t n_cus, int64_t workspace_bytes) {
  const LinearPlan simple = {LinearPlan::kSimple, 0, 1, 0, 0.0};
  // (most products of up to 8 rows are faster than the staged kernel could stream the weights alone: the same choice without its plan, 6 ns of the
  // call's host time for 4 x 4096 x 4096 instead of some 45)
  if (m <= OKV_LIN_SIMPLE_ROWS && few_rows_simple_us(m, n_out, n_in, n_cus) < 1.14 * (2.91 + (double)n_out * n_in * 2 / 8.1e6)) return simple;
  const LinearPlan staged = staged_plan(m, n_out, n_in, n_cus);
  const bool staged_runs = staged.cuts == 1 || (staged.cuts > 1 && (int64_t)staged.cuts * m * n_out * 4 <= workspace_bytes);
  if (m <= OKV_LIN_SIMPLE_ROWS && !staged_runs) return simple;
  if (m <= 16 && staged.cuts > 0 && few_rows_simple(m, n_out, n_in, n_cus, staged)) return simple;
  if (staged_runs && m <= 64) return staged;
  const LinearPlan tile = tile_plan(m, n_out, n_in, n_cus, workspace_bytes);
  if (staged_runs) {
    const double by_intake = staged_us_by_intake(staged, m, n_out, n_in, n_cus);
    if (m <= OKV_LINEAR_MAX_ROWS) return tile.us < (n_out > 20480 && n_in < 4096 ? 0.88 : 0.93) * by_intake ? tile : staged;
    return tile.us < 0.96 * by_intake || tile.us < 0.955 * staged_us_by_bytes(staged, m, n_out, n_in, n_cus) ? tile : staged;
  }
  if (m > OKV_LINEAR_MAX_ROWS) return tile;
  const double q = n_out / 16.0 / n_cus, rounds = q <= 1.0 ? 1.0 : 0.82 * std::ceil(q) + 0.18 * q;
  const int fragments = (m + 15) / 16;
  const double simple_us = 1.7 + 0.066 * fragments + rounds * n_in / 128.0 * (0.065 + 0.114 * fragments) * (1.0 - 0.27 * (1.0 - std::min(1.0, q)));
  const double tile_us = tile.cuts > 1 ? tile.us - 2.0 : 0.95 * tile.us - 1.2;
  return tile_us < simple_us ? tile : simple;
}

}  // namespace

int64_t linear_workspace_bytes(int32_t m, int32_t n_out, int32_t n_in, int32_t n_cus) {
  // up to OKV_LINEAR_MAX_ROWS rows a shape that the staged kernel does not take asks for none
  const LinearPlan plan = choose_linear(m, n_out, n_in, n_cus, m > OKV_LINEAR_MAX_ROWS || staged_plan(m, n_out, n_in, n_cus).cuts ? INT64_MAX : 0);
  // a single cut of the staged kernel still goes through a share when a layer norm follows
  return plan.kind == LinearPlan::kStaged || plan.cuts > 1 ? (int64_t)plan.cuts * m * n_out * 4 : 0;
}

LinearRoute linear_route(int32_t m, int32_t n_out, int32_t n_in, int32_t n_cus, int64_t workspace_bytes) {
  const LinearPlan plan = choose_linear(m, n_out, n_in, n_cus, workspace_bytes);
  if (plan.kind == LinearPlan::kSimple) return {plan.kind, (m + 15) / 16 * 16, 16, 1};
  if (plan.kind == LinearPlan::kStaged) return {plan.kind, (m + 15) / 16 * 16, 16 * plan.waves, plan.cuts};
  return {plan.kind, kTileForms[plan.form].rows, kTileForms[plan.form].cols, plan.cuts};
}

hipError_t launch_linear(const LinearLaunch &l, hipStream_t stream) {
  LinearArgs a;
  a.x = static_cast<const uint4 *>(l.x);
  a.w = static_cast<const uint4 *>(l.w_packed);
  a.bias = static_cast<const _Float16 *>(l.bias);
  a.residual = static_cast<const _Float16 *>(l.residual);
  for (int s = 0; s < 3; ++s) a.out[s] = static_cast<_Float16 *>(s < l.n_seg ? l.out[s] : l.out[0]);
  a.m = l.m;
  a.n_in = l.n_in;
  a.n_kb = l.n_in / 32;
  a.seg0_cols = l.first_cols ? l.first_cols : l.n_out / l.n_seg;
  a.seg_cols = l.n_seg > 1 ? (l.n_out - a.seg0_cols) / (l.n_seg - 1) : l.n_out;
  a.relu = l.relu;
  const int n_tiles = l.n_out / 16;
  a.n_tiles = n_tiles;
  a.n_out = l.n_out;
  a.ln_gamma = static_cast<const _Float16 *>(l.ln_gamma);
  a.ln_beta = static_cast<const _Float16 *>(l.ln_beta);
  a.ln_out = nullptr;
  a.ln_eps = l.ln_eps;
  const int64_t have = l.workspace ? l.workspace_bytes : 0;
  const LinearPlan plan = choose_linear(l.m, l.n_out, l.n_in, l.n_cus, have);
  const bool fast = plan.kind == LinearPlan::kStaged;
  a.splits = plan.kind == LinearPlan::kSimple ? 1 : plan.cuts;
  a.shares = static_cast<float *>(l.workspace);
  a.to_shares = a.splits > 1;
  // a layer norm of the result rides on the share reduction when there is one to ride on (the staged kernel then writes
  // its share also when there is a single cut; with the tile kernel's hundreds of rows a pass of its own over the fp16
  // result moves less than fp32 shares would)
  const bool fuse_ln = l.ln_out && l.n_seg == 1 && l.n_out <= kLnMaxWidth && (fast || a.splits > 1) &&
                       have >= (int64_t)a.splits * l.m * l.n_out * 4;
  if (fuse_ln) {
    a.to_shares = 1;
    a.ln_out = static_cast<_Float16 *>(l.ln_out);
  }
  hipError_t e = hipErrorInvalidValue;
  if (plan.kind == LinearPlan::kTile) e = launch_linear_tile(a, plan.form, stream);
  else switch ((l.m + 15) / 16) {
    case 1: e = launch_linear_mf<1>(a, n_tiles, fast, plan.waves, stream); break;
    case 2: e = launch_linear_mf<2>(a, n_tiles, fast, plan.waves, stream); break;
    case 3: e = launch_linear_mf<3>(a, n_tiles, fast, plan.waves, stream); break;
    case 4: e = launch_linear_mf<4>(a, n_tiles, fast, plan.waves, stream); break;
    case 5: e = launch_linear_mf<5>(a, n_tiles, fast, plan.waves, stream); break;
    case 6: e = launch_linear_mf<6>(a, n_tiles, fast, plan.waves, stream); break;
    case 7: e = launch_linear_mf<7>(a, n_tiles, fast, plan.waves, stream); break;
    case 8: e = launch_linear_mf<8>(a, n_tiles, fast, plan.waves, stream); break;
    case 9: e = launch_linear_mf<9>(a, n_tiles, fast, plan.waves, stream); break;
    case 10: e = launch_linear_mf<10>(a, n_tiles, fast, plan.waves, stream); break;
    case 11: e = launch_linear_mf<11>(a, n_tiles, fast, plan.waves, stream); break;
    case 12: e = launch_linear_mf<12>(a, n_tiles, fast, plan.waves, stream); break;
  }
  if (e != hipSuccess || !l.ln_out || fuse_ln) return e;
  return launch_layernorm(l.out[0], l.ln_gamma, l.ln_beta, l.ln_out, l.m, l.n_out, l.ln_eps, stream);   // the same in two steps
}

hipError_t launch_pack_weight(void *dst, const void *src, int32_t n_out, int32_t n_in, hipStream_t stream) {
  const int64_t total = (int64_t)n_out * n_in / 8;
  const unsigned blocks = (unsigned)std::min<int64_t>((total + 255) / 256, 1 << 16);
  hipLaunchKernelGGL(pack_weight_kernel, dim3(blocks), dim3(256), 0, stream, static_cast<uint4 *>(dst),
                     static_cast<const uint4 *>(src), n_out, n_in);
  return hipGetLastError();
}

hipError_t launch_layernorm(const void *x, const void *gamma, const void *beta, void *out, int32_t m, int32_t h, float eps,
                            hipStream_t stream) {
  if ((h >> 3) > kLnMaxThreads)
    hipLaunchKernelGGL(layernorm_kernel<2>, dim3(m), dim3(ln_threads(h)), 0, stream, static_cast<const uint4 *>(x),
                       static_cast<const uint4 *>(gamma), static_cast<const uint4 *>(beta), static_cast<uint4 *>(out), h, eps);
  else
  hipLaunchKernelGGL(layernorm_kernel<1>, dim3(m), dim3(ln_threads(h)), 0, stream, static_cast<const uint4 *>(x),
                     static_cast<const uint4 *>(gamma), static_cast<const uint4 *>(beta), static_cast<uint4 *>(out), h, eps);
  return hipGetLastError();
}

}  // namespace okv
