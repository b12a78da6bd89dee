// Host-side launch interface of the HIP kernels (internal to libsugg).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.hpp"

namespace sugg {

// One kernel of a work item: where its rows start, its index in the batch and
// its global optimisation ids (ascending; bit b of a version <-> opt[b]).
struct alignas(16) KRec {
  int64_t row_off;
  int32_t kid;
  int32_t pad;
  uint8_t opt[16];
};

// Row stride of the FP32 weight copy: E weights and the intercept, padded to
// a multiple of 4 so every row starts 16-byte aligned.
__host__ __device__ inline int w32_ld(int E) { return (E + 4) & ~3; }

// Arguments of the judge: plain composed log-speedups of given subsets.
template <typename T>
struct JudgeArgs {
  const T* counters;
  const T* cycles;
  int32_t E;
  int32_t D;
  const T* W;              // [D, ldw]: E weights then the intercept
  int32_t ldw;             // row stride of W
  const T* mu;
  const T* isg;
  const int64_t* row_off;  // [K+1]
  const int32_t* nopts;    // [K]
  const int64_t* opt_off;  // [K+1]
  const int32_t* opt_ids;
  int32_t K;
  int32_t C;               // candidates per kernel
  const int32_t* cand;     // [K, C] subset bitmasks, < 0 = none
  T* out;                  // [K, C]; 0 for S = 0, NaN for none
  const T* ref;            // [K, C] reference values (with flag)
  double tol;
  int32_t* flag;           // [K] or null: 1 where some candidate differs from ref by > tol
  int32_t accumulate;      // nonzero: keep flags already set (no clearing)
  int32_t* status;
};

// Arguments of the fused scoring kernel (predict / suggest).
template <typename T>
struct PathArgs {
  const JudgeArgs<T>* judge;   // non-null: run the judge instead (same dispatch)
  const int32_t* kmask;        // [K] or null: only kernels with kmask != 0 are scored and written
  const T* counters;       // [N, E]
  const T* cycles;         // [N]
  int32_t E;
  int32_t D;
  const Item* items;       // work list
  const KRec* recs;        // kernels of the items, item after item
  int32_t n_items;
  int32_t K;
  int32_t uni_B;           // >= 0: all kernels have uni_B optimisations and item i
  int32_t uni_nk;          //       holds kernels [i*uni_nk, (i+1)*uni_nk) (items unused)
  int32_t uni_ops;         // nonzero (with uni_B >= 0): every kernel has the same global
  uint64_t uni_opt_lo;     //   optimisation ids, byte b of (lo, hi) = id of local bit b;
  uint64_t uni_opt_hi;     //   the kernel records are then not read
  int32_t* queue;          // [2] next item, finished workgroups; zero at launch, re-armed by the kernel
  const T* mu;             // [E]
  const T* isg;            // [E] 1 / sigma
  const T* W;              // [D, ldw]: E weights then the intercept
  int32_t ldw;             // row stride of W
  T* grid;                 // [N, grid_ld] or null
  int32_t grid_ld;
  T* table;                // [N] or null
  int32_t* idx_out;        // [K, n] or null (no ranking)
  T* score_out;
  int32_t* count_out;
  int32_t n;
  T tau;
  int32_t* status;
};

struct PathLaunch {
  int waves;       // waves per workgroup (1..8)
  int unroll;      // rows per lane group per iteration (1, 2, 4)
  int grid;        // workgroups (persistent); 0 = occupancy-derived
};

// Fused normalise -> candidate predict -> compose [-> rank]; VPL = columns
// per lane (E <= 16 * VPL), instantiated for VPL 4, 8, 16.
template <typename T, int VPL>
hipError_t launch_path_vpl(const PathArgs<T>& a, int max_item_rows, int max_item_kernels, int max_B,
                           const PathLaunch& cfg, hipStream_t s);
// Split form for batches of equal kernels (same B <= 6, same ids, rows kernel
// after kernel): 16-version workgroups write chain edges to edges[N]; the
// last of a kernel's workgroups (arrivals[k], zero between launches, re-armed
// by that workgroup) composes and ranks.  Same results as the fused kernel.
template <typename T>
hipError_t launch_path_split(const PathArgs<T>& a, int32_t* arrivals, T* edges, hipStream_t s);

// The streaming form of the scoring pass: workgroups take chunks of
// consecutive whole kernels in memory order (mixed B), one chunk each.
struct alignas(16) Chunk {
  int64_t row0;   // first row
  int32_t k0;     // first kernel
  int32_t nk;     // kernels
  int32_t R;      // rows
  int32_t pad[3];
};
// One kernel of a chunk (kernel order, one record per kernel of the batch):
// its first row relative to its chunk's, its B and global ids (bit b <-> op[b]).
struct alignas(16) CRec {
  int16_t rel;
  int8_t B;
  int8_t skip;    // 0; in a workgroup's copy 1 where a mask does not select the kernel
  uint8_t op[12];
};
static_assert(sizeof(CRec) == 16 && SUGG_MAX_OPTS <= 12, "chunk kernel record");
template <typename T>
struct ChunkArgs {
  const T* counters;
  const T* cycles;
  int32_t E;
  int32_t D;
  const T* W;
  int32_t ldw;
  const T* mu;
  const T* isg;
  const CRec* recs;          // [K]
  const Chunk* chunks;
  int32_t n_chunks;
  int32_t max_rows;          // largest chunk
  int32_t max_nk;            // most kernels in a chunk
  int32_t wide;              // nonzero: workgroups of 1024 (or 512) threads, one row per lane group and stage
  const int32_t* kmask;      // [K] or null: only kernels with kmask != 0 are scored and written
  int32_t packed;            // with kmask: workgroups go to the chunks with a selected kernel (each lane
                             //   reads the flags of a chunk)
  T* grid;                   // [N, grid_ld] or null (then no ranking)
  int32_t grid_ld;
  T* table;                  // nullable
  int32_t* idx_out;          // nullable (then no ranking)
  T* score_out;
  int32_t* count_out;
  int32_t n;
  T tau;
  int32_t* status;
};
// unroll: rows per lane group per stage (1, 2, 4); one workgroup per chunk
template <typename T>
hipError_t launch_path_chunks(const ChunkArgs<T>& a, int unroll, hipStream_t s);
// dynamic LDS of the streaming form
size_t path_chunk_lds(size_t tsize, int D, int E, int max_rows, int max_nk);

template <typename T>
hipError_t launch_path(const PathArgs<T>& a, int max_item_rows, int max_item_kernels,
                       int max_B, const PathLaunch& cfg, hipStream_t s);

// Generic segmented top-n.
template <typename T>
hipError_t launch_rank(const T* scores, const int64_t* seg_off, int32_t nseg, int32_t skip_head,
                       int32_t n, T tau, int32_t* idx_out, T* score_out, int32_t* count_out,
                       hipStream_t s, int64_t seg_len = 0);   // seg_off null: segments of seg_len

// Threshold band of short suggestion lists (entries outside the list with
// score >= lo, ascending, at most C per segment; flag 1 on overflow).
template <typename T>
hipError_t launch_band(const T* scores, const int64_t* seg_off, int32_t nseg, int32_t skip_head,
                       const int32_t* top_idx, const int32_t* top_count, int32_t n, double lo, int32_t C,
                       int32_t* cand_out, T* ref_out, int32_t* flag_out, hipStream_t s);

// A serving query between the surrogate's tables and the plain pass, a batch
// of kernels with B optimisations each.
constexpr int kMaxBand = 64;
struct ServeTailArgs {
  const float* ys;         // [K << B] the surrogate's tables
  const float* sc;         // [K, n] values of the lists in idx / count; null: rank here
  const float* counters;   // [K << B, E]
  const float* cycles;
  int32_t E, B, K, n, cap; // cap: at most this many band subsets
  const float* W;          // [D, ldw]: E weights then the intercept
  int32_t ldw;
  const float* mu;
  const float* isg;
  const int64_t* row_off;  // [K+1]
  const int64_t* opt_off;  // [K+1]
  const int32_t* opt_ids;
  float tau;
  double lo;               // band: values from here
  double tol;              // largest |surrogate - plain| of a kept subset
  int32_t* idx;            // [K, n] the answer: subsets, plain values, length
  float* score;
  int32_t* count;
  int32_t* flag;           // [K] 1: answer by the plain pass
  int32_t* status;
};
hipError_t launch_serve_tail(const ServeTailArgs& a, hipStream_t s);

// FP64 column statistics of x = ln(c / cyc) over all N rows; lcyc (nullable,
// [N]) receives every row's ln(cyc); isg64, mu32, isg32 (all or none) further
// copies of the statistics.
template <typename T>
hipError_t launch_colstats(const T* counters, const T* cycles, int64_t N, int32_t E,
                           double* partial, int32_t nchunks, double* mu64, double* sig64,
                           T* mu_t, T* isg_t, int32_t* status, hipStream_t s, double* lcyc = nullptr,
                           double* isg64 = nullptr, float* mu32 = nullptr, float* isg32 = nullptr);
int colstats_chunks(int64_t N);

// z = (x - mu) / sigma in the plan dtype.
template <typename T>
hipError_t launch_standardize(const T* counters, const T* cycles, int64_t N, int32_t E, const T* mu,
                              const T* isg, T* z, int32_t* status, hipStream_t s);

// z of the rows listed in rows[nrows] (e.g. each kernel's baseline version).
template <typename T>
hipError_t launch_standardize_rows(const T* counters, const T* cycles, const int64_t* rows, int64_t nrows, int32_t E,
                                   const T* mu, const T* isg, T* z, int32_t* status, hipStream_t s);
// the same values rounded to BF16, row i at z + i * ldz (the surrogate's input)
hipError_t launch_standardize_rows_bf16(const float* counters, const float* cycles, const int64_t* rows, int64_t nrows,
                                        int32_t E, const float* mu, const float* isg, __bf16* z, int32_t ldz,
                                        int32_t* status, hipStream_t s);

// FP64 z and ln(cycles) for the regression.
template <typename T>
hipError_t launch_zfeat64(const T* counters, const T* cycles, int64_t N, int32_t E,
                          const double* mu64, const double* sig64, double* z64, double* lcyc64,
                          hipStream_t s);

// A run of before versions of the same optimisations (see launch_gram_rows).
struct GramSeg {
  int64_t base;    // first entry of the row list
  int32_t first;   // classes: first kernel in the kernel list; pairs: the kernel
  int32_t sel;     // classes: the version; pairs: the local bit of the optimisation
  uint64_t bits;   // four bits per optimisation of the class, ascending id: its local bit
};
// A before version: its row, and the local bits of the optimisations it is a
// before version of (after version of the j-th: row + 2^bit).
struct alignas(16) GramRow {
  int64_t row;
  uint64_t bits;
};
// The row list of the segments: entry q of a segment is version `sel` of
// kernel klist[first + q] (classes: kernels with the same optimisations), or
// the q-th version without bit `sel` of kernel `first` (pairs).
hipError_t launch_gram_rows(const GramSeg* segs, int nseg, int64_t n, bool pairs, const int32_t* klist,
                            const int64_t* row_off, GramRow* out, hipStream_t s);

// One chunk of rows that are before versions of the ids in mask.
struct GramWork {
  int64_t begin;   // into the row list
  uint64_t mask;   // global ids
  int32_t n;
  int32_t pad;
};

struct GramArgs {
  const void* counters;     // [N, E], plan dtype
  const double* lcyc;       // [N] ln(cycles)
  const double* mu;         // [E]
  const double* sig;        // [E]
  int32_t E;
  const GramRow* rows;
  const GramWork* work;
  int32_t n_work;
  double* partial;          // [n_work, gram_stride(E)] lower triangle of 16 x 16 blocks
};

int gram_blocks(int E);       // block columns: E padded, and the labels' and ones' block
int64_t gram_stride(int E);   // doubles of one lower triangle
int gram_slices(int n_work, int D, int E);   // slices of the chunks' sums
template <typename T>
hipError_t launch_gram(const GramArgs& a, hipStream_t s);
// sums of the chunks' partials per id into reduced [D, gram_stride] (the
// label row 0 holds the id's); slices: [gram_slices, D, gram_stride]
hipError_t launch_gram_reduce(const GramArgs& a, int D, double* slices, double* reduced, hipStream_t s);

// Solve every optimisation's normal equations.
struct SolveArgs {
  int32_t E;
  int32_t D;
  int32_t nb;             // gram_blocks(E)
  double lambda;
  const double* reduced;  // [D, gram_stride(E)]
  double* A;          // [D, solve_workspace(E)] when the system does not fit in LDS
  double* W64;        // [D, E+1]
  float* W32;         // [D, w32_ld(E)]
  int32_t* status;
};

size_t solve_workspace(int E);   // doubles per optimisation (0: LDS)
hipError_t launch_solve(const SolveArgs& a, hipStream_t s);

hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s);

// Arguments of the all-paths composition and greedy re-profiling kernels.
template <typename T>
struct PathsArgs {
  const T* counters;
  const T* cycles;
  int32_t E, D, ldw;
  const T* W;
  const T* mu;
  const T* isg;
  const int64_t* row_off;
  const int32_t* nopts;
  const int64_t* opt_off;
  const int32_t* opt_ids;
  int32_t K, Bmax, n;
  T tau;
  T* table;          // allpaths: [N]
  int32_t* idx_out;  // allpaths (nullable): [K, n]
  T* score_out;
  int32_t* count_out;
  int32_t* path_out;  // greedy: [K, Bmax + 1]
  int32_t* steps_out; // greedy: [K]
  T* gain_out;        // greedy: [K]
  int32_t* status;
};

template <typename T>
hipError_t launch_paths(const PathsArgs<T>& a, bool greedy, hipStream_t s);
template <typename T>
size_t paths_lds_bytes(int D, int E, int Bmax);

// ---- surrogate MLP --------------------------------------------------------
enum GemmEpilogue : int {
  kEpiWgrad = 0,       // FP32 split-K partial of a weight gradient
  kEpiFwdHidden = 1,   // + bias, keep pre-activation, GELU, BF16 row-major and transposed
  kEpiFwdOut = 2,      // + bias -> Y; with targets: squared error partials and dY
  kEpiBwdHidden = 3,   // * GELU'(pre-activation) -> BF16 row-major and transposed
  kEpiFwdRank = 4      // + bias -> Y (optional) and each row's top n above tau (the tile spans N)
};

// C[M x N] = A[M x K] . Bt[N x K]^T, BF16 operands, FP32 accumulation.
struct GemmArgs {
  const __bf16* A;
  int lda;
  const __bf16* Bt;
  int ldb;
  int M, N, K;
  int k_per_split;       // K range of one split (grid z), multiple of 32
  const float* bias;     // [N]
  float* Cf;             // FP32 output (pre-activation, Y or split partials)
  int ldcf;
  __bf16* Cb;            // BF16 row-major output
  int ldcb;
  __bf16* Ct;            // BF16 transposed output [N x M]
  int ldct;
  const float* gact;     // pre-activation for GELU'
  int ldg;
  const float* target;   // [M x N] targets
  int ldt;
  const int32_t* trow;   // nullable: output row r's target is row trow[r] of target
  int32_t* idx_out;      // kEpiFwdRank: [M x n] columns of each row's top n (-1 padded),
  float* score_out;      //   their values (NaN padded) and the count; columns >= skip
  int32_t* count_out;    //   with value > tau, by value descending then column ascending
  int n, skip;
  float tau;
  float* loss_part;      // one partial per output tile
  float scale;           // dY = scale * (Y - T)
};

// info (nullable, 4 ints): the launched instance as (tile rows, tile columns,
// K splits, 1 if the variant without bounds checks ran)
hipError_t launch_gemm(const GemmArgs& g, int epi, int splits, hipStream_t s, int32_t* info = nullptr);
// the output layer with the ranking epilogue: N must be 64 or 128, n <= 8
hipError_t launch_gemm_rank(const GemmArgs& g, hipStream_t s, int32_t* info = nullptr);
hipError_t launch_pack(const float* src, int rows, int cols, __bf16* dst, int ldd, __bf16* dst_t, int ldt,
                       hipStream_t s);
hipError_t launch_loss_sum(const float* part, int n, float scale, float* loss, hipStream_t s);
hipError_t launch_adam(float* p, const float* g, float* m, float* v, int64_t n, float lr, float b1, float b2,
                       float eps, int step, hipStream_t s);
// Rows idx[0..rows) of the FP32 matrix src [src_rows x cols] to BF16
// row-major dst and transposed dst_t (as launch_pack); an index outside
// [0, src_rows) reads row 0 and sets kStatusBadIndex in status.  The rows
// read are written to rows_out [rows].
struct GatherArgs {
  const float* src;
  int64_t src_rows;
  int cols;
  const int32_t* idx;
  int rows;
  __bf16* dst;
  int ldd;
  __bf16* dst_t;
  int ldt;
  int32_t* rows_out;
  int32_t* status;
};
hipError_t launch_gather_pack(const GatherArgs& g, hipStream_t s);
// A weight gradient dW[M x N] = A[M x K] . Bt[N x K]^T split over K and a
// hidden-layer backward (kEpiBwdHidden, one split) that do not depend on each
// other, in one launch where their instances allow (else two launches; the
// results are the same either way).
hipError_t launch_gemm_pair(const GemmArgs& gw, int splits, const GemmArgs& gb, hipStream_t s,
                            int32_t* info_w = nullptr, int32_t* info_b = nullptr);
// The end of up to three weight gradients in one launch: split-K sums (in
// split order) of the partials part [splits x n] into out [n], and row sums
// of the transposed BF16 activation gradient x [rows x cols] (leading
// dimension ld; its bias gradient) into bias_out [rows].
struct WgradJob {
  const float* part;
  int64_t n;
  int splits;
  float* out;
  const __bf16* x;
  int rows, cols, ld;
  float* bias_out;
};
struct FinishArgs {
  WgradJob job[3];
  int njobs;
  const float* loss_part;   // launch_train_update: the loss as launch_loss_sum
  int loss_n;
  int loss_quads;           // nonzero: four parts per tile, summed in order first
  float loss_scale;
  float* loss;
};
hipError_t launch_wgrad_finish(const FinishArgs& a, hipStream_t s);
// Adam (as launch_adam) over the surrogate's flat parameters p (gradients in
// g), writing the updated weights of its three layers to their BF16 working
// copies (row-major w[l]; transposed wt[l] where non-null, leading dimension =
// rows).
struct AdamPackArgs {
  float* p;
  const float* g;
  float* m;
  float* v;
  int64_t n;
  float lr, b1, b2, eps, c1, c2;
  int64_t off[3];     // first parameter of each weight matrix
  int rows[3], cols[3];
  __bf16* w[3];
  __bf16* wt[3];
};
// launch_wgrad_finish (three jobs, the last layer's first, whose outputs are
// the parts of a.g; with the loss), that Adam with step's bias corrections, and
// launch_gather_pack of the next mini-batch (nullable) in one launch.
hipError_t launch_train_update(const AdamPackArgs& a, const FinishArgs& f, int step, const GatherArgs* next,
                               hipStream_t s);

// The output layer of a training step and the backward through it, hidden
// width 512 (mlp_train.hip): dy [M x out], dyt (leading dimension ldt), da2
// [M x 512], da2t and the loss in four parts per 64 x 64 tile.
struct OutBackwardArgs {
  const __bf16* h2;        // [M x 512]
  const __bf16* w3;        // [out x 512]
  const __bf16* w3t;       // [512 x out]
  const float* b3;
  const float* a2;         // [M x 512] pre-activations
  const float* target;     // rows of out; row r's is trow[r] (nullable: r)
  const int32_t* trow;
  int M;
  float scale;             // dY = scale * (Y - T)
  __bf16 *dy, *dyt, *da2, *da2t;
  int ldt;
  float* loss_part;
};
hipError_t launch_out_backward(const OutBackwardArgs& a, int out, hipStream_t s);
// Two weight gradients in one launch where both run the exact 64 x 64 tile
// with K stage 128 (else two launches; the results are the same).
hipError_t launch_wgrad_pair(const GemmArgs& g1, int splits1, const GemmArgs& g2, int splits2, hipStream_t s,
                             int32_t* info1, int32_t* info2);

// ---- frozen inference in one launch (mlp_fused.hip) --------------------------
constexpr int kFusedHidden = 512;   // the hidden width it serves
constexpr int kFusedTile = 64;      // rows per workgroup
typedef __bf16 frag8 __attribute__((ext_vector_type(8)));
// The three weight matrices [N x K] (at params + off) in operand order.
struct FragArgs {
  const float* params;
  int64_t off[3];
  int N[3], K[3], steps[3];   // steps = ceil(K / 16)
  frag8* out[3];              // [N / 32][steps][64]
};
hipError_t launch_mlp_frag(const FragArgs& a, hipStream_t s);
struct FusedArgs {
  const __bf16* xb;          // [M x in] input, or (counters non-null) Tier 1 of rows[M] of the counters
  const float* counters;     // [N x in], 16-byte aligned
  const float* cycles;
  const int64_t* rows;
  const float* mu;
  const float* isg;
  int32_t* status;
  int in, out;
  int64_t M;
  const frag8 *w1, *w2, *w3;
  const float *b1, *b2, *b3;
  float* y;                  // [M x out] or null
  int32_t* idx_out;          // null: no ranking; as GemmArgs (out 64 or 128)
  float* score_out;
  int32_t* count_out;
  int n, skip;
  float tau;
};
// out a multiple of 32, in of 8 up to 512
hipError_t launch_mlp_fused(const FusedArgs& a, hipStream_t s);

}  // namespace sugg
