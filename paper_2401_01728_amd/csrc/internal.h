// Internal interfaces between the library's translation units (not part of the ABI).
#pragma once
#include <vector>
#include "common.h"

// ---- update.hip ------------------------------------------------------------------
// Where a weight version keeps the parameters of a flat vector: as they come, or with the four matrices of every `per_block`
// parameters in blocks of 32 columns (rv_mat).  [0, n) of a call is whole blocks then; all numbers are multiples of 64.
struct rv_ver_map {
  uint32_t per_block = 0;      // 0: as they come
  uint32_t at[4] = {0, 0, 0, 0}, rows[4] = {0, 0, 0, 0}, cols[4] = {1, 1, 1, 1};
};
// position in the version of the parameter at e = base + (less than per_block); base is the same in all lanes of a wave
__device__ __forceinline__ uint64_t rv_ver_at(const rv_ver_map& m, uint64_t base, uint64_t e) {
  uint64_t first = base / m.per_block * m.per_block;
  if (e - first >= m.per_block) first += m.per_block;
  const uint32_t r = (uint32_t)(e - first);
  uint32_t at = r;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t i = r - m.at[k];
    if (r >= m.at[k] && i < m.rows[k] * m.cols[k]) {
      const uint32_t row = i / m.cols[k], c = i - row * m.cols[k];
      at = m.at[k] + (c >> 5) * (m.rows[k] * 32) + row * 32 + (c & 31);
    }
  }
  return first + at;
}
// Workgroup -> tile of a kernel that writes versions through the map: an XCD (workgroup ids go to the 8 of them in turn) takes 32
// consecutive tiles at a time, so that the 64-byte pieces two neighbouring rows leave in one line meet in one L2.
__device__ __forceinline__ unsigned rv_ver_tile(unsigned block, unsigned blocks) {
  const unsigned whole = blocks / 256 * 256;
  return block < whole ? block / 256 * 256 + block % 8 * 32 + block % 256 / 8 : block;
}
// copy_kind: 0 none, 1 bf16 bits, 2 fp32, 3 bf16 bits through `map`; acc: the gradient is acc + g (kinds 2 and 3)
rv_status rv_launch_update(float* w, const float* g, size_t n, float eta, void* copy, int copy_kind,
                           hipStream_t st, const rv_ver_map& map = rv_ver_map(), const float* acc = nullptr);
rv_status rv_launch_update_momentum(float* w, const float* g, float* v, size_t n, float eta, float mu, float wd,
                                    void* copy, int copy_kind, hipStream_t st, const rv_ver_map& map = rv_ver_map(),
                                    const float* acc = nullptr);
rv_status rv_launch_accumulate(float* acc, const float* g, size_t n, bool first, hipStream_t st);
rv_status rv_launch_copy(float* dst, const float* src, size_t n, hipStream_t st);
// master <- w and copy <- w in the version's type
rv_status rv_launch_set(const float* w, size_t n, float* master, void* copy, int copy_kind, hipStream_t st,
                        const rv_ver_map& map);

// the RV_VER_PAD bytes at offset `at` of each of n version slots <- 0 (at: a multiple of 4)
rv_status rv_launch_clear_pads(char* const* ver, int n, size_t at, hipStream_t st);

// ---- average.hip -----------------------------------------------------------------
// rv_cluster_average with write-back, and the mean also stored to C weight versions (copy_kind)
rv_status rv_average_publish(float* const* masters, void* const* versions, int copy_kind, const rv_ver_map& map, int C, size_t n, int R,
                             const float* grad, int grad_replica, float eta, hipStream_t st);

// A bf16 matrix as the decoder keeps its own ones: element (r, c) at r * ld + (c / 32) * bs + c % 32.  Rows of pitch ld are
// bs = 32; "blocked" is ld = 32, bs = 32 * (number of rows): blocks of 32 columns, each a contiguous run of 64-byte rows, which is
// what a 32-deep tile of a matrix product reads (gemm_bf16.hip).  The matrices a product reads - the weight versions and
// the activations and gradients that are operands - are blocked; what only other kernels read, and what callers hand in or
// get, is in rows.
struct rv_mat {
  uint16_t* p;
  int64_t ld, bs;
};
__host__ __device__ inline int64_t rv_at(const rv_mat& m, int64_t r, int c) { return r * m.ld + (int64_t)(c >> 5) * m.bs + (c & 31); }
inline rv_mat rv_rows(const void* p, int64_t ld) { return {(uint16_t*)p, ld, 32}; }
inline rv_mat rv_blocks(const void* p, int64_t rows) { return {(uint16_t*)p, 32, 32 * rows}; }

// ---- gemm_bf16.hip ----------------------------------------------------------------
#include "../../include/rv_kernels.h"
struct rv_gemm_args {
  // a_bs, b_bs 32: the operand lies in rows of pitch lda, ldb; else in blocks of 32 columns (rv_mat): 32 and 32 * its rows
  const uint16_t* A = nullptr; int64_t lda = 0, a_bs = 32; int a_kmajor = 0;
  const uint16_t* B = nullptr; int64_t ldb = 0, b_bs = 32; int b_kmajor = 0;
  int M = 0, N = 0, K = 0;
  int epi = 0;
  void* out = nullptr; int64_t ldo = 0;   // primary output [M, ldo]
  void* out2 = nullptr;                   // second output, same pitch (GELU value / bf16 copy)
  // != 0 (32 M): `out` of the GELU' product, `out2` of the GELU product, upd_ver of a weight gradient in blocks of 32 columns
  int64_t bsv = 0;
  const uint16_t* bias = nullptr;         // bf16 [N]
  const float* resid = nullptr; int64_t ldr = 0;
  const uint16_t* zin = nullptr;          // bf16 [M, ldo] pre-activations for GELU'
  int tile = 0;                           // 0 = choose, else the code of a tile form
  // who else is on the chip while this product runs (automatic tile choice only):
  //   0  nobody: shortest time of this launch alone
  //   1  the other streams of a stage step, and the launch is on the step's critical chain:
  //      the 256x256 tile as soon as it covers half the chip
  //   2  the same, off the critical chain: the 256x256 tile (least CU time per flop)
  // in every case a split form instead where the rule for the shape takes one (whole_form)
  int sharing = 0;
  // weight-gradient products of the grouped launch only: the delayed update of Eq. 2 applied in
  // the epilogue.  upd_w = fp32 master tile base (same [M, ldo] layout as out), upd_ver = bf16
  // weight-version tile base; the gradient itself is stored to `out` only if store_out.
  // GELU' epilogue only: if given, fp32 [ceil(M / tile rows), ldo] (tile rows >= 32) partial column sums of the
  // output (the bias gradient of the Linear whose pre-activation gradient this is), one row per
  // tile row; the number of rows written comes back in colpart_rows
  float* colpart = nullptr;
  mutable int colpart_rows = 0;
  float* upd_w = nullptr;
  uint16_t* upd_ver = nullptr;
  float upd_eta = 0.f;
  bool store_out = true;
};
rv_status rv_gemm_bf16(const rv_gemm_args& g, hipStream_t st);
// the product cut into S stretches along K: part[S][M][N] = their sums, for a kernel that adds them
#define RV_GEMM_PARTS_MAX 8
rv_status rv_gemm_part(const rv_gemm_args& g, int S, float* part, hipStream_t st);
struct rv_part_form { int tile, S; };   // S 1: the whole product is as good
rv_part_form rv_gemm_part_form(int M, int N, int K);
// up to RV_GEMM_GROUP_MAX weight-gradient products (both operands k-major, fp32 output) in one launch; more than the four
// of one block only in the split form
#define RV_GEMM_GROUP_BLOCK 4
#define RV_GEMM_GROUP_MAX 16
#define RV_WGRAD_SPLIT_K 2048
rv_status rv_stage_update_range(rv_stage* s, size_t off, size_t n, hipStream_t st);
// RV_WGRAD_IN_ORDER: every product summed in order of k, as rv_gemm_bf16 with tile 5256 does; SPLIT: in tiles whose contraction
// is split, as with tile 1128; BY_TOKENS: the latter where the products of the launch are small and of fewer than RV_WGRAD_SPLIT_K tokens
enum rv_wgrad_form { RV_WGRAD_IN_ORDER, RV_WGRAD_SPLIT, RV_WGRAD_BY_TOKENS };
rv_status rv_gemm_wgrad_grouped(const rv_gemm_args* gs, int count, hipStream_t st, rv_wgrad_form form);
// IN_ORDER or SPLIT for count products [M[k], N[k]] over K tokens
rv_wgrad_form rv_gemm_wgrad_form(int count, const int* M, const int* N, int K);

// ---- norm.hip ---------------------------------------------------------------------
rv_status rv_ln_fwd(const void* x, int x_is_bf16, float* xcopy, const uint16_t* gamma, const uint16_t* beta,
                    rv_mat y, float* mean, float* rstd, int T, int d, float eps, hipStream_t st);
// the same of x = part[0] + .. + part[S-1] + bias + resid, which it also writes to xsum (S in {2, 4, 8}); y.p null: only xsum, and
// its bf16 rounding to out16
rv_status rv_ln_fwd_parts(const float* part, int S, const uint16_t* bias, const float* resid, float* xsum, const uint16_t* gamma,
                          const uint16_t* beta, rv_mat y, float* mean, float* rstd, uint16_t* out16, int T, int d, float eps,
                          hipStream_t st);
int rv_ln_bwd_rows(int T, int d);    // rows per workgroup of the backward: 2, 4, 8 or (d > 1024) 16
int rv_ln_bwd_parts(int T, int d);   // partial rows it writes with them (each 3*d floats)
rv_status rv_ln_bwd(const uint16_t* dy, const float* x, const float* mean, const float* rstd,
                    const uint16_t* gamma, const float* dres, float* dx, rv_mat dx_bf16, float* part,
                    int T, int d, hipStream_t st, int rows);   // (dx_bf16.p may be null)
// the same with dy = part[0] + .. + part[S-1] (S in {2, 4, 8}, fp32 [T,d] each), not rounded
rv_status rv_ln_bwd_parts_in(const float* dy_part, int S, const float* x, const float* mean, const float* rstd, const uint16_t* gamma,
                             const float* dres, float* dx, rv_mat dx_bf16, float* part, int T, int d, hipStream_t st, int rows);
// o fp32 [T,d] = a bf16 [T,d] widened, and part fp32 [rv_widen_parts(T), d] = column sums of a over
// blocks of 32 rows
int rv_widen_parts(int T);
rv_status rv_widen_colsum(const uint16_t* a, float* o, float* part, int T, int d, hipStream_t st);
// out[c] = sum_r src[r * pitch + c] for r < R, c < N, each job of a list in the same launch.  w (may be
// null) with ver: the fp32 master vector and the bf16 weight-version vector the column sums update,
// w <- w - eta * sum (Eq. 2); out null: the sums themselves are not written.
#define RV_REDUCE_MAX 36
struct rv_reduce_job {
  const float* src;
  float* out;
  float* w;
  uint16_t* ver;
  int64_t pitch;
  int R, N;
};
rv_status rv_reduce_rows(const rv_reduce_job* jobs, int njobs, float eta, hipStream_t st);

// ---- attention.hip ----------------------------------------------------------------
rv_status rv_attn_fwd(const uint16_t* qkv, rv_mat out, float* lse2, int mb, int S, int d, int H,
                      hipStream_t st);
// colpart (may be null): fp32 [mb*S/32, 3d] partial rows of the column sums of dqkv (the qkv
// bias gradient), one per (sequence, 32-token block); reduce with rv_reduce_rows
int rv_attn_colsum_parts(int mb, int S);
rv_status rv_attn_bwd(const uint16_t* qkv, rv_mat out, const uint16_t* dout, const float* lse2,
                      float* Dbuf, rv_mat dqkv, int mb, int S, int d, int H, hipStream_t st,
                      float* colpart = nullptr);

// ---- stage bookkeeping -------------------------------------------------------------
struct rv_slot {
  bool live = false;
  int64_t mb = 0;
  int ver = -1;          // weight-version slot bound at forward time
  char* base = nullptr;  // activation stash of this microbatch
};

// do [a, a + na) and [b, b + nb) bytes meet (null: no)
inline bool rv_overlap(const void* a, size_t na, const void* b, size_t nb) {
  return a && b && (const char*)a < (const char*)b + nb && (const char*)b < (const char*)a + na;
}

#define RV_VER_PAD 16   // bytes behind the parameters of every weight version; zero on an MLP stage (tiny_request_rest)

struct rv_stage {
  int kind = 0, dtype = 0, n_layers = 0, microbatch = 0, tau = 0;
  float eta = 0.f, ln_eps = 1e-5f;
  std::vector<int64_t> dims;
  hipStream_t st = nullptr;   // stream the next kernel is enqueued on (the caller's, or aux inside a step)
  hipStream_t aux = nullptr;  // second stream for the backward half of rv_stage_step
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;
  // third stream: the weight-gradient products of a decoder block run beside the next block's
  // input-gradient chain
  int upd_dst = -1;           // version slot the running backward publishes into
  bool in_step = false;       // inside rv_stage_step: forward and backward share the chip
  hipStream_t wgs = nullptr;
  hipEvent_t ev_wg_ready = nullptr, ev_wg_done[2] = {nullptr, nullptr};
  size_t P = 0;
  float* master = nullptr;  // [P] fp32
  float* grad = nullptr;    // [P] fp32, gradient of the last backward
  float* vel = nullptr;     // [P] fp32 momentum buffer (allocated by rv_stage_set_optimizer)
  float momentum = 0.f, weight_decay = 0.f;
  float* gacc = nullptr;    // [P] fp32 sum of the gradients of the current accumulation group
  int accum = 1, acc_count = 0;   // microbatches per update; backwards so far in the group
  bool defer = false;       // backward leaves its update pending (folded into the next cluster sync)
  bool keep_grad = false;   // decoder: also store the parameter gradient when the update is applied in the
                            // epilogues that produce it (rv_stage_keep_grad)
  bool fused = false;       // the running backward applies the update where the gradient is produced: plain Eq. 2,
                            // on an MLP stage the momentum form as well
  bool grad_valid = false;  // `grad` holds the whole gradient of the last backward
  size_t ver_elem = 0;      // bytes per parameter in a version slot (2 or 4)
  rv_ver_map ver_map;       // decoder: the matrices of a version lie in blocks of columns
  std::vector<char*> ver;   // tau+2 version slots: one is always free of readers, so an update can be
                            // written piece by piece while the backward still reads its own version
  std::vector<int> ver_ref; // in-flight microbatches bound to each slot
  int cur = 0;              // slot holding the newest version
  std::vector<rv_slot> slots;
  size_t slot_bytes = 0;
  char* stash = nullptr;    // (tau+1) * slot_bytes
  char* work = nullptr;     // scratch shared by all calls of this stage
  size_t work_bytes = 0;
  void* impl = nullptr;     // kind-specific plan (offsets, shapes)
  // rv_cluster_sync_fork .. join: the version slot the averaging is writing on another stream
  // (-1: none), and the stage whose ev_sync_done closes it
  int sync_dst = -1;
  rv_stage* sync_owner = nullptr;
  hipEvent_t ev_sync_ready = nullptr, ev_sync_done = nullptr;
  // rv_stage_profile: event pairs around every launch of the block's grouped weight-gradient
  // product, on the stream it is launched on
  bool prof_on = false;
  std::vector<hipEvent_t> prof_ev;   // start, stop, start, stop, ...
};

// ---- mlp.hip -----------------------------------------------------------------------
rv_status rv_mlp_plan(rv_stage* s);   // fills P, slot_bytes, work_bytes, impl
void rv_mlp_free(rv_stage* s);
rv_status rv_mlp_forward(rv_stage* s, rv_slot& slot, const void* in, void* out);
rv_status rv_mlp_backward(rv_stage* s, rv_slot& slot, const void* grad_out, void* grad_in);

// ---- decoder.hip -------------------------------------------------------------------
rv_status rv_dec_plan(rv_stage* s);
bool rv_dec_less_work(rv_stage* s);   // plan a smaller work buffer (work_bytes), if there is one; nothing may be on the way
void rv_dec_free(rv_stage* s);
// what the kernels of a forward, of a backward would refuse, to be asked before a microbatch is admitted or anything is enqueued
bool rv_dec_takes_forward(const rv_stage* s);
bool rv_dec_takes_backward(const rv_stage* s, const void* grad_out, const void* grad_in);
rv_status rv_dec_forward(rv_stage* s, rv_slot& slot, const void* in, void* out);
rv_status rv_dec_backward(rv_stage* s, rv_slot& slot, const void* grad_out, void* grad_in);
rv_status rv_dec_step(rv_stage* s, rv_slot& fwd, const void* in, void* out, rv_slot& bwd, const void* grad_out, void* grad_in);
