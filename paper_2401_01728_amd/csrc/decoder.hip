// Decoder stage: L pre-LayerNorm transformer blocks as one peer's forward_pass and its
// exact gradient at the stashed weight version (paper Alg. 1; Eq. 2).  Host-side
// sequencing only; the work is in gemm_bf16.hip, attention.hip and norm.hip.
//
//   u  = LN1(x);  qkv = u Wqkv + bqkv;  a = CausalSoftmax(q k^T / sqrt(dh)) v
//   x1 = x + a Wo + bo;   v2 = LN2(x1);  z = v2 W1 + b1;  g = GELU(z);  y = x1 + g W2 + b2
//
// The residual stream (x, x1, y) and its gradient are fp32 inside the stage; matrix
// product operands are bf16.  Per microbatch and block the stash keeps x, x1 (fp32), the
// LN statistics, u, qkv, a, v2, z, g (bf16) and the softmax log-sums: everything the
// backward reads, so nothing is recomputed except the attention probabilities.
#include <algorithm>
#include <new>
#include "internal.h"

namespace {

size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

struct DecPlan {
  int L, d, H, f, S, mb, T;
  // element offsets inside one block's parameters (same in the fp32 master and the bf16 version)
  size_t ln1g, ln1b, wqkv, bqkv, wo, bo, ln2g, ln2b, w1, b1, w2, b2, per_block;
  // byte offsets inside one block's stash
  size_t s_x, s_m1, s_r1, s_u, s_qkv, s_a, s_lse, s_x1, s_m2, s_r2, s_v2, s_z, s_g, blk_bytes;
  // byte offsets inside the work buffer.  What a block's side work reads (dy, dx1, dz, dqkv and the partial rows of the
  // column sums) alternates between `sets` sets, so that it can run beside the blocks below: block l uses set l % sets,
  // its dy buffer l % (sets + 1) (block l - 1 writes the dy of block l - 2 while the side work of block l still reads
  // its own).  deep: a set for every block, nothing is overwritten within a backward.
  bool deep;
  int sets, dy_sets, group;   // group: blocks whose side work goes out together (deep only)
  bool early;                 // the feed-forward pair of the weight-gradient products leaves ahead of the other two (begin)
  rv_wgrad_form wgrad, wgrad_last;   // of a block's products; of the two that leave last by themselves, of the first block
  size_t w_dres, w_dtmp, w_D, w_part_dy, w_ytmp;
  // products whose contraction is cut over workgroups, the LayerNorm behind them adding the pieces (S 1: none), and where
  // the pieces go: those of the forward and of the backward apart, a step runs both at once
  rv_part_form f_wo, f_w2, b_w1, b_wqkv;
  size_t w_pf, w_pb;
  size_t w_dy, dy_bytes;                                                   // dy buffers: w_dy + i * dy_bytes
  size_t w_set, set_bytes;                                                 // sets: w_set + i * set_bytes, and in a set
  size_t o_dx1_16, o_dz, o_dqkv, o_part_ln[2], o_part_dz, o_part_qkv;
};

// A stage whose sets for every block fit in this many bytes gets them (deep).
constexpr size_t kDeepBytes = 512u << 20;
constexpr int kCUs = 256;
int tiles256(int M, int N) { return ((M + 255) / 256) * ((N + 255) / 256); }
constexpr int kGroupBlocks = RV_GEMM_GROUP_MAX / 4;
static_assert(9 * kGroupBlocks <= RV_REDUCE_MAX, "the column sums of a group fit in one launch");

// the work buffer, with a set of buffers for every block or with alternating ones
void plan_work(rv_stage* s, DecPlan* p, bool deep) {
  const size_t T = p->T, d = p->d;
  p->deep = deep;
  p->sets = deep ? p->L : 2;
  p->dy_sets = deep ? p->L : 3;
  p->group = 1;
  if (p->deep && p->wgrad == RV_WGRAD_SPLIT && p->T < RV_WGRAD_SPLIT_K) {
    // A block whose products do not give every CU a tile leaves with three others: a launch is a few microseconds, and the
    // event pair in front of it 11 of host time, however small it is.  Stage step of 12 blocks of d 448 (172 tiles) on
    // 256 tokens, two / three / four blocks at a time, 815 / 785 / 745 us.  Blocks that fill the chip lose by waiting for each other:
    // d 896 (448 tiles), 256 tokens, one / three at a time 400 / 407, d 832 in separate calls 1398 / 1422.
    auto tiles = [](int64_t M, int64_t N) { return ((M + 127) / 128) * ((N + 127) / 128); };
    if (2 * tiles(p->d, p->f) + tiles(p->d, p->d) + tiles(p->d, 3 * p->d) < 256) p->group = kGroupBlocks;
  }
  size_t w = 0;
  p->w_dres = w; w += align_up(T * d * 4);
  p->w_dtmp = w; w += align_up(T * d * 2);
  p->w_D = w; w += align_up(T * p->H * 4);
  p->w_part_dy = w; w += align_up((size_t)rv_widen_parts(p->T) * d * 4);   // of the arriving gradient (32-row blocks)
  p->w_ytmp = w; w += align_up(T * d * 4);
  p->f_wo = rv_gemm_part_form(p->T, p->d, p->d); p->f_w2 = rv_gemm_part_form(p->T, p->d, p->f);
  p->b_w1 = rv_gemm_part_form(p->T, p->d, p->f); p->b_wqkv = rv_gemm_part_form(p->T, p->d, 3 * p->d);
  auto most = [](const rv_part_form& a, const rv_part_form& b) { const int S = a.S > b.S ? a.S : b.S; return (size_t)(S > 1 ? S : 0); };
  p->w_pf = w; w += align_up(most(p->f_wo, p->f_w2) * T * d * 4);
  p->w_pb = w; w += align_up(most(p->b_w1, p->b_wqkv) * T * d * 4);
  p->w_dy = w; w += p->dy_bytes * p->dy_sets;
  p->w_set = w; w += p->set_bytes * p->sets;
  s->work_bytes = w;
}

}  // namespace

rv_status rv_dec_plan(rv_stage* s) {
  const int64_t d = s->dims[0], H = s->dims[1], f = s->dims[2], S = s->dims[3];
  if (d < 64 || d > 4096 || d % 64 || H < 1 || d % H || f < 64 || f % 64 || f > (1 << 16) || S < 64 ||
      S % 64 || S > (1 << 16))
    return RV_E_INVAL;
  const int64_t dh = d / H;
  if (dh != 64 && dh != 128) return RV_E_INVAL;
  if ((int64_t)s->microbatch * S > (1 << 24)) return RV_E_INVAL;
  DecPlan* p = new (std::nothrow) DecPlan();
  if (!p) return RV_E_NOMEM;
  s->impl = p;
  p->L = s->n_layers; p->d = (int)d; p->H = (int)H; p->f = (int)f; p->S = (int)S; p->mb = s->microbatch;
  p->T = p->mb * p->S;
  size_t o = 0;
  p->ln1g = o; o += d; p->ln1b = o; o += d;
  p->wqkv = o; o += (size_t)d * 3 * d; p->bqkv = o; o += 3 * d;
  p->wo = o; o += (size_t)d * d; p->bo = o; o += d;
  p->ln2g = o; o += d; p->ln2b = o; o += d;
  p->w1 = o; o += (size_t)d * f; p->b1 = o; o += f;
  p->w2 = o; o += (size_t)f * d; p->b2 = o; o += d;
  p->per_block = o;
  const int pm[4] = {p->f, p->d, p->d, p->d}, pn[4] = {p->d, p->f, p->d, 3 * p->d};   // dW2, dW1, dWo, dWqkv
  p->early = 2 * tiles256(p->d, p->f) >= kCUs;
  // (a launch of an early block that does not fill the chip is split on few tokens by itself)
  p->wgrad = p->early ? RV_WGRAD_BY_TOKENS : rv_gemm_wgrad_form(4, pm, pn, p->T);
  // (stage step of 4 blocks of d 1024, 4096 tokens, these 64 tiles split / in order 1789 / 1817 us)
  p->wgrad_last = rv_gemm_wgrad_form(2, pm + 2, pn + 2, p->T);
  s->P = o * p->L;
  // the matrices of a weight version lie in blocks of 32 columns
  const size_t at[4] = {p->wqkv, p->wo, p->w1, p->w2};
  const int64_t rows[4] = {d, d, d, f}, cols[4] = {3 * d, d, f, d};
  s->ver_map.per_block = (uint32_t)o;
  for (int k = 0; k < 4; ++k) { s->ver_map.at[k] = (uint32_t)at[k]; s->ver_map.rows[k] = (uint32_t)rows[k]; s->ver_map.cols[k] = (uint32_t)cols[k]; }
  const size_t T = p->T;
  size_t b = 0;
  p->s_x = b; b += align_up(T * d * 4);
  p->s_m1 = b; b += align_up(T * 4); p->s_r1 = b; b += align_up(T * 4);
  p->s_u = b; b += align_up(T * d * 2);
  p->s_qkv = b; b += align_up(T * 3 * d * 2);
  p->s_a = b; b += align_up(T * d * 2);
  p->s_lse = b; b += align_up(T * H * 4);
  p->s_x1 = b; b += align_up(T * d * 4);
  p->s_m2 = b; b += align_up(T * 4); p->s_r2 = b; b += align_up(T * 4);
  p->s_v2 = b; b += align_up(T * d * 2);
  p->s_z = b; b += align_up(T * f * 2);
  p->s_g = b; b += align_up(T * f * 2);
  p->blk_bytes = b;
  s->slot_bytes = b * p->L;
  // one set; partial rows of the bias gradients: of dz (one per tile row of the product that makes it, at least 32 rows)
  // and of dqkv (32-token blocks)
  const size_t part_ln = (size_t)rv_ln_bwd_parts(p->T, d) * 3 * d;
  size_t q = 0;
  p->o_dx1_16 = q; q += align_up(T * d * 2);
  p->o_dz = q; q += align_up(T * f * 2);
  p->o_dqkv = q; q += align_up(T * 3 * d * 2);
  for (size_t& o : p->o_part_ln) { o = q; q += align_up(part_ln * 4); }
  p->o_part_dz = q; q += align_up((size_t)((T + 31) / 32) * f * 4);
  p->o_part_qkv = q; q += align_up((size_t)rv_attn_colsum_parts(p->mb, p->S) * 3 * d * 4);
  p->set_bytes = q;
  p->dy_bytes = align_up(T * d * 2);
  plan_work(s, p, (size_t)p->L * (p->set_bytes + p->dy_bytes) <= kDeepBytes);
  return RV_OK;
}

bool rv_dec_less_work(rv_stage* s) {
  DecPlan* p = (DecPlan*)s->impl;
  if (!p->deep) return false;
  const size_t had = s->work_bytes;
  plan_work(s, p, false);
  if (s->work_bytes < had) return true;
  plan_work(s, p, true);   // (one or two blocks: the alternating sets are more)
  return false;
}

void rv_dec_free(rv_stage* s) {
  delete (DecPlan*)s->impl;
  s->impl = nullptr;
}

namespace {

// out = A B: A [M,K], B a weight [K,N] (wt 0) or its transpose, W [N,K] (wt 1); the outputs that are operands
// later, GELU(z) and dz, leave in blocks of columns
rv_status gemm(int sharing, hipStream_t st, rv_mat A, const void* W, int wt, int M, int N, int K, int epi, void* out, int64_t ldo,
               void* out2 = nullptr, const void* bias = nullptr, const float* resid = nullptr, const void* zin = nullptr,
               float* colpart = nullptr, int* colpart_rows = nullptr) {
  rv_gemm_args g;
  g.colpart = colpart;
  g.sharing = sharing;
  g.A = A.p; g.lda = A.ld; g.a_bs = A.bs;
  const rv_mat B = rv_blocks(W, wt ? N : K);
  g.B = B.p; g.ldb = B.ld; g.b_bs = B.bs; g.b_kmajor = !wt;
  g.M = M; g.N = N; g.K = K; g.epi = epi; g.out = out; g.ldo = ldo; g.out2 = out2;
  if (epi == RV_EPI_BF16_BIAS_GELU || epi == RV_EPI_BF16_DGELU) g.bsv = (int64_t)M * 32;
  g.bias = (const uint16_t*)bias; g.resid = resid; g.ldr = ldo; g.zin = (const uint16_t*)zin;
  const rv_status rc = rv_gemm_bf16(g, st);
  if (colpart_rows) *colpart_rows = g.colpart_rows;
  return rc;
}

rv_status gemm_part(const rv_part_form& form, hipStream_t st, rv_mat A, const void* W, int wt, int M, int N, int K, float* part) {
  rv_gemm_args g;
  g.A = A.p; g.lda = A.ld; g.a_bs = A.bs;
  const rv_mat B = rv_blocks(W, wt ? N : K);
  g.B = B.p; g.ldb = B.ld; g.b_bs = B.bs; g.b_kmajor = !wt;
  g.M = M; g.N = N; g.K = K; g.tile = form.tile;
  return rv_gemm_part(g, form.S, part, st);
}

// the forward of block l of one microbatch, on st
rv_status forward_block(const rv_stage* s, const rv_slot& slot, const void* in, void* out, int l, hipStream_t st) {
  const DecPlan& p = *(const DecPlan*)s->impl;
  const int T = p.T, d = p.d, f = p.f;
  const int sh = s->in_step ? 2 : 0;   // in a step the backward chain is the longer one
  const uint16_t* w = (const uint16_t*)s->ver[slot.ver] + (size_t)l * p.per_block;
  char* sb = slot.base + (size_t)l * p.blk_bytes;
  float* x = (float*)(sb + p.s_x);
  float* x1 = (float*)(sb + p.s_x1);
  const rv_mat u = rv_blocks(sb + p.s_u, T);
  uint16_t* qkv = (uint16_t*)(sb + p.s_qkv);
  const rv_mat a = rv_blocks(sb + p.s_a, T);
  const rv_mat v2 = rv_blocks(sb + p.s_v2, T);
  uint16_t* z = (uint16_t*)(sb + p.s_z);
  const rv_mat g = rv_blocks(sb + p.s_g, T);
  float* pf = (float*)(s->work + p.w_pf);
  if (l == 0)
    RV_TRY(rv_ln_fwd(in, 1, x, w + p.ln1g, w + p.ln1b, u, (float*)(sb + p.s_m1), (float*)(sb + p.s_r1), T, d, s->ln_eps, st));
  else if (p.f_w2.S > 1)   // (x is what it adds up)
    RV_TRY(rv_ln_fwd_parts(pf, p.f_w2.S, w - p.per_block + p.b2, (const float*)(sb - p.blk_bytes + p.s_x1), x, w + p.ln1g, w + p.ln1b, u,
                           (float*)(sb + p.s_m1), (float*)(sb + p.s_r1), nullptr, T, d, s->ln_eps, st));
  else
    RV_TRY(rv_ln_fwd(x, 0, nullptr, w + p.ln1g, w + p.ln1b, u, (float*)(sb + p.s_m1), (float*)(sb + p.s_r1), T, d,
                     s->ln_eps, st));
  RV_TRY(gemm(sh, st, u, w + p.wqkv, 0, T, 3 * d, d, RV_EPI_BF16_BIAS, qkv, 3 * d, nullptr, w + p.bqkv));
  RV_TRY(rv_attn_fwd(qkv, a, (float*)(sb + p.s_lse), p.mb, p.S, d, p.H, st));
  if (p.f_wo.S > 1) {
    RV_TRY(gemm_part(p.f_wo, st, a, w + p.wo, 0, T, d, d, pf));
    RV_TRY(rv_ln_fwd_parts(pf, p.f_wo.S, w + p.bo, x, x1, w + p.ln2g, w + p.ln2b, v2, (float*)(sb + p.s_m2), (float*)(sb + p.s_r2),
                           nullptr, T, d, s->ln_eps, st));
  } else {
    RV_TRY(gemm(sh, st, a, w + p.wo, 0, T, d, d, RV_EPI_F32_BIAS_RESID, x1, d, nullptr, w + p.bo, x));
    RV_TRY(rv_ln_fwd(x1, 0, nullptr, w + p.ln2g, w + p.ln2b, v2, (float*)(sb + p.s_m2), (float*)(sb + p.s_r2), T, d,
                     s->ln_eps, st));
  }
  RV_TRY(gemm(sh, st, v2, w + p.w1, 0, T, f, d, RV_EPI_BF16_BIAS_GELU, z, f, g.p, w + p.b1));
  if (p.f_w2.S > 1) {
    RV_TRY(gemm_part(p.f_w2, st, g, w + p.w2, 0, T, d, f, pf));
    if (l + 1 < p.L) return RV_OK;   // the next block's LayerNorm adds the pieces
    return rv_ln_fwd_parts(pf, p.f_w2.S, w + p.b2, x1, nullptr, nullptr, nullptr, rv_mat{}, nullptr, nullptr, (uint16_t*)out, T, d,
                           s->ln_eps, st);
  }
  if (l + 1 < p.L) {
    float* xn = (float*)(slot.base + (size_t)(l + 1) * p.blk_bytes + p.s_x);
    return gemm(sh, st, g, w + p.w2, 0, T, d, f, RV_EPI_F32_BIAS_RESID, xn, d, nullptr, w + p.b2, x1);
  }
  return gemm(sh, st, g, w + p.w2, 0, T, d, f, RV_EPI_F32_BIAS_RESID_BF16, s->work + p.w_ytmp, d, out, w + p.b2, x1);
}

// The backward of one microbatch, issued block by block from the last: begin, block(L-1) .. block(0), end.
//
// Everything that only feeds the parameter gradient - the four weight-gradient products of a
// block, the reductions behind the bias and LayerNorm gradients, the block's delayed update -
// is side work: nothing in the chain dy -> dx that the block below waits for reads it.  It
// goes to a stream of its own and runs beside the next block's chain (measured step time
// against issuing it in line: d 1024 -7 %, d 2048 -1 %, d 1600 -5 %).
//
// The host's part in this: a launch takes 2.7 us to issue, making the side stream wait for the chain 11 us (record 1.5,
// wait 9 .. 10).  A small stage is bounded by that, so where every block has buffers of its own (deep) the side stream is
// made to wait once per launch of products, the column sums behind the last LayerNorm of a block ride with those
// of the next, and no wait guards the reuse of a buffer.  Stage step of 12 blocks of d 448 on 256 tokens 1193 -> 924 us
// (with forward and backward issued in turn, see rv_dec_step); bounded by the device, 4 blocks of d 1024 on 128 tokens
// forward and backward 0.70 -> 0.69 ms, on 4096 tokens the same.
struct Backward {
  rv_stage* s;
  const DecPlan& p;
  const rv_slot& slot;
  const void* grad_out;
  void* grad_in;
  hipStream_t st, ws;          // the chain's stream, the side stream
  int sh;
  uint16_t* vdst = nullptr;
  rv_mat dres16 = {};   // bf16 gradient of the current block's output
  // the side work that has come into being and not left yet
  rv_reduce_job sums[RV_REDUCE_MAX];
  rv_gemm_args prods[RV_GEMM_GROUP_MAX];
  int n_sums = 0, n_prods = 0;
  bool early;
  int wg_pos[4] = {2, 2, 2, 2};   // launch points (see begin) of dW2, dW1, dWo, dWqkv
  int whole = 0;                  // blocks below this one (and it) still lack part of their gradient: updates done down to it

  Backward(rv_stage* s_, const rv_slot& slot_, const void* go, void* gi, hipStream_t st_)
      : s(s_), p(*(const DecPlan*)s_->impl), slot(slot_), grad_out(go), grad_in(gi), st(st_), ws(s_->wgs),
        sh(s_->in_step ? 1 : 0), early(p.early) {}

  uint16_t* dy_buf(int l) const { return (uint16_t*)(s->work + p.w_dy + (size_t)(l % p.dy_sets) * p.dy_bytes); }
  char* set(int l) const { return s->work + p.w_set + (size_t)(l % p.sets) * p.set_bytes; }

  rv_status side_begin() {
    RV_HIP_TRY(hipEventRecord(s->ev_wg_ready, st));
    RV_HIP_TRY(hipStreamWaitEvent(ws, s->ev_wg_ready, 0));
    return RV_OK;
  }
  // The column sums of a block (bias and LayerNorm-affine gradients) are listed as their partial
  // rows come into being.  fused update (plain Eq. 2): every kernel that completes a parameter gradient applies it at
  // once to the fp32 master and writes the bf16 rounding into the new weight version `vdst`
  void colsum(const float* part, int rows, int64_t pitch, int n, float* dst) {
    const size_t off = (size_t)(dst - s->grad);
    sums[n_sums++] = rv_reduce_job{part, !s->fused || s->keep_grad ? dst : nullptr, s->fused ? s->master + off : nullptr,
                                   s->fused ? vdst + off : nullptr, pitch, rows, n};
  }
  rv_status send_sums(hipStream_t to) {
    const int n = n_sums;
    n_sums = 0;
    return n ? rv_reduce_rows(sums, n, s->eta, to) : RV_OK;
  }
  rv_status send_prods(rv_wgrad_form form) {
    const int n = n_prods;
    n_prods = 0;
    if (!n) return RV_OK;
    if (s->prof_on) {   // measurement aid: bracket the launch with events on its own stream
      hipEvent_t e0 = nullptr, e1 = nullptr;
      RV_HIP_TRY(hipEventCreate(&e0));
      s->prof_ev.push_back(e0);
      RV_HIP_TRY(hipEventCreate(&e1));
      s->prof_ev.push_back(e1);
      RV_HIP_TRY(hipEventRecord(e0, ws));
      RV_TRY(rv_gemm_wgrad_grouped(prods, n, ws, form));
      RV_HIP_TRY(hipEventRecord(e1, ws));
      return RV_OK;
    }
    return rv_gemm_wgrad_grouped(prods, n, ws, form);
  }
  // blocks l .. whole - 1 have their whole gradient: unless the epilogues have applied it already, their delayed update
  rv_status update_from(int l, hipStream_t to) {
    const int n = whole - l;
    whole = l;
    if (s->fused || n <= 0) return RV_OK;
    return rv_stage_update_range(s, (size_t)l * p.per_block, (size_t)n * p.per_block, to);
  }

  // dy = A W^T (A [T,K], W [d,K]) and the backward of the LayerNorm in front of that Linear, joined with the residual branch
  rv_status product_and_norm(const rv_part_form& form, rv_mat A, const uint16_t* W, int K, const float* x, const float* mean,
                             const float* rstd, const uint16_t* gamma, rv_mat dx16, float* part) {
    const int T = p.T, d = p.d, rows = rv_ln_bwd_rows(T, d);
    float* dres = (float*)(s->work + p.w_dres);
    if (form.S > 1) {
      float* pb = (float*)(s->work + p.w_pb);
      RV_TRY(gemm_part(form, st, A, W, 1, T, d, K, pb));
      return rv_ln_bwd_parts_in(pb, form.S, x, mean, rstd, gamma, dres, dres, dx16, part, T, d, st, rows);
    }
    uint16_t* dtmp = (uint16_t*)(s->work + p.w_dtmp);
    RV_TRY(gemm(sh, st, A, W, 1, T, d, K, RV_EPI_BF16, dtmp, d));
    return rv_ln_bwd(dtmp, x, mean, rstd, gamma, dres, dres, dx16, part, T, d, st, rows);
  }

  rv_status begin() {
    vdst = s->fused ? (uint16_t*)s->ver[s->upd_dst] : nullptr;
    whole = p.L;
    const int T = p.T, d = p.d;
    // gradient of the last block's output: fp32 copy for the residual path, bf16 as operand
    // (summed over tokens it is also the gradient of the last block's b2: partial sums on the way)
    float* part_dy = (float*)(s->work + p.w_part_dy);
    dres16 = rv_rows(grad_out, d);
    if (rv_overlap(grad_out, (size_t)T * d * 2, grad_in, (size_t)T * d * 2)) {
      // the first block's backward writes grad_in without waiting for the side stream, where the last block's dW2
      // still reads the arriving gradient: that goes to its place among the gradients of the other blocks first
      uint16_t* dy = dy_buf(p.L - 1);
      RV_HIP_TRY(hipMemcpyAsync(dy, grad_out, (size_t)T * d * 2, hipMemcpyDeviceToDevice, st));
      dres16 = rv_rows(dy, d);
    }
    RV_TRY(rv_widen_colsum(dres16.p, (float*)(s->work + p.w_dres), part_dy, T, d, st));
    colsum(part_dy, rv_widen_parts(T), d, d, s->grad + (size_t)(p.L - 1) * p.per_block + p.b2);
    // When the four weight-gradient products of a block go to the side stream.  Launch points:
    // 0 behind the GELU' product (dz exists: dW2 and dW1 can run), 1 behind the second LayerNorm's
    // backward (dx1 exists: dWo), 2 behind the attention backward (dqkv exists: all four).  One
    // launch of all four at point 2 is the least launch work; going out earlier puts the products
    // beside the chain's LayerNorm and attention kernels instead of beside its next products.
    // Measured step time against the single launch, tiles of 256 x 256 on 256 CUs:
    //   dW2 + dW1 at point 0, dWo + dWqkv at point 2:  -4.7 % where they are 512 and 256 tiles
    //   (d 2048, ffn 8192), 0 % at 350 and 182 tiles (d 1600, ffn 6400), +1.3 % at 128 and 64 tiles
    //   (d 1024, ffn 4096);
    //   dWo on its own at point 1 as well:  -2.8 %, -1.2 %, +7 % in the same order.
    // So: the feed-forward pair goes out early when it fills the chip at least once, and dWo leaves
    // dWqkv only when the two together are not a whole number of rounds anyway.  (All four behind the
    // first LayerNorm's backward, one event pair less per block: +4 % at d 2048, d 1024 and 6 blocks of
    // d 768 on 1152 tokens.)
    if (early) {
      wg_pos[0] = wg_pos[1] = 0;
      if (!p.deep && (tiles256(p.d, p.d) + tiles256(p.d, 3 * p.d)) % kCUs != 0) wg_pos[2] = 1;
    }
    return RV_OK;
  }

  rv_status block(int l) {
    const int T = p.T, d = p.d, f = p.f, par = l & 1;
    uint16_t* dtmp = (uint16_t*)(s->work + p.w_dtmp);
    float* Dbuf = (float*)(s->work + p.w_D);
    const int ln_parts = rv_ln_bwd_parts(T, d);
    // block l may overwrite what the side work of block l+2 read only after that is done
    if (!p.deep && l + 2 < p.L) RV_HIP_TRY(hipStreamWaitEvent(st, s->ev_wg_done[par], 0));
    char* set_l = set(l);
    const rv_mat dx1_16 = rv_blocks(set_l + p.o_dx1_16, T);      // bf16 dx1 of this block
    const rv_mat dz = rv_blocks(set_l + p.o_dz, T);
    const rv_mat dqkv = rv_blocks(set_l + p.o_dqkv, T);
    float* part2 = (float*)(set_l + p.o_part_ln[0]);             // LayerNorm 2 / 1 partial sums
    float* part1 = (float*)(set_l + p.o_part_ln[1]);
    const uint16_t* w = (const uint16_t*)s->ver[slot.ver] + (size_t)l * p.per_block;
    float* gl = s->grad + (size_t)l * p.per_block;
    const char* sb = slot.base + (size_t)l * p.blk_bytes;
    const float* x = (const float*)(sb + p.s_x);
    const float* x1 = (const float*)(sb + p.s_x1);
    const rv_mat u = rv_blocks(sb + p.s_u, T);
    const uint16_t* qkv = (const uint16_t*)(sb + p.s_qkv);
    const rv_mat a = rv_blocks(sb + p.s_a, T);
    const rv_mat v2 = rv_blocks(sb + p.s_v2, T);
    const uint16_t* z = (const uint16_t*)(sb + p.s_z);
    const rv_mat g = rv_blocks(sb + p.s_g, T);
    rv_gemm_args wg[4];
    auto wgrad = [&](int k, rv_mat A, rv_mat B, int M, int N, float* out) {
      wg[k].A = A.p; wg[k].lda = A.ld; wg[k].a_bs = A.bs; wg[k].a_kmajor = 1;
      wg[k].B = B.p; wg[k].ldb = B.ld; wg[k].b_bs = B.bs; wg[k].b_kmajor = 1;
      wg[k].M = M; wg[k].N = N; wg[k].K = T; wg[k].epi = RV_EPI_F32; wg[k].out = out; wg[k].ldo = N;
      if (s->fused) {   // Eq. 2 in the product's epilogue: master and new weight version at the same offset
        const size_t off = (size_t)(out - s->grad);
        wg[k].upd_w = s->master + off; wg[k].upd_ver = vdst + off; wg[k].bsv = (int64_t)M * 32; wg[k].upd_eta = s->eta;
        wg[k].store_out = s->keep_grad;
      }
    };
    // the weight-gradient products whose launch point is `pos` join the list
    // (the stage's first block, the last of the chain, has nothing to run beside: its feed-forward pair leaves early where a
    // block's products go out by themselves, and what is left at the end is a third: with the last sums on the chain's stream
    // four microbatches of 6 blocks of d 768, 1152 tokens 5451 -> 5345 us, stage step of 4 of d 1024, 4096 tokens 1812 -> 1773)
    const bool pair_first = early || (p.deep && p.group == 1 && l == 0);
    auto take = [&](int pos) {
      for (int k = 0; k < 4; ++k)
        if ((k < 2 && pair_first ? 0 : wg_pos[k]) == pos) prods[n_prods++] = wg[k];
    };
    // Where the listed side work leaves.  One buffer set per block: the products at points 0 and 2 (2 of every group-th
    // block where the group has several), each time with the sums listed so far - a block's last sums with the
    // next launch.  Alternating sets: the products as above, the sums of a block in one launch at its end (with four
    // launches per block, each behind an event pair of its own, the host bounded small stages), or along with the
    // products where those leave early (one launch at the end made the stage step 0.8 % longer at 12 blocks of
    // d 1600, 8192 tokens).
    const bool leaves = !p.deep || l % p.group == 0;
    // feed-forward half
    wgrad(0, g, dres16, f, d, gl + p.w2);                                                      // dW2 = g^T dy
    // dz = (dy W2^T) * GELU'(z); its column sums (the b1 gradient) leave the same epilogue as partial rows
    float* part_dz = (float*)(set_l + p.o_part_dz);
    int dz_parts = 0;
    RV_TRY(gemm(sh, st, dres16, w + p.w2, 1, T, f, d, RV_EPI_BF16_DGELU, dz.p, f, nullptr, nullptr, nullptr, z,
                part_dz, &dz_parts));
    wgrad(1, v2, dz, d, f, gl + p.w1);                                                         // dW1 = v2^T dz
    colsum(part_dz, dz_parts, f, f, gl + p.b1);
    take(0);
    if (pair_first && leaves) {
      RV_TRY(side_begin());
      RV_TRY(send_prods(p.wgrad));
      RV_TRY(send_sums(ws));
      if (p.deep) RV_TRY(update_from(l + 1, ws));
    }
    // dv2 = dz W1^T
    RV_TRY(product_and_norm(p.b_w1, dz, w + p.w1, f, x1, (const float*)(sb + p.s_m2), (const float*)(sb + p.s_r2), w + p.ln2g, dx1_16,
                            part2));
    colsum(part2, ln_parts, 3 * (int64_t)d, d, gl + p.ln2g);
    colsum(part2 + d, ln_parts, 3 * (int64_t)d, d, gl + p.ln2b);
    colsum(part2 + 2 * d, ln_parts, 3 * (int64_t)d, d, gl + p.bo);                                     // dbo = sum dx1
    // attention half
    wgrad(2, a, dx1_16, d, d, gl + p.wo);                                                      // dWo = a^T dx1
    take(1);
    if (early && !p.deep) {
      RV_TRY(side_begin());
      RV_TRY(send_sums(ws));
      RV_TRY(send_prods(p.wgrad));
    }
    RV_TRY(gemm(sh, st, dx1_16, w + p.wo, 1, T, d, d, RV_EPI_BF16, dtmp, d));                   // da = dx1 Wo^T
    // (the attention backward also leaves partial column sums of dqkv: the qkv bias gradient)
    float* part_qkv = (float*)(set_l + p.o_part_qkv);
    RV_TRY(rv_attn_bwd(qkv, a, dtmp, (const float*)(sb + p.s_lse), Dbuf, dqkv, p.mb, p.S, d, p.H, st, part_qkv));
    wgrad(3, u, dqkv, d, 3 * d, gl + p.wqkv);                                              // dWqkv = u^T dqkv
    colsum(part_qkv, rv_attn_colsum_parts(p.mb, p.S), 3 * d, 3 * d, gl + p.bqkv);
    take(2);
    if (leaves) {
      RV_TRY(side_begin());
      RV_TRY(send_prods(l == 0 && pair_first && !early ? p.wgrad_last : p.wgrad));
      if (early || p.deep) RV_TRY(send_sums(ws));
      if (p.deep) RV_TRY(update_from(l + 1, ws));   // (block l lacks what its last LayerNorm gives)
    }
    const rv_mat dy_below = l > 0 ? rv_blocks(dy_buf(l - 1), T) : rv_rows(grad_in, d);
    // du
    RV_TRY(product_and_norm(p.b_wqkv, dqkv, w + p.wqkv, 3 * d, x, (const float*)(sb + p.s_m1), (const float*)(sb + p.s_r1), w + p.ln1g,
                            dy_below, part1));
    colsum(part1, ln_parts, 3 * (int64_t)d, d, gl + p.ln1g);
    colsum(part1 + d, ln_parts, 3 * (int64_t)d, d, gl + p.ln1b);
    // the residual gradient leaving this block is dy of the block below: its b2 gradient
    if (l > 0) colsum(part1 + 2 * d, ln_parts, 3 * (int64_t)d, d, s->grad + (size_t)(l - 1) * p.per_block + p.b2);
    dres16 = dy_below;
    if (p.deep) {
      if (l > 0) return RV_OK;
      // the last sums are the chain's own, behind it on its stream: no hop to the side stream and back
      RV_HIP_TRY(hipEventRecord(s->ev_wg_done[0], ws));
      RV_TRY(send_sums(st));
      RV_HIP_TRY(hipStreamWaitEvent(st, s->ev_wg_done[0], 0));
      return update_from(0, st);
    }
    RV_TRY(side_begin());
    RV_TRY(send_sums(ws));
    // every gradient of block l is complete behind this point of `ws` (its b2 gradient came from the block above)
    RV_TRY(update_from(l, ws));
    RV_HIP_TRY(hipEventRecord(s->ev_wg_done[par], ws));
    return RV_OK;
  }

  // the chain's stream (and with it the caller's) continues behind the last side work
  rv_status end() {
    if (p.deep) return RV_OK;   // block(0) has seen to it
    RV_HIP_TRY(hipStreamWaitEvent(st, s->ev_wg_done[0], 0));
    if (p.L > 1) RV_HIP_TRY(hipStreamWaitEvent(st, s->ev_wg_done[1], 0));
    return RV_OK;
  }
};

}  // namespace

// Matrix products address an operand in 32 bits (T * f: also GELU(z) and dz).
bool rv_dec_takes_forward(const rv_stage* s) {
  const DecPlan& p = *(const DecPlan*)s->impl;
  return (int64_t)p.T * std::max(p.d, p.f) < (1ll << 31);
}
// The arriving gradient is such an operand where it lies, and begins at 16 bytes then; one that shares memory with grad_in is
// copied first.
bool rv_dec_takes_backward(const rv_stage* s, const void* grad_out, const void* grad_in) {
  const DecPlan& p = *(const DecPlan*)s->impl;
  const size_t bytes = (size_t)p.T * p.d * 2;
  return (int64_t)p.T * std::max(3 * p.d, p.f) < (1ll << 31) &&
         (((uintptr_t)grad_out & 15) == 0 || rv_overlap(grad_out, bytes, grad_in, bytes));
}

rv_status rv_dec_forward(rv_stage* s, rv_slot& slot, const void* in, void* out) {
  const int L = ((const DecPlan*)s->impl)->L;
  for (int l = 0; l < L; ++l) RV_TRY(forward_block(s, slot, in, out, l, s->st));
  return RV_OK;
}

rv_status rv_dec_backward(rv_stage* s, rv_slot& slot, const void* grad_out, void* grad_in) {
  Backward b(s, slot, grad_out, grad_in, s->st);
  RV_TRY(b.begin());
  for (int l = b.p.L - 1; l >= 0; --l) RV_TRY(b.block(l));
  return b.end();
}

// A forward on the stage's stream beside a backward on the auxiliary one, issued in turn block by block: the backward is
// the longer chain, and behind a whole forward its first launch would wait for as long as that takes to issue.
rv_status rv_dec_step(rv_stage* s, rv_slot& fwd, const void* in, void* out, rv_slot& bwd, const void* grad_out, void* grad_in) {
  Backward b(s, bwd, grad_out, grad_in, s->aux);
  RV_TRY(b.begin());
  for (int l = 0; l < b.p.L; ++l) {
    RV_TRY(b.block(b.p.L - 1 - l));
    RV_TRY(forward_block(s, fwd, in, out, l, s->st));
  }
  return b.end();
}
