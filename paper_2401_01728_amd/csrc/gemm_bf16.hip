// bf16 MFMA matrix products of the decoder stage (forward, dX and dW of every Linear),
// fp32 accumulation, for gfx950.
//
//   C[M,N] = sum_k A(m,k) B(k,n)        K % 64 == 0, N % 8 == 0, M % 8 == 0
//
// Each operand is either "k-contiguous" (A[m*lda+k], B[n*ldb+k]) or "k-major"
// (A[k*lda+m], B[k*ldb+n]) - in rows, or in blocks of 32 columns: element (r, c) of a matrix of R rows at
// (c / 32) * 32 R + 32 r + c % 32, so that the 32-deep tile of a k-contiguous operand is ONE run of rows x 64 bytes (as rows: so many
// pieces of 64, each half a line) and that of a k-major one BN / 32 runs of 2 KiB.  Both are one address form,
// r * ld + (c / 32) * bs + c % 32, rows being bs = 32.  Blocks against rows, alone,
// us: 4096x2048x8192 (k-contiguous W) 172 -> 147, 8192x6400x1600 with GELU' 242 -> 216, 4096x8192x2048 with GELU 142 -> 137, weight
// gradients the same; weights cold, 128x1024x4096 21.1 -> 16.0 (32x64 split), 2048x1024x3072 32.0 -> 24.3 (64x64 split).  Stage steps:
// d 2048, 4096 tokens 11.49 -> 10.87 ms, d 1024 1.773 -> 1.714, d 1600, 8192 tokens 22.5 -> 21.9; 6 blocks of d 768 on 1152
// tokens, four microbatches 5345 -> 5095 us.  What it costs: the average that publishes versions 353 -> 372 us over four of 50 M
// parameters (a row of a blocked version is pieces of 64 bytes).  The three products of a Linear y = x W, W stored [in,out]:
//   forward  y  = x W      : A = x  k-contiguous, B = W  k-major
//   dX       dx = dy W^T   : A = dy k-contiguous, B = W  k-contiguous (its rows are the n's)
//   dW       dW = x^T dy   : A = x  k-major,      B = dy k-major      (contraction over tokens)
//
// Tiling: a workgroup of 4 or 8 waves owns a BM x BN tile and walks K in steps of BK = 32; a wave owns a block of MFMA products (v_mfma_f32_32x32x16_bf16 or _16x16x32_bf16).  Operand tiles go
// global -> LDS directly (global_load_lds_dwordx4) through a ring of NS stages, unpadded, bank
// conflicts removed by an XOR swizzle (see "direct-to-LDS pipeline" below);
//   k-contiguous operands sit in LDS as [row][BK k], read as one 16-byte fragment per lane;
//   k-major operands sit as [BK k][cols] and are read with the LDS transpose read
//   (ds_read_b64_tr_b16), which hands each lane four consecutive k of one column: no register
//   transposes, no transposed copies of activations in HBM.
// The MFMA is issued with the B fragment as its first operand, so a lane ends up with
// four CONSECUTIVE n of one row m: epilogues store 8 (bf16) or 16 (fp32) bytes per lane.
#include <type_traits>
#include "internal.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// GELU(z) = z * Phi(z) and its derivative Phi(z) + z * phi(z).  The upper tail of the normal
// distribution, q = 1 - Phi(|z|) = erfc(|z|/sqrt 2)/2, comes from the three-term
// rational-exponential form of erfc (Abramowitz & Stegun 7.1.25, |error| < 1.3e-5 on q - the
// results are rounded to bf16, whose half-ulp is 2e-3 relative):
//   q = (a1 t + a2 t^2 + a3 t^3)/2 * exp(-z^2/2),   t = 1/(1 + 0.47047 |z|/sqrt 2).
// Computing the tail directly loses no digits to cancellation for negative arguments, and
//   GELU(z) = max(z, 0) - |z| q
// needs no select.  The same exponential serves phi(z).  Nine instructions, two of them
// transcendental.
__device__ __forceinline__ float tail_q(float z, float& e) {
  const float t = __builtin_amdgcn_rcpf(__fmaf_rn(fabsf(z), 0.33267254f, 1.0f));
  e = __builtin_amdgcn_exp2f(z * z * -0.72134752f);
  float p = __fmaf_rn(0.3739278f, t, -0.0479399f);
  p = __fmaf_rn(p, t, 0.1740121f);
  return p * t * e;
}
__device__ __forceinline__ float gelu_f(float z) {
  float e;
  const float q = tail_q(z, e);
  return __fmaf_rn(-fabsf(z), q, fmaxf(z, 0.f));
}
__device__ __forceinline__ float dgelu_f(float z) {
  float e;
  const float q = tail_q(z, e);
  const float cdf = z < 0.f ? q : 1.0f - q;
  return __fmaf_rn(z * 0.3989422804014327f, e, cdf);
}

#ifndef RV_RESID_LDS
#define RV_RESID_LDS 1
#endif
struct Epi {
  void* out; int64_t ldo;
  void* out2;
  const uint16_t* bias;
  const float* resid; int64_t ldr;
  const uint16_t* zin;
  float* upd_w;   // EPI_F32_UPD: fp32 master tile updated in place (out2 = its bf16 weight version)
  float eta;
  float* colpart; // EPI_BF16_DGELU: partial column sums of the output, one row (pitch ldo) per tile row
  // where (m, n) lies in the output that may be in blocks of 32 columns: `out` of EPI_BF16_DGELU, `out2` of
  // EPI_BF16_BIAS_GELU and of EPI_F32_UPD (rows: ldb = ldo, bsb = 32)
  int64_t ldb, bsb;
  __device__ __forceinline__ int64_t blocked(int m, int n) const { return (int64_t)m * ldb + (n >> 5) * bsb + (n & 31); }
};

enum { EPI_BF16 = RV_EPI_BF16, EPI_BF16_BIAS = RV_EPI_BF16_BIAS, EPI_F32_BIAS_RESID = RV_EPI_F32_BIAS_RESID,
       EPI_BF16_BIAS_GELU = RV_EPI_BF16_BIAS_GELU, EPI_BF16_DGELU = RV_EPI_BF16_DGELU, EPI_F32 = RV_EPI_F32,
       EPI_F32_BIAS_RESID_BF16 = RV_EPI_F32_BIAS_RESID_BF16,
       // grouped weight-gradient launch only: out f32 = acc if out is given; if upd_w is given the
       // delayed update of Eq. 2 right here, w <- w - eta * acc (one fused multiply-add, as the
       // stand-alone update kernel does it) and out2 bf16 = the new w
       EPI_F32_UPD = 7 };

constexpr bool epi_has_bias(int epi) {
  return epi == EPI_BF16_BIAS || epi == EPI_F32_BIAS_RESID || epi == EPI_BF16_BIAS_GELU || epi == EPI_F32_BIAS_RESID_BF16;
}
constexpr bool epi_has_resid(int epi) { return epi == EPI_F32_BIAS_RESID || epi == EPI_F32_BIAS_RESID_BF16; }

__device__ __forceinline__ void add_bias4(f32x4& a, u32x2 b) {
  a.x += __uint_as_float(b.x << 16); a.y += __uint_as_float(b.x & 0xFFFF0000u);
  a.z += __uint_as_float(b.y << 16); a.w += __uint_as_float(b.y & 0xFFFF0000u);
}

// four consecutive columns n..n+3 of row m; b = their bias, r = their residual (already loaded)
template <int EPI>
__device__ __forceinline__ void epilogue4(const Epi& e, int m, int n, f32x4 a, u32x2 b, f32x4 r) {
  if (epi_has_bias(EPI)) add_bias4(a, b);
  if (EPI == EPI_BF16 || EPI == EPI_BF16_BIAS) {
    u32x2 o; o.x = rv_pack_bf16x2(a.x, a.y); o.y = rv_pack_bf16x2(a.z, a.w);
    *reinterpret_cast<u32x2*>((uint16_t*)e.out + (int64_t)m * e.ldo + n) = o;
  } else if (epi_has_resid(EPI)) {
    a += r;
    *reinterpret_cast<f32x4*>((float*)e.out + (int64_t)m * e.ldo + n) = a;
    if (EPI == EPI_F32_BIAS_RESID_BF16) {
      u32x2 o; o.x = rv_pack_bf16x2(a.x, a.y); o.y = rv_pack_bf16x2(a.z, a.w);
      *reinterpret_cast<u32x2*>((uint16_t*)e.out2 + (int64_t)m * e.ldo + n) = o;
    }
  } else if (EPI == EPI_BF16_BIAS_GELU) {
    u32x2 o; o.x = rv_pack_bf16x2(a.x, a.y); o.y = rv_pack_bf16x2(a.z, a.w);
    *reinterpret_cast<u32x2*>((uint16_t*)e.out + (int64_t)m * e.ldo + n) = o;
    u32x2 g;
    g.x = rv_pack_bf16x2(gelu_f(a.x), gelu_f(a.y));
    g.y = rv_pack_bf16x2(gelu_f(a.z), gelu_f(a.w));
    *reinterpret_cast<u32x2*>((uint16_t*)e.out2 + e.blocked(m, n)) = g;
  } else if (EPI == EPI_BF16_DGELU) {
    u32x2 z = *reinterpret_cast<const u32x2*>(e.zin + (int64_t)m * e.ldo + n);
    a.x *= dgelu_f(__uint_as_float(z.x << 16)); a.y *= dgelu_f(__uint_as_float(z.x & 0xFFFF0000u));
    a.z *= dgelu_f(__uint_as_float(z.y << 16)); a.w *= dgelu_f(__uint_as_float(z.y & 0xFFFF0000u));
    u32x2 o; o.x = rv_pack_bf16x2(a.x, a.y); o.y = rv_pack_bf16x2(a.z, a.w);
    *reinterpret_cast<u32x2*>((uint16_t*)e.out + e.blocked(m, n)) = o;
  } else if (EPI == EPI_F32) {
    *reinterpret_cast<f32x4*>((float*)e.out + (int64_t)m * e.ldo + n) = a;
  } else if (EPI == EPI_F32_UPD) {
    // (no update asked for: the gradient tile alone; the update path is f32_tile_through_lds)
    *reinterpret_cast<f32x4*>((float*)e.out + (int64_t)m * e.ldo + n) = a;
  }
}

// A wave's part of a tile is accumulated in products of 32x32 (V = f32x16) or 16x16 (V = f32x4), [TM][TN] of them.  Either
// way a lane holds of each of its TM rows - row l % 32 or l % 16 of a product - runs of four consecutive columns: "quads", four
// to a product of 32x32 (columns 8 r + 4 (l / 32)), one to a product of 16x16 (columns 4 (l / 16)).
template <typename V> constexpr int kEdge = sizeof(V) == 64 ? 32 : 16;       // of a product
template <typename V, int TN> constexpr int kQuads = sizeof(V) == 64 ? 4 * TN : TN;
template <typename V>
__device__ __forceinline__ int quad_row(int i) { return i * kEdge<V> + (threadIdx.x & (kEdge<V> - 1)); }
template <typename V>
__device__ __forceinline__ int quad_col(int c) {
  const int l = threadIdx.x & 63;
  return sizeof(V) == 64 ? (c >> 2) * 32 + 8 * (c & 3) + 4 * (l >> 5) : c * 16 + 4 * (l >> 4);
}
template <int TM, int TN>
__device__ __forceinline__ f32x4 quad(const f32x4 (&acc)[TM][TN], int i, int c) { return acc[i][c]; }
template <int TM, int TN>
__device__ __forceinline__ f32x4 quad(const f32x16 (&acc)[TM][TN], int i, int c) {
  const int r = 4 * (c & 3);
  return f32x4{acc[i][c >> 2][r], acc[i][c >> 2][r + 1], acc[i][c >> 2][r + 2], acc[i][c >> 2][r + 3]};
}

// What an epilogue reads (bias, residual) is requested for a whole batch of column groups, at
// addresses clamped into the matrix, before the first result is formed: a batch costs one
// memory round trip, not one per group of four columns.
template <typename V, int TM, int TN, int EPI>
__device__ __forceinline__ void write_tile(const V (&acc)[TM][TN], const Epi& e, int mw, int nw, int M, int N) {
  constexpr int Q = kQuads<V, TN>, QB = Q < 8 ? Q : 8, IB = 8 / QB < TM ? 8 / QB : TM;   // quads, rows per batch of residual loads
  static_assert(Q % QB == 0 && TM % IB == 0, "whole batches");
  u32x2 bias4[Q];
#pragma unroll
  for (int c = 0; c < Q; ++c) {
    bias4[c] = u32x2{0u, 0u};
    if (epi_has_bias(EPI)) {
      const int n = nw + quad_col<V>(c);
      bias4[c] = *reinterpret_cast<const u32x2*>(e.bias + (n < N ? n : N - 4));
    }
  }
#pragma unroll
  for (int i0 = 0; i0 < TM; i0 += IB)
#pragma unroll
    for (int c0 = 0; c0 < Q; c0 += QB) {
      f32x4 res[IB][QB];
#pragma unroll
      for (int i = 0; i < IB; ++i)
#pragma unroll
        for (int c = 0; c < QB; ++c) {
          res[i][c] = f32x4{0.f, 0.f, 0.f, 0.f};
          if (epi_has_resid(EPI)) {
            const int m = mw + quad_row<V>(i0 + i), n = nw + quad_col<V>(c0 + c);
            res[i][c] = *reinterpret_cast<const f32x4*>(e.resid + (int64_t)(m < M ? m : M - 1) * e.ldr + (n < N ? n : N - 4));
          }
        }
#pragma unroll
      for (int i = 0; i < IB; ++i)
#pragma unroll
        for (int c = 0; c < QB; ++c) {
          const int m = mw + quad_row<V>(i0 + i), n = nw + quad_col<V>(c0 + c);
          if (m >= M || n >= N) continue;
          epilogue4<EPI>(e, m, n, quad(acc, i0 + i, c0 + c), bias4[c0 + c], res[i][c]);
        }
    }
}

// Workgroup -> tile map (tiles_m > 0; a negative tiles_m selects the natural order).
// Workgroups are dealt to the 8 XCDs round-robin (id % 8), and each
// XCD has its own L2.  First give every XCD a CONTIGUOUS range of tile numbers, then walk
// that range in bands of 8 tile-rows, column by column: the ~32 tiles an XCD has in flight
// form an 8 x 4 patch, so it pulls 12 operand tiles per k-step through its L2 instead of 33.
__device__ __forceinline__ void tile_of_block(int tiles_m, int tiles_n, int band_rows, int& bm, int& bn) {
  const int total = tiles_m * tiles_n;
  int id = blockIdx.x;
  if (tiles_m < 0) {   // natural order: consecutive workgroups walk down one column of tiles
    tiles_m = -tiles_m; bm = id % tiles_m; bn = id / tiles_m; return;
  }
  const int per = total / 8;
  if (id < per * 8) id = (id % 8) * per + id / 8;       // the remainder keeps its natural order
  const int GM = band_rows;
  const int band = id / (GM * tiles_n);
  const int first = band * GM;
  const int rows = tiles_m - first < GM ? tiles_m - first : GM;
  const int in = id - band * GM * tiles_n;
  bm = first + in % rows;
  bn = in / rows;
}

// bf16 outputs leave through LDS: every wave parks its accumulator tile (after bias / GELU /
// GELU') as bf16 in a [BM][BN] image of the workgroup tile, then the workgroup writes the
// image out row by row, 16 bytes per lane, whole 128-byte lines per row segment - instead
// of 8-byte pieces of 32 different rows per store instruction.  The GELU epilogue makes two
// trips (pre-activation, then activation).  The image reuses the operand ring.
__host__ __device__ constexpr int stage_pitch(int bn) { return bn * 2 + 16; }
__host__ __device__ constexpr bool staged_epi(int epi) {
  return epi == EPI_BF16 || epi == EPI_BF16_BIAS || epi == EPI_BF16_BIAS_GELU || epi == EPI_BF16_DGELU;
}

template <int BM, int BN, int NT, typename V, int TM, int TN, int EPI>
__device__ __forceinline__ void write_tile_staged(const V (&acc)[TM][TN], const Epi& e, int m0, int n0,
                                                  int wm0, int wn0, int M, int N, char* smem) {
  constexpr int PITCH = stage_pitch(BN);
  constexpr int PASSES = EPI == EPI_BF16_BIAS_GELU ? 2 : 1;
  const int l = threadIdx.x & 63;
  __syncthreads();   // every wave has finished reading operands from the ring
  if (EPI == EPI_BF16_DGELU) {
    // the pre-activation tile comes in the way the result goes out: whole rows, 16 bytes per
    // lane, through the image; a lane then finds its own four values where it will put the result
    // (eight loads per lane in flight before the first is parked: two memory round trips per
    // tile instead of one per 16-byte piece)
    constexpr int CPR = BN / 8, PIECES = BM * CPR / NT, BATCH = NT >= 512 ? 8 : 4;
    static_assert(BM * CPR % NT == 0 && PIECES % BATCH == 0, "whole batches");
#pragma unroll 1
    for (int p0 = 0; p0 < PIECES; p0 += BATCH) {
      u32x4 v[BATCH];
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int idx = threadIdx.x + (p0 + u) * NT, row = idx / CPR, c = idx % CPR;
        const int gm = m0 + row, gn = n0 + c * 8;
        v[u] = u32x4{0u, 0u, 0u, 0u};
        if (gm < M && gn < N) v[u] = *reinterpret_cast<const u32x4*>(e.zin + (int64_t)gm * e.ldo + gn);
      }
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int idx = threadIdx.x + (p0 + u) * NT, row = idx / CPR, c = idx % CPR;
        *reinterpret_cast<u32x4*>(smem + row * PITCH + c * 16) = v[u];
      }
    }
    __syncthreads();
  }
  // GELU' epilogue: column sums of the results over this wave's rows, kept per lane while the tile
  // is packed (the bias gradient of the Linear below the GELU, one partial row per tile row)
  constexpr int Q = kQuads<V, TN>;
  f32x4 cs[Q];
  const bool want_cs = EPI == EPI_BF16_DGELU && e.colpart != nullptr;
  float* red = reinterpret_cast<float*>(smem + BM * PITCH);   // [2 wave rows][BN], behind the image
  if (EPI == EPI_BF16_DGELU) {
#pragma unroll
    for (int c = 0; c < Q; ++c) cs[c] = 0.f;
  }
  u32x2 bias4[Q];                                // this lane's bias values, loaded once
#pragma unroll
  for (int c = 0; c < Q; ++c) {
    bias4[c] = u32x2{0u, 0u};
    if (EPI == EPI_BF16_BIAS || EPI == EPI_BF16_BIAS_GELU) {
      const int gn = n0 + wn0 + quad_col<V>(c);
      bias4[c] = *reinterpret_cast<const u32x2*>(e.bias + (gn < N ? gn : N - 4));
    }
  }
#pragma unroll
  for (int pass = 0; pass < PASSES; ++pass) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int ml = wm0 + quad_row<V>(i);
#pragma unroll
      for (int c = 0; c < Q; ++c) {
        const int nl = wn0 + quad_col<V>(c);
        const int gm = m0 + ml, gn = n0 + nl;
        f32x4 a = quad(acc, i, c);
        if (EPI == EPI_BF16_BIAS || EPI == EPI_BF16_BIAS_GELU) {
          add_bias4(a, bias4[c]);
          if (pass == 1) { a.x = gelu_f(a.x); a.y = gelu_f(a.y); a.z = gelu_f(a.z); a.w = gelu_f(a.w); }
        }
        if (EPI == EPI_BF16_DGELU) {
          const u32x2 z = *reinterpret_cast<const u32x2*>(smem + ml * PITCH + nl * 2);
          a.x *= dgelu_f(__uint_as_float(z.x << 16)); a.y *= dgelu_f(__uint_as_float(z.x & 0xFFFF0000u));
          a.z *= dgelu_f(__uint_as_float(z.y << 16)); a.w *= dgelu_f(__uint_as_float(z.y & 0xFFFF0000u));
          const bool ok = gm < M && gn < N;   // (a select and no branch: what is past the end is not summed)
#pragma unroll
          for (int k = 0; k < 4; ++k) cs[c][k] += ok ? a[k] : 0.f;
        }
        u32x2 o; o.x = rv_pack_bf16x2(a.x, a.y); o.y = rv_pack_bf16x2(a.z, a.w);
        *reinterpret_cast<u32x2*>(smem + ml * PITCH + nl * 2) = o;
        if (EPI == EPI_BF16_DGELU && c % 2 == 1) __builtin_amdgcn_sched_barrier(0);   // (all quads' pre-activations at once spill)
      }
    }
    if (EPI == EPI_BF16_DGELU && want_cs) {   // (workgroup-uniform)
#pragma unroll
      for (int c = 0; c < Q; ++c) {
        f32x4 v;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = rv_row_sum(cs[c][k]);
        if ((l & 15) == 0) *reinterpret_cast<f32x4*>(red + (wm0 ? BN : 0) + wn0 + quad_col<V>(c)) = v;
      }
    }
    __syncthreads();
    if (EPI == EPI_BF16_DGELU && want_cs) {
      for (int c = threadIdx.x; c < BN; c += NT)
        if (n0 + c < N) e.colpart[(int64_t)(m0 / BM) * e.ldo + n0 + c] = red[c] + red[BN + c];
    }
    uint16_t* dst = (uint16_t*)(pass == 0 ? e.out : e.out2);
    constexpr int CPR = BN / 8, PIECES = BM * CPR / NT, BATCH = NT >= 512 ? 8 : 4;
    static_assert(BM * CPR % NT == 0 && PIECES % BATCH == 0, "whole batches");
#pragma unroll 1
    for (int p0 = 0; p0 < PIECES; p0 += BATCH) {
      u32x4 v[BATCH];
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int idx = threadIdx.x + (p0 + u) * NT, row = idx / CPR, c = idx % CPR;
        v[u] = *reinterpret_cast<const u32x4*>(smem + row * PITCH + c * 16);
      }
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int idx = threadIdx.x + (p0 + u) * NT, row = idx / CPR, c = idx % CPR;
        const int gm = m0 + row, gn = n0 + c * 8;
        const bool blk = EPI == EPI_BF16_DGELU || (EPI == EPI_BF16_BIAS_GELU && pass == 1);
        if (gm < M && gn < N) *reinterpret_cast<u32x4*>(dst + (blk ? e.blocked(gm, gn) : (int64_t)gm * e.ldo + gn)) = v[u];
      }
    }
    if (pass + 1 < PASSES) __syncthreads();
  }
}

// ---- direct-to-LDS pipeline ---------------------------------------------------------------
// Tiles go global -> LDS with global_load_lds_dwordx4: no staging registers, no LDS write
// instructions.  One such instruction fills 1 KiB of LDS (lane i -> base + 16 i), so the
// tile is unpadded and bank conflicts are removed by an XOR swizzle of the 16-byte chunk
// index instead; because a lane's LDS slot is fixed, the swizzle is applied to the GLOBAL
// address a lane fetches.
//   k-contiguous tile [rows][32]: four rows to a 256-byte bank line; a 16-byte read goes out in groups of lanes 0-3, 12-15, 20-27 / 4-11,
//                                 16-19, 28-31 and the same of the upper half, which with fragments of 16 rows are one chunk of
//                                 rows 0-3 and 12-15 and the next one of rows 4-11: physical chunk = c ^ (-(row / 4) & 3) is free of
//                                 conflicts with them and with fragments of 32 rows.  (c ^ (row / 4 & 3) is so with 32 rows alone: with 16,
//                                 every read of 8192x8192x8192 took twice its LDS cycles, 2.04e8 for 1.03e8)
//   k-major tile [BK][cols]     : half a wave's transposing read takes 32 bytes of rows k .. k + 3 and k + 8 .. k + 11
//                                 (fragments of 16 rows) or 64 bytes of rows k .. k + 3 (of 32): physical chunk =
//                                 c ^ ((k & 3) << 2) ^ ((k & 8) >> 2); split forms with 64 columns (fragments of 32 rows),
//                                 two rows to a 256-byte bank line, c ^ ((k & 2) << 1)
// NS stages form a ring (see gemm_dtl_body): the products are bound by how fast operand tiles arrive, inside a stage step
// even more than alone (with seven of eight MFMAs taken out the step is 3 % shorter, without
// the loads 24 %), so a workgroup keeps two or three 32-deep tiles in flight.  (One 64-deep tile, requested behind the barrier
// that opens the one before, on the four-wave tiles: 10 - 20 % slower alone, 4 blocks of d 1024 on 4096 tokens 1796 / 1747 us a step.)
__host__ __device__ constexpr int dtl_tile_bytes(int rows, int bk) { return rows * bk * 2; }

template <int BK>
__device__ __forceinline__ int kc_swizzle(int row) {
  static_assert(BK == 32, "four chunks to a row, four rows to a bank line");
  return -(row >> 2) & 3;
}
template <int ROWS>
__device__ __forceinline__ int km_swizzle(int k) { return ROWS == 64 ? (k & 2) << 1 : ((k & 3) << 2) ^ ((k & 8) >> 2); }

template <bool KM, int ROWS, int BK, int NW>
struct Dtl {
  static constexpr int N = ROWS * BK / 8 / (64 * NW);   // loads per lane per tile
  int off[N];
};

template <bool KM, int ROWS, int BK, int NW>
__device__ __forceinline__ void dtl_init(Dtl<KM, ROWS, BK, NW>& s, int64_t ld, int64_t bs, int r0, int rows, int wave) {
  const int l = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < Dtl<KM, ROWS, BK, NW>::N; ++i) {
    const int slot = (i * NW + wave) * 64 + l;
    if (!KM) {
      constexpr int CPR = BK / 8;
      const int row = slot / CPR, c = (slot % CPR) ^ kc_swizzle<BK>(row);
      int gr = r0 + row;
      gr = gr < rows ? gr : rows - 1;
      s.off[i] = gr * (int)ld + (c * 8 / 32) * (int)bs + c * 8 % 32;
    } else {
      constexpr int CPR = ROWS / 8;
      const int kr = slot / CPR, c = (slot % CPR) ^ km_swizzle<ROWS>(kr);
      int col = r0 + c * 8;
      col = col < rows ? col : rows - 8;
      s.off[i] = kr * (int)ld + (col >> 5) * (int)bs + (col & 31);
    }
  }
}

// rows kr .. + 3 and kr + 4 .. + 7 of a k-major tile, transposed: a lane gets eight consecutive k of one column
template <int ROWS>
__device__ __forceinline__ bf16x8 dtl_read_tr(const char* lds, int kr, int col) {
  const int c = (col >> 3) ^ km_swizzle<ROWS>(kr);
  const char* p = lds + kr * (ROWS * 2) + c * 16 + (col & 7) * 2;
  s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p));
  s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (s16x4 __attribute__((address_space(3)))*)(p + 4 * (ROWS * 2)));
  s16x8 r = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, r);
}

// Fragment of one v_mfma_f32_16x16x32_bf16 (whole tiles): rows row0 .. + 15, k-step kk of 32.  Lane l holds row l % 16, k = 8 (l / 16) .. + 7.
template <bool KM, int ROWS, int BK>
__device__ __forceinline__ bf16x8 dtl_frag(const char* lds, int row0, int kk) {
  const int l = threadIdx.x & 63;
  if (!KM) {
    const int row = row0 + (l & 15);
    const int c = (kk * 4 + (l >> 4)) ^ kc_swizzle<BK>(row);
    return *reinterpret_cast<const bf16x8*>(lds + row * (BK * 2) + c * 16);
  } else {
    static_assert(!KM || ROWS > 64, "the swizzle of narrower tiles is that of 32-row fragments");
    const int q = l >> 4, i = l & 15;
    const int kr = kk * 32 + 8 * q + (i >> 2);
    const int col = row0 + 4 * (i & 3);
    return dtl_read_tr<ROWS>(lds, kr, col);
  }
}

// Fragment of one v_mfma_f32_32x32x16_bf16: rows row0 .. + 31, k-step kk of 16.  Lane l holds row l % 32, k = 8 (l / 32) .. + 7.
template <bool KM, int ROWS, int BK>
__device__ __forceinline__ bf16x8 dtl_frag32(const char* lds, int row0, int kk) {
  const int l = threadIdx.x & 63;
  if (!KM) {
    const int row = row0 + (l & 31);
    const int c = (kk * 2 + (l >> 5)) ^ kc_swizzle<BK>(row);
    return *reinterpret_cast<const bf16x8*>(lds + row * (BK * 2) + c * 16);
  } else {
    const int q = l >> 4, i = l & 15;
    const int kr = kk * 16 + 8 * (q >> 1) + (i >> 2);
    const int col = row0 + 16 * (q & 1) + 4 * (i & 3);
    return dtl_read_tr<ROWS>(lds, kr, col);
  }
}

// Issued as inline assembly: the compiler would otherwise make every later LDS read wait for ALL outstanding loads, which
// defeats the ring.  The kernels order them with explicit vmcnt waits and barriers.
// Direct-to-LDS load in the scalar-base form: wave-uniform 64-bit base in SGPRs, per-lane byte
// offset in one VGPR (no per-load address arithmetic), LDS block = lb + IMM through M0.
__device__ __forceinline__ void dtl_load_s(const void* base, unsigned off, int m0v) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(off), "s"(base), "s"(m0v)
               : "memory", "m0");
}
// s_waitcnt vmcnt(n) only (expcnt, lgkmcnt left at "no wait"); n < 64
#define RV_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (((n) >> 4) << 14) | 0x0F70)

extern __shared__ __align__(1024) char dtl_smem[];

// Epilogue of a weight-gradient tile with the delayed update of Eq. 2 folded in:
//   w <- w - eta * acc (fp32 master, in place), bf16(w) into the new weight version, acc itself
// to `out` only on request.  The master tile is fetched through LDS, half a tile at a time,
// with direct-to-LDS loads (one instruction = one 256-column fp32 row): all rows of the half
// are in flight together, so the read costs one memory round trip per half instead of one per
// accumulator group, and it needs no registers.  Row pitch BN*4 + 16 bytes spreads a wave's
// 32 rows over the banks.
__host__ __device__ constexpr int upd_image_bytes(int bm, int bn) { return (bm / 2) * (bn * 4 + 16); }

// MODE 0: the update above (source and fp32 result = e.upd_w, bf16 result = e.out2, the gradient itself to e.out
//         on request).  MODE 1: out = acc + bias + residual (source = e.resid, fp32 result = e.out, and with
//         BF16OUT its rounding to e.out2) - the same staging: at 4-byte results per lane-quad the direct form costs
//         more L2 requests than a short product's whole main loop.
// The results go back into the LDS rows they came from and leave the way the rows came in: whole rows, 16 bytes
// per lane, one 128-byte line per 8 lanes, instead of 32-byte pieces of 32 different rows per store instruction.
template <int BM, int BN, int NW, typename V, int TM, int TN, int MODE, bool BF16OUT>
__device__ __forceinline__ void f32_tile_through_lds(const V (&acc)[TM][TN], const Epi& e, int m0, int n0,
                                                     int wm0, int wn0, int M, int N, char* smem) {
  static_assert(BN == 256, "one direct-to-LDS instruction moves one 256-column fp32 row");
  constexpr int HALF = BM / 2, PITCH = BN * 4 + 16, RPW = HALF / NW;   // rows per wave in the row-wise phases
  static_assert(HALF % NW == 0 && RPW % 8 == 0, "row batches of eight");
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63;
  const float* srcm = MODE == 0 ? e.upd_w : e.resid;
  const int64_t lds_src = MODE == 0 ? e.ldo : e.ldr;
  float* dst32 = MODE == 0 ? e.upd_w : (float*)e.out;
  constexpr int Q = kQuads<V, TN>;
  u32x2 bias4[Q];
#pragma unroll
  for (int c = 0; c < Q; ++c) {
    bias4[c] = u32x2{0u, 0u};
    if (MODE == 1) {
      const int n = n0 + wn0 + quad_col<V>(c);
      bias4[c] = *reinterpret_cast<const u32x2*>(e.bias + (n < N ? n : N - 4));
    }
  }
  int gn = n0 + l * 4;
  const bool col_ok = gn < N;
  gn = col_ok ? gn : N - 4;                    // ragged tiles fetch valid memory and ignore it below
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    __syncthreads();   // LDS is free: the operand ring (h = 0) or the other half's rows (h = 1)
    for (int r = wave; r < HALF; r += NW) {
      int gm = m0 + h * HALF + r;
      gm = gm < M ? gm : M - 1;
      const float* src = srcm + (int64_t)gm * lds_src + gn;
      const int m0v = __builtin_amdgcn_readfirstlane((int)(size_t)smem + r * PITCH);
      asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                   :
                   : "v"(src), "s"(m0v)
                   : "memory", "m0");
    }
    RV_WAIT_VMCNT(0);
    __syncthreads();
    if (wm0 == h * HALF) {
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int ml = quad_row<V>(i);
        const int gm = m0 + wm0 + ml;
#pragma unroll
        for (int c = 0; c < Q; ++c) {
          const int nl = wn0 + quad_col<V>(c);
          f32x4* p = reinterpret_cast<f32x4*>(smem + ml * PITCH + nl * 4);
          const f32x4 w = *p;
          f32x4 a = quad(acc, i, c);
          f32x4 r;
          if (MODE == 0) {
            r.x = __fmaf_rn(-e.eta, a.x, w.x); r.y = __fmaf_rn(-e.eta, a.y, w.y);
            r.z = __fmaf_rn(-e.eta, a.z, w.z); r.w = __fmaf_rn(-e.eta, a.w, w.w);
            if (e.out && gm < M && n0 + nl < N)
              *reinterpret_cast<f32x4*>((float*)e.out + (int64_t)gm * e.ldo + n0 + nl) = a;
          } else {
            add_bias4(a, bias4[c]);
            r = a + w;
          }
          *p = r;
        }
      }
    }
    __syncthreads();   // the half's results are in LDS
#pragma unroll 1
    for (int rb = 0; rb < RPW; rb += 8) {
      f32x4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const f32x4*>(smem + (wave + (rb + u) * NW) * PITCH + l * 16);
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int gm = m0 + h * HALF + wave + (rb + u) * NW;
        if (gm < M && col_ok) {
          const int64_t o = (int64_t)gm * e.ldo + gn;
          *reinterpret_cast<f32x4*>(dst32 + o) = v[u];
          if (BF16OUT) {
            u32x2 q; q.x = rv_pack_bf16x2(v[u].x, v[u].y); q.y = rv_pack_bf16x2(v[u].z, v[u].w);
            *reinterpret_cast<u32x2*>((uint16_t*)e.out2 + (MODE == 0 ? e.blocked(gm, gn) : o)) = q;
          }
        }
      }
    }
  }
}

template <int BM, int BN, int BK, int NS, int NW, bool AKM, bool BKM, int EPI>
__device__ __forceinline__ void gemm_dtl_body(const uint16_t* __restrict__ A, int64_t lda, int64_t a_bs,
                                              const uint16_t* __restrict__ B, int64_t ldb, int64_t b_bs, int M, int N,
                                              int K, int bm, int bn, const Epi& e) {
  // Products of 16x16: the matrix cores do 1717 TFLOP/s out of LDS at the board's power cap with those, 1586 with 32x32 ones
  // (registers alone 2028 / 1807; half the accumulator traffic per flop).  Stage steps at the cap 2 % shorter (8 blocks of d 2048
  // 10.92 -> 10.72 ms), below it, after seconds under load, 0.3 - 0.7 %.
  // NW waves laid out 2 (m) x NW/2 (n)
  typedef f32x4 V;
  constexpr int WM = BM / 2, WN = BN / (NW / 2), TM = WM / 16, TN = WN / 16;
  constexpr int A_BYTES = dtl_tile_bytes(BM, BK), B_BYTES = dtl_tile_bytes(BN, BK);
  constexpr int BUF = A_BYTES + B_BYTES;
  constexpr int NL = NW;                                                    // loader waves per tile
  char* smem = dtl_smem;

  const int m0 = bm * BM, n0 = bn * BN;
  const int wave = threadIdx.x >> 6;
  const int wm0 = (wave & 1) * WM, wn0 = (wave >> 1) * WN;

  V acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = 0.f;

  const int lw = wave;                 // this wave's share of a tile's loads
  Dtl<AKM, BM, BK, NL> da;
  Dtl<BKM, BN, BK, NL> db;
  dtl_init<AKM, BM, BK, NL>(da, lda, a_bs, m0, M, lw);
  dtl_init<BKM, BN, BK, NL>(db, ldb, b_bs, n0, N, lw);
  const int nk = K / BK;
  {
    // Ring of NS slots, the slot hand-over INSIDE a k-tile.  A tile is one step of 32 in k, multiplied in two halves: the upper
    // TM / 2 rows of fragments, column by column, then the lower ones.  Between the halves (all fragments of the tile are
    // in registers) the workgroup meets once: tile s+1 has landed and nobody reads tile s's slot any more.  Behind
    // that barrier, among the multiplications of the lower half, the upper fragments of tile s+1 are read, each column's B fragment
    // as soon as its last multiplication is out (no second set of registers), and the loads of tile s+NS go into
    // the slot just left - so NS-1 tiles are in flight while one is being used, and the matrix core does not wait at a
    // tile boundary.
    constexpr int NA = Dtl<AKM, BM, BK, NL>::N, NB = Dtl<BKM, BN, BK, NL>::N, LPS = NA + NB;
    constexpr int HM = TM / 2, STRIDE = HM * TN / LPS; // MFMAs per load in the lower half
    static_assert(BK == 32 && TM % 2 == 0 && HM <= TN && STRIDE >= 1, "a column to each lower fragment, a load to every STRIDE MFMAs");
    static_assert((NS - 1) * LPS < 64, "vmcnt range");
    unsigned oa[NA], ob[NB];               // per-lane byte offsets of this wave's loads inside a tile
#pragma unroll
    for (int i = 0; i < NA; ++i) oa[i] = (unsigned)da.off[i] * 2u;
#pragma unroll
    for (int i = 0; i < NB; ++i) ob[i] = (unsigned)db.off[i] * 2u;
    auto baseA = [&](int t) { return AKM ? A + (int64_t)t * BK * lda : A + (int64_t)t * (BK / 32) * a_bs; };
    auto baseB = [&](int t) { return BKM ? B + (int64_t)t * BK * ldb : B + (int64_t)t * (BK / 32) * b_bs; };
    // wait until at most `tiles` of this wave's newest tile loads are still in flight
    auto wait_tiles = [&](int tiles) {
      if (NS >= 4 && tiles >= 3) RV_WAIT_VMCNT(3 * LPS);
      else if (NS >= 3 && tiles >= 2) RV_WAIT_VMCNT(2 * LPS);
      else if (tiles >= 1) RV_WAIT_VMCNT(1 * LPS);
      else RV_WAIT_VMCNT(0);
    };
    static_assert(NS <= 4, "wait_tiles covers up to three tiles in flight behind the awaited one");
    const int pre = nk < NS ? nk : NS;
    for (int t = 0; t < pre; ++t) {
      const int lb = __builtin_amdgcn_readfirstlane((int)(size_t)(smem + t * BUF) + lw * 1024);
      const uint16_t* pa = baseA(t);
      const uint16_t* pb = baseB(t);
#pragma unroll
      for (int q = 0; q < NA; ++q) dtl_load_s(pa, oa[q], lb + q * NL * 1024);
#pragma unroll
      for (int q = 0; q < NB; ++q) dtl_load_s(pb, ob[q], lb + A_BYTES + q * NL * 1024);
    }
    wait_tiles(pre - 1);
    __syncthreads();
    // A wave whose part of a ragged tile lies past the end of the result only takes its share of the loads (a width of 1600 is
    // six tiles and a quarter: of the last one's eight waves two have something to multiply).  8192x1600x6400 alone 152 -> 146 us,
    // 8192x1600x1600 48 -> 46; 12 blocks of d 1600 on 8192 tokens in separate calls 20.47 -> 20.24 ms, as a stage step, where the other
    // streams take what a wave leaves, the same; widths of 832, 1088 and 2112 within 0.5 % either way.
    if (__builtin_amdgcn_readfirstlane(m0 + wm0 >= M || n0 + wn0 >= N)) {
      int slot = 0;
      for (int s = 0; s + 1 < nk; ++s) {
        if (s + NS < nk) RV_WAIT_VMCNT((NS - 2) * LPS);
        else wait_tiles(nk - 2 - s);
        __syncthreads();
        if (s + NS < nk) {
          const int lb = __builtin_amdgcn_readfirstlane((int)(size_t)(smem + slot * BUF) + lw * 1024);
          const uint16_t* pa = baseA(s + NS);
          const uint16_t* pb = baseB(s + NS);
#pragma unroll
          for (int q = 0; q < NA; ++q) dtl_load_s(pa, oa[q], lb + q * NL * 1024);
#pragma unroll
          for (int q = 0; q < NB; ++q) dtl_load_s(pb, ob[q], lb + A_BYTES + q * NL * 1024);
        }
        slot = slot + 1 == NS ? 0 : slot + 1;
      }
    } else {
    bf16x8 fa[TM], fb[TN];
#pragma unroll
    for (int i = 0; i < HM; ++i) fa[i] = dtl_frag<AKM, BM, BK>(smem, wm0 + i * 16, 0);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[j] = dtl_frag<BKM, BN, BK>(smem + A_BYTES, wn0 + j * 16, 0);
    // the upper half of the tile at `cur`, and the reads of its lower fragments, one behind the first MFMA of each column
    // (all of them behind the first column's MFMAs: warm stage steps 0.6 % longer, see the loads below)
    auto upper_half = [&](const char* cur) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int i = 0; i < HM; ++i) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
          if (i == 0 && j < HM) {
            __builtin_amdgcn_sched_barrier(0);
            fa[HM + j] = dtl_frag<AKM, BM, BK>(cur, wm0 + (HM + j) * 16, 0);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
    };
    // the lower half; with `nxt` the first fragments of the tile there, with `pa` the loads of a tile into the block at `lb`, the
    // first one behind the first MFMA.  (Three MFMAs later, together with the reads above: 8 blocks of d 2048 9.28 -> 9.43 ms,
    // 12 of d 1600 18.04 -> 18.20, warm; products of 32x32 9.35 and 18.10.)
    auto lower_half = [&](auto has_next, const char* nxt, auto has_load, const uint16_t* pa, const uint16_t* pb, int lb) {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
#pragma unroll
        for (int i = 0; i < HM; ++i) {
          acc[HM + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[HM + i], acc[HM + i][j], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          if (has_next && j == 0) fa[i] = dtl_frag<AKM, BM, BK>(nxt, wm0 + i * 16, 0);
          const int m = j * HM + i;
          if (has_load && m % STRIDE == 0 && m / STRIDE < LPS) {
            const int q = m / STRIDE;
            if (q < NA) dtl_load_s(pa, oa[q], lb + q * NL * 1024);
            else dtl_load_s(pb, ob[q - NA], lb + A_BYTES + (q - NA) * NL * 1024);
          }
          if (has_next && i == HM - 1) fb[j] = dtl_frag<BKM, BN, BK>(nxt + A_BYTES, wn0 + j * 16, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    constexpr std::true_type yes;
    constexpr std::false_type no;
    int slot = 0;                            // ring slot of tile s
    int s = 0;
    for (; s + NS < nk; ++s) {               // passes that still have a tile s+NS to fetch
      const int nslot = slot + 1 == NS ? 0 : slot + 1;
      upper_half(smem + slot * BUF);
      RV_WAIT_VMCNT((NS - 2) * LPS);         // tile s+1 (tiles s+2 .. s+NS-1 may still fly)
      __syncthreads();                       // all of tile s+1 is in LDS; all fragment reads of tile s are done
      const int lb = __builtin_amdgcn_readfirstlane((int)(size_t)(smem + slot * BUF) + lw * 1024);
      lower_half(yes, smem + nslot * BUF, yes, baseA(s + NS), baseB(s + NS), lb);
      slot = nslot;
    }
    for (; s + 1 < nk; ++s) {                // the last NS-1 hand-overs: nothing left to fetch
      const int nslot = slot + 1 == NS ? 0 : slot + 1;
      upper_half(smem + slot * BUF);
      wait_tiles(nk - 2 - s);                // tiles s+2 .. nk-1 may still fly
      __syncthreads();
      lower_half(yes, smem + nslot * BUF, no, nullptr, nullptr, 0);
      slot = nslot;
    }
    upper_half(smem + slot * BUF);
    lower_half(no, nullptr, no, nullptr, nullptr, 0);
    }
  }
  if constexpr (staged_epi(EPI)) {
    write_tile_staged<BM, BN, 64 * NW, V, TM, TN, EPI>(acc, e, m0, n0, wm0, wn0, M, N, smem);
  } else if constexpr (EPI == EPI_F32_UPD) {
    if (e.upd_w) f32_tile_through_lds<BM, BN, NW, V, TM, TN, 0, true>(acc, e, m0, n0, wm0, wn0, M, N, smem);   // workgroup-uniform
    else write_tile<V, TM, TN, EPI>(acc, e, m0 + wm0, n0 + wn0, M, N);
  } else if constexpr (epi_has_resid(EPI) && NW == 8 && RV_RESID_LDS) {
    f32_tile_through_lds<BM, BN, NW, V, TM, TN, 1, EPI == EPI_F32_BIAS_RESID_BF16>(acc, e, m0, n0, wm0, wn0, M, N, smem);
  } else {
    write_tile<V, TM, TN, EPI>(acc, e, m0 + wm0, n0 + wn0, M, N);
  }
}

template <int BM, int BN, int BK, int NS, int NW, int WPE, bool AKM, bool BKM, int EPI>
__global__ __launch_bounds__(64 * NW, WPE) void gemm_dtl_kernel(const uint16_t* __restrict__ A, int64_t lda, int64_t a_bs,
                                                                 const uint16_t* __restrict__ B, int64_t ldb, int64_t b_bs,
                                                                 int M, int N, int K, int tiles_m, int tiles_n,
                                                                 int band_rows, Epi e) {
  int bm, bn;
  tile_of_block(tiles_m, tiles_n, band_rows, bm, bn);
  gemm_dtl_body<BM, BN, BK, NS, NW, AKM, BKM, EPI>(A, lda, a_bs, B, ldb, b_bs, M, N, K, bm, bn, e);
}

// ---- few tiles: the contraction split inside a workgroup ------------------------------------
// A product whose 128x128 or 256x256 tiles do not cover the chip lasts as long as ONE workgroup's
// walk along K: each 32-deep step costs a barrier and what is left of a memory round trip, and most
// CUs have no tile at all.  Here a workgroup of G groups of NW waves takes a smaller tile and group
// g the k-tiles g, g + G, ... of it, each group with its own ring of NS slots - the walk is G times
// shorter and a CU keeps G (NS - 1) k-tiles on the way.  (Interleaved k-tiles, so that the two
// halves of a 128-byte line of a k-contiguous operand are asked for together.)  The G partial
// tiles meet in LDS as fp32 images and are added in group order; the epilogue runs on rows of the image,
// eight columns per lane, with what it reads from memory requested before the partial tiles are parked.
__host__ __device__ constexpr int split_pitch(int bn) { return bn + 4; }   // floats
template <int BM, int BN, int G, int NS> constexpr int split_lds() {
  constexpr int ring = G * NS * (dtl_tile_bytes(BM, 32) + dtl_tile_bytes(BN, 32)), image = G * BM * split_pitch(BN) * 4;
  return ring > image ? ring : image;
}
__device__ __forceinline__ void bf16x8_to_f32(f32x4 (&v)[2], u32x4 b) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    v[h].x = __uint_as_float(b[2 * h] << 16); v[h].y = __uint_as_float(b[2 * h] & 0xFFFF0000u);
    v[h].z = __uint_as_float(b[2 * h + 1] << 16); v[h].w = __uint_as_float(b[2 * h + 1] & 0xFFFF0000u);
  }
}
// eight bf16 at an 8-byte boundary (biases, weight versions, the rounded copy of an fp32 result)
__device__ __forceinline__ u32x4 load8(const uint16_t* p) {
  const u32x2 a = reinterpret_cast<const u32x2*>(p)[0], b = reinterpret_cast<const u32x2*>(p)[1];
  return u32x4{a.x, a.y, b.x, b.y};
}
__device__ __forceinline__ void store8(void* base, int64_t at, u32x4 v) {
  u32x2* p = reinterpret_cast<u32x2*>((uint16_t*)base + at);
  p[0] = u32x2{v.x, v.y}; p[1] = u32x2{v.z, v.w};
}
__device__ __forceinline__ u32x4 f32_to_bf16x8(const f32x4 (&v)[2]) {
  u32x4 o;
  o.x = rv_pack_bf16x2(v[0].x, v[0].y); o.y = rv_pack_bf16x2(v[0].z, v[0].w);
  o.z = rv_pack_bf16x2(v[1].x, v[1].y); o.w = rv_pack_bf16x2(v[1].z, v[1].w);
  return o;
}

template <int BM, int BN, int G, int NW, int NS, bool AKM, bool BKM, int EPI>
__device__ __forceinline__ void gemm_split_body(const uint16_t* __restrict__ A, int64_t lda, int64_t a_bs,
                                                const uint16_t* __restrict__ B, int64_t ldb, int64_t b_bs, int M, int N, int K, int bm, int bn, const Epi& e) {
  constexpr int BK = 32, NT = 64 * NW * G;               // a group's NW waves: NW / 2 (m) x 2 (n)
  constexpr int WM = BM / (NW / 2), WN = BN / 2, TM = WM / 32, TN = WN / 32;
  constexpr int A_BYTES = dtl_tile_bytes(BM, BK), BUF = A_BYTES + dtl_tile_bytes(BN, BK);
  constexpr int NA = Dtl<AKM, BM, BK, NW>::N, NB = Dtl<BKM, BN, BK, NW>::N, LPT = NA + NB;
  static_assert(NS >= 3 && NS <= 5 && LPT * (NS - 2) < 64, "ring");
  const int m0 = bm * BM, n0 = bn * BN;
  const int group = __builtin_amdgcn_readfirstlane(threadIdx.x / (64 * NW)), wave = (threadIdx.x >> 6) % NW, l = threadIdx.x & 63;
  const int wm0 = wave / 2 * WM, wn0 = wave % 2 * WN;
  char* ring = dtl_smem + group * (NS * BUF);

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = 0.f;

  Dtl<AKM, BM, BK, NW> da;
  Dtl<BKM, BN, BK, NW> db;
  dtl_init<AKM, BM, BK, NW>(da, lda, a_bs, m0, M, wave);
  dtl_init<BKM, BN, BK, NW>(db, ldb, b_bs, n0, N, wave);
  const int nk = K / BK, turns = (nk + G - 1) / G;
  const int mine = (nk - group + G - 1) / G;               // k-tiles of this group: group, group + G, ...
  auto issue = [&](int i) {                                // its i-th k-tile into slot i % NS
    const int t = i * G + group;
    const int lb = __builtin_amdgcn_readfirstlane((int)(size_t)(ring + (i % NS) * BUF) + wave * 1024);
    const uint16_t* pa = AKM ? A + (int64_t)t * BK * lda : A + (int64_t)t * a_bs;
    const uint16_t* pb = BKM ? B + (int64_t)t * BK * ldb : B + (int64_t)t * b_bs;
#pragma unroll
    for (int q = 0; q < NA; ++q) dtl_load_s(pa, (unsigned)da.off[q] * 2u, lb + q * NW * 1024);
#pragma unroll
    for (int q = 0; q < NB; ++q) dtl_load_s(pb, (unsigned)db.off[q] * 2u, lb + A_BYTES + q * NW * 1024);
  };
  // The epilogue works on rows of the tile, eight columns per lane.  What it reads from memory is requested here, ahead of
  // the operand tiles: asked for behind the walk along K it was a memory round trip of its own.
  constexpr int CPR = BN / 8, PIECES = (BM * CPR + NT - 1) / NT, PITCH = split_pitch(BN);
  constexpr bool RESID = epi_has_resid(EPI), BIAS = epi_has_bias(EPI), ZIN = EPI == EPI_BF16_DGELU, UPD = EPI == EPI_F32_UPD;
  f32x4 in[PIECES][2];
  u32x4 bias[PIECES], zin[PIECES];
  int64_t at[PIECES];
  bool ok[PIECES];
#pragma unroll
  for (int p = 0; p < PIECES; ++p) {
    const int idx = threadIdx.x + p * NT, row = idx / CPR, gm = m0 + row, gn = n0 + idx % CPR * 8;
    ok[p] = row < BM && gm < M && gn < N;
    const int mc = gm < M ? gm : M - 1, nc = gn < N ? gn : N - 8;
    at[p] = (int64_t)mc * e.ldo + nc;
    if (BIAS) bias[p] = load8(e.bias + nc);
    if (ZIN) zin[p] = *reinterpret_cast<const u32x4*>(e.zin + at[p]);
    if (RESID || (UPD && e.upd_w)) {
      const f32x4* src = reinterpret_cast<const f32x4*>(RESID ? e.resid + (int64_t)mc * e.ldr + nc : e.upd_w + at[p]);
      in[p][0] = src[0]; in[p][1] = src[1];
    }
  }
#pragma unroll
  for (int i = 0; i < NS - 1; ++i)
    if (i < mine) issue(i);
  for (int i = 0; i < turns; ++i) {
    // this group's k-tile i has landed once at most its newer ones are outstanding
    const int newer = mine - 1 - i;
    if (NS >= 5 && newer >= 3) RV_WAIT_VMCNT(LPT * (NS >= 5 ? 3 : 0));
    else if (NS >= 4 && newer >= 2) RV_WAIT_VMCNT(LPT * (NS >= 4 ? 2 : 0));
    else if (newer >= 1) RV_WAIT_VMCNT(LPT);
    else RV_WAIT_VMCNT(0);
    __syncthreads();                                       // every wave's part of it has; everyone left k-tile i - 1
    if (i + NS - 1 < mine) issue(i + NS - 1);
    if (i < mine) {                                        // (wave-uniform)
      const char* curA = ring + (i % NS) * BUF;
      const char* curB = curA + A_BYTES;
      bf16x8 fa[2][TM], fb[2][TN];
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
        for (int a = 0; a < TM; ++a) fa[kk][a] = dtl_frag32<AKM, BM, BK>(curA, wm0 + a * 32, kk);
#pragma unroll
        for (int b = 0; b < TN; ++b) fb[kk][b] = dtl_frag32<BKM, BN, BK>(curB, wn0 + b * 32, kk);
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
          for (int b = 0; b < TN; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[kk][b], fa[kk][a], acc[a][b], 0, 0, 0);
    }
  }
  __syncthreads();                                         // the rings are free
  float* image = reinterpret_cast<float*>(dtl_smem);
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int c = 0; c < 4 * TN; ++c)
      *reinterpret_cast<f32x4*>(image + (group * BM + wm0 + quad_row<f32x16>(i)) * PITCH + wn0 + quad_col<f32x16>(c)) = quad(acc, i, c);
  __syncthreads();
#pragma unroll
  for (int p = 0; p < PIECES; ++p) {
    const int idx = threadIdx.x + p * NT, row = idx / CPR, c = idx % CPR * 8;
    if (BM * CPR % NT != 0 && row >= BM) break;
    f32x4 v[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      v[h] = *reinterpret_cast<const f32x4*>(image + row * PITCH + c + 4 * h);
#pragma unroll
      for (int g = 1; g < G; ++g) v[h] += *reinterpret_cast<const f32x4*>(image + (g * BM + row) * PITCH + c + 4 * h);
    }
    if (BIAS) {
      f32x4 b[2];
      bf16x8_to_f32(b, bias[p]);
      v[0] += b[0]; v[1] += b[1];
    }
    if (ZIN) {
      f32x4 z[2];
      bf16x8_to_f32(z, zin[p]);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int k = 0; k < 4; ++k) v[h][k] = ok[p] ? v[h][k] * dgelu_f(z[h][k]) : 0.f;
      if (e.colpart) {                                     // for the column sums below
        *reinterpret_cast<f32x4*>(image + row * PITCH + c) = v[0];
        *reinterpret_cast<f32x4*>(image + row * PITCH + c + 4) = v[1];
      }
    }
    if (!ok[p]) continue;
    const int gm = m0 + row, gn = n0 + c;
    if (EPI == EPI_BF16 || EPI == EPI_BF16_BIAS || EPI == EPI_BF16_BIAS_GELU)
      *reinterpret_cast<u32x4*>((uint16_t*)e.out + at[p]) = f32_to_bf16x8(v);
    if (EPI == EPI_BF16_DGELU) *reinterpret_cast<u32x4*>((uint16_t*)e.out + e.blocked(gm, gn)) = f32_to_bf16x8(v);
    if (EPI == EPI_BF16_BIAS_GELU) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int k = 0; k < 4; ++k) v[h][k] = gelu_f(v[h][k]);
      *reinterpret_cast<u32x4*>((uint16_t*)e.out2 + e.blocked(gm, gn)) = f32_to_bf16x8(v);
    }
    if (RESID) {
      v[0] += in[p][0]; v[1] += in[p][1];
      if (EPI == EPI_F32_BIAS_RESID_BF16) store8(e.out2, at[p], f32_to_bf16x8(v));
    }
    if ((RESID || EPI == EPI_F32 || UPD) && e.out) {
      f32x4* dst = reinterpret_cast<f32x4*>((float*)e.out + at[p]);
      dst[0] = v[0]; dst[1] = v[1];
    }
    if (UPD && e.upd_w) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int k = 0; k < 4; ++k) v[h][k] = __fmaf_rn(-e.eta, v[h][k], in[p][h][k]);
      f32x4* dst = reinterpret_cast<f32x4*>(e.upd_w + at[p]);
      dst[0] = v[0]; dst[1] = v[1];
      store8(e.out2, e.blocked(gm, gn), f32_to_bf16x8(v));
    }
  }
  if (ZIN && e.colpart) {                                  // (uniform) NT / BN row lanes per column, added in order
    constexpr int RL = NT / BN < 4 ? NT / BN : 4;
    __syncthreads();
    float* part = image + BM * PITCH;
    const int c = threadIdx.x % BN, rl = threadIdx.x / BN;
    if (rl < RL) {
      float s = 0.f;
#pragma unroll 8
      for (int r = rl; r < BM; r += RL) s += image[r * PITCH + c];
      part[rl * BN + c] = s;
    }
    __syncthreads();
    if (rl == 0 && n0 + c < N) {
      float s = part[c];
#pragma unroll
      for (int q = 1; q < RL; ++q) s += part[q * BN + c];
      e.colpart[(int64_t)(m0 / BM) * e.ldo + n0 + c] = s;
    }
  }
}

// Workgroup -> stretch of the contraction and tile: every XCD (workgroup ids go to the 8 of them in turn) takes a contiguous
// range of a stretch's tiles, column by column in bands of up to 8 tile rows, so that a panel of the weights - cold, in HBM -
// is fetched into one or two of the L2s and not into all that hold a tile row.
__device__ __forceinline__ void split_tile(int tiles_m, int tiles_n, int S, int& ks, int& bm, int& bn) {
  const int tiles = tiles_m * tiles_n, total = tiles * S, base = total / 8, rem = total % 8;
  const int g = blockIdx.x % 8, v = g * base + (g < rem ? g : rem) + blockIdx.x / 8;
  ks = v / tiles;
  const int t = v - ks * tiles, band = t / (8 * tiles_n), first = band * 8;
  const int rows = tiles_m - first < 8 ? tiles_m - first : 8, in = t - band * 8 * tiles_n;
  bm = first + in % rows;
  bn = in / rows;
}

template <int BM, int BN, int G, int NW, int NS, bool AKM, bool BKM, int EPI>
__global__ __launch_bounds__(64 * NW * G, NW * G / 4) void gemm_split_kernel(const uint16_t* __restrict__ A, int64_t lda, int64_t a_bs,
                                                                const uint16_t* __restrict__ B, int64_t ldb, int64_t b_bs, int M, int N, int K,
                                                                int tiles_m, int tiles_n, Epi e) {
  int ks, bm, bn;
  split_tile(tiles_m, tiles_n, 1, ks, bm, bn);
  gemm_split_body<BM, BN, G, NW, NS, AKM, BKM, EPI>(A, lda, a_bs, B, ldb, b_bs, M, N, K, bm, bn, e);
}

// ---- few tiles and a long contraction: split over workgroups as well ------------------------
// A product of so few tiles that most CUs have none is cut into S stretches of k-tiles, a workgroup to each tile of each: every
// one stores its sum as fp32 to part[stretch][M][N], and the kernel that reads the result - a LayerNorm, which passes over
// whole rows anyway - adds the S of them in order (norm.hip): no exchange between workgroups, no launch of its own.
template <int BM, int BN, int G, int NW, int NS, bool BKM>
__global__ __launch_bounds__(64 * NW * G, NW * G / 4) void gemm_part_kernel(const uint16_t* __restrict__ A, int64_t lda, int64_t a_bs,
                                                               const uint16_t* __restrict__ B, int64_t ldb, int64_t b_bs, int M, int N, int K,
                                                               int tiles_m, int tiles_n, int S, float* part) {
  int ks, bm, bn;
  split_tile(tiles_m, tiles_n, S, ks, bm, bn);
  const int nk = K / 32, t0 = nk * ks / S, t1 = nk * (ks + 1) / S;
  Epi e{part + (int64_t)ks * M * N, N, nullptr, nullptr, nullptr, 0, nullptr, nullptr, 0.f, nullptr, 0, 0};
  gemm_split_body<BM, BN, G, NW, NS, false, BKM, EPI_F32>(A + t0 * a_bs, lda, a_bs, B + t0 * (BKM ? 32 * ldb : b_bs), ldb, b_bs,
                                                          M, N, (t1 - t0) * 32, bm, bn, e);
}

// Several independent products of one kind in a single launch (the four weight-gradient
// products of a decoder block): a workgroup finds its problem from the running tile count.
// One launch fills the chip where four small grids would each leave most CUs idle.
struct GroupedProblem {
  const uint16_t* A; const uint16_t* B; float* out;
  float* upd_w; uint16_t* upd_ver; float eta;
  int lda, a_bs, ldb, b_bs, ldo, ldv, bsv, M, N, K, tiles_m, tiles_n, first_tile;   // ldv, bsv: of the weight version
};
template <int MAX>
struct GroupedArgs {
  GroupedProblem p[MAX];
  int count;
};

// the problem, tile row and tile column of a workgroup
template <int MAX>
__device__ __forceinline__ const GroupedProblem& grouped_tile(const GroupedArgs<MAX>& ga, int& bm, int& bn) {
  // Workgroup ids are dealt to the 8 XCDs in turn, and each XCD pulls its operand panels
  // through its own L2.  Give XCD g a CONTIGUOUS range of the tile numbering (so it works on
  // one problem at a time, not on a slice of all of them) and number a problem's tiles in bands
  // of two tile rows, column by column (so a run of 8 tiles is a 2 x 4 patch: 6 operand panels).
  const int total = gridDim.x, base = total / 8, rem = total % 8;
  const int g = blockIdx.x % 8, i = blockIdx.x / 8;
  const int v = g * base + (g < rem ? g : rem) + i;
  int pi = 0;
#pragma unroll
  for (int k = 1; k < MAX; ++k)
    if (k < ga.count && v >= ga.p[k].first_tile) pi = k;
  const GroupedProblem& q = ga.p[pi];
  const int local = v - q.first_tile;
  constexpr int GB = 2;
  const int band = local / (GB * q.tiles_n), first_row = band * GB;
  const int rows = q.tiles_m - first_row < GB ? q.tiles_m - first_row : GB;
  const int in = local - band * GB * q.tiles_n;
  bm = first_row + in % rows;
  bn = in / rows;
  return q;
}
__device__ __forceinline__ Epi grouped_epi(const GroupedProblem& q) {
  return Epi{q.out, q.ldo, q.upd_ver, nullptr, nullptr, 0, nullptr, q.upd_w, q.eta, nullptr, q.ldv, q.bsv};
}

template <int BM, int BN, int BK, int NS, int NW, int WPE>
__global__ __launch_bounds__(64 * NW, WPE) void gemm_dtl_grouped_wgrad_kernel(GroupedArgs<RV_GEMM_GROUP_BLOCK> ga) {
  int bm, bn;
  const GroupedProblem& q = grouped_tile(ga, bm, bn);
  gemm_dtl_body<BM, BN, BK, NS, NW, true, true, EPI_F32_UPD>(q.A, q.lda, q.a_bs, q.B, q.ldb, q.b_bs, q.M, q.N, q.K, bm, bn, grouped_epi(q));
}
template <int BM, int BN, int G, int NW, int NS, int MAX>
__global__ __launch_bounds__(64 * NW * G, NW * G / 4) void gemm_split_grouped_wgrad_kernel(GroupedArgs<MAX> ga) {
  int bm, bn;
  const GroupedProblem& q = grouped_tile(ga, bm, bn);
  gemm_split_body<BM, BN, G, NW, NS, true, true, EPI_F32_UPD>(q.A, q.lda, q.a_bs, q.B, q.ldb, q.b_bs, q.M, q.N, q.K, bm, bn, grouped_epi(q));
}

template <int BM, int BN, int BK, int NS, int NW, int WPE, bool AKM, bool BKM, int EPI>
rv_status launch_dtl(const rv_gemm_args& g, hipStream_t st) {
  constexpr int ring = NS * (dtl_tile_bytes(BM, BK) + dtl_tile_bytes(BN, BK));
  // the GELU' epilogue keeps two rows of fp32 column sums (one per wave row) behind the image
  constexpr int image = staged_epi(EPI) ? BM * stage_pitch(BN) + (EPI == EPI_BF16_DGELU ? 2 * BN * 4 : 0)
                        : (epi_has_resid(EPI) && NW == 8 && BM == 256 && BN == 256 ? upd_image_bytes(BM, BN) : 0);
  constexpr int smem = ring > image ? ring : image;
  auto kern = gemm_dtl_kernel<BM, BN, BK, NS, NW, WPE, AKM, BKM, EPI>;
  // once per instantiation; a function-local static is initialised exactly once, also under threads
  static const hipError_t configured =
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  if (configured != hipSuccess) return RV_E_DEVICE;
  int tm = (g.M + BM - 1) / BM, tn = (g.N + BN - 1) / BN;
  Epi e{g.out, g.ldo, g.out2, g.bias, g.resid, g.ldr, g.zin, nullptr, 0.f, g.epi == EPI_BF16_DGELU ? g.colpart : nullptr,
        g.bsv ? 32 : g.ldo, g.bsv ? g.bsv : 32};
  g.colpart_rows = (g.M + BM - 1) / BM;
  const int ntiles = tm * tn;
  // Measured: alone, the XCD-banded map pays only for the small tile.  Inside a stage step a
  // launch holds about a third of every XCD's CUs, and what an XCD runs of it at one time should
  // share operand panels: bands of 8 tile rows (2 for 32 or more tile rows, either tile size)
  // against the natural order: stage steps -1.3 % / -0.6 % / -1.9 % (d 1600 / 2048 / 1024).
  int band = 8;
  if (g.sharing != 0) band = tm >= 32 ? 2 : 8;
  else if (!(BM == 128 && BN == 128)) tm = -tm;
  hipLaunchKernelGGL(kern, dim3(ntiles), dim3(64 * NW), smem, st, g.A, g.lda, g.a_bs, g.B, g.ldb, g.b_bs, g.M, g.N, g.K,
                     tm, tn, band, e);
  return rv_launch_status();
}

template <int BM, int BN, int G, int NW, int NS, bool AKM, bool BKM, int EPI>
rv_status launch_split(const rv_gemm_args& g, hipStream_t st) {
  constexpr int smem = split_lds<BM, BN, G, NS>();
  static_assert(smem <= 160 * 1024, "LDS of one CU");
  auto kern = gemm_split_kernel<BM, BN, G, NW, NS, AKM, BKM, EPI>;
  static const hipError_t configured =
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  if (configured != hipSuccess) return RV_E_DEVICE;
  const int tm = (g.M + BM - 1) / BM, tn = (g.N + BN - 1) / BN;
  Epi e{g.out, g.ldo, g.out2, g.bias, g.resid, g.ldr, g.zin, nullptr, 0.f, g.epi == EPI_BF16_DGELU ? g.colpart : nullptr,
        g.bsv ? 32 : g.ldo, g.bsv ? g.bsv : 32};
  g.colpart_rows = tm;
  hipLaunchKernelGGL(kern, dim3(tm * tn), dim3(64 * NW * G), smem, st, g.A, g.lda, g.a_bs, g.B, g.ldb, g.b_bs, g.M, g.N, g.K, tm, tn, e);
  return rv_launch_status();
}

template <int BM, int BN, int G, int NW, int NS, bool BKM>
rv_status launch_part(const rv_gemm_args& g, int S, float* part, hipStream_t st) {
  constexpr int smem = split_lds<BM, BN, G, NS>();
  static_assert(smem <= 160 * 1024, "LDS of one CU");
  auto kern = gemm_part_kernel<BM, BN, G, NW, NS, BKM>;
  static const hipError_t configured =
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  if (configured != hipSuccess) return RV_E_DEVICE;
  const int tm = (g.M + BM - 1) / BM, tn = (g.N + BN - 1) / BN;
  hipLaunchKernelGGL(kern, dim3(tm * tn * S), dim3(64 * NW * G), smem, st, g.A, g.lda, g.a_bs, g.B, g.ldb, g.b_bs, g.M, g.N, g.K, tm, tn, S, part);
  return rv_launch_status();
}
template <bool BKM>
rv_status pick_part(const rv_gemm_args& g, int S, float* part, hipStream_t st) {
  switch (g.tile) {
    case 1032: return launch_part<32, 64, 8, 2, 3, BKM>(g, S, part, st);
    case 1064: return launch_part<64, 64, 4, 4, 4, BKM>(g, S, part, st);
    case 1065: return launch_part<64, 64, 2, 4, 4, BKM>(g, S, part, st);
    case 1128: return launch_part<128, 128, 2, 4, 4, BKM>(g, S, part, st);
  }
  return RV_E_INVAL;
}

// Tile choice (codes: 5256, 2256, 2192, 2128, 1128, 1065, 1064, 1032).
//   5256  256x256, eight waves of 128x64, BK 32, ring of four slots run in the pipelined form
//         (three tiles in flight, loads dealt out behind the MFMAs), one workgroup per CU:
//         lowest LDS traffic per MFMA, two waves per SIMD cover each other's stalls;
//   2192  128x256, four waves of 64x128, ring of three slots, two workgroups per CU;
//   2128  128x128, four waves of 64x64, ring of four slots, two workgroups per CU;
//   1128  128x128, 1065 / 1064 64x64, 1032 32x64: the contraction split inside the workgroup over
//         2, 2 / 4 and 8 groups of waves.
// The automatic choice among the first three minimises  rounds * tile area * workgroups per CU / efficiency,
// rounds = ceil(tiles / (256 CUs * workgroups per CU)), efficiencies ratios of times before 2192 and 2128 had
// the pipelined ring, 2192's 0.92 -> 0.98 with it (us, bound loads / ring: 4096x1024x4096 2128 43.7 / 38.0, 4096x6144x2048 2192 116 / 98,
// 8192x1600x6400 2192 189 / 154; 5256 75, 103, 150).  Over 200 launches of 512 .. 8192 rows and 256 .. 8192 in k alone on average 2.1 % above
// the best of the three (0.3 % before the ring; 3.0 % from 64 tiles of 256x256 on), most on short contractions: 6784x7552x256 with GELU 91 where
// 2128 takes 69, 5120x6848x1024 85 / 72 (2192).
// Whether the contraction is split is decided by the modelled time, us,
//   rounds * (f + turns * t) + out * M N / 1e6,  turns = k-tiles per group,
// t between t0 (a launch that leaves most CUs idle) and t1 (one that fills them; with 2192 and 2128 as they were before the pipelined ring:
// with 0.88 of their times four microbatches of 6 blocks of d 768, 1152 tokens take 0.2 - 0.5 % longer), fitted to 488 launches of 64 .. 8192 rows
// alone, operands in blocks of columns, weights cold.  A product of few tiles is one walk along K: 256x448x1792 takes 43 us
// with 5256, 22 with 2128 and 7 with 1032; 512x4096x1024 with GELU' 32 / 17 / 11 (1065); 1152x768x3072 65 / 36 / 14 (1064);
// 1152x2048x8192 152 / 108 / 72 (1128); 2048x1024x4096 82 / 44 / 29 (1065); 8192x6400x1600 183 / 204 / 261.
// A split form is taken where the model has it a tenth faster, on the shape alone, so that a product has the same bits beside
// other streams as by itself; and not from 64 tiles of 256x256 on: it takes more CU time per flop, which the other streams
// of a step could have used.  Stage steps, split where a tenth faster / not from 64 tiles on / nowhere, us:
//   4 blocks d 1024, 4096 tokens 1762 / 1718 / 1714    6 blocks d 768, 1152 tokens, 4 microbatches 4847 / 4850 / 5260
//   8 blocks d 832, 2048 tokens  1535 / 1443           9 blocks d 896, 4032 tokens (64 tiles)     3382 / 3520
//   12 blocks d 640, 2880 tokens 2230 / - / 2400       7 blocks d 1536, 1536 tokens, 2 microbatches 5890 / - / 6230
struct TileForm { int code, bm, bn, k, per_cu; float f, t0, t1, out; };
constexpr TileForm kForms[] = {
    {5256, 256, 256, 32, 1, 8.9f, 0.51f, 0.64f, 0.63f}, {2192, 128, 256, 32, 2, 6.1f, 0.45f, 0.77f, 0.66f},
    {2128, 128, 128, 64, 2, 3.1f, 0.65f, 0.91f, 0.77f}, {1128, 128, 128, 64, 1, 4.3f, 0.47f, 0.48f, 0.68f},
    {1065, 64, 64, 64, 2, 3.1f, 0.27f, 0.37f, 0.50f},   {1064, 64, 64, 128, 1, 3.9f, 0.43f, 0.40f, 0.11f},
    {1032, 32, 64, 256, 1, 3.3f, 0.66f, 0.57f, 0.f}};
// the modelled time of a form whose contraction is cut into S stretches
float form_time(const TileForm& c, int M, int N, int K, int S) {
  const float tiles = (float)((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn) * S, slots = 256.f * c.per_cu;
  const float fill = tiles < slots ? tiles / slots : 1.f;
  return ceilf(tiles / slots) * (c.f + ceilf((float)K / S / c.k) * (c.t0 + (c.t1 - c.t0) * fill * fill)) + c.out * 1e-6f * M * N * S;
}
int in_order_form(int M, int N) {
  auto cost = [&](int bm, int bn, int bpc, double eff) {
    const long tiles = (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn);
    return (double)((tiles + 256 * bpc - 1) / (256 * bpc)) * bm * bn * bpc / eff;
  };
  const double c256 = cost(256, 256, 1, 1.0), c192 = cost(128, 256, 2, 0.98), c128 = cost(128, 128, 2, 0.83);
  return c256 <= c192 && c256 <= c128 ? 5256 : c192 <= c128 ? 2192 : 2128;
}
// the form of a whole product where nobody shares the chip, and its modelled time (k32: form 1032 is there)
int whole_form(int M, int N, int K, bool k32, float& time) {
  int best = in_order_form(M, N);
  for (const TileForm& c : kForms)
    if (c.code == best) time = form_time(c, M, N, K, 1);
  if (((M + 255) / 256) * ((N + 255) / 256) >= 64) return best;
  float least = 0.9f * time;
  for (const TileForm& c : kForms) {
    if (c.code >= 2000 || (c.code == 1032 && !k32)) continue;
    const float t = form_time(c, M, N, K, 1);
    if (t < least) { best = c.code; least = time = t; }
  }
  return best;
}

template <bool AKM, bool BKM, int EPI>
rv_status pick_tile(const rv_gemm_args& g, hipStream_t st) {
  int tile = g.tile;
  if (tile == 0) {
    float time;   // (whether the contraction is split: by the shape alone)
    tile = whole_form(g.M, g.N, g.K, !AKM, time);
    const long t256 = (long)((g.M + 255) / 256) * ((g.N + 255) / 256);
    // Measured inside the stage step (d = 1024, 1600, 2048): what a launch leaves of the chip is
    // used by the other streams, so CU time per flop counts for more than its own duration.
    if (tile >= 2000 && (g.sharing == 2 || (g.sharing && t256 >= 128))) tile = 5256;
  }
  if constexpr (!AKM) {
    if (tile == 1032) return launch_split<32, 64, 8, 2, 3, AKM, BKM, EPI>(g, st);
  }
  if (tile == 1064) return launch_split<64, 64, 4, 4, 4, AKM, BKM, EPI>(g, st);
  if (tile == 1065) return launch_split<64, 64, 2, 4, 4, AKM, BKM, EPI>(g, st);
  if (tile == 1128) return launch_split<128, 128, 2, 4, 4, AKM, BKM, EPI>(g, st);
  if (tile == 2256) return launch_dtl<256, 256, 32, 4, 4, 1, AKM, BKM, EPI>(g, st);
  if (tile == 2192) return launch_dtl<128, 256, 32, 3, 4, 2, AKM, BKM, EPI>(g, st);
  if (tile == 2128) return launch_dtl<128, 128, 32, 4, 4, 2, AKM, BKM, EPI>(g, st);
  if (tile == 5256) return launch_dtl<256, 256, 32, 4, 8, 2, AKM, BKM, EPI>(g, st);
  return RV_E_INVAL;
}

}  // namespace

namespace {
// tile offsets are kept in 32 bits, and a matrix in blocks of columns is whole blocks
bool operand_fits(const rv_gemm_args& g) {
  auto fits = [](int64_t rows, int64_t cols, int64_t ld, int64_t bs) {
    if (bs == 32) return rows * ld < (1ll << 31);
    return ld == 32 && bs == rows * 32 && cols % 32 == 0 && rows * cols < (1ll << 31);
  };
  return (g.a_kmajor ? fits(g.K, g.M, g.lda, g.a_bs) : fits(g.M, g.K, g.lda, g.a_bs)) &&
         (g.b_kmajor ? fits(g.K, g.N, g.ldb, g.b_bs) : fits(g.N, g.K, g.ldb, g.b_bs)) &&
         (!g.bsv || (g.bsv == (int64_t)g.M * 32 && g.N % 32 == 0 && (int64_t)g.M * g.N < (1ll << 31)));
}
}  // namespace

rv_status rv_gemm_bf16(const rv_gemm_args& g, hipStream_t st) {
  if (!g.A || !g.B || !g.out || g.M < 8 || g.N < 8 || g.K < 64) return RV_E_INVAL;
  if (g.K % 64 || g.N % 8 || g.M % 8 || g.lda % 8 || g.ldb % 8 || g.ldo % 4) return RV_E_INVAL;
  if ((((uintptr_t)g.A) | ((uintptr_t)g.B) | ((uintptr_t)g.out)) & 15) return RV_E_INVAL;
  // bf16 outputs (and the pre-activation input of GELU') move in 16-byte row pieces: pitch % 8
  if ((staged_epi(g.epi) || g.epi == EPI_F32_BIAS_RESID_BF16) && g.ldo % 8) return RV_E_INVAL;
  if (staged_epi(g.epi) && g.epi == EPI_BF16_BIAS_GELU && (((uintptr_t)g.out2) & 15)) return RV_E_INVAL;
  if (g.epi == EPI_BF16_DGELU && (((uintptr_t)g.zin) & 15)) return RV_E_INVAL;
  if (!operand_fits(g)) return RV_E_INVAL;
  const bool need_bias = g.epi == EPI_BF16_BIAS || g.epi == EPI_F32_BIAS_RESID ||
                         g.epi == EPI_BF16_BIAS_GELU || g.epi == EPI_F32_BIAS_RESID_BF16;
  if (need_bias && (!g.bias || (((uintptr_t)g.bias) & 7))) return RV_E_INVAL;
  if ((g.epi == EPI_F32_BIAS_RESID || g.epi == EPI_F32_BIAS_RESID_BF16) &&
      (!g.resid || g.ldr % 4 || (((uintptr_t)g.resid) & 15)))
    return RV_E_INVAL;
  if ((g.epi == EPI_BF16_BIAS_GELU || g.epi == EPI_F32_BIAS_RESID_BF16) && !g.out2) return RV_E_INVAL;
  if (g.epi == EPI_BF16_DGELU && !g.zin) return RV_E_INVAL;
  // only the layout/epilogue pairs the stage uses are instantiated
  if (!g.a_kmajor && g.b_kmajor) {          // forward products
    switch (g.epi) {
      case EPI_BF16_BIAS: return pick_tile<false, true, EPI_BF16_BIAS>(g, st);
      case EPI_F32_BIAS_RESID: return pick_tile<false, true, EPI_F32_BIAS_RESID>(g, st);
      case EPI_F32_BIAS_RESID_BF16: return pick_tile<false, true, EPI_F32_BIAS_RESID_BF16>(g, st);
      case EPI_BF16_BIAS_GELU: return pick_tile<false, true, EPI_BF16_BIAS_GELU>(g, st);
    }
  } else if (!g.a_kmajor && !g.b_kmajor) {  // input-gradient products
    switch (g.epi) {
      case EPI_BF16: return pick_tile<false, false, EPI_BF16>(g, st);
      case EPI_BF16_DGELU: return pick_tile<false, false, EPI_BF16_DGELU>(g, st);
    }
  } else if (g.a_kmajor && g.b_kmajor) {    // weight-gradient products
    if (g.epi == EPI_F32) return pick_tile<true, true, EPI_F32>(g, st);
  }
  return RV_E_INVAL;
}

// The form and the number of stretches of a product whose partial sums the next kernel can add: the least modelled time,
// with 4 bytes per partial sum read back at 5 TB/s, if that takes a tenth off the best whole product; S = 1: none does.
// Weights cold, best whole form / cut (with the reading back), us: 64x2048x8192 30.1 / 11.3 (64x64 tiles, S 8), 128x1024x4096
// 11.6 / 7.1 (32x64, 4), 1024x2048x8192 66.9 / 46.0 (128x128, 2), 1152x1600x6400 50.2 / 35.7,
// 256x448x1792 7.2 / 5.9.  Over 130 products of 64 .. 2048 rows the modelled ratio is below the measured one by 0.1 .. 0.2 on the
// short walks and above it by as much on the long ones; a modelled tenth was 0 .. 30 % measured.
// Four stages of 4 blocks of d 1024 on 128 tokens, forward and backward, with their average 3137 -> 2761 us, stage step of 12
// blocks of d 448 on 256 tokens 924 -> 852 us (with what split_tile and the early requests give).
// Not from 64 tiles of 256x256 on, as with the split forms of whole products.  Stage steps, cut / whole, us: 4 blocks d 2048, 2048 tokens
// 3367 / 3069, 2 of d 4096, 4608 tokens 11080 / 9200 (separate calls 11530 / 10910), 3 of d 4096, 1024 tokens 4537 / 4262 (separate
// calls 4853 / 5017: the one form that loses).  Below, cut against the forms without: 4 of d 2048, 1024 tokens 2100 / 2550, of
// d 1600, 2048 tokens (56 tiles) 2170 / 2344, of d 1024, 3072 tokens (48) 1390 / 1513.
rv_part_form rv_gemm_part_form(int M, int N, int K) {
  float whole;
  whole_form(M, N, K, true, whole);
  rv_part_form best = {0, 1};
  if (((M + 255) / 256) * ((N + 255) / 256) >= 64) return best;
  float least = 0.9f * whole;
  for (const TileForm& c : kForms) {
    if (c.code >= 2000) continue;
    for (int S = 2; S <= RV_GEMM_PARTS_MAX && S * c.k <= K; S *= 2) {
      const float time = form_time(c, M, N, K, S) + (float)M * N * S * 4.f / 5e6f;   // (written: in the form's own time)
      if (time < least) { least = time; best = {c.code, S}; }
    }
  }
  return best;
}

// the product's operands as in g (a_kmajor 0), its sums over S stretches of the contraction to part[S][M][N]
rv_status rv_gemm_part(const rv_gemm_args& g, int S, float* part, hipStream_t st) {
  if (!g.A || !g.B || !part || g.a_kmajor || g.M < 8 || g.N < 8 || g.K < 64 || S < 1 || S > RV_GEMM_PARTS_MAX || S > g.K / 32) return RV_E_INVAL;
  if (g.K % 64 || g.N % 8 || g.M % 8 || g.lda % 8 || g.ldb % 8) return RV_E_INVAL;
  if ((((uintptr_t)g.A) | ((uintptr_t)g.B) | ((uintptr_t)part)) & 15) return RV_E_INVAL;
  if (!operand_fits(g)) return RV_E_INVAL;
  return g.b_kmajor ? pick_part<true>(g, S, part, st) : pick_part<false>(g, S, part, st);
}

namespace {
template <int MAX>
rv_status launch_grouped(void (*kern)(GroupedArgs<MAX>), int BM, int BN, int threads, int smem, const rv_gemm_args* gs, int count,
                         hipStream_t st) {
  GroupedArgs<MAX> ga;
  int tiles = 0;
  for (int k = 0; k < count; ++k) {
    const rv_gemm_args& g = gs[k];
    GroupedProblem& q = ga.p[k];
    q.A = g.A; q.B = g.B; q.out = g.store_out ? (float*)g.out : nullptr;
    q.upd_w = g.upd_w; q.upd_ver = g.upd_ver; q.eta = g.upd_eta;
    q.lda = (int)g.lda; q.a_bs = (int)g.a_bs; q.ldb = (int)g.ldb; q.b_bs = (int)g.b_bs; q.ldo = (int)g.ldo;
    q.ldv = (int)(g.bsv ? 32 : g.ldo); q.bsv = (int)(g.bsv ? g.bsv : 32);
    q.M = g.M; q.N = g.N; q.K = g.K;
    q.tiles_m = (g.M + BM - 1) / BM;
    q.tiles_n = (g.N + BN - 1) / BN;
    q.first_tile = tiles;
    tiles += q.tiles_m * q.tiles_n;
  }
  for (int k = count; k < MAX; ++k) ga.p[k] = ga.p[0];
  ga.count = count;
  hipLaunchKernelGGL(kern, dim3(tiles), dim3(threads), smem, st, ga);
  return rv_launch_status();
}
template <int BM, int BN, int BK, int NS, int NW>
rv_status launch_grouped_dtl(const rv_gemm_args* gs, int count, hipStream_t st) {
  constexpr int ring = NS * (dtl_tile_bytes(BM, BK) + dtl_tile_bytes(BN, BK));
  constexpr int smem = ring > upd_image_bytes(BM, BN) ? ring : upd_image_bytes(BM, BN);
  static_assert(smem <= 160 * 1024, "LDS of one CU");
  auto kern = gemm_dtl_grouped_wgrad_kernel<BM, BN, BK, NS, NW, 2>;
  static const hipError_t configured =
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  if (configured != hipSuccess) return RV_E_DEVICE;
  return launch_grouped(kern, BM, BN, 64 * NW, smem, gs, count, st);
}
template <int BM, int BN, int G, int NW, int NS, int MAX>
rv_status launch_grouped_split(const rv_gemm_args* gs, int count, hipStream_t st) {
  constexpr int smem = split_lds<BM, BN, G, NS>();
  static_assert(smem <= 160 * 1024, "LDS of one CU");
  auto kern = gemm_split_grouped_wgrad_kernel<BM, BN, G, NW, NS, MAX>;
  static const hipError_t configured =
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  if (configured != hipSuccess) return RV_E_DEVICE;
  return launch_grouped(kern, BM, BN, 64 * NW * G, smem, gs, count, st);
}
}  // namespace

namespace {
int tiles_of(int count, const int* M, const int* N, int edge) {
  int tiles = 0;
  for (int k = 0; k < count; ++k) tiles += ((M[k] + edge - 1) / edge) * ((N[k] + edge - 1) / edge);
  return tiles;
}
}  // namespace

// 256x256 tiles, eight waves (measured against 128x128 and 128x256 tiles, alone and inside the
// stage step of d 1024, 2048 and 1600: fewest LDS bytes per MFMA, so it takes the least CU time
// from the kernels that run beside it, and the step is 3-4 % shorter)
// A block whose 256x256 tiles do not cover the chip and whose walk along the tokens is short takes
// 128x128 tiles with the walk split in two, four times as many: 24 -> 12 us (d 448, ffn 1792, 256
// tokens, 44 tiles), 37 -> 34 us (768, 3072, 1152 tokens, 108); even at 30 us with 128 tokens of a
// 1024-wide block, where the update's 126 MB bound it.  Longer walks keep the CU time per flop down: stage steps of
// four blocks, ms, split / in order (the separate calls differ the same way):
//   tokens           512          1024         1536         2048         3072         4096
//   d 1024   0.710/0.732  0.870/0.876  1.090/1.074  1.240/1.220  1.584/1.535  1.979/1.881
//   d 768    0.514/0.520  0.656/0.651  0.772/0.786  0.917/0.904  1.156/1.095  1.377/1.357
//   d 448    0.390/0.410  0.425/0.443  0.486/0.496  0.531/0.568  0.669/0.690  0.786/0.818
// From RV_WGRAD_SPLIT_K tokens on the split form where the model of the forms has the whole block a quarter faster: that is a narrow
// one, whose 256x256 tiles are a tenth of the chip.  Stage steps, in order / split, us: d 128, 4032 tokens 726 / 539; d 320, 6272 tokens 2266 /
// 2000; d 256, 2688 tokens 1226 / 1164; d 448, 4160 tokens, four microbatches in separate calls 4340 / 3915; the one
// seen to lose, d 384 on 3584 tokens in separate calls, 2443 / 2500.
// Asked for the four products of a block together, however many launches they leave in (the few tiles that a wide block sends by
// themselves share the chip with the others: dWo of d 1600, 8192 tokens, 49 tiles, split 11 ms of CU time, in order 7; stage step
// 21.53 / 21.43 and, another run, 21.39 / 21.37 ms),
// and for what leaves last by itself, with nothing behind it to share the chip (decoder.hip).
rv_wgrad_form rv_gemm_wgrad_form(int count, const int* M, const int* N, int K) {
  const int tiles = tiles_of(count, M, N, 256), small = tiles_of(count, M, N, 128);
  const float whole = ceilf(tiles / 256.f) * (8.9f + K / 32 * 0.55f), split = ceilf(small / 256.f) * (4.3f + K / 64 * 0.48f);
  return tiles < 256 && (K < RV_WGRAD_SPLIT_K || split < 0.75f * whole) ? RV_WGRAD_SPLIT : RV_WGRAD_IN_ORDER;
}

rv_status rv_gemm_wgrad_grouped(const rv_gemm_args* gs, int count, hipStream_t st, rv_wgrad_form form) {
  if (!gs || count < 1 || count > (form == RV_WGRAD_SPLIT ? RV_GEMM_GROUP_MAX : RV_GEMM_GROUP_BLOCK)) return RV_E_INVAL;
  for (int k = 0; k < count; ++k) {
    const rv_gemm_args& g = gs[k];
    if (!g.A || !g.B || !g.out || !g.a_kmajor || !g.b_kmajor || g.epi != EPI_F32) return RV_E_INVAL;
    if (g.M < 8 || g.N < 8 || g.K < 64 || g.K % 64 || g.N % 8 || g.M % 8 || g.lda % 8 || g.ldb % 8 || g.ldo % 4)
      return RV_E_INVAL;
    if ((((uintptr_t)g.A) | ((uintptr_t)g.B) | ((uintptr_t)g.out)) & 15) return RV_E_INVAL;
    if (!operand_fits(g)) return RV_E_INVAL;
    if ((g.upd_w != nullptr) != (g.upd_ver != nullptr)) return RV_E_INVAL;
    if (!g.upd_w && !g.store_out) return RV_E_INVAL;
    if ((((uintptr_t)g.upd_w) & 15) || (((uintptr_t)g.upd_ver) & 7)) return RV_E_INVAL;
  }
  if (form == RV_WGRAD_BY_TOKENS) {
    int M[RV_GEMM_GROUP_BLOCK], N[RV_GEMM_GROUP_BLOCK];
    for (int k = 0; k < count; ++k) { M[k] = gs[k].M; N[k] = gs[k].N; }
    form = gs[0].K < RV_WGRAD_SPLIT_K && tiles_of(count, M, N, 256) < 256 ? RV_WGRAD_SPLIT : RV_WGRAD_IN_ORDER;
  }
  if (form == RV_WGRAD_IN_ORDER) return launch_grouped_dtl<256, 256, 32, 4, 8>(gs, count, st);
  return count > RV_GEMM_GROUP_BLOCK ? launch_grouped_split<128, 128, 2, 4, 4, RV_GEMM_GROUP_MAX>(gs, count, st)
                                     : launch_grouped_split<128, 128, 2, 4, 4, RV_GEMM_GROUP_BLOCK>(gs, count, st);
}

extern "C" rv_status rv_k_gemm_bf16(const void* A, int64_t lda, int a_kmajor, const void* B, int64_t ldb,
                                    int b_kmajor, int M, int N, int K, int epilogue, void* out, int64_t ldo,
                                    void* out2, const void* bias, const float* resid, int64_t ldr,
                                    const void* zin, int tile, void* stream) {
  rv_gemm_args g;
  g.A = (const uint16_t*)A; g.lda = lda; g.a_kmajor = a_kmajor;
  g.B = (const uint16_t*)B; g.ldb = ldb; g.b_kmajor = b_kmajor;
  g.M = M; g.N = N; g.K = K; g.epi = epilogue; g.out = out; g.ldo = ldo; g.out2 = out2;
  g.bias = (const uint16_t*)bias; g.resid = resid; g.ldr = ldr; g.zin = (const uint16_t*)zin; g.tile = tile;
  return rv_gemm_bf16(g, (hipStream_t)stream);
}

extern "C" rv_status rv_k_gemm_bf16_blocks(const void* A, int a_blocks, int a_kmajor, const void* B, int b_blocks, int b_kmajor, int M,
                                           int N, int K, int epilogue, void* out, void* out2, int out_blocks, const void* bias,
                                           const float* resid, const void* zin, int tile, int parts, void* stream) {
  if (M < 1 || N < 1 || K < 1 || (out_blocks && epilogue != EPI_BF16_BIAS_GELU && epilogue != EPI_BF16_DGELU)) return RV_E_INVAL;
  auto operand = [](const void* p, int blocks, int64_t rows, int64_t cols) { return blocks ? rv_blocks(p, rows) : rv_rows(p, cols); };
  const rv_mat a = a_kmajor ? operand(A, a_blocks, K, M) : operand(A, a_blocks, M, K);
  const rv_mat b = b_kmajor ? operand(B, b_blocks, K, N) : operand(B, b_blocks, N, K);
  rv_gemm_args g;
  g.A = a.p; g.lda = a.ld; g.a_bs = a.bs; g.a_kmajor = a_kmajor;
  g.B = b.p; g.ldb = b.ld; g.b_bs = b.bs; g.b_kmajor = b_kmajor;
  g.M = M; g.N = N; g.K = K; g.epi = epilogue; g.out = out; g.ldo = N; g.out2 = out2; g.bsv = out_blocks ? (int64_t)M * 32 : 0;
  g.bias = (const uint16_t*)bias; g.resid = resid; g.ldr = N; g.zin = (const uint16_t*)zin; g.tile = tile;
  return parts ? rv_gemm_part(g, parts, (float*)out, (hipStream_t)stream) : rv_gemm_bf16(g, (hipStream_t)stream);
}

extern "C" rv_status rv_k_gemm_part_form(int M, int N, int K, int* tile, int* parts) {
  if (!tile || !parts || M < 8 || N < 8 || K < 64) return RV_E_INVAL;
  const rv_part_form form = rv_gemm_part_form(M, N, K);
  *tile = form.tile;
  *parts = form.S;
  return RV_OK;
}

extern "C" rv_status rv_k_gemm_part(const void* A, int64_t lda, const void* B, int64_t ldb, int b_kmajor, int M, int N, int K,
                                    int tile, int parts, float* part, void* stream) {
  rv_gemm_args g;
  g.A = (const uint16_t*)A; g.lda = lda; g.B = (const uint16_t*)B; g.ldb = ldb; g.b_kmajor = b_kmajor;
  g.M = M; g.N = N; g.K = K; g.tile = tile;
  return rv_gemm_part(g, parts, part, (hipStream_t)stream);
}

extern "C" rv_status rv_k_gemm_wgrad_grouped(int count, const void* const* X, const int64_t* lda,
                                             const void* const* dY, const int64_t* ldb, const int* M, const int* N,
                                             int K, float* const* dW, void* stream) {
  if (count < 1 || count > RV_GEMM_GROUP_BLOCK || !X || !lda || !dY || !ldb || !M || !N || !dW) return RV_E_INVAL;
  rv_gemm_args g[RV_GEMM_GROUP_BLOCK];
  for (int k = 0; k < count; ++k) {
    g[k].A = (const uint16_t*)X[k]; g[k].lda = lda[k]; g[k].a_kmajor = 1;
    g[k].B = (const uint16_t*)dY[k]; g[k].ldb = ldb[k]; g[k].b_kmajor = 1;
    g[k].M = M[k]; g[k].N = N[k]; g[k].K = K; g[k].epi = EPI_F32; g[k].out = dW[k]; g[k].ldo = N[k];
  }
  return rv_gemm_wgrad_grouped(g, count, (hipStream_t)stream, RV_WGRAD_IN_ORDER);
}

extern "C" rv_status rv_k_gemm_wgrad_update(int count, const void* const* X, const int64_t* lda, const void* const* dY,
                                            const int64_t* ldb, const int* M, const int* N, int K, float* const* dW,
                                            float* const* w, void* const* ver, float eta, void* stream) {
  if (count < 1 || count > RV_GEMM_GROUP_BLOCK || !X || !lda || !dY || !ldb || !M || !N || (!dW && !w) || !w != !ver) return RV_E_INVAL;
  rv_gemm_args g[RV_GEMM_GROUP_BLOCK];
  for (int k = 0; k < count; ++k) {
    g[k].A = (const uint16_t*)X[k]; g[k].lda = lda[k]; g[k].a_kmajor = 1;
    g[k].B = (const uint16_t*)dY[k]; g[k].ldb = ldb[k]; g[k].b_kmajor = 1;
    g[k].M = M[k]; g[k].N = N[k]; g[k].K = K; g[k].epi = EPI_F32; g[k].ldo = N[k];
    g[k].out = dW ? dW[k] : w[k];   // (not written without dW)
    g[k].store_out = dW != nullptr;
    if (w) { g[k].upd_w = w[k]; g[k].upd_ver = (uint16_t*)ver[k]; g[k].upd_eta = eta; }
  }
  return rv_gemm_wgrad_grouped(g, count, (hipStream_t)stream, RV_WGRAD_BY_TOKENS);
}
