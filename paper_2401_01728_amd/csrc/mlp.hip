// fp32 MLP stage (Linear -> ReLU -> ... -> Linear): the forward_pass of a peer in the
// paper's Alg. 1 and its exact gradient with the delayed update of Eq. 2.
//
// Stash per microbatch: the input of every Linear (a_0 .. a_{n-1}).  Because a_{i+1} =
// ReLU(z_i), "a_{i+1} > 0" is the ReLU gate of layer i, so pre-activations are not kept.
//
// Every product has fp32 precision and a fixed order of additions (deterministic).  It runs on the fp32 matrix instructions
// (v_mfma_f32_32x32x2_f32 and v_mfma_f32_16x16x4_f32: full fp32 products and sums at twice the rate of plain vector FMAs,
// which may not be packed here), the large ones on the bf16 instructions with each operand in three pieces.  Four forms:
//   tiny   a whole forward, or a whole backward with its update, in ONE launch: workgroups
//          repeat the small chain of activations (or of gradients) each for itself in LDS and
//          share out the results, so that no layer waits for a launch of its own;
//   split  a 32x32 result tile per workgroup, the contraction dealt out over its four or eight waves,
//          operands straight from memory to registers;
//   wave   a 32x32 result tile per wave, for thin results of short contractions;
//   tiled  LDS tiles of 128x128 or 64x64 results, the operands in three bf16 planes.
// In all but the tiny form one launch per layer and direction: the forward product; or the input
// gradient, the weight gradient with the update in its epilogue, and the bias gradient together
// (they read the same gradient and do not depend on one another).
#include <new>
#include <type_traits>
#include "internal.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef f32x4 f32x4_u __attribute__((aligned(4)));   // four floats at any float's address

template <int V> struct Int { static constexpr int value = V; };   // a constant as an argument
template <int N, int I = 0, typename F>
__device__ __forceinline__ void each(F f) {                // f(0), .. f(N - 1)
  if constexpr (I < N) { f(Int<I>()); each<N, I + 1>(f); }
}

constexpr int kTinyLayers = 4, kTinyRows = 64;

struct MlpPlan {
  int n = 0;
  std::vector<size_t> offW, offB;   // into the flat parameter vector
  std::vector<size_t> offA;         // a_i inside a stash slot (floats)
  size_t maxw = 0;
  bool tiny = false;
};

// What happens to a finished parameter gradient: stored, and with the update of Eq. 2 (or its
// momentum form) applied on the spot where one is due.  Offsets are into the flat vector.
struct Upd {
  float* grad;
  float* w;            // null: gradient only
  float* vel;          // null: plain step
  float* ver;
  float eta, mu, wd;
};
__device__ __forceinline__ float next_velocity(const Upd& u, float w, float v, float g) {   // as update_momentum_kernel
  return __fmaf_rn(u.mu, v, __fmaf_rn(u.wd, w, g));
}
// N results of a lane at once: everything they read is requested before the first is formed (a
// store between two loads keeps the second one waiting for a round trip of its own); ok[k] = false: no
// such parameter (o[k] is a valid offset all the same).
template <int N>
struct Apply {
  float w[N], v[N];
  __device__ __forceinline__ void request(const Upd& u, const size_t (&o)[N]) {
    if (u.w) {
#pragma unroll
      for (int k = 0; k < N; ++k) w[k] = u.w[o[k]];
      if (u.vel) {
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = u.vel[o[k]];
      }
    }
  }
  __device__ __forceinline__ void complete(const Upd& u, const size_t (&o)[N], const float (&g)[N], const bool (&ok)[N]) {
    if (u.w) {
      if (u.vel) {
#pragma unroll
        for (int k = 0; k < N; ++k) {
          v[k] = next_velocity(u, w[k], v[k], g[k]);
          w[k] = __fmaf_rn(-u.eta, v[k], w[k]);
          if (ok[k]) u.vel[o[k]] = v[k];
        }
      } else {
#pragma unroll
        for (int k = 0; k < N; ++k) w[k] = __fmaf_rn(-u.eta, g[k], w[k]);
      }
#pragma unroll
      for (int k = 0; k < N; ++k)
        if (ok[k]) { u.w[o[k]] = w[k]; u.ver[o[k]] = w[k]; }
    }
#pragma unroll
    for (int k = 0; k < N; ++k)
      if (ok[k]) u.grad[o[k]] = g[k];
  }
};

// One product C[M,N] = sum_k A(m,k) B(k,n).  An operand is k-contiguous (A[m*lda + k],
// B[n*ldb + k]) or k-major (A[k*lda + m], B[k*ldb + n]).
struct Prod {
  const float* A; const float* B;
  int lda, ldb, M, N, K, tiles_n, tiles;
};
enum { FWD, DX, DW };
struct Out {
  float* C;            // FWD, DX: [M,N]
  const float* bias;   // FWD
  const float* gate;   // DX: kept where gate[m,n] > 0 (null: no gate)
  int relu;            // FWD
  Upd u; size_t off;   // DW: parameter offset of the tile's matrix
};
// R results of a lane, rows m[] of column n: what they read is requested, then they are completed
template <int OP, int R>
struct Finish {
  size_t i[R];
  bool ok[R];
  float b, gate[R];
  Apply<R> a;
  __device__ __forceinline__ void request(const Out& o, const int (&m)[R], int n, int M, int N) {
    const int nc = n < N ? n : N - 1;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      ok[r] = m[r] < M && n < N;
      i[r] = (size_t)(m[r] < M ? m[r] : M - 1) * N + nc;
      if (OP == DW) i[r] += o.off;
    }
    if (OP == FWD) b = o.bias[nc];
    if (OP == DX) {
#pragma unroll
      for (int r = 0; r < R; ++r) gate[r] = o.gate ? o.gate[i[r]] : 1.f;
    }
    if (OP == DW) a.request(o.u, i);
  }
  __device__ __forceinline__ void complete(const Out& o, const float (&v)[R]) {
    if (OP == DW) { a.complete(o.u, i, v, ok); return; }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float x = OP == DX ? (gate[r] > 0.f ? v[r] : 0.f) : o.relu ? fmaxf(v[r] + b, 0.f) : v[r] + b;
      if (ok[r]) o.C[i[r]] = x;
    }
  }
};
template <int OP, int R>
__device__ __forceinline__ void finish(const Out& o, const int (&m)[R], int n, int M, int N, const float (&v)[R]) {
  Finish<OP, R> f;
  f.request(o, m, n, M, N);
  f.complete(o, v);
}

// ---- tiled ---------------------------------------------------------------------------------
// The fp32 walk, for the tiles that three planes do not do for.  LDS keeps an operand the way memory has it: k-contiguous rows of
// 32 (pitch 36 floats: sixteen rows of 16-byte reads fall on all 64 banks), k-major rows of the tile's width (pitch + 8:
// rows k and k + 4, read together, are 32 banks apart).  A lane takes k = 8 g + 4 (lane / 32) + e, e = 0..3, for the four
// matrix instructions of group g: one 16-byte read of a k-contiguous tile, four 4-byte reads of a k-major one.
constexpr int BK = 32;
template <bool KM, int ROWS> struct Lds {
  static constexpr int PITCH = KM ? ROWS + 8 : BK + 4;
  static constexpr int FLOATS = KM ? BK * PITCH : ROWS * PITCH;
  static constexpr int PIECES = ROWS * BK / 4 / 256;       // 16-byte pieces per thread and tile
};

// A thread's share of a tile D deep, element by element at clamped indexes: what lies past the end of k is zeroed when the piece
// is parked (results of rows past the other end are not stored).
template <bool KM, int ROWS, int D>
__device__ __forceinline__ void tile_load(f32x4* v, const float* __restrict__ g, int ld, int r0, int rows, int k0, int K) {
  const float* base = KM ? g + (int64_t)k0 * ld + r0 : g + (int64_t)r0 * ld + k0;
#pragma unroll
  for (int i = 0; i < ROWS * D / 4 / 256; ++i) {
    const int p = threadIdx.x % 256 + 256 * i;
    const int k = KM ? p / (ROWS / 4) : p % (D / 4) * 4, r = KM ? p % (ROWS / 4) * 4 : p / (D / 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      int ke = KM ? k : k + e, re = KM ? r + e : r;
      ke = k0 + ke < K ? ke : K - 1 - k0; re = r0 + re < rows ? re : rows - 1 - r0;
      v[i][e] = base[KM ? (int64_t)ke * ld + re : (int64_t)re * ld + ke];
    }
  }
}
template <bool KM, int ROWS>
__device__ __forceinline__ void tile_park(const f32x4* v, float* s, int left) {   // left: K - k0
#pragma unroll
  for (int i = 0; i < Lds<KM, ROWS>::PIECES; ++i) {
    const int p = threadIdx.x % 256 + 256 * i;
    const int row = KM ? p / (ROWS / 4) : p / (BK / 4), c = KM ? p % (ROWS / 4) : p % (BK / 4);
    f32x4 x = v[i];
    if (left < BK) {                                       // (uniform)
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = (KM ? row : c * 4 + e) < left ? x[e] : 0.f;
    }
    *reinterpret_cast<f32x4*>(s + row * Lds<KM, ROWS>::PITCH + c * 4) = x;
  }
}
template <bool KM, int ROWS>
__device__ __forceinline__ f32x4 tile_frag(const float* s, int row0, int g) {
  const int l = threadIdx.x & 63, row = row0 + (l & 31), k = 8 * g + 4 * (l >> 5);
  constexpr int P = Lds<KM, ROWS>::PITCH;
  if (!KM) return *reinterpret_cast<const f32x4*>(s + row * P + k);
  return f32x4{s[k * P + row], s[(k + 1) * P + row], s[(k + 2) * P + row], s[(k + 3) * P + row]};
}

// A tile of BT x BT results is formed by four waves, 2 x 2, in products of 32x32.  Walks along K: on the bf16 matrix
// instructions (planes_walk), and where that does not do on the fp32 ones.
template <int BT> constexpr int kTileEdge = BT / 64;      // products to a wave's side
template <int BT> using TileAcc = f32x16[kTileEdge<BT>][kTileEdge<BT>];

template <int BT, bool AKM, bool BKM>
__device__ __forceinline__ void fp32_walk(TileAcc<BT>& acc, const Prod& p, int m0, int n0, float* s) {
  constexpr int T = kTileEdge<BT>, AF = Lds<AKM, BT>::FLOATS;
  const int wave = threadIdx.x % 256 >> 6, wm = (wave & 1) * 32 * T, wn = (wave >> 1) * 32 * T;
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j) acc[i][j] = 0.f;
  for (int k0 = 0; k0 < p.K; k0 += BK) {
    f32x4 va[Lds<AKM, BT>::PIECES], vb[Lds<BKM, BT>::PIECES];
    tile_load<AKM, BT, BK>(va, p.A, p.lda, m0, p.M, k0, p.K);
    tile_load<BKM, BT, BK>(vb, p.B, p.ldb, n0, p.N, k0, p.K);
    __syncthreads();
    tile_park<AKM, BT>(va, s, p.K - k0);
    tile_park<BKM, BT>(vb, s + AF, p.K - k0);
    __syncthreads();
#pragma unroll
    for (int g = 0; g < BK / 8; ++g) {
      f32x4 fa[T], fb[T];
#pragma unroll
      for (int i = 0; i < T; ++i) fa[i] = tile_frag<AKM, BT>(s, wm + i * 32, g);
#pragma unroll
      for (int j = 0; j < T; ++j) fb[j] = tile_frag<BKM, BT>(s + AF, wn + j * 32, g);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
          for (int j = 0; j < T; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][e], fb[j][e], acc[i][j], 0, 0, 0);
    }
  }
}

// A float is the sum of three bf16 numbers: the nearest one (a0), the one nearest to what is left, and what is left then.  bf16
// ends at 2^-133 and the last bit of a float below 2^-110 lies lower: operands are multiplied by 2^16 on the way in and the sums
// by 2^-32 on the way out, and so every float below 2^112 is the sum of its pieces, exactly.  (Without that a gradient's row at
// 1e-36 came out 3e-5 off.)  Of the nine products of pieces six are formed; the three left out are together at most 2^-24
// of the product, of either sign.
// Six bf16 instructions of 32 cycles stand against eight fp32 ones of 64.  a0 b0 is summed by itself: the instruction drops what
// lies below its sum towards minus infinity several times in 16 k, and with all six in one sum 1024-4096-4096-1024 on
// 1024 rows is 1.43e-6 from 64 bits and 4096 in k low by 2e-7 in the mean (fp32 instructions 1.28e-6 and 0).
// Operands of one sign (uniform), 4096 / 16384 / 65536 in k: 3.0e-7 / 6.0e-7 / 1.25e-6 from 64 bits and -4e-9 / -5e-8 / -4.0e-7 of it
// in the mean (fp32 instructions 8.4e-7 / 1.7e-6 / 3.5e-6 and 4e-9 / 6e-8 / 8.5e-7 towards zero).
// LDS keeps the planes of an operand as memory has it: k-contiguous rows of 32 bytes, read as one 16-byte fragment per
// lane, k-major rows of the tile's width, read by the transposing LDS read; 16-byte chunks are exchanged so that neither way
// of reading nor the 8-byte writes have bank conflicts.
// What bounds it: with two workgroups to a CU the matrix cores (1024 rows, 4096 -> 8192 forward 344 us = 200 TFLOP/s, 1200 of
// bf16), with one the LDS and barrier latency of a wave alone on its SIMD (4096 -> 4096 forward 197 us, 174 TFLOP/s).  Against the
// fp32 walk that ran here before, 1024 rows, forward / backward with the update, us: 4096 -> 4096 310 / 548 -> 197 / 371,
// 1024 -> 4096 90 / 159 -> 60 / 111; 2051 rows, 1030 -> 2052 177 / 244 -> 84 / 160; distance from 64 bits 0.31 - 0.36 times.
// (The factors of 2^16, on the vector ALU, are up to 5 % of a walk: 187 / 367 without, and 6 instructions of it behind a matrix
// instruction instead of the 5 before: 202 / 380.)
constexpr int SK = 16, kSlots = 3;                         // of k to a step
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
template <bool KM, int ROWS> struct Planes {
  static constexpr int BYTES = ROWS * SK * 2;              // of one plane
  static constexpr int PIECES = ROWS * SK / 4 / 256;       // 16-byte pieces of memory per thread and step
};
// The pieces of a step that is whole in k, one load each at a lane offset from a uniform base: rows past the end are clamped, and
// of a k-major operand whole pieces - the last may reach into the row behind (so not in the last row of all: see planes_walk).
template <bool KM, int ROWS>
__device__ __forceinline__ void plane_offsets(int ld, int r0, int rows, unsigned (&off)[Planes<KM, ROWS>::PIECES]) {
#pragma unroll
  for (int i = 0; i < Planes<KM, ROWS>::PIECES; ++i) {
    const int p = threadIdx.x % 256 + 256 * i;
    const int k = KM ? p / (ROWS / 4) : p % (SK / 4) * 4, r = KM ? p % (ROWS / 4) * 4 : p / (SK / 4);
    const int last = (KM ? (rows - 1) / 4 * 4 : rows - 1) - r0, rc = r < last ? r : last;
    off[i] = KM ? k * ld + rc : rc * ld + k;
  }
}
template <bool KM, int ROWS>
__device__ __forceinline__ void planes_load(f32x4* v, const unsigned (&off)[Planes<KM, ROWS>::PIECES], const float* __restrict__ g, int ld,
                                            int r0, int k0) {
  const float* base = KM ? g + (int64_t)k0 * ld + r0 : g + (int64_t)r0 * ld + k0;
#pragma unroll
  for (int i = 0; i < Planes<KM, ROWS>::PIECES; ++i) v[i] = *reinterpret_cast<const f32x4_u*>(base + off[i]);
}
template <bool KM, int ROWS>
__device__ __forceinline__ int plane_chunk(int row, int c) {   // byte of 16-byte chunk c of a row
  return KM ? row * (ROWS * 2) + (c ^ (ROWS == 64 ? (row & 2) << 1 : (row & 3) << 2)) * 16 : row * 32 + (c ^ (row >> 3 & 1)) * 16;
}
constexpr float kUp = 0x1p16f, kDown = 0x1p-32f;
template <bool KM, int ROWS>
__device__ __forceinline__ void planes_park(const f32x4* v, char* s, int left) {   // left: K - k0
#pragma unroll
  for (int i = 0; i < Planes<KM, ROWS>::PIECES; ++i) {
    const int p = threadIdx.x % 256 + 256 * i;
    const int row = KM ? p / (ROWS / 4) : p / (SK / 4), c = KM ? p % (ROWS / 4) : p % (SK / 4);
    f32x4 x = v[i];
    if (left < SK) {                                       // (uniform)
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = (KM ? row : c * 4 + e) < left ? x[e] : 0.f;
    }
    x *= kUp;
    char* d = s + plane_chunk<KM, ROWS>(row, c >> 1) + (c & 1) * 8;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const u32x2 h = {rv_pack_bf16x2(x[0], x[1]), rv_pack_bf16x2(x[2], x[3])};
      *reinterpret_cast<u32x2*>(d + q * Planes<KM, ROWS>::BYTES) = h;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] -= __uint_as_float(e & 1 ? h[e >> 1] & 0xFFFF0000u : h[e >> 1] << 16);
    }
  }
}
// rows row0 .. + 31 of plane q for v_mfma_f32_32x32x16_bf16: lane l holds row l % 32, k = 8 (l / 32) .. + 7
template <bool KM, int ROWS>
__device__ __forceinline__ bf16x8 plane_frag(const char* s, int row0, int plane) {
  const int l = threadIdx.x & 63;
  s += plane * Planes<KM, ROWS>::BYTES;
  if (!KM) return *reinterpret_cast<const bf16x8*>(s + plane_chunk<KM, ROWS>(row0 + (l & 31), l >> 5));
  typedef s16x4 __attribute__((address_space(3)))* lds4;
  const int q = l >> 4, i = l & 15, k = 8 * (q >> 1) + (i >> 2), col = row0 + 16 * (q & 1) + 4 * (i & 3);
  const char* at = s + plane_chunk<KM, ROWS>(k, col >> 3) + (col & 7) * 2;
  const s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(at));
  const s16x4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(at + 4 * (ROWS * 2)));
  return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7));
}
template <int BT, bool AKM, bool BKM> constexpr int kSlotBytes = 3 * (Planes<AKM, BT>::BYTES + Planes<BKM, BT>::BYTES);

// While step s is multiplied, step s + 2 goes into the slot that step s - 1 was read from and step s + 2 + D is requested (D steps
// are on the way: on 128x128 tiles what the registers hold; on 64x64 ones 8 in place of 4 are no faster on long walks and make
// the code longer, 129 -> 3001 on 300 rows backward 33 us in place of 20): one barrier a step.  Fragments have one set of registers: the order of the products lets those of pieces 1 and 2 be read anew behind
// the last products of the step before, those of piece 0 behind the first of their own.  Two workgroups share a CU.
template <int BT, bool AKM, bool BKM>
__device__ __forceinline__ void planes_walk(TileAcc<BT>& acc, const Prod& p, int m0, int n0, char* smem) {
  constexpr int T = kTileEdge<BT>, PA = Planes<AKM, BT>::BYTES, SLOT = kSlotBytes<BT, AKM, BKM>;
  const int wave = threadIdx.x % 256 >> 6, wm = (wave & 1) * 32 * T, wn = (wave >> 1) * 32 * T;
  TileAcc<BT> low;
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j) { acc[i][j] = 0.f; low[i][j] = 0.f; }
  constexpr int D = T == 2 ? 2 : 4;
  f32x4 va[D][Planes<AKM, BT>::PIECES], vb[D][Planes<BKM, BT>::PIECES];   // step s in set s % D
  unsigned oa[Planes<AKM, BT>::PIECES], ob[Planes<BKM, BT>::PIECES];
  plane_offsets<AKM, BT>(p.lda, m0, p.M, oa);
  plane_offsets<BKM, BT>(p.ldb, n0, p.N, ob);
  bf16x8 a[3][T], b[3][T];
  const int ns = (p.K + SK - 1) / SK;
  const int Kw = p.K - ((AKM && p.M % 4) || (BKM && p.N % 4) ? 1 : 0);   // steps that end here at the latest are loaded by pieces
  auto fetch = [&](auto set, int s) {
    constexpr int S = decltype(set)::value;
    if (s >= ns) return;
    if ((s + 1) * SK <= Kw) {                              // (uniform)
      planes_load<AKM, BT>(va[S], oa, p.A, p.lda, m0, s * SK);
      planes_load<BKM, BT>(vb[S], ob, p.B, p.ldb, n0, s * SK);
    } else {
      tile_load<AKM, BT, SK>(va[S], p.A, p.lda, m0, p.M, s * SK, p.K);
      tile_load<BKM, BT, SK>(vb[S], p.B, p.ldb, n0, p.N, s * SK, p.K);
    }
  };
  auto park = [&](auto set, int s, char* to) {
    constexpr int S = decltype(set)::value;
    if (s >= ns) return;
    planes_park<AKM, BT>(va[S], to, p.K - s * SK);
    planes_park<BKM, BT>(vb[S], to + 3 * PA, p.K - s * SK);
  };
  auto frags = [&](int piece, const char* from) {
#pragma unroll
    for (int i = 0; i < T; ++i) a[piece][i] = plane_frag<AKM, BT>(from, wm + i * 32, piece);
#pragma unroll
    for (int j = 0; j < T; ++j) b[piece][j] = plane_frag<BKM, BT>(from + 3 * PA, wn + j * 32, piece);
  };
  auto products = [&](TileAcc<BT>& to, int pa, int pb) {
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
      for (int j = 0; j < T; ++j) to[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[pa][i], b[pb][j], to[i][j], 0, 0, 0);
  };
  char *cur = smem, *nxt = smem + SLOT, *free = smem + 2 * SLOT;
  // steps 0 and 1 in their slots, 2 .. D + 1 on the way, the first fragments read.  (Both kinds of loop have a start of their own:
  // behind loads that may not have been issued the compiler waits for all there are, in every turn of the loop.)
  auto begin = [&](auto load, auto store) {
    each<D>([&](auto set) { load(set, decltype(set)::value); });
    store(Int<0>(), 0, cur);
    load(Int<0>(), D);
    store(Int<1>(), 1, nxt);
    load(Int<1>(), D + 1);
    __syncthreads();
    frags(1, cur);
    frags(2, cur);
  };
  auto step = [&](int s, auto set, auto whole) {
    constexpr int S = (decltype(set)::value + 2) % D;      // of step s + 2
    constexpr bool WHOLE = decltype(whole)::value != 0;    // step s + 2 + D is loaded by pieces
    const bool next = WHOLE || s + 1 < ns;
    // the order in which a stretch's instructions are issued: behind each matrix instruction some of the others
    auto deal = [&](auto matrix, auto lds) {
#pragma unroll
      for (int q = 0; q < decltype(matrix)::value * T * T; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, T == 2 ? 6 : 11, 0);
        __builtin_amdgcn_sched_group_barrier(0x080, decltype(lds)::value, 0);
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    if (!WHOLE) {
      park(Int<S>(), s + 2, free);
      fetch(Int<S>(), s + 2 + D);
    }
    frags(0, cur);
    products(low, 1, 1);
    if (WHOLE) deal(Int<1>(), Int<T == 2 ? 2 : 4>());
    if (WHOLE) {
      planes_park<AKM, BT>(va[S], free, SK);
      planes_load<AKM, BT>(va[S], oa, p.A, p.lda, m0, (s + 2 + D) * SK);
    }
    products(low, 1, 0);
    products(low, 0, 1);
    if (WHOLE) deal(Int<2>(), Int<T == 2 ? 1 : 2>());
    if (next) frags(1, nxt);
    if (WHOLE) {
      planes_park<BKM, BT>(vb[S], free + 3 * PA, SK);
      planes_load<BKM, BT>(vb[S], ob, p.B, p.ldb, n0, (s + 2 + D) * SK);
    }
    products(low, 2, 0);
    products(low, 0, 2);
    if (WHOLE) deal(Int<2>(), Int<T == 2 ? 2 : 4>());
    if (next) frags(2, nxt);
    products(acc, 0, 0);
    if (WHOLE) deal(Int<1>(), Int<T == 2 ? 2 : 4>());
    __syncthreads();
    char* t = cur; cur = nxt; nxt = free; free = t;
  };
  int s = 0;
  if ((2 * D + 2) * SK <= Kw) {
    begin(
        [&](auto set, int s) {
          planes_load<AKM, BT>(va[decltype(set)::value], oa, p.A, p.lda, m0, s * SK);
          planes_load<BKM, BT>(vb[decltype(set)::value], ob, p.B, p.ldb, n0, s * SK);
        },
        [&](auto set, int s, char* to) {
          planes_park<AKM, BT>(va[decltype(set)::value], to, SK);
          planes_park<BKM, BT>(vb[decltype(set)::value], to + 3 * PA, SK);
        });
    do {
      each<D>([&](auto set) { step(s + decltype(set)::value, set, Int<1>()); });
      s += D;
    } while ((s + 2 * D + 2) * SK <= Kw);
  } else {
    begin(fetch, park);
  }
  for (; s < ns; s += D)
    each<D>([&](auto set) {
      if (s + decltype(set)::value < ns) step(s + decltype(set)::value, set, Int<0>());
    });
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j) acc[i][j] = (acc[i][j] + low[i][j]) * kDown;
}

// BT: 128 or 64 (tiled), kHalves (64, by two halves of a workgroup), 32 (split over NT / 64 waves), kSlim (the same, 32x16),
// kWave (a 32x32 tile per wave)
constexpr int kWave = 1, kHalves = 2, kSlim = 16;
template <int BT, int NT, bool AKM, bool BKM> constexpr int mlp_lds_bytes() {
  if constexpr (BT == kHalves) return mlp_lds_bytes<64, NT, AKM, BKM>();
  else
  // (kWave: the bias sums beside it)
  return 4 * (BT == kWave ? NT / 32 * 33 : BT == 32 || BT == kSlim ? NT / 64 * 32 * 33
              : NT / 256 * std::max(Lds<AKM, BT>::FLOATS + Lds<BKM, BT>::FLOATS, kSlots * kSlotBytes<BT, AKM, BKM> / 4));
}
// A workgroup of 512 threads takes two tiles, side by side: both have the same number of steps and so of barriers; the last
// one's second tile may be past the end (it walks along on the last tile and keeps nothing).
// With HALVES the two of them take half of one tile's steps each and the second one's sums are added to the first one's: a wave alone
// on its SIMD waits for LDS and barriers most of a 64x64 tile's step (4096 -> 1024 on 1024 rows forward 104 us, in halves 79).
template <int BT, bool AKM, bool BKM, int OP, bool HALVES = false>
__device__ __forceinline__ void tiled_body(const Prod& p, const Out& o, int tile, float* smem, int part = 0) {
  constexpr int T = kTileEdge<BT>;
  const int all = (p.M + BT - 1) / BT * p.tiles_n;
  const bool live = tile < all;        // (uniform in 256 threads)
  tile = live ? tile : all - 1;
  const int m0 = tile / p.tiles_n * BT, n0 = tile % p.tiles_n * BT;
  const int wave = threadIdx.x % 256 >> 6, l = threadIdx.x & 63, wm = (wave & 1) * 32 * T, wn = (wave >> 1) * 32 * T;
  TileAcc<BT> acc;
  if constexpr (HALVES) {
    static_assert(!AKM && BKM, "operands of a forward product");
    Prod h = p;
    const int steps = (p.K + SK - 1) / SK, mine = (steps + 1) / 2, k1 = mine * SK;
    if (part) { h.A += k1; h.B += (int64_t)k1 * p.ldb; h.K -= k1; } else { h.K = k1; }
    planes_walk<BT, AKM, BKM>(acc, h, m0, n0, reinterpret_cast<char*>(smem));
    if (part && steps - mine < mine) __syncthreads();      // (the barrier of the step that the first half has more)
    const float* mem = smem + (part ? 0 : mlp_lds_bytes<BT, 256, AKM, BKM>() / 4);
    f32x4* x = reinterpret_cast<f32x4*>(const_cast<float*>(mem)) + threadIdx.x % 256;
#pragma unroll
    for (int r = 0; r < 16 * T * T; r += 4) {
      f32x16& v = acc[r / 16 / T][r / 16 % T];
      if (part) x[r / 4 * 256] = f32x4{v[r % 16], v[r % 16 + 1], v[r % 16 + 2], v[r % 16 + 3]};
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16 * T * T; r += 4) {
      f32x16& v = acc[r / 16 / T][r / 16 % T];
      if (!part) {
        const f32x4 y = x[r / 4 * 256];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[r % 16 + e] += y[e];
      }
    }
  } else {
    planes_walk<BT, AKM, BKM>(acc, p, m0, n0, reinterpret_cast<char*>(smem));
  }
  // The pieces of an infinity hold a NaN, and large numbers may pass the largest one on the way: a tile with a result that is not
  // finite is walked again in fp32, and with it the other one of its workgroup.
  bool finite = true;
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) finite = finite && fabsf(acc[i][j][r]) < __builtin_inff();
  if (__syncthreads_or(!finite))
    fp32_walk<BT, AKM, BKM>(acc, p, m0, n0, smem);
  if (!live || (HALVES && part)) return;
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
      for (int rb = 0; rb < 16; rb += 8) {
        int m[8];
        float v[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          m[r] = m0 + wm + i * 32 + 8 * ((rb + r) >> 2) + 4 * (l >> 5) + (r & 3);
          v[r] = acc[i][j][rb + r];
        }
        finish<OP, 8>(o, m, n0 + wn + j * 32 + (l & 31), p.M, p.N, v);
      }
}

// ---- split ---------------------------------------------------------------------------------
// NW waves on one 32x32 tile; wave w takes the 8-deep groups w, w + NW, ... of the contraction, up to eight of
// them on the way; the partial tiles are added in wave order.
constexpr int kSplitWaves = 8;
template <bool KM>
__device__ __forceinline__ f32x4 direct_frag(const float* __restrict__ g, int ld, int row, int k, int K, bool whole) {
  f32x4 v;
  if (whole) {
    if (!KM) return *reinterpret_cast<const f32x4_u*>(g + (int64_t)row * ld + k);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = g[(int64_t)(k + e) * ld + row];
    return v;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int kc = k + e < K ? k + e : K - 1;
    const float x = KM ? g[(int64_t)kc * ld + row] : g[(int64_t)row * ld + kc];
    v[e] = k + e < K ? x : 0.f;
  }
  return v;
}
template <int NW, bool AKM, bool BKM, int OP>
__device__ __forceinline__ void split_body(const Prod& p, const Out& o, int tile, float* smem) {
  const int m0 = tile / p.tiles_n * 32, n0 = tile % p.tiles_n * 32;
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, h = l >> 5;
  const int ra = m0 + (l & 31) < p.M ? m0 + (l & 31) : p.M - 1, rb = n0 + (l & 31) < p.N ? n0 + (l & 31) : p.N - 1;
  constexpr int U = 4;                                     // two sets of so many groups are on the way
  const int ng = (p.K + 7) / 8, whole = p.K / 8;
  f32x4 fa[2][U], fb[2][U];
  auto request = [&](int set, int g0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int g = g0 + u * NW;                  // wave-uniform
      fa[set][u] = 0.f; fb[set][u] = 0.f;
      if (g < ng) {
        fa[set][u] = direct_frag<AKM>(p.A, p.lda, ra, 8 * g + 4 * h, p.K, g < whole);
        fb[set][u] = direct_frag<BKM>(p.B, p.ldb, rb, 8 * g + 4 * h, p.K, g < whole);
      }
    }
  };
  // what the results read comes with the first operands, and the next operands while the present ones are multiplied:
  // behind one another these were a memory round trip each (two sets of eight groups instead hold registers that a
  // second workgroup of the CU would use: 442-461-220-2087-99 on 450 rows 272 -> 291 us)
  constexpr int R = 32 * 32 / (64 * NW);
  int m[R];
  const int nl = threadIdx.x & 31;
#pragma unroll
  for (int i = 0; i < R; ++i) m[i] = m0 + (threadIdx.x >> 5) + 2 * NW * i;
  Finish<OP, R> f;
  request(0, wave);
  if (wave + U * NW < ng) request(1, wave + U * NW);
  f.request(o, m, n0 + nl, p.M, p.N);
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  auto products = [&](int set) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[set][u][e], fb[set][u][e], acc, 0, 0, 0);
  };
  for (int g0 = wave; g0 < ng; g0 += 2 * U * NW) {
    products(0);
    if (g0 + 2 * U * NW < ng) request(0, g0 + 2 * U * NW);
    if (g0 + U * NW >= ng) break;
    products(1);
    if (g0 + 3 * U * NW < ng) request(1, g0 + 3 * U * NW);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) smem[(wave * 32 + 8 * (r >> 2) + 4 * h + (r & 3)) * 33 + (l & 31)] = acc[r];
  __syncthreads();
  float v[R];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int ml = m[i] - m0;
    v[i] = smem[ml * 33 + nl];
#pragma unroll
    for (int w = 1; w < NW; ++w) v[i] += smem[(w * 32 + ml) * 33 + nl];
  }
  f.complete(o, v);
}

// The same on 32x16 tiles, in products of 16x16: where 32x32 tiles leave half of the CUs without one.  A group is 16 deep, so
// that a wave has a contraction of up to 1024 on the way at once and touches fewer lines to a request.
template <bool AKM, bool BKM, int OP>
__device__ __forceinline__ void slim_body(const Prod& p, const Out& o, int tile, float* smem) {
  constexpr int NW = kSplitWaves, U = 4, P = 17;
  const int m0 = tile / p.tiles_n * 32, n0 = tile % p.tiles_n * 16;
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, q = l >> 4;
  const int ra0 = m0 + (l & 15) < p.M ? m0 + (l & 15) : p.M - 1, ra1 = m0 + 16 + (l & 15) < p.M ? m0 + 16 + (l & 15) : p.M - 1;
  const int rb = n0 + (l & 15) < p.N ? n0 + (l & 15) : p.N - 1;
  const int ng = (p.K + 15) / 16, whole = p.K / 16;
  f32x4 fa[2][U][2], fb[2][U];
  auto request = [&](int set, int g0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int g = g0 + u * NW;                  // wave-uniform
      fa[set][u][0] = 0.f; fa[set][u][1] = 0.f; fb[set][u] = 0.f;
      if (g < ng) {
        fa[set][u][0] = direct_frag<AKM>(p.A, p.lda, ra0, 16 * g + 4 * q, p.K, g < whole);
        fa[set][u][1] = direct_frag<AKM>(p.A, p.lda, ra1, 16 * g + 4 * q, p.K, g < whole);
        fb[set][u] = direct_frag<BKM>(p.B, p.ldb, rb, 16 * g + 4 * q, p.K, g < whole);
      }
    }
  };
  const int ml = threadIdx.x >> 4, nl = threadIdx.x & 15;   // one result to a thread
  const int m[1] = {m0 + ml};
  Finish<OP, 1> f;
  request(0, wave);
  if (wave + U * NW < ng) request(1, wave + U * NW);
  f.request(o, m, n0 + nl, p.M, p.N);
  f32x4 acc[2] = {0.f, 0.f};
  auto products = [&](int set) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[set][u][t][e], fb[set][u][e], acc[t], 0, 0, 0);
  };
  for (int g0 = wave; g0 < ng; g0 += 2 * U * NW) {
    products(0);
    if (g0 + 2 * U * NW < ng) request(0, g0 + 2 * U * NW);
    if (g0 + U * NW >= ng) break;
    products(1);
    if (g0 + 3 * U * NW < ng) request(1, g0 + 3 * U * NW);
  }
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) smem[(wave * 32 + 16 * t + 4 * q + r) * P + (l & 15)] = acc[t][r];
  __syncthreads();
  float v[1] = {smem[ml * P + nl]};
#pragma unroll
  for (int w = 1; w < NW; ++w) v[0] += smem[(w * 32 + ml) * P + nl];
  f.complete(o, v);
}

// ---- one wave per tile ---------------------------------------------------------------------
// A short contraction behind a thin result (see pick): a 32x32 tile per wave straight from its accumulators,
// nothing to add up between waves, no LDS, no barrier.  What bounds it is the results' own memory traffic.
template <int NT, bool AKM, bool BKM, int OP>
__device__ __forceinline__ void wave_body(const Prod& p, const Out& o, int group) {
  const int tile = __builtin_amdgcn_readfirstlane(group * (NT / 64) + (threadIdx.x >> 6));
  const int m0 = tile / p.tiles_n * 32, n0 = tile % p.tiles_n * 32;
  if (m0 >= p.M) return;
  const int l = threadIdx.x & 63, h = l >> 5;
  const int ra = m0 + (l & 31) < p.M ? m0 + (l & 31) : p.M - 1, rb = n0 + (l & 31) < p.N ? n0 + (l & 31) : p.N - 1;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  constexpr int U = 4;
  const int ng = (p.K + 7) / 8, whole = p.K / 8;
  for (int g0 = 0; g0 < ng; g0 += U) {
    f32x4 fa[U], fb[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int g = g0 + u;
      fa[u] = 0.f; fb[u] = 0.f;
      if (g < ng) {
        fa[u] = direct_frag<AKM>(p.A, p.lda, ra, 8 * g + 4 * h, p.K, g < whole);
        fb[u] = direct_frag<BKM>(p.B, p.ldb, rb, 8 * g + 4 * h, p.K, g < whole);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[u][e], fb[u][e], acc, 0, 0, 0);
  }
#pragma unroll
  for (int rb = 0; rb < 16; rb += 8) {
    if (m0 + 2 * rb >= p.M) break;                         // (uniform) rows 2 rb .. 2 rb + 15 of the tile
    int m[8];
    float v[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      m[r] = m0 + 8 * ((rb + r) >> 2) + 4 * h + (r & 3);
      v[r] = acc[rb + r];
    }
    finish<OP, 8>(o, m, n0 + (l & 31), p.M, p.N, v);
  }
}

// column sums of D[M,N] (the bias gradient): 32 columns per workgroup, NT / 32 row lanes whose
// sums are added in order
template <int NT>
__device__ __forceinline__ void bias_body(const float* __restrict__ D, int M, int N, const Upd& u, size_t off, int blk,
                                          float* smem) {
  constexpr int RL = NT / 32;
  const int cl = threadIdx.x & 31, rl = threadIdx.x >> 5, c = blk * 32 + cl, cc = c < N ? c : N - 1;
  float s[4] = {0.f, 0.f, 0.f, 0.f};
  for (int r = rl; r < M; r += 4 * RL) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int rr = r + q * RL;
      const float x = D[(int64_t)(rr < M ? rr : M - 1) * N + cc];
      s[q] += rr < M ? x : 0.f;
    }
  }
  smem[rl * 33 + cl] = (s[0] + s[1]) + (s[2] + s[3]);
  __syncthreads();
  if (rl == 0 && c < N) {
    float t = smem[cl];
#pragma unroll
    for (int w = 1; w < RL; ++w) t += smem[w * 33 + cl];
    const size_t i[1] = {off + c};
    const float g[1] = {t};
    const bool ok[1] = {true};
    Apply<1> a;
    a.request(u, i);
    a.complete(u, i, g, ok);
  }
}

template <int BT, int NT, bool AKM, bool BKM, int OP>
__device__ __forceinline__ void mlp_body(const Prod& p, const Out& o, int tile, float* smem) {
  if constexpr (BT == kWave) {
    wave_body<NT, AKM, BKM, OP>(p, o, tile);
  } else if constexpr (BT == kSlim) {
    slim_body<AKM, BKM, OP>(p, o, tile, smem);
  } else if constexpr (BT == 32) {
    split_body<NT / 64, AKM, BKM, OP>(p, o, tile, smem);
  } else if constexpr (BT == kHalves) {
    static_assert(NT == 512, "eight waves a tile");
    const int part = __builtin_amdgcn_readfirstlane(threadIdx.x / 256);
    tiled_body<64, AKM, BKM, OP, true>(p, o, tile, smem + part * (mlp_lds_bytes<64, 256, AKM, BKM>() / 4), part);
  } else {
    static_assert(NT == 256 || NT == 512, "four waves a tile");
    const int part = NT == 256 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / 256);
    tiled_body<BT, AKM, BKM, OP>(p, o, tile * (NT / 256) + part, smem + part * (mlp_lds_bytes<BT, 256, AKM, BKM>() / 4));
  }
}
extern __shared__ __align__(16) float mlp_smem[];

template <int BT, int NT>
__global__ __launch_bounds__(NT, 2) void mlp_fwd_kernel(Prod p, Out o, float* __restrict__ copy) {
  // The stage's input goes into the stash beside the product that reads it, by workgroups of their own behind its
  // tiles, four 16-byte pieces of a lane in flight.  (Dealt out over the tiles, one float at a time ahead of the
  // product, it was what a narrow layer behind a wide input lasted: there are few tiles then.  4096 -> 32 on 1024 rows
  // 98 -> 40 us, 1024 -> 32 19.4 -> 11.2; 4096 -> 4096 on 1024 rows, where there are 256 tiles, 321 -> 304.)
  if ((int)blockIdx.x >= p.tiles) {
    const int64_t n = (int64_t)p.M * p.K, step = (int64_t)(gridDim.x - p.tiles) * NT * 4;
    int64_t i = ((int64_t)(blockIdx.x - p.tiles) * NT + threadIdx.x) * 4;
    for (; i + 3 * step + 4 <= n; i += 4 * step) {
      f32x4 v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = *reinterpret_cast<const f32x4_u*>(p.A + i + k * step);
#pragma unroll
      for (int k = 0; k < 4; ++k) *reinterpret_cast<f32x4_u*>(copy + i + k * step) = v[k];
    }
    for (; i < n; i += step)
      for (int64_t e = i; e < i + 4 && e < n; ++e) copy[e] = p.A[e];
    return;
  }
  mlp_body<BT, NT, false, true, FWD>(p, o, blockIdx.x, mlp_smem);
}

// input gradient (tiles 0 .. dx.tiles), weight gradient, bias gradient in one launch
template <int BX, int BW, int NT>
__global__ __launch_bounds__(NT, 2) void mlp_bwd_kernel(Prod dx, Out ox, Prod dw, Out ow, const float* __restrict__ d, int M, int N,
                                                     size_t offb) {
  int b = blockIdx.x;
  if (b < dx.tiles) { mlp_body<BX, NT, false, false, DX>(dx, ox, b, mlp_smem); return; }
  b -= dx.tiles;
  if (b < dw.tiles) { mlp_body<BW, NT, true, true, DW>(dw, ow, b, mlp_smem); return; }
  bias_body<NT>(d, M, N, ow.u, offb, b - dw.tiles, mlp_smem);
}

Prod product(const float* A, int lda, const float* B, int ldb, int M, int N, int K, int bt, int nt) {
  const int edge = bt == kWave || bt == kSlim ? 32 : bt == kHalves ? 64 : bt, en = bt == kSlim ? 16 : edge;
  const int tn = (N + en - 1) / en, tiles = (M + edge - 1) / edge * tn, waves = nt / 64;
  const int per = bt == kWave ? waves : bt > 32 ? nt / 256 : 1;   // tiles a workgroup (kHalves: 1)
  return Prod{A, B, lda, ldb, M, N, K, tn, (tiles + per - 1) / per};   // (tiles: workgroups)
}
int tile_count(int M, int N, int bt) { return (M + bt - 1) / bt * ((N + bt - 1) / bt); }
constexpr int kCUs = 256;
// The largest tile that still gives every CU one (of 64x64 tiles half of them: such a workgroup
// keeps up with two CUs' worth of 32x32 ones, whose operands all come through L2; fitted to fp32 tiles, which took a seventh to a half
// longer than the present ones).  Measured: a stage step of
// 1024-4096-4096-1024 on 1024 rows 0.90 ms (171 TFLOP/s), 300-1000-1000-77 on 100 rows with momentum 60 us.
// A result of at most 32 rows or columns fills at best half of such a tile's matrix instructions, so there the tile
// count says nothing about the chip: it takes 32x32 tiles, one per wave where the contraction is short (the work is the
// results' memory traffic), split where it is long.  Times in us against the tiles that the count alone would take:
//   4 -> 1e5 on 8 rows, forward 10.8 -> 6.3 (32x32 split 29.5)  1e5 -> 4 on 8 rows, backward 16.7 -> 12.8 (49.5)
//   8 -> 2048 on 8192 rows, backward 92 -> 85                    8192 -> 8192 on 8 rows, forward 118 -> 68
//   slower: 4 -> 1e5 on 8 rows, backward 310 -> 339; 16384 -> 100 on 16 rows, backward 10.2 -> 11.5
int pick(int M, int N, int K) {
  const int thin = std::min(M, N);
  if (thin <= 32 && tile_count(M, N, 64) >= kCUs / 2) return K <= 128 ? kWave : 32;
  return thin > 64 && tile_count(M, N, 128) >= kCUs ? 128 : tile_count(M, N, 64) >= kCUs / 2 ? 64 : 32;
}
// 32x16 tiles where 32x32 ones leave CUs without one: a forward product up to half of them, an input gradient up to a quarter, for the
// weight gradient's tiles come beside it (and more below).  us, 32x32 / 32x16: forward 1000 -> 1000 on 100 rows 10.5 / 8.8, 4096 -> 256 on
// 16 29.1 / 19.4, 128 -> 128 on 64 6.9 / 5.2; backward 300 -> 1000 on 100 rows 11.1 / 9.1, 256 -> 4000 on 20 31.4 / 22.9;
// past the quarter 200 -> 200 on 500 rows 7.3 / 8.9, 1000 -> 1000 on 100 15.6 / 19.7, 1000 -> 77 on 100 5.3 / 7.7.
bool slim(int M, int N, int bt, int cus) { return bt == 32 && tile_count(M, N, 32) <= cus; }
int threads(int bt) { return bt == 32 || bt == kSlim || bt == kHalves ? 64 * kSplitWaves : 256; }

template <typename K>
rv_status allow_lds(K kern, int bytes) {
  return hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess ? RV_OK : RV_E_DEVICE;
}
// workgroups that copy the stage's input beside a forward product's tiles
int copy_groups(int M, int K, int nt) {
  const int64_t per = 16 * nt;   // floats a workgroup copies per turn
  return (int)std::min<int64_t>(4 * kCUs, ((int64_t)M * K + per - 1) / per);
}
// A workgroup of 32x16 tiles has a CU to itself and workgroups are dealt to the eight XCDs in turn, so the copying ones of a first
// layer run on the CUs that the tiles leave of each XCD, a short turn after another, and behind the tiles where they leave none.
// That pays only where the walk is long against it: us, 32x32 / 32x16: no CU left, 128 -> 128 on 1000 rows 4.8 / 6.3, 256 -> 256 on 500 5.0 / 6.8,
// 1400 -> 256 on 500 (84 copying workgroups) 14.4 / 12.5, 1400 -> 128 on 1000 (171) 14.8 / 15.3, 2000 -> 128 on 1000 (245) 20.0 / 18.5;
// four of an XCD left, 500 -> 100 on 1000 (two turns) 7.2 / 5.7, 1000 -> 100 on 1000 (four) 10.6 / 9.7; one left, 300 -> 128 on 970 (five)
// 6.4 / 6.8, 1000 -> 128 on 970 (15) 10.5 / 11.2.
bool slim_forward(int M, int N, int K, int bt, bool copy) {
  if (!slim(M, N, bt, kCUs / 2)) return false;
  const int copies = copy ? copy_groups(M, K, 64 * kSplitWaves) : 0, groups = (M + 31) / 32 * ((N + 15) / 16);
  const int left = kCUs / 8 - (groups + 7) / 8, each = (copies + 7) / 8;   // of an XCD
  return groups + copies <= kCUs || each <= left * std::max(1, K / 250) || 5 * copies <= K - 750;
}
// The input gradient of mb rows, width K and contraction N beside a weight gradient of `others` workgroups, bias ones among them.  It
// has to be the longer walk: us, 32x32 / 32x16, 20 -> 128 on 1000 rows 9.8 / 10.5, 128 -> 300 on 300 6.5 / 7.0, 20 -> 1000 on 1000 10.5 / 11.1,
// 100 -> 600 on 500 8.0 / 7.7, 64 -> 1000 on 64 10.2 / 8.3; contractions of 128, 1000 -> 128 on 60 4.6 / 4.8, 300 -> 128 on 100 4.7 / 4.7.  And workgroups have
// a CU to themselves here too: another turn of the CUs is worth it only for a long walk: 1900 -> 600 on 20 rows 9.4 / 13.8, 300 -> 600 on 100
// 8.2 / 7.9, 1000 -> 900 on 60 11.9 / 11.2, 100 -> 900 on 500 10.7 / 9.0.
bool slim_backward(int mb, int K, int N, int bx, int others) {
  if (!slim(mb, K, bx, kCUs / 4) || N < 256 || N <= mb) return false;
  return (mb + 31) / 32 * ((K + 15) / 16) + others <= kCUs || tile_count(mb, K, 32) + others > kCUs || N >= 800;
}
template <int BT, int NT>
rv_status launch_fwd(hipStream_t st, const Prod& p, const Out& o, float* copy) {
  constexpr int lds = mlp_lds_bytes<BT, NT, false, true>();
  static const rv_status ok = allow_lds(mlp_fwd_kernel<BT, NT>, lds);
  RV_TRY(ok);
  const int extra = copy ? copy_groups(p.M, p.K, NT) : 0;
  hipLaunchKernelGGL((mlp_fwd_kernel<BT, NT>), dim3(p.tiles + extra), dim3(NT), lds, st, p, o, copy);
  return rv_launch_status();
}
template <int BX, int BW, int NT>
rv_status launch_bwd(hipStream_t st, const Prod& dx, const Out& ox, const Prod& dw, const Out& ow, const float* d, int M, int N,
                     size_t offb) {
  constexpr int l1 = mlp_lds_bytes<BX, NT, false, false>(), l2 = mlp_lds_bytes<BW, NT, true, true>(), lds = l1 > l2 ? l1 : l2;
  static const rv_status ok = allow_lds(mlp_bwd_kernel<BX, BW, NT>, lds);
  RV_TRY(ok);
  hipLaunchKernelGGL((mlp_bwd_kernel<BX, BW, NT>), dim3(dx.tiles + dw.tiles + (N + 31) / 32), dim3(NT), lds, st, dx, ox, dw, ow, d, M,
                     N, offb);
  return rv_launch_status();
}

// ---- tiny ----------------------------------------------------------------------------------
struct Tiny {
  int mb, dim[kTinyLayers + 1];
  unsigned offW[kTinyLayers], offB[kTinyLayers], offA[kTinyLayers], zero;   // zero: the number of parameters
  unsigned over[kTinyLayers];   // t / tn of a layer's gradient tiles, tn to a row: t * over >> 16 (t * tn < 65536)
  int skip[kTinyLayers];        // the layer's gradient tiles modulo the waves of the launch
};
constexpr int kTinyDepth = 128;   // contraction a wave requests at a time
constexpr int kTinyThreads = 512, kTinyWaves = kTinyThreads / 64;
__host__ __device__ constexpr int tiny_pitch(int w) { return (w + 15) / 16 * 16 + 4; }   // rows of whole 16-wide groups, 16-byte aligned

// What bounds these kernels is one memory round trip after another (1 - 2 us each: the lines were
// written by other launches, which leaves every XCD's L2 without them) and the number of lines a
// load instruction touches.  So a wave requests everything its first tiles of a layer read up to two layers
// ahead (what the registers hold), the rows of a transposed weight tile come in 16-byte pieces, and no load waits behind
// a branch: an index past an end is clamped where its result is not stored, and points at a zero behind the
// parameters where it enters a sum (the zero on the other side would not do: zero times an infinity is no zero).
// These kernels run through their code once, so its length is time too, about 0.3 us to a KiB: the copy of the input moved as
// pieces of 16 bytes (element by element with a test each: forward + 0.8 us), rows of gradient tiles by a multiplication in
// place of divisions, lane offsets of 32 bits.  A launch of 64-128-64 on 8 rows, forward / backward, 5.8 / 8.6 us before
// that and 5.5 / 7.3 with it; 16 microbatches through two such stages 437 -> 386 us, which is what issuing them takes.
// element i of a vector of less than 4 GiB: a lane offset from a uniform base, without 64-bit arithmetic per lane
template <typename T>
__device__ __forceinline__ T& at(T* base, unsigned i) {
  return *reinterpret_cast<T*>(reinterpret_cast<std::conditional_t<std::is_const<T>::value, const char, char>*>(base) + i * 4u);
}
template <int N>
__device__ __forceinline__ void pin(float (&v)[N]) {   // the values have arrived here
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(v[i]));
}

// One 16-column tile of a product over the activations in LDS: acc[t] = rows 16 t .. of
// act[., 0..K) x B.  A lane takes k = 16 u + 4 (lane / 16) + e of group u; kTinyDepth of whole groups are requested
// at a time, what is left of K past them (`rest`) with the first: there act is zero from column K on, and so is
// W[zero].   BT = false: B(k, c) = W[k * ldw + c];   true: B(k, c) = W[c * ldw + k]
struct TinyB { float b[kTinyDepth / 4], rest[4]; };
template <bool BT>
__device__ __forceinline__ void tiny_request(TinyB& r, const float* __restrict__ W, unsigned ldw, int K, int k0, int c) {
  const unsigned q = (threadIdx.x & 63) >> 4, lane = (BT ? c * ldw + 4u * q : 4u * q * ldw + c) * 4u;   // bytes
  const float* g = W + (BT ? (unsigned)k0 : (unsigned)k0 * ldw);   // uniform
#pragma unroll
  for (int u = 0; u < kTinyDepth / 16; ++u) {
    if (k0 + 16 * u + 16 <= K) {
      if (BT) {
        const f32x4 v = *reinterpret_cast<const f32x4_u*>(reinterpret_cast<const char*>(g) + lane);
#pragma unroll
        for (int e = 0; e < 4; ++e) r.b[4 * u + e] = v[e];
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) r.b[4 * u + e] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(g + (unsigned)e * ldw) + lane);
      }
    }
    g += BT ? 16u : 16u * ldw;
  }
}
template <bool BT>
__device__ __forceinline__ void tiny_request_rest(TinyB& r, const float* __restrict__ W, unsigned zero, unsigned ldw, int K, int c) {
  const int k = K / 16 * 16 + 4 * ((threadIdx.x & 63) >> 4);
  if (K % 16 != 0) {                                       // (uniform)
#pragma unroll
    for (int e = 0; e < 4; ++e) r.rest[e] = at(W, k + e < K ? (BT ? c * ldw + (unsigned)(k + e) : (unsigned)(k + e) * ldw + c) : zero);
  }
}
template <int MT, bool BT>
__device__ __forceinline__ void tiny_tile(f32x4 (&acc)[MT], TinyB& r, const float* act, int pitch, const float* __restrict__ W,
                                          unsigned ldw, int K, int c) {
  const int l = threadIdx.x & 63, q = l >> 4;
#pragma unroll
  for (int t = 0; t < MT; ++t) acc[t] = 0.f;
  auto group = [&](const float* b, int kg) {
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const f32x4 a = *reinterpret_cast<const f32x4*>(act + (t * 16 + (l & 15)) * pitch + kg + 4 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], acc[t], 0, 0, 0);
    }
  };
  for (int k0 = 0;;) {
    pin(r.b);
#pragma unroll
    for (int u = 0; u < kTinyDepth / 16; ++u)
      if (k0 + 16 * u + 16 <= K) group(r.b + 4 * u, k0 + 16 * u);
    k0 += kTinyDepth;
    if (k0 + 16 > K) break;
    tiny_request<BT>(r, W, ldw, K, k0, c);
  }
  if (K % 16 != 0) {
    pin(r.rest);
    group(r.rest, K / 16 * 16);
  }
}

// rows [mb][w] of memory -> LDS, rows and columns past the end zero.  All is requested before the first value is used: piece by piece
// this was a round trip to a piece.
template <int MT>
__device__ __forceinline__ void tiny_rows(float* s, const float* __restrict__ g, int mb, int w) {
  constexpr int R = 16 * MT / kTinyWaves, C = MT == 4 ? 2 : 5;   // pieces of 64: rows of up to 64 or 256, and the pitch
  const int pitch = tiny_pitch(w), wave = threadIdx.x >> 6, l = threadIdx.x & 63;
  float v[C][R];
#pragma unroll
  for (int k = 0; k < C; ++k)
    if (64 * k < w) {                                      // (uniform)
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int m = wave + kTinyWaves * r, c = l + 64 * k;
        v[k][r] = at(g, (m < mb ? m : mb - 1) * w + (c < w ? c : w - 1));
      }
    }
#pragma unroll
  for (int k = 0; k < C; ++k)
    if (64 * k < pitch) {                                  // (uniform)
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int m = wave + kTinyWaves * r, c = l + 64 * k;
        if (c < pitch) s[m * pitch + c] = m < mb && c < w ? v[k][r] : 0.f;
      }
    }
}

struct TinyFwdReq { TinyB b; float bias[1]; };
template <int NL, int MT>
__global__ __launch_bounds__(kTinyThreads) void tiny_fwd_kernel(Tiny p, const float* __restrict__ w, const float* __restrict__ in,
                                                                float* __restrict__ stash, float* __restrict__ out, int half) {
  extern __shared__ __align__(16) float act[];
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, q = l >> 4;
  // every workgroup needs every hidden activation; the last layer is shared out
  auto first = [&](int i) { return i == NL - 1 ? (int)blockIdx.x * kTinyWaves + wave : wave; };
  auto request = [&](TinyFwdReq& r, int i, int t) {
    const int N = p.dim[i + 1], c = t * 16 + (l & 15), cc = c < N ? c : N - 1;
    tiny_request<false>(r.b, w + p.offW[i], N, p.dim[i], 0, cc);
    tiny_request_rest<false>(r.b, w + p.offW[i], p.zero - p.offW[i], N, p.dim[i], cc);
    r.bias[0] = at(w, p.offB[i] + cc);
  };
  TinyFwdReq req[NL];
  request(req[0], 0, first(0));
  request(req[1], 1, first(1));
  // (the stash copy of the input: the first piece of a thread is on its way with the rows)
  const int n = p.mb * p.dim[0], i0 = (blockIdx.x * kTinyThreads + threadIdx.x) * 4;
  float* copy = stash + p.offA[0];
  f32x4 piece = 0.f;
  if (i0 + 4 <= n) piece = *reinterpret_cast<const f32x4_u*>(in + i0);
  tiny_rows<MT>(act, in, p.mb, p.dim[0]);
  if (i0 + 4 <= n) *reinterpret_cast<f32x4_u*>(copy + i0) = piece;
  for (int i = i0 + 4 <= n ? i0 + 4 * kTinyThreads * gridDim.x : i0; i < n; i += 4 * kTinyThreads * gridDim.x)
#pragma unroll 1
    for (int e = i; e < i + 4 && e < n; ++e) copy[e] = in[e];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int K = p.dim[i], N = p.dim[i + 1];
    const bool last = i == NL - 1;
    const float* src = act + (i & 1) * half;
    float* dst = act + ((i + 1) & 1) * half;
    const int dp = tiny_pitch(N), tiles = (N + 15) / 16, step = last ? kTinyWaves * gridDim.x : kTinyWaves;
    TinyFwdReq& cur = req[i];
    if (i + 2 < NL) request(req[i + 2], i + 2, first(i + 2));
    for (int t = first(i); t < tiles; t += step) {
      if (t != first(i)) request(cur, i, t);
      const int c = t * 16 + (l & 15);
      f32x4 acc[MT];
      tiny_tile<MT, false>(acc, cur.b, src, tiny_pitch(K), w + p.offW[i], N, K, c < N ? c : N - 1);
      pin(cur.bias);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = mt * 16 + 4 * q + r;
          float v = acc[mt][r] + cur.bias[0];
          if (!last) {
            v = c < N ? fmaxf(v, 0.f) : 0.f;
            dst[m * dp + c] = v;
            if (t % gridDim.x == blockIdx.x && m < p.mb && c < N) at(stash, p.offA[i + 1] + m * N + c) = v;
          } else if (m < p.mb && c < N) {
            at(out, m * N + c) = v;
          }
        }
    }
    if (!last) __syncthreads();
  }
}

template <int MT> struct TinyBwdReq { TinyB b; float gate[4 * MT], a[4 * MT], w[4], v[4]; };
template <int NL, int MT>
__global__ __launch_bounds__(kTinyThreads) void tiny_bwd_kernel(Tiny p, const float* __restrict__ w, const float* __restrict__ stash,
                                                                const float* __restrict__ dout, float* __restrict__ din, Upd u,
                                                                int half) {
  extern __shared__ __align__(16) float act[];
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, q = l >> 4;
  const int waves = gridDim.x * kTinyWaves, me = blockIdx.x * kTinyWaves + wave;
  // d_{i-1} = (d_i W_i^T) where a_i > 0: a whole copy per workgroup, the stage's own input gradient shared out
  auto request_chain = [&](TinyBwdReq<MT>& r, int i, int t) {
    const int K = p.dim[i], N = p.dim[i + 1], c = t * 16 + (l & 15), cc = c < K ? c : K - 1;
    tiny_request<true>(r.b, w + p.offW[i], N, N, 0, cc);
    tiny_request_rest<true>(r.b, w + p.offW[i], p.zero - p.offW[i], N, N, cc);
#pragma unroll
    for (int k = 0; k < 4 * MT; ++k) {
      const int m = k / 4 * 16 + 4 * q + k % 4;
      r.gate[k] = at(stash, p.offA[i] + (m < p.mb ? m : p.mb - 1) * K + cc);
    }
  };
  // dW_i = a_i^T d_i and db_i = column sums of d_i (a row K of ones below a_i): 16x16 tiles dealt out over all waves
  auto row = [&](int i, int t) -> int { return (unsigned)t * p.over[i] >> 16; };   // of tiles
  auto offsets = [&](int i, int t, unsigned (&o)[4]) {     // of a lane's four results
    const int K = p.dim[i], N = p.dim[i + 1], tn = (N + 15) / 16, tk = row(i, t), k = tk * 16 + 4 * q, c = (t - tk * tn) * 16 + (l & 15);
    const unsigned cc = c < N ? c : N - 1, bias = p.offB[i] + cc, weight = p.offW[i] + k * N + cc;
#pragma unroll
    for (int r = 0; r < 4; ++r) o[r] = k + r < K ? weight + r * N : bias;
  };
  auto request_grad = [&](TinyBwdReq<MT>& r, int i, int t) {
    const int K = p.dim[i], kr = row(i, t) * 16 + (l & 15);
#pragma unroll
    for (int k = 0; k < 4 * MT; ++k) {
      const int m = 4 * k + q;
      r.a[k] = at(stash, p.offA[i] + (m < p.mb ? m : p.mb - 1) * K + (kr < K ? kr : K - 1));
    }
    if (u.w) {
      unsigned o[4];
      offsets(i, t, o);
#pragma unroll
      for (int k = 0; k < 4; ++k) r.w[k] = at(u.w, o[k]);
      if (u.vel) {
#pragma unroll
        for (int k = 0; k < 4; ++k) r.v[k] = at(u.vel, o[k]);
      }
    }
  };
  auto grad_tiles = [&](int i) { return (p.dim[i] + 16) / 16 * ((p.dim[i + 1] + 15) / 16); };
  auto request = [&](TinyBwdReq<MT>& r, int i, int tc, int tg) {
    if (i > 0 || din) request_chain(r, i, tc);
    request_grad(r, i, tg < grad_tiles(i) ? tg : 0);
  };
  auto first_chain = [&](int i) { return i == 0 ? me : wave; };

  int first_grad[NL];                                      // this wave's first tile of layer i (the deal goes on from layer to layer)
#pragma unroll
  for (int i = NL - 1, t = me; i >= 0; --i) {
    first_grad[i] = t;
    t -= p.skip[i];
    if (t < 0) t += waves;
  }
  constexpr int AHEAD = MT == 1 || (MT == 2 && NL == 2) ? 2 : 1;   // layers requested ahead (what the registers hold)
  TinyBwdReq<MT> req[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i)
#pragma unroll
    for (int k = 0; k < 4; ++k) { req[i].w[k] = 0.f; req[i].v[k] = 0.f; }
#pragma unroll
  for (int i = NL - 1; i >= NL - AHEAD; --i) request(req[i], i, first_chain(i), first_grad[i]);
  tiny_rows<MT>(act, dout, p.mb, p.dim[NL]);
  __syncthreads();
#pragma unroll
  for (int i = NL - 1; i >= 0; --i) {
    const int side = (NL - 1 - i) & 1;
    const int K = p.dim[i], N = p.dim[i + 1];
    const float* d = act + side * half;                    // dL/dz_i
    float* below = act + (side ^ 1) * half;
    const int dp = tiny_pitch(N), bp = tiny_pitch(K), gt = grad_tiles(i), tg = first_grad[i];
    TinyBwdReq<MT>& cur = req[i];
    if (i >= AHEAD) request(req[i - AHEAD], i - AHEAD, first_chain(i - AHEAD), first_grad[i - AHEAD]);
    if (i > 0 || din) {
      const bool share = i == 0;
      const int tiles = (K + 15) / 16;
      for (int t = first_chain(i); t < tiles; t += share ? waves : kTinyWaves) {
        if (t != first_chain(i)) request_chain(cur, i, t);
        const int c = t * 16 + (l & 15);
        f32x4 acc[MT];
        tiny_tile<MT, true>(acc, cur.b, d, dp, w + p.offW[i], N, N, c < K ? c : K - 1);
        pin(cur.gate);
#pragma unroll
        for (int k = 0; k < 4 * MT; ++k) {
          const int m = k / 4 * 16 + 4 * q + k % 4;
          const float v = acc[k / 4][k % 4];
          if (!share) below[m * bp + c] = m < p.mb && c < K && cur.gate[k] > 0.f ? v : 0.f;
          else if (m < p.mb && c < K) at(din, m * K + c) = v;
        }
      }
    }
    for (int t = tg; t < gt; t += waves) {
      if (t != tg) request_grad(cur, i, t);
      const int tn = (N + 15) / 16, tk = row(i, t), kr = tk * 16 + (l & 15), c = (t - tk * tn) * 16 + (l & 15);
      f32x4 acc = 0.f;
      pin(cur.a); pin(cur.w); pin(cur.v);
#pragma unroll
      for (int k = 0; k < 4 * MT; ++k) {                   // four rows of the microbatch at a time; past its end both are zero
        const float a = 4 * k + q < p.mb ? kr < K ? cur.a[k] : 1.f : 0.f;
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, d[(4 * k + q) * dp + c], acc, 0, 0, 0);
      }
      unsigned to[4];
      offsets(i, t, to);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (c < N && tk * 16 + 4 * q + r <= K) {
          const unsigned o = to[r];
          at(u.grad, o) = acc[r];
          if (u.w) {
            float x = cur.w[r];
            if (u.vel) {
              const float v = next_velocity(u, x, cur.v[r], acc[r]);
              at(u.vel, o) = v;
              x = __fmaf_rn(-u.eta, v, x);
            } else {
              x = __fmaf_rn(-u.eta, acc[r], x);
            }
            at(u.w, o) = x;
            at(u.ver, o) = x;
          }
        }
    }
    if (i > 0) __syncthreads();
  }
}

int tiny_half(const rv_stage* s) {   // floats of one LDS activation buffer
  const int rows = (s->microbatch + 15) / 16;
  return 16 * (rows > 2 ? 4 : rows) * tiny_pitch((int)((MlpPlan*)s->impl)->maxw);
}
Tiny tiny_desc(const rv_stage* s, int wgs) {
  const MlpPlan* p = (const MlpPlan*)s->impl;
  Tiny t = {};
  t.mb = s->microbatch; t.zero = (unsigned)s->P;
  for (int i = 0; i <= p->n; ++i) t.dim[i] = (int)s->dims[i];
  for (int i = 0; i < p->n; ++i) { t.offW[i] = (unsigned)p->offW[i]; t.offB[i] = (unsigned)p->offB[i]; t.offA[i] = (unsigned)p->offA[i]; }
  for (int i = 0; i < p->n; ++i) {
    const int tn = (t.dim[i + 1] + 15) / 16;
    t.over[i] = (65536u + tn - 1) / tn;
    t.skip[i] = (t.dim[i] + 16) / 16 * tn % (wgs * kTinyWaves);
  }
  return t;
}
template <typename F>
rv_status tiny_by_shape(int n, int mt, F f) {   // layers (2, 3, 4) and 16-row groups as constants
  auto rows = [&](auto nl) { return mt == 1 ? f(nl, Int<1>()) : mt == 2 ? f(nl, Int<2>()) : f(nl, Int<4>()); };
  return n == 2 ? rows(Int<2>()) : n == 3 ? rows(Int<3>()) : rows(Int<4>());
}
// [mb, wa] and [mb, wb] floats
bool overlap(const rv_stage* s, const void* a, int64_t wa, const void* b, int64_t wb) {
  const size_t row = (size_t)s->microbatch * 4;
  return rv_overlap(a, row * wa, b, row * wb);
}
}  // namespace

rv_status rv_mlp_plan(rv_stage* s) {
  MlpPlan* p = new (std::nothrow) MlpPlan();
  if (!p) return RV_E_NOMEM;
  s->impl = p;
  p->n = s->n_layers;
  size_t off = 0, offa = 0;
  for (int i = 0; i <= p->n; ++i) {
    if (s->dims[i] < 1 || s->dims[i] > (1 << 20)) return RV_E_INVAL;
    p->maxw = std::max(p->maxw, (size_t)s->dims[i]);
  }
  for (int i = 0; i < p->n; ++i) {
    p->offW.push_back(off); off += (size_t)s->dims[i] * s->dims[i + 1];
    p->offB.push_back(off); off += (size_t)s->dims[i + 1];
    p->offA.push_back(offa); offa += (size_t)s->microbatch * s->dims[i];
  }
  s->P = off;
  s->slot_bytes = offa * 4;
  s->work_bytes = 2 * (size_t)s->microbatch * p->maxw * 4;
  // One launch per direction, or one per layer and direction?  Forward + backward of one microbatch, us on the device (one per
  // direction / one per layer):
  //   8 rows    16-16-16 8.2 / 10.8   64-128-64 11.8 / 13.7   64-64-64-64 12.6 / 19.1   64-64-64-64-64 15.4 / 25.5
  //   16 rows   128-128-128-128 21.3 / 23.0   20-60-200-60-20 21.6 / 29.8   144-144-144-144 27.9 / 22.7   200-200-200 25.3 / 16.8
  //   32 rows   64-64-64-64 15.7 / 20.1   96-96-96-96 24.4 / 23.1   112-112-112-112 26.3 / 22.8
  //   64 rows   16-16-16 12.3 / 12.4   48-48-48-48 24.3 / 20.9   64-64-64-64-64 39.2 / 28.5
  // The limit was fitted when a launch of a layer took about 5 us whatever it did, and the repeated chain about 8 + 2.5 (g - 1) us and
  // (0.2 + 0.11 g) ns per parameter, g = 1, 2, 4 groups of 16 rows; both are shorter now, the layers' by more.  By device time alone one
  // launch is taken too often past 128 wide and with four groups; but issuing a launch takes the host 2.7 us, which is what such
  // stages last where calls follow one another.  With four groups rows wider than 64 lose whatever the other widths.
  const int g = s->microbatch <= 16 ? 1 : s->microbatch <= 32 ? 2 : 4;
  p->tiny = p->n >= 2 && p->n <= kTinyLayers && s->microbatch <= kTinyRows && p->maxw <= (g == 4 ? 64 : 256) &&
            (20.0 + 11.0 * g) * (double)off < 1e5 * (10.0 * p->n - 5.5 - 2.5 * g);
  return RV_OK;
}

void rv_mlp_free(rv_stage* s) {
  delete (MlpPlan*)s->impl;
  s->impl = nullptr;
}

rv_status rv_mlp_forward(rv_stage* s, rv_slot& slot, const void* in, void* out) {
  MlpPlan* p = (MlpPlan*)s->impl;
  const float* w = (const float*)s->ver[slot.ver];
  float* stash = (float*)slot.base;
  const int mb = s->microbatch;
  // a caller may hand the same buffer in and out: then nothing may be written before all of it is read
  const bool in_place = overlap(s, in, s->dims[0], out, s->dims[p->n]);
  if (p->tiny && !in_place) {
    const int half = tiny_half(s), mt = (mb + 15) / 16;
    const int wgs = ((int)s->dims[p->n] + 16 * kTinyWaves - 1) / (16 * kTinyWaves);
    const Tiny t = tiny_desc(s, wgs);
    const size_t lds = 2 * (size_t)half * 4;
    return tiny_by_shape(p->n, mt, [&](auto nl, auto m) -> rv_status {
      constexpr auto kern = tiny_fwd_kernel<decltype(nl)::value, decltype(m)::value>;
      static const rv_status ok = allow_lds(kern, 160 * 1024);
      RV_TRY(ok);
      hipLaunchKernelGGL(kern, dim3(wgs), dim3(kTinyThreads), lds, s->st, t, w, (const float*)in, stash, (float*)out, half);
      return rv_launch_status();
    });
  }
  const bool copy_first = in_place && p->n == 1;
  if (copy_first) RV_HIP_TRY(hipMemcpyAsync(stash, in, (size_t)mb * s->dims[0] * 4, hipMemcpyDeviceToDevice, s->st));
  for (int i = 0; i < p->n; ++i) {
    const bool last = i == p->n - 1, first = i == 0 && !copy_first;
    const int K = (int)s->dims[i], N = (int)s->dims[i + 1];
    int bt = pick(mb, N, K);
    if (slim_forward(mb, N, K, bt, first)) bt = kSlim;
    // one tile to a CU; the shortest walks are mostly beginning (1024 -> 1024 rows, us, whole / halves: 32 in k 6.3 / 6.6, 64 7.2 / 7.2, 100 9.0 / 8.5,
    // 128 9.2 / 8.6, 200 10.9 / 10.6)
    if (bt == 64 && tile_count(mb, N, 64) <= kCUs && K >= 80) bt = kHalves;
    const Prod pr = product(first ? (const float*)in : stash + p->offA[i], K, w + p->offW[i], N, mb, N, K, bt, threads(bt));
    Out o = {};
    o.C = last ? (float*)out : stash + p->offA[i + 1]; o.bias = w + p->offB[i]; o.relu = !last;
    float* copy = first ? stash : nullptr;
    const rv_status rc = bt == 128  ? launch_fwd<128, 256>(s->st, pr, o, copy)
                         : bt == 64 ? launch_fwd<64, 256>(s->st, pr, o, copy)
                         : bt == kWave ? launch_fwd<kWave, 256>(s->st, pr, o, copy)
                         : bt == kSlim ? launch_fwd<kSlim, 64 * kSplitWaves>(s->st, pr, o, copy)
                         : bt == kHalves ? launch_fwd<kHalves, 512>(s->st, pr, o, copy)
                                    : launch_fwd<32, 64 * kSplitWaves>(s->st, pr, o, copy);
    RV_TRY(rc);
  }
  return rv_launch_status();
}

// The gradient of every layer, and the update where the epilogues can apply it (s->fused: plain
// or momentum step of a backward that updates); otherwise the caller follows with rv_stage_update_range.
rv_status rv_mlp_backward(rv_stage* s, rv_slot& slot, const void* grad_out, void* grad_in) {
  MlpPlan* p = (MlpPlan*)s->impl;
  const float* w = (const float*)s->ver[slot.ver];
  const float* stash = (const float*)slot.base;
  const int mb = s->microbatch;
  Upd u = {s->grad, nullptr, nullptr, nullptr, s->eta, s->momentum, s->weight_decay};
  if (s->fused) { u.w = s->master; u.vel = s->vel; u.ver = (float*)s->ver[s->upd_dst]; }
  if (p->tiny && !overlap(s, grad_out, s->dims[p->n], grad_in, s->dims[0])) {
    const int half = tiny_half(s), mt = (mb + 15) / 16;
    int tiles = 0;
    for (int i = 0; i < p->n; ++i) tiles += ((int)s->dims[i] + 16) / 16 * (((int)s->dims[i + 1] + 15) / 16);
    const int wgs = std::min(64, (tiles + kTinyWaves - 1) / kTinyWaves);
    const Tiny t = tiny_desc(s, wgs);
    const size_t lds = 2 * (size_t)half * 4;
    return tiny_by_shape(p->n, mt, [&](auto nl, auto m) -> rv_status {
      constexpr auto kern = tiny_bwd_kernel<decltype(nl)::value, decltype(m)::value>;
      static const rv_status ok = allow_lds(kern, 160 * 1024);
      RV_TRY(ok);
      hipLaunchKernelGGL(kern, dim3(wgs), dim3(kTinyThreads), lds, s->st, t, w, stash, (const float*)grad_out, (float*)grad_in, u,
                         half);
      return rv_launch_status();
    });
  }
  float* ping = (float*)s->work;
  float* pong = ping + (size_t)mb * p->maxw;
  const float* d = (const float*)grad_out;   // dL/dz_i, already gated
  if (p->n == 1 && overlap(s, grad_out, s->dims[1], grad_in, s->dims[0])) {
    // the one launch reads the gradient for all its parts while the input gradient is written over it
    RV_HIP_TRY(hipMemcpyAsync(ping, grad_out, (size_t)mb * s->dims[1] * 4, hipMemcpyDeviceToDevice, s->st));
    d = ping;
  }
  for (int i = p->n - 1; i >= 0; --i) {
    const int K = (int)s->dims[i], N = (int)s->dims[i + 1];
    const float* a = stash + p->offA[i];
    const bool want_dx = i > 0 || grad_in;
    float* dst = i == 0 ? (float*)grad_in : (d == ping ? pong : ping);
    // 64x64 tiles beside a walk that is dealt out over eight waves go two to a workgroup: weight-gradient tiles always, those of an input
    // gradient where the weight gradient's walk is much the longer one (us, four waves / eight: 700 -> 60 on 1000 rows 14.8 / 12.2, 1024 -> 128
    // on 1024 15.7 / 12.3, 500 -> 250 on 2000 28.2 / 22.3, 2000 -> 60 on 300 9.2 / 7.9; 2000 -> 77 on 300 9.8 / 10.6, 1024 -> 200 on 1024 17.7 / 18.9)
    const int bx = pick(mb, K, N), bw = pick(K, N, mb);
    const bool pairs = (bx == 32 && bw == 64) || (bx == 64 && bw == 32 && mb >= (N <= 64 ? 4 : 6) * N);
    const int nt = std::max(bx, bw) == 32 || pairs ? threads(32) : 256;
    const Prod pw = product(a, K, d, N, K, N, mb, bw, nt);
    const int form = nt == threads(32) && want_dx && slim_backward(mb, K, N, bx, pw.tiles + (N + 31) / 32) ? kSlim : bx;
    Prod px = product(d, N, w + p->offW[i], N, mb, K, N, form, nt);
    if (!want_dx) px.tiles = 0;
    Out ox = {}, ow = {};
    ox.C = dst; ox.gate = i > 0 ? a : nullptr;
    ow.u = u; ow.off = p->offW[i];
    auto go = [&](auto launch) { return launch(s->st, px, ox, pw, ow, d, mb, N, p->offB[i]); };
    // Beside 128x128 tiles, which are made for four waves, a split form has four instead of eight, also where the input
    // gradient's walk is the longer one: 32x32 weight-gradient tiles with eight waves for both took (one layer, backward, us)
    // 49 instead of 23 at 4096 -> 1024 on 8 rows, 188 / 87 at 4096 -> 4096 on 16, 273 / 98 on 64.
    auto by_bw = [&](auto x) {
      constexpr int BX = decltype(x)::value, NT = BX <= 32 ? 64 * kSplitWaves : 256;
      if constexpr (BX == kSlim)
        return bw == 64 ? go(launch_bwd<BX, 64, NT>) : bw == 32 ? go(launch_bwd<BX, 32, NT>) : go(launch_bwd<BX, kWave, NT>);
      else
      return bw == 128 ? go(launch_bwd<BX, 128, 256>) : bw == 64 ? go(launch_bwd<BX, 64, BX == 32 ? NT : 256>)
             : bw == 32 && BX == 64 && pairs ? go(launch_bwd<BX, 32, BX == 64 ? 64 * kSplitWaves : NT>)
             : bw == 32 ? go(launch_bwd<BX, 32, NT>) : go(launch_bwd<BX, kWave, BX == 32 ? NT : 256>);
    };
    const rv_status rc = form == kSlim ? by_bw(Int<kSlim>()) : bx == 128 ? by_bw(Int<128>()) : bx == 64 ? by_bw(Int<64>()) : bx == 32 ? by_bw(Int<32>()) : by_bw(Int<kWave>());
    RV_TRY(rc);
    if (want_dx) d = dst;
  }
  return rv_launch_status();
}
