// Cluster average: the arithmetic of Parallel Multi-Ring All-Reduce (paper section 3.2,
// built on the ring all-reduce of section 2.3) for C replicas resident in one HBM.
//
// The network rounds disappear on one GPU; what remains of the algorithm is the
// partition (ring -> segment -> C chunks) and the order of the additions: chunk j is
// accumulated starting at replica j and walking the ring, then divided by C once.
// Each input element is read exactly once and each output written once, so the kernel
// is bound by HBM: (C+1)*4 bytes per element (+4 with a folded-in gradient; 2C*4 with
// write-back).
//
// Layout: one workgroup owns a tile of TILE consecutive elements.  Chunks are millions of
// elements long, so almost every tile lies inside one chunk: its rotation j is
// wave-uniform, the C replica base pointers are fetched with scalar loads in rotated
// order and each lane streams C independent 16-byte loads before the first add.
// Tiles that straddle a chunk boundary and the ragged tail take an element-wise path that
// computes the owning chunk per element.
//
// For the stages' own averaging (rv_cluster_sync) the same pass also leaves the mean as every
// stage's new weight version (Versions below): reading the written-back masters again, replica by replica,
// cost 6 (bf16) bytes per element and replica where storing the mean here costs 2 (an averaging
// iteration over four stages of 50 M parameters: 6.47 -> 6.17 ms).
#include "internal.h"

#define RV_MAX_C 64
#define RV_MAX_R 4096

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef f4 f4_u __attribute__((aligned(4)));   // 16-byte accesses at any float's address
typedef unsigned int u2 __attribute__((ext_vector_type(2)));

struct RepTable {
  float* p[RV_MAX_C];
};

// where the mean goes as a weight version: kind 0 nowhere, 2 fp32, 3 bf16 through the map
struct Versions {
  void* p[RV_MAX_C];
  int kind;
  rv_ver_map map;
};

constexpr int kThreads = 256;
constexpr int kTile = kThreads * 4;    // elements per tile: one float4 per lane
constexpr int kBatch = 8;              // replicas requested at a time when C is no compile-time constant

// Owning chunk of element i: ring r = ceil((i+1) R / n) - 1, then the same rule inside
// the ring's segment.
__device__ __forceinline__ int chunk_of(uint64_t i, uint64_t n, int R, int C) {
  uint64_t r = ((i + 1) * (uint64_t)R - 1) / n;
  uint64_t lo = (r * n) / (uint64_t)R;
  uint64_t hi = ((r + 1) * n) / (uint64_t)R;
  uint64_t s = hi - lo;
  return (int)(((i - lo + 1) * (uint64_t)C - 1) / s);
}

// Rings given by explicit boundaries (segments of unequal size, as when clusters split the
// model differently and a peer sits in several rings): off[0] = 0 <= ... <= off[R] = n.
#define RV_MAX_EXPLICIT_R 64
struct RingOffsets {
  uint64_t off[RV_MAX_EXPLICIT_R + 1];
};
__device__ __forceinline__ void ring_of(const RingOffsets& ro, int R, uint64_t i, uint64_t& lo, uint64_t& hi) {
  int r = 0;
  while (r + 1 < R && i >= ro.off[r + 1]) ++r;     // empty rings are stepped over
  lo = ro.off[r]; hi = ro.off[r + 1];
}
__device__ __forceinline__ int chunk_of_v(const RingOffsets& ro, int R, uint64_t i, int C) {
  uint64_t lo, hi;
  ring_of(ro, R, i, lo, hi);
  return (int)(((i - lo + 1) * (uint64_t)C - 1) / (hi - lo));
}

__device__ __forceinline__ float elem_mean(const RepTable& tab, int C, int j, uint64_t i,
                                           const float* grad, int gr, float eta) {
  float acc = 0.f;
  for (int s = 0; s < C; ++s) {
    int c = j + s; if (c >= C) c -= C;
    float v = tab.p[c][i];
    if (grad != nullptr && c == gr) v = __fsub_rn(v, __fmul_rn(grad[i], eta));
    acc = (s == 0) ? v : __fadd_rn(acc, v);
  }
  return __fdiv_rn(acc, (float)C);
}

// The C replica base pointers are fetched with scalar loads in ring order starting at j
// (wave-uniform), every lane issues its C independent 16-byte loads, then adds them in
// that order.  (A compile-time rotation of the SUM order over naturally ordered loads was
// tried: the compiler folds the C unrolled variants back into a dynamically indexed
// register array in scratch memory, which costs a third of the bandwidth.)
// C is a compile-time constant up to 16; beyond, kBatch loads are in flight at a time.  (With the
// element path for every C but 1, 2, 3, 4, 8 and 16, C = 6 over
// 1e8 elements written back took 1.68 ms, 2.9 TB/s; this way 0.87 ms, 5.5.)
template <bool HAS_GRAD>
__device__ __forceinline__ f4 replica_term(const RepTable& tab, int c, uint64_t e, const float* grad, int gr, float eta) {
  f4 v = __builtin_nontemporal_load(reinterpret_cast<const f4_u*>(tab.p[c] + e));
  if (HAS_GRAD && c == gr) {
    const f4 g = __builtin_nontemporal_load(reinterpret_cast<const f4_u*>(grad + e));
    v.x = __fsub_rn(v.x, __fmul_rn(g.x, eta));
    v.y = __fsub_rn(v.y, __fmul_rn(g.y, eta));
    v.z = __fsub_rn(v.z, __fmul_rn(g.z, eta));
    v.w = __fsub_rn(v.w, __fmul_rn(g.w, eta));
  }
  return v;
}
__device__ __forceinline__ void add_term(f4& a, f4 v) {
  a.x = __fadd_rn(a.x, v.x); a.y = __fadd_rn(a.y, v.y);
  a.z = __fadd_rn(a.z, v.z); a.w = __fadd_rn(a.w, v.w);
}
template <int CT, bool HAS_GRAD>
__device__ __forceinline__ void tile_fast(const RepTable& tab, const Versions& ver, int Crt, int j, uint64_t base, float* out,
                                          int write_back, const float* grad, int gr, float eta) {
  const int C = CT > 0 ? CT : Crt;
  const float c_num = (float)C;
  j = __builtin_amdgcn_readfirstlane(j);
  const uint64_t e = base + (uint64_t)threadIdx.x * 4;
  f4 a;
  if constexpr (CT > 0) {
    f4 v[CT];
#pragma unroll
    for (int s = 0; s < CT; ++s) {
      int c = j + s; if (c >= CT) c -= CT;
      v[s] = replica_term<HAS_GRAD>(tab, c, e, grad, gr, eta);
    }
    a = v[0];
#pragma unroll
    for (int s = 1; s < CT; ++s) add_term(a, v[s]);
  } else {
    int s = 0;
    for (; s + kBatch <= C; s += kBatch) {
      f4 v[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        int c = j + s + u; if (c >= C) c -= C;
        v[u] = replica_term<HAS_GRAD>(tab, c, e, grad, gr, eta);
      }
      if (s == 0) a = v[0]; else add_term(a, v[0]);
#pragma unroll
      for (int u = 1; u < kBatch; ++u) add_term(a, v[u]);
    }
    for (; s < C; ++s) {
      int c = j + s; if (c >= C) c -= C;
      add_term(a, replica_term<HAS_GRAD>(tab, c, e, grad, gr, eta));   // (C > 16: s > 0 here)
    }
  }
  a.x = __fdiv_rn(a.x, c_num);
  a.y = __fdiv_rn(a.y, c_num);
  a.z = __fdiv_rn(a.z, c_num);
  a.w = __fdiv_rn(a.w, c_num);
  if (out != nullptr) __builtin_nontemporal_store(a, reinterpret_cast<f4_u*>(out + e));
  if (write_back) {
#pragma unroll
    for (int c = 0; c < C; ++c)
      __builtin_nontemporal_store(a, reinterpret_cast<f4_u*>(tab.p[c] + e));
  }
  if (ver.kind == 3) {
    u2 h;
    h.x = rv_pack_bf16x2(a.x, a.y); h.y = rv_pack_bf16x2(a.z, a.w);
    const uint64_t at = rv_ver_at(ver.map, base, e);
#pragma unroll
    for (int c = 0; c < C; ++c) *reinterpret_cast<u2*>((uint16_t*)ver.p[c] + at) = h;
  } else if (ver.kind == 2) {
#pragma unroll
    for (int c = 0; c < C; ++c) __builtin_nontemporal_store(a, reinterpret_cast<f4*>((float*)ver.p[c] + e));
  }
}

// floor(x / d) for x < 2^52 from an fp64 estimate (inv_d = 1/d rounded) and one exact
// correction step: the estimate is within one of the quotient, q*d fits in 64 bits.
__device__ __forceinline__ uint64_t floor_div(uint64_t x, uint64_t d, double inv_d) {
  uint64_t q = (uint64_t)((double)x * inv_d);
  if (q * d > x) --q;
  else if ((q + 1) * d <= x) ++q;
  return q;
}

struct DivConsts {
  double inv_n, inv_R, inv_C;
};

// Chunk that owns element i and the (exclusive) end of that chunk: the same arithmetic as
// chunk_of, without 64-bit integer division (it runs once per workgroup).
__device__ __forceinline__ void locate(uint64_t i, uint64_t n, int R, int C, const DivConsts& dc, int& j,
                                       uint64_t& chunk_end) {
  const uint64_t r = floor_div((i + 1) * (uint64_t)R - 1, n, dc.inv_n);
  const uint64_t lo = floor_div(r * n, (uint64_t)R, dc.inv_R), hi = floor_div((r + 1) * n, (uint64_t)R, dc.inv_R);
  const uint64_t s = hi - lo;
  j = (int)floor_div((i - lo + 1) * (uint64_t)C - 1, s, 1.0 / (double)s);
  chunk_end = lo + floor_div((uint64_t)(j + 1) * s, (uint64_t)C, dc.inv_C);
}

// One workgroup per tile.  CT == 0: C at run time.
template <int CT, bool HAS_GRAD, bool EXPL>
__global__ __launch_bounds__(kThreads) void average_kernel(RepTable tab, Versions ver, int Crt, uint64_t n, int R,
                                                           float* out, int write_back,
                                                           const float* grad, int gr, float eta,
                                                           DivConsts dc, RingOffsets ro) {
  const int C = CT > 0 ? CT : Crt;
  const uint64_t base = (uint64_t)(ver.kind == 3 ? rv_ver_tile(blockIdx.x, gridDim.x) : blockIdx.x) * kTile, last = base + kTile - 1;
  int j;
  uint64_t chunk_end;
  if (EXPL) {
    uint64_t lo, hi;
    ring_of(ro, R, base, lo, hi);
    const uint64_t sz = hi - lo;
    j = (int)floor_div((base - lo + 1) * (uint64_t)C - 1, sz, 1.0 / (double)sz);
    chunk_end = lo + floor_div((uint64_t)(j + 1) * sz, (uint64_t)C, dc.inv_C);
  } else {
    locate(base, n, R, C, dc, j, chunk_end);   // wave-uniform, no barrier needed
  }
  if (last < chunk_end) {                      // chunk_end <= n: the tile is whole and inside one chunk
    tile_fast<CT, HAS_GRAD>(tab, ver, Crt, j, base, out, write_back, grad, gr, eta);
    return;
  }
  for (int k = threadIdx.x; k < kTile; k += kThreads) {
    const uint64_t i = base + k;
    if (i >= n) break;
    const int je = EXPL ? chunk_of_v(ro, R, i, C) : chunk_of(i, n, R, C);
    const float m = elem_mean(tab, C, je, i, HAS_GRAD ? grad : nullptr, gr, eta);
    if (out != nullptr) out[i] = m;
    if (write_back)
      for (int c = 0; c < C; ++c) tab.p[c][i] = m;
    for (int c = 0; ver.kind && c < C; ++c) {
      if (ver.kind == 3) ((uint16_t*)ver.p[c])[rv_ver_at(ver.map, base, i)] = rv_f32_to_bf16(m);
      else ((float*)ver.p[c])[i] = m;
    }
  }
}

template <int CT>
void launch(const RepTable& tab, const Versions& ver, int C, uint64_t n, int R, float* out, int wb, const float* grad,
            int gr, float eta, const RingOffsets* ro, hipStream_t st) {
  const unsigned blocks = (unsigned)((n + kTile - 1) / kTile);
  const DivConsts dc{1.0 / (double)n, 1.0 / (double)R, 1.0 / (double)C};
  static const RingOffsets none = {};
#define RV_AVG_LAUNCH(G, E)                                                                                   \
  hipLaunchKernelGGL((average_kernel<CT, G, E>), dim3(blocks), dim3(kThreads), 0, st, tab, ver, C, n, R, out, \
                     wb, grad, gr, eta, dc, E ? *ro : none)
  if (ro) { if (grad) RV_AVG_LAUNCH(true, true); else RV_AVG_LAUNCH(false, true); }
  else    { if (grad) RV_AVG_LAUNCH(true, false); else RV_AVG_LAUNCH(false, false); }
#undef RV_AVG_LAUNCH
}

template <int CT, typename... A>
void launch_for(int C, const A&... a) {   // CT = C up to 16
  if constexpr (CT <= 16) {
    if (C == CT) launch<CT>(a...); else launch_for<CT + 1>(C, a...);
  } else {
    launch<0>(a...);
  }
}

}  // namespace

static rv_status average_impl(float* const* replicas, int C, size_t n, int R, const RingOffsets* ro,
                              float* mean_out, int write_back, const float* grad, int grad_replica, float eta,
                              void* const* versions, int ver_kind, const rv_ver_map& map, void* stream) {
  if (replicas == nullptr || C < 1 || C > RV_MAX_C || R < 1 || R > RV_MAX_R || n == 0)
    return RV_E_INVAL;
  if (mean_out == nullptr && !write_back) return RV_E_INVAL;
  if (grad != nullptr && (grad_replica < 0 || grad_replica >= C)) return RV_E_INVAL;
  if (n > ((uint64_t)1 << 40)) return RV_E_INVAL;   // keeps (i+1)*R inside 64 bits
  RepTable tab = {};
  Versions ver = {};
  ver.kind = ver_kind;
  ver.map = map;
  for (int c = 0; c < C; ++c) {
    if (replicas[c] == nullptr) return RV_E_INVAL;
    for (int k = 0; k < c; ++k)
      if (replicas[k] == replicas[c]) return RV_E_INVAL;
    if (replicas[c] == mean_out) return RV_E_INVAL;
    tab.p[c] = replicas[c];
    if (ver_kind) ver.p[c] = versions[c];
  }
  launch_for<1>(C, tab, ver, C, (uint64_t)n, R, mean_out, write_back ? 1 : 0, grad, grad_replica, eta, ro, (hipStream_t)stream);
  return rv_launch_status();
}

rv_status rv_average_publish(float* const* masters, void* const* versions, int ver_kind, const rv_ver_map& map, int C, size_t n, int R,
                             const float* grad, int grad_replica, float eta, hipStream_t st) {
  return average_impl(masters, C, n, R, nullptr, nullptr, 1, grad, grad_replica, eta, versions, ver_kind, map, st);
}

extern "C" rv_status rv_cluster_average(float* const* replicas, int C, size_t n, int R,
                                        float* mean_out, int write_back, const float* grad,
                                        int grad_replica, float eta, void* stream) {
  return average_impl(replicas, C, n, R, nullptr, mean_out, write_back, grad, grad_replica, eta, nullptr, 0, rv_ver_map(), stream);
}

extern "C" rv_status rv_cluster_average_v(float* const* replicas, int C, size_t n, const int64_t* ring_offsets,
                                          int R, float* mean_out, int write_back, const float* grad,
                                          int grad_replica, float eta, void* stream) {
  if (ring_offsets == nullptr || R < 1 || R > RV_MAX_EXPLICIT_R) return RV_E_INVAL;
  if (ring_offsets[0] != 0 || ring_offsets[R] != (int64_t)n) return RV_E_INVAL;
  RingOffsets ro = {};
  for (int r = 0; r <= R; ++r) {
    if (r > 0 && ring_offsets[r] < ring_offsets[r - 1]) return RV_E_INVAL;
    ro.off[r] = (uint64_t)ring_offsets[r];
  }
  return average_impl(replicas, C, n, R, &ro, mean_out, write_back, grad, grad_replica, eta, nullptr, 0, rv_ver_map(), stream);
}
