// Delayed block SGD update (paper Eq. 2; Eq. 4 restricts it to the peer's own block):
// w <- w - eta * g on the flat fp32 master vector, one fused multiply-add per element,
// optionally emitting the new weights as the next weight version (bf16 for the
// decoder's matrix products, fp32 for the MLP stage).
//
// HBM-bound streaming kernel: reads w and g (4+4 B), writes w (4 B) and the version
// copy (2 or 4 B) per parameter.  16-byte accesses, one vector per lane and as many workgroups
// as tiles (measured best: 5.8 TB/s with the bf16 copy, 6.5 without).  A decoder stage taking the
// plain step does not come here: its update happens in the kernels that produce the gradient.
#include "common.h"
#include "internal.h"

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef unsigned int u2 __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256;
constexpr int kVec = 1;
constexpr int kTile = kThreads * kVec * 4;

// COPY: 0 none, 1 bf16, 2 fp32, 3 bf16 where the map puts it.  Without the bf16 version w and g stream through with non-temporal
// accesses (nothing is read twice; measured 76 % -> 81 % of HBM peak).  With it, only g does: every
// non-temporal access to w or to the version measured 3-5 % slower there (73 % -> 69-70 %), and so
// did 8 consecutive parameters per lane for a 16-byte bf16 store (the lanes of a wave must stay
// 16 bytes apart on w and g).
// ADD: the gradient is acc + g, the sum of a group's microbatches before this one and this one's: the last accumulation pass
// and the update in one, 8 B/param less than one after the other.
template <int COPY, bool ADD>
__global__ __launch_bounds__(kThreads) void update_kernel(float* __restrict__ w,
                                                          const float* __restrict__ g, uint64_t n,
                                                          float eta, void* __restrict__ copy,
                                                          int aligned, rv_ver_map map, const float* __restrict__ acc) {
  const uint64_t base = (uint64_t)(COPY == 3 ? rv_ver_tile(blockIdx.x, gridDim.x) : blockIdx.x) * kTile;
  if (aligned && base + kTile <= n) {
    f4 wv[kVec], gv[kVec];
#pragma unroll
    for (int u = 0; u < kVec; ++u) {
      uint64_t e = base + (uint64_t)(u * kThreads + threadIdx.x) * 4;
      if (COPY == 1 || COPY == 3) wv[u] = *reinterpret_cast<const f4*>(w + e);
      else wv[u] = __builtin_nontemporal_load(reinterpret_cast<const f4*>(w + e));
      gv[u] = __builtin_nontemporal_load(reinterpret_cast<const f4*>(g + e));
      if (ADD) gv[u] += __builtin_nontemporal_load(reinterpret_cast<const f4*>(acc + e));
    }
#pragma unroll
    for (int u = 0; u < kVec; ++u) {
      uint64_t e = base + (uint64_t)(u * kThreads + threadIdx.x) * 4;
      f4 r;
      r.x = __fmaf_rn(-eta, gv[u].x, wv[u].x);
      r.y = __fmaf_rn(-eta, gv[u].y, wv[u].y);
      r.z = __fmaf_rn(-eta, gv[u].z, wv[u].z);
      r.w = __fmaf_rn(-eta, gv[u].w, wv[u].w);
      if (COPY == 1 || COPY == 3) *reinterpret_cast<f4*>(w + e) = r;
      else __builtin_nontemporal_store(r, reinterpret_cast<f4*>(w + e));
      if (COPY == 1 || COPY == 3) {
        u2 pk;
        pk.x = rv_pack_bf16x2(r.x, r.y);
        pk.y = rv_pack_bf16x2(r.z, r.w);
        *reinterpret_cast<u2*>(reinterpret_cast<uint16_t*>(copy) + (COPY == 3 ? rv_ver_at(map, base, e) : e)) = pk;
      } else if (COPY == 2) {
        __builtin_nontemporal_store(r, reinterpret_cast<f4*>(reinterpret_cast<float*>(copy) + e));
      }
    }
    return;
  }
  for (int k = threadIdx.x; k < kTile; k += kThreads) {
    uint64_t i = base + k;
    if (i >= n) break;
    float r = __fmaf_rn(-eta, ADD ? acc[i] + g[i] : g[i], w[i]);
    w[i] = r;
    if (COPY == 1 || COPY == 3) reinterpret_cast<uint16_t*>(copy)[COPY == 3 ? rv_ver_at(map, base, i) : i] = rv_f32_to_bf16(r);
    if (COPY == 2) reinterpret_cast<float*>(copy)[i] = r;
  }
}

// The optimiser of the paper's single-cluster experiments (section 4.1: SGD with momentum
// 0.9 and weight decay 5e-4) as a variant of the same update, in the usual form
//   d = g + wd * w;   v <- mu * v + d;   w <- w - eta * v
// (three fused multiply-adds per element; wd = mu = 0 gives Eq. 2 bit for bit).
// 22 B/param with a bf16 copy: reads w, g, v, writes w, v, copy.
template <int COPY, bool ADD>
__global__ __launch_bounds__(kThreads) void update_momentum_kernel(float* __restrict__ w,
                                                                   const float* __restrict__ g,
                                                                   float* __restrict__ v, uint64_t n,
                                                                   float eta, float mu, float wd,
                                                                   void* __restrict__ copy, int aligned, rv_ver_map map,
                                                                   const float* __restrict__ acc) {
  const uint64_t base = (uint64_t)(COPY == 3 ? rv_ver_tile(blockIdx.x, gridDim.x) : blockIdx.x) * kTile;
  auto step = [&](float wi, float gi, float& vi) {
    const float d = __fmaf_rn(wd, wi, gi);
    vi = __fmaf_rn(mu, vi, d);
    return __fmaf_rn(-eta, vi, wi);
  };
  if (aligned && base + kTile <= n) {
#pragma unroll
    for (int u = 0; u < kVec; ++u) {
      const uint64_t e = base + (uint64_t)(u * kThreads + threadIdx.x) * 4;
      const f4 wv = *reinterpret_cast<const f4*>(w + e);
      f4 gv = __builtin_nontemporal_load(reinterpret_cast<const f4*>(g + e));
      if (ADD) gv += __builtin_nontemporal_load(reinterpret_cast<const f4*>(acc + e));
      f4 vv = *reinterpret_cast<const f4*>(v + e);
      f4 r;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        float vi = vv[c];
        r[c] = step(wv[c], gv[c], vi);
        vv[c] = vi;
      }
      *reinterpret_cast<f4*>(w + e) = r;
      *reinterpret_cast<f4*>(v + e) = vv;
      if (COPY == 1 || COPY == 3) {
        u2 pk;
        pk.x = rv_pack_bf16x2(r.x, r.y);
        pk.y = rv_pack_bf16x2(r.z, r.w);
        *reinterpret_cast<u2*>(reinterpret_cast<uint16_t*>(copy) + (COPY == 3 ? rv_ver_at(map, base, e) : e)) = pk;
      } else if (COPY == 2) {
        *reinterpret_cast<f4*>(reinterpret_cast<float*>(copy) + e) = r;
      }
    }
    return;
  }
  for (int k = threadIdx.x; k < kTile; k += kThreads) {
    const uint64_t i = base + k;
    if (i >= n) break;
    float vi = v[i];
    const float r = step(w[i], ADD ? acc[i] + g[i] : g[i], vi);
    w[i] = r; v[i] = vi;
    if (COPY == 1 || COPY == 3) reinterpret_cast<uint16_t*>(copy)[COPY == 3 ? rv_ver_at(map, base, i) : i] = rv_f32_to_bf16(r);
    if (COPY == 2) reinterpret_cast<float*>(copy)[i] = r;
  }
}

// Gradient accumulation (section 4.2 of the paper: the gradients of several microbatches are
// summed before one update): acc <- g for the first microbatch of a group, acc <- acc + g
// after.  12 B/param (8 for the first).
template <bool FIRST>
__global__ __launch_bounds__(kThreads) void accumulate_kernel(float* __restrict__ acc, const float* __restrict__ g,
                                                              uint64_t n, int aligned) {
  const uint64_t base = (uint64_t)blockIdx.x * kTile;
  if (aligned && base + kTile <= n) {
#pragma unroll
    for (int u = 0; u < kVec; ++u) {
      const uint64_t e = base + (uint64_t)(u * kThreads + threadIdx.x) * 4;
      f4 gv = *reinterpret_cast<const f4*>(g + e);
      if (!FIRST) gv += *reinterpret_cast<const f4*>(acc + e);
      *reinterpret_cast<f4*>(acc + e) = gv;
    }
    return;
  }
  for (int k = threadIdx.x; k < kTile; k += kThreads) {
    const uint64_t i = base + k;
    if (i >= n) break;
    acc[i] = FIRST ? g[i] : acc[i] + g[i];
  }
}

// set_params: a flat vector becomes the master and, converted, a weight version, in one pass
template <int COPY>
__global__ __launch_bounds__(kThreads) void set_kernel(const float* w, uint64_t n, float* master, void* __restrict__ copy, rv_ver_map map) {
  const uint64_t base = (uint64_t)(COPY == 3 ? rv_ver_tile(blockIdx.x, gridDim.x) : blockIdx.x) * (kThreads * 4);
  const uint64_t e = base + threadIdx.x * 4;
  if (e + 4 <= n) {
    typedef f4 f4_u __attribute__((aligned(4)));           // the caller's vector may start anywhere
    const f4 v = *reinterpret_cast<const f4_u*>(w + e);
    *reinterpret_cast<f4*>(master + e) = v;
    if (COPY == 3) {
      u2 pk;
      pk.x = rv_pack_bf16x2(v.x, v.y); pk.y = rv_pack_bf16x2(v.z, v.w);
      *reinterpret_cast<u2*>(reinterpret_cast<uint16_t*>(copy) + rv_ver_at(map, base, e)) = pk;
    } else {
      *reinterpret_cast<f4*>(reinterpret_cast<float*>(copy) + e) = v;
    }
    return;
  }
  for (uint64_t i = e; i < n; ++i) {
    const float v = w[i];
    master[i] = v;
    if (COPY == 3) reinterpret_cast<uint16_t*>(copy)[rv_ver_at(map, base, i)] = rv_f32_to_bf16(v);
    else reinterpret_cast<float*>(copy)[i] = v;
  }
}

// One launch for 64 version slots: with a 16-byte hipMemsetAsync each, creating an MLP stage of tau = 4 / 100 took
// 79 / 408 us instead of 62 / 170 (60 / 159 without the pads).
constexpr int kPadSlots = 64;
// dst <- src, fp32, both at 16 bytes: what the stage hands out (parameters, gradient).  201 MB of parameters 93 us with the
// runtime's copy, 66 us (6.1 TB/s) here; 5.5 MB 4.4 us with either, so the smaller vectors stay with the runtime's.
constexpr int kCopyVec = 2;
constexpr size_t kCopyFrom = 32u << 20;   // bytes
__global__ __launch_bounds__(kThreads) void copy_kernel(float* __restrict__ dst, const float* __restrict__ src, uint64_t n) {
  const uint64_t base = (uint64_t)blockIdx.x * (kThreads * kCopyVec * 4) + threadIdx.x * 4;
  f4 v[kCopyVec];
#pragma unroll
  for (int u = 0; u < kCopyVec; ++u)
    if (base + u * kThreads * 4 + 4 <= n) v[u] = __builtin_nontemporal_load(reinterpret_cast<const f4*>(src + base + u * kThreads * 4));
#pragma unroll
  for (int u = 0; u < kCopyVec; ++u) {
    const uint64_t e = base + u * kThreads * 4;
    if (e + 4 <= n) __builtin_nontemporal_store(v[u], reinterpret_cast<f4*>(dst + e));
    else for (uint64_t i = e; i < n; ++i) dst[i] = src[i];
  }
}

struct PadSlots { uint32_t* p[kPadSlots]; };
__global__ __launch_bounds__(kPadSlots * RV_VER_PAD / 4) void clear_pads_kernel(PadSlots a, int n) {
  const int slot = threadIdx.x / (RV_VER_PAD / 4);
  if (slot < n) a.p[slot][threadIdx.x % (RV_VER_PAD / 4)] = 0;
}

}  // namespace

rv_status rv_launch_update(float* w, const float* g, size_t n, float eta, void* copy, int copy_kind,
                           hipStream_t st, const rv_ver_map& map, const float* acc) {
  if (n == 0) return RV_OK;
  int aligned = ((((uintptr_t)w) | ((uintptr_t)g) | ((uintptr_t)acc)) & 15) == 0;
  if (copy && (((uintptr_t)copy) & 15)) aligned = 0;
  const int kind = copy ? copy_kind : 0;
  if (acc && kind < 2) return RV_E_INVAL;      // (only a stage has one)
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)((n + kTile - 1) / kTile)), dim3(kThreads), 0, st, w, g, n, eta, kind ? copy : nullptr, aligned,
                       map, acc);
    return rv_launch_status();
  };
  if (acc) return kind == 3 ? go(update_kernel<3, true>) : go(update_kernel<2, true>);
  return kind == 0 ? go(update_kernel<0, false>) : kind == 1 ? go(update_kernel<1, false>)
         : kind == 3 ? go(update_kernel<3, false>) : go(update_kernel<2, false>);
}

rv_status rv_launch_update_momentum(float* w, const float* g, float* v, size_t n, float eta, float mu, float wd,
                                    void* copy, int copy_kind, hipStream_t st, const rv_ver_map& map, const float* acc) {
  if (n == 0) return RV_OK;
  int aligned = ((((uintptr_t)w) | ((uintptr_t)g) | ((uintptr_t)v) | ((uintptr_t)acc)) & 15) == 0;
  if (copy && (((uintptr_t)copy) & 15)) aligned = 0;
  const int kind = copy ? copy_kind : 0;
  if (acc && kind < 2) return RV_E_INVAL;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)((n + kTile - 1) / kTile)), dim3(kThreads), 0, st, w, g, v, n, eta, mu, wd,
                       kind ? copy : nullptr, aligned, map, acc);
    return rv_launch_status();
  };
  if (acc) return kind == 3 ? go(update_momentum_kernel<3, true>) : go(update_momentum_kernel<2, true>);
  return kind == 0 ? go(update_momentum_kernel<0, false>) : kind == 1 ? go(update_momentum_kernel<1, false>)
         : kind == 3 ? go(update_momentum_kernel<3, false>) : go(update_momentum_kernel<2, false>);
}

rv_status rv_launch_accumulate(float* acc, const float* g, size_t n, bool first, hipStream_t st) {
  if (n == 0) return RV_OK;
  const int aligned = ((((uintptr_t)acc) | ((uintptr_t)g)) & 15) == 0;
  const unsigned blocks = (unsigned)((n + kTile - 1) / kTile);
  if (first) hipLaunchKernelGGL(accumulate_kernel<true>, dim3(blocks), dim3(kThreads), 0, st, acc, g, n, aligned);
  else hipLaunchKernelGGL(accumulate_kernel<false>, dim3(blocks), dim3(kThreads), 0, st, acc, g, n, aligned);
  return rv_launch_status();
}

rv_status rv_launch_clear_pads(char* const* ver, int n, size_t at, hipStream_t st) {
  for (int k = 0; k < n; k += kPadSlots) {
    PadSlots a = {};
    const int m = n - k < kPadSlots ? n - k : kPadSlots;
    for (int i = 0; i < m; ++i) a.p[i] = reinterpret_cast<uint32_t*>(ver[k + i] + at);
    hipLaunchKernelGGL(clear_pads_kernel, dim3(1), dim3(kPadSlots * RV_VER_PAD / 4), 0, st, a, m);
  }
  return rv_launch_status();
}

rv_status rv_launch_copy(float* dst, const float* src, size_t n, hipStream_t st) {
  if (n == 0) return RV_OK;
  if (n * 4 < kCopyFrom || ((((uintptr_t)dst) | ((uintptr_t)src)) & 15)) {
    RV_HIP_TRY(hipMemcpyAsync(dst, src, n * 4, hipMemcpyDeviceToDevice, st));
    return RV_OK;
  }
  const uint64_t tile = (uint64_t)kThreads * kCopyVec * 4;
  hipLaunchKernelGGL(copy_kernel, dim3((unsigned)((n + tile - 1) / tile)), dim3(kThreads), 0, st, dst, src, (uint64_t)n);
  return rv_launch_status();
}

rv_status rv_launch_set(const float* w, size_t n, float* master, void* copy, int copy_kind, hipStream_t st, const rv_ver_map& map) {
  if (n == 0) return RV_OK;
  const unsigned blocks = (unsigned)((n + kThreads * 4 - 1) / (kThreads * 4));
  if (copy_kind == 3)
    hipLaunchKernelGGL(set_kernel<3>, dim3(blocks), dim3(kThreads), 0, st, w, n, master, copy, map);
  else
    hipLaunchKernelGGL(set_kernel<2>, dim3(blocks), dim3(kThreads), 0, st, w, n, master, copy, map);
  return rv_launch_status();
}

extern "C" rv_status rv_block_update(float* w, const float* g, size_t n, float eta, void* bf16_out,
                                     void* stream) {
  if (w == nullptr || g == nullptr || n == 0) return RV_E_INVAL;
  if ((const float*)w == g) return RV_E_INVAL;
  return rv_launch_update(w, g, n, eta, bf16_out, bf16_out ? 1 : 0, (hipStream_t)stream);
}

extern "C" rv_status rv_block_update_momentum(float* w, const float* g, float* v, size_t n, float eta,
                                              float momentum, float weight_decay, void* bf16_out, void* stream) {
  if (w == nullptr || g == nullptr || v == nullptr || n == 0) return RV_E_INVAL;
  if ((const float*)w == g || (const float*)v == g || w == v) return RV_E_INVAL;
  if (!(momentum >= 0.f) || !(weight_decay >= 0.f)) return RV_E_INVAL;
  return rv_launch_update_momentum(w, g, v, n, eta, momentum, weight_decay, bf16_out, bf16_out ? 1 : 0,
                                   (hipStream_t)stream);
}
