// HIP kernels for gfx950 (CDNA4) besides the exterior contractions (hec.hpp,
// hec_*.hip): fixed-order split-K reduction, the FP64 root trace, the FP64
// cross-diagram sum, the layout conversion of uploaded leaves, and every
// launcher.  Tensor layout and descriptors: desc.hpp.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <mutex>

#include "desc.hpp"
#include "hec.hpp"
#include "kernels.hpp"

namespace cdag {

// ------------------------------------------------------------------ split-K reduce
// Bound by memory (it reads splits x the output once).  A thread takes 16 bytes
// of the output at a time, four splits' loads in flight: with one element per
// thread the reduction of FP32 K33s at N = 64 (16 splits, 0.92 GB) took 0.33 ms
// (3.5 TB/s), this form 0.21 (5.7 TB/s).
template <typename T>
__global__ void __launch_bounds__(256) splitk_reduce(char* __restrict__ arena, const RedDesc* __restrict__ descs,
                                                     Span n_desc, int64_t n_items) {
  constexpr int W = 16 / (int)sizeof(T), PER = kRedBlock / 256;   // elements per vector, per thread
  typedef T VT __attribute__((ext_vector_type(W)));
  typedef VT VU __attribute__((aligned(sizeof(T))));              // slices of odd length
  for (int64_t item = blockIdx.x; item < n_items; item += gridDim.x) {
    const RedDesc& r = *desc_of(descs, n_desc, item);
    const int64_t total = 2LL * r.nt * r.mn;
    const T* ws = reinterpret_cast<const T*>(arena + r.ws_off);
    T* out = reinterpret_cast<T*>(arena + r.c_off);
    const int splits = r.splits;
#pragma unroll
    for (int q = 0; q < PER / W; ++q) {
      const int64_t e = (item - r.item_begin) * kRedBlock + (int64_t)(q * 256 + (int)threadIdx.x) * W;
      if (e + W <= total) {
        double s[W];
#pragma unroll
        for (int x = 0; x < W; ++x) s[x] = 0.0;
#pragma unroll 4
        for (int k = 0; k < splits; ++k) {   // fixed order
          const VT v = *reinterpret_cast<const VU*>(ws + (int64_t)k * total + e);
#pragma unroll
          for (int x = 0; x < W; ++x) s[x] += (double)v[x];
        }
        VT v;
#pragma unroll
        for (int x = 0; x < W; ++x) v[x] = (T)s[x];
        *reinterpret_cast<VU*>(out + e) = v;
      } else {
        for (int64_t i = e; i < total; ++i) {
          double s = 0.0;
          for (int k = 0; k < splits; ++k) s += (double)ws[(int64_t)k * total + i];
          out[i] = (T)s;
        }
      }
    }
  }
}

// ------------------------------------------------------------------ root trace (FP64)
// The traces of one launch (device code and summation order: hec.hpp), in one
// of two layouts of the same order.  WG = false: one wave per (root, t), four
// per workgroup, for launches with many traces.  WG = true: one workgroup per
// (root, t), for launches with few traces (small waves), which one wave each
// would spread over few compute units with several rounds of loads per wave.
template <typename T, bool WG>
__global__ void __launch_bounds__(256, 3) hca_trace(char* __restrict__ arena, const HcaDesc* __restrict__ descs,
                                                    Span n_desc, int64_t n_items) {
  if constexpr (WG) {
    __shared__ double part[2][4];
    for (int64_t item = blockIdx.x; item < n_items; item += gridDim.x)
      trace_group<T, 4>(arena, descs, n_desc, item, true, (int)threadIdx.x, part);
  } else {
    const int wave = (int)threadIdx.x >> 6;
    for (int64_t base = (int64_t)blockIdx.x * 4; base < n_items; base += (int64_t)gridDim.x * 4) {
      const int64_t item = base + wave;
      if (item >= n_items) break;
      trace_wave<T, 4>(arena, descs, n_desc, item);
    }
  }
}

// ------------------------------------------------------------------ cross-diagram sum (FP64)
// The last kernel of an execute: one workgroup per (correlator, t), then
// workgroups that copy the correlators to the host.  Thread i sums the entries
// i, i + 256, ... in that order; the 256 partial sums are then added in a fixed
// tree (halves 128, 64, then 32 .. 1 within a wave).  The order is fixed, so
// the result does not change from run to run.
//
// host (may be nullptr): pinned memory laid out as [corr_bytes of
// correlators][sums] like the arena from corr_off; the kernel stores both
// there, so no copy follows it.
//
// Bound by the latency of an entry's two dependent loads (once per 256
// entries), or by the host link for many correlators.  With one workgroup per
// correlator walking over t it took 9.8 us (8 time slices, 6 graphs) and 53 us
// (32 slices, 2,000 graphs), and the copy that followed it 9 and 29 us with the
// gap before it; this form, the copy included, takes 2.3 and 22 us (1 MB at
// 45 GB/s).
__global__ void __launch_bounds__(256) xsum_kernel(char* __restrict__ arena, const XsumDesc* __restrict__ descs,
                                                   const XsumEntry* __restrict__ entries, Span n_desc, int64_t n_items,
                                                   int64_t corr_off, int64_t corr_bytes, char* __restrict__ host) {
  typedef double v2d __attribute__((ext_vector_type(2)));
  __shared__ double red[2][128];
  const int tid = threadIdx.x;
  for (int64_t item = blockIdx.x; item < n_items; item += gridDim.x) {
    const XsumDesc& x = descs[find_desc(&descs[0].item_begin, sizeof(XsumDesc) / 4, n_desc.n, item)];
    const int t = (int)(item - x.item_begin);
    double sr = 0.0, si = 0.0;
    for (int e = x.e_begin + tid; e < x.e_end; e += 256) {
      const double* C = reinterpret_cast<const double*>(arena + entries[e].root_off);
      const double cr = C[2 * t], ci = C[2 * t + 1];
      sr += entries[e].w_re * cr - entries[e].w_im * ci;
      si += entries[e].w_re * ci + entries[e].w_im * cr;
    }
    if (tid >= 128) {
      red[0][tid - 128] = sr;
      red[1][tid - 128] = si;
    }
    __syncthreads();
    if (tid < 128) {
      sr += red[0][tid];
      si += red[1][tid];
    }
    __syncthreads();
    if (tid >= 64 && tid < 128) {
      red[0][tid] = sr;
      red[1][tid] = si;
    }
    __syncthreads();
    if (tid < 64) {
      sr += red[0][tid + 64];
      si += red[1][tid + 64];
#pragma unroll
      for (int w = 32; w > 0; w >>= 1) {
        sr += __shfl_down(sr, w);
        si += __shfl_down(si, w);
      }
      if (tid == 0) {
        const int64_t off = x.out_off + 16LL * t;
        *reinterpret_cast<v2d*>(arena + off) = v2d{sr, si};
        if (host) *reinterpret_cast<v2d*>(host + (off - corr_off)) = v2d{sr, si};
      }
    }
    __syncthreads();
  }
  if (host == nullptr) return;
  // the workgroups past the sums' (every one of a grid of less) copy the correlators
  const int64_t first = n_items < (int64_t)gridDim.x ? n_items : 0;
  const int64_t step = ((int64_t)gridDim.x - first) * 256, b = (int64_t)blockIdx.x - first;
  if (b < 0) return;
  const v2d* src = reinterpret_cast<const v2d*>(arena + corr_off);
  for (int64_t i = b * 256 + tid; i < corr_bytes / 16; i += step) reinterpret_cast<v2d*>(host)[i] = src[i];
}

// ------------------------------------------------------------------ layout conversion
// Interleaved complex [nt][e] (S: double or float) -> the device layout
// [nt][2][e] in T, converted on the device (the path that copies host data
// straight into device memory, without a pinned staging copy in device layout).
template <typename S, typename T>
__global__ void __launch_bounds__(256) to_planar(const S* __restrict__ src, T* __restrict__ dst, int64_t nt,
                                                 int64_t e) {
  const int64_t total = nt * e;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    const int64_t t = i / e, x = i - t * e;
    const S re = src[2 * i], im = src[2 * i + 1];
    dst[2 * t * e + x] = (T)re;
    dst[(2 * t + 1) * e + x] = (T)im;
  }
}

// ------------------------------------------------------------------ host transfers
// The uploads, or the spills, of one plan step in one launch: workgroup b moves
// the chunk (mb.chunk bytes) that it holds of its move, between device memory
// and pinned host memory, every load of a thread ahead of its first store.
//
// A replayed graph runs its copies one after another, as copy kernels of 5 to 6
// us each for small tensors (16 leaf slices of 128 KiB: 100 us a pass); one
// launch keeps every tensor's reads in flight on the link at once (15 slices in
// 37 us, 53 GB/s).  Chunks of one load per thread for a small batch, which
// spreads it over more compute units (4 tensors of 32 KiB 8.6 -> 4.7 us), of four
// for a large one (the 15 slices above take 43 us in small chunks).
template <int Q>
__device__ __forceinline__ void move_chunk(const char* src, char* dst, int64_t left) {
  typedef double v2d __attribute__((ext_vector_type(2)));
  const int tid = threadIdx.x;
  v2d r[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (16 * (tid + 256 * q) < left) r[q] = reinterpret_cast<const v2d*>(src)[tid + 256 * q];
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (16 * (tid + 256 * q) < left) reinterpret_cast<v2d*>(dst)[tid + 256 * q] = r[q];
}

__global__ void __launch_bounds__(256) move_kernel(const MoveBatch mb) {
  int i = 0;
  while (i + 1 < mb.n && mb.begin[i + 1] <= (int)blockIdx.x) ++i;
  const Move m = mb.move[i];
  const int64_t off = (int64_t)((int)blockIdx.x - mb.begin[i]) * mb.chunk;
  const int64_t left = m.bytes - off < mb.chunk ? m.bytes - off : mb.chunk;
  const char* src = static_cast<const char*>(m.src) + off;
  char* dst = static_cast<char*>(m.dst) + off;
  if ((((uintptr_t)src | (uintptr_t)dst | (uint64_t)left) & 15) == 0) {
    if (mb.chunk <= kMoveChunk) move_chunk<1>(src, dst, left);
    else move_chunk<4>(src, dst, left);
  } else {   // slices of odd length: whole complex64 values (8 bytes)
    for (int64_t e = threadIdx.x; e < left / 8; e += 256)
      reinterpret_cast<double*>(dst)[e] = reinterpret_cast<const double*>(src)[e];
  }
}

// ------------------------------------------------------------------ launchers
namespace {
// Persistent launches: at most as many workgroups as can be resident at once
// (compute units x occupancy of the kernel); each loops over work items with
// a grid stride.  The occupancy query is made once per kernel.
unsigned persistent_grid(const void* kernel, int block, int64_t items) {
  static std::mutex mu;
  static std::map<std::pair<const void*, int>, int> cache;   // (kernel, device) -> resident workgroups
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) dev = -1;
  const auto key = std::make_pair(kernel, dev);
  int resident;
  {
    std::lock_guard<std::mutex> lock(mu);
    auto it = cache.find(key);
    if (it == cache.end()) {
      int cus = 0, per_cu = 0;
      if (dev < 0 || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
          hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, 0) != hipSuccess || per_cu < 1)
        resident = 1 << 16;
      else
        resident = cus * per_cu;
      cache.emplace(key, resident);
    } else {
      resident = it->second;
    }
  }
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(items, resident));
}
// traces per launch from which one wave per trace still fills 256 compute
// units with a workgroup of four waves each
constexpr int64_t kHcaWaveItems = 4 * 256;
unsigned grid_for(int64_t items) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>(items, kMaxGrid)); }

void set_args(KernelCall& k, char* arena, const void* desc, int n_desc, int64_t n_items) {
  k.arena = arena;
  k.desc = desc;
  k.n_desc = span(n_desc, n_items);
  k.n_items = n_items;
}
}  // namespace

void KernelCall::bind() {
  args[0] = &arena;
  args[1] = &desc;
  if (entries != nullptr) {
    args[2] = &entries;
    args[3] = &n_desc;
    args[4] = &n_items;
    args[5] = &corr_off;
    args[6] = &corr_bytes;
    args[7] = &host;
    return;
  }
  args[2] = &n_desc;
  args[3] = &n_items;
  args[4] = &tdesc;     // exterior contractions only
  args[5] = &n_tdesc;
  args[6] = &n_titems;
}

hipError_t launch(KernelCall& k, hipStream_t s) {
  k.bind();
  return hipLaunchKernel(k.fn, dim3(k.grid), dim3(k.block), k.args, 0, s);
}

// variant: see desc.hpp (grid 0: persistent, 1: one workgroup per work item).
// interior: every contraction of the launch passes hec_interior for the
// variant's tile and the precision's k-step (the host checks it).
hipError_t hec_call(int prec, int variant, bool interior, char* arena, int64_t desc_off, int n_desc, int64_t n_items,
                    KernelCall* k, int64_t tdesc_off, int n_tdesc, int64_t n_titems) {
  const bool traces = n_titems > 0;
  if (variant == kGenVariantId) {        // contractions over any index pairs: FP64 and FP32
    if (prec > 1 || traces) return hipErrorInvalidValue;
    k->fn = prec == 0 ? hec_general_f64() : hec_general_f32();
    k->block = kTileShapes[1].nth;
    k->grid = grid_for(n_items);
    set_args(*k, arena, arena + desc_off, n_desc, n_items);
    return hipSuccess;
  }
  if (variant < 0 || variant >= kAllVariants || prec < 0 || prec > 3) return hipErrorInvalidValue;
  const int tile = variant_tile(variant), stages = variant_stages(variant);
  const bool persistent = variant_grid(variant) == 0;
  const void* fn = prec == 0   ? hec_kernel_f64(tile, stages, persistent, interior, traces)
                   : prec == 1 ? hec_kernel_f32(tile, stages, persistent, interior, traces)
                   : prec == 2 ? hec_kernel_bf16x2(tile, stages, persistent, interior, traces)
                               : hec_kernel_bf16x3(tile, stages, persistent, interior, traces);
  if (fn == nullptr) return hipErrorInvalidValue;
  k->fn = fn;
  k->block = kTileShapes[tile].nth;
  set_args(*k, arena, arena + desc_off, n_desc, n_items);
  if (traces) {
    // one workgroup per contraction work item, then the trace workgroups
    const int64_t blocks = n_items + trace_blocks(k->block, n_titems);
    if (blocks > kMaxGrid) return hipErrorInvalidValue;
    k->grid = (unsigned)blocks;
    k->tdesc = arena + tdesc_off;
    k->n_tdesc = span(n_tdesc, n_titems);
    k->n_titems = n_titems;
  } else {
    k->grid = persistent ? persistent_grid(fn, k->block, n_items) : grid_for(n_items);
    k->tdesc = nullptr;
    k->n_tdesc = span(0, 0);
    k->n_titems = 0;
  }
  return hipSuccess;
}

hipError_t reduce_call(int prec, char* arena, int64_t desc_off, int n_desc, int64_t n_items, KernelCall* k) {
  k->fn = prec == 0 ? reinterpret_cast<const void*>(&splitk_reduce<double>)
                    : reinterpret_cast<const void*>(&splitk_reduce<float>);
  k->grid = grid_for(n_items);
  k->block = 256;
  set_args(*k, arena, arena + desc_off, n_desc, n_items);
  return hipSuccess;
}

// The trace layout by launch size: one wave per trace while that still gives
// every compute unit a workgroup (256 CUs), else one workgroup per trace.
hipError_t hca_call(int prec, char* arena, int64_t desc_off, int n_desc, int64_t n_items, KernelCall* k) {
  const bool wg = n_items < kHcaWaveItems;
  k->fn = prec == 0 ? (wg ? reinterpret_cast<const void*>(&hca_trace<double, true>)
                          : reinterpret_cast<const void*>(&hca_trace<double, false>))
                    : (wg ? reinterpret_cast<const void*>(&hca_trace<float, true>)
                          : reinterpret_cast<const void*>(&hca_trace<float, false>));
  k->grid = grid_for(wg ? n_items : (n_items + 3) / 4);
  k->block = 256;
  set_args(*k, arena, arena + desc_off, n_desc, n_items);
  return hipSuccess;
}

hipError_t xsum_call(char* arena, int64_t desc_off, int64_t entries_off, int n_desc, int64_t n_items,
                     int64_t corr_off, int64_t corr_bytes, char* host, KernelCall* k) {
  k->fn = reinterpret_cast<const void*>(&xsum_kernel);
  // 16 KB of correlators per copying workgroup, at most one per compute unit
  const int64_t copiers = host ? std::min<int64_t>(256, (corr_bytes + 16383) / 16384) : 0;
  k->grid = grid_for(n_items + copiers);
  k->block = 256;
  set_args(*k, arena, arena + desc_off, n_desc, n_items);
  k->entries = arena + entries_off;
  k->corr_off = corr_off;
  k->corr_bytes = corr_bytes;
  k->host = host;
  return hipSuccess;
}

hipError_t launch_hec(int prec, int variant, bool interior, char* arena, int64_t desc_off, int n_desc,
                      int64_t n_items, hipStream_t s) {
  KernelCall k;
  hipError_t e = hec_call(prec, variant, interior, arena, desc_off, n_desc, n_items, &k);
  return e != hipSuccess ? e : launch(k, s);
}

hipError_t launch_reduce(int prec, char* arena, int64_t desc_off, int n_desc, int64_t n_items, hipStream_t s) {
  KernelCall k;
  const hipError_t e = reduce_call(prec, arena, desc_off, n_desc, n_items, &k);
  return e != hipSuccess ? e : launch(k, s);
}

hipError_t launch_hca(int prec, char* arena, int64_t desc_off, int n_desc, int64_t n_items, hipStream_t s) {
  KernelCall k;
  const hipError_t e = hca_call(prec, arena, desc_off, n_desc, n_items, &k);
  return e != hipSuccess ? e : launch(k, s);
}

int make_moves(const Move* moves, int n, MoveBatch* mb) {
  int64_t bytes = 0, chunks = 0;
  for (int i = 0; i < n && i < kMaxMoves; ++i) bytes += moves[i].bytes;
  mb->chunk = bytes <= kMoveSmall ? kMoveChunk : 4 * kMoveChunk;
  mb->n = 0;
  while (mb->n < n && mb->n < kMaxMoves) {
    const int64_t more = (moves[mb->n].bytes + mb->chunk - 1) / mb->chunk;
    if (mb->n > 0 && chunks + more > kMaxGrid) break;
    if (chunks + more > INT32_MAX / 256) return -1;
    mb->move[mb->n] = moves[mb->n];
    mb->begin[mb->n++] = (int32_t)chunks;
    chunks += more;
  }
  mb->begin[mb->n] = (int32_t)chunks;
  return mb->n;
}

const void* move_fn() { return reinterpret_cast<const void*>(&move_kernel); }

hipError_t launch_moves(const Move* moves, int n, hipStream_t s) {
  for (int done = 0; done < n;) {
    MoveBatch mb;
    const int k = make_moves(moves + done, n - done, &mb);
    if (k <= 0) return hipErrorInvalidValue;
    void* args[1] = {&mb};
    if (mb.begin[k] > 0) {
      const hipError_t e = hipLaunchKernel(move_fn(), dim3((unsigned)mb.begin[k]), dim3(256), args, 0, s);
      if (e != hipSuccess) return e;
    }
    done += k;
  }
  return hipSuccess;
}

hipError_t launch_to_planar(bool src_double, bool dst_double, const void* src, void* dst, int64_t nt, int64_t e,
                           hipStream_t s) {
  const dim3 grid(grid_for((nt * e + 255) / 256)), block(256);
  if (src_double && dst_double)
    hipLaunchKernelGGL((to_planar<double, double>), grid, block, 0, s, (const double*)src, (double*)dst, nt, e);
  else if (src_double)
    hipLaunchKernelGGL((to_planar<double, float>), grid, block, 0, s, (const double*)src, (float*)dst, nt, e);
  else if (dst_double)
    hipLaunchKernelGGL((to_planar<float, double>), grid, block, 0, s, (const float*)src, (double*)dst, nt, e);
  else
    hipLaunchKernelGGL((to_planar<float, float>), grid, block, 0, s, (const float*)src, (float*)dst, nt, e);
  return hipGetLastError();
}

}  // namespace cdag
