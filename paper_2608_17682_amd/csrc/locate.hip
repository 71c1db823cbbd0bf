// The cell containing each ray origin: its nearest site (Sec. 3.1, the single
// nearest-neighbour query that starts the walk).  Distances are compared in
// FP64 from the FP32 inputs, ties going to the smallest index.
//
// Two exact strategies:
//  * brute force (few origins, e.g. one per pinhole view): a grid of
//    (chunk, origin) workgroups each reduce a chunk of sites, a second pass
//    reduces the chunks;
//  * greedy walk over the Delaunay adjacency from a hint (many origins, e.g.
//    thin-lens samples): move to the closest neighbour while one is closer.
//    Exact because a site that is not the nearest to x always has a Delaunay
//    neighbour closer to x; with (distance, index) ordered lexicographically
//    the walk strictly descends, so it ends after at most N moves.
#include <hip/hip_runtime.h>

#include "host_common.hpp"
#include "locate_impl.hpp"
#include "voro_device.hpp"
#include "walk_impl.hpp"

namespace voro {

struct BestD {
  double d2;
  int idx;
  int pad;
};

__device__ __forceinline__ bool better(double da, int ia, double db, int ib) {
  return (da < db) || (da == db && (unsigned)ia < (unsigned)ib);
}

__device__ __forceinline__ void wave_best(double& bd, int& bi) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    const double od = __shfl_xor(bd, m);
    const int oi = __shfl_xor(bi, m);
    if (better(od, oi, bd, bi)) {
      bd = od;
      bi = oi;
    }
  }
}

// The workgroup's nearest site to (ox, oy, oz) in its chunk; valid in thread 0.
// wide: four sites a thread and turn, so that their loads overlap.
__device__ __forceinline__ BestD block_nearest(const float* __restrict__ sites, int n, int chunk,
                                               int chunks, bool wide, double ox, double oy,
                                               double oz) {
  const long per = ((long)n + chunks - 1) / chunks;
  const long lo = (long)chunk * per;
  const unsigned len = (unsigned)max(0l, min((long)n, lo + per) - lo);
  const float* __restrict__ p = sites + 3 * lo;
  const unsigned step = blockDim.x;
  constexpr int kNone = 0x7fffffff;
  double bd = __builtin_huge_val();
  int bi = kNone;
  auto take = [&](unsigned i, float x, float y, float z) {
    const double dx = (double)x - ox;
    const double dy = (double)y - oy;
    const double dz = (double)z - oz;
    const double d2 = __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz));
    if (better(d2, (int)i, bd, bi)) {
      bd = d2;
      bi = (int)i;
    }
  };
  unsigned i = threadIdx.x;   // (unsigned: a turn past a single chunk of 2^31 - 1 sites)
  for (; wide && i + 3 * step < len; i += 4 * step) {
    float x[4], y[4], z[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float* q = p + 3 * (size_t)(i + k * step);
      x[k] = q[0];
      y[k] = q[1];
      z[k] = q[2];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) take(i + k * step, x[k], y[k], z[k]);
  }
  for (; i < len; i += step) {
    const float* q = p + 3 * (size_t)i;
    take(i, q[0], q[1], q[2]);
  }
  wave_best(bd, bi);
  __shared__ double sd[16];
  __shared__ int si[16];
  const int wave = threadIdx.x >> 6;
  const int nw = blockDim.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    sd[wave] = bd;
    si[wave] = bi;
  }
  __syncthreads();
  if (threadIdx.x == 0)
    for (int k = 1; k < nw; ++k)
      if (better(sd[k], si[k], bd, bi)) {
        bd = sd[k];
        bi = si[k];
      }
  return BestD{bd, bi == kNone ? kNone : (int)(lo + bi), 0};
}

// origins: device memory, or null for the camera centres in c
__global__ void __launch_bounds__(1024) k_locate_brute(const float* __restrict__ sites, int n,
                                                      const float* __restrict__ origins,
                                                      ViewCenters c, BestD* __restrict__ partial,
                                                      int chunks, bool wide) {
  const int u = blockIdx.y;
  const float ox = origins ? origins[3 * (size_t)u] : c.c[3 * u];
  const float oy = origins ? origins[3 * (size_t)u + 1] : c.c[3 * u + 1];
  const float oz = origins ? origins[3 * (size_t)u + 2] : c.c[3 * u + 2];
  const BestD r = block_nearest(sites, n, blockIdx.x, chunks, wide, ox, oy, oz);
  if (threadIdx.x == 0) partial[(size_t)u * chunks + blockIdx.x] = r;
}

// queue: a multi-view launch's tile-queue counters, zeroed here, or null
__global__ void __launch_bounds__(64) k_locate_final(const BestD* __restrict__ partial, int chunks,
                                                     unsigned* __restrict__ queue,
                                                     int32_t* __restrict__ out) {
  const int u = blockIdx.x;
  if (queue && u == 0 && threadIdx.x < kViewsQueues) queue[threadIdx.x] = 0u;
  double bd = __builtin_huge_val();
  int bi = 0x7fffffff;
  for (int c = threadIdx.x; c < chunks; c += 64) {
    const BestD r = partial[(size_t)u * chunks + c];
    if (better(r.d2, r.idx, bd, bi)) {
      bd = r.d2;
      bi = r.idx;
    }
  }
  wave_best(bd, bi);
  if (threadIdx.x == 0) out[u] = bi;
}

// The multi-view launch's start in one kernel: the cells of the camera centres
// (which travel as kernel arguments), and the tile-queue counters zeroed.
// Workgroup (chunk, view) leaves its chunk's nearest site in `partial`; the one
// that takes the last ticket reduces them and puts the ticket back to zero (as
// the walk behind this kernel does, so that no bad value outlives a call).
// Stores and loads of the partial results are device-scope atomics, as the
// workgroups run on XCDs with L2s of their own.  One launch instead of three:
// 100k-site frames spent 18 us on them, thumbnails of 512 sites 10 of 61 us.
// Each ticket takes the chip about 20 ns, one after the other: worth it up to
// kTicketBlocks workgroups (BruteShape).
__global__ void __launch_bounds__(1024) k_views_locate(const float* __restrict__ sites, int n,
                                                      ViewCenters c, BestD* partial, int chunks,
                                                      int V, unsigned* ticket, unsigned* queue,
                                                      int32_t* __restrict__ out) {
  const int u = blockIdx.y;
  const BestD r = block_nearest(sites, n, blockIdx.x, chunks, true, c.c[3 * u], c.c[3 * u + 1],
                                c.c[3 * u + 2]);
  __shared__ bool s_last;
  if (threadIdx.x == 0) {
    BestD* p = partial + (size_t)u * chunks + blockIdx.x;
    __hip_atomic_store(&p->d2, r.d2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&p->idx, r.idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) ==
             (unsigned)(chunks * V) - 1u;
  }
  __syncthreads();
  if (!s_last) return;
  if (threadIdx.x < kViewsQueues) queue[threadIdx.x] = 0u;
  if (threadIdx.x == 0) *ticket = 0u;
  for (int v = threadIdx.x >> 6; v < V; v += (int)(blockDim.x >> 6)) {
    double bd = __builtin_huge_val();
    int bi = 0x7fffffff;
    for (int k = threadIdx.x & 63; k < chunks; k += 64) {
      BestD* p = partial + (size_t)v * chunks + k;
      const double d = __hip_atomic_load(&p->d2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int i = __hip_atomic_load(&p->idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (better(d, i, bd, bi)) {
        bd = d;
        bi = i;
      }
    }
    wave_best(bd, bi);
    if ((threadIdx.x & 63) == 0) out[v] = bi;
  }
}

__global__ void __launch_bounds__(256) k_locate_walk(DevScene s, const float* __restrict__ origins,
                                                     const int32_t* __restrict__ hint, int U,
                                                     int32_t* __restrict__ out,
                                                     unsigned long long* stats) {
  const int u = blockIdx.x * blockDim.x + threadIdx.x;
  uint32_t capped = 0;
  if (u < U) {
    int h = hint ? hint[u] : 0;
    if (h < 0 || h >= s.n) h = 0;
    bool cap = false;
    out[u] = nearest_walk(s, origins[3 * (size_t)u], origins[3 * (size_t)u + 1],
                          origins[3 * (size_t)u + 2], h, &cap);
    capped = cap ? 1u : 0u;
  }
  if (stats) {
    const uint32_t c = wave_sum_u32(capped);
    if ((threadIdx.x & 63) == 0 && c) atomicAdd(&stats[VORO_STAT_LOCATE_CAP], (unsigned long long)c);
  }
}

// How the brute-force search of U origins over n sites is split.
//
// Chunks of 1,024 sites (four a thread) while that gives no more than four
// workgroups per CU; beyond, of 4,096, as starting and reducing a workgroup then
// costs more than its loads (64 origins, 300k sites: 33 us, 20 with 4,096).  More
// than eight chunks are a multiple of eight, so that the workgroups of a chunk
// run on one XCD and find it in that L2 (64 origins, 700k sites: 76 -> 40 us).
// Sites that the L2s together do not hold are read in narrow turns where eight
// origins or more share them (64 origins, 8M sites: 785 us in wide turns, 600).
// A multi-view launch of up to kTicketBlocks workgroups takes one kernel; the
// tickets of more take longer than the second kernel (16 views, 262k sites: 95
// us for the call with tickets, 23 without).  Chunks of more than 4,096 sites
// then get four times the threads (one origin, 4M sites: 18.7 -> 13.5 us).
constexpr int kTicketBlocks = 256;
constexpr int kSmallChunkBlocks = 1024;
constexpr int kCachedSites = 3 << 20;

struct BruteShape {
  int chunks, threads;
  bool ticket, wide;
  BruteShape(int n, int U) {
    auto of = [n](int per) {
      const int c = min(n / per + (n % per != 0), kLocateChunks);
      return c > 8 ? (c + 7) & ~7 : c;
    };
    chunks = of(1024);
    if (chunks * U > kSmallChunkBlocks) chunks = of(4096);
    ticket = chunks * U <= kTicketBlocks;
    threads = ticket && n > 4096 * kLocateChunks ? 1024 : 256;
    wide = n <= kCachedSites || U < 8;
  }
};

// Brute-force nearest sites of U <= kLocateBruteMax origins into out (device);
// partials: U * kLocateChunks * 16 bytes of device scratch.  origins null: the
// camera centres in c, with the launch's queue counters to be zeroed.
static voro_status launch_locate_brute(const voro_scene* scene, void* partials,
                                       const float* origins, const ViewCenters& c, int U,
                                       unsigned* queue, int32_t* out, hipStream_t st) {
  BestD* partial = reinterpret_cast<BestD*>(partials);
  const BruteShape b(scene->n_sites, U);
  hipLaunchKernelGGL(k_locate_brute, dim3(b.chunks, U), dim3(b.threads), 0, st, scene->sites,
                     scene->n_sites, origins, c, partial, b.chunks, b.wide);
  hipLaunchKernelGGL(k_locate_final, dim3(U), dim3(64), 0, st, partial, b.chunks, queue, out);
  return check_launch(origins ? "voro_locate_origins (brute force)"
                              : "views: cells of the camera centres");
}

// Cells of V camera centres into out (device), the queue counters zeroed;
// partials as above, ticket: a device word that is zero between launches.
voro_status launch_views_locate(const voro_scene* scene, void* partials, const ViewCenters& c,
                                int V, unsigned* ticket, unsigned* queue, int32_t* out,
                                hipStream_t st) {
  const BruteShape b(scene->n_sites, V);
  if (!b.ticket) return launch_locate_brute(scene, partials, nullptr, c, V, queue, out, st);
  hipLaunchKernelGGL(k_views_locate, dim3(b.chunks, V), dim3(b.threads), 0, st, scene->sites,
                     scene->n_sites, c, reinterpret_cast<BestD*>(partials), b.chunks, V, ticket,
                     queue, out);
  return check_launch("views: cells of the camera centres");
}

}  // namespace voro

using namespace voro;

extern "C" voro_status voro_locate_origins(const voro_scene* scene, const void* ws,
                                           size_t ws_bytes, const float* origins,
                                           const int32_t* hint, int32_t U, int32_t* cell_out,
                                           uint64_t* stats, void* stream) {
  voro_status st;
  if ((st = check_scene(scene)) != VORO_OK) return st;
  if ((st = check_ws(scene, ws, ws_bytes)) != VORO_OK) return st;
  if (U < 0) return fail(VORO_EINVAL, "U must be >= 0");
  if (U == 0) return VORO_OK;
  if (!origins || !cell_out) return fail(VORO_EINVAL, "origins and cell_out must not be NULL");
  if ((st = check_device()) != VORO_OK) return st;
  const hipStream_t s = (hipStream_t)stream;
  if (!hint && U <= kLocateBruteMax) {
    const WsLayout L = ws_layout(scene->n_sites, scene->n_edges);
    // the partials' region of the workspace is scratch (const only in the signature)
    return launch_locate_brute(scene, (char*)const_cast<void*>(ws) + L.locate, origins,
                               ViewCenters{}, U, nullptr, cell_out, s);
  }
  const DevScene d = dev_scene(scene, ws);
  hipLaunchKernelGGL(k_locate_walk, dim3((U + 255) / 256), dim3(256), 0, s, d, origins, hint, U,
                     cell_out, reinterpret_cast<unsigned long long*>(stats));
  return check_launch("voro_locate_origins (walk)");
}
