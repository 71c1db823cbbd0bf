// The per-ray walk, forward and adjoint, as device functions shared by the
// explicit-ray kernels and the persistent multi-view kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "voro.h"
#include "voro_device.hpp"

namespace voro {

struct WalkParams {
  float t_stop;
  float skip_w;
  float tie_window;
  int max_steps;
  int edge16;  // rank neighbours from the half-precision edge vectors
};

struct RayIn {
  float ox, oy, oz;
  float dx, dy, dz;
  float tmax;
  int start;
};

struct RayOut {
  float r, g, b, T;
  int k;
  float dist, dist_a, dist_w;  // distortion loss and its running totals (when asked for)
};

// saved forward totals and upstream gradient of one ray; with the
// distortion loss also its saved value and totals sum w sbar, sum w, and
// its upstream gradient
struct Upstream {
  float Cr, Cg, Cb, Tf;
  float gr, gg, gb, gT;
  float D, DA, DW, gD;
};

// Distortion loss (Sec. 5.3): s(t) = t / (1 + t) maps depth into [0, 1).
// Along a ray the intervals are ordered, so the pair sum runs on prefix
// sums: segment k adds 2 w_k (sbar_k W - A) + w_k^2 ds_k / 3, with W, A the
// sums of w and w sbar over the earlier segments.
__device__ __forceinline__ float dist_s(float t) { return t / (1.0f + t); }

// Gradient targets of the adjoint kernels.  Position and density gradients
// go to a per-cell accumulator in the workspace, dp in xyz and dsigma in w,
// so that one 16-byte slot (one cache line) takes all four terms of a cell;
// a second kernel then adds it into the caller's arrays.  Texel gradients go
// straight to the caller's array.
struct Grads {
  float4* cell;    // [N] workspace accumulator: (dp.x, dp.y, dp.z, dsigma)
  float* texels;   // [N,R,R,4], or [N,2,R,R,4] for the full appearance model
  int maps;        // texture maps per cell (1 or 2)
  unsigned rr_mul; // key / R^2 = umulhi(key, rr_mul) >> rr_shift (set_grad_layout)
  int rr_shift;
};

// Exact quotients by RR = R^2 (4 <= RR <= 256) of any key in [0, 2^31): with
// 2^L >= RR and m = ceil(2^(31+L) / RR), m RR - 2^(31+L) < RR <= 2^L, so the
// error key (m RR - 2^(31+L)) / (RR 2^(31+L)) stays below 1 / RR.
inline void set_grad_layout(Grads& g, const voro_scene* s) {
  g.maps = s->tex_maps == 2 ? 2 : 1;
  const unsigned RR = (unsigned)(s->tex_res * s->tex_res);
  int L = 0;
  while ((1u << L) < RR) ++L;
  g.rr_mul = (unsigned)(((1ull << (31 + L)) + RR - 1) / RR);
  g.rr_shift = L - 1;
}

struct Counters {
  uint32_t rays = 0, steps = 0, deg = 0, maxsteps = 0, nan = 0, bad = 0, redecide = 0,
           skipped = 0;
};

// wave-reduce the per-lane counters and add them to stats (one lane per
// counter and wave).  Every lane of the wave must call this.
__device__ __forceinline__ void flush_counters(Counters c, bool contribute, int lane,
                                               unsigned long long* stats) {
  if (!contribute) c = Counters();
  const uint32_t v[8] = {c.rays, c.steps, c.deg, c.maxsteps, c.nan, c.bad, c.redecide, c.skipped};
  const int idx[8] = {VORO_STAT_RAYS,  VORO_STAT_STEPS,     VORO_STAT_DEGREE_SUM,
                      VORO_STAT_MAX_STEPS, VORO_STAT_NAN, VORO_STAT_BAD_START,
                      VORO_STAT_FP64_REDECIDE, VORO_STAT_SKIPPED};
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const uint32_t s = wave_sum_u32(v[k]);
    if (lane == 0 && s) atomicAdd(&stats[idx[k]], (unsigned long long)s);
  }
}

// Per-workgroup stats in LDS (index = VORO_STAT_*) for the persistent
// kernels, whose waves walk one ray per lane group per tile: after each tile
// the lanes add their counters there (per-ray events as one ballot count per
// wave, per-step sums as LDS atomics), so no counter and no cross-lane
// shuffle address stays live across the tile loop.
constexpr int kWgStats = 10;

__device__ __forceinline__ void wg_stats_clear(unsigned long long* s) {
  if (threadIdx.x < kWgStats) s[threadIdx.x] = 0ull;
}

// Every lane of the wave must call this; a lane's counters cover at most one
// ray since they were zeroed.
__device__ __forceinline__ void tile_counters_to_lds(const Counters& c, bool contribute,
                                                     bool capped, int lane,
                                                     unsigned long long* s) {
  const unsigned n_rays = __popcll(__ballot(contribute && c.rays != 0u));
  const unsigned n_bad = __popcll(__ballot(contribute && c.bad != 0u));
  const unsigned n_max = __popcll(__ballot(contribute && c.maxsteps != 0u));
  const unsigned n_nan = __popcll(__ballot(contribute && c.nan != 0u));
  const unsigned n_cap = __popcll(__ballot(contribute && capped));
  if (contribute) {
    if (c.steps) atomicAdd(&s[VORO_STAT_STEPS], (unsigned long long)c.steps);
    if (c.deg) atomicAdd(&s[VORO_STAT_DEGREE_SUM], (unsigned long long)c.deg);
    if (c.redecide) atomicAdd(&s[VORO_STAT_FP64_REDECIDE], (unsigned long long)c.redecide);
    if (c.skipped) atomicAdd(&s[VORO_STAT_SKIPPED], (unsigned long long)c.skipped);
  }
  if (lane == 0) {
    if (n_rays) atomicAdd(&s[VORO_STAT_RAYS], (unsigned long long)n_rays);
    if (n_bad) atomicAdd(&s[VORO_STAT_BAD_START], (unsigned long long)n_bad);
    if (n_max) atomicAdd(&s[VORO_STAT_MAX_STEPS], (unsigned long long)n_max);
    if (n_nan) atomicAdd(&s[VORO_STAT_NAN], (unsigned long long)n_nan);
    if (n_cap) atomicAdd(&s[VORO_STAT_LOCATE_CAP], (unsigned long long)n_cap);
  }
}

// after a barrier that follows every wave's last tile.  The thread index is
// read afresh (empty asm) so that the slot address is not kept live, or
// spilled, from the kernel's start.
__device__ __forceinline__ void wg_stats_flush(const unsigned long long* s,
                                               unsigned long long* stats) {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  if (t < kWgStats && s[t]) atomicAdd(&stats[t], s[t]);
}

// One step of the walk: the exit of cell `cur` entered at t_in.  lrow: the
// cell's edge row staged in LDS by the wave (one lane per ray), or null to
// gather it from global memory.  E16: rank a gathered row from its
// half-precision copy first (a template switch, so the exact walk's kernels
// do not carry that code's registers); a staged row is searched in FP32
// either way, which reads it from LDS and costs less than the ranking.
template <int LPR, bool E16 = false>
__device__ __forceinline__ Exit step_exit(const DevScene& s, const WalkParams& w, const RayIn& r,
                                          const Cell& c, int cur, float t_in, int sub,
                                          const float4* lrow = nullptr, int llen = 0) {
  const float qx = fmaf(t_in, r.dx, r.ox) - c.px;
  const float qy = fmaf(t_in, r.dy, r.oy) - c.py;
  const float qz = fmaf(t_in, r.dz, r.oz) - c.pz;
  Best b;
  bool searched = false;
  if constexpr (LPR == 1 && E16) if (!lrow) {
    // Rank in half precision.  When the bounds leave a single face that can
    // hold the smallest FP32 crossing, and every other face lies beyond the
    // tie window from it, that face's FP32 record gives exactly what the
    // FP32 search would (its crossing, its id, no FP64 re-decision);
    // otherwise the row is searched in FP32.  Either way the walk is the
    // exact walk.
    const Rank16 h = rank16(s.edges16, c.off, c.deg, qx, qy, qz, r.dx, r.dy, r.dz);
    if (!h.unsure && h.k1 >= 0 && h.lo2 > h.hi) {
      const float4 E = s.edges[c.off + h.k1];
      const float u = cross_u(E, 2.0f * qx, 2.0f * qy, 2.0f * qz, r.dx, r.dy, r.dz);
      const float t1 = 0.5f * u;
      const float win = w.tie_window * fmaxf(1.0f, fabsf(t_in + t1));
      if (0.5f * h.lo2 - t1 > win) {
        b.t1 = t1;
        b.j1 = __float_as_int(E.w);
        b.t2 = 0.5f * h.lo2;
        searched = true;
      }
    } else if (!h.unsure && h.k1 < 0) {
      b.t1 = kInf;  // no face lies ahead
      b.j1 = -1;
      b.t2 = kInf;
      searched = true;
    }
  }
  if (searched) {
  } else if (LPR == 1 && lrow) {
    b = exit_search<1, true>(lrow, 0, llen, 0, qx, qy, qz, r.dx, r.dy, r.dz);
  } else {
    b = exit_search<LPR>(s.edges, c.off, c.deg, sub, qx, qy, qz, r.dx, r.dy, r.dz);
  }
  return decide_exit(b, s.cells, s.edges, cur, c.off, c.deg, t_in, w.tie_window, r.ox, r.oy, r.oz,
                     r.dx, r.dy, r.dz, qx, qy, qz);
}

// Full appearance model: the vector from the site to the point where the ray
// meets cell c (its entry point t_in; the clipped exit point in the start
// cell, step k = 0).  Zero when that point is the site itself.
__device__ __forceinline__ void hit_vector(const RayIn& r, const Cell& c, int k, float t_in,
                                           float exit_t, float& hx, float& hy, float& hz) {
  const float th = k > 0 ? t_in : fminf(exit_t, r.tmax);
  hx = fmaf(th, r.dx, r.ox) - c.px;
  hy = fmaf(th, r.dy, r.oy) - c.py;
  hz = fmaf(th, r.dz, r.oz) - c.pz;
}

// The taps a ray uses for every cell: the single map at +w (appearance 0)
// or the view map at -w (appearance 1; unused by appearance 2).
template <int APP>
__device__ __forceinline__ Taps ray_taps(const RayIn& r, int R) {
  return APP ? make_taps(-r.dx, -r.dy, -r.dz, R) : make_taps(r.dx, r.dy, r.dz, R);
}

// Forward walk state of one ray, so that a lane can hold a ray across the
// steps of a loop it shares with other rays (fwd_begin, fwd_step, fwd_end).
template <int APP>
struct FwdState {
  Taps tp;
  float Ysh[APP == 2 ? 16 : 1];
  float T, Cr, Cg, Cb, t_in;
  float dP, dQ, dW, dA, s0;
  int cur, k;
  // the record of cell cur, loaded as soon as cur is known (the exit
  // decision of the previous step), so that its latency overlaps that
  // step's texel lookup and compositing
  Cell nc;
};

// false: nothing to walk (tmax <= 0 or an invalid start cell)
template <int APP>
__device__ __forceinline__ bool fwd_begin(FwdState<APP>& st, const DevScene& s, const RayIn& r,
                                          Counters& cnt) {
  st.T = 1.0f;
  st.Cr = st.Cg = st.Cb = 0.0f;
  st.t_in = 0.0f;
  st.dP = st.dQ = st.dW = st.dA = st.s0 = 0.0f;
  st.k = 0;
  st.cur = r.start;
  if (!(r.tmax > 0.0f)) return false;
  if (r.start < 0 || r.start >= s.n) {
    cnt.bad++;
    return false;
  }
  cnt.rays++;
  st.nc = load_cell(s.cells, r.start);
  st.tp = ray_taps<APP>(r, s.res);
  if constexpr (APP == 2) sh3_basis(r.dx, r.dy, r.dz, st.Ysh);
  return true;
}

// Stored exits of a ray: step k's exit (parameter t by bit pattern, next
// cell) at p[k * stride] for k < cap, written by the forward and read by the
// adjoint instead of searching the step's edge row again (null: none).
using i32x2 = int __attribute__((ext_vector_type(2)));
struct ExitTrace {
  int2* p;
  unsigned stride;
  int cap;
};

// One visited cell (lrow: its edge row staged in LDS, or null); true when
// the ray has ended.
template <int LPR, int TEX, int APP, bool E16 = false>
__device__ __forceinline__ bool fwd_step(FwdState<APP>& st, const DevScene& s,
                                         const WalkParams& w, const RayIn& r, int sub,
                                         int32_t* rec, int max_record, Counters& cnt,
                                         bool dist_on, const float4* lrow = nullptr,
                                         int llen = 0, const ExitTrace& xt = {}) {
  const int cur = st.cur;
  const float t_in = st.t_in;
  const Cell c = st.nc;
  const Exit ex = step_exit<LPR, E16>(s, w, r, c, cur, t_in, sub, lrow, llen);
  if (xt.p && sub == 0 && st.k < xt.cap) {
    // streamed out (only the adjoint reads it back): a non-temporal store
    // leaves the caches to the walk's records
    const i32x2 e = {__float_as_int(ex.t), ex.next};
    __builtin_nontemporal_store(e, reinterpret_cast<i32x2*>(xt.p + (size_t)st.k * xt.stride));
  }
  if (ex.next >= 0) st.nc = load_cell(s.cells, ex.next);
  cnt.redecide += ex.redecided ? 1u : 0u;
  cnt.deg += (uint32_t)c.deg;
  const Segment sg = segment(ex.t, r.tmax, t_in, c.sigma);
  const float wk = st.T * sg.alpha;
  if (dist_on) {
    const float s1 = dist_s(fmaxf(t_in, fminf(ex.t, r.tmax)));
    const float sb = 0.5f * (st.s0 + s1);
    st.dP = fmaf(2.0f * wk, fmaf(sb, st.dW, -st.dA), st.dP);
    st.dQ = fmaf(wk * wk, s1 - st.s0, st.dQ);
    st.dW += wk;
    st.dA = fmaf(wk, sb, st.dA);
    st.s0 = s1;
  }
  if (wk >= w.skip_w) {
    float cr, cg, cb;
    if constexpr (APP == 0) {
      texel_rgb<TEX>(s.texels, cur, s.res, st.tp, cr, cg, cb);
    } else if constexpr (APP == 2) {
      sh3_colour<TEX>(s.texels, cur, st.Ysh, cr, cg, cb);
    } else {
      float hx, hy, hz;
      hit_vector(r, c, st.k, t_in, ex.t, hx, hy, hz);
      const bool on_site = hx == 0.0f && hy == 0.0f && hz == 0.0f;
      const Taps ts = make_taps(on_site ? r.dx : hx, on_site ? r.dy : hy,
                                on_site ? r.dz : hz, s.res);
      float lr, lg, lb;
      float4 ta, tb, te, tf;
      full_logits<TEX>(s.texels, cur, s.res, ts, st.tp, lr, lg, lb, ta, tb, te, tf);
      cr = sigmoid_f(lr);
      cg = sigmoid_f(lg);
      cb = sigmoid_f(lb);
    }
    st.Cr = fmaf(wk, cr, st.Cr);
    st.Cg = fmaf(wk, cg, st.Cg);
    st.Cb = fmaf(wk, cb, st.Cb);
  } else {
    cnt.skipped++;
  }
  st.T = st.T * sg.trans;
  if (rec && sub == 0 && st.k < max_record) rec[st.k] = cur;
  ++st.k;
  if (st.T < w.t_stop) return true;
  if (!(ex.t < r.tmax) || ex.next < 0) return true;
  if (st.k >= w.max_steps) {
    cnt.maxsteps++;
    return true;
  }
  st.t_in = fmaxf(t_in, fminf(ex.t, r.tmax));
  st.cur = ex.next;
  return false;
}

template <int APP>
__device__ __forceinline__ RayOut fwd_end(const FwdState<APP>& st, bool walked, Counters& cnt) {
  RayOut out;
  out.r = st.Cr;
  out.g = st.Cg;
  out.b = st.Cb;
  out.T = st.T;
  out.k = st.k;
  out.dist = fmaf(st.dQ, 1.0f / 3.0f, st.dP);
  out.dist_a = st.dA;
  out.dist_w = st.dW;
  if (walked) {
    cnt.steps += (uint32_t)st.k;
    if (st.T != st.T) cnt.nan++;
  }
  return out;
}

template <int LPR, int TEX, int APP, bool E16 = false>
__device__ __forceinline__ RayOut walk_forward(const DevScene& s, const WalkParams& w,
                                               const RayIn& r, int sub, int32_t* rec,
                                               int max_record, Counters& cnt,
                                               bool dist_on = false, const ExitTrace& xt = {}) {
  FwdState<APP> st;
  const bool walk = fwd_begin<APP>(st, s, r, cnt);
  if (walk)
    while (!fwd_step<LPR, TEX, APP, E16>(st, s, w, r, sub, rec, max_record, cnt, dist_on,
                                         nullptr, 0, xt)) {
    }
  return fwd_end<APP>(st, walk, cnt);
}

// Orders a wave's own LDS accesses for the compiler (the hardware keeps them in
// order).
__device__ __forceinline__ void lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
}

// Ranks the distinct keys of the lanes with `open`: each such lane writes its
// number to a bucket chosen by its key and reads back whose stayed; lanes whose
// key is that lane's have their leader, the others go on with another hash.
// Every round settles at least one key.  Every lane of the wave must call this;
// bucket: 256 bytes of the wave's LDS.  rank: of the lane's key (-1: not open),
// leads: the lane that stands for its key.  Stops, and returns a number above
// `most`, once there are more than `most` keys.
__device__ __forceinline__ int rank_keys(int key, bool open, unsigned char* bucket, int lane,
                                         int most, int& rank, bool& leads) {
  rank = -1;
  leads = false;
  int total = 0;
  unsigned mul = 2654435761u;
  do {
    const unsigned h = ((unsigned)key * mul) >> 24;
    int lead = lane;
    if (open) bucket[h] = (unsigned char)lane;
    lds_order();
    if (open) lead = bucket[h];
    lds_order();
    const bool won = open && __builtin_amdgcn_ds_bpermute(4 * lead, key) == key;
    const bool own = won && lead == lane;
    const unsigned long long m = __ballot(own);
    const int r = total + __popcll(m & ((1ull << lane) - 1ull));
    const int lr = __builtin_amdgcn_ds_bpermute(4 * lead, r);
    rank = won ? lr : rank;
    leads = leads || own;
    total += __popcll(m);
    open = open && !won;
    mul = (mul * 0x9E3779B1u + 0x7F4A7C15u) | 1u;
  } while (__any(open) && total <= most);
  return total;
}

// Wave-cooperative staging of edge rows (one lane per ray).  Rays of a
// coherent tile stand in few distinct cells at a time: 6 a step on the
// 100k-site scene, 16 on the 4M-site one (28 in one step of ten).  When the
// live lanes of the wave sit in at most kStageCells cells of at most
// 64 kStageLoads faces together, the wave reads those rows packed, 64 records
// a load, and keeps in its LDS slab, in their order, the faces that do not
// point away from every ray of the wave: about half.  If these fit, every live
// lane searches its row there; otherwise each lane gathers its own row from
// global memory.  The choice is per wave and step (mixing both within one step
// was slower: the two loops then run one after the other), and the exit search
// decides the same either way: a face left out is no exit of any of the rays.
//
// What bounds the walk: gathers, for scenes beyond the L2 (texture data path
// busy 0.98 of the 4M-site forward's cycles), and VALU issue, 14 instructions
// per face, for smaller ones (0.74 of a 100k-site frame's).  Staging serves
// both.  Rows copied one after the other (a trip to memory each, at most
// eight): 100k-site frame 577 us, two maps 1280x840 922, spherical harmonics
// 775, 4M-site forward + backward 58.4 ms, 311k thin-lens rays 465 us; packed
// and culled, eight cells: 541, 836, 713 us, 58.4 ms, 465 us; up to 32 cells
// ranked by rank_keys: 539, 829, 658 us, 54.5 ms, 431 us, each record's row
// found by bisection over the lanes; by counting the marks of the rows' starts
// (one trip to LDS instead of five): 495, 780, 597 us, 54.6 ms, 378 us.  (Ranks
// counted from the leaders' mask and the next row's start by a lane shift,
// without their LDS permutes, were slower again: 530, 820, 696 us, 59.4 ms.)
// Loading each texel ahead of the search (580 us a frame) or eight gathered records at a time
// (638 us) costs registers and with them a wave per SIMD.
constexpr int kStageCells = 32;      // two rows of 16 lanes (scan)
constexpr int kStageRecords = 256;   // in the slab
constexpr int kStageLoads = 8;       // of 64 records each
// a wave's slab, the rows' numbers (256 bytes) and its cone of directions (a
// search reads up to three records past its row: they may be these)
constexpr int kStageBytesPerWave = kStageRecords * 16 + 256 + 32;
constexpr int kStageMaxGap = 8;

// The directions of a wave's rays: centre c and a radius with |w - c| <= rho
// for every ray (wave-uniform).
// Held in the wave's LDS, as registers are short in the walk.
struct __align__(16) Cone {
  float cx, cy, cz, rho;
};

__device__ __forceinline__ float wave_uniform(float x) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}

__device__ __forceinline__ Cone wave_cone(const RayIn& r, bool has) {
  float x = has ? r.dx : 0.0f, y = has ? r.dy : 0.0f, z = has ? r.dz : 0.0f;
  float n = has ? 1.0f : 0.0f;
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    x += __shfl_xor(x, m);
    y += __shfl_xor(y, m);
    z += __shfl_xor(z, m);
    n += __shfl_xor(n, m);
  }
  const float inv = 1.0f / fmaxf(n, 1.0f);
  Cone k;
  k.cx = wave_uniform(x * inv);
  k.cy = wave_uniform(y * inv);
  k.cz = wave_uniform(z * inv);
  float d = has ? fabsf(r.dx - k.cx) + fabsf(r.dy - k.cy) + fabsf(r.dz - k.cz) : 0.0f;
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) d = fmaxf(d, __shfl_xor(d, m));
  // max |w - c|_inf <= |w - c|_1; the last term covers the FP32 roundings
  k.rho = wave_uniform(d * 1.0001f + 4e-6f);
  return k;
}

// Every lane of the wave must call this; alive: the lane's walk goes on, at
// cell cur with record c.  Returns the lane's staged row and its length, or
// null when the wave's rows were not staged (then staged = false on every
// lane).  Faces that no ray of the wave can leave through (m.w < 0 over the
// whole cone) are left out of the slab.
__device__ __forceinline__ const float4* stage_rows(const float4* __restrict__ edges, float4* slab,
                                                    bool alive, int cur, const Cell& c, int lane,
                                                    int& len, bool& staged) {
  staged = false;
  int* info = reinterpret_cast<int*>(slab + kStageRecords);
  int rank;
  bool leads;
  // (the slab's previous rows have been read by every lane: LDS operations of
  // one wave complete in order)
  const int n = rank_keys(cur, alive, reinterpret_cast<unsigned char*>(info), lane, kStageCells,
                          rank, leads);
  if (n > kStageCells) return nullptr;
  using i32x2 = int __attribute__((ext_vector_type(2)));
  i32x2* rows = reinterpret_cast<i32x2*>(info);
  // (no longer than what cannot be staged anyway, so that the sum of 32 lengths
  // stays an int: rows of a malformed adjacency can overlap)
  if (leads) rows[rank] = i32x2{c.off, min(c.deg, 64 * kStageLoads + 1)};
  lds_order();
  // lane m < n: row m, its records at [from, from + deg) of the packed rows
  i32x2 row = i32x2{0, 0};
  if (lane < n) row = rows[lane];
  int sum = row.y;
  sum += __builtin_amdgcn_update_dpp(0, sum, 0x111, 0xF, 0xF, false);  // row_shr:1
  sum += __builtin_amdgcn_update_dpp(0, sum, 0x112, 0xF, 0xF, false);
  sum += __builtin_amdgcn_update_dpp(0, sum, 0x114, 0xF, 0xF, false);
  sum += __builtin_amdgcn_update_dpp(0, sum, 0x118, 0xF, 0xF, false);
  const int low = __builtin_amdgcn_readlane(sum, 15);
  sum += lane >= 16 ? low : 0;
  const int used = __builtin_amdgcn_readlane(sum, 31);  // (rows past n have none)
  if (used > 64 * kStageLoads) return nullptr;
  const int from = sum - row.y;
  const int delta = row.x - from;
  // a byte per packed record, set where a row starts (a row without faces would
  // share its start: such cells are left to the gathered search)
  unsigned char* flag = reinterpret_cast<unsigned char*>(slab);
  if (__any(lane < n && row.y == 0)) return nullptr;
  reinterpret_cast<i32x2*>(flag)[lane] = i32x2{0, 0};
  lds_order();
  if (lane < n) flag[from] = 1;
  lds_order();
  const Cone cone = *reinterpret_cast<const Cone*>(info + 64);
  unsigned char f[kStageLoads];
#pragma unroll
  for (int i = 0; i < kStageLoads; ++i) f[i] = flag[64 * i + lane];
  lds_order();
  int start = 0, kept = 0, first = -1;
#pragma unroll
  for (int half = 0; half < kStageLoads; half += 4) {
    if (64 * half >= used) break;
    // four loads under way at a time
    float4 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (64 * (half + i) >= used) break;
      const int r = 64 * (half + i) + lane;
      // the last row that starts at or before r
      const unsigned long long starts = __ballot(f[half + i] != 0);
      const int m = first + __popcll(starts & (~0ull >> (63 - lane)));
      first += __popcll(starts);
      const int d = __builtin_amdgcn_ds_bpermute(4 * m, delta);
      v[i] = edges[r < used ? r + d : 0];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (64 * (half + i) >= used) break;
      const float4 E = v[i];
      const float b = dot3(E.x, E.y, E.z, cone.cx, cone.cy, cone.cz);
      const float e = fabsf(E.x) + fabsf(E.y) + fabsf(E.z);
      const bool keep = 64 * (half + i) + lane < used && !(fmaf(e, cone.rho, b) < 0.0f);
      const unsigned long long mask = __ballot(keep);
      const int at = kept + __popcll(mask & ((1ull << lane) - 1ull));
      if (keep && at < kStageRecords) slab[at] = E;
      const int lo = from - 64 * (half + i);
      if (lo > 0) start = kept + __popcll(lo >= 64 ? mask : mask & ((1ull << lo) - 1ull));
      kept += __popcll(mask);
    }
  }
  if (kept > kStageRecords) return nullptr;
  const int next = __builtin_amdgcn_ds_bpermute(4 * lane + 4, start);
  int span = start | (((lane + 1 < n ? next : kept) - start) << 16);
  span = __builtin_amdgcn_ds_bpermute(4 * rank, span);
  len = span >> 16;
  lds_order();
  staged = true;
  return slab + (span & 0xffff);
}

// Waves per SIMD that a forward kernel with one lane per ray is held to.  The
// persistent kernels of the larger models, which hold their queue's state as
// well, are faster without spills (800x800 frame, two maps: 100k sites 884 us at
// five waves, 764 at three, 4,000 sites 682 and 491; spherical harmonics 845 at
// four, 736 at three, and 582 and 481).
template <int APP, bool E16, bool PERSIST = false>
constexpr int kFwdWaves = PERSIST && APP ? 3 : APP == 2 ? 4 : E16 ? 4 : 5;

// walk_forward with one lane per ray and staged rows.  Every lane of the
// wave must call this (has_ray = false for lanes without a ray); slab: the
// wave's kStageBytesPerWave of LDS.
template <int TEX, int APP, bool E16 = false>
__device__ __forceinline__ RayOut walk_forward_staged(const DevScene& s, const WalkParams& w,
                                                      const RayIn& r, bool has_ray, int lane,
                                                      float4* slab, int32_t* rec, int max_record,
                                                      Counters& cnt, bool dist_on = false,
                                                      const ExitTrace& xt = {}) {
  FwdState<APP> st;
  const bool walk = has_ray && fwd_begin<APP>(st, s, r, cnt);
  bool alive = walk;
  const Cone cone = wave_cone(r, walk);
  if (lane == 0) *reinterpret_cast<Cone*>(reinterpret_cast<int*>(slab + kStageRecords) + 64) = cone;
  lds_order();
  // after a step whose rows could not be staged the wave waits `wait` steps
  // before it tries again, doubling the wait up to kStageMaxGap while it
  // keeps failing (rays that have spread apart seldom meet again soon, and
  // each failed try costs a ranking, up to the round that finds more than
  // kStageCells cells, and the loads of rows whose faces turn out too many)
  int wait = 0, gap = 1;
  while (__any(alive)) {
    const float4* row = nullptr;
    int len = 0;
    if (wait == 0) {
      // the row bounds for the staging (the record fwd_step will use)
      Cell c;
      if (alive) c = st.nc;
      bool staged;
      row = stage_rows(s.edges, slab, alive, st.cur, c, lane, len, staged);
      if (staged) {
        gap = 1;
      } else {
        wait = gap;
        gap = min(2 * gap, kStageMaxGap);
      }
    } else {
      --wait;
    }
    if (alive) {
      if (row)
        alive = !fwd_step<1, TEX, APP, E16>(st, s, w, r, 0, rec, max_record, cnt, dist_on, row, len, xt);
      else
        alive =
            !fwd_step<1, TEX, APP, E16>(st, s, w, r, 0, rec, max_record, cnt, dist_on, nullptr, 0, xt);
    }
  }
  return fwd_end<APP>(st, walk, cnt);
}

// ------------------------------------------------------------- adjoint
//
// Adjoint of walk_forward for L = g.C + g_T T_final.  The walk is replayed
// with identical decisions (each exit searched again, or read from the
// forward's stored exits) and, per segment k (App. X of the derivation in
// the oracle's adjoint module):
//   dL/dtau_k  = g.(T_{k+1} c_k - S_k) - g_T T_final,  S_k = C - sum_{j<=k} w_j c_j
//   dL/dsigma  += dL/dtau_k delta_k,    dL/dtexel_q += w_k b_q g
//   the exit end of the segment moves with its bisector crossing (+D) and
//   the entry end, the crossing that last advanced t, with -D, where
//   D = sigma_k dL/dtau_k; for the bisector of (a, b) crossed at t,
//   dt/dp_a = (x - p_a)/beta, dt/dp_b = (p_b - x)/beta, beta = (p_b - p_a).w.
//
// Gradient traffic.  A visited cell receives contributions from its own
// segment and from its two faces on the ray, i.e. from three consecutive
// steps.  Each lane keeps a sliding window (previous cell, current cell, next
// cell) and emits a cell's finished record - dsigma, dp (3), 12 texel terms -
// once, one step after leaving it.  The records of a wave that share a key
// (cell, texel quad) are summed before they go to the workgroup's table and
// from there to global memory.  Faces whose far cell has already been emitted
// (only after zero-length segments) go straight to the atomics.

__device__ __forceinline__ void atomic_site(const Grads& g, int cell, float x, float y, float z) {
  float* p = reinterpret_cast<float*>(g.cell + cell);
  atomicAdd(p, x);
  atomicAdd(p + 1, y);
  atomicAdd(p + 2, z);
}

// A record's key is (cell * maps + map) * R^2 + texel quad.  Address of term
// c (0..15): 0 dsigma, 1-3 dp, 4-15 the texel terms of taps (r0,c0),
// (r0,c0+1), (r0+1,c0), (r0+1,c0+1) x RGB of that map.
__device__ __forceinline__ float* record_addr(const Grads& g, int key, int c, int RR, int R) {
  const int cm = (int)(__umulhi((unsigned)key, g.rr_mul) >> g.rr_shift);
  const int base = key - cm * RR;
  const int cell = g.maps == 2 ? (cm >> 1) : cm;
  if (c < 4) return reinterpret_cast<float*>(g.cell + cell) + (c == 0 ? 3 : c - 1);
  const int t = (c - 4) / 3;
  const int ch = (c - 4) - 3 * t;
  return g.texels + ((size_t)cm * (size_t)RR + (size_t)base) * 4 + (t & 1) * 4 + (t >> 1) * 4 * R +
         ch;
}

// Workgroup gradient table in LDS: a four-way cache of 16 FP32 sums per record
// key (cell * R^2 + texel quad).  A wave adds to an entry under the entry's
// lock (the sign bit of its key word); a key whose four ways all hold other
// keys takes one of them over, and the sums it held go to global memory.  The
// rest reach global memory when the workgroup flushes.
//
// What bounds the adjoint: device float atomics leave a CU at most 64 bytes at
// a time and the chip at 20 G requests/s, wherever the line is held, and LDS
// float atomics take 3 cycles per active lane (193 per full wave; a read and a
// write together 5.6).  So records are summed across the wave first, by
// exact key and in FP32 (emit_records), the sums are added by plain reads and writes, and entries
// that later rays cannot reach any more make room for new ones.  4M sites, 8
// views: device requests 817 M -> 130 M, LDS busy 0.78 -> 0.25, adjoint 51.9 ->
// 29.7 ms; 100k sites, 800x800: 1.17 -> 0.72 ms (two maps: 2.40 -> 1.50 ms).
// Taking over a fixed way per key instead of one that moves on with the steps
// left finished cells in place: 32.0 ms at 4M sites.  Locking with a loop over
// single slots instead of one 16-byte read of a set cost 240 us of the 100k
// adjoint; LDS float atomics on the merged sums instead of the lock, 100 us.
// 512 entries are what leaves room for three workgroups per CU beside the
// merge areas (four waves per SIMD instead of three spill inside the walk:
// 63.6 against 62.0 ms per 4M-site step).
constexpr int kBwdWaves = 3;      // waves per SIMD of every adjoint kernel
constexpr int kTableCap = 512;
constexpr int kTableTries = 16;   // rounds before a contended sum goes to global memory
constexpr int kTableLock = (int)0x80000000;

struct GradTable {
  int* keys;    // [kTableCap], -1 = empty, key | kTableLock = held by a wave
  float* vals;  // [kTableCap + 1][16]; the last is written for keys without an entry
};

// all threads of the workgroup; needs a barrier before the table is used
__device__ __forceinline__ void table_clear(const GradTable& t) {
  for (int i = threadIdx.x; i < kTableCap; i += blockDim.x) t.keys[i] = -1;
  for (int i = threadIdx.x; i < kTableCap * 16; i += blockDim.x) t.vals[i] = 0.0f;
}

// Lock the entry of `key`, taking one over if need be: its slot, or -1 when
// another lane or wave holds the entry that would be taken (never waits).
// old: the key whose sums the entry holds, -1 if none.  age moves the way
// that is taken over.
__device__ __forceinline__ int table_lock(const GradTable& t, int key, unsigned age, int& old) {
  const unsigned h = (unsigned)key * 2654435761u;
  const int set = (int)(((unsigned long long)h * (unsigned)(kTableCap / 4)) >> 32);
  using i32x4 = int __attribute__((ext_vector_type(4)));
  const i32x4 k = *reinterpret_cast<const volatile i32x4*>(t.keys + 4 * set);
  const int turn = (h + age) & 3;   // the way taken over when all four are full
  int way = turn;
  int e = turn == 0 ? k.x : turn == 1 ? k.y : turn == 2 ? k.z : k.w;
#pragma unroll
  for (int w = 3; w >= 0; --w) {
    way = k[w] == -1 ? w : way;
    e = k[w] == -1 ? -1 : e;
  }
#pragma unroll
  for (int w = 3; w >= 0; --w) {
    const bool hit = (k[w] & ~kTableLock) == key;
    way = hit ? w : way;
    e = hit ? k[w] : e;
  }
  old = e;
  if (e < -1) return -1;  // held
  const int slot = 4 * set + way;
  return atomicCAS(&t.keys[slot], e, key | kTableLock) == e ? slot : -1;
}

// all threads of the workgroup, after a barrier: every entry to global
// memory once (16 consecutive threads per entry, one term each), and the
// table left empty (a barrier must follow)
__device__ __forceinline__ void table_flush(const GradTable& t, const Grads& g, int RR,
                                            int R) {
  for (int i = threadIdx.x; i < kTableCap * 16; i += blockDim.x) {
    const int key = t.keys[i >> 4];
    if (key < 0) continue;
    const float x = t.vals[i];
    t.vals[i] = 0.0f;
    if (x != 0.0f) atomicAdd(record_addr(g, key, i & 15, RR, R), x);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kTableCap; i += blockDim.x) t.keys[i] = -1;
}

// One wave's LDS area for merging its records: row c < 16 holds term c of
// every lane, row 16 the lanes' ranks and other words of the merge.
constexpr int kMergeStride = 68;  // 16-byte rows that start four banks apart
constexpr int kMergeFloats = 17 * kMergeStride;

// Merge the wave's records by key and add the sums to the workgroup table.
// Every lane of the wave must call this (key < 0: no record).  The texel term
// of tap t and channel ch is tap weight t x m_ch.  C0 = 4 marks a texel-only
// record.  settle() runs before the first global atomic.
//
// The wave's keys are ranked; then, 16 at a time, a 16 x 64 matrix of
// zeros and ones (rank of lane k is m) times the 64 x 16 matrix of the lanes'
// terms gives each key's 16 sums in FP32 on the matrix cores, laid out so that
// 16 lanes hold one key's terms: the table's and the atomics' order.  A wave
// of 64 rays stands in about 6 distinct (cell, quad)s a step on the 100k-site
// scene and 16 on the 4M-site one; a butterfly over lane ^ m, which it
// replaces, left 20 and 38 records and took three times the VALU work.
template <int C0, class F>
__device__ __forceinline__ void emit_records(int key, float ds, float px, float py, float pz,
                                             const Taps& tp, float mr, float mg, float mb, int lane,
                                             int RR, int R, const Grads& g, const GradTable& tab,
                                             float* area, unsigned age, F&& settle) {
  if (!__any(key >= 0)) return;
  float* rank_row = area + 16 * kMergeStride;
  int* word = reinterpret_cast<int*>(rank_row);
  area[0 * kMergeStride + lane] = ds;
  area[1 * kMergeStride + lane] = px;
  area[2 * kMergeStride + lane] = py;
  area[3 * kMergeStride + lane] = pz;
  const float q[4] = {tp.w00, tp.w01, tp.w10, tp.w11};
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    area[(4 + 3 * t) * kMergeStride + lane] = q[t] * mr;
    area[(5 + 3 * t) * kMergeStride + lane] = q[t] * mg;
    area[(6 + 3 * t) * kMergeStride + lane] = q[t] * mb;
  }
  const int n = lane & 15;
  const int grp = lane >> 4;
  int rank;
  bool leads;
  const int total =
      rank_keys(key, key >= 0, reinterpret_cast<unsigned char*>(word), lane, 64, rank, leads);
  for (int base = 0; base < total; base += 16) {
    using f32x4 = float __attribute__((ext_vector_type(4)));
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    word[lane] = rank - base;
    lds_order();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const f32x4 b = *reinterpret_cast<const f32x4*>(area + n * kMergeStride + 16 * grp + 4 * j);
      const int4 rk = *reinterpret_cast<const int4*>(word + 16 * grp + 4 * j);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(rk.x == n ? 1.0f : 0.0f, b.x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(rk.y == n ? 1.0f : 0.0f, b.y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(rk.z == n ? 1.0f : 0.0f, b.z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(rk.w == n ? 1.0f : 0.0f, b.w, acc, 0, 0, 0);
    }
    lds_order();
    const bool now = rank >= base && rank < base + 16;
    if (leads && now) word[rank - base] = key;
    lds_order();
    const int cnt = min(16, total - base);
    int mine = lane < cnt ? word[lane] : -1;
    if (base == 0) settle();
    const float big = fabsf(acc.x) + fabsf(acc.y) + fabsf(acc.z) + fabsf(acc.w);
    if (__any(!(big < kInf))) {
      // an infinity or NaN would reach every sum (0 x inf): each record of
      // this pass goes to global memory by itself
      for (int c = C0; c < 16; ++c) {
        const float x = area[c * kMergeStride + lane];
        if (now && x != 0.0f) atomicAdd(record_addr(g, key, c, RR, R), x);
      }
      continue;
    }
    const float a4[4] = {acc.x, acc.y, acc.z, acc.w};
    for (int it = 0; __any(mine >= 0); ++it) {
      // the last round sends what found no entry to global memory
      int slot = -1, old = -1;
      const bool last = it >= kTableTries;
      if (mine >= 0 && !last) slot = table_lock(tab, mine, age, old);
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
      // what becomes of the sums the entry holds: kept (-2), none (-1), or
      // another key's, to be sent
      if (slot >= 0) old = old == mine ? -2 : old;
      if (lane < 16) {
        word[lane] = slot >= 0 ? slot : kTableCap;
        word[16 + lane] = slot >= 0 ? old : last ? mine : -1;
      }
      lds_order();
      const int4 sl = *reinterpret_cast<const int4*>(word + 4 * grp);
      const int4 ky = *reinterpret_cast<const int4*>(word + 16 + 4 * grp);
      const int s4[4] = {sl.x, sl.y, sl.z, sl.w};
      const int k4[4] = {ky.x, ky.y, ky.z, ky.w};
      float x4[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) x4[i] = tab.vals[16 * s4[i] + n];
#pragma unroll
      for (int i = 0; i < 4; ++i) tab.vals[16 * s4[i] + n] = a4[i] + (k4[i] == -2 ? x4[i] : 0.0f);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
      if (slot >= 0)
        __hip_atomic_store(&tab.keys[slot], mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (__any(old >= 0 || (last && mine >= 0))) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float x = last ? a4[i] : x4[i];
          if (k4[i] >= 0 && x != 0.0f) atomicAdd(record_addr(g, k4[i], n, RR, R), x);
        }
      }
      if (slot >= 0 || last) mine = -1;
    }
  }
}

// Every lane of the wave must call this; has_ray = false for lanes without a
// ray.  The loop runs until every lane's walk has ended, so the record merge
// always sees the full wave.
//
// Full appearance model (APP = 1): with c = sigmoid(l), dL/dl = w_k g c(1-c)
// per channel feeds the surface-map taps (in the cell's delayed record) and
// the view-map taps (a record of its own, sent at once).  The surface
// direction adds dL/dx = J^T dL/d(u,v) for the hit point x, J the
// octahedral map's Jacobian at x - p_i: -dL/dx goes to the site, and
// dL/dt_hit = dL/dx . w to the crossing that placed x (the entry face, or
// the start cell's exit face) through the same dt/dp as the segment ends.
//
// Distortion loss (dist_on): with G_k = dL_dist/dw_k, the chain through
// w_k = T_k - T_{k+1} gives dL_dist/dtau_k = G_k T_{k+1} - sum_{j>k} G_j w_j,
// and sum_j G_j w_j = 2 L_dist, so the suffix follows from the saved loss;
// the interval ends move with their crossings through
// dL_dist/dt = (dL/dsbar / 2 -+ dL/dds) s'(t), s'(t) = 1/(1+t)^2.
template <int LPR, int TEX, int APP>
__device__ __forceinline__ void walk_backward(const DevScene& s, const WalkParams& w, const RayIn& r,
                                              const Upstream& u, bool has_ray, int sub, int lane,
                                              const Grads& g, const GradTable& tab,
                                              float* area, Counters& cnt,
                                              bool dist_on = false, const ExitTrace& xt = {}) {
  const int R = s.res;
  const int RR = R * R;
  constexpr int MAPS = APP ? 2 : 1;
  bool active = has_ray && r.tmax > 0.0f;
  if (active && (r.start < 0 || r.start >= s.n)) {
    cnt.bad++;
    active = false;
  }
  if (active) cnt.rays++;
  const bool lead = sub == 0;
  // no weights without a ray: its direction is none, and a NaN in an idle lane
  // would send the whole wave's records past the merge
  Taps tp{};
  if (active) tp = ray_taps<APP>(r, R);
  float T = 1.0f, Pr = 0.0f, Pg = 0.0f, Pb = 0.0f, t_in = 0.0f;
  float dW = 0.0f, dA = 0.0f, dGW = 0.0f, s0 = 0.0f;  // distortion prefix sums
  int cur = active ? r.start : 0;
  // the current cell's position and density: loaded with the previous
  // step's exit (a step with a stored exit needs nothing else of its cell).
  // Single map only: the full model's adjoint would lose a wave per SIMD to
  // the registers it holds.
  constexpr bool kCarry = APP == 0;
  float4 here = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  if (kCarry && active) here = s.cells[2 * (size_t)cur];
  // Loads run ahead of their use (single map): the texels of the cell entered
  // next, the stored exits of the next two steps and the far site of the next
  // one's exit face are all under way while a step's records are merged.  They
  // fill the registers that three waves per SIMD leave (168; spilled to 128 for
  // a fourth wave they cost 40%, without them four waves were 4% slower).
  TexQuad<TEX> tx;
  int2 e0 = make_int2(0, -1), e1 = make_int2(0, -1);
  float4 ahead = here;
  if (kCarry && active) {
    tx.load(s.texels, (size_t)cur * (size_t)RR + (size_t)tp.base, R);
    if (xt.p) {
      e0 = xt.p[0];
      if (xt.cap > 1) e1 = xt.p[xt.stride];
      if (e0.y >= 0 && e0.y < s.n) ahead = s.cells[2 * (size_t)e0.y];
    }
  }

  int k = 0;
  // previous cell's record (emitted one step late): its texel multipliers
  // and, for APP = 1, its surface taps
  int a_cell = -1;
  float a_ds = 0.0f, a_px = 0.0f, a_py = 0.0f, a_pz = 0.0f;
  float a_mr = 0.0f, a_mg = 0.0f, a_mb = 0.0f;
  Taps a_tp = tp;
  // position gradient already received by the cell entered next
  int c_cell = -1;
  float c_px = 0.0f, c_py = 0.0f, c_pz = 0.0f;
  // the entry face: cells (fa, fb) and dt/dp_fa, dt/dp_fb
  int fa = -1, fb = -1;
  float uax = 0.0f, uay = 0.0f, uaz = 0.0f, ubx = 0.0f, uby = 0.0f, ubz = 0.0f;
  // wait for the loads under way before the records' global atomics follow
  // them (their counter is shared and in order)
  auto settle = [&] {
    if constexpr (kCarry) {
      asm volatile("" : "+v"(e1.x), "+v"(e1.y), "+v"(ahead.x), "+v"(ahead.y), "+v"(ahead.z), "+v"(ahead.w));
      tx.settle();
    }
  };
  unsigned age = 0;
  for (;;) {
    if (!__any(active)) break;
    int e_key = -1;
    float e_ds = 0.0f, e_px = 0.0f, e_py = 0.0f, e_pz = 0.0f;
    float e_mr = 0.0f, e_mg = 0.0f, e_mb = 0.0f;
    Taps e_tp = tp;
    int v_key = -1;  // APP = 1: this cell's view-map record
    float v_mr = 0.0f, v_mg = 0.0f, v_mb = 0.0f;
    if (active) {
      Cell c;
      Exit ex;
      const bool stored = xt.p && k < xt.cap;
      if (stored) {
        // the forward's exit of this step (a next cell outside the scene,
        // which only a trace from another walk could hold, ends the ray)
        const int2 e = kCarry ? e0 : xt.p[(size_t)k * xt.stride];
        ex.t = __int_as_float(e.x);
        ex.next = e.y >= 0 && e.y < s.n ? e.y : -1;
        ex.redecided = false;
      }
      if (kCarry && stored) {
        c.px = here.x;
        c.py = here.y;
        c.pz = here.z;
        c.sigma = here.w;
        c.off = 0;
        c.deg = 0;
      } else {
        c = load_cell(s.cells, cur);
        if (!stored) ex = step_exit<LPR>(s, w, r, c, cur, t_in, sub);
      }
      float4 pn = here;
      float cr, cg, cb;
      if constexpr (kCarry) {
        quad_rgb<TEX>(tx, tp, cr, cg, cb);
        if (stored) {
          pn = ahead;
          e0 = e1;
          if (k + 2 < xt.cap) e1 = xt.p[(size_t)(k + 2) * xt.stride];
          if (k + 1 < xt.cap && e0.y >= 0 && e0.y < s.n) ahead = s.cells[2 * (size_t)e0.y];
        } else if (ex.next >= 0) {
          pn = s.cells[2 * (size_t)ex.next];
        }
        if (ex.next >= 0) tx.load(s.texels, (size_t)ex.next * (size_t)RR + (size_t)tp.base, R);
      }
      cnt.redecide += ex.redecided ? 1u : 0u;
      cnt.deg += (uint32_t)c.deg;
      const Segment sg = segment(ex.t, r.tmax, t_in, c.sigma);
      const float wk = T * sg.alpha;
      Taps ts = tp;
      float gxx = 0.0f, gxy = 0.0f, gxz = 0.0f, dldt = 0.0f;
      float glr = 0.0f, glg = 0.0f, glb = 0.0f;
      if constexpr (APP == 1) {
        float hx, hy, hz;
        hit_vector(r, c, k, t_in, ex.t, hx, hy, hz);
        const bool on_site = hx == 0.0f && hy == 0.0f && hz == 0.0f;
        ts = make_taps(on_site ? r.dx : hx, on_site ? r.dy : hy, on_site ? r.dz : hz, R);
        float lr, lg, lb;
        float4 ta, tb, te, tf;
        full_logits<TEX>(s.texels, cur, R, ts, tp, lr, lg, lb, ta, tb, te, tf);
        cr = sigmoid_f(lr);
        cg = sigmoid_f(lg);
        cb = sigmoid_f(lb);
        glr = wk * u.gr * cr * (1.0f - cr);
        glg = wk * u.gg * cg * (1.0f - cg);
        glb = wk * u.gb * cb * (1.0f - cb);
        if (!on_site) {
          // dL/d(u,v) of the bilinear surface lookup (taps held fixed)
          const float kR = 0.5f * (float)(R - 1);
          const float fx = ts.w01 + ts.w11;
          const float fy = ts.w10 + ts.w11;
          const float dur = kR * fmaf(fy, tf.x - te.x, (1.0f - fy) * (tb.x - ta.x));
          const float dug = kR * fmaf(fy, tf.y - te.y, (1.0f - fy) * (tb.y - ta.y));
          const float dub = kR * fmaf(fy, tf.z - te.z, (1.0f - fy) * (tb.z - ta.z));
          const float dvr = kR * fmaf(fx, tf.x - tb.x, (1.0f - fx) * (te.x - ta.x));
          const float dvg = kR * fmaf(fx, tf.y - tb.y, (1.0f - fx) * (te.y - ta.y));
          const float dvb = kR * fmaf(fx, tf.z - tb.z, (1.0f - fx) * (te.z - ta.z));
          const float gu = dot3(glr, glg, glb, dur, dug, dub);
          const float gv = dot3(glr, glg, glb, dvr, dvg, dvb);
          float ju[3], jv[3];
          oct_jacobian(hx, hy, hz, ju, jv);
          gxx = fmaf(gu, ju[0], gv * jv[0]);
          gxy = fmaf(gu, ju[1], gv * jv[1]);
          gxz = fmaf(gu, ju[2], gv * jv[2]);
          dldt = dot3(gxx, gxy, gxz, r.dx, r.dy, r.dz);
        }
      }
      Pr = fmaf(wk, cr, Pr);
      Pg = fmaf(wk, cg, Pg);
      Pb = fmaf(wk, cb, Pb);
      const float Tn = T * sg.trans;
      const float Sr = u.Cr - Pr;
      const float Sg = u.Cg - Pg;
      const float Sb = u.Cb - Pb;
      float dtau =
          fmaf(u.gb, Tn * cb - Sb, fmaf(u.gg, Tn * cg - Sg, u.gr * (Tn * cr - Sr))) - u.gT * u.Tf;
      float dist_in = 0.0f, dist_ex = 0.0f;  // dL_dist/dt of the interval's ends
      if (dist_on) {
        const float t1 = fmaxf(t_in, fminf(ex.t, r.tmax));
        const float s1 = dist_s(t1);
        const float sb = 0.5f * (s0 + s1);
        const float dsv = s1 - s0;
        const float Wle = dW + wk;
        const float Ale = fmaf(wk, sb, dA);
        const float Gk = 2.0f * (fmaf(sb, dW, -dA) + (u.DA - Ale) - sb * (u.DW - Wle)) +
                         (2.0f / 3.0f) * wk * dsv;
        const float GWle = fmaf(Gk, wk, dGW);
        dtau = fmaf(u.gD, fmaf(Gk, Tn, -(2.0f * u.D - GWle)), dtau);
        const float gsb = 2.0f * wk * (dW - (u.DW - Wle));
        const float gds = wk * wk * (1.0f / 3.0f);
        const float i0 = 1.0f / (1.0f + t_in);
        const float i1 = 1.0f / (1.0f + t1);
        dist_in = u.gD * fmaf(0.5f, gsb, -gds) * (i0 * i0);
        dist_ex = u.gD * fmaf(0.5f, gsb, gds) * (i1 * i1);
        dW = Wle;
        dA = Ale;
        dGW = GWle;
        s0 = s1;
      }
      // this cell's record starts with what its entry face already sent it,
      // less the hit point's own pull on the site
      float m_px = (c_cell == cur ? c_px : 0.0f) - gxx;
      float m_py = (c_cell == cur ? c_py : 0.0f) - gxy;
      float m_pz = (c_cell == cur ? c_pz : 0.0f) - gxz;
      int n_cell = -1;
      float n_px = 0.0f, n_py = 0.0f, n_pz = 0.0f;
      if (sg.delta > 0.0f) {
        const float D = c.sigma * dtau;
        // dL/dt of the entry end (the hit point rides on it when k > 0) and
        // of the exit end (the start cell's hit point rides on it)
        const float Din = (k > 0 ? dldt : 0.0f) - D + dist_in;
        const float Dex = D + (k == 0 ? dldt : 0.0f) + dist_ex;
        if (fa >= 0) {
          if (fa == a_cell) {
            a_px = fmaf(Din, uax, a_px);
            a_py = fmaf(Din, uay, a_py);
            a_pz = fmaf(Din, uaz, a_pz);
          } else if (lead) {
            atomic_site(g, fa, Din * uax, Din * uay, Din * uaz);
          }
          if (fb == cur) {
            m_px = fmaf(Din, ubx, m_px);
            m_py = fmaf(Din, uby, m_py);
            m_pz = fmaf(Din, ubz, m_pz);
          } else if (fb == a_cell) {
            a_px = fmaf(Din, ubx, a_px);
            a_py = fmaf(Din, uby, a_py);
            a_pz = fmaf(Din, ubz, a_pz);
          } else if (lead) {
            atomic_site(g, fb, Din * ubx, Din * uby, Din * ubz);
          }
        }
        if (ex.t < r.tmax && ex.next >= 0) {
          // exit end: along the exit face (cur -> next)
          if constexpr (!kCarry) pn = s.cells[2 * (size_t)ex.next];
          const float nx = pn.x - c.px;
          const float ny = pn.y - c.py;
          const float nz = pn.z - c.pz;
          const float beta = dot3(nx, ny, nz, r.dx, r.dy, r.dz);
          const float xx = fmaf(ex.t, r.dx, r.ox);
          const float xy = fmaf(ex.t, r.dy, r.oy);
          const float xz = fmaf(ex.t, r.dz, r.oz);
          const float ib = 1.0f / beta;
          uax = (xx - c.px) * ib;
          uay = (xy - c.py) * ib;
          uaz = (xz - c.pz) * ib;
          ubx = (pn.x - xx) * ib;
          uby = (pn.y - xy) * ib;
          ubz = (pn.z - xz) * ib;
          fa = cur;
          fb = ex.next;
          m_px = fmaf(Dex, uax, m_px);
          m_py = fmaf(Dex, uay, m_py);
          m_pz = fmaf(Dex, uaz, m_pz);
          n_cell = ex.next;
          n_px = Dex * ubx;
          n_py = Dex * uby;
          n_pz = Dex * ubz;
        }
      }
      // the previous cell is complete: emit it
      if (lead && a_cell >= 0) {
        e_key = (a_cell * MAPS) * RR + a_tp.base;
        e_ds = a_ds;
        e_px = a_px;
        e_py = a_py;
        e_pz = a_pz;
        e_mr = a_mr;
        e_mg = a_mg;
        e_mb = a_mb;
        e_tp = a_tp;
      }
      if constexpr (APP == 1) {
        if (lead) {
          v_key = (2 * cur + 1) * RR + tp.base;
          v_mr = glr;
          v_mg = glg;
          v_mb = glb;
        }
      }
      a_cell = cur;
      a_ds = dtau * sg.delta;
      a_px = m_px;
      a_py = m_py;
      a_pz = m_pz;
      if constexpr (APP == 0) {
        a_mr = wk * u.gr;
        a_mg = wk * u.gg;
        a_mb = wk * u.gb;
      } else {
        a_mr = glr;
        a_mg = glg;
        a_mb = glb;
        a_tp = ts;
      }
      c_cell = n_cell;
      c_px = n_px;
      c_py = n_py;
      c_pz = n_pz;
      T = Tn;
      ++k;
      bool stop = T < w.t_stop || !(ex.t < r.tmax) || ex.next < 0;
      if (!stop && k >= w.max_steps) {
        cnt.maxsteps++;
        stop = true;
      }
      if (stop) {
        active = false;
        cnt.steps += (uint32_t)k;
        if (T != T) cnt.nan++;
      } else {
        t_in = fmaxf(t_in, fminf(ex.t, r.tmax));
        cur = ex.next;
        if constexpr (kCarry) here = pn;
      }
    }
    emit_records<0>(e_key, e_ds, e_px, e_py, e_pz, e_tp, e_mr, e_mg, e_mb, lane,
                                   RR, R, g, tab, area, age++, settle);
    if constexpr (APP == 1)
      emit_records<4>(v_key, 0.0f, 0.0f, 0.0f, 0.0f, tp, v_mr, v_mg, v_mb, lane, RR, R,
                                 g, tab, area, age, [] {});
  }
  // the last visited cell, and the unvisited cell behind an early-stopped ray's exit face
  emit_records<0>(lead && a_cell >= 0 ? (a_cell * MAPS) * RR + a_tp.base : -1,
                                 a_ds, a_px, a_py, a_pz, a_tp, a_mr, a_mg, a_mb, lane, RR, R, g,
                                 tab, area, age, [] {});
  emit_records<0>(lead && c_cell >= 0 ? (c_cell * MAPS) * RR + tp.base : -1, 0.0f,
                                 c_px, c_py, c_pz, tp, 0.0f, 0.0f, 0.0f, lane, RR, R, g, tab, area, age, [] {});
}

}  // namespace voro

namespace voro {
// host helpers (defined in walk.hip)
DevScene dev_scene(const voro_scene* s, const void* ws);
WalkParams walk_params(const voro_params* p);
}  // namespace voro
