// HIP kernels of the per-iteration path (gfx950, 64-wide wavefronts).
//
//  - fwd_level / bwd_level: one level of the batched supernodal forward and
//    backward solves of all subdomains at once (local solves of eq. oras).
//    One workgroup (4 waves) per tile of <= 64 panel rows; each lane owns a
//    row, the four waves split the input columns, the input vector (gathered
//    through index lists, restriction fused in) sits in LDS, and the panel is
//    streamed column by column (64 rows x 16 B = 1 KiB coalesced per wave).
//  - spmv / spmv_real: CSR products, a group of lanes per row.
//  - prolong: partition-of-unity weighted sum of the local solutions.
//  - Gram-Schmidt reductions: per-block partial sums reduced in a fixed order
//    (no atomics), so every result is bitwise repeatable.
#include <hip/hip_cooperative_groups.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>

#include "device.hpp"

namespace helm {
namespace dev {

namespace {

constexpr int kWG = 256;
constexpr int kChunk = kLevelChunkMax;  // input columns staged in LDS per pass (at most)

__device__ __forceinline__ void cfma(double& ar, double& ai, double2 a, double2 v) {
  ar = fma(a.x, v.x, ar);
  ar = fma(-a.y, v.y, ar);
  ai = fma(a.x, v.y, ai);
  ai = fma(a.y, v.x, ai);
}

__device__ __forceinline__ double2 widen(double2 a) { return a; }
__device__ __forceinline__ double2 widen(float2 a) { return make_double2((double)a.x, (double)a.y); }

__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int64_t uni64(int64_t x) {
  return ((int64_t)uni((int)(x >> 32)) << 32) | (uint32_t)uni((int)x);
}

// Panel tiles are read through buffer loads: the tile's base and the column
// offset are scalar, a lane adds one constant offset, and a lane whose entry is
// not wanted (rows past the tile, columns past its share, the zero triangle of
// a diagonal block) passes an offset past the buffer, which returns zero and
// fetches nothing.  The hardware tests lane offset >= size - scalar offset, so
// the scalar offset must not pass the size either (the difference would wrap):
// it is clamped to it, where every lane offset is out of range.
// The sweeps of a large operator are bound by HBM: without the zero triangles
// (6 % of the panel entries at one million unknowns in 64 subdomains) they fetch
// 21.3 GB instead of 22.9, and the address arithmetic leaves the vector unit:
// local solves 3.57 -> 3.45 ms, with complex64 panels 2.02 -> 1.98 ms.
constexpr int kBufNt = 2;                 // cache policy: non-temporal
constexpr int kBufSkip = 0x7ffffff0;      // an offset no tile reaches
__device__ __forceinline__ __amdgpu_buffer_rsrc_t panel_rsrc(const void* p, int64_t off, int bytes) {
  // raw buffer: no stride, range checked in bytes
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(reinterpret_cast<const char*>(p)) + uni64(off), 0,
                                           uni(bytes), 0x00020000);
}
template <class PT>
__device__ __forceinline__ PT ldb(__amdgpu_buffer_rsrc_t r, int voff, int soff);
template <>
__device__ __forceinline__ double2 ldb<double2>(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, kBufNt));
}
template <>
__device__ __forceinline__ float2 ldb<float2>(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, kBufNt));
}

// x / d for 0 <= x < 4096 and 1 <= d <= 64 as one multiplication: floor(x m /
// 2^20) with m = floor(2^20 / d) + 1 (the error x / 2^20 stays below 1 / d).
// The compiler's division by a run-time value is some thirty vector
// instructions and a short task had ten of them: local solves of 168,075
// unknowns 343 -> 328 us.
struct DivTable {
  uint32_t m[65];
  constexpr DivTable() : m() {
    for (uint32_t d = 1; d <= 64; ++d) m[d] = (1u << 20) / d + 1;
  }
};
__constant__ const DivTable kDiv{};
__device__ __forceinline__ int div20(int x, uint32_t m) { return (int)(((uint32_t)x * m) >> 20); }

// Lanes of a tile: a tile with few rows spreads its columns over G = 64 / R
// lane groups of R = nrows lanes (the last 64 mod R lanes idle).
struct Lanes {
  int R, G, grp, row;
  uint32_t mg;  // divides by G
  __device__ __forceinline__ explicit Lanes(int nrows) {
    const int lane = threadIdx.x & 63;
    R = nrows <= 32 ? max(nrows, 1) : 64;
    const uint32_t mr = kDiv.m[R];
    G = div20(64, mr);
    grp = div20(lane, mr);
    row = lane - grp * R;
    mg = kDiv.m[G];
  }
};

// A wave's share of a tile's panel: columns kbeg .. kend - 1 of a tile stored
// column-major, ld rows apart; a lane takes columns kbeg + grp, kbeg + grp + G,
// ... and keeps those in [lo, hi).
template <class PT>
struct Panel {
  __amdgpu_buffer_rsrc_t r;
  int bytes;       // of the buffer (uniform)
  int voff;        // of this lane in a group of G columns
  int step;        // bytes per group of G columns (uniform)
  int base;        // bytes of column kbeg (uniform)
  int n;           // groups (uniform)
  int i0;          // this lane's first group ...
  unsigned cnt;    // ... and number of groups
  __device__ __forceinline__ Panel(__amdgpu_buffer_rsrc_t rs, int size, int ld, int kbeg, int kend, const Lanes& l,
                                   bool on, int lo, int hi) {
    r = rs;
    bytes = uni(size);
    voff = (l.grp * ld + l.row) * (int)sizeof(PT);
    step = uni(l.G * ld * (int)sizeof(PT));
    base = uni(kbeg * ld * (int)sizeof(PT));
    n = uni(kend > kbeg ? div20(kend - kbeg + l.G - 1, l.mg) : 0);
    const int first = kbeg + l.grp;  // column of group 0
    hi = min(hi, kend);
    i0 = div20(max(lo - first + l.G - 1, 0), l.mg);
    const int e = div20(max(hi - first + l.G - 1, 0), l.mg);
    cnt = on && e > i0 ? (unsigned)(e - i0) : 0u;
  }
  __device__ __forceinline__ PT load(int i) const {
    return ldb<PT>(r, (unsigned)(i - i0) < cnt ? voff : kBufSkip, min(base + i * step, bytes));
  }
};

// The first eight groups of a panel share.
template <class PT>
__device__ __forceinline__ void tile_load(const Panel<PT>& p, PT (&a)[8]) {
#pragma unroll
  for (int u = 0; u < 8; ++u) a[u] = p.load(u);
}

// Streams a panel share against vin (vin[0] is the entry of the share's first
// column for this lane group, G entries per group; kmax: its last entry), the
// first eight groups already in a.  Eight loads stay in flight per lane: each
// register is refilled right after its column is used, instead of eight loads
// being issued and drained in turn (a chain of short levels, the coarse
// correction: 192 -> 168 us).  Groups sum into two accumulators alternately.
template <class PT>
__device__ __forceinline__ void tile_dot(const Panel<PT>& p, const double2* vin, int G, int kmax, PT (&a)[8],
                                         double& ar, double& ai) {
  double br = 0, bi = 0;
  int i = 0;
  for (; i + 8 < p.n; i += 8) {
#pragma unroll
    for (int u = 0; u < 8; u += 2) {
      cfma(ar, ai, widen(a[u]), vin[(i + u) * G]);
      a[u] = p.load(i + u + 8);
      cfma(br, bi, widen(a[u + 1]), vin[(i + u + 1) * G]);
      a[u + 1] = p.load(i + u + 9);
    }
  }
  // the last group; entries past the last column meet zero panel entries
#pragma unroll
  for (int u = 0; u < 8; u += 2) {
    if (i + u >= p.n) break;  // uniform
    cfma(ar, ai, widen(a[u]), vin[min((i + u) * G, kmax)]);
    cfma(br, bi, widen(a[u + 1]), vin[min((i + u + 1) * G, kmax)]);
  }
  ar += br;
  ai += bi;
}

// Calls f(i) for the child-update entries routed to front row fr, in list
// order: rows with at most two read them from their index pair (one load),
// longer lists from fcon_ptr / fcon_idx.
template <class F>
__device__ __forceinline__ void for_children(const Batch& b, int fr, F&& f) {
  const int2 c = b.fcon2[fr];
  if (c.x >= 0) {
    f(c.x);
    if (c.y >= 0) f(c.y);
  } else if (c.x < -1) {
    for (int e = -2 - c.x; e < b.fcon_ptr[fr + 1]; ++e) f(b.fcon_idx[e]);
  }
}

// Work split of a workgroup (4 waves) over the tiles of its task.
struct Split {
  int my;      // tile slot of this wave
  int part;    // this wave's share of the tile's columns
  int wpt, sh; // waves per tile (1, 2 or 4), its logarithm
  int region;  // LDS entries per tile slot
  bool has;    // the slot holds a tile
  // ceil(n / wpt)
  __device__ __forceinline__ int share(int n) const { return (n + wpt - 1) >> sh; }
};

__device__ __forceinline__ Split split_of(int wpt, int ntile, int chunk) {
  Split sp;
  // the wave index is the same on all lanes: scalar, so the wave's tile
  // descriptor is a scalar load
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  sp.wpt = wpt;
  sp.sh = wpt >> 1;
  sp.my = wv >> sp.sh;
  sp.part = wv & (wpt - 1);
  sp.region = chunk >> (2 - sp.sh);
  sp.has = sp.my < ntile;
  return sp;
}

// One workgroup task of a forward level (vin: chunk LDS entries, at least
// 4 / wpt times the widest tile of a task with wpt < 4; red: 4 x 64 LDS
// entries).
template <class PT>
__device__ __forceinline__ void fwd_task(const Task& task, const Batch& b, const double2* __restrict__ bin,
                                         double2* vin, double2 (*red)[64], int chunk) {
  const Split sp = split_of(task.wpt, task.ntile, chunk);
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Tile t{};
  if (sp.has) t = b.tf[task.tile0 + sp.my];
  const int s = t.sn, c0 = t.c0, w = t.w, frow0 = t.aux;
  double2* vt = vin + sp.my * sp.region;
  const Lanes l(t.nrows);
  const int bytes = t.nrows * t.ncols * (int)sizeof(PT);
  const __amdgpu_buffer_rsrc_t rs = panel_rsrc(b.pf, t.off * (int64_t)sizeof(PT), bytes);
  const double2* __restrict__ ub = reinterpret_cast<const double2*>(b.ubuf);
  // the children's updates to this lane's output row (rows past the pivot
  // block) are fetched before the panel, off the critical path
  const bool out = sp.has && sp.part == 0 && lane < t.nrows;
  const int row = t.row0 + lane;
  double er = 0, ei = 0;
  int uo = 0;
  if (out && row >= w) {
    uo = b.sn_uoff[s] + row - w;
    for_children(b, frow0 + row, [&](int i) {
      const double2 u = ub[i];
      er += u.x;
      ei += u.y;
    });
  }
  double ar = 0, ai = 0;
  // all waves of a workgroup run the same number of passes: one, unless the
  // workgroup holds a single wide tile
  for (int cb = 0; cb == 0 || (sp.wpt == 4 && cb < t.ncols); cb += sp.region) {
    const int cn = sp.has ? min(sp.region, t.ncols - cb) : 0;
    for (int k = sp.part * 64 + lane; k < cn; k += 64 * sp.wpt) {
      const int kk = cb + k;
      double2 v = bin[b.bidx[c0 + kk]];
      for_children(b, frow0 + kk, [&](int i) {
        const double2 u = ub[i];
        v.x -= u.x;
        v.y -= u.y;
      });
      vt[k] = v;
    }
    __syncthreads();
    {
      const int per = sp.share(cn);
      const int k0 = cb + sp.part * per, k1 = min(cb + cn, k0 + per);
      const Panel<PT> p(rs, bytes, t.nrows, k0, k1, l, l.row < t.nrows && l.grp < l.G, 0, t.row0 + l.row < w ? t.row0 + l.row + 1 : t.ncols);
      PT a[8];
      tile_load(p, a);
      if (p.n > 0) tile_dot(p, vt + (k0 - cb + l.grp), l.G, cn - 1 - (k0 - cb + l.grp), a, ar, ai);
    }
    __syncthreads();
  }
  red[wv][lane] = make_double2(ar, ai);
  __syncthreads();
  if (out) {
    double rr = 0, ii = 0;
    for (int q = 0; q < sp.wpt; ++q)
      for (int g = lane; g < l.G * l.R; g += l.R) {
        rr += red[wv + q][g].x;
        ii += red[wv + q][g].y;
      }
    if (row < w)
      reinterpret_cast<double2*>(b.y)[c0 + row] = make_double2(rr, ii);
    else
      reinterpret_cast<double2*>(b.ubuf)[uo] = make_double2(rr + er, ii + ei);
  }
}

template <class PT>
__device__ __forceinline__ void bwd_task(const Task& task, const Batch& b, double2* vin, double2 (*red)[64],
                                         int chunk) {
  const Split sp = split_of(task.wpt, task.ntile, chunk);
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  Tile t{};
  if (sp.has) t = b.tb[task.tile0 + sp.my];
  const int c0 = t.c0, w = t.w;
  const int64_t roff = t.aux;
  double2* vt = vin + sp.my * sp.region;
  const Lanes l(t.nrows);
  const int bytes = t.nrows * t.ncols * (int)sizeof(PT);
  const __amdgpu_buffer_rsrc_t rs = panel_rsrc(b.pb, t.off * (int64_t)sizeof(PT), bytes);
  const double2* __restrict__ yv = reinterpret_cast<const double2*>(b.y);
  const double2* xv = reinterpret_cast<const double2*>(b.x);
  double ar = 0, ai = 0;
  for (int cb = 0; cb == 0 || (sp.wpt == 4 && cb < t.ncols); cb += sp.region) {
    const int cn = sp.has ? min(sp.region, t.ncols - cb) : 0;
    for (int k = sp.part * 64 + lane; k < cn; k += 64 * sp.wpt) {
      const int c = t.col0 + cb + k;
      vt[k] = c < w ? yv[c0 + c] : xv[b.rows[roff + (c - w)]];
    }
    __syncthreads();
    {
      const int per = sp.share(cn);
      const int k0 = cb + sp.part * per, k1 = min(cb + cn, k0 + per);
      const Panel<PT> p(rs, bytes, t.nrows, k0, k1, l, l.row < t.nrows && l.grp < l.G, l.row, t.ncols);
      PT a[8];
      tile_load(p, a);
      if (p.n > 0) tile_dot(p, vt + (k0 - cb + l.grp), l.G, cn - 1 - (k0 - cb + l.grp), a, ar, ai);
    }
    __syncthreads();
  }
  red[wv][lane] = make_double2(ar, ai);
  __syncthreads();
  if (sp.has && sp.part == 0 && lane < t.nrows) {
    double rr = 0, ii = 0;
    for (int q = 0; q < sp.wpt; ++q)
      for (int g = lane; g < l.G * l.R; g += l.R) {
        rr += red[wv + q][g].x;
        ii += red[wv + q][g].y;
      }
    reinterpret_cast<double2*>(b.x)[c0 + t.row0 + lane] = make_double2(rr, ii);
  }
}

// The input-column buffer is dynamic LDS sized per level (chunk entries), so
// levels of narrow tiles keep more workgroups resident per CU.
// The grid holds at most as many workgroups as fit on the device at once;
// each sweeps tasks blockIdx.x, blockIdx.x + gridDim.x, ... (widest first),
// so a level costs no workgroup launches beyond the first wave of them.
// Complex64 panels: five workgroups per CU.  Local solves with six / five / four
// registers' worth: one million unknowns in 64 subdomains 2.004 / 1.992 / 1.984 ms,
// in 16 2.144 / 2.104 / 2.113, 608,375 unknowns in 20 1.098 / 1.036 / 1.041 (six
// hold too few loads in flight per wave where the upper levels have few tiles).
// Complex128 panels: four (six: 3.65 -> 3.69 ms for the two-level preconditioner).
template <class PT, int kCoarse>
__global__ __launch_bounds__(kWG, sizeof(PT) == 8 ? 5 : 4) void fwd_level_kernel(const Task* __restrict__ tasks, int ntasks, Batch b,
                                                        const double2* __restrict__ bin, int chunk) {
  extern __shared__ double2 vin[];
  __shared__ double2 red[4][64];
  for (int t = blockIdx.x; t < ntasks; t += gridDim.x) {
    fwd_task<PT>(tasks[t], b, bin, vin, red, chunk);
    __syncthreads();  // red and vin are rewritten by the next task
  }
}

template <class PT, int kCoarse>
__global__ __launch_bounds__(kWG, sizeof(PT) == 8 ? 5 : 4) void bwd_level_kernel(const Task* __restrict__ tasks, int ntasks, Batch b,
                                                        int chunk) {
  extern __shared__ double2 vin[];
  __shared__ double2 red[4][64];
  for (int t = blockIdx.x; t < ntasks; t += gridDim.x) {
    bwd_task<PT>(tasks[t], b, vin, red, chunk);
    __syncthreads();
  }
}

// ---- both sweeps in one launch ----------------------------------------------
// A sweep level by level costs a launch per level, and every level ends in a
// tail of a few workgroups while the next one's panels wait; on an operator
// whose levels do not fill the device several times over that is most of the
// time.  Here one launch takes all tasks of both sweeps, of all batches, in
// level order.  A workgroup draws the next task from a counter (and its record
// one task ahead), loads what does not depend on other tasks (indices, inputs
// from the caller, the first panel columns), waits for the tiles it does
// depend on, and streams its panel.
//
// Dependencies: counters per supernode.  A forward tile waits until every
// forward tile of its supernode's children has finished (they hold the
// updates it gathers), a backward tile until every backward tile of the parent
// has (the ancestors' results are then complete, since the parent waited for
// its own parent), a root's backward tiles for its forward tiles.  A sweep
// raises each counter from zero to a known amount.  The kernel that follows it
// on its stream (prolongation, coarse update) clears counters and state for the
// next one and counts a generation (flow_clear), so eager and captured launches
// may alternate, and no sweep depends on how an earlier one went: applications of
// one context that overlap, which the callers have to order, draw from one ticket
// and spoil each other's results, but the last clear comes after all of them.  A
// sweep cleared under a wait sees the generation change and gives up.  (With
// counters that ran on from sweep to sweep, an overlap left them off their targets
// for the life of the context.)
//
// Progress: a task's dependencies have smaller numbers, and numbers are drawn
// in order by workgroups already running, so the smallest unfinished task
// never waits for one that no workgroup holds, whatever the number of
// resident workgroups.  The wait is bounded all the same; a workgroup that
// gives up writes NaN, which the solvers report.
//
// Memory: what tasks pass to each other (y, x, the update vectors) is written
// and read with agent-scope accesses, coherent across the XCDs' L2s without
// writing back or invalidating them; a wave adds to a counter once its stores
// have completed.  Everything else is constant during the launch.
//
// Measured (MI355X): one hop between workgroups (poll, load, store, add) 1.06
// us, a level of the 16,810-unknown coarse solve 9 us against 11 us with a
// launch per level (coarse correction 194 -> 168 us), the local solves of
// 4,913 unknowns in 8 subdomains 156 -> 71 us, of 168,075 unknowns in 30
// (complex64 panels, 1.05 GB) 461 -> 330 us (76 and 345 us with the input
// indices in LDS and a loop of dependent loads after the wait, instead of
// registers and four loads at once).  What bounds it now is the chain
// of latencies in a task (indices, inputs, hop, children's updates, panel,
// reduction, stores), about 5 us per level on the small operator.
constexpr int kFlowPolls = 1 << 20;  // about a second, a thousand times the longest sweep

__device__ __forceinline__ double2 ld_agent(const double2* p) {
  const double* d = reinterpret_cast<const double*>(p);
  return make_double2(__hip_atomic_load(d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                      __hip_atomic_load(d + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void st_agent(double2* p, double2 v) {
  double* d = reinterpret_cast<double*>(p);
  __hip_atomic_store(d, v.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(d + 1, v.y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t cnt_load(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t cnt_add(uint32_t* p) {
  return __hip_atomic_fetch_add(p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void cnt_store(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Clears the counters and the state of a sweep that has ended (thread id of
// nthreads of the kernel after it; one store per thread and counter).
__device__ __forceinline__ void flow_clear(const FlowState& f, int64_t id, int64_t nthreads) {
  if (id >= f.counters) return;
  for (int64_t k = id; k < f.counters; k += nthreads) cnt_store(f.cnt + kFlowHead + kFlowPad * k, 0u);
  if (id == 0) {
    cnt_store(f.cnt + kFlowTicket, 0u);
    cnt_store(f.cnt + kFlowTicket + 1, 0u);
    cnt_store(f.cnt + kFlowGaveUp, 0u);
  }
  if (threadIdx.x == 0) cnt_add(f.cnt + kFlowGeneration);  // every workgroup that cleared something
}

// Waits until the counters of the task's tiles have reached their targets:
// lane u of the first wave polls tile u's counter, since a thousand workgroups
// polling from every wave slow down the additions they wait for (same-address
// traffic: 11 ns per access).  False if it gave up.
__device__ __forceinline__ bool flow_wait(const FlowTask& task, uint32_t* cnt, uint32_t generation) {
  const int u = threadIdx.x;
  const int32_t c = u < 4 ? task.t[u].wait : -1;
  const uint32_t target = u < 4 ? task.t[u].need : 0;
  const uint32_t* p = cnt + kFlowHead + (int64_t)kFlowPad * c;
  for (int i = 0; i < kFlowPolls; ++i) {
    bool done = true;
    if (c >= 0) done = cnt_load(p) >= target;
    if (__all(done)) return true;
    if ((i & 255) == 255) {
      if (cnt_load(cnt + kFlowGaveUp)) return false;
      if (cnt_load(cnt + kFlowGeneration) != generation) break;
    }
    __builtin_amdgcn_s_sleep(1);
  }
  cnt_store(cnt + kFlowGaveUp, 1u);
  return false;
}

// Sum over the children's update entries of front row fr, whose index pair
// is c (list order, as for_children).
__device__ __forceinline__ double2 flow_children(const FlowBatch& b, int fr, int2 c) {
  const double2* ub = reinterpret_cast<const double2*>(b.ubuf);
  double2 e = make_double2(0.0, 0.0);
  if (c.x >= 0) {
    e = ld_agent(ub + c.x);
    if (c.y >= 0) {
      const double2 u = ld_agent(ub + c.y);
      e.x += u.x;
      e.y += u.y;
    }
  } else if (c.x < -1) {
    for (int q = -2 - c.x; q < b.fcon_ptr[fr + 1]; ++q) {
      const double2 u = ld_agent(ub + b.fcon_idx[q]);
      e.x += u.x;
      e.y += u.y;
    }
  }
  return e;
}

// task: in LDS.  nx: the number drawn for the next task (first lane of the
// workgroup); *word: this lane's word of that task's record (first wave).
template <class PT, bool kBwd>
__device__ __forceinline__ void flow_task(const FlowTask& task, const FlowArgs& a, const FlowBatch& b,
                                          const double2* __restrict__ bin, double2* vin,
                                          double2 (*red)[64], int* gave_up, uint32_t generation, int nx_bound, uint32_t nx,
                                          const FlowTask* __restrict__ tasks, uint32_t& word) {
  const int lane = threadIdx.x & 63, wv = uni(threadIdx.x >> 6);
  const Split sp = split_of(uni(task.t[0].wpt), 4, a.chunk);
  const int wpt = sp.wpt, part = sp.part, region = sp.region;
  const FlowTile& t = task.t[sp.my];
  const int nrows = uni(t.nrows), ncols = uni(t.ncols), ld = uni(t.ld), c0 = uni(t.c0), w = uni(t.w), aux = uni(t.aux),
            col0 = uni(t.col0), row0 = uni(t.row0);
  const bool waits = uni(task.t[0].waits) != 0;
  double2* vt = vin + sp.my * region;
  const Lanes l(nrows);
  const int bytes = ncols > 0 ? ((ncols - 1) * ld + nrows) * (int)sizeof(PT) : 0;
  const __amdgpu_buffer_rsrc_t rs = panel_rsrc(kBwd ? b.pb : b.pf, t.off * (int64_t)sizeof(PT), bytes);
  const double2* __restrict__ ub = reinterpret_cast<const double2*>(b.ubuf);
  const bool out = part == 0 && lane < nrows;
  const bool dots = l.row < nrows && l.grp < l.G;
  const int row = row0 + lane;
  const bool upd = !kBwd && out && row >= w;
  const bool many = wpt == 4 && ncols > region;  // several passes
  const int ks = part * 64 + lane, kst = 64 * wpt;
  const int2 co = upd ? b.fcon2[aux + row] : make_int2(-1, -1);
  double er = 0, ei = 0;
  double ar = 0, ai = 0;
  for (int cb = 0; cb == 0 || (many && cb < ncols); cb += region) {
    const int cn = min(region, ncols - cb);
    // before the wait: the indices of this pass's inputs (at most four per
    // lane), the caller's entries (forward), and the first eight panel
    // columns of every lane
    int2 ci[4];
    double2 v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = ks + q * kst;
      ci[q] = make_int2(-1, -1);
      v[q] = make_double2(0.0, 0.0);
      if (k >= cn) continue;
      if (kBwd) {
        const int c = col0 + cb + k;
        ci[q].x = c < w ? c0 + c : -1 - b.rows[(int64_t)aux + (c - w)];
      } else {
        ci[q] = b.fcon2[aux + cb + k];
        v[q] = bin[b.bidx[c0 + cb + k]];
      }
    }
    const int per = sp.share(cn);
    const int kb = cb + part * per, ke = min(cb + cn, kb + per);
    // forward pivot rows end at the diagonal, backward rows begin there
    const Panel<PT> p(rs, bytes, ld, kb, ke, l, dots, kBwd ? l.row : 0,
                      !kBwd && row0 + l.row < w ? row0 + l.row + 1 : ncols);
    PT pre[8];
    tile_load(p, pre);
    if (cb == 0) {
      if (waits) {
        if (wv == 0) {
          const bool ok = flow_wait(task, a.cnt, generation);
          if (lane == 0) *gave_up = ok ? 0 : 1;
        }
        __syncthreads();
      }
      asm volatile("" ::: "memory");  // no load of the other tasks' results above the wait
      if (upd) {
        const double2 e = flow_children(b, aux + row, co);
        er = e.x;
        ei = e.y;
      }
    }
    // then the other tasks' results, all loads before the first use
    if (kBwd) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (ks + q * kst < cn)
          v[q] = ld_agent(ci[q].x >= 0 ? reinterpret_cast<const double2*>(b.y) + ci[q].x
                                       : reinterpret_cast<const double2*>(b.x) + (-1 - ci[q].x));
    } else {
      double2 u[4], u2[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (ci[q].x >= 0) u[q] = ld_agent(ub + ci[q].x);
        if (ci[q].x >= 0 && ci[q].y >= 0) u2[q] = ld_agent(ub + ci[q].y);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (ci[q].x >= 0) {
          v[q].x -= u[q].x;
          v[q].y -= u[q].y;
          if (ci[q].y >= 0) {
            v[q].x -= u2[q].x;
            v[q].y -= u2[q].y;
          }
        } else if (ci[q].x < -1) {
          for (int e = -2 - ci[q].x; e < b.fcon_ptr[aux + cb + ks + q * kst + 1]; ++e) {
            const double2 x = ld_agent(ub + b.fcon_idx[e]);
            v[q].x -= x.x;
            v[q].y -= x.y;
          }
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (ks + q * kst < cn) vt[ks + q * kst] = v[q];
    if (cb == 0 && wv == 0) {  // the next task's record
      const int n = uni((int)nx);
      if (n < nx_bound) word = reinterpret_cast<const uint32_t*>(tasks + n)[lane];
    }
    __syncthreads();
    if (p.n > 0) tile_dot(p, vt + (kb - cb + l.grp), l.G, cn - 1 - (kb - cb + l.grp), pre, ar, ai);
    if (many) __syncthreads();
  }
  red[wv][lane] = make_double2(ar, ai);
  __syncthreads();
  if (nrows > 0 && part == 0) {
    if (out) {
      double rr = 0, ii = 0;
      for (int q = 0; q < wpt; ++q)
        for (int g = lane; g < l.G * l.R; g += l.R) {
          rr += red[wv + q][g].x;
          ii += red[wv + q][g].y;
        }
      if (waits && *gave_up) rr = ii = __builtin_nan("");
      double2* dst;
      if (kBwd)
        dst = reinterpret_cast<double2*>(b.x) + c0 + row;
      else
        dst = row < w ? reinterpret_cast<double2*>(b.y) + c0 + row
                      : reinterpret_cast<double2*>(b.ubuf) + t.uoff + (row - w);
      st_agent(dst, make_double2(rr + er, ii + ei));
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the stores have reached the coherence point
    if (lane == 0) cnt_add(a.cnt + kFlowHead + (int64_t)kFlowPad * t.sig);
  }
}

// Three workgroups per CU: a fourth (128 registers) made the chains longer, 339
// against 328 us for 168,075 unknowns.
template <class PT, int kCoarse>
__global__ __launch_bounds__(kWG, 3) void flow_kernel(FlowArgs a, int t0, int t1, int ticket_word,
                                                   const double2* __restrict__ bin) {
  extern __shared__ double2 vin[];
  __shared__ double2 red[4][64];
  __shared__ FlowTask rec[2];
  __shared__ int next, gave_up;
  const FlowTask* __restrict__ tasks = a.tasks + t0;
  const int n = t1 - t0;
  const uint32_t generation = uni((int)cnt_load(a.cnt + kFlowGeneration));
  uint32_t* const ticket = a.cnt + ticket_word;
  if (threadIdx.x < 64) {
    uint32_t d = 0;
    if (threadIdx.x == 0) next = (int)(d = cnt_add(ticket));
    const int t = uni((int)d);
    if (t < n)
      reinterpret_cast<uint32_t*>(&rec[0])[threadIdx.x] = reinterpret_cast<const uint32_t*>(tasks + t)[threadIdx.x];
  }
  __syncthreads();
  int t = uni(next);
  for (int cur = 0; t < n; cur ^= 1) {
    // the next task is drawn, and its record loaded, while this one runs
    uint32_t nx = 0, word = 0;
    if (threadIdx.x == 0) nx = cnt_add(ticket);
    const FlowTask& task = rec[cur];
    const FlowBatch& b = a.b[uni(task.t[0].batch)];
    if (uni(task.t[0].bwd))
      flow_task<PT, true>(task, a, b, bin, vin, red, &gave_up, generation, n, nx, tasks, word);
    else
      flow_task<PT, false>(task, a, b, bin, vin, red, &gave_up, generation, n, nx, tasks, word);
    if (threadIdx.x < 64) reinterpret_cast<uint32_t*>(&rec[cur ^ 1])[threadIdx.x] = word;
    if (threadIdx.x == 0) next = (int)nx;
    __syncthreads();  // vin and red are rewritten by the next task
    t = uni(next);
  }
}

// Forward solve of narrow supernodes (w <= 64), one wave per supernode.
// Lane k holds gathered input k; lane l owns row l of every 64-row tile, and
// the wave streams up to four tiles side by side (column k of each), so a
// supernode's whole panel is one stream of loads after a single gather.
__device__ __forceinline__ double bcast(double x, int k) {
  const long long v = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)v, k);
  const int hi = __builtin_amdgcn_readlane((int)(v >> 32), k);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// acc[q] += tile q (rows lane, columns 0..w-1) * v, NQ tiles at byte offset
// 64 q w of the buffer (tile q has rows[q] rows, none for q >= nq), eight loads
// in flight per lane.  Lanes past a tile's last row skip their loads, and in
// the first tile (diag) the lanes above the diagonal.
template <class PT, int NQ>
__device__ __forceinline__ void sn_stream(__amdgpu_buffer_rsrc_t r, int bytes, int w, const int* rows, bool diag, double2 v,
                                          double2* acc) {
  constexpr int KU = 8 / NQ, esz = (int)sizeof(PT);
  const int lane = threadIdx.x & 63;
  for (int k = 0; k < w; k += KU) {
    PT a[KU][NQ];
#pragma unroll
    for (int u = 0; u < KU; ++u)
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const bool on = lane < rows[q] && k + u < w && !(q == 0 && diag && lane < k + u);
        a[u][q] = ldb<PT>(r, on ? lane * esz : kBufSkip, min((q * 64 * w + (k + u) * rows[q]) * esz, bytes));
      }
#pragma unroll
    for (int u = 0; u < KU; ++u) {
      if (k + u >= w) break;
      const double2 x = make_double2(bcast(v.x, k + u), bcast(v.y, k + u));
#pragma unroll
      for (int q = 0; q < NQ; ++q) cfma(acc[q].x, acc[q].y, widen(a[u][q]), x);
    }
  }
}

template <class PT>
__global__ __launch_bounds__(kWG) void fwd_sn_kernel(const SnJob* __restrict__ jobs, int njobs, Batch b,
                                                     const double2* __restrict__ bin) {
  const int lane = threadIdx.x & 63;
  const double2* __restrict__ ub = reinterpret_cast<const double2*>(b.ubuf);
  // the job index is wave-uniform, so the job lives in scalar registers
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int j = blockIdx.x * 4 + wave; j < njobs; j += gridDim.x * 4) {
    const SnJob jb = jobs[j];
    const int m = jb.m, w = jb.w;
    // inputs: restricted right-hand side minus the children's updates
    double2 v = make_double2(0.0, 0.0);
    if (lane < w) {
      v = bin[b.bidx[jb.c0 + lane]];
      for_children(b, jb.frow0 + lane, [&](int i) {
        const double2 u = ub[i];
        v.x -= u.x;
        v.y -= u.y;
      });
    }
    for (int q0 = 0; q0 * 64 < m; q0 += 4) {
      const int nq = min(4, (m - q0 * 64 + 63) / 64);
      int rows[4];
      double2 acc[4];
      // rows past the pivot block start from the children's updates
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        rows[q] = q < nq ? min(64, m - (q0 + q) * 64) : 0;
        acc[q] = make_double2(0.0, 0.0);
        const int row = (q0 + q) * 64 + lane;
        if (q < nq && lane < rows[q] && row >= w)
          for_children(b, jb.frow0 + row, [&](int i) {
            const double2 u = ub[i];
            acc[q].x += u.x;
            acc[q].y += u.y;
          });
      }
      const int bytes = min(256, m - q0 * 64) * w * (int)sizeof(PT);
      const __amdgpu_buffer_rsrc_t rs =
          panel_rsrc(b.pf, (jb.off + (int64_t)q0 * 64 * w) * (int64_t)sizeof(PT), bytes);
      if (nq == 1)
        sn_stream<PT, 1>(rs, bytes, w, rows, q0 == 0, v, acc);
      else if (nq == 2)
        sn_stream<PT, 2>(rs, bytes, w, rows, q0 == 0, v, acc);
      else
        sn_stream<PT, 4>(rs, bytes, w, rows, q0 == 0, v, acc);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = (q0 + q) * 64 + lane;
        if (q < nq && lane < rows[q]) {
          if (row < w)
            reinterpret_cast<double2*>(b.y)[jb.c0 + row] = acc[q];
          else
            reinterpret_cast<double2*>(b.ubuf)[jb.uoff + row - w] = acc[q];
        }
      }
    }
  }
}

// Whole forward + backward solve of a small batch (the coarse matrix) in one
// cooperative launch: the workgroups sweep each level's tasks and meet at a
// grid-wide barrier before the next level, instead of one launch per level.
__global__ __launch_bounds__(kWG) void batch_solve_coop_kernel(Batch b, const double2* __restrict__ bin,
                                                               LevelRanges lv) {
  __shared__ double2 vin[kChunk];
  __shared__ double2 red[4][64];
  cooperative_groups::grid_group grid = cooperative_groups::this_grid();
  for (int l = 0; l < lv.nf; ++l) {
    for (int64_t t = lv.f[l] + blockIdx.x; t < lv.f[l + 1]; t += gridDim.x) {
      fwd_task<double2>(b.kf[t], b, bin, vin, red, kChunk);
      __syncthreads();
    }
    grid.sync();
  }
  for (int l = 0; l < lv.nb; ++l) {
    for (int64_t t = lv.b[l] + blockIdx.x; t < lv.b[l + 1]; t += gridDim.x) {
      bwd_task<double2>(b.kb[t], b, vin, red, kChunk);
      __syncthreads();
    }
    grid.sync();
  }
}

// One row of a CSR matrix per G lanes; each lane takes U entries per pass
// (entries base + u G + lane), loading all U columns, then all U values and
// x entries before the multiply-adds, so a wave keeps U gathers in flight
// instead of one dependent col -> x chain per entry.  With kXcd, workgroup b
// runs on XCD b % 8 (workgroups are dealt round-robin) and takes the
// (b / 8)-th block of that XCD's row range [xr[b % 8], xr[b % 8 + 1]).
// Entries are complex (VT = double2), or real parts and imaginary parts
// stored as separate real entries (VT = double): an imaginary entry carries
// bit 31 in its column index and multiplies i x[col].  A of the Helmholtz
// problem is complex only on the absorbing boundary, so the split storage
// moves 12 B per entry instead of 20 B.
template <class VT>
__device__ __forceinline__ void spmv_fma(double& ar, double& ai, int c, VT v, const double2* __restrict__ x);
template <>
__device__ __forceinline__ void spmv_fma<double2>(double& ar, double& ai, int c, double2 v,
                                                  const double2* __restrict__ x) {
  cfma(ar, ai, v, x[c]);
}
template <>
__device__ __forceinline__ void spmv_fma<double>(double& ar, double& ai, int c, double v,
                                                 const double2* __restrict__ x) {
  const double2 xv = x[c & 0x7fffffff];
  const bool im = c < 0;  // i x = (-x.y, x.x)
  ar = fma(v, im ? -xv.y : xv.x, ar);
  ai = fma(v, im ? xv.x : xv.y, ai);
}

template <int G, int U, bool kXcd, class VT>
__global__ __launch_bounds__(kWG) void spmv_kernel(int64_t n, const int64_t* __restrict__ ptr,
                                                   const int32_t* __restrict__ col, const VT* __restrict__ val,
                                                   const int64_t* __restrict__ xr, const double2* __restrict__ x,
                                                   const double2* __restrict__ bvec, double2* __restrict__ y) {
  int64_t row, end = n;
  if (kXcd) {
    row = xr[blockIdx.x & 7] + ((int64_t)(blockIdx.x >> 3) * kWG + threadIdx.x) / G;
    end = xr[(blockIdx.x & 7) + 1];
  } else {
    row = ((int64_t)blockIdx.x * kWG + threadIdx.x) / G;
  }
  const int l = threadIdx.x % G;
  double ar = 0, ai = 0;
  if (row < end) {
    const int64_t p1 = ptr[row + 1];
    for (int64_t base = ptr[row] + l; base < p1; base += G * U) {
      int c[U];
      VT v[U];
      bool ok[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        ok[u] = base + u * G < p1;
        c[u] = ok[u] ? col[base + u * G] : 0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = ok[u] ? val[base + u * G] : VT{};
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (ok[u]) spmv_fma<VT>(ar, ai, c[u], v[u], x);
    }
  }
#pragma unroll
  for (int o = G / 2; o > 0; o >>= 1) {
    ar += __shfl_xor(ar, o, G);
    ai += __shfl_xor(ai, o, G);
  }
  if (row < end && l == 0) {
    if (bvec) {
      double2 bb = bvec[row];
      y[row] = make_double2(bb.x - ar, bb.y - ai);
    } else {
      y[row] = make_double2(ar, ai);
    }
  }
}

// Sliced ELL (slices of 64 rows = one wavefront): slice s holds rows
// perm[64 s .. 64 s + 63], padded to the slice's longest row, stored
// column-major inside the slice so each lane owns a row and every load of a
// wave is one contiguous 1 KiB (values) / 256 B (columns) line.
__global__ __launch_bounds__(kWG) void sell_kernel(int64_t n, int64_t nslices, const int64_t* __restrict__ soff,
                                                   const int32_t* __restrict__ swidth,
                                                   const int32_t* __restrict__ perm, const int32_t* __restrict__ col,
                                                   const double2* __restrict__ val, const double2* __restrict__ x,
                                                   const double2* __restrict__ bvec, double2* __restrict__ y) {
  // XCD-aware order: workgroups are dealt round-robin to the 8 XCDs, so
  // workgroup b works on block (b % 8) * per + b / 8 and every XCD sweeps a
  // contiguous eighth of the rows (their x entries stay in its own L2)
  const unsigned per = gridDim.x / 8;
  const int64_t vb = (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
  const int64_t s = vb * (kWG / 64) + (threadIdx.x >> 6);
  if (s >= nslices) return;
  const int lane = threadIdx.x & 63;
  const int64_t slot = s * 64 + lane;
  const int64_t off = soff[s] + lane;
  const int wdt = swidth[s];
  double ar = 0, ai = 0, br = 0, bi = 0;
  int j = 0;
  for (; j + 4 <= wdt; j += 4) {
    const int c0 = col[off + (int64_t)(j + 0) * 64], c1 = col[off + (int64_t)(j + 1) * 64];
    const int c2 = col[off + (int64_t)(j + 2) * 64], c3 = col[off + (int64_t)(j + 3) * 64];
    const double2 v0 = val[off + (int64_t)(j + 0) * 64], v1 = val[off + (int64_t)(j + 1) * 64];
    const double2 v2 = val[off + (int64_t)(j + 2) * 64], v3 = val[off + (int64_t)(j + 3) * 64];
    cfma(ar, ai, v0, x[c0]);
    cfma(br, bi, v1, x[c1]);
    cfma(ar, ai, v2, x[c2]);
    cfma(br, bi, v3, x[c3]);
  }
  for (; j < wdt; ++j) cfma(ar, ai, val[off + (int64_t)j * 64], x[col[off + (int64_t)j * 64]]);
  ar += br;
  ai += bi;
  if (slot >= n) return;
  const int row = perm[slot];
  if (bvec) {
    const double2 bb = bvec[row];
    y[row] = make_double2(bb.x - ar, bb.y - ai);
  } else {
    y[row] = make_double2(ar, ai);
  }
}

template <int G>
__global__ __launch_bounds__(kWG) void spmv_real_kernel(int64_t n, const int64_t* __restrict__ ptr,
                                                        const int32_t* __restrict__ col,
                                                        const double* __restrict__ val,
                                                        const double2* __restrict__ x, double2* __restrict__ y,
                                                        FlowState done) {
  const int64_t id = (int64_t)blockIdx.x * kWG + threadIdx.x;
  flow_clear(done, id, (int64_t)gridDim.x * kWG);
  const int64_t row = id / G;
  const int l = threadIdx.x % G;
  double ar = 0, ai = 0;
  if (row < n) {
    const int64_t p1 = ptr[row + 1];
    for (int64_t p = ptr[row] + l; p < p1; p += G) {
      double a = val[p];
      double2 v = x[col[p]];
      ar = fma(a, v.x, ar);
      ai = fma(a, v.y, ai);
    }
  }
#pragma unroll
  for (int o = G / 2; o > 0; o >>= 1) {
    ar += __shfl_xor(ar, o, G);
    ai += __shfl_xor(ai, o, G);
  }
  if (row < n && l == 0) y[row] = make_double2(ar, ai);
}

// Both fine-grid products of the coarse solution cx, row by row (G lanes
// per row): q = Z cx (real Z) and t = r - (A Z) cx, A Z in split storage
// (real entries; bit 31 of the column marks an imaginary part).
template <int G>
__global__ __launch_bounds__(kWG) void coarse_update_kernel(int64_t n, const int64_t* __restrict__ zptr,
                                                            const int32_t* __restrict__ zcol,
                                                            const double* __restrict__ zval,
                                                            const int64_t* __restrict__ aptr,
                                                            const int32_t* __restrict__ acol,
                                                            const double* __restrict__ aval,
                                                            const double2* __restrict__ cx,
                                                            const double2* __restrict__ r, double2* __restrict__ q,
                                                            double2* __restrict__ t, FlowState done) {
  const int64_t id = (int64_t)blockIdx.x * kWG + threadIdx.x;
  flow_clear(done, id, (int64_t)gridDim.x * kWG);
  const int64_t row = id / G;
  const int l = threadIdx.x % G;
  double qr = 0, qi = 0, ar = 0, ai = 0;
  if (row < n) {
    const int64_t z1 = zptr[row + 1], a1 = aptr[row + 1];
    for (int64_t p = zptr[row] + l; p < z1; p += G) {
      const double z = zval[p];
      const double2 v = cx[zcol[p]];
      qr = fma(z, v.x, qr);
      qi = fma(z, v.y, qi);
    }
    for (int64_t p = aptr[row] + l; p < a1; p += G) spmv_fma<double>(ar, ai, acol[p], aval[p], cx);
  }
#pragma unroll
  for (int o = G / 2; o > 0; o >>= 1) {
    qr += __shfl_xor(qr, o, G);
    qi += __shfl_xor(qi, o, G);
    ar += __shfl_xor(ar, o, G);
    ai += __shfl_xor(ai, o, G);
  }
  if (row < n && l == 0) {
    q[row] = make_double2(qr, qi);
    const double2 rr = r[row];
    t[row] = make_double2(rr.x - ar, rr.y - ai);
  }
}

__global__ __launch_bounds__(kWG) void prolong_kernel(int64_t n, const int64_t* __restrict__ ptr,
                                                      const int32_t* __restrict__ idx, const double* __restrict__ w,
                                                      const double2* __restrict__ xl, const double2* __restrict__ q,
                                                      double2* __restrict__ z, FlowState done) {
  const int64_t g = (int64_t)blockIdx.x * kWG + threadIdx.x;
  flow_clear(done, g, (int64_t)gridDim.x * kWG);
  if (g >= n) return;
  double ar = 0, ai = 0;
  if (q) {
    ar = q[g].x;
    ai = q[g].y;
  }
  for (int64_t p = ptr[g]; p < ptr[g + 1]; ++p) {
    double2 v = xl[idx[p]];
    double c = w[p];
    ar = fma(c, v.x, ar);
    ai = fma(c, v.y, ai);
  }
  z[g] = make_double2(ar, ai);
}

// ---- Gram-Schmidt ----------------------------------------------------------

__global__ __launch_bounds__(kWG) void gs_dots_final_kernel(PtrSetC parts, int nblk, int ncol, PtrSet hs_, PtrSet haccs,
                                                            int accumulate) {
  __shared__ double2 sm[kWG];
  const double2* __restrict__ partial = reinterpret_cast<const double2*>(parts.p[blockIdx.y]);
  double2* __restrict__ h = reinterpret_cast<double2*>(hs_.p[blockIdx.y]);
  double2* __restrict__ hacc = reinterpret_cast<double2*>(haccs.p[blockIdx.y]);
  const int k = blockIdx.x, tid = threadIdx.x;
  double ar = 0, ai = 0;
  for (int b = tid; b < nblk; b += kWG) {
    double2 v = partial[(int64_t)b * ncol + k];
    ar += v.x;
    ai += v.y;
  }
  sm[tid] = make_double2(ar, ai);
  __syncthreads();
  for (int st = kWG / 2; st > 0; st >>= 1) {
    if (tid < st) {
      sm[tid].x += sm[tid + st].x;
      sm[tid].y += sm[tid + st].y;
    }
    __syncthreads();
  }
  if (tid == 0) {
    h[k] = sm[0];
    if (hacc) {
      if (accumulate)
        hacc[k] = make_double2(hacc[k].x + sm[0].x, hacc[k].y + sm[0].y);
      else
        hacc[k] = sm[0];
    }
  }
}

// One CGS2 pass over a 64-row tile of V (all ncol columns staged in LDS,
// padded to avoid bank conflicts):
//   kUpdate: w -= V h                (h: device, ncol entries)
//   kDots:   partial[blk*ncol + k] = sum_rows conj(V[i,k]) w[i]
//   kNorm:   partial[blk] = sum_rows |w[i]|^2   (real, stored in .x)
constexpr int kGsRows = 64;
constexpr int kGsMaxCols = 64;

template <bool kUpdate, bool kDots, bool kNorm>
__global__ __launch_bounds__(kWG) void gs_pass_kernel(int64_t n, PtrSetC Vs, int64_t ld, int ncol, PtrSetC hs_,
                                                      PtrSet ws, PtrSet parts) {
  // right-hand side blockIdx.y
  const double2* __restrict__ V = reinterpret_cast<const double2*>(Vs.p[blockIdx.y]);
  const double2* __restrict__ h = reinterpret_cast<const double2*>(hs_.p[blockIdx.y]);
  double2* __restrict__ w = reinterpret_cast<double2*>(ws.p[blockIdx.y]);
  double2* __restrict__ partial = reinterpret_cast<double2*>(parts.p[blockIdx.y]);
  // dynamic LDS: tile[ncol][kGsRows + 1], then h, the new w, and the
  // per-wave partial sums of the update and of the dots
  extern __shared__ double2 lds[];
  double2 (*tile)[kGsRows + 1] = reinterpret_cast<double2 (*)[kGsRows + 1]>(lds);
  double2* hs = lds + (size_t)ncol * (kGsRows + 1);
  double2* wn = hs + kGsMaxCols;
  double2* ured = wn + kGsRows;         // [4][kGsRows]
  double2* dred = ured + 4 * kGsRows;   // [4][kGsMaxCols]
  double* red = reinterpret_cast<double*>(dred + 4 * kGsMaxCols);
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (kUpdate && tid < ncol) hs[tid] = h[tid];
  double dr = 0, di = 0;  // dots: column `lane`, rows [16 wv, 16 wv + 16) of every tile
  double nrm = 0;         // norm: row `tid` of every tile
  const int64_t ntiles = (n + kGsRows - 1) / kGsRows;
  // Software pipeline: wave q holds columns q, q + 4, ... of the next tile
  // (and wave 0 the next tile's w) in registers; they are loaded right after
  // the current tile is staged, so the loads overlap its arithmetic.
  constexpr int kU = kGsMaxCols / 4;
  double2 a[kU];
  double2 wnext = make_double2(0.0, 0.0);
  auto load_next = [&](int64_t tb) {
    const int64_t i = tb * kGsRows + lane;
    const bool valid = tb < ntiles && i < n;
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int k = wv + 4 * u;
      a[u] = (k < ncol && valid) ? V[(int64_t)k * ld + i] : make_double2(0.0, 0.0);
    }
    if (tid < kGsRows) wnext = valid ? w[i] : make_double2(0.0, 0.0);
  };
  load_next(blockIdx.x);
  for (int64_t tb = blockIdx.x; tb < ntiles; tb += gridDim.x) {
    const int64_t i = tb * kGsRows + lane;
    const bool valid = i < n;
#pragma unroll
    for (int u = 0; u < kU; ++u)
      if (wv + 4 * u < ncol) tile[wv + 4 * u][lane] = a[u];
    const double2 wcur = wnext;
    __syncthreads();
    load_next(tb + gridDim.x);
    if (kUpdate) {
      // wave q sums the columns k = q mod 4 of row `lane`
      double ur = 0, ui = 0;
      for (int k = wv; k < ncol; k += 4) cfma(ur, ui, tile[k][lane], hs[k]);
      ured[wv * kGsRows + lane] = make_double2(ur, ui);
      __syncthreads();
    }
    if (tid < kGsRows) {
      double2 wi = wcur;
      if (kUpdate) {
        for (int q = 0; q < 4; ++q) {
          wi.x -= ured[q * kGsRows + tid].x;
          wi.y -= ured[q * kGsRows + tid].y;
        }
        if (valid) w[i] = wi;
      }
      wn[tid] = wi;
      if (kNorm) nrm = fma(wi.x, wi.x, fma(wi.y, wi.y, nrm));
    }
    __syncthreads();
    if (kDots && lane < ncol) {
      for (int r = wv * 16; r < wv * 16 + 16; ++r) {
        const double2 v = tile[lane][r], x = wn[r];
        dr = fma(v.x, x.x, dr);
        dr = fma(v.y, x.y, dr);
        di = fma(v.x, x.y, di);
        di = fma(-v.y, x.x, di);
      }
    }
    __syncthreads();  // the next tile overwrites tile and wn
  }
  if (kDots) {
    if (lane < ncol) dred[wv * kGsMaxCols + lane] = make_double2(dr, di);
    __syncthreads();
    if (tid < ncol) {
      double ar = 0, ai = 0;
      for (int q = 0; q < 4; ++q) {
        ar += dred[q * kGsMaxCols + tid].x;
        ai += dred[q * kGsMaxCols + tid].y;
      }
      partial[(int64_t)blockIdx.x * ncol + tid] = make_double2(ar, ai);
    }
  }
  if (kNorm) {
    if (tid < kGsRows) red[tid] = nrm;
    __syncthreads();
    if (tid == 0) {
      double sum = 0;
      for (int r = 0; r < kGsRows; ++r) sum += red[r];
      partial[blockIdx.x] = make_double2(sum, 0.0);
    }
  }
}

// Delayed CGS2 (two passes over V per Arnoldi step instead of three): the
// last column v_j of V (ncol = j + 1 columns) was orthogonalised once when it
// was made; its second pass is folded into the next step.
// Pass A: partial dots V^H w (ncol entries) and V^H v_j (ncol more, the last
// being |v_j|^2) of every 64-row tile, staged through LDS so lane k of each
// wave sums column k over a quarter of the tile's rows;
// partial[blk * 2 ncol + k] and partial[blk * 2 ncol + ncol + k].
template <int kU>  // columns per wave (ncol <= 4 kU): fewer prefetch registers for short bases
__global__ __launch_bounds__(kWG) void gs_dots_kernel(int64_t n, PtrSetC Vs, int64_t ld, int ncol, PtrSet ws,
                                                      PtrSet parts) {
  const double2* __restrict__ V = reinterpret_cast<const double2*>(Vs.p[blockIdx.y]);
  const double2* __restrict__ w = reinterpret_cast<const double2*>(ws.p[blockIdx.y]);
  double2* __restrict__ partial = reinterpret_cast<double2*>(parts.p[blockIdx.y]);
  extern __shared__ double2 lds[];
  double2 (*tile)[kGsRows + 1] = reinterpret_cast<double2 (*)[kGsRows + 1]>(lds);
  double2* wn = lds + (size_t)ncol * (kGsRows + 1);
  double2* dred = wn + kGsRows;           // [4][kGsMaxCols]
  double2* ered = dred + 4 * kGsMaxCols;  // [4][kGsMaxCols]
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), j = ncol - 1;
  double dr = 0, di = 0, er = 0, ei = 0;  // dots of column `lane` with w and with v_j
  const int64_t ntiles = (n + kGsRows - 1) / kGsRows;
  double2 a[kU];
  double2 wnext = make_double2(0.0, 0.0);
  auto load_next = [&](int64_t tb) {
    const int64_t i = tb * kGsRows + lane;
    const bool valid = tb < ntiles && i < n;
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int k = wv + 4 * u;
      a[u] = (k < ncol && valid) ? V[(int64_t)k * ld + i] : make_double2(0.0, 0.0);
    }
    if (tid < kGsRows) wnext = valid ? w[i] : make_double2(0.0, 0.0);
  };
  load_next(blockIdx.x);
  for (int64_t tb = blockIdx.x; tb < ntiles; tb += gridDim.x) {
#pragma unroll
    for (int u = 0; u < kU; ++u)
      if (wv + 4 * u < ncol) tile[wv + 4 * u][lane] = a[u];
    if (tid < kGsRows) wn[tid] = wnext;
    __syncthreads();
    load_next(tb + gridDim.x);
    if (lane < ncol) {
      for (int r = wv * 16; r < wv * 16 + 16; ++r) {
        const double2 v = tile[lane][r], x = wn[r], y = tile[j][r];
        dr = fma(v.x, x.x, dr);
        dr = fma(v.y, x.y, dr);
        di = fma(v.x, x.y, di);
        di = fma(-v.y, x.x, di);
        er = fma(v.x, y.x, er);
        er = fma(v.y, y.y, er);
        ei = fma(v.x, y.y, ei);
        ei = fma(-v.y, y.x, ei);
      }
    }
    __syncthreads();  // the next tile overwrites tile and wn
  }
  if (lane < ncol) {
    dred[wv * kGsMaxCols + lane] = make_double2(dr, di);
    ered[wv * kGsMaxCols + lane] = make_double2(er, ei);
  }
  __syncthreads();
  if (tid < ncol) {
    double ar = 0, ai = 0, br = 0, bi = 0;
    for (int q = 0; q < 4; ++q) {
      ar += dred[q * kGsMaxCols + tid].x;
      ai += dred[q * kGsMaxCols + tid].y;
      br += ered[q * kGsMaxCols + tid].x;
      bi += ered[q * kGsMaxCols + tid].y;
    }
    partial[(int64_t)blockIdx.x * 2 * ncol + tid] = make_double2(ar, ai);
    partial[(int64_t)blockIdx.x * 2 * ncol + ncol + tid] = make_double2(br, bi);
  }
}

// Pass B of delayed CGS2 with one row per thread (no staging: every row
// needs all ncol columns, and the coefficients are shared by all rows):
// v_j <- (v_j - V_{<j} cv) * cv[j].x, w <- w - V_{<j} cw - v_j(old) cw[j],
// partial squared norms of the new w in partial[blockIdx.x].x.
__global__ __launch_bounds__(kWG) void gs_update_rows_kernel(int64_t n, PtrSetC Vs, PtrSet Vw, int64_t ld, int ncol,
                                                             PtrSetC cws, PtrSetC cvs, PtrSet ws, PtrSet parts) {
  const double2* __restrict__ V = reinterpret_cast<const double2*>(Vs.p[blockIdx.y]);
  double2* __restrict__ vw = reinterpret_cast<double2*>(Vw.p[blockIdx.y]);
  double2* __restrict__ w = reinterpret_cast<double2*>(ws.p[blockIdx.y]);
  double2* __restrict__ partial = reinterpret_cast<double2*>(parts.p[blockIdx.y]);
  __shared__ double2 cw[kGsMaxCols], cv[kGsMaxCols];
  __shared__ double red[kWG / 64];
  const int tid = threadIdx.x, j = ncol - 1;
  if (tid < ncol) {
    cw[tid] = reinterpret_cast<const double2*>(cws.p[blockIdx.y])[tid];
    cv[tid] = reinterpret_cast<const double2*>(cvs.p[blockIdx.y])[tid];
  }
  __syncthreads();
  double nrm = 0;
  for (int64_t i = (int64_t)blockIdx.x * kWG + tid; i < n; i += (int64_t)gridDim.x * kWG) {
    double ur = 0, ui = 0, vr = 0, vi = 0;
    int k = 0;
    for (; k + 8 <= j; k += 8) {
      double2 a[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) a[u] = V[(int64_t)(k + u) * ld + i];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        cfma(ur, ui, a[u], cw[k + u]);
        cfma(vr, vi, a[u], cv[k + u]);
      }
    }
    for (; k < j; ++k) {
      const double2 a = V[(int64_t)k * ld + i];
      cfma(ur, ui, a, cw[k]);
      cfma(vr, vi, a, cv[k]);
    }
    const double2 vo = V[(int64_t)j * ld + i];
    double2 wi = w[i];
    const double2 dj = cw[j];
    const double ia = cv[j].x;
    wi.x -= ur + (vo.x * dj.x - vo.y * dj.y);
    wi.y -= ui + (vo.x * dj.y + vo.y * dj.x);
    w[i] = wi;
    vw[(int64_t)j * ld + i] = make_double2((vo.x - vr) * ia, (vo.y - vi) * ia);
    nrm = fma(wi.x, wi.x, fma(wi.y, wi.y, nrm));
  }
  for (int o = 32; o > 0; o >>= 1) nrm += __shfl_xor(nrm, o, 64);
  if ((tid & 63) == 0) red[tid >> 6] = nrm;
  __syncthreads();
  if (tid == 0) {
    double sum = 0;
    for (int q = 0; q < kWG / 64; ++q) sum += red[q];
    partial[blockIdx.x] = make_double2(sum, 0.0);
  }
}

// Coefficients of pass B from the reduced dots of pass A (dots[0, ncol): t =
// V^H w, dots[ncol, 2 ncol): g = V^H v_j): s = g_{<j}, a = sqrt(g_j - |s|^2),
// h_j = (t_j - s^H t_{<j}) / a; cw_k = t_k - s_k h_j / a (k < j),
// cw_j = h_j / a; cv_k = s_k, cv_j = 1 / a.  out (host-bound) gets
// [t_0 .. t_{j-1}, h_j, (slot for |w|), s_0 .. s_{j-1}, a].  ncol <= 64.
__device__ __forceinline__ void dcgs2_coefs(const double2* t, int ncol, double2* __restrict__ cw,
                                            double2* __restrict__ cv, double2* __restrict__ out) {
  const double2* g = t + ncol;
  const int j = ncol - 1, k = threadIdx.x;  // one wave, lane k < j owns column k
  const double2 gk = k < j ? g[k] : make_double2(0.0, 0.0);
  const double2 tk = k < j ? t[k] : make_double2(0.0, 0.0);
  double ss = gk.x * gk.x + gk.y * gk.y;
  double str = gk.x * tk.x + gk.y * tk.y;  // conj(s_k) t_k
  double sti = gk.x * tk.y - gk.y * tk.x;
  for (int o = 32; o > 0; o >>= 1) {
    ss += __shfl_xor(ss, o, 64);
    str += __shfl_xor(str, o, 64);
    sti += __shfl_xor(sti, o, 64);
  }
  const double2 gj = g[j], tj = t[j];
  double a2 = gj.x - ss;
  if (!(a2 > 0)) a2 = gj.x;  // no usable correction: keep v_j as it is
  const double a = sqrt(a2), ia = 1.0 / a;
  const double hr = (tj.x - str) * ia, hi = (tj.y - sti) * ia;
  if (k < j) {
    // s_k h_j / a
    const double pr = (gk.x * hr - gk.y * hi) * ia, pi = (gk.x * hi + gk.y * hr) * ia;
    cw[k] = make_double2(tk.x - pr, tk.y - pi);
    cv[k] = gk;
    out[k] = tk;
    out[j + 2 + k] = gk;
  } else if (k == j) {
    cw[j] = make_double2(hr * ia, hi * ia);
    cv[j] = make_double2(ia, 0.0);
    out[j] = make_double2(hr, hi);
    out[2 * j + 2] = make_double2(a, 0.0);
  }
}

__global__ __launch_bounds__(64) void dcgs2_coef_kernel(PtrSetC dots, int ncol, PtrSet cws, PtrSet cvs, PtrSet outs) {
  const int r = blockIdx.y;
  dcgs2_coefs(reinterpret_cast<const double2*>(dots.p[r]), ncol, reinterpret_cast<double2*>(cws.p[r]),
              reinterpret_cast<double2*>(cvs.p[r]), reinterpret_cast<double2*>(outs.p[r]));
}

// The sum a workgroup of kWG threads takes over nblk <= kWG partials (thread t
// holds partial t, the threads add pairwise), on one wave: lane l stands for
// threads l, l + 64, l + 128, l + 192 and holds their partials a; lane 0's
// result.
__device__ __forceinline__ double wave_sum(const double* a) {
  static_assert(kWG == 256, "four threads per lane");
  double v = (a[0] + a[2]) + (a[1] + a[3]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  return v;
}

// Reduction of the pass-A dots (nblk <= kWG partials) and the coefficients in
// one launch: a workgroup per right-hand side, its 16 waves taking four columns
// at a time.  Same sums, in the same order, as gs_dots_final_kernel.  Dependent
// launches of this size take 4.5 us each; with norm_scale_kernel two fewer per
// step: 110 -> 108 us per step at 4,913 unknowns, 238 -> 232 for eight
// right-hand sides.  Above kWG partials (16,384 unknowns) one workgroup reads
// them slower than the columns' workgroups do (37,485 unknowns, eight right-hand
// sides: 499 us fused, 494 not).
__global__ __launch_bounds__(1024) void dcgs2_final_kernel(PtrSetC parts, int nblk, int ncol, PtrSet cws, PtrSet cvs,
                                                           PtrSet outs) {
  __shared__ double2 t[2 * kGsMaxCols];
  const int r = blockIdx.y, wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const double2* __restrict__ partial = reinterpret_cast<const double2*>(parts.p[r]);
  for (int k0 = wv; k0 < 2 * ncol; k0 += 64) {
    double2 v[4][4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int k = k0 + 16 * u, b = lane + 64 * q;
        v[u][q] = k < 2 * ncol && b < nblk ? partial[(int64_t)b * 2 * ncol + k] : make_double2(0.0, 0.0);
      }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const double re[4] = {v[u][0].x, v[u][1].x, v[u][2].x, v[u][3].x};
      const double im[4] = {v[u][0].y, v[u][1].y, v[u][2].y, v[u][3].y};
      const double2 sum = make_double2(wave_sum(re), wave_sum(im));
      if (lane == 0 && k0 + 16 * u < 2 * ncol) t[k0 + 16 * u] = sum;
    }
  }
  __syncthreads();
  if (wv == 0)
    dcgs2_coefs(t, ncol, reinterpret_cast<double2*>(cws.p[r]), reinterpret_cast<double2*>(cvs.p[r]),
                reinterpret_cast<double2*>(outs.p[r]));
}

__global__ __launch_bounds__(kWG) void norm_final2_kernel(PtrSetC parts, int nblk, PtrSet outs) {
  __shared__ double sm[kWG];
  const double2* __restrict__ partial = reinterpret_cast<const double2*>(parts.p[blockIdx.y]);
  double2* __restrict__ out = reinterpret_cast<double2*>(outs.p[blockIdx.y]);
  double s = 0;
  for (int b = threadIdx.x; b < nblk; b += kWG) s += partial[b].x;
  sm[threadIdx.x] = s;
  __syncthreads();
  for (int st = kWG / 2; st > 0; st >>= 1) {
    if (threadIdx.x < st) sm[threadIdx.x] += sm[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = make_double2(sqrt(sm[0]), 0.0);
}

__global__ __launch_bounds__(kWG) void norm_partial_kernel(int64_t n, const double2* __restrict__ w,
                                                           double* __restrict__ partial) {
  __shared__ double sm[kWG];
  double s = 0;
  for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < n; i += (int64_t)gridDim.x * kWG) {
    double2 v = w[i];
    s = fma(v.x, v.x, s);
    s = fma(v.y, v.y, s);
  }
  sm[threadIdx.x] = s;
  __syncthreads();
  for (int st = kWG / 2; st > 0; st >>= 1) {
    if (threadIdx.x < st) sm[threadIdx.x] += sm[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = sm[0];
}

__global__ __launch_bounds__(kWG) void norm_final_kernel(const double* __restrict__ partial, int nblk,
                                                         double2* __restrict__ out) {
  __shared__ double sm[kWG];
  double s = 0;
  for (int b = threadIdx.x; b < nblk; b += kWG) s += partial[b];
  sm[threadIdx.x] = s;
  __syncthreads();
  for (int st = kWG / 2; st > 0; st >>= 1) {
    if (threadIdx.x < st) sm[threadIdx.x] += sm[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = make_double2(sqrt(sm[0]), 0.0);
}

__global__ __launch_bounds__(kWG) void scale_by_inv_kernel(int64_t n, PtrSetC ws, PtrSetC nrms, PtrSet vs) {
  const double2* __restrict__ w = reinterpret_cast<const double2*>(ws.p[blockIdx.y]);
  const double2* __restrict__ nrm = reinterpret_cast<const double2*>(nrms.p[blockIdx.y]);
  double2* __restrict__ v = reinterpret_cast<double2*>(vs.p[blockIdx.y]);
  const int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (i >= n) return;
  const double d = nrm[0].x;
  const double inv = d != 0.0 ? 1.0 / d : 0.0;
  const double2 a = w[i];
  v[i] = make_double2(a.x * inv, a.y * inv);
}

// norm_final2_kernel and scale_by_inv_kernel in one launch: every wave reduces
// the nblk <= kWG partials itself (the same sum), wave 0 of right-hand side r also
// stores the norm and, with a host buffer, copies the step's nout
// Hessenberg entries (the norm at entry inorm) there.
__global__ __launch_bounds__(kWG) void norm_scale_kernel(int64_t n, PtrSetC ws, PtrSetC parts, int nblk, PtrSet nrms,
                                                         PtrSet vs, const double2* __restrict__ hcol, int nout,
                                                         int inorm, double2* __restrict__ host) {
  const int r = blockIdx.y;
  const double2* __restrict__ w = reinterpret_cast<const double2*>(ws.p[r]);
  const double2* __restrict__ partial = reinterpret_cast<const double2*>(parts.p[r]);
  const int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x;
  const double2 a = w[min(i, n - 1)];
  double p[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int b = (threadIdx.x & 63) + 64 * q;
    p[q] = b < nblk ? partial[b].x : 0.0;
  }
  const double d = sqrt(__shfl(wave_sum(p), 0, 64));
  if (blockIdx.x == 0 && threadIdx.x < 64) {
    const double2 nv = make_double2(d, 0.0);
    if (threadIdx.x == 0) reinterpret_cast<double2*>(nrms.p[r])[0] = nv;
    if (host)
      for (int e = threadIdx.x; e < nout; e += 64) host[e] = e == inorm ? nv : hcol[e];
  }
  const double inv = d != 0.0 ? 1.0 / d : 0.0;
  if (i < n) reinterpret_cast<double2*>(vs.p[r])[i] = make_double2(a.x * inv, a.y * inv);
}

__global__ __launch_bounds__(kWG) void scale_kernel(int64_t n, const double2* __restrict__ w, double alpha,
                                                    double2* __restrict__ v) {
  const int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (i >= n) return;
  const double2 a = w[i];
  v[i] = make_double2(a.x * alpha, a.y * alpha);
}

__global__ __launch_bounds__(kWG) void gemv_acc_kernel(int64_t n, const double2* __restrict__ Z, int64_t ld, int k,
                                                       const double2* __restrict__ y, double2* __restrict__ x) {
  __shared__ double2 ys[1024];
  for (int j = threadIdx.x; j < k; j += kWG) ys[j] = y[j];
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (i >= n) return;
  double ar = 0, ai = 0;
  for (int j = 0; j < k; ++j) cfma(ar, ai, Z[(int64_t)j * ld + i], ys[j]);
  double2 xi = x[i];
  x[i] = make_double2(xi.x + ar, xi.y + ai);
}

__global__ __launch_bounds__(kWG) void fill_zero_kernel(int64_t n, double* __restrict__ p) {
  const int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (i < n) p[i] = 0.0;
}

__global__ __launch_bounds__(kWG) void copy_kernel(int64_t n, const double* __restrict__ a, double* __restrict__ b) {
  const int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (i < n) b[i] = a[i];
}

inline unsigned blocks_for(int64_t n, int per = kWG) { return (unsigned)((n + per - 1) / per); }

__global__ __launch_bounds__(kWG) void copy_tiles_kernel(const uint64_t* __restrict__ src, uint64_t* __restrict__ dst,
                                                         const int64_t* __restrict__ from,
                                                         const int64_t* __restrict__ to,
                                                         const int64_t* __restrict__ words, int64_t ntiles) {
  for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
    const uint64_t* a = src + from[t];
    uint64_t* d = dst + to[t];
    const int64_t n = words[t];
    for (int64_t i = threadIdx.x; i < n; i += kWG) d[i] = a[i];
  }
}

}  // namespace

int waves_per_tile(int ncols) { return ncols <= 96 ? 1 : (ncols <= 384 ? 2 : 4); }

void copy_tiles(const void* src, void* dst, const int64_t* from, const int64_t* to, const int64_t* words,
                int64_t ntiles, hipStream_t s) {
  if (ntiles <= 0) return;
  const unsigned grid = (unsigned)std::min<int64_t>(ntiles, 1 << 20);
  copy_tiles_kernel<<<grid, kWG, 0, s>>>(reinterpret_cast<const uint64_t*>(src), reinterpret_cast<uint64_t*>(dst),
                                         from, to, words, ntiles);
}

// Workgroups of a level kernel resident on the current device at once
// (cached per kernel, LDS size and device).
static int resident_grid(const void* fn, size_t lds) {
  static std::mutex mu;
  static std::map<std::tuple<const void*, size_t, int>, int> cache;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 1 << 30;
  const auto key = std::make_tuple(fn, lds, dev);
  std::lock_guard<std::mutex> lock(mu);
  auto it = cache.find(key);
  if (it != cache.end()) return it->second;
  int ncu = 0, per = 0;
  int g = 1 << 30;  // unknown: one workgroup per task
  if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, kWG, lds) == hipSuccess && per > 0 && ncu > 0)
    g = per * ncu;
  cache.emplace(key, g);
  return g;
}

template <class K, class... A>
static void level_go(K kernel, int64_t ntasks, size_t lds, hipStream_t s, A... args) {
  const int64_t g = std::min<int64_t>(ntasks, resident_grid(reinterpret_cast<const void*>(kernel), lds));
  kernel<<<(unsigned)g, kWG, lds, s>>>(args...);
}

void fwd_level(const Batch& b, int64_t task0, int64_t ntasks, const double* bin, int chunk, bool coarse,
               hipStream_t s) {
  if (ntasks <= 0) return;
  const Task* k = b.kf + task0;
  const int nt = (int)ntasks;
  const double2* in = reinterpret_cast<const double2*>(bin);
  const size_t lds = sizeof(double2) * (size_t)chunk;
  if (coarse)
    level_go(fwd_level_kernel<double2, 1>, ntasks, lds, s, k, nt, b, in, chunk);
  else if (b.c64)
    level_go(fwd_level_kernel<float2, 0>, ntasks, lds, s, k, nt, b, in, chunk);
  else
    level_go(fwd_level_kernel<double2, 0>, ntasks, lds, s, k, nt, b, in, chunk);
}

void fwd_sn(const Batch& b, int64_t job0, int64_t njobs, const double* bin, hipStream_t s) {
  if (njobs <= 0) return;
  const SnJob* j = b.snj + job0;
  const int nj = (int)njobs;
  const double2* in = reinterpret_cast<const double2*>(bin);
  const int64_t wgs = (njobs + 3) / 4;
  if (b.c64)
    level_go(fwd_sn_kernel<float2>, wgs, 0, s, j, nj, b, in);
  else
    level_go(fwd_sn_kernel<double2>, wgs, 0, s, j, nj, b, in);
}

void bwd_level(const Batch& b, int64_t task0, int64_t ntasks, int chunk, bool coarse, hipStream_t s) {
  if (ntasks <= 0) return;
  const Task* k = b.kb + task0;
  const int nt = (int)ntasks;
  const size_t lds = sizeof(double2) * (size_t)chunk;
  if (coarse)
    level_go(bwd_level_kernel<double2, 1>, ntasks, lds, s, k, nt, b, chunk);
  else if (b.c64)
    level_go(bwd_level_kernel<float2, 0>, ntasks, lds, s, k, nt, b, chunk);
  else
    level_go(bwd_level_kernel<double2, 0>, ntasks, lds, s, k, nt, b, chunk);
}

void flow(const FlowArgs& a, bool c64, bool coarse, int t0, int t1, const double* bin, hipStream_t s) {
  if (t1 <= t0) return;
  const double2* in = reinterpret_cast<const double2*>(bin);
  const size_t lds = sizeof(double2) * (size_t)a.chunk;
  const int word = kFlowTicket + (t0 > 0);  // a second launch of one sweep draws from the other ticket
  if (coarse)
    level_go(flow_kernel<double2, 1>, t1 - t0, lds, s, a, t0, t1, word, in);
  else if (c64)
    level_go(flow_kernel<float2, 0>, t1 - t0, lds, s, a, t0, t1, word, in);
  else
    level_go(flow_kernel<double2, 0>, t1 - t0, lds, s, a, t0, t1, word, in);
}

int coop_grid() {
  int dev = 0, ncu = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, batch_solve_coop_kernel, kWG, 0) != hipSuccess) return 0;
  return per * ncu;
}

hipError_t batch_solve_coop(const Batch& b, const double* bin, const LevelRanges& lv, int grid, hipStream_t s) {
  Batch bb = b;
  const double2* in = reinterpret_cast<const double2*>(bin);
  LevelRanges l = lv;
  void* args[] = {&bb, &in, &l};
  return hipLaunchCooperativeKernel(reinterpret_cast<const void*>(batch_solve_coop_kernel), dim3(grid), dim3(kWG),
                                    args, 0, s);
}

template <int G, int U, bool R, class VT>
void spmv_go(int64_t n, const int64_t* ptr, const int32_t* col, const VT* v2, const int64_t* xr, int64_t xrows,
             const double2* x2, const double2* b2, double2* y2, hipStream_t s) {
  // with R, 8 x the block count of the longest XCD range, else one block per kWG / G rows
  const unsigned grid = R ? 8 * blocks_for(xrows * G) : blocks_for(n * G);
  spmv_kernel<G, U, R, VT><<<grid, kWG, 0, s>>>(n, ptr, col, v2, xr, x2, b2, y2);
}

template <bool R, class VT>
void spmv_launch(int64_t n, const int64_t* ptr, const int32_t* col, const VT* v2, const int64_t* xr,
                 int64_t xrows, const double2* x2, const double2* b2, double2* y2, int cfg, hipStream_t s) {
  switch (cfg) {
    case spmv_cfg(4, 4): spmv_go<4, 4, R, VT>(n, ptr, col, v2, xr, xrows, x2, b2, y2, s); break;
    case spmv_cfg(4, 8): spmv_go<4, 8, R, VT>(n, ptr, col, v2, xr, xrows, x2, b2, y2, s); break;
    case spmv_cfg(8, 1): spmv_go<8, 1, R, VT>(n, ptr, col, v2, xr, xrows, x2, b2, y2, s); break;
    case spmv_cfg(8, 2): spmv_go<8, 2, R, VT>(n, ptr, col, v2, xr, xrows, x2, b2, y2, s); break;
    case spmv_cfg(8, 4): spmv_go<8, 4, R, VT>(n, ptr, col, v2, xr, xrows, x2, b2, y2, s); break;
    case spmv_cfg(16, 1): spmv_go<16, 1, R, VT>(n, ptr, col, v2, xr, xrows, x2, b2, y2, s); break;
    case spmv_cfg(16, 2): spmv_go<16, 2, R, VT>(n, ptr, col, v2, xr, xrows, x2, b2, y2, s); break;
    case spmv_cfg(32, 1): spmv_go<32, 1, R, VT>(n, ptr, col, v2, xr, xrows, x2, b2, y2, s); break;
    default: spmv_go<4, 1, R, VT>(n, ptr, col, v2, xr, xrows, x2, b2, y2, s); break;
  }
}

int64_t xcd_ranges(int64_t n, const int64_t* ptr, int64_t xr[9]) {
  xr[0] = 0;
  int64_t r = 0, longest = 0;
  for (int k = 1; k < 8; ++k) {
    const int64_t target = (ptr[n] * k) / 8;
    while (r < n && ptr[r] < target) ++r;
    xr[k] = r;
  }
  xr[8] = n;
  for (int k = 0; k < 8; ++k) longest = std::max<int64_t>(longest, xr[k + 1] - xr[k]);
  return longest;
}

void spmv(int64_t n, const int64_t* ptr, const int32_t* col, const double* val, const int64_t* xr, int64_t xrows,
          const double* x, const double* b, double* y, int cfg, hipStream_t s) {
  if (n <= 0) return;
  auto v2 = reinterpret_cast<const double2*>(val);
  auto x2 = reinterpret_cast<const double2*>(x);
  auto b2 = reinterpret_cast<const double2*>(b);
  auto y2 = reinterpret_cast<double2*>(y);
  if (xr)
    spmv_launch<true, double2>(n, ptr, col, v2, xr, xrows, x2, b2, y2, cfg, s);
  else
    spmv_launch<false, double2>(n, ptr, col, v2, nullptr, 0, x2, b2, y2, cfg, s);
}

void spmv_split(int64_t n, const int64_t* ptr, const int32_t* col, const double* val, const double* x,
                const double* b, double* y, int cfg, hipStream_t s) {
  if (n <= 0) return;
  spmv_launch<false, double>(n, ptr, col, val, nullptr, 0, reinterpret_cast<const double2*>(x),
                             reinterpret_cast<const double2*>(b), reinterpret_cast<double2*>(y), cfg, s);
}

void sell_spmv(int64_t n, int64_t nslices, const int64_t* soff, const int32_t* swidth, const int32_t* perm,
               const int32_t* col, const double* val, const double* x, const double* b, double* y, hipStream_t s) {
  if (n <= 0) return;
  const unsigned nb = (unsigned)((nslices + 3) / 4);
  sell_kernel<<<(nb + 7) / 8 * 8, kWG, 0, s>>>(
      n, nslices, soff, swidth, perm, col, reinterpret_cast<const double2*>(val), reinterpret_cast<const double2*>(x),
      reinterpret_cast<const double2*>(b), reinterpret_cast<double2*>(y));
}

void spmv_real(int64_t n, const int64_t* ptr, const int32_t* col, const double* val, const double* x, double* y,
               int G, hipStream_t s, const FlowState& done) {
  if (n <= 0) return;
  auto x2 = reinterpret_cast<const double2*>(x);
  auto y2 = reinterpret_cast<double2*>(y);
  switch (G) {
    case 8: spmv_real_kernel<8><<<blocks_for(n * 8), kWG, 0, s>>>(n, ptr, col, val, x2, y2, done); break;
    case 16: spmv_real_kernel<16><<<blocks_for(n * 16), kWG, 0, s>>>(n, ptr, col, val, x2, y2, done); break;
    case 32: spmv_real_kernel<32><<<blocks_for(n * 32), kWG, 0, s>>>(n, ptr, col, val, x2, y2, done); break;
    case 64: spmv_real_kernel<64><<<blocks_for(n * 64), kWG, 0, s>>>(n, ptr, col, val, x2, y2, done); break;
    default: spmv_real_kernel<4><<<blocks_for(n * 4), kWG, 0, s>>>(n, ptr, col, val, x2, y2, done); break;
  }
}

void coarse_update(int64_t n, const int64_t* zptr, const int32_t* zcol, const double* zval, const int64_t* aptr,
                   const int32_t* acol, const double* aval, const double* cx, const double* r, double* q, double* t,
                   int G, hipStream_t s, const FlowState& done) {
  if (n <= 0) return;
  auto c2 = reinterpret_cast<const double2*>(cx);
  auto r2 = reinterpret_cast<const double2*>(r);
  auto q2 = reinterpret_cast<double2*>(q);
  auto t2 = reinterpret_cast<double2*>(t);
  if (G == 8)
    coarse_update_kernel<8><<<blocks_for(n * 8), kWG, 0, s>>>(n, zptr, zcol, zval, aptr, acol, aval, c2, r2, q2, t2,
                                                            done);
  else if (G == 2)
    coarse_update_kernel<2><<<blocks_for(n * 2), kWG, 0, s>>>(n, zptr, zcol, zval, aptr, acol, aval, c2, r2, q2, t2,
                                                            done);
  else if (G == 1)
    coarse_update_kernel<1><<<blocks_for(n), kWG, 0, s>>>(n, zptr, zcol, zval, aptr, acol, aval, c2, r2, q2, t2,
                                                            done);
  else
    coarse_update_kernel<4><<<blocks_for(n * 4), kWG, 0, s>>>(n, zptr, zcol, zval, aptr, acol, aval, c2, r2, q2, t2,
                                                            done);
}

void prolong(int64_t n, const int64_t* ptr, const int32_t* idx, const double* w, const double* xl, const double* q,
             double* z, hipStream_t s, const FlowState& done) {
  if (n <= 0) return;
  prolong_kernel<<<blocks_for(n), kWG, 0, s>>>(n, ptr, idx, w, reinterpret_cast<const double2*>(xl),
                                               reinterpret_cast<const double2*>(q), reinterpret_cast<double2*>(z),
                                               done);
}

int gs_blocks(int64_t n) {
  int64_t b = (n + kWG * 4 - 1) / (kWG * 4);
  if (b < 1) b = 1;
  if (b > 2048) b = 2048;
  return (int)b;
}

void gs_final(int nr, const PtrSetC& partial, int nblk, int ncol, const PtrSet& h, const PtrSet& hacc,
              int accumulate, hipStream_t s) {
  gs_dots_final_kernel<<<dim3((unsigned)ncol, (unsigned)nr), kWG, 0, s>>>(partial, nblk, ncol, h, hacc, accumulate);
}

int gs_tiles(int64_t n) {
  const int64_t t = (n + kGsRows - 1) / kGsRows;
  return (int)(t < 2048 ? t : 2048);  // workgroups; each loops over 64-row tiles
}

void gs_pass(int mode, int nr, int64_t n, const PtrSetC& V, int64_t ld, int ncol, const PtrSetC& h, const PtrSet& w,
             const PtrSet& partial, hipStream_t s) {
  const dim3 grid((unsigned)gs_tiles(n), (unsigned)nr);
  const size_t lds = sizeof(double2) * ((size_t)ncol * (kGsRows + 1) + kGsMaxCols + kGsRows + 4 * kGsRows +
                                        4 * kGsMaxCols) +
                     sizeof(double) * kGsRows;
  if (mode == 0)
    gs_pass_kernel<false, true, false><<<grid, kWG, lds, s>>>(n, V, ld, ncol, h, w, partial);
  else if (mode == 1)
    gs_pass_kernel<true, true, false><<<grid, kWG, lds, s>>>(n, V, ld, ncol, h, w, partial);
  else
    gs_pass_kernel<true, false, true><<<grid, kWG, lds, s>>>(n, V, ld, ncol, h, w, partial);
}

void gs_dual(bool update, int nr, int64_t n, const PtrSetC& V, const PtrSet& Vw, int64_t ld, int ncol,
             const PtrSetC& cw, const PtrSetC& cv, const PtrSet& w, const PtrSet& partial, hipStream_t s) {
  const dim3 grid((unsigned)gs_tiles(n), (unsigned)nr);
  const size_t lds = sizeof(double2) * ((size_t)ncol * (kGsRows + 1) + kGsRows + 8 * kGsMaxCols);
  if (update)
    gs_update_rows_kernel<<<grid, kWG, 0, s>>>(n, V, Vw, ld, ncol, cw, cv, w, partial);
  else if (ncol <= 16)
    gs_dots_kernel<4><<<grid, kWG, lds, s>>>(n, V, ld, ncol, w, partial);
  else if (ncol <= 32)
    gs_dots_kernel<8><<<grid, kWG, lds, s>>>(n, V, ld, ncol, w, partial);
  else
    gs_dots_kernel<kGsMaxCols / 4><<<grid, kWG, lds, s>>>(n, V, ld, ncol, w, partial);
}
void dcgs2_coef(int nr, const PtrSetC& partial, int nblk, int ncol, const PtrSet& dots, const PtrSet& cw,
                const PtrSet& cv, const PtrSet& out, hipStream_t s) {
  if (nblk <= kWG) {
    dcgs2_final_kernel<<<dim3(1, (unsigned)nr), 1024, 0, s>>>(partial, nblk, ncol, cw, cv, out);
    return;
  }
  gs_final(nr, partial, nblk, 2 * ncol, dots, PtrSet{}, 0, s);
  PtrSetC d{};
  for (int r = 0; r < nr; ++r) d.p[r] = dots.p[r];
  dcgs2_coef_kernel<<<dim3(1, (unsigned)nr), 64, 0, s>>>(d, ncol, cw, cv, out);
}

bool norm_scale(int nr, int64_t n, const PtrSetC& w, const PtrSetC& partial, int nblk, const PtrSet& nrm,
                const PtrSet& v, const double* hcol, int nout, int inorm, double* host, hipStream_t s) {
  if (n <= 0) return false;
  if (nblk <= kWG) {
    norm_scale_kernel<<<dim3(blocks_for(n), (unsigned)nr), kWG, 0, s>>>(
        n, w, partial, nblk, nrm, v, reinterpret_cast<const double2*>(hcol), nout, inorm,
        reinterpret_cast<double2*>(host));
    return host != nullptr;
  }
  norm_final2_kernel<<<dim3(1, (unsigned)nr), kWG, 0, s>>>(partial, nblk, nrm);
  PtrSetC d{};
  for (int r = 0; r < nr; ++r) d.p[r] = nrm.p[r];
  scale_by_inv_kernel<<<dim3(blocks_for(n), (unsigned)nr), kWG, 0, s>>>(n, w, d, v);
  return false;
}

void norm2(int64_t n, const double* w, double* partial, int nblk, double* out, hipStream_t s) {
  norm_partial_kernel<<<(unsigned)nblk, kWG, 0, s>>>(n, reinterpret_cast<const double2*>(w), partial);
  norm_final_kernel<<<1, kWG, 0, s>>>(partial, nblk, reinterpret_cast<double2*>(out));
}

void scale(int64_t n, const double* w, double alpha, double* v, hipStream_t s) {
  if (n <= 0) return;
  scale_kernel<<<blocks_for(n), kWG, 0, s>>>(n, reinterpret_cast<const double2*>(w), alpha,
                                             reinterpret_cast<double2*>(v));
}

void gemv_acc(int64_t n, const double* Z, int64_t ld, int k, const double* y, double* x, hipStream_t s) {
  if (n <= 0 || k <= 0) return;
  gemv_acc_kernel<<<blocks_for(n), kWG, 0, s>>>(n, reinterpret_cast<const double2*>(Z), ld, k,
                                                reinterpret_cast<const double2*>(y), reinterpret_cast<double2*>(x));
}

// ---- fixed scratch of the allocation-free entry point ----------------------
//
// One file-scope array per device (each GPU the library runs on holds its own
// copy until the process ends).  In host code `scratch` names a host-side
// stand-in, not the device array: its device address is looked up once per
// device with hipGetSymbolAddress and only that address is ever handed to
// kernels or copies.

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t scratch_init(int device) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[device]) return hipSuccess;
  int cur = -1;
  hipError_t e = hipGetDevice(&cur);
  if (e != hipSuccess) return e;
  if (cur != device) return hipErrorInvalidDevice;  // the caller makes `device` current
  void* ptr = nullptr;
  e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  g_scratch_ptr[device] = ptr;
  return hipSuccess;
}

void* scratch_ptr(int device) {
  if (device < 0 || device >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  return g_scratch_ptr[device];
}

void fill_zero(int64_t n, double* p, hipStream_t s) {
  if (n <= 0) return;
  fill_zero_kernel<<<blocks_for(n), kWG, 0, s>>>(n, p);
}

void copy(int64_t n, const double* src, double* dst, hipStream_t s) {
  if (n <= 0) return;
  copy_kernel<<<blocks_for(n), kWG, 0, s>>>(n, src, dst);
}

}  // namespace dev
}  // namespace helm
