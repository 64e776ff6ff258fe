// Multi-right-hand-side kernels (pseudo-block GMRES: S Krylov spaces advanced
// together, the operator and the preconditioner applied to all S vectors in
// one pass over A and over the factor panels).
//
// Block vectors are interleaved: entry (i, r) of an n x S block sits at
// i * S + r, so every gather of a row fetches S contiguous complex values.
// The level kernels stream each panel tile once for all S columns, as small
// dense contractions on MFMA.
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "device.hpp"

namespace helm {
namespace dev {

namespace {

constexpr int kWG = 256;

__device__ __forceinline__ void cfma(double& ar, double& ai, double2 a, double2 v) {
  ar = fma(a.x, v.x, ar);
  ar = fma(-a.y, v.y, ar);
  ai = fma(a.x, v.y, ai);
  ai = fma(a.y, v.x, ai);
}
__device__ __forceinline__ double2 widen(double2 a) { return a; }
__device__ __forceinline__ double2 widen(float2 a) { return make_double2((double)a.x, (double)a.y); }

// ---- MFMA form for 16 right-hand sides --------------------------------------
// A tile (<= 64 rows x ncols) times the 16-column input block is a small
// dense contraction: it runs on v_mfma_{f64,f32}_16x16x4 as four 16-row
// blocks, the complex product split into four real MFMAs
//   Dre += Are Bre - Aim Bim,  Dim += Are Bim + Aim Bre.
// Operand layout of the 16x16x4 MFMA: lane l holds A[l % 16][l / 16] and
// B[l / 16][l % 16]; accumulator register j of lane l is D[row][l % 16] with
// row = 4 (l / 16) + j for FP32 and row = 4 j + l / 16 for FP64 (both
// checked on the device).
// Complex128 panels use FP64 MFMA; complex64 panels use FP32 MFMA with the
// input block rounded to FP32 (FP32 accumulation; the outer flexible GMRES
// stays in FP64).
typedef double dv4 __attribute__((ext_vector_type(4)));
typedef float fv4 __attribute__((ext_vector_type(4)));

template <class T>
struct Mf;
template <>
struct Mf<double> {
  using V4 = dv4;
  using C2 = double2;
  static __device__ __forceinline__ V4 mma(double a, double b, V4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lk, int j) { return 4 * j + lk; }
};
template <>
struct Mf<float> {
  using V4 = fv4;
  using C2 = float2;
  static __device__ __forceinline__ V4 mma(float a, float b, V4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lk, int j) { return 4 * lk + j; }
};

// ---- staged MFMA form ------------------------------------------------------
template <class T>
__global__ __launch_bounds__(kWG) void gather_fwd_kernel(const int32_t* __restrict__ sns, Batch b,
                                                         const double2* __restrict__ bin,
                                                         const double2* __restrict__ ubb,
                                                         typename Mf<T>::C2* __restrict__ G) {
  using C2 = typename Mf<T>::C2;
  const int sn = sns[blockIdx.x];
  const int c0 = b.sn_c0[sn], w = b.sn_w[sn], frow0 = b.sn_frow0[sn];
  C2* g = G + b.goff_f[sn] * 16;
  // workgroup blockIdx.y of gridDim.y takes every gridDim.y-th 256 entries;
  // an entry's input index and child-update pair are loaded together, then
  // the input and the (at most two) updates; a row with more children walks
  // its list
  for (int e = blockIdx.y * kWG + threadIdx.x; e < w * 16; e += gridDim.y * kWG) {
    const int k = e >> 4, r = e & 15;
    const int fr = frow0 + k;
    const int bi = b.bidx[c0 + k];
    const int2 c2 = b.fcon2[fr];
    double2 v = bin[(int64_t)bi * 16 + r];
    const double2 u0 = *(c2.x >= 0 ? ubb + (int64_t)c2.x * 16 + r : bin + r);
    const double2 u1 = *(c2.y >= 0 ? ubb + (int64_t)c2.y * 16 + r : bin + r);
    if (c2.x >= 0) {
      v.x -= u0.x;
      v.y -= u0.y;
      if (c2.y >= 0) {
        v.x -= u1.x;
        v.y -= u1.y;
      }
    } else if (c2.x < -1) {
      for (int q = -2 - c2.x; q < b.fcon_ptr[fr + 1]; ++q) {
        const double2 u = ubb[(int64_t)b.fcon_idx[q] * 16 + r];
        v.x -= u.x;
        v.y -= u.y;
      }
    }
    g[e] = C2{(T)v.x, (T)v.y};
  }
}

// Panel loads are streamed once per sweep: non-temporal, so they do not
// evict the staged input blocks and vectors from the caches.
typedef double dvec2 __attribute__((ext_vector_type(2)));
typedef float fvec2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ double2 ldp(const double2* p) {
  const dvec2 v = __builtin_nontemporal_load(reinterpret_cast<const dvec2*>(p));
  return make_double2(v.x, v.y);
}
__device__ __forceinline__ float2 ldp(const float2* p) {
  const fvec2 v = __builtin_nontemporal_load(reinterpret_cast<const fvec2*>(p));
  return make_float2(v.x, v.y);
}

// Streams the k-steps k0 = ks0, ks0 + kst, ... < cn (a k-step is four
// columns) of a panel tile P (nr rows, column-major) against the input block
// Bk (16 right-hand sides per column) into the accumulators of the row
// blocks rb < nrb.  The loads of the next k-step are issued before the MFMAs
// of the current one, into the other of two register sets, so no loaded
// register is copied (a copy would make the wave wait for the load just
// issued).  Every load is issued unconditionally, at a clamped address: rows
// past nr read row nr - 1 (rows whose results are never stored), columns
// past cn read column cn - 1 and meet a zero B entry, so the waits the
// compiler places count exactly the other set's loads.
template <class T>
__device__ __forceinline__ void mfma_stream(const typename Mf<T>::C2* __restrict__ P, int nr, int cn,
                                            const typename Mf<T>::C2* __restrict__ Bk, int ks0, int kst,
                                            typename Mf<T>::V4* dre, typename Mf<T>::V4* dim) {
  using C2 = typename Mf<T>::C2;
  if (ks0 >= cn) return;  // uniform: the wave has no k-step
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
  const int nrb = (nr + 15) >> 4;
  int roff[4];
#pragma unroll
  for (int rb = 0; rb < 4; ++rb) roff[rb] = min(16 * rb + lr, nr - 1);
  auto load = [&](int k0, C2& bv, C2 (&a)[4]) {
    const int k = min(k0 + lk, cn - 1);
    bv = Bk[k * 16 + lr];
    const C2* pc = P + (int64_t)k * nr;
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) a[rb] = ldp(pc + roff[rb]);
  };
  auto step = [&](int k0, const C2& b, const C2 (&a)[4]) {
    const C2 bv = k0 + lk < cn ? b : C2{0, 0};
    const decltype(bv.y) nby = -bv.y;  // a.y (-b.y) is -(a.y b.y) exactly
    // row blocks past the tile are skipped (uniform branches: nrb is the
    // same on every lane)
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
      if (rb < nrb) {
        dre[rb] = Mf<T>::mma(a[rb].x, bv.x, dre[rb]);
        dim[rb] = Mf<T>::mma(a[rb].x, bv.y, dim[rb]);
        dre[rb] = Mf<T>::mma(a[rb].y, nby, dre[rb]);
        dim[rb] = Mf<T>::mma(a[rb].y, bv.x, dim[rb]);
      }
    }
  };
  C2 b0, a0[4], b1, a1[4];
  load(ks0, b0, a0);
  // the k-steps go in pairs (an odd count loads a step past cn and skips
  // its MFMAs); the scheduling barriers keep each k-step's loads ahead of
  // the MFMAs of the step before it
  for (int k0 = ks0; k0 < cn; k0 += 2 * kst) {
    load(k0 + kst, b1, a1);
    __builtin_amdgcn_sched_barrier(0);
    step(k0, b0, a0);
    __builtin_amdgcn_sched_barrier(0);
    load(k0 + 2 * kst, b0, a0);
    __builtin_amdgcn_sched_barrier(0);
    if (k0 + kst < cn) step(k0 + kst, b1, a1);  // uniform
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Children's updates routed to front row fr, for right-hand side r: the
// first two entries of the row's list come as one index pair (fcon2), so
// the values are one load away; a row with more than two walks its list.
// uu holds the pair's values, loaded beforehand (a missing entry is not
// used); the sum is taken in list order.
__device__ __forceinline__ void add_children(const Batch& b, int fr, int2 c2, const double2* uu, const double2* ubb,
                                             int r, double& ar, double& ai) {
  if (c2.x >= 0) {
    ar += uu[0].x;
    ai += uu[0].y;
    if (c2.y >= 0) {
      ar += uu[1].x;
      ai += uu[1].y;
    }
  } else if (c2.x < -1) {
    for (int e = -2 - c2.x; e < b.fcon_ptr[fr + 1]; ++e) {
      const double2 u = ubb[(int64_t)b.fcon_idx[e] * 16 + r];
      ar += u.x;
      ai += u.y;
    }
  }
}

// The level kernels' launch bounds keep their register budget at or below
// 256 (at least three waves per SIMD for complex128): with a larger budget
// the compiler may hold MFMA accumulators in AGPRs and move them through
// VGPRs around every MFMA.
template <class T, int kFwd, int kCoarse>
__global__ __launch_bounds__(kWG, sizeof(T) == 4 ? 4 : 3) void level_mfma_kernel(const Tile* __restrict__ tiles, Batch b,
                                                         const typename Mf<T>::C2* __restrict__ G,
                                                         double2* __restrict__ out, double2* __restrict__ ubb) {
  using C2 = typename Mf<T>::C2;
  using V4 = typename Mf<T>::V4;
  // partial sums of the 4 waves, two row blocks at a time: [wave][rb2][j][lane]
  __shared__ C2 red[4][2][4][64];
  const Tile t = tiles[blockIdx.x];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sn = t.sn, c0 = b.sn_c0[sn], w = b.sn_w[sn];
  const C2* __restrict__ P = reinterpret_cast<const C2*>(kFwd ? b.pf : b.pb) + t.off;
  const C2* Bk = G + (b.goff_f[sn] + t.col0) * 16;  // the staged forward input block
  V4 dre[4], dim[4];
#pragma unroll
  for (int rb = 0; rb < 4; ++rb) dre[rb] = dim[rb] = V4{0, 0, 0, 0};
  // 4 waves per tile: wave q takes the k-steps q, q + 4, ... of the tile;
  // the partial accumulators are summed through LDS
  mfma_stream<T>(P, t.nrows, t.ncols, Bk, 4 * wv, 16, dre, dim);
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int j = 0; j < 4; ++j) red[wv][q][j][lane] = C2{dre[2 * h + q][j], dim[2 * h + q][j]};
    __syncthreads();
    // 512 outputs (32 rows x 16 right-hand sides) of this half, 2 per
    // thread: the update rows' child-update pairs and values are loaded for
    // both outputs before either is stored
    const int frow0 = b.sn_frow0[sn], uoff = b.sn_uoff[sn];
    int2 c2[2];
    double2 uu[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int o = threadIdx.x + i * kWG, rloc = 32 * h + (o >> 4), r = o & 15, row = t.row0 + rloc;
      const bool upd = kFwd && rloc < t.nrows && row >= w;
      const int2 c = b.fcon2[upd ? frow0 + row : 0];
      c2[i] = upd ? c : make_int2(-1, -1);
      uu[i][0] = *(c2[i].x >= 0 ? ubb + (int64_t)c2[i].x * 16 + r : out + r);
      uu[i][1] = *(c2[i].y >= 0 ? ubb + (int64_t)c2[i].y * 16 + r : out + r);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int o = threadIdx.x + i * kWG;
      const int rloc = 32 * h + (o >> 4), r = o & 15;
      if (rloc < t.nrows) {
        const int q = (rloc >> 4) - 2 * h, rr = rloc & 15;
        int l, j;
        if (sizeof(T) == 8) {  // FP64: row = 4 j + l / 16
          j = rr >> 2;
          l = (rr & 3) * 16 + r;
        } else {               // FP32: row = 4 (l / 16) + j
          j = rr & 3;
          l = (rr >> 2) * 16 + r;
        }
        double ar = 0, ai = 0;
#pragma unroll
        for (int wq = 0; wq < 4; ++wq) {
          ar += (double)red[wq][q][j][l].x;
          ai += (double)red[wq][q][j][l].y;
        }
        const int row = t.row0 + rloc;
        if (!kFwd || row < w) {
          out[(int64_t)(c0 + row) * 16 + r] = make_double2(ar, ai);
        } else {
          add_children(b, frow0 + row, c2[i], uu[i], ubb, r, ar, ai);
          ubb[(int64_t)(uoff + row - w) * 16 + r] = make_double2(ar, ai);
        }
      }
    }
    __syncthreads();
  }
}

// Narrow tiles (at most 96 input columns, 192 with complex64 panels): one wave per tile, all four
// 16-row blocks of the tile in that wave, so there is no cross-wave
// reduction; the accumulators go straight to y / the update vectors (FP64
// accumulator register j of lane l holds row 4 j + l / 16, FP32 row
// 4 (l / 16) + j, right-hand side l % 16).
template <class T, int kFwd, int kCoarse>
__global__ __launch_bounds__(kWG, sizeof(T) == 4 ? 5 : 4) void level_mfma_narrow_kernel(const Tile* __restrict__ tiles, int64_t ntiles,
                                                                Batch b, const typename Mf<T>::C2* __restrict__ G,
                                                                double2* __restrict__ out,
                                                                double2* __restrict__ ubb) {
  using C2 = typename Mf<T>::C2;
  using V4 = typename Mf<T>::V4;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lr = lane & 15, lk = lane >> 4;
  const int64_t ti = (int64_t)blockIdx.x * (kWG / 64) + wv;
  if (ti >= ntiles) return;  // a whole wave; the kernel has no barrier
  const Tile t = tiles[ti];
  const int sn = t.sn, c0 = b.sn_c0[sn], w = b.sn_w[sn];
  const C2* __restrict__ P = reinterpret_cast<const C2*>(kFwd ? b.pf : b.pb) + t.off;
  const C2* Bk = G + (b.goff_f[sn] + t.col0) * 16;  // the staged forward input block
  const int nr = t.nrows, nrb = (nr + 15) >> 4;
  V4 dre[4], dim[4];
#pragma unroll
  for (int rb = 0; rb < 4; ++rb) dre[rb] = dim[rb] = V4{0, 0, 0, 0};
  mfma_stream<T>(P, nr, t.ncols, Bk, 0, 4, dre, dim);
  // per row block, the update rows' child-update pairs, then their values,
  // then the stores (rows without updates read y, any valid address)
  const int frow0 = b.sn_frow0[sn], uoff = b.sn_uoff[sn];
#pragma unroll
  for (int rb = 0; rb < 4; ++rb) {
    if (rb >= nrb) break;
    int2 c2[4];
    double2 uu[4][2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int rloc = 16 * rb + Mf<T>::row(lk, j), row = t.row0 + rloc;
      const bool upd = kFwd && rloc < nr && row >= w;
      const int2 c = b.fcon2[upd ? frow0 + row : 0];
      c2[j] = upd ? c : make_int2(-1, -1);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uu[j][0] = *(c2[j].x >= 0 ? ubb + (int64_t)c2[j].x * 16 + lr : out + lr);
      uu[j][1] = *(c2[j].y >= 0 ? ubb + (int64_t)c2[j].y * 16 + lr : out + lr);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int rloc = 16 * rb + Mf<T>::row(lk, j);
      if (rloc >= nr) continue;
      double ar = (double)dre[rb][j], ai = (double)dim[rb][j];
      const int row = t.row0 + rloc;
      if (!kFwd || row < w) {
        out[(int64_t)(c0 + row) * 16 + lr] = make_double2(ar, ai);
      } else {
        add_children(b, frow0 + row, c2[j], uu[j], ubb, lr, ar, ai);
        ubb[(int64_t)(uoff + row - w) * 16 + lr] = make_double2(ar, ai);
      }
    }
  }
}

// Stages a pass of a tile's input block into G: entries e = base + q stride
// (q < 8) of the cn columns from cb, entry e being column col0 + cb + e / S
// and right-hand side e % S.  Forward: the restricted right-hand side,
// gathered through bidx (restriction, nested-dissection permutation and
// pivot order in one index), minus the children's updates routed to the
// column's front row (at most two, read through fcon2; longer lists through
// fcon_idx).  Backward: the forward result for the pivot columns, the
// ancestors' backward results (through the supernode's row list) for the
// others.  All eight entries' index loads are issued first, then all value
// loads, so a pass costs two memory round trips.  The backward loads are
// unconditional (entries past the pass read a valid dummy address and are
// not stored), so no load waits behind a branch.
template <class T, int kFwd, int S = 16>
__device__ __forceinline__ void stage_pass(const Batch& b, const Tile& t, int cb, int cn, int base, int stride,
                                           typename Mf<T>::C2* G, const double2* __restrict__ src,
                                           const double2* aux) {
  using C2 = typename Mf<T>::C2;
  constexpr int kQ = 8;
  if constexpr (!kFwd) {
    int rv[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const int e = base + q * stride;
      const int c = t.col0 + cb + e / S;
      // an ancestor column reads its position from the row list; the
      // others read bidx[0] (any valid address) and ignore it
      const bool up = e < cn * S && c >= t.w;
      rv[q] = *(up ? b.rows + t.aux + (c - t.w) : b.bidx);
    }
    double2 v[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const int e = base + q * stride;
      const int c = t.col0 + cb + e / S, r = e % S;
      const bool in = e < cn * S;
      v[q] = *(!in ? src + r : (c < t.w ? src + (int64_t)(t.c0 + c) * S + r : aux + (int64_t)rv[q] * S + r));
    }
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const int e = base + q * stride;
      if (e < cn * S) G[e] = C2{(T)v[q].x, (T)v[q].y};
    }
  } else {
    int idx[kQ];
    int2 ch[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const int e = base + q * stride;
      const bool in = e < cn * S;
      const int c = in ? t.col0 + cb + e / S : 0;  // column 0 is always there
      idx[q] = b.bidx[t.c0 + c];
      const int2 f = b.fcon2[t.aux + c];
      ch[q] = in ? f : make_int2(-1, -1);
    }
    // the inputs and the (at most two) updates of four entries at a time, all
    // loads before the first use; missing updates read the input instead
#pragma unroll
    for (int h = 0; h < kQ; h += kQ / 2) {
      double2 v[kQ / 2], u0[kQ / 2], u1[kQ / 2];
#pragma unroll
      for (int q = 0; q < kQ / 2; ++q) {
        const int r = (base + (h + q) * stride) % S;
        const int2 c2 = ch[h + q];
        const double2* in = src + (int64_t)idx[h + q] * S + r;
        v[q] = *in;
        u0[q] = *(c2.x >= 0 ? aux + (int64_t)c2.x * S + r : in);
        u1[q] = *(c2.y >= 0 ? aux + (int64_t)c2.y * S + r : in);
      }
#pragma unroll
      for (int q = 0; q < kQ / 2; ++q) {
        const int e = base + (h + q) * stride;
        if (e >= cn * S) continue;
        const int r = e % S;
        const int2 c2 = ch[h + q];
        double2 w = v[q];
        if (c2.x >= 0) {
          w.x -= u0[q].x;
          w.y -= u0[q].y;
          if (c2.y >= 0) {
            w.x -= u1[q].x;
            w.y -= u1[q].y;
          }
        } else if (c2.x < -1) {
          const int fr = t.aux + t.col0 + cb + e / S;
          for (int k = -2 - c2.x; k < b.fcon_ptr[fr + 1]; ++k) {
            const double2 u = aux[(int64_t)b.fcon_idx[k] * S + r];
            w.x -= u.x;
            w.y -= u.y;
          }
        }
        G[e] = C2{(T)w.x, (T)w.y};
      }
    }
  }
}

constexpr int kCB = 128;  // input columns staged per pass of a wide tile (4 waves)
constexpr int kCBn = 32;  // per pass of a narrow tile (one wave)
// stage_pass stages eight entries per thread
static_assert(kCB * 16 == 8 * kWG && kCBn * 16 == 8 * 64, "a pass is eight entries per thread");

// Output row rloc (of the tile) for right-hand side r: forward pivot rows
// and backward rows go to out; forward update rows add the children's
// updates routed to that front row and go to the supernode's update vector.
template <int kFwd>
__device__ __forceinline__ void put_row(const Batch& b, const Tile& t, int rloc, int r, double ar, double ai,
                                        double2* out, double2* ubb) {
  const int row = t.row0 + rloc;
  if (!kFwd || row < t.w) {
    out[(int64_t)(t.c0 + row) * 16 + r] = make_double2(ar, ai);
  } else {
    const int fr = t.aux + row;
    for (int e = b.fcon_ptr[fr]; e < b.fcon_ptr[fr + 1]; ++e) {
      const double2 u = ubb[(int64_t)b.fcon_idx[e] * 16 + r];
      ar += u.x;
      ai += u.y;
    }
    ubb[(int64_t)(b.sn_uoff[t.sn] + row - t.w) * 16 + r] = make_double2(ar, ai);
  }
}

// One level of the 16-right-hand-side backward sweep, the input gather
// fused in (a backward tile holds all input columns of its rows, so a narrow
// supernode's input is gathered once; the forward sweep keeps the staged
// gather, whose supernodes have several row tiles over the same input): a
// workgroup stages its tile's input block (16 right-hand sides per column)
// in LDS a pass of columns at a time and multiplies the panel tile into it
// on MFMA.  Workgroups [0, nwide) take one wide tile each (its k-steps
// shared by the four waves, wave q taking q, q + 4, ..., partial sums added
// through LDS); the others take four narrow tiles, a wave each.
template <class T, int kFwd, int kCoarse>
__global__ __launch_bounds__(kWG, 3) void level_fused_kernel(const Tile* __restrict__ tiles, int64_t ntiles,
                                                          int64_t nwide, Batch b, const double2* __restrict__ src,
                                                          const double2* aux, double2* out, double2* ubb) {
  using C2 = typename Mf<T>::C2;
  using V4 = typename Mf<T>::V4;
  __shared__ C2 G[kCB * 16];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lr = lane & 15,
            lk = lane >> 4;
  V4 dre[4], dim[4];
#pragma unroll
  for (int rb = 0; rb < 4; ++rb) dre[rb] = dim[rb] = V4{0, 0, 0, 0};
  const C2* __restrict__ panels = reinterpret_cast<const C2*>(kFwd ? b.pf : b.pb);
  if ((int64_t)blockIdx.x < nwide) {
    const Tile t = tiles[blockIdx.x];
    for (int cb = 0; cb < t.ncols; cb += kCB) {
      const int cn = min(kCB, t.ncols - cb);
      stage_pass<T, kFwd>(b, t, cb, cn, threadIdx.x, kWG, G, src, aux);
      __syncthreads();
      mfma_stream<T>(panels + t.off + (int64_t)cb * t.nrows, t.nrows, cn, G, 4 * wv, 16, dre, dim);
      __syncthreads();
    }
    // partial sums of the 4 waves, two row blocks at a time, in the staging
    // buffer: [wave][rb2][j][lane] (4 x 2 x 4 x 64 = kCB x 16 entries)
    C2 (*red)[2][4][64] = reinterpret_cast<C2 (*)[2][4][64]>(G);
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int j = 0; j < 4; ++j) red[wv][q][j][lane] = C2{dre[2 * h + q][j], dim[2 * h + q][j]};
      __syncthreads();
      // 512 outputs (32 rows x 16 right-hand sides) of this half, 2 per thread
      for (int o = threadIdx.x; o < 512; o += kWG) {
        const int rloc = 32 * h + (o >> 4), r = o & 15;
        if (rloc < t.nrows) {
          const int q = (rloc >> 4) - 2 * h, rr = rloc & 15;
          int l, j;
          if (sizeof(T) == 8) {  // FP64: row = 4 j + l / 16
            j = rr >> 2;
            l = (rr & 3) * 16 + r;
          } else {               // FP32: row = 4 (l / 16) + j
            j = rr & 3;
            l = (rr >> 2) * 16 + r;
          }
          double ar = 0, ai = 0;
#pragma unroll
          for (int wq = 0; wq < 4; ++wq) {
            ar += (double)red[wq][q][j][l].x;
            ai += (double)red[wq][q][j][l].y;
          }
          put_row<kFwd>(b, t, rloc, r, ar, ai, out, ubb);
        }
      }
      __syncthreads();
    }
    return;
  }
  // narrow tiles: a wave each, the staging buffer split into four
  const int64_t g0 = nwide + ((int64_t)blockIdx.x - nwide) * 4;
  const int64_t ti = g0 + wv;
  const bool has = ti < ntiles;
  Tile t{};
  if (has) t = tiles[ti];
  int np = 0;  // passes: the most any tile of the workgroup needs (uniform)
  for (int q = 0; q < 4; ++q)
    if (g0 + q < ntiles) np = max(np, (tiles[g0 + q].ncols + kCBn - 1) / kCBn);
  C2* Gw = G + wv * kCBn * 16;
  const int nr = t.nrows, nrb = (nr + 15) >> 4;
  const C2* __restrict__ P = panels + t.off;
  for (int p = 0; p < np; ++p) {
    const int cb = p * kCBn;
    const int cn = has ? max(0, min(kCBn, t.ncols - cb)) : 0;
    stage_pass<T, kFwd>(b, t, cb, cn, lane, 64, Gw, src, aux);
    __syncthreads();
    mfma_stream<T>(P + (int64_t)cb * nr, nr, cn, Gw, 0, 4, dre, dim);
    __syncthreads();
  }
  if (!has) return;
#pragma unroll
  for (int rb = 0; rb < 4; ++rb) {
    if (rb >= nrb) break;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int rloc = 16 * rb + Mf<T>::row(lk, j);
      if (rloc < nr) put_row<kFwd>(b, t, rloc, lr, (double)dre[rb][j], (double)dim[rb][j], out, ubb);
    }
  }
}

// ---- MFMA form for 2, 4 and 8 right-hand sides ------------------------------
// With at most eight right-hand sides the 16 columns of an MFMA hold the real
// and the imaginary parts side by side: with B1 = [Bre | Bim] and
// B2 = [-Bim | Bre], D = Are B1 + Aim B2 = [Dre | Dim], two MFMAs per four
// columns and 16 rows instead of four.  Always FP64 MFMA, also for complex64
// panels (widened in registers): these widths accumulate in FP64.
// Measured at 8 columns, 168,075 unknowns, complex64 panels (1.05 GB), one
// forward or backward level of one of two batches: 76 / 131 us with one lane
// per tile row and FP64 vector arithmetic, 22 / 20 us so (five right-hand sides
// solved together: 37.4 -> 12.2 ms).  Bound by latencies on operators of that
// size (staging, panel, epilogue), by HBM on large ones.
//
// Panel entries through raw buffer loads (range checked in bytes against the
// buffer's size, out of range reads give zero; non-temporal): the k-step's offset
// is scalar, a lane's offset constant.  The check is lane offset >= size - scalar
// offset, so the scalar offset must not pass the size.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const void* p, int bytes) {
  const int64_t a = reinterpret_cast<int64_t>(p);
  const int lo = __builtin_amdgcn_readfirstlane((int)a), hi = __builtin_amdgcn_readfirstlane((int)(a >> 32));
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(((int64_t)hi << 32) | (uint32_t)lo), 0,
                                           __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}
template <class PT>
__device__ __forceinline__ PT ldb(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  constexpr int kNt = 2;
  if constexpr (sizeof(PT) == 16)
    return __builtin_bit_cast(PT, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, kNt));
  else
    return __builtin_bit_cast(PT, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, kNt));
}

// Streams the k-steps k0 = ks0, ks0 + kst, ... < cn of a panel tile (nr rows,
// ld apart, at most NRB 16-row blocks) against the staged block Bk (S
// right-hand sides per column).  D k-steps of panel loads stay in flight, each
// register set refilled right after its MFMAs; rows past nr read row nr - 1,
// columns past cn lie past the buffer.  (64-bit lane addresses took 50 more
// registers in the backward kernels, three waves per SIMD instead of five: a step
// of 8 right-hand sides at 168,075 unknowns 1,051 -> 1,034 us, at 370,301 2,189 ->
// 2,146, complex64 panels.  Twice the k-steps with complex64: 1,071 and 2,210;
// four waves in the forward kernels, which then spill: 1,130 and 2,252.)  (With two k-steps in flight a level of a small operator took
// 20-25 us, most of it panel latency.)
template <class PT, int S, int NRB, int D>
__device__ __forceinline__ void mfma_stream_small(const PT* __restrict__ P, int ld, int nr, int cn,
                                                  const double2* __restrict__ Bk, int ks0, int kst, dv4* d) {
  if (ks0 >= cn) return;  // uniform: the wave has no k-step
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4, r = lr & 7;
  const bool im = lr >= 8, used = r < S;
  const int rs = used ? r : 0;
  constexpr int esz = sizeof(PT);
  const int bytes = ((cn - 1) * ld + nr) * esz;
  const __amdgpu_buffer_rsrc_t buf = tile_rsrc(P, bytes);
  int voff[NRB];
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) voff[rb] = (lk * ld + min(16 * rb + lr, nr - 1)) * esz;
  PT a[D][NRB];
  auto load = [&](int k0, PT (&w)[NRB]) {
    const int soff = __builtin_amdgcn_readfirstlane(min(k0 * ld * esz, bytes));
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) w[rb] = ldb<PT>(buf, voff[rb], soff);
  };
  auto step = [&](int k0, const PT (&w)[NRB]) {
    const double2 b = Bk[min(k0 + lk, cn - 1) * S + rs];
    const bool in = used && k0 + lk < cn;
    const double b1 = in ? (im ? b.y : b.x) : 0.0, b2 = in ? (im ? b.x : -b.y) : 0.0;
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
      if (rb == 0 || 16 * rb < nr) {  // uniform
        const double2 v = widen(w[rb]);
        d[rb] = Mf<double>::mma(v.x, b1, d[rb]);
        d[rb] = Mf<double>::mma(v.y, b2, d[rb]);
      }
  };
#pragma unroll
  for (int u = 0; u < D; ++u) load(ks0 + u * kst, a[u]);
  int n = (cn - ks0 + kst - 1) / kst, k0 = ks0;  // k-steps from k0 on
  for (; n >= 2 * D; n -= D, k0 += D * kst) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      step(k0 + u * kst, a[u]);
      load(k0 + (u + D) * kst, a[u]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  for (; n > 0; n -= D, k0 += D * kst) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      if (u < n) step(k0 + u * kst, a[u]);
      if (u + D < n) load(k0 + (u + D) * kst, a[u]);
    }
  }
}

// Stores the rows row0 + 4 j + lk (j < 4, those below nr) of a tile, component
// c = 2 r + (0: real, 1: imaginary) of the interleaved block rows: forward
// pivot rows and backward rows go to out; forward update rows add the
// children's updates and go to the supernode's update vector.  Index pairs,
// then values, then stores.
template <int kFwd, int S>
__device__ __forceinline__ void put_small(const Batch& b, const Tile& t, int uoff, int rloc0, int nr, int c, double* v,
                                          double* out, double* ubb) {
  const int lk = (threadIdx.x & 63) >> 4;
  if constexpr (!kFwd) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int rloc = rloc0 + 4 * j + lk;
      if (rloc < nr) out[(int64_t)(t.c0 + t.row0 + rloc) * (2 * S) + c] = v[j];
    }
  } else {
    int2 c2[4];
    double u0[4], u1[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int rloc = rloc0 + 4 * j + lk, row = t.row0 + rloc;
      const bool upd = rloc < nr && row >= t.w;
      const int2 f = b.fcon2[t.aux + (upd ? row : 0)];
      c2[j] = upd ? f : make_int2(-1, -1);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {  // a missing child reads out's first row instead
      u0[j] = *(c2[j].x >= 0 ? ubb + (int64_t)c2[j].x * (2 * S) + c : out + c);
      u1[j] = *(c2[j].y >= 0 ? ubb + (int64_t)c2[j].y * (2 * S) + c : out + c);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int rloc = rloc0 + 4 * j + lk, row = t.row0 + rloc;
      if (rloc >= nr) continue;
      double x = v[j];
      if (row < t.w) {
        out[(int64_t)(t.c0 + row) * (2 * S) + c] = x;
        continue;
      }
      if (c2[j].x >= 0) {
        x += u0[j];
        if (c2[j].y >= 0) x += u1[j];
      } else if (c2[j].x < -1) {
        for (int e = -2 - c2[j].x; e < b.fcon_ptr[t.aux + row + 1]; ++e)
          x += ubb[(int64_t)b.fcon_idx[e] * (2 * S) + c];
      }
      ubb[(int64_t)(uoff + row - t.w) * (2 * S) + c] = x;
    }
  }
}

// One level of a sweep for S right-hand sides.  Workgroups [0, nwide split),
// split = 4 / NRB, take a wide tile's rows in ranges of NRB 16-row blocks (1, 2
// or 4: levels of few tiles spread over the device), the k-steps shared by the
// four waves, partial sums added through LDS; with NRB = 4 the others take four
// narrow tiles, a wave each.  Every workgroup stages its tile's inputs in LDS, a pass of
// columns at a time (eight entries per thread).
template <class PT, int kFwd, int S, int kCoarse, int NRB>
__global__ __launch_bounds__(kWG, 3) void level_small_kernel(const Tile* __restrict__ tiles, int64_t ntiles,
                                                             int64_t nwide, Batch b, const double2* __restrict__ src,
                                                             const double2* aux,
                                                             double* out, double* ubb) {
  constexpr int kC = 8 * kWG / S, kCn = kC / 4;  // columns per pass: wide tile, narrow tile
  constexpr int split = 4 / NRB, D = 8 / NRB;
  __shared__ double2 G[8 * kWG];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lr = lane & 15,
            r = lr & 7;
  const int c = 2 * r + (lr >> 3);  // component of this lane's MFMA column
  const PT* __restrict__ panels = reinterpret_cast<const PT*>(kFwd ? b.pf : b.pb);
  dv4 d[NRB];
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) d[rb] = dv4{0, 0, 0, 0};
  if ((int64_t)blockIdx.x < nwide * split) {
    const Tile t = tiles[blockIdx.x / split];
    constexpr int h = 64 / split;
    const int r0 = (int)(blockIdx.x % split) * h, nr = min(h, t.nrows - r0);
    if (nr <= 0) return;  // the whole workgroup
    const int uoff = kFwd ? b.sn_uoff[t.sn] : 0;
    for (int cb = 0; cb < t.ncols; cb += kC) {
      const int cn = min(kC, t.ncols - cb);
      stage_pass<double, kFwd, S>(b, t, cb, cn, threadIdx.x, kWG, G, src, aux);
      __syncthreads();
      mfma_stream_small<PT, S, NRB, D>(panels + t.off + (int64_t)cb * t.nrows + r0, t.nrows, nr, cn, G, 4 * wv, 16, d);
      __syncthreads();
    }
    // partial sums of the four waves: [wave][rb][j][lane] (4 x 4 x 4 x 64
    // doubles = the staging buffer)
    double (*red)[4][4][64] = reinterpret_cast<double (*)[4][4][64]>(G);
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
      for (int j = 0; j < 4; ++j) red[wv][rb][j][lane] = d[rb][j];
    __syncthreads();
    // wave q sums and stores row block q (row = 4 j + l / 16)
    if (r < S && 16 * wv < nr) {
      double v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        v[j] = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[j] += red[q][wv][j][lane];
      }
      put_small<kFwd, S>(b, t, uoff, r0 + 16 * wv, r0 + nr, c, v, out, ubb);
    }
    return;
  }
  if constexpr (NRB == 4) {
  const int64_t g0 = nwide + ((int64_t)blockIdx.x - nwide * split) * 4;
  const int64_t ti = g0 + wv;
  const bool has = ti < ntiles;
  Tile t{};
  if (has) t = tiles[ti];
  int np = 0;  // passes: the most any tile of the workgroup needs (uniform)
  for (int q = 0; q < 4; ++q)
    if (g0 + q < ntiles) np = max(np, (tiles[g0 + q].ncols + kCn - 1) / kCn);
  double2* Gw = G + wv * kCn * S;
  const int uoff = kFwd && has ? b.sn_uoff[t.sn] : 0;
  for (int p = 0; p < np; ++p) {
    const int cb = p * kCn;
    const int cn = has ? max(0, min(kCn, t.ncols - cb)) : 0;
    stage_pass<double, kFwd, S>(b, t, cb, cn, lane, 64, Gw, src, aux);
    __syncthreads();
    mfma_stream_small<PT, S, NRB, D>(panels + t.off + (int64_t)cb * t.nrows, t.nrows, t.nrows, cn, Gw, 0, 4, d);
    __syncthreads();
  }
  if (!has || r >= S) return;
#pragma unroll
  for (int rb = 0; rb < 4; ++rb)
    if (16 * rb < t.nrows) {
      double v[4] = {d[rb][0], d[rb][1], d[rb][2], d[rb][3]};
      put_small<kFwd, S>(b, t, uoff, 16 * rb, t.nrows, c, v, out, ubb);
    }
  }
}

// Entry n of the 16 a row's lanes hold, on all lanes of the row (DPP broadcast
// within 16 lanes).
template <int N>
__device__ __forceinline__ int row_bcast(int x) {
  return __builtin_amdgcn_update_dpp(0, x, 0x150 + N, 0xf, 0xf, false);
}
template <int N>
__device__ __forceinline__ double row_bcast(double x) {
  const long long v = __double_as_longlong(x);
  const int lo = row_bcast<N>((int)v), hi = row_bcast<N>((int)(v >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Calls f(u, col, val, x entry) for the entries [p, p1) of a sparse row, in order
// (u: the entry's place in its group), for one of S interleaved right-hand sides;
// xs(c) is the x entry of column c.  With 16 right-hand sides the row's sixteen
// lanes load sixteen entries at once and hand them round: one load of columns
// and one of values per sixteen entries instead of sixteen each (the loads of a
// product are bound by the L1s' 64 B per clock: 782 -> 558 us at one million
// unknowns, with real instead of complex entries).  Gathers go eight at a time.
template <int N0, class X, class F, int... N>
__device__ __forceinline__ void row_group8(int c, double v, int cnt, X&& xs, F&& f, std::integer_sequence<int, N...>) {
  const int cc[8] = {row_bcast<N0 + N>(c)...};
  const double vv[8] = {row_bcast<N0 + N>(v)...};
  double2 xv[8];
#pragma unroll
  for (int u = 0; u < 8; ++u)
    if (N0 + u < cnt) xv[u] = xs(cc[u]);
#pragma unroll
  for (int u = 0; u < 8; ++u)
    if (N0 + u < cnt) f(u, cc[u], vv[u], xv[u]);
}

template <int S, class X, class F>
__device__ __forceinline__ void for_row(const int32_t* __restrict__ col, const double* __restrict__ val, int64_t p,
                                        int64_t p1, X&& xs, F&& f) {
  if constexpr (S == 16) {
    const int r = threadIdx.x & 15;
    for (; p < p1; p += 16) {
      const int cnt = (int)min((int64_t)16, p1 - p);
      const int64_t q = p + min(r, cnt - 1);
      const int c = col[q];
      const double v = val[q];
      constexpr std::make_integer_sequence<int, 8> seq{};
      row_group8<0>(c, v, cnt, xs, f, seq);
      if (cnt > 8) row_group8<8>(c, v, cnt, xs, f, seq);
    }
  } else {
    for (; p + 8 <= p1; p += 8) {
      int c[8];
      double v[8];
      double2 xv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) c[u] = col[p + u];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = val[p + u];
#pragma unroll
      for (int u = 0; u < 8; ++u) xv[u] = xs(c[u]);
#pragma unroll
      for (int u = 0; u < 8; ++u) f(u, c[u], v[u], xv[u]);
    }
    for (int u = 0; p < p1; ++p, ++u) f(u, col[p], val[p], xs(col[p]));
  }
}

// Block SpMV: S consecutive lanes share a row and take one right-hand side each,
// so every x gather is one contiguous S x 16 B line.  A row without imaginary parts
// (as many entries in the split storage as in the complex one: with real
// velocities all but the rows on absorbing faces) reads its real entries only; the
// others read the complex ones.
// Even entries sum into a, odd ones into b, alike on both routes.  With kXcd, XCD k
// sweeps the rows [xr[k], xr[k+1]) (as in the single-vector kernel).
template <int S, bool kXcd>
__global__ __launch_bounds__(kWG) void spmv_block_kernel(
    int64_t n, const int64_t* __restrict__ aptr, const int32_t* __restrict__ acol, const double2* __restrict__ aval,
    const int64_t* __restrict__ sptr, const int32_t* __restrict__ scol, const double* __restrict__ sval,
    const int64_t* __restrict__ xr, const double2* __restrict__ x, const double2* __restrict__ bvec,
    double2* __restrict__ y) {
  const int r = threadIdx.x % S;
  int64_t i = ((int64_t)(kXcd ? blockIdx.x >> 3 : blockIdx.x) * kWG + threadIdx.x) / S, end = n;
  if (kXcd) {
    i += xr[blockIdx.x & 7];
    end = xr[(blockIdx.x & 7) + 1];
  }
  if (i >= end) return;
  const int64_t e = i * S + r;
  double ar = 0, ai = 0, br = 0, bi = 0;
  int64_t p = aptr[i];
  const int64_t p1 = aptr[i + 1], q = sptr[i], q1 = sptr[i + 1];
  if (q1 - q == p1 - p) {
    for_row<S>(scol, sval, q, q1, [&](int c) { return x[(int64_t)c * S + r]; }, [&](int u, int, double v, double2 xv) {
      double& sr = u & 1 ? br : ar;
      double& si = u & 1 ? bi : ai;
      sr = fma(v, xv.x, sr);
      si = fma(v, xv.y, si);
    });
  } else {
    for (; p + 8 <= p1; p += 8) {
      int c[8];
      double2 v[8], xv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) c[u] = acol[p + u];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = aval[p + u];
#pragma unroll
      for (int u = 0; u < 8; ++u) xv[u] = x[(int64_t)c[u] * S + r];
#pragma unroll
      for (int u = 0; u < 8; u += 2) {
        cfma(ar, ai, v[u], xv[u]);
        cfma(br, bi, v[u + 1], xv[u + 1]);
      }
    }
    for (; p + 2 <= p1; p += 2) {
      const int c0 = acol[p], c1 = acol[p + 1];
      const double2 v0 = aval[p], v1 = aval[p + 1];
      cfma(ar, ai, v0, x[(int64_t)c0 * S + r]);
      cfma(br, bi, v1, x[(int64_t)c1 * S + r]);
    }
    if (p < p1) cfma(ar, ai, aval[p], x[(int64_t)acol[p] * S + r]);
  }
  ar += br;
  ai += bi;
  if (bvec) {
    const double2 bb = bvec[e];
    y[e] = make_double2(bb.x - ar, bb.y - ai);
  } else {
    y[e] = make_double2(ar, ai);
  }
}

template <int S>
__global__ __launch_bounds__(kWG) void spmv_real_block_kernel(int64_t n, const int64_t* __restrict__ ptr,
                                                              const int32_t* __restrict__ col,
                                                              const double* __restrict__ val,
                                                              const double2* __restrict__ x, double2* __restrict__ y) {
  const int64_t e = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (e >= n * S) return;
  const int64_t row = e / S;
  const int r = (int)(e % S);
  double ar = 0, ai = 0;
  const int64_t p1 = ptr[row + 1];
  int64_t p = ptr[row];
  // eight entries per step (loads first, then the multiply-adds in order)
  for (; p + 8 <= p1; p += 8) {
    int c[8];
    double a[8];
    double2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) c[u] = col[p + u];
#pragma unroll
    for (int u = 0; u < 8; ++u) a[u] = val[p + u];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = x[(int64_t)c[u] * S + r];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      ar = fma(a[u], v[u].x, ar);
      ai = fma(a[u], v[u].y, ai);
    }
  }
  for (; p < p1; ++p) {
    const double a = val[p];
    const double2 v = x[(int64_t)col[p] * S + r];
    ar = fma(a, v.x, ar);
    ai = fma(a, v.y, ai);
  }
  y[e] = make_double2(ar, ai);
}

// t = x - (A Z) cx for S interleaved right-hand sides (A Z in split storage: bit
// 31 of a column marks an imaginary part).
template <int S>
__global__ __launch_bounds__(kWG) void coarse_update_block_kernel(int64_t n, const int64_t* __restrict__ aptr,
                                                                  const int32_t* __restrict__ acol,
                                                                  const double* __restrict__ aval,
                                                                  const double2* __restrict__ cx,
                                                                  const double2* __restrict__ x,
                                                                  double2* __restrict__ t) {
  const int64_t e = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (e >= n * S) return;
  const int64_t row = e / S;
  const int r = (int)(e % S);
  double ar = 0, ai = 0;
  for_row<S>(acol, aval, aptr[row], aptr[row + 1], [&](int c) { return cx[(int64_t)(c & 0x7fffffff) * S + r]; },
             [&](int, int c, double a, double2 v) {
               const bool im = c < 0;  // i v = (-v.y, v.x)
               ar = fma(a, im ? -v.y : v.x, ar);
               ai = fma(a, im ? v.x : v.y, ai);
             });
  const double2 xx = x[e];
  t[e] = make_double2(xx.x - ar, xx.y - ai);
}

// z = Z cx + sum of the weighted local results, cx null for one level.  The
// coarse part is formed here from the coarse solution, which the caches hold,
// instead of being written by the coarse update and read back (16 right-hand sides
// at one million unknowns: the coarse stage 796 -> 642 us, this one 167 -> 218).
template <int S>
__global__ __launch_bounds__(kWG) void prolong_block_kernel(int64_t n, const int64_t* __restrict__ ptr,
                                                            const int32_t* __restrict__ idx,
                                                            const double* __restrict__ w,
                                                            const double2* __restrict__ xl,
                                                            const int64_t* __restrict__ zptr,
                                                            const int32_t* __restrict__ zcol,
                                                            const double* __restrict__ zval,
                                                            const double2* __restrict__ cx, double2* __restrict__ z) {
  const int64_t e = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (e >= n * S) return;
  const int64_t g = e / S;
  const int r = (int)(e % S);
  double ar = 0, ai = 0;
  auto add = [&](int, int, double c, double2 v) {
    ar = fma(c, v.x, ar);
    ai = fma(c, v.y, ai);
  };
  if (cx) for_row<S>(zcol, zval, zptr[g], zptr[g + 1], [&](int c) { return cx[(int64_t)c * S + r]; }, add);
  for_row<S>(idx, w, ptr[g], ptr[g + 1], [&](int i) { return xl[(int64_t)i * S + r]; }, add);
  z[e] = make_double2(ar, ai);
}

template <int S>
__global__ __launch_bounds__(kWG) void pack_kernel(int64_t n, PtrSetC src, double2* __restrict__ dst) {
  const int64_t e = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (e >= n * S) return;
  const int64_t i = e / S;
  const int r = (int)(e % S);
  const double2* p = reinterpret_cast<const double2*>(src.p[r]);
  dst[e] = p ? p[i] : make_double2(0.0, 0.0);
}

template <int S>
__global__ __launch_bounds__(kWG) void unpack_kernel(int64_t n, const double2* __restrict__ src, PtrSet dst) {
  const int64_t e = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (e >= n * S) return;
  const int64_t i = e / S;
  const int r = (int)(e % S);
  double2* p = reinterpret_cast<double2*>(dst.p[r]);
  if (p) p[i] = src[e];
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kWG - 1) / kWG); }

// Calls f(std::integral_constant<int, S>) for the supported block widths.
template <class F>
void with_width(int S, F&& f) {
  switch (S) {
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 16: f(std::integral_constant<int, 16>{}); break;
    default: break;
  }
}

}  // namespace

// Launch of level_small_kernel: all tiles take four waves on levels of at most
// 2048 tiles (a wave per tile would leave most of the 1024 SIMDs idle), and a
// tile's rows are split over workgroups while those stay within 512, two per
// CU (a block step of 8 right-hand sides at 138,000 unknowns: 1,094 us unsplit,
// 1,018 so).
template <class PT, int kFwd, int S, int kCoarse>
static void small_go(const Batch& b, const Tile* tiles, int64_t ntiles, int64_t nwide, const double* src,
                     const double* aux, double* out, double* ubb, hipStream_t s) {
  if (ntiles <= 2048) nwide = ntiles;
  auto in = reinterpret_cast<const double2*>(src);
  auto au = reinterpret_cast<const double2*>(aux);
  if (ntiles <= 128)
    level_small_kernel<PT, kFwd, S, kCoarse, 1><<<(unsigned)(4 * ntiles), kWG, 0, s>>>(tiles, ntiles, nwide, b, in, au, out, ubb);
  else if (ntiles <= 256)
    level_small_kernel<PT, kFwd, S, kCoarse, 2><<<(unsigned)(2 * ntiles), kWG, 0, s>>>(tiles, ntiles, nwide, b, in, au, out, ubb);
  else
    level_small_kernel<PT, kFwd, S, kCoarse, 4><<<(unsigned)(nwide + (ntiles - nwide + 3) / 4), kWG, 0, s>>>(
        tiles, ntiles, nwide, b, in, au, out, ubb);
}

template <int kFwd, int S>
static void small_launch(const Batch& b, const Tile* tiles, int64_t ntiles, int64_t nwide, const double* src,
                         const double* aux, double* out, double* ubb, bool coarse, hipStream_t s) {
  if (coarse)
    small_go<double2, kFwd, S, 1>(b, tiles, ntiles, nwide, src, aux, out, ubb, s);
  else if (b.c64)
    small_go<float2, kFwd, S, 0>(b, tiles, ntiles, nwide, src, aux, out, ubb, s);
  else
    small_go<double2, kFwd, S, 0>(b, tiles, ntiles, nwide, src, aux, out, ubb, s);
}

template <int kFwd>
static void level_small(const Batch& b, const Tile* tiles, int64_t ntiles, int64_t nwide, int S, const double* src,
                        const double* aux, double* out, double* ubb, bool coarse, hipStream_t s) {
  if (S == 2)
    small_launch<kFwd, 2>(b, tiles, ntiles, nwide, src, aux, out, ubb, coarse, s);
  else if (S == 4)
    small_launch<kFwd, 4>(b, tiles, ntiles, nwide, src, aux, out, ubb, coarse, s);
  else
    small_launch<kFwd, 8>(b, tiles, ntiles, nwide, src, aux, out, ubb, coarse, s);
}

void fwd_level_block(const Batch& b, int64_t tile0, int64_t ntiles, int64_t nwide, int S, const double* bin, double* yb,
                     double* ubb, bool coarse, hipStream_t s) {
  if (ntiles <= 0) return;
  level_small<1>(b, b.tf + tile0, ntiles, nwide, S, bin, ubb, yb, ubb, coarse, s);
}

void bwd_level_block(const Batch& b, int64_t tile0, int64_t ntiles, int64_t nwide, int S, const double* yb, double* xb,
                     bool coarse, hipStream_t s) {
  if (ntiles <= 0) return;
  level_small<0>(b, b.tb + tile0, ntiles, nwide, S, yb, xb, xb, nullptr, coarse, s);
}

// Tiles [tile0, tile0 + nwide) go to the 4-wave kernel, the rest (narrow,
// at the end of the level) to the one-wave-per-tile kernel.
template <class T, int kFwd, int kCoarse>
void level_mfma_launch(const Batch& b, const Tile* tiles, int64_t ntiles, int64_t nwide,
                       const typename Mf<T>::C2* G, double2* out, double2* u, hipStream_t s) {
  if (nwide > 0) level_mfma_kernel<T, kFwd, kCoarse><<<(unsigned)nwide, kWG, 0, s>>>(tiles, b, G, out, u);
  const int64_t nn = ntiles - nwide;
  if (nn > 0)
    level_mfma_narrow_kernel<T, kFwd, kCoarse><<<(unsigned)((nn + 3) / 4), kWG, 0, s>>>(tiles + nwide, nn, b, G, out,
                                                                                        u);
}

void fwd_level_mfma(const Batch& b, const int32_t* sns, int64_t nsn, int gy, int64_t tile0, int64_t ntiles,
                    int64_t nwide, const double* bin, double* yb, double* ubb, void* stage, bool coarse,
                    hipStream_t s) {
  if (ntiles <= 0) return;
  auto in = reinterpret_cast<const double2*>(bin);
  auto y = reinterpret_cast<double2*>(yb);
  auto u = reinterpret_cast<double2*>(ubb);
  if (b.c64 && !coarse) {
    auto G = reinterpret_cast<float2*>(stage);
    gather_fwd_kernel<float><<<dim3((unsigned)nsn, (unsigned)gy), kWG, 0, s>>>(sns, b, in, u, G);
    level_mfma_launch<float, 1, 0>(b, b.tf + tile0, ntiles, nwide, G, y, u, s);
  } else {
    auto G = reinterpret_cast<double2*>(stage);
    gather_fwd_kernel<double><<<dim3((unsigned)nsn, (unsigned)gy), kWG, 0, s>>>(sns, b, in, u, G);
    if (coarse)
      level_mfma_launch<double, 1, 1>(b, b.tf + tile0, ntiles, nwide, G, y, u, s);
    else
      level_mfma_launch<double, 1, 0>(b, b.tf + tile0, ntiles, nwide, G, y, u, s);
  }
}

// One launch per level: nwide wide tiles (the level's first ones) take a
// workgroup each, the narrow ones four per workgroup.
template <class T, int kCoarse>
void bwd_fused_launch(const Batch& b, const Tile* tiles, int64_t ntiles, int64_t nwide, const double2* y, double2* x,
                      hipStream_t s) {
  const int64_t grid = nwide + (ntiles - nwide + 3) / 4;
  level_fused_kernel<T, 0, kCoarse><<<(unsigned)grid, kWG, 0, s>>>(tiles, ntiles, nwide, b, y, x, x, nullptr);
}

void bwd_level_mfma(const Batch& b, int64_t tile0, int64_t ntiles, int64_t nwide, const double* yb, double* xb,
                    bool coarse, hipStream_t s) {
  if (ntiles <= 0) return;
  auto y = reinterpret_cast<const double2*>(yb);
  auto x = reinterpret_cast<double2*>(xb);
  if (b.c64 && !coarse)
    bwd_fused_launch<float, 0>(b, b.tb + tile0, ntiles, nwide, y, x, s);
  else if (coarse)
    bwd_fused_launch<double, 1>(b, b.tb + tile0, ntiles, nwide, y, x, s);
  else
    bwd_fused_launch<double, 0>(b, b.tb + tile0, ntiles, nwide, y, x, s);
}

void spmv_block(int64_t n, const SpmvBlock& A, const int64_t* xr, int64_t xrows, int S, const double* x,
                const double* b, double* y, hipStream_t s) {
  if (n <= 0) return;
  with_width(S, [&](auto w) {
    constexpr int W = decltype(w)::value;
    auto v2 = reinterpret_cast<const double2*>(A.aval);
    auto x2 = reinterpret_cast<const double2*>(x);
    auto b2 = reinterpret_cast<const double2*>(b);
    auto y2 = reinterpret_cast<double2*>(y);
    if (xr)
      spmv_block_kernel<W, true><<<8 * blocks_for(xrows * W), kWG, 0, s>>>(n, A.aptr, A.acol, v2, A.sptr, A.scol,
                                                                           A.sval, xr, x2, b2, y2);
    else
      spmv_block_kernel<W, false><<<blocks_for(n * W), kWG, 0, s>>>(n, A.aptr, A.acol, v2, A.sptr, A.scol, A.sval,
                                                                    nullptr, x2, b2, y2);
  });
}

void spmv_real_block(int64_t n, const int64_t* ptr, const int32_t* col, const double* val, int S, const double* x,
                     double* y, hipStream_t s) {
  if (n <= 0) return;
  with_width(S, [&](auto w) {
    constexpr int W = decltype(w)::value;
    spmv_real_block_kernel<W><<<blocks_for(n * W), kWG, 0, s>>>(n, ptr, col, val, reinterpret_cast<const double2*>(x),
                                                                 reinterpret_cast<double2*>(y));
  });
}

void coarse_update_block(int64_t n, const int64_t* aptr, const int32_t* acol, const double* aval, int S,
                         const double* cx, const double* x, double* t, hipStream_t s) {
  if (n <= 0) return;
  with_width(S, [&](auto w) {
    constexpr int W = decltype(w)::value;
    coarse_update_block_kernel<W><<<blocks_for(n * W), kWG, 0, s>>>(
        n, aptr, acol, aval, reinterpret_cast<const double2*>(cx), reinterpret_cast<const double2*>(x),
        reinterpret_cast<double2*>(t));
  });
}

void prolong_block(int64_t n, const int64_t* ptr, const int32_t* idx, const double* wt, int S, const double* xl,
                   const int64_t* zptr, const int32_t* zcol, const double* zval, const double* cx, double* z,
                   hipStream_t s) {
  if (n <= 0) return;
  with_width(S, [&](auto w) {
    constexpr int W = decltype(w)::value;
    prolong_block_kernel<W><<<blocks_for(n * W), kWG, 0, s>>>(
        n, ptr, idx, wt, reinterpret_cast<const double2*>(xl), zptr, zcol, zval, reinterpret_cast<const double2*>(cx),
        reinterpret_cast<double2*>(z));
  });
}

void pack(int64_t n, int S, const PtrSetC& src, double* dst, hipStream_t s) {
  if (n <= 0) return;
  with_width(S, [&](auto w) {
    constexpr int W = decltype(w)::value;
    pack_kernel<W><<<blocks_for(n * W), kWG, 0, s>>>(n, src, reinterpret_cast<double2*>(dst));
  });
}

void unpack(int64_t n, int S, const double* src, const PtrSet& dst, hipStream_t s) {
  if (n <= 0) return;
  with_width(S, [&](auto w) {
    constexpr int W = decltype(w)::value;
    unpack_kernel<W><<<blocks_for(n * W), kWG, 0, s>>>(n, reinterpret_cast<const double2*>(src), dst);
  });
}

}  // namespace dev
}  // namespace helm
