// Copies between views linearised in different orders (Sec. 2 array
// extents: row-major or column-major).  dst(a) = src(a) for every multi-index
// a: a batched 2-D transpose of records through LDS.  A workgroup takes one
// tile of TP x TQ records: for each of TP positions p along the destination's
// fastest axis P it loads TQ records that are consecutive in the source (along
// Q), and for each of the TQ positions q along Q it stores TP records that are
// consecutive in the destination.  Each lane moves one unit (U bytes) of one
// record per step; consecutive lanes take consecutive records of one column
// (planar, AoSoA) or consecutive units of one record (AoS), so every wave
// access is one contiguous run.  The LDS image is [unit][q][p] with padded
// rows, which keeps the column writes nearly free of bank conflicts.
//
// No one resource is full: a tile's loads, its barrier and its stores follow
// each other, so half of a wave's cycles wait for memory, while vector issue
// takes half of the time and scalar issue a third (15.6 Mi records of 3 x f32,
// AoS to column-major SoA: 92 us, 4.1 TB/s; 1.01 times the needed bytes read,
// 1.05 written).  The lines at the runs' ends lie off the line grid and belong to
// two tiles; neighbouring tiles run on the same XCD, whose L2 merges all but 2 %
// of them (without that order 20-30 % slower).  Runs are 256 bytes on axes that
// hold them.  A lane keeps its place in the run and steps through the rows with
// one addition, eight accesses in flight; with 64-bit index arithmetic per unit
// and 128-byte runs the same copy took 237 us.
#include "kernels.hpp"

namespace lm {

// 64-bit quotient x / L by multiply-high with m = ceil(2^64 / L) (exact for
// x * L < 2^64), or a shift when L is a power of two (m = 0).
__device__ __forceinline__ uint64_t xp_div(uint64_t x, uint64_t m, const Div& d) {
  return m ? __umul64hi(x, m) : (x >> d.sh);
}

// Address of unit u of record i of a physical side.
template <int U>
__device__ __forceinline__ uint8_t* xp_addr(const Side& s, uint64_t lmag, uint64_t i, uint32_t u) {
  const uint32_t byte = u * U;
  const uint32_t c = byte >> s.log2cs, bo = byte & (s.cs - 1u);
  switch (s.layout) {
    case LY_AOS:
      return (uint8_t*)s.blob[0] + i * s.rec_bytes + byte;
    case LY_PLANAR:
      return (uint8_t*)(s.mb ? s.blob[c] : s.blob[0]) + (s.mb ? 0ull : (uint64_t)c * s.n * s.cs) + i * s.cs + bo;
    default: {  // AoSoA: block, column, lane
      const uint64_t blk = xp_div(i, lmag, s.div_L);
      const uint64_t lane = i - blk * s.lanes;
      return (uint8_t*)s.blob[0] + blk * s.lanes * s.rec_bytes + (uint64_t)c * s.lanes * s.cs + lane * s.cs + bo;
    }
  }
}

template <int U>
struct Unit;
template <> struct Unit<1> { typedef uint8_t T; };
template <> struct Unit<2> { typedef uint16_t T; };
template <> struct Unit<4> { typedef uint32_t T; };
template <> struct Unit<8> { typedef uint64_t T; };

// One side's walk over a tile: `rows` positions along one axis, each with a
// run of `len` records consecutive in this side's memory.  `base` is the record
// of (row 0, position 0), `stride` the records between rows.  Every unit is
// visited twice: get(k, valid, address), for XK units of a lane one after
// another, so that XK accesses are in flight, then put(k, valid, row, position,
// unit) for the same ones.
constexpr uint32_t XK = 8;

template <int U, int L, uint32_t T, typename Get, typename Put>
__device__ __forceinline__ void xp_walk(const Side& s, uint64_t lmag, uint32_t u0, uint32_t nu, const Div& dnu,
                                        uint64_t base, uint64_t stride, uint32_t rows, uint32_t len, uint32_t log2len,
                                        Get&& get, Put&& put) {
  if constexpr (L == LY_AOS) {
    // a row is one run of len * nu units
    const uint32_t run = len * nu, total = rows * run;
    const Div dr = make_div_dev(run);
    uint8_t* p0 = (uint8_t*)s.blob[0] + base * s.rec_bytes;
    const uint64_t rb = stride * s.rec_bytes;
    for (uint32_t i0 = threadIdx.x; i0 < total; i0 += XK * T) {
      uint32_t row[XK], x[XK];
#pragma unroll
      for (uint32_t k = 0; k < XK; ++k) {
        const uint32_t i = i0 + k * T, j = i < total ? i : total - 1u;
        row[k] = fdiv(j, dr);
        x[k] = j - row[k] * run;
        get(k, i < total, p0 + row[k] * rb + x[k] * U);
      }
#pragma unroll
      for (uint32_t k = 0; k < XK; ++k) {
        const uint32_t r = fdiv(x[k], dnu);
        put(k, i0 + k * T < total, row[k], r, x[k] - r * nu);
      }
    }
  } else {
    // per unit: lanes over the positions of a row; a lane keeps its position
    const uint32_t pos = threadIdx.x & ((1u << log2len) - 1u), row0 = threadIdx.x >> log2len;
    const uint32_t step = T >> log2len;  // rows between a lane's steps (tile edges are at most 128)
    const uint32_t at = pos < len ? pos : len - 1u;
    if (rows <= step) {  // short axes: one row a lane
      const bool ok = row0 < rows && pos < len;
      const uint64_t i = base + (row0 < rows ? row0 : 0u) * stride + at;
      for (uint32_t u = 0; u < nu; ++u) {
        get(0, ok, xp_addr<U>(s, lmag, i, u0 + u));
        put(0, ok, row0, pos, u);
      }
      return;
    }
    for (uint32_t u = 0; u < nu; ++u) {
      uint8_t* p = nullptr;
      if constexpr (L == LY_PLANAR) p = xp_addr<U>(s, 0, base + row0 * stride + at, u0 + u);
      const uint64_t pb = step * stride * s.cs;
      for (uint32_t r0 = row0; r0 < rows; r0 += XK * step) {
#pragma unroll
        for (uint32_t k = 0; k < XK; ++k) {
          const uint32_t r = r0 + k * step;
          const bool ok = r < rows && pos < len;
          if constexpr (L == LY_PLANAR) {
            get(k, ok, p);
            p += pb;
          } else {
            get(k, ok, xp_addr<U>(s, lmag, base + (r < rows ? r : row0) * stride + at, u0 + u));
          }
        }
#pragma unroll
        for (uint32_t k = 0; k < XK; ++k) put(k, r0 + k * step < rows && pos < len, r0 + k * step, pos, u);
      }
    }
  }
}

// T: threads of a workgroup, 64 (tiny tiles) or 256.
template <int U, int SL, int DL, uint32_t T>
__global__ __launch_bounds__(T) void k_xpose(const XposeArgs a) {
  typedef typename Unit<U>::T W;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
  W* img = (W*)lds_raw;
  const uint32_t lp = a.log2P, lq = a.log2Q, nu = a.nunits;
  const uint32_t row = (1u << lp) + xpose_pad(U);
  for (uint64_t b = blockIdx.x; b < a.ntiles; b += gridDim.x) {
    const uint64_t t = a.xcd ? xcd_tile((uint32_t)b, (uint32_t)a.ntiles) : b;
    // tile -> (units, middle index, tile along Q, tile along P): neighbours
    // along P share the lines at their runs' ends in the destination
    uint64_t p0, q0, sbase = 0, dbase = 0;
    uint32_t u0;
    auto locate = [&](auto x) {
      typedef decltype(x) I;
      I rest = x / (I)a.nPt;
      p0 = (uint64_t)(x - rest * (I)a.nPt) << lp;
      I m = rest / (I)a.nQt;
      q0 = (uint64_t)(rest - m * (I)a.nQt) << lq;
      for (uint32_t k = 0; k < a.nmid; ++k) {  // last middle axis varies fastest
        const uint32_t j = a.nmid - 1u - k;
        rest = m / (I)a.mext[j];
        const uint64_t y = m - rest * (I)a.mext[j];
        m = rest;
        sbase += y * a.msrc[j];
        dbase += y * a.mdst[j];
      }
      u0 = (uint32_t)m * nu;
    };
    if (a.xcd) locate((uint32_t)t);  // fewer than 2^24 tiles
    else locate(t);
    const uint32_t np = (uint32_t)(a.eP - p0 < (1u << lp) ? a.eP - p0 : (1u << lp));
    const uint32_t nq = (uint32_t)(a.eQ - q0 < (1u << lq) ? a.eQ - q0 : (1u << lq));
    sbase += p0 * a.sP + q0;  // source record of (p, q) = sbase + p sP + q
    dbase += q0 * a.dQ + p0;  // destination record of (p, q) = dbase + q dQ + p
    W v[XK];
    xp_walk<U, SL, T>(a.src, a.src_lmag, u0, nu, a.div_units, sbase, a.sP, np, nq, lq,
                   [&](uint32_t k, bool ok, const uint8_t* p) { v[k] = ok ? *(const W*)p : (W)0; },
                   [&](uint32_t k, bool ok, uint32_t p, uint32_t q, uint32_t u) {
                     if (ok) img[((u << lq) + q) * row + p] = v[k];
                   });
    __syncthreads();
    uint8_t* to[XK];
    xp_walk<U, DL, T>(a.dst, a.dst_lmag, u0, nu, a.div_units, dbase, a.dQ, nq, np, lp,
                   [&](uint32_t k, bool ok, uint8_t* p) { to[k] = p; },
                   [&](uint32_t k, bool ok, uint32_t q, uint32_t p, uint32_t u) {
                     if (ok) *(W*)to[k] = img[((u << lq) + q) * row + p];
                   });
    __syncthreads();
  }
}

template <int U, int SL, int DL>
static void launch_t(const XposeArgs& a, uint32_t grid, uint32_t lds, hipStream_t st) {
  if (a.log2T == 6u) hipLaunchKernelGGL((k_xpose<U, SL, DL, 64u>), dim3(grid), dim3(64), lds, st, a);
  else hipLaunchKernelGGL((k_xpose<U, SL, DL, kThreads>), dim3(grid), dim3(kThreads), lds, st, a);
}

template <int U, int SL>
static hipError_t launch_dl(const XposeArgs& a, uint32_t grid, uint32_t lds, hipStream_t st) {
  switch (a.dst.layout) {
    case LY_AOS: launch_t<U, SL, LY_AOS>(a, grid, lds, st); break;
    case LY_PLANAR: launch_t<U, SL, LY_PLANAR>(a, grid, lds, st); break;
    default: launch_t<U, SL, LY_AOSOA>(a, grid, lds, st); break;
  }
  return hipGetLastError();
}

template <int U>
static hipError_t launch_sl(const XposeArgs& a, uint32_t grid, uint32_t lds, hipStream_t st) {
  switch (a.src.layout) {
    case LY_AOS: return launch_dl<U, LY_AOS>(a, grid, lds, st);
    case LY_PLANAR: return launch_dl<U, LY_PLANAR>(a, grid, lds, st);
    default: return launch_dl<U, LY_AOSOA>(a, grid, lds, st);
  }
}

hipError_t launch_xpose(const XposeArgs& a, uint32_t unit, uint32_t grid, uint32_t lds, hipStream_t st) {
  switch (unit) {
    case 1: return launch_sl<1>(a, grid, lds, st);
    case 2: return launch_sl<2>(a, grid, lds, st);
    case 4: return launch_sl<4>(a, grid, lds, st);
    case 8: return launch_sl<8>(a, grid, lds, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lm
