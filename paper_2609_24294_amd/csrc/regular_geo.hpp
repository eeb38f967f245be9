// regular_geo.hpp -- where the blocks of a regular strided array lie, and the
// views of blocks and runs that the kernels gather and scatter through.
//
// The functions are __host__ __device__ (plain C++ without HIP): a host test
// compares them with 64-bit arithmetic over sizes that no buffer is made for.
#pragma once

#include <stdint.h>

#if defined(__HIP_DEVICE_COMPILE__)
#define ZFPX_GEO __host__ __device__ __attribute__((always_inline)) inline
#elif defined(__HIPCC__)
#define ZFPX_GEO __host__ __device__ inline
#else
#define ZFPX_GEO inline
#endif

namespace zfpx {

struct BlockView {
  int64_t rbase[4];
  int64_t lstride;
  int64_t sx;
  int32_t nlev, nrow;
  int32_t rlen[4];
  int32_t x0;  // first x of the block
};

// A tile whose 64 blocks all lie in one run: everything but the x offset is
// wave-uniform (scalar registers), so whole blocks load through a scalar row
// base plus a per-lane offset.
struct RunView {
  int64_t rbase[4];
  int64_t lstride;
  int32_t nlev, nrow, block0;
  int32_t minlen;  // shortest row of the group
  int32_t rlen[4];
};

// Regular strided array as a geometry.
struct RegularDev {
  int64_t nx, ny, nz;
  int64_t sx, sy, sz;
  int32_t nbx, nby;
};

// 4x4x4 blocks of an nx x ny x nz array (sizes >= 0), or -1 if their number
// passes 64 bits.
inline int64_t regular_blocks(int64_t nx, int64_t ny, int64_t nz) {
  if (nx == 0 || ny == 0 || nz == 0) return 0;
  const int64_t bx = (nx - 1) / 4 + 1, by = (ny - 1) / 4 + 1, bz = (nz - 1) / 4 + 1;
  int64_t n;
  if (__builtin_mul_overflow(bx, by, &n) || __builtin_mul_overflow(n, bz, &n)) return -1;
  return n;
}

struct RegularGeo {
  static constexpr bool kStreamLoads = false;
  RegularDev g;
  // Positions within a row are 32-bit, a row may be longer (nx up to four
  // times the number of blocks, 2^33): they count from the last multiple of
  // 2^30 points at or before the block, which joins the row's base, and the
  // length from there is cut at 2^31 - 1, far past the last block of a tile
  // that starts within those 2^30 points.  Rows of up to 2^30 points count
  // from their start.
  static constexpr uint32_t kSpanBlocks = 1u << 28;
  static ZFPX_GEO int64_t origin(uint32_t bx) { return 4 * (int64_t)(bx & ~(kSpanBlocks - 1)); }
  ZFPX_GEO int32_t length_from(int64_t x) const {
    const int64_t n = g.nx - x;
    return (int32_t)(n < INT32_MAX ? n : INT32_MAX);
  }
  // u / d for u < d + 64: at most one row further where d >= 64; below, an
  // exact multiply (u < 128).
  static ZFPX_GEO uint32_t wraps(uint32_t u, uint32_t d) {
    if (d >= 64) return u >= d ? 1u : 0u;
    return (u * ((65536u + d - 1) / d)) >> 16;
  }
  // Block b0 + lane: the divisions are those of the wave-uniform b0.
  ZFPX_GEO void locate_tile(int32_t b0, int lane, int, BlockView& v) const {
    const uint32_t t0 = (uint32_t)b0 / (uint32_t)g.nbx;
    uint32_t bx = (uint32_t)b0 - t0 * (uint32_t)g.nbx + (uint32_t)lane;
    uint32_t bz = t0 / (uint32_t)g.nby;
    uint32_t by = t0 - bz * (uint32_t)g.nby;
    const uint32_t rows = wraps(bx, (uint32_t)g.nbx);
    bx -= rows * (uint32_t)g.nbx;
    by += rows;
    const uint32_t planes = wraps(by, (uint32_t)g.nby);
    by -= planes * (uint32_t)g.nby;
    bz += planes;
    const int64_t x = origin(bx);
    const int64_t y0 = 4 * (int64_t)by, z0 = 4 * (int64_t)bz;
    const int64_t off = z0 * g.sz + x * g.sx;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      int64_t y = y0 + i < g.ny ? y0 + i : g.ny - 1;
      v.rbase[i] = off + y * g.sy;
      v.rlen[i] = length_from(x);
    }
    v.lstride = g.sz;
    v.sx = g.sx;
    v.nlev = (int32_t)(g.nz - z0 < 4 ? g.nz - z0 : 4);
    v.nrow = (int32_t)(g.ny - y0 < 4 ? g.ny - y0 : 4);
    v.x0 = (int32_t)(4 * (bx & (kSpanBlocks - 1)));
  }
  // A tile within one row of blocks (every tile but those at row ends) of an
  // array with unit x stride: the same view as a plan's run.  Rows of fewer
  // blocks than a tile have none.
  ZFPX_GEO bool one_run(int32_t b0, int nact, RunView& r) const {
    if (nact > g.nbx) return false;
    const uint32_t t = (uint32_t)b0 / (uint32_t)g.nbx;
    const uint32_t bx0 = (uint32_t)b0 - t * (uint32_t)g.nbx;
    if (bx0 + (uint32_t)nact > (uint32_t)g.nbx) return false;
    const uint32_t bz = t / (uint32_t)g.nby;
    const int64_t x = origin(bx0);
    const int64_t y0 = 4 * (int64_t)(t - bz * (uint32_t)g.nby), z0 = 4 * (int64_t)bz;
    const int32_t len = length_from(x);
#pragma unroll
    for (int i = 0; i < 4; i++) {
      r.rbase[i] = z0 * g.sz + x + (y0 + i < g.ny ? y0 + i : g.ny - 1) * g.sy;
      r.rlen[i] = len;
    }
    r.lstride = g.sz;
    r.nlev = (int32_t)(g.nz - z0 < 4 ? g.nz - z0 : 4);
    r.nrow = (int32_t)(g.ny - y0 < 4 ? g.ny - y0 : 4);
    r.block0 = b0 - (int32_t)(bx0 & (kSpanBlocks - 1));
    r.minlen = len;
    return true;
  }
};

}  // namespace zfpx
