// elbm_pull.hpp -- addressing of the blocked population layout and the pull
// g_i = P_i(x - c_i) of a site's populations, for the step kernels and the
// auxiliary kernels.
#pragma once

#include <type_traits>

#include "elbm_internal.hpp"
#include "elbm_q19.hpp"
#include "elbm_site.hpp"

namespace elbm {

template <class R>
__device__ __forceinline__ R sel3(const R (&a)[3], int d) {
  return d == 0 ? a[0] : (d == 1 ? a[1] : a[2]);
}

// Addressing.  Bases are uniform (scalar registers) and a lane's byte
// offset a 32-bit vector register, so loads and stores take the
// scalar-base + vector-offset form.  The buffer base is passed through
// in_sgpr() once per tile and the per-direction bases are formed with
// scalar adds; the explicit global address space keeps the accesses global
// rather than generic.
using gaddr = uint64_t;
template <class T>
using gptr = __attribute__((address_space(1))) T*;

template <class T>
__device__ __forceinline__ gaddr buffer_base(const T* buf) {
  return in_sgpr((gaddr)(uintptr_t)buf);
}
// Load of one population as a raw buffer load from a range of `bytes`
// bytes at `base` (scalar descriptor, vector byte offset); an offset past
// the range reads 0.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(gaddr base, uint32_t bytes) {
  // word 3: 32-bit data format, the raw-buffer setting of this architecture
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(base), (short)0, (int)bytes,
                                           0x00020000);
}
// soff: a uniform byte offset added to the base (scalar operand)
template <class T>
__device__ __forceinline__ T ld_buf(__amdgpu_buffer_rsrc_t r, uint32_t boff, uint32_t soff) {
  if constexpr (sizeof(T) == 8) {
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, boff, soff, 0));
  } else if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, boff, soff, 0));
  } else {
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b16(r, boff, soff, 0));
  }
}

// Non-temporal store of one population into a range of `bytes` bytes at
// `base`, as a raw buffer store: the descriptor is formed in scalar
// registers and the lane's byte offset is the only vector operand, so a
// store costs no vector address arithmetic.  An offset at or past `bytes`
// is discarded by the hardware range check.
template <class T>
__device__ __forceinline__ void st_nt(gaddr base, uint32_t bytes, uint32_t boff, T v) {
  const __amdgpu_buffer_rsrc_t r = rsrc(base, bytes);
  constexpr int kNT = 2;  // cache policy: non-temporal
  if constexpr (sizeof(T) == 8) {
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, boff, 0, kNT);
  } else if constexpr (sizeof(T) == 4) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, boff, 0, kNT);
  } else {
    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, v), r, boff, 0, kNT);
  }
}

// Byte address of the block that holds the wavefront's 64 sites in `buf`
// (the sites of a wavefront are 64 consecutive, 64-aligned indices, so the
// block is uniform).
template <int Q, class T>
__device__ __forceinline__ gaddr block_base(const T* buf, uint32_t s) {
  const uint32_t blk = __builtin_amdgcn_readfirstlane(s >> 6);
  return buffer_base(buf) + (uint64_t)blk * ((uint64_t)Q * kLane * sizeof(T));
}

// Quotient of s < 2^31 by n < 2^20 through one FP64 multiply: (s + 1/2)/n is
// at least 1/(2n) away from an integer, far more than the rounding error.
__device__ __forceinline__ uint32_t qdiv(uint32_t s, double inv_n) {
  return (uint32_t)(((double)s + 0.5) * inv_n);
}

// Source coordinates of one site for digit 0 (c = 0), 1 (c = +1: pull from
// -1) and 2 (c = -1), as element offsets: x, y * nx, z * nx * ny.
struct Where {
  uint32_t xs[3], ys[3], zs[3];
};

template <int D, class Box>
__device__ __forceinline__ Where locate(const Box& d, uint32_t s) {
  const uint32_t nx = (uint32_t)d.nx, ny = (uint32_t)d.ny, nz = (uint32_t)d.nz;
  uint32_t x, y, z;
  if constexpr (D == 1) {
    x = s;
    y = 0;
    z = 0;
  } else {
    const uint32_t row = qdiv(s, d.inv_nx);
    x = s - row * nx;
    z = (D == 3) ? qdiv(row, d.inv_ny) : 0u;
    y = row - z * ny;
  }
  Where w;
  w.xs[0] = x;
  w.xs[1] = x == 0 ? nx - 1 : x - 1;
  w.xs[2] = x == nx - 1 ? 0 : x + 1;
  w.ys[0] = y * nx;
  w.ys[1] = (y == 0 ? ny - 1 : y - 1) * nx;
  w.ys[2] = (y == ny - 1 ? 0 : y + 1) * nx;
  const uint32_t nxy = nx * ny;
  w.zs[0] = z * nxy;
  w.zs[1] = (z == 0 ? nz - 1 : z - 1) * nxy;
  w.zs[2] = (z == nz - 1 ? 0 : z + 1) * nxy;
  return w;
}

// Direction index of the digits (dx, dy, dz) on lattice L, or -1 if L has
// no such direction.
template <class L>
struct Dirs;
template <int D>
struct Dirs<Lattice<D>> {
  static constexpr int index(int dx, int dy, int dz) {
    return ((D < 2 && dy != 0) || (D < 3 && dz != 0)) ? -1 : dx + 3 * dy + 9 * dz;
  }
};
template <>
struct Dirs<LatticeQ19> {
  static constexpr int index(int dx, int dy, int dz) {
    return (dx != 0 && dy != 0 && dz != 0)
               ? -1
               : (dx + 3 * dy + 9 * dz) - 2 * ((dx + 3 * dy + 9 * dz) >= 13) -
                     2 * ((dx + 3 * dy + 9 * dz) >= 18) - 2 * ((dx + 3 * dy + 9 * dz) >= 22);
  }
};

// Pull of the Q populations when the wavefront's 64 sites lie in one x-row
// (one descriptor per source row (c_y, c_z), the three x positions as
// per-lane offsets).  Box: a SimDesc or a BoxDesc.
template <class L, class T, class Box>
__device__ __forceinline__ void load_row_l(const Box& d, const T* src, uint32_t s,
                                           T (&raw)[L::Q]) {
  constexpr int D = L::Dim, Q = L::Q;
  const uint32_t nx = (uint32_t)d.nx, ny = (uint32_t)d.ny, nz = (uint32_t)d.nz;
  const uint32_t row = __builtin_amdgcn_readfirstlane(D == 1 ? 0u : qdiv(s, d.inv_nx));
  const uint32_t x = s - row * nx;
  uint32_t ys[3] = {0u, 0u, 0u}, zs[3] = {0u, 0u, 0u};
  if constexpr (D > 1) {
    const uint32_t z = D == 3 ? __builtin_amdgcn_readfirstlane(qdiv(row, d.inv_ny)) : 0u;
    const uint32_t y = row - z * ny;
    ys[0] = y * nx;
    ys[1] = (y == 0 ? ny - 1 : y - 1) * nx;
    ys[2] = (y == ny - 1 ? 0 : y + 1) * nx;
    const uint32_t nxy = nx * ny;
    zs[0] = z * nxy;
    zs[1] = (z == 0 ? nz - 1 : z - 1) * nxy;
    zs[2] = (z == nz - 1 ? 0 : z + 1) * nxy;
  }
  constexpr uint32_t es = sizeof(T);
  uint32_t xo[3];
  const uint32_t xm = x == 0 ? nx - 1 : x - 1, xp = x == nx - 1 ? 0 : x + 1;
  xo[0] = (uint32_t)pidx<Q>(x, 0) * es;
  xo[1] = (uint32_t)pidx<Q>(xm, 0) * es;
  xo[2] = (uint32_t)pidx<Q>(xp, 0) * es;
  const gaddr base = buffer_base(src);
  const uint32_t rowbytes = nx * (uint32_t)Q * es;
#pragma unroll
  for (int dz = 0; dz < (D > 2 ? 3 : 1); ++dz)
#pragma unroll
    for (int dy = 0; dy < (D > 1 ? 3 : 1); ++dy) {
      const __amdgpu_buffer_rsrc_t r = rsrc(base + (uint64_t)(zs[dz] + ys[dy]) * Q * es, rowbytes);
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        const int i = Dirs<L>::index(dx, dy, dz);
        if (i < 0) continue;
        raw[i] = ld_buf<T>(r, xo[dx], (uint32_t)i * kLane * es);
      }
    }
}

// Pull of the Q populations of site s (s < N), any box.
template <class L, class T, class Box>
__device__ __forceinline__ void load_l(const Box& d, const T* src, uint32_t s, T (&raw)[L::Q]) {
  const Where w = locate<L::Dim>(d, s);
  const gaddr base = buffer_base(src);
#pragma unroll
  for (int i = 0; i < L::Q; ++i) {
    const uint32_t sp = w.zs[L::dg(i, 2)] + w.ys[L::dg(i, 1)] + w.xs[L::dg(i, 0)];
    raw[i] = *(const gptr<T>)(base + pidx<L::Q>(sp, i) * sizeof(T));
  }
}

}  // namespace elbm
