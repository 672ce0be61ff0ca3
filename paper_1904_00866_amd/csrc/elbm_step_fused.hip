// elbm_step_fused.hip -- several time steps of a D2Q9 box in one launch.
//
// A workgroup owns a tile of sites and advances it `nsub` steps: it pulls the
// tile and a frame of nsub - 1 sites around it from the source buffer, keeps
// the post-collision populations of each step in LDS (in their storage format,
// rounded as a buffer would hold them), pulls the next step from there, and
// writes the tile after the last.  The frame's sites are computed by the
// neighbouring workgroups too; each step the frame shrinks by one site.  The
// arithmetic of a site is the step kernel's own code, so the result has the
// bits of nsub single steps, in every byte of the buffer.
//
// What it buys: a small box, whose step is a launch and the latency of one
// site's arithmetic, pays one launch for nsub steps (64^2 in FP32, six steps:
// 3.3 -> 1.4 us a step), and a large one moves its state once per nsub steps:
// LBGK becomes two times faster (FP64 4096^2, three steps: 416 -> 172 us a
// step), FP64 closed form 405 -> 325.  The FP32 closed form is bound by its
// FP64 arithmetic then: 14.2M vector instructions a step at 1500^2, of single
// steps 13.7M (the frame's sites cost what the pull from LDS saves), about 25
// us of issue in 34 us a step (single steps 38).  A box whose tiles are mostly
// frame computes far more (fusion_of() has the limits).
// It records no diagnostics (those belong to the last step of a call, which is
// launched singly when it records).
#include "elbm_step_impl.hpp"

namespace elbm {
namespace {

// New populations of a site into the workgroup's LDS region.
template <class T, int SITES>
struct ToRegion {
  T (*lds)[SITES];
  uint32_t at;
  __device__ __forceinline__ void begin() const {}
  __device__ __forceinline__ void operator()(int i, T v) const { lds[i][at] = v; }
};

// g modulo n for -2^20 < g < 2^21, n < 2^20 (inv_n = 1/n).
__device__ __forceinline__ uint32_t wrap_mod(int g, uint32_t n, double inv_n) {
  const int q = (int)floor(((double)g + 0.5) * inv_n);
  return (uint32_t)(g - q * (int)n);
}

// Byte offset of element (0, s) of the blocked layout with nine directions,
// ((s / 64) 9) 64 + s % 64 elements: 32 bits, so a buffer holds less than 4 GiB
// (the host sees to that).
template <class T>
__device__ __forceinline__ uint64_t offset9(uint32_t s) {
  return (uint32_t)((((s & ~63u) << 3) + s) * (uint32_t)sizeof(T));
}

// The region of RX x RY sites is spread over WAVES wavefronts, UNITS sites per
// thread: unit u of thread t is region site u 64 WAVES + t, x fastest.
template <class S, int MODE, class R, int RX, int RY, int WAVES>
__global__ void __launch_bounds__(64 * WAVES) k_fused(const BatchArgs args, int nsub) {
  using T = typename S::T;
  using L = Lattice<2>;
  constexpr int Q = L::Q, SITES = RX * RY, THREADS = 64 * WAVES, UNITS = SITES / THREADS;
  static_assert(UNITS * THREADS == SITES && RX % 16 == 0, "region shape");
  __shared__ T lds[Q][SITES];
  const int b = blockIdx.x;
  int si = 0;
  for (int k = 1; k < args.n; ++k)
    if (b >= args.d[k].block_begin) si = k;
  const SimDesc& d = args.d[si];
  const T* __restrict__ src = static_cast<const T*>(d.src);
  T* __restrict__ dst = static_cast<T*>(d.dst);
  const uint32_t nx = (uint32_t)d.nx, ny = (uint32_t)d.ny;
  const int frame = nsub - 1, ix = RX - 2 * frame, iy = RY - 2 * frame;
  const uint32_t tiles_x = (nx + ix - 1) / ix, tiles_y = (ny + iy - 1) / iy;
  // one contiguous run of tiles per XCD, as in the step kernel
  const uint32_t lb = (uint32_t)(b - d.block_begin);
  const uint32_t tile = (lb & 7u) * ((uint32_t)d.nblocks >> 3) + (lb >> 3);
  if (tile >= tiles_x * tiles_y) return;  // padding workgroup
  const uint32_t ty = tile / tiles_x;
  const int x0 = (int)((tile - ty * tiles_x) * ix) - frame, y0 = (int)(ty * iy) - frame;

  Slot<T> raw[UNITS][Q];
#if ELBM_LOAD_PRIO
  __builtin_amdgcn_s_setprio(ELBM_LOAD_PRIO);
#endif
  // a tile whose frame and its neighbours lie inside the box needs no wrapping
  const bool inner = x0 > 0 && y0 > 0 && x0 + RX < (int)nx && y0 + RY < (int)ny;
#pragma unroll
  for (int u = 0; u < UNITS; ++u) {
    const int at = u * THREADS + (int)threadIdx.x;
    uint32_t xs[3], ys[3];
    if (inner) {
      const uint32_t x = (uint32_t)(x0 + at % RX), y = (uint32_t)(y0 + at / RX) * nx;
      xs[0] = x;
      xs[1] = x - 1;
      xs[2] = x + 1;
      ys[0] = y;
      ys[1] = y - nx;
      ys[2] = y + nx;
    } else {
      const uint32_t x = wrap_mod(x0 + at % RX, nx, d.inv_nx);
      const uint32_t y = wrap_mod(y0 + at / RX, ny, d.inv_ny);
      xs[0] = x;
      xs[1] = x == 0 ? nx - 1 : x - 1;
      xs[2] = x == nx - 1 ? 0 : x + 1;
      ys[0] = y * nx;
      ys[1] = (y == 0 ? ny - 1 : y - 1) * nx;
      ys[2] = (y == ny - 1 ? 0 : y + 1) * nx;
    }
    const gaddr base = buffer_base(src);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      using U = typename std::conditional<sizeof(T) == 2, uint16_t, T>::type;
      raw[u][i] = Slot<T>(*(const gptr<U>)(base + offset9<T>(ys[i / 3] + xs[i % 3]) +
                                           (uint64_t)(i * kLane * sizeof(T))));
    }
  }
#if ELBM_LOAD_PRIO
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_setprio(0);
#endif
  Acc acc;
  acc.init();
#pragma unroll 1
  for (int j = 1;; ++j) {
    bool deferred[UNITS];
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
      ToRegion<T, SITES> out{lds, (uint32_t)(u * THREADS) + threadIdx.x};
      constexpr int kPhase = MODE == kClosed ? kPhaseCommon : kPhaseAll;
      deferred[u] = site_update<2, S, MODE, R, false, kPhase>(d, src, out, 0u, true, raw[u], acc, 0).deferred;
    }
    if constexpr (MODE == kClosed) {
#pragma unroll
      for (int u = 0; u < UNITS; ++u) {
        if (__any(deferred[u])) {
          ToRegion<T, SITES> out{lds, (uint32_t)(u * THREADS) + threadIdx.x};
          if (deferred[u])
            (void)site_update<2, S, MODE, R, false, kPhaseRareReg>(d, src, out, 0u, true, raw[u], acc, 0);
        }
      }
    }
    if (j == nsub) break;
    __syncthreads();
    // the next step's pull.  Sites whose neighbours are not known any more
    // take the values of the nearest that is (ordinary numbers for the
    // wavefront's votes); nothing reads what they write.
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
      const int at = u * THREADS + (int)threadIdx.x;
      const int lx = min(max(at % RX, j), RX - 1 - j), ly = min(max(at / RX, j), RY - 1 - j);
      const int c = ly * RX + lx;
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        const T v = lds[i][c - L::c(i, 1) * RX - L::c(i, 0)];
        if constexpr (sizeof(T) == 2) raw[u][i] = (uint32_t)__builtin_bit_cast(uint16_t, v);
        else raw[u][i] = v;
      }
    }
    __syncthreads();
  }
  const gaddr base = buffer_base(dst);
  // each thread stores what it has just written
#pragma unroll
  for (int u = 0; u < UNITS; ++u) {
    const int at = u * THREADS + (int)threadIdx.x;
    const int lx = at % RX, ly = at / RX, x = x0 + lx, y = y0 + ly;
    // The places that pad the last tile of kBlock sites hold site 0's new
    // populations after a single step (its lanes past the box repeat that site).
    // A checkpoint copies them too, so the wavefront of site 0 writes them (100^2
    // FP64, five steps a launch: 1.64 us a step without, 1.66 with; 1.73 where
    // every wavefront of the workgroup wrote them after the other stores).
    if (u == 0 && __builtin_expect(x0 == -frame && y0 == -frame && nx * ny % kBlock != 0, 0)) {
      const int at0 = frame * RX + frame;
      static_assert(THREADS >= 256, "site 0 lies in the first unit");
      if (__any(lx == frame && ly == frame)) {
        const uint32_t lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        const uint32_t N = nx * ny, end = (N + kBlock - 1) / kBlock * kBlock;
        for (uint32_t s = N + lane; s < end; s += 64) {
#pragma unroll
          for (int i = 0; i < Q; ++i)
            *(gptr<T>)(base + offset9<T>(s) + (uint64_t)(i * kLane * sizeof(T))) = lds[i][at0];
        }
      }
    }
    if (lx >= frame && lx < RX - frame && ly >= frame && ly < RY - frame && x < (int)nx &&
        y < (int)ny) {
      const uint32_t s = (uint32_t)y * nx + (uint32_t)x;
#pragma unroll
      for (int i = 0; i < Q; ++i)
        *(gptr<T>)(base + offset9<T>(s) + (uint64_t)(i * kLane * sizeof(T))) = lds[i][at];
    }
  }
}

// Geometries beside the smallest are built where fusion_of() chooses them.
template <class S, int MODE, class R>
hipError_t launch_fused(const BatchArgs& a, int grid, int nsub, int geom, hipStream_t st) {
  constexpr int es = sizeof(typename S::T);
  constexpr bool fp64 = std::is_same<R, double>::value;
  if (geom == kFused16x16) {
    k_fused<S, MODE, R, 16, 16, 4><<<grid, 256, 0, st>>>(a, nsub);
    return hipGetLastError();
  }
  if constexpr (kIsMixed<R>) {
    if (geom == kFused64x16) {
      k_fused<S, MODE, R, 64, 16, 4><<<grid, 256, 0, st>>>(a, nsub);
      return hipGetLastError();
    }
  } else if constexpr (MODE == kBGK || (es == 4 && !(S::dev && fp64))) {
    if (geom == kFused32x32) {
      k_fused<S, MODE, R, 32, 32, 8><<<grid, 512, 0, st>>>(a, nsub);
      return hipGetLastError();
    }
  }
  return hipErrorInvalidValue;
}

template <int MODE, class R>
FusedLauncher fused_for(int storage) {
  switch (storage) {
    case kStoreF64:
      if constexpr (std::is_same<R, double>::value) return &launch_fused<StoreF64, MODE, R>;
      return nullptr;
    case kStoreF32: return &launch_fused<StoreF32, MODE, R>;
    case kStoreF32Dev: return &launch_fused<StoreF32Dev, MODE, R>;
    case kStoreF16Dev: return &launch_fused<StoreF16Dev, MODE, R>;
    default: return nullptr;
  }
}

}  // namespace

FusedLauncher fused_launcher(int lattice, int storage, int mode, int fp64, int entropy) {
  if (lattice != 2 || entropy != 0) return nullptr;
  if (mode == kBGK) return fused_for<kBGK, double>(storage);
  if (mode != kClosed) return nullptr;  // the root solvers' passes re-read the source
  if (fp64 == kArithF64) return fused_for<kClosed, double>(storage);
  if (fp64 == kArithMixed) return fused_for<kClosed, Mixed>(storage);
  if (fp64 == kArithF32) return fused_for<kClosed, float>(storage);
  return nullptr;
}

}  // namespace elbm
