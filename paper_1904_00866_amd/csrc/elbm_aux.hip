// elbm_aux.hip -- auxiliary kernels of the ELBM library: validation and
// placement of initial states, gathers of f(x,t), moments, and the
// fixed-order reduction of the per-workgroup diagnostics records.
//
// Pull convention: the buffer read by the next step holds P_i(y) with
// P_i(x - c_i) = f_i(x, t), i.e. the post-collision values of the previous
// step before streaming (Eq. (5b) is carried out by the reader).
#include "elbm_internal.hpp"
#include "elbm_burg.hpp"
#include "elbm_pull.hpp"
#include "elbm_q19.hpp"
#include "elbm_site.hpp"

namespace elbm {

namespace {

// What bounds the readings below is their traffic: Q populations in, D + 1 or
// Q doubles out, each once.  One thread per site in the step kernel's XCD
// order (a run of 64 shifted by one site reaches into the next block's line,
// which is then in the same L2), with its row-descriptor loads where a
// wavefront's sites lie in one x-row and 32-bit site coordinates.  With
// 64-bit divisions per direction and blocks dealt round the XCDs the moments
// of a 512^3 FP32 box took 4.2 ms, now 3.5 ms (5.3 TB/s); 256^3 in FP16,
// 0.56 -> 0.27 ms.

// Site of this thread: workgroup b of a grid that is a multiple of 8 takes
// block (b mod 8) grid / 8 + b / 8, so that each XCD has one contiguous eighth.
__device__ __forceinline__ uint32_t site_of_thread() {
  const uint32_t b = blockIdx.x, chunk = gridDim.x >> 3;
  return ((b & 7u) * chunk + (b >> 3)) * blockDim.x + threadIdx.x;
}

// The pre-collision populations of site s, as stored.
template <class L, class T>
__device__ __forceinline__ void pull(const BoxDesc& b, const T* buf, uint32_t s, T (&raw)[L::Q]) {
  if (b.nx % kLane == 0) load_row_l<L>(b, buf, s, raw);
  else load_l<L>(b, buf, s, raw);
}

// Site index of x - c_i (sign = +1) or x + c_i (sign = -1).
template <class L, int SIGN>
__device__ __forceinline__ uint32_t neighbour(const Where& w, int i) {
  const auto dg = [&](int a) {
    const int k = L::dg(i, a);
    return SIGN > 0 || k == 0 ? k : 3 - k;
  };
  return w.zs[dg(2)] + w.ys[dg(1)] + w.xs[dg(0)];
}

// rho0 > 0 and u0 inside the hull of the velocities: |u_a| < 1, and on
// D3Q19 (no corner velocities, hull2 set) also |u_x| + |u_y| + |u_z| < 2.
__global__ void k_validate(int64_t N, int D, int hull2, const double* __restrict__ rho0,
                           const double* __restrict__ u0, unsigned long long* bad) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int ok = 1;
  if (s < N) {
    ok = rho0[s] > 0.0 && isfinite(rho0[s]);
    double l1 = 0.0;
    for (int a = 0; a < D; ++a) {
      ok = ok && fabs(u0[a * N + s]) < 1.0;
      l1 += fabs(u0[a * N + s]);
    }
    if (hull2) ok = ok && l1 < 2.0;
  }
  const unsigned long long nb = __ballot(!ok);
  if ((threadIdx.x & 63) == 0 && nb) atomicAdd(bad, (unsigned long long)__popcll(nb));
}

// f^eq(rho0, u0) in pull convention: f_i of site x goes to x - c_i.
template <class L, class S>
__global__ void k_init(const BoxDesc b, typename S::T* __restrict__ buf,
                       const double* __restrict__ rho0, const double* __restrict__ u0) {
  constexpr int D = L::Dim;
  constexpr int Q = L::Q;
  const uint32_t s = site_of_thread();
  if (s >= b.N) return;
  double fv[Q];
  double u[3] = {0.0, 0.0, 0.0};
  for (int a = 0; a < D; ++a) u[a] = u0[a * b.N + s];
  if (b.entropy == 1) {
    // Burg's entropy: f^eq_i = W_i / d_i (elbm_burg.hpp)
    double mu[4];
    burg_multipliers<L>(rho0[s], 1.0 / rho0[s], u, mu);
#pragma unroll
    for (int i = 0; i < Q; ++i) fv[i] = L::W(i) / burg_den<L>(mu, i);
  } else if constexpr (Q == 19) {
    // f^eq_i = rho W_i prod_a X_a^c_ia / Z  (EquilibriumQ19)
    EquilibriumQ19<double> eq;
    eq.build(u);
    const double cF = rho0[s] / eq.Z9;
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      double p = cF * (9.0 * L::W(i));
#pragma unroll
      for (int a = 0; a < 3; ++a)
        p *= L::dg(i, a) == 0 ? 1.0 : (L::dg(i, a) == 1 ? eq.X[a] : eq.Y[a]);
      fv[i] = p;
    }
  } else {
    Equilibrium<double, D> eq;
    eq.build(u);
#pragma unroll
    for (int i = 0; i < Q; ++i)
      fv[i] = rho0[s] * (eq.e(0, L::dg(i, 0)) * eq.e(1, L::dg(i, 1))) * eq.e(2, L::dg(i, 2));
  }
  const Where w = locate<D>(b, s);
#pragma unroll
  for (int i = 0; i < Q; ++i)
    buf[pidx<Q>(neighbour<L, 1>(w, i), i)] =
        Codec<S, double>::enc(fv[i], L::invW(i), b.rho_ref);
}

// Given f(x, t) in pull convention: each stored element (i, y) takes
// f_i(y + c_i), so that the writes are whole blocks and the reads carry the
// shifts.
template <class L, class S>
__global__ void k_put(const BoxDesc b, typename S::T* __restrict__ buf,
                      const double* __restrict__ f) {
  constexpr int Q = L::Q;
  const uint32_t s = site_of_thread();
  if (s >= b.N) return;
  const Where w = locate<L::Dim>(b, s);
  double fv[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) fv[i] = f[i * b.N + neighbour<L, -1>(w, i)];
#pragma unroll
  for (int i = 0; i < Q; ++i)
    buf[pidx<Q>(s, i)] = Codec<S, double>::enc(fv[i], L::invW(i), b.rho_ref);
}

// f(x, t) of every site.
template <class L, class S>
__global__ void k_populations(const BoxDesc b, const typename S::T* __restrict__ buf,
                              double* __restrict__ out) {
  constexpr int Q = L::Q;
  const uint32_t s = site_of_thread();
  if (s >= b.N) return;
  typename S::T raw[Q];
  pull<L>(b, buf, s, raw);
#pragma unroll
  for (int i = 0; i < Q; ++i)
    __builtin_nontemporal_store(Codec<S, double>::dec(raw[i], L::W(i), b.rho_ref),
                                out + i * b.N + s);
}

template <class L, class S>
__global__ void k_gather(const BoxDesc b, const typename S::T* __restrict__ buf,
                         const int64_t* __restrict__ sites, int64_t n, int which,
                         double* __restrict__ out) {
  constexpr int Q = L::Q;
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int64_t s = sites[k];
  if (s < 0 || s >= b.N) {
    for (int i = 0; i < Q; ++i) out[i * n + k] = NAN;
    return;
  }
  const Where w = locate<L::Dim>(b, (uint32_t)s);
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const uint32_t src = which == 0 ? neighbour<L, 1>(w, i) : (uint32_t)s;
    out[i * n + k] = Codec<S, double>::dec(buf[pidx<Q>(src, i)], L::W(i), b.rho_ref);
  }
}

template <class L, class S>
__global__ void k_moments(const BoxDesc b, const typename S::T* __restrict__ buf,
                          double* __restrict__ rho, double* __restrict__ u) {
  constexpr int D = L::Dim;
  constexpr int Q = L::Q;
  const uint32_t s = site_of_thread();
  if (s >= b.N) return;
  typename S::T raw[Q];
  pull<L>(b, buf, s, raw);
  double r = 0.0, j[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const double g = Codec<S, double>::dec(raw[i], L::W(i), b.rho_ref);
    r += g;
#pragma unroll
    for (int a = 0; a < D; ++a) {
      if (L::c(i, a) > 0) j[a] += g;
      else if (L::c(i, a) < 0) j[a] -= g;
    }
  }
  rho[s] = r;
  // a NaN or an infinity among the populations leaves no velocity component
  // defined, also those that its direction does not enter
#pragma unroll
  for (int a = 0; a < D; ++a) u[a * b.N + s] = isfinite(r) ? j[a] / r : NAN;
}

// Fixed-order reduction of the per-workgroup records by one workgroup per
// chunk of them: thread t folds the chunk's records t, t + kBlock, ... in
// order, then a fixed tree combines the threads.  A box of many workgroups
// is folded in two launches (one workgroup over the 524,288 records of 512^3
// takes 1.1 ms; the two launches 17 us): the first leaves the kPartWords
// 64-bit words of each chunk's result in the pad words of the chunk's own
// first records (which every step writes as zero and nothing else reads), the
// second folds those.
struct Partial {
  unsigned long long c[kNumCounts];
  double v[5];
  float mn, mx;
};
constexpr int kPartWords = sizeof(Partial) / 8;
static_assert(sizeof(Partial) == 8 * kPartWords && sizeof(CountRec::pad) == 8,
              "a partial result is spread over the records' 8-byte pads");
constexpr int kOneLaunch = 4096;  // records up to which one workgroup folds them alone
constexpr int kMaxParts = kBlock;

__device__ __forceinline__ void fold(Partial& p, const Partial& q) {
#pragma unroll
  for (int m = 0; m < kNumCounts; ++m) p.c[m] += q.c[m];
#pragma unroll
  for (int m = 0; m < 5; ++m) p.v[m] += q.v[m];
  p.mn = fminf(p.mn, q.mn);
  p.mx = fmaxf(p.mx, q.mx);
}

// PARTS: fold the partial results of ceil(n / chunk) chunks; else the
// records of chunk blockIdx.x.  With `out`, the result goes there, otherwise
// into the pads of the chunk.
template <bool PARTS>
__global__ void k_reduce(CountRec* __restrict__ cr, const SumRec* __restrict__ sr, int n,
                         int chunk, Reduced* __restrict__ out) {
  __shared__ Partial sp[kBlock / 64];
  const int t = threadIdx.x;
  Partial p{};
  p.mn = INFINITY;
  p.mx = -INFINITY;
  if constexpr (PARTS) {
    if ((int64_t)t * chunk < n) {
      unsigned long long w[kPartWords];
#pragma unroll
      for (int m = 0; m < kPartWords; ++m)
        w[m] = *reinterpret_cast<const unsigned long long*>(cr[t * chunk + m].pad);
      __builtin_memcpy(&p, w, sizeof p);
    }
  } else {
    const int k0 = blockIdx.x * chunk, k1 = min(n, k0 + chunk);
    for (int k = k0 + t; k < k1; k += kBlock) {
      const CountRec& q = cr[k];
      Partial w{};
#pragma unroll
      for (int m = 0; m < kNumCounts; ++m) w.c[m] = q.cnt[m];
      w.mn = q.amin;
      w.mx = q.amax;
      if (sr) {
        const SumRec& z = sr[k];
        w.v[0] = z.rho; w.v[1] = z.j[0]; w.v[2] = z.j[1]; w.v[3] = z.j[2]; w.v[4] = z.H;
      }
      fold(p, w);
    }
  }
  // the wavefront's 64 partial results by a shuffle tree, then the wavefronts
  // in order
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    Partial q;
#pragma unroll
    for (int m = 0; m < kNumCounts; ++m) q.c[m] = __shfl_down(p.c[m], o);
#pragma unroll
    for (int m = 0; m < 5; ++m) q.v[m] = __shfl_down(p.v[m], o);
    q.mn = __shfl_down(p.mn, o);
    q.mx = __shfl_down(p.mx, o);
    fold(p, q);
  }
  if ((t & 63) == 0) sp[t >> 6] = p;
  __syncthreads();
  if (t != 0) return;
  for (int w = 1; w < kBlock / 64; ++w) fold(p, sp[w]);
  if (out) {
    for (int m = 0; m < kNumCounts; ++m) out->cnt[m] = (int64_t)p.c[m];
    out->amin = p.mn;
    out->amax = p.mx;
    out->rho = p.v[0];
    out->j[0] = p.v[1]; out->j[1] = p.v[2]; out->j[2] = p.v[3];
    out->H = p.v[4];
  } else {
    unsigned long long w[kPartWords];
    __builtin_memcpy(w, &p, sizeof p);
    CountRec* c0 = cr + (int64_t)blockIdx.x * chunk;
#pragma unroll
    for (int m = 0; m < kPartWords; ++m)
      *reinterpret_cast<unsigned long long*>(c0[m].pad) = w[m];
  }
}

__global__ void k_copy_f64(const double* __restrict__ a, double* __restrict__ b, int64_t n) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s < n) b[s] = a[s];
}

inline unsigned grid_for(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }
// a multiple of 8 workgroups (site_of_thread)
inline unsigned grid_for_box(const BoxDesc& b) { return (grid_for(b.N, 256) + 7) / 8 * 8; }

// lattice: 1, 2, 3 (D1Q3, D2Q9, D3Q27) or 19 (D3Q19)
template <template <class, class> class Fn, class... A>
hipError_t dispatch(int lattice, int storage, A&&... a) {
#define ELBM_ST(LL)                                                            \
  switch (storage) {                                                           \
    case kStoreF64: return Fn<LL, StoreF64>::run(a...);                        \
    case kStoreF32: return Fn<LL, StoreF32>::run(a...);                        \
    case kStoreF32Dev: return Fn<LL, StoreF32Dev>::run(a...);                  \
    case kStoreF16Dev: return Fn<LL, StoreF16Dev>::run(a...);                  \
    default: return hipErrorInvalidValue;                                      \
  }
  switch (lattice) {
    case 1: ELBM_ST(Lattice<1>)
    case 2: ELBM_ST(Lattice<2>)
    case 3: ELBM_ST(Lattice<3>)
    case 19: ELBM_ST(LatticeQ19)
    default: return hipErrorInvalidValue;
  }
#undef ELBM_ST
}

template <class L, class S>
struct ScatterFn {
  static hipError_t run(const BoxDesc& b, void* buf, const double* rho0, const double* u0,
                        const double* f, int which, hipStream_t st) {
    if (b.N == 0) return hipSuccess;
    auto* p = static_cast<typename S::T*>(buf);
    if (which == 0) k_init<L, S><<<grid_for_box(b), 256, 0, st>>>(b, p, rho0, u0);
    else k_put<L, S><<<grid_for_box(b), 256, 0, st>>>(b, p, f);
    return hipGetLastError();
  }
};

template <class L, class S>
struct GatherFn {
  static hipError_t run(const BoxDesc& b, const void* buf, const int64_t* sites, int64_t n,
                        int which, double* out, hipStream_t st) {
    if (n == 0) return hipSuccess;
    const auto* p = static_cast<const typename S::T*>(buf);
    if (!sites) k_populations<L, S><<<grid_for_box(b), 256, 0, st>>>(b, p, out);
    else k_gather<L, S><<<grid_for(n, 256), 256, 0, st>>>(b, p, sites, n, which, out);
    return hipGetLastError();
  }
};

template <class L, class S>
struct MomentsFn {
  static hipError_t run(const BoxDesc& b, const void* buf, double* rho, double* u,
                        hipStream_t st) {
    if (b.N == 0) return hipSuccess;
    k_moments<L, S><<<grid_for_box(b), 256, 0, st>>>(b, static_cast<const typename S::T*>(buf),
                                                     rho, u);
    return hipGetLastError();
  }
};

}  // namespace

hipError_t launch_validate_init(const BoxDesc& b, const double* rho0, const double* u0,
                                unsigned long long* bad, hipStream_t st) {
  if (b.N == 0) return hipSuccess;
  k_validate<<<grid_for(b.N, 256), 256, 0, st>>>(b.N, b.D, b.lattice == 19, rho0, u0, bad);
  return hipGetLastError();
}

hipError_t launch_scatter(const BoxDesc& b, void* buf, const double* rho0, const double* u0,
                          const double* f, int which, hipStream_t st) {
  return dispatch<ScatterFn>(b.lattice, b.storage, b, buf, rho0, u0, f, which, st);
}

hipError_t launch_gather(const BoxDesc& b, const void* buf, const int64_t* sites, int64_t n,
                         int which, double* out, hipStream_t st) {
  return dispatch<GatherFn>(b.lattice, b.storage, b, buf, sites, n, which, out, st);
}

hipError_t launch_moments(const BoxDesc& b, const void* buf, double* rho, double* u,
                          hipStream_t st) {
  return dispatch<MomentsFn>(b.lattice, b.storage, b, buf, rho, u, st);
}

hipError_t launch_reduce(void* counts, const void* sums, int nblocks, Reduced* out,
                         hipStream_t st) {
  auto* cr = static_cast<CountRec*>(counts);
  const auto* sr = static_cast<const SumRec*>(sums);
  if (nblocks <= kOneLaunch) {
    k_reduce<false><<<1, kBlock, 0, st>>>(cr, sr, nblocks, nblocks, out);
    return hipGetLastError();
  }
  // at least kOneLaunch / kMaxParts records a chunk; the last may be short,
  // but never shorter than a partial result
  static_assert(kOneLaunch / kMaxParts >= kPartWords, "a chunk's pads hold its result");
  int parts = kMaxParts;
  int chunk = (nblocks + parts - 1) / parts;
  while ((nblocks - 1) % chunk + 1 < kPartWords) ++chunk;
  parts = (nblocks + chunk - 1) / chunk;
  k_reduce<false><<<parts, kBlock, 0, st>>>(cr, sr, nblocks, chunk, nullptr);
  k_reduce<true><<<1, kBlock, 0, st>>>(cr, nullptr, nblocks, chunk, out);
  return hipGetLastError();
}

hipError_t launch_copy_f64(const double* src, double* dst, int64_t n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  k_copy_f64<<<grid_for(n, 256), 256, 0, st>>>(src, dst, n);
  return hipGetLastError();
}

StepLauncher step_launcher(int lattice, int storage, int mode, int fp64, int entropy) {
  if (entropy == 1) return step_launcher_burg(lattice, storage, mode, fp64);
  if (entropy != 0) return nullptr;
  switch (lattice) {
    case 1: return step_launcher_d1(storage, mode, fp64);
    case 2: return step_launcher_d2(storage, mode, fp64);
    case 3: return step_launcher_d3(storage, mode, fp64);
    case 19: return step_launcher_q19(storage, mode, fp64);
    default: return nullptr;
  }
}

}  // namespace elbm
