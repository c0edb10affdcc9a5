// Resident Krylov iterations of small grids: one cooperative launch runs a
// whole chunk of iterations of one solve with its vectors held in registers.
//
// A small grid's iteration is latency, not traffic: at 32^3 each pass of the
// two-reduction BiCGStab took 9-11 us as a launch of its own, of which the
// 64 workgroups spent most in dependent trips to memory (plane loads, partial
// store, arrival counter, the last workgroup's reduction) and the kernel
// boundary.  Here every workgroup keeps one tile -- the tile a per-pass
// launch gives it -- with r, p, v, t, x and the shadow residual in registers
// from the first iteration of the chunk to the last, and a pass costs one
// exchange between the workgroups:
//   * the operator's output (v = A p, then t = A s) goes to its vector with
//     agent-scope stores; the neighbours read their halo cells of it back.
//     Every workgroup keeps r and p of its halo cells as well and updates
//     them with the own cells' operations, so nothing else is exchanged;
//   * the tile's partial sums go to a slot of their own once those stores
//     have completed, so a partial that has arrived says that the halo has.
//     Every workgroup waits for all partials, adds them in the per-pass
//     form's order and applies the finalizer to its own copy of the scalars:
//     no arrival counter, no last workgroup, no cache-wide fence.
// A slot waits to be written holding kEmpty, a NaN payload no sum produces;
// three sets of slots take turns, so that a workgroup can empty the set of
// the exchange before while the others read the current one.
//
// Measured (us an iteration, one launch per pass -> resident):
//   two-reduction BiCGStab, FP64   32^3 20.4 -> 9.5    64^3 26.5 -> 16.4
//   CG, one reduction, FP64        32^3 10.5 -> 5.0    64^3 14.9 -> 7.5
//
// Tiles, per-thread order of the dot products, reduction order and
// finalizers are those of the per-pass kernels, so the iterates are bitwise
// theirs.  Waits are bounded: a workgroup that gives up sets the scalar
// block's `timeout` and leaves, and so does every other at its next wait.
#include <stddef.h>

#include <atomic>

#include "device.hpp"
#include "internal.hpp"
#include "phases.hpp"

namespace wfa {

namespace {

constexpr uint64_t kEmpty = 0x7ff85eed0badf00dull;   // slot not written yet
constexpr int kRing = 3;
constexpr int kSpinLimit = 1 << 20;   // polls of one wait (each a trip to memory)

template <typename T>
struct ResArgs {
  Geo geo;
  Op<T> op;
  const float* kappa;
  T* x;
  const T* rh;
  T* t;
  T *r[2], *p[2], *v[2];
  double* ring;      // kRing sets of kMaxReduce x ntiles slots
  Scalars* sc;
  int iters;
  int parity;
  int hashed;
};

template <typename T>
__device__ __forceinline__ void st_agent(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T ld_agent(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What one workgroup shares in LDS.
template <typename T, bool CELL, int Z>
struct ResShared {
  using TS = TileShape<2>;
  T u[Z][TS::LH * TS::LW];                          // staged vector, with its x-y halo
  float k[CELL ? Z : 1][CELL ? TS::LH * TS::LW : 1];  // diffusivity, the same layout
  double red[kWaves * kMaxReduce];
  Scalars sc;
  int bad;
};

// One tile's cells as a thread sees them: its RY = 2 rows of up to Z planes,
// the x-y halo cell it loads of each plane, and the z-halo cells below and
// above its rows.
template <typename T, bool CELL, int Z>
struct ResTile {
  using TS = TileShape<2>;
  static constexpr int LW = TS::LW, LH = TS::LH, TY = TS::TY;
  static constexpr int RY = 2;
  const Geo& g;
  const Op<T>& op;
  ResShared<T, CELL, Z>& sh;
  size_t base;            // first cell of the tile's first plane
  size_t plane;
  int nzt;                // planes of this tile
  bool own[RY];
  int poff[RY], lidx[RY];
  uint32_t ins_xy[RY];
  int hl = -1, hoff = 0;
  bool hval = false;
  bool zlo, zhi;          // the z neighbours exist
  int k0;
  float kc[CELL ? Z : 1][RY], kzh[2][RY];

  __device__ ResTile(const Geo& geo, const Op<T>& o, ResShared<T, CELL, Z>& s, int tile,
                     const float* __restrict__ kappa)
      : g(geo), op(o), sh(s) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int tx = tile % g.tiles_x;
    const int rest = tile / g.tiles_x;
    const int ty = rest % g.tiles_y;
    const int tz = rest / g.tiles_y;
    const int x0 = tx * kTX, y0 = ty * TY;
    k0 = tz * g.zc;
    nzt = min(g.zc, g.nz - k0);
    plane = (size_t)g.plane;
    base = (size_t)k0 * plane;
    zlo = k0 > 0;
    zhi = k0 + nzt < g.nz;
    const int i = x0 + lane, nx = g.nx, ny = g.ny;
#pragma unroll
    for (int r = 0; r < RY; ++r) {
      const int j = y0 + wave * RY + r;
      own[r] = i < nx && j < ny;
      poff[r] = own[r] ? i + nx * j : 0;
      lidx[r] = (wave * RY + r + 1) * LW + lane + 1;
      ins_xy[r] = (i > 0 ? 1u : 0u) | (i < nx - 1 ? 2u : 0u) | (j > 0 ? 4u : 0u) |
                  (j < ny - 1 ? 8u : 0u);
    }
    const int hs = threadIdx.x;
    int hi = 0, hj = 0;
    if (hs < kTX) { hi = x0 + hs; hj = y0 - 1; hl = hs + 1; }
    else if (hs < 2 * kTX) { hi = x0 + hs - kTX; hj = y0 + TY; hl = (LH - 1) * LW + hs - kTX + 1; }
    else if (hs < 2 * kTX + TY) { hi = x0 - 1; hj = y0 + hs - 2 * kTX; hl = (hs - 2 * kTX + 1) * LW; }
    else if (hs < TS::NHALO) { hi = x0 + kTX; hj = y0 + hs - 2 * kTX - TY; hl = (hs - 2 * kTX - TY + 1) * LW + LW - 1; }
    if (hl >= 0) {
      hval = hi >= 0 && hi < nx && hj >= 0 && hj < ny;
      hoff = hval ? hi + nx * hj : 0;
    }
    if constexpr (CELL) {
      float kh[Z];
      load_own(kappa, kc, 1.f);
      load_halo(kappa, kh, kzh, 1.f);
#pragma unroll
      for (int k = 0; k < Z; ++k) {
#pragma unroll
        for (int r = 0; r < RY; ++r) sh.k[k][lidx[r]] = kc[k][r];
        if (hl >= 0) sh.k[k][hl] = kh[k];
      }
    }
  }

  __device__ size_t at(int k, int r) const { return base + (size_t)k * plane + poff[r]; }

  template <typename V>
  __device__ void load_own(const V* a, V (&o)[Z][RY], V none = V(0)) const {
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int r = 0; r < RY; ++r) o[k][r] = (k < nzt && own[r]) ? a[at(k, r)] : none;
  }
  // halo cells written before this launch (plain loads) ...
  template <typename V>
  __device__ void load_halo(const V* a, V (&h)[Z], V (&z)[2][RY], V none = V(0)) const {
    halo(h, z, none, [&](size_t i) { return a[i]; });
  }
  // ... and by another workgroup of it
  __device__ void load_halo_agent(const T* a, T (&h)[Z], T (&z)[2][RY]) const {
    halo(h, z, T(0), [&](size_t i) { return ld_agent(a + i); });
  }
  template <typename V, class F>
  __device__ void halo(V (&h)[Z], V (&z)[2][RY], V none, F ld) const {
#pragma unroll
    for (int k = 0; k < Z; ++k)
      h[k] = (hval && k < nzt) ? ld(base + (size_t)k * plane + hoff) : none;
#pragma unroll
    for (int r = 0; r < RY; ++r) {
      z[0][r] = (zlo && own[r]) ? ld(base - plane + poff[r]) : none;
      z[1][r] = (zhi && own[r]) ? ld(base + (size_t)nzt * plane + poff[r]) : none;
    }
  }
  __device__ void store_own(T* a, const T (&o)[Z][RY]) const {
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int r = 0; r < RY; ++r)
        if (k < nzt && own[r]) a[at(k, r)] = o[k][r];
  }
  __device__ void store_own_agent(T* a, const T (&o)[Z][RY]) const {
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int r = 0; r < RY; ++r)
        if (k < nzt && own[r]) st_agent(a + at(k, r), o[k][r]);
  }

  // A u of the own cells (0 elsewhere), u staged with its halo.
  __device__ void apply(const T (&u)[Z][RY], const T (&h)[Z], const T (&z)[2][RY],
                        T (&Au)[Z][RY]) {
#pragma unroll
    for (int k = 0; k < Z; ++k) {
#pragma unroll
      for (int r = 0; r < RY; ++r) sh.u[k][lidx[r]] = u[k][r];
      if (hl >= 0) sh.u[k][hl] = h[k];
    }
    __syncthreads();
    T kz[RY];
#pragma unroll
    for (int r = 0; r < RY; ++r) kz[r] = T(0);
#pragma unroll
    for (int k = 0; k < Z; ++k) {
      const uint32_t ins_z = (k0 + k > 0 ? 16u : 0u) | (k0 + k < g.nz - 1 ? 32u : 0u);
#pragma unroll
      for (int r = 0; r < RY; ++r) {
        Au[k][r] = T(0);
        if (k < nzt && own[r]) {
          const int l = lidx[r];
          const T* Lu = sh.u[k];
          const bool last = k + 1 >= nzt;
          const T lo = k > 0 ? u[k > 0 ? k - 1 : 0][r] : z[0][r];
          const T hi = last ? z[1][r] : u[k + 1 < Z ? k + 1 : k][r];
          const T nb[6] = {Lu[l - 1], Lu[l + 1], Lu[l - LW], Lu[l + LW], lo, hi};
          T kn[6] = {T(1), T(1), T(1), T(1), T(1), T(1)};
          T kP = T(1);
          if constexpr (CELL) {
            const float* Lk = sh.k[k];
            kP = (T)kc[k][r];
            kn[0] = (T)Lk[l - 1]; kn[1] = (T)Lk[l + 1];
            kn[2] = (T)Lk[l - LW]; kn[3] = (T)Lk[l + LW];
            kn[4] = (T)(k > 0 ? kc[k > 0 ? k - 1 : 0][r] : kzh[0][r]);
            kn[5] = (T)(last ? kzh[1][r] : kc[k + 1 < Z ? k + 1 : k][r]);
          }
          T dg;
          Au[k][r] = cell_apply<T, CELL>(op, u[k][r], nb, kP, kn, ins_xy[r] | ins_z, dg, kz[r],
                                         k > 0);
        }
      }
    }
  }
};

// One exchange: publishes this tile's sums and returns the grid's, in thread
// 0 (the order of publish_and_finalize).  The caller's agent-scope stores
// are complete before the sums can be seen.  `seq` numbers the exchanges of
// the solve.  False once a wait has given up.
template <int NV>
__device__ __forceinline__ bool exchange(double (&v)[NV], double* ring, int tile, int nt, int seq,
                                         double* red, int* bad) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  block_sum<NV>(v, red);
  double* set = ring + (size_t)(seq % kRing) * kMaxReduce * nt;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      uint64_t bits = (uint64_t)__double_as_longlong(v[q]);
      if (bits == kEmpty) bits = 0x7ff8000000000000ull;
      st_agent((uint64_t*)set + (size_t)q * nt + tile, bits);
    }
  }
  double s[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) s[q] = 0.0;
  for (int c = threadIdx.x; c < nt; c += kThreads) {
    uint64_t got[NV];
    int spins = 0;
    bool all;
    do {
      all = true;
#pragma unroll
      for (int q = 0; q < NV; ++q) got[q] = ld_agent((const uint64_t*)set + (size_t)q * nt + c);
#pragma unroll
      for (int q = 0; q < NV; ++q) all = all && got[q] != kEmpty;
    } while (!all && ++spins < kSpinLimit);
    if (!all) *bad = 1;
#pragma unroll
    for (int q = 0; q < NV; ++q) s[q] += __longlong_as_double((long long)got[q]);
  }
#pragma unroll
  for (int q = 0; q < NV; ++q) v[q] = s[q];
  block_sum<NV>(v, red);
  // every workgroup has read the set before: empty this tile's slots of it
  if (threadIdx.x < kMaxReduce)
    st_agent((uint64_t*)ring + (size_t)((seq + kRing - 1) % kRing) * kMaxReduce * nt +
                 (size_t)threadIdx.x * nt + tile,
             (uint64_t)kEmpty);
  return *bad == 0;
}

// The scalars go back without the timeout word, which any workgroup may set.
template <class Sh>
__device__ __forceinline__ void leave(Sh& sh, Scalars* sc, bool first_tile, int seq) {
  constexpr int kWords = sizeof(Scalars) / 4;
  constexpr int kTimeout = offsetof(Scalars, timeout) / 4;
  if (threadIdx.x == 0) sh.sc.seq = seq;
  __syncthreads();
  if (sh.bad) {
    if (threadIdx.x == 0) st_agent(&sc->timeout, 1);
  } else if (first_tile && threadIdx.x < kWords && threadIdx.x != kTimeout) {
    ((uint32_t*)sc)[threadIdx.x] = ((const uint32_t*)&sh.sc)[threadIdx.x];
  }
}

// Two-reduction BiCGStab: passes AC and B2 (PhAC, PhB2) on resident tiles.
template <typename T, bool CELL, int Z>
__global__ void __launch_bounds__(kThreads) k_resident_bicgstab2(ResArgs<T> a) {
  constexpr int RY = 2;
  __shared__ ResShared<T, CELL, Z> sh;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int nt = a.geo.ntiles;
  if (threadIdx.x == 0) {
    sh.sc = *a.sc;
    sh.bad = 0;
  }
  __syncthreads();
  if (sh.sc.status != ST_RUN || sh.sc.restart) return;
  ResTile<T, CELL, Z> tl(a.geo, a.op, sh, tile, a.kappa);
  int par = a.parity;
  int seq = sh.sc.seq;
  T r[Z][RY], p[Z][RY], v[Z][RY], t[Z][RY], x[Z][RY], rh[Z][RY];
  T hr[Z], hp[Z], hv[Z], ht[Z];
  T zr[2][RY], zp[2][RY], zv[2][RY], zt[2][RY];
  const bool first0 = sh.sc.first != 0;
  tl.load_own(a.r[par], r);
  tl.load_halo(a.r[par], hr, zr);
#pragma unroll
  for (int k = 0; k < Z; ++k) {
    hp[k] = hv[k] = ht[k] = T(0);
#pragma unroll
    for (int q = 0; q < RY; ++q) p[k][q] = v[k][q] = t[k][q] = x[k][q] = T(0);
  }
#pragma unroll
  for (int q = 0; q < RY; ++q)
#pragma unroll
    for (int e = 0; e < 2; ++e) zp[e][q] = zv[e][q] = zt[e][q] = T(0);
  if (!first0) {
    tl.load_own(a.p[par], p);
    tl.load_own(a.v[par], v);
    tl.load_own(a.t, t);
    tl.load_halo(a.p[par], hp, zp);
    tl.load_halo(a.v[par], hv, zv);
    tl.load_halo(a.t, ht, zt);
  }
  if (!sh.sc.x_zero) tl.load_own(a.x, x);
  if (a.hashed) {
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int q = 0; q < RY; ++q) rh[k][q] = hashed_shadow<T>(tl.at(k, q));
  } else {
    tl.load_own(a.rh, rh);
  }

  T u[Z][RY], hu[Z], zu[2][RY];
  for (int it = 0; it < a.iters; ++it) {
    // ---- pass AC: the update of the iteration before, v' = A p'
    double s3[3] = {0.0, 0.0, 0.0};
    {
      const T alpha = (T)sh.sc.alpha, omega = (T)sh.sc.omega, beta = (T)sh.sc.beta;
      const int first = sh.sc.first;
#pragma unroll
      for (int k = 0; k < Z; ++k)
#pragma unroll
        for (int q = 0; q < RY; ++q) {
          if (!first) {
            const T s = minus_ax(r[k][q], alpha, v[k][q]);
            const T rn = minus_ax(s, omega, t[k][q]);
            x[k][q] = next_x(x[k][q], p[k][q], s, alpha, omega);
            p[k][q] = next_p(rn, p[k][q], v[k][q], beta, omega);
            r[k][q] = rn;
          } else {
            p[k][q] = r[k][q];
          }
          if (k < tl.nzt && tl.own[q]) {
            dot_acc(s3[1], (double)rh[k][q], (double)r[k][q]);
            dot_acc(s3[2], (double)r[k][q], (double)r[k][q]);
          }
        }
      auto update = [&](T& hr_, T& hp_, T hv_, T ht_) {
        if (first) { hp_ = hr_; return; }
        const T rn = minus_ax(minus_ax(hr_, alpha, hv_), omega, ht_);
        hp_ = next_p(rn, hp_, hv_, beta, omega);
        hr_ = rn;
      };
#pragma unroll
      for (int k = 0; k < Z; ++k) update(hr[k], hp[k], hv[k], ht[k]);
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int q = 0; q < RY; ++q) update(zr[e][q], zp[e][q], zv[e][q], zt[e][q]);
    }
    par ^= 1;
    tl.apply(p, hp, zp, v);
    tl.store_own_agent(a.v[par], v);
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int q = 0; q < RY; ++q)
        if (k < tl.nzt && tl.own[q]) dot_acc(s3[0], (double)rh[k][q], (double)v[k][q]);
    bool ok = exchange<3>(s3, a.ring, tile, nt, seq++, sh.red, &sh.bad);
    if (!ok) break;
    tl.store_own(a.p[par], p);
    tl.load_halo_agent(a.v[par], hv, zv);
    if (threadIdx.x == 0) FinAC{&sh.sc}(s3);
    __syncthreads();
    if (sh.sc.status != ST_RUN || sh.sc.restart) break;

    // ---- pass B2: t = A s
    double s4[4] = {0.0, 0.0, 0.0, 0.0};
    {
      const T alpha = (T)sh.sc.alpha;
#pragma unroll
      for (int k = 0; k < Z; ++k) {
        hu[k] = minus_ax(hr[k], alpha, hv[k]);
#pragma unroll
        for (int q = 0; q < RY; ++q) u[k][q] = minus_ax(r[k][q], alpha, v[k][q]);
      }
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int q = 0; q < RY; ++q) zu[e][q] = minus_ax(zr[e][q], alpha, zv[e][q]);
    }
    tl.apply(u, hu, zu, t);
    tl.store_own_agent(a.t, t);
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int q = 0; q < RY; ++q)
        if (k < tl.nzt && tl.own[q]) {
          dot_acc(s4[0], (double)t[k][q], (double)u[k][q]);
          dot_acc(s4[1], (double)t[k][q], (double)t[k][q]);
          dot_acc(s4[2], (double)rh[k][q], (double)u[k][q]);
          dot_acc(s4[3], (double)rh[k][q], (double)t[k][q]);
        }
    ok = exchange<4>(s4, a.ring, tile, nt, seq++, sh.red, &sh.bad);
    if (!ok) break;
    tl.load_halo_agent(a.t, ht, zt);
    if (threadIdx.x == 0) FinB2{&sh.sc}(s4);
    __syncthreads();
    if (sh.sc.status != ST_RUN || sh.sc.restart) break;
  }
  tl.store_own(a.r[par], r);
  if (!sh.sc.x_zero) tl.store_own(a.x, x);
  leave(sh, a.sc, tile == 0, seq);
}

// CG with one reduction per iteration (PhCg1): w = A r exchanged, one
// exchange an iteration.  v holds w, p holds s (double-buffered), t holds p.
template <typename T, bool CELL, int Z>
__global__ void __launch_bounds__(kThreads) k_resident_cg1(ResArgs<T> a) {
  constexpr int RY = 2;
  __shared__ ResShared<T, CELL, Z> sh;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int nt = a.geo.ntiles;
  if (threadIdx.x == 0) {
    sh.sc = *a.sc;
    sh.bad = 0;
  }
  __syncthreads();
  if (sh.sc.status != ST_RUN || sh.sc.restart) return;
  ResTile<T, CELL, Z> tl(a.geo, a.op, sh, tile, a.kappa);
  int par = a.parity;
  int seq = sh.sc.seq;
  T r[Z][RY], w[Z][RY], s[Z][RY], p[Z][RY], x[Z][RY];
  T hr[Z], hw[Z], hs[Z], zr[2][RY], zw[2][RY], zs[2][RY];
  const int stage0 = sh.sc.stage;
  tl.load_own(a.r[par], r);
  tl.load_halo(a.r[par], hr, zr);
#pragma unroll
  for (int k = 0; k < Z; ++k) {
    hw[k] = hs[k] = T(0);
#pragma unroll
    for (int q = 0; q < RY; ++q) w[k][q] = s[k][q] = p[k][q] = x[k][q] = T(0);
  }
#pragma unroll
  for (int q = 0; q < RY; ++q)
#pragma unroll
    for (int e = 0; e < 2; ++e) zw[e][q] = zs[e][q] = T(0);
  if (stage0 > 0) {
    tl.load_own(a.v[par], w);
    tl.load_halo(a.v[par], hw, zw);
  }
  if (stage0 > 1) {
    tl.load_own(a.p[par], s);
    tl.load_halo(a.p[par], hs, zs);
    tl.load_own(a.t, p);
  }
  if (!sh.sc.x_zero) tl.load_own(a.x, x);

  int stage = stage0;
  for (int it = 0; it < a.iters; ++it) {
    double s2[2] = {0.0, 0.0};
    const T alpha = (T)sh.sc.alpha, beta = (T)sh.sc.beta;
    stage = sh.sc.stage;
    auto s_new = [&](T w_, T s_) { return stage == 1 ? w_ : fma_t(beta, s_, w_); };
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int q = 0; q < RY; ++q) {
        if (stage != 0) {
          s[k][q] = s_new(w[k][q], s[k][q]);
          p[k][q] = stage == 1 ? r[k][q] : fma_t(beta, p[k][q], r[k][q]);
          x[k][q] = fma_t(alpha, p[k][q], x[k][q]);
          r[k][q] = fma_t(-alpha, s[k][q], r[k][q]);
        }
        if (k < tl.nzt && tl.own[q]) dot_acc(s2[0], (double)r[k][q], (double)r[k][q]);
      }
    if (stage != 0) {
#pragma unroll
      for (int k = 0; k < Z; ++k) {
        hs[k] = s_new(hw[k], hs[k]);
        hr[k] = fma_t(-alpha, hs[k], hr[k]);
      }
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int q = 0; q < RY; ++q) {
          zs[e][q] = s_new(zw[e][q], zs[e][q]);
          zr[e][q] = fma_t(-alpha, zs[e][q], zr[e][q]);
        }
    }
    par ^= 1;
    tl.apply(r, hr, zr, w);
    tl.store_own_agent(a.v[par], w);
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int q = 0; q < RY; ++q)
        if (k < tl.nzt && tl.own[q]) dot_acc(s2[1], (double)w[k][q], (double)r[k][q]);
    if (!exchange<2>(s2, a.ring, tile, nt, seq++, sh.red, &sh.bad)) break;
    tl.store_own(a.r[par], r);
    tl.load_halo_agent(a.v[par], hw, zw);
    if (threadIdx.x == 0) FinCg1{&sh.sc}(s2);
    __syncthreads();
    if (sh.sc.status != ST_RUN || sh.sc.restart) break;
  }
  if (stage != 0) {
    tl.store_own(a.p[par], s);
    tl.store_own(a.t, p);
    tl.store_own(a.x, x);
  }
  leave(sh, a.sc, tile == 0, seq);
}

// A kernel and the workgroups of it that fit on the current device at once
// (looked up once per device).
template <typename T>
struct Entry {
  void (*kernel)(ResArgs<T>) = nullptr;
  int fit = 0;
};

template <typename T, void (*K)(ResArgs<T>)>
Entry<T> entry() {
  constexpr int kDevices = 16;
  static std::atomic<int> known[kDevices];
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevices) return {};
  int fit = known[dev].load(std::memory_order_relaxed);
  if (fit == 0) {
    int per_cu = 0, cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)K, kThreads, 0) !=
            hipSuccess)
      return {};
    fit = per_cu * cus;
    known[dev].store(fit, std::memory_order_relaxed);
  }
  return {K, fit};
}

template <typename T, bool CELL, int Z>
Entry<T> entry_of(int kind) {
  return kind == kResidentCg1 ? entry<T, k_resident_cg1<T, CELL, Z>>()
                              : entry<T, k_resident_bicgstab2<T, CELL, Z>>();
}

template <typename T>
Entry<T> entry_for(const Launch<T>& L, int kind) {
  const int zc = L.tl.geo.zc;
  if (zc <= 2) return L.cell ? entry_of<T, true, 2>(kind) : entry_of<T, false, 2>(kind);
  if (zc <= 4) return L.cell ? entry_of<T, true, 4>(kind) : entry_of<T, false, 4>(kind);
  return {};
}

}  // namespace

template <typename T>
bool resident_fits(const Launch<T>& L, int kind) {
  const Geo& g = L.tl.geo;
  if (L.tl.ry != 2 || g.ntiles > kResidentTiles) return false;
  return entry_for<T>(L, kind).fit >= g.ntiles;
}

template <typename T>
hipError_t launch_resident(const Launch<T>& L, int kind, T* x, T* const (&r)[2], const T* rh,
                           T* const (&p)[2], T* const (&v)[2], T* t, int iters, int parity) {
  ResArgs<T> a{};
  a.geo = L.tl.geo;
  a.op = L.op;
  a.kappa = L.kappa;
  a.x = x; a.rh = rh; a.t = t;
  for (int q = 0; q < 2; ++q) { a.r[q] = r[q]; a.p[q] = p[q]; a.v[q] = v[q]; }
  a.ring = L.ring;
  a.sc = L.sc;
  a.iters = iters;
  a.parity = parity;
  a.hashed = L.shadow;
  void* args[] = {(void*)&a};
  return hipLaunchCooperativeKernel((const void*)entry_for<T>(L, kind).kernel, dim3(a.geo.ntiles),
                                    dim3(kThreads), args, 0, L.stream);
}

// The solve's scalars, with every slot of the ring empty.
__global__ void __launch_bounds__(kThreads)
k_set_resident(Scalars* __restrict__ dst, Scalars v, uint64_t* __restrict__ ring, int slots) {
  if (threadIdx.x == 0) *dst = v;
  for (int e = threadIdx.x; e < slots; e += kThreads) ring[e] = kEmpty;
}

void launch_set_resident(Scalars* dst, const Scalars& v, double* ring, int ntiles, hipStream_t s) {
  hipLaunchKernelGGL(k_set_resident, dim3(1), dim3(kThreads), 0, s, dst, v, (uint64_t*)ring,
                     kRing * kMaxReduce * ntiles);
}

#define WFA_RES(T)                                                                             \
  template bool resident_fits<T>(const Launch<T>&, int);                                      \
  template hipError_t launch_resident<T>(const Launch<T>&, int, T*, T* const (&)[2], const T*, \
                                         T* const (&)[2], T* const (&)[2], T*, int, int);
WFA_RES(float)
WFA_RES(double)
#undef WFA_RES

}  // namespace wfa
