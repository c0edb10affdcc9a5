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
//   * the operator's output (v = A p, then t = A s) of a tile's boundary
//     cells goes to an exchange vector with agent-scope stores; the
//     neighbours read their halo cells of it back.  Every workgroup keeps r
//     and p of its halo cells as well and updates them with the own cells'
//     operations, so nothing else is exchanged;
//   * the tile's partial sums go to slots of their own.  Every workgroup
//     waits for all partials, adds them in the per-pass form's order and
//     applies the finalizer to its own copy of the scalars: no arrival
//     counter, no last workgroup, no cache-wide fence.
// A cell or slot that waits to be written holds a NaN payload no arithmetic
// produces (`Empty`), so a value's arrival is its own signal: nothing waits
// for a store to complete before another announces it.  Three exchange
// vectors and three sets of slots take turns: once a workgroup has passed
// exchange e, every other has arrived there and is done with e - 1, whose
// cells and slots it then empties; those stores are complete before it
// arrives at e + 1, and so before anyone waits for exchange e + 2.
//
// A pass is one dependent chain of some 8000 cycles, so what bounds it is the
// latency of each link.  A one-way trip between two XCDs takes 0.5-0.7 us (a
// store past the caches until another XCD's load sees it); around it stand
// the update, two barriers, the sums and the finalizer.  Every load of a link
// is issued at once, without a branch; the operator's rows are formed once
// per launch (in LDS, or for a constant diffusivity in registers); the
// finalizer runs on registers.
//
// Measured (us an iteration, one launch per pass -> resident):
//   two-reduction BiCGStab, FP64   32^3 20.0 -> 5.8    64^3 25.8 -> 9.4
//   CG, one reduction, FP64        32^3 10.5 -> 3.0    64^3 14.4 -> 4.4
//   (8.9 / 15.1 and 4.6 / 7.1 where a pass waited for its stores before it
//   published its sums, with branches around the cells outside the grid)
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

template <typename T>
struct Empty;          // the value not written yet, and what stands in for it
template <>
struct Empty<double> {
  using Bits = uint64_t;
  static constexpr Bits value = 0x7ff85eed0badf00dull, nan = 0x7ff8000000000000ull;
};
template <>
struct Empty<float> {
  using Bits = uint32_t;
  static constexpr Bits value = 0x7fc5eed1u, nan = 0x7fc00000u;
};
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
  T* set[kRing];     // exchange vectors; set[0] is not read when the launch starts
  double* ring;      // `copies` rings of kRing sets of kMaxReduce x ntiles slots
  int copies;
  Scalars* sc;
  int iters;
  int parity;
  int hashed;
};

// Vectors are addressed through buffer resources with byte offsets, so that
// a cell outside the grid (offset kNowhere) reads 0 and is not written
// without a branch: a pass is a short chain, and each branch around a load
// had put the loads behind it in series.
constexpr int kNowhere = 0x7ffff000;
constexpr int kAgent = 16;   // sc1: the access goes past this XCD's caches
using Rsrc = __amdgpu_buffer_rsrc_t;
__device__ __forceinline__ Rsrc rsrc(const void* p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
template <typename V, int AUX>
__device__ __forceinline__ V buf_load(Rsrc r, int off) {
  if constexpr (sizeof(V) == 8)
    return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, AUX));
  else
    return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, AUX));
}
template <int AUX, typename V>
__device__ __forceinline__ void buf_store(Rsrc r, int off, V v) {
  if constexpr (sizeof(V) == 8) {
    using B = decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0, 0, 0));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(B, v), r, off, 0, AUX);
  } else {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, off, 0, AUX);
  }
}
// Exchanged values: stored past the caches, the empty one never among them.
template <typename T>
__device__ __forceinline__ void put_value(Rsrc r, int off, T v) {
  using E = Empty<T>;
  const auto bits = __builtin_bit_cast(typename E::Bits, v);
  buf_store<kAgent>(r, off, bits == E::value ? E::nan : bits);
}
template <typename T>
__device__ __forceinline__ void put_empty(Rsrc r, int off) {
  buf_store<kAgent>(r, off, Empty<T>::value);
}
template <typename T>
__device__ __forceinline__ bool is_empty(T v) {
  return __builtin_bit_cast(typename Empty<T>::Bits, v) == Empty<T>::value;
}

template <typename T>
__device__ __forceinline__ T* pick(T* const (&pair)[2], int par) {
  return par ? pair[1] : pair[0];
}

// What one workgroup shares in LDS.
template <typename T, bool CELL, int Z>
struct ResShared {
  using TS = TileShape<2>;
  static constexpr int kPlane = TS::LH * TS::LW + 2;   // the last slot: threads without a halo cell
  T u[Z][kPlane];                                      // staged vector, with its x-y halo
  T coef[CELL ? 7 : 1][CELL ? Z * 2 : 1][CELL ? kThreads : 1];   // own cells' operator rows
  double red[2][kWaves * kMaxReduce];
  Scalars sc;
  int bad;
};

// One tile's cells as a thread sees them: its RY = 2 rows of up to Z planes,
// the x-y halo cell it keeps of each plane, and the z-halo cells below and
// above its rows.
template <typename T, bool CELL, int Z>
struct ResTile {
  using TS = TileShape<2>;
  static constexpr int LW = TS::LW, LH = TS::LH, TY = TS::TY;
  static constexpr int RY = 2;
  using Own = T[Z][RY];
  using Halo = T[Z];
  using HaloZ = T[2][RY];
  const Op<T>& op;
  ResShared<T, CELL, Z>& sh;
  size_t bytes;           // of one vector
  int off[Z][RY];         // byte offsets of the own cells,
  int hoff[Z], zoff[2][RY];   // of the halo cells,
  int boff[Z][RY];        // and of the own cells another tile reads
  bool own[RY];
  int cell0[RY], plane;   // index of the own cells of the first plane
  int lidx[RY], hl;
  int nzt;                // planes of this tile
  T diag[CELL ? 1 : Z][RY];      // constant diffusivity: the operator's rows, from the
  uint32_t ins[RY], ins0, ins1;  // faces inside (x and y by row; first and last plane)

  __device__ ResTile(const Geo& g, const Op<T>& o, ResShared<T, CELL, Z>& s, int tile,
                     const float* __restrict__ kappa)
      : op(o), sh(s) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int tx = tile % g.tiles_x;
    const int rest = tile / g.tiles_x;
    const int ty = rest % g.tiles_y;
    const int tz = rest / g.tiles_y;
    const int x0 = tx * kTX, y0 = ty * TY;
    const int k0 = tz * g.zc;
    nzt = min(g.zc, g.nz - k0);
    const bool zlo = k0 > 0, zhi = k0 + nzt < g.nz;
    const int i = x0 + lane, nx = g.nx, ny = g.ny;
    plane = (int)g.plane;
    bytes = (size_t)g.plane * g.nz * sizeof(T);
    const int base = k0 * plane;
    constexpr int W = sizeof(T);
#pragma unroll
    for (int r = 0; r < RY; ++r) {
      const int j = y0 + wave * RY + r;
      own[r] = i < nx && j < ny;
      cell0[r] = base + (own[r] ? i + nx * j : 0);
      lidx[r] = (wave * RY + r + 1) * LW + lane + 1;
      ins[r] = (i > 0 ? 1u : 0u) | (i < nx - 1 ? 2u : 0u) | (j > 0 ? 4u : 0u) |
               (j < ny - 1 ? 8u : 0u);
      const bool edge = (lane == 0 && x0 > 0) || (lane == kTX - 1 && i < nx - 1) ||
                        (j == y0 && y0 > 0) || (j == y0 + TY - 1 && j < ny - 1);
#pragma unroll
      for (int k = 0; k < Z; ++k) {
        off[k][r] = own[r] && k < nzt ? (cell0[r] + k * plane) * W : kNowhere;
        boff[k][r] = edge || (k == 0 && zlo) || (k == nzt - 1 && zhi) ? off[k][r] : kNowhere;
      }
      zoff[0][r] = own[r] && zlo ? (cell0[r] - plane) * W : kNowhere;
      zoff[1][r] = own[r] && zhi ? (cell0[r] + nzt * plane) * W : kNowhere;
    }
    ins0 = zlo ? 16u : 0u;
    ins1 = zhi ? 32u : 0u;
    const int hs = threadIdx.x;
    int hi = -1, hj = 0;
    hl = LH * LW;
    if (hs < kTX) { hi = x0 + hs; hj = y0 - 1; hl = hs + 1; }
    else if (hs < 2 * kTX) { hi = x0 + hs - kTX; hj = y0 + TY; hl = (LH - 1) * LW + hs - kTX + 1; }
    else if (hs < 2 * kTX + TY) { hi = x0 - 1; hj = y0 + hs - 2 * kTX; hl = (hs - 2 * kTX + 1) * LW; }
    else if (hs < TS::NHALO) { hi = x0 + kTX; hj = y0 + hs - 2 * kTX - TY; hl = (hs - 2 * kTX - TY + 1) * LW + LW - 1; }
    const bool hval = hi >= 0 && hi < nx && hj >= 0 && hj < ny;
#pragma unroll
    for (int k = 0; k < Z; ++k)
      hoff[k] = hval && k < nzt ? (base + k * plane + hi + nx * hj) * W : kNowhere;
    operator_rows(kappa);
  }

  __device__ uint32_t inside(int k, int r) const {
    return ins[r] | (k > 0 ? 16u : ins0) | (k < nzt - 1 ? 32u : ins1);
  }

  // The operator's rows: the couplings of the six faces (0 where there is no
  // neighbour) and the diagonal, formed as cell_apply forms them.
  __device__ T row(int k, int r, T kP, const T (&kN)[6], T (&D)[6]) const {
#pragma clang fp contract(off)
    const uint32_t in = inside(k, r);
    T dg = T(1);
#pragma unroll
    for (int f = 0; f < 6; ++f) {
      D[f] = T(0);
      if (in & (1u << f)) {
        if (CELL) {
          const T kf = T(2) * kP * kN[f] * pos_rcp(kP + kN[f]);
          dg += fma_t(op.cD, kf, op.out[f]);
          D[f] = fma_t(op.cD, kf, op.in[f]);
        } else {
          dg += op.cD + op.out[f];
          D[f] = op.cD + op.in[f];
        }
      } else if (op.dir & (1u << f)) {
        dg += CELL ? fma_t(op.cD, kP, op.out[f]) : op.cD + op.out[f];
      }
    }
    return dg;
  }
  __device__ void operator_rows(const float* __restrict__ kappa) {
    if constexpr (CELL) {
      const Rsrc kr = rsrc(kappa, bytes / sizeof(T) * 4);
      constexpr int W = sizeof(T);
      auto ld = [&](int o) {
        const float v = buf_load<float, 0>(kr, o == kNowhere ? kNowhere : o / W * 4);
        return o == kNowhere ? 1.f : v;
      };
      float kc[Z][RY], kz[2][RY];
      float* Lk = (float*)&sh.u[0][0];   // the diffusivity in the staged vector's place
      constexpr int LP = ResShared<T, CELL, Z>::kPlane;
#pragma unroll
      for (int k = 0; k < Z; ++k) {
#pragma unroll
        for (int r = 0; r < RY; ++r) {
          kc[k][r] = ld(off[k][r]);
          Lk[k * LP + lidx[r]] = kc[k][r];
        }
        Lk[k * LP + hl] = ld(hoff[k]);
      }
#pragma unroll
      for (int r = 0; r < RY; ++r)
#pragma unroll
        for (int e = 0; e < 2; ++e) kz[e][r] = ld(zoff[e][r]);
      __syncthreads();
#pragma unroll
      for (int k = 0; k < Z; ++k)
#pragma unroll
        for (int r = 0; r < RY; ++r) {
          const float* L = Lk + k * LP + lidx[r];
          const float lo = k > 0 ? kc[k > 0 ? k - 1 : 0][r] : kz[0][r];
          const float hi = k + 1 >= nzt ? kz[1][r] : kc[k + 1 < Z ? k + 1 : k][r];
          const T kN[6] = {(T)L[-1], (T)L[1], (T)L[-LW], (T)L[LW], (T)lo, (T)hi};
          T D[6];
          const T dg = row(k, r, (T)kc[k][r], kN, D);
#pragma unroll
          for (int f = 0; f < 6; ++f) sh.coef[f][k * RY + r][threadIdx.x] = D[f];
          sh.coef[6][k * RY + r][threadIdx.x] = dg;
        }
      __syncthreads();
    } else {
      const T one[6] = {T(1), T(1), T(1), T(1), T(1), T(1)};
      T D[6];
#pragma unroll
      for (int k = 0; k < Z; ++k)
#pragma unroll
        for (int r = 0; r < RY; ++r) diag[k][r] = row(k, r, T(1), one, D);
    }
  }

  __device__ Rsrc vec(const T* a) const { return rsrc(a, bytes); }
  __device__ void load_own(const T* a, Own& o) const {
    const Rsrc b = vec(a);
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int r = 0; r < RY; ++r) o[k][r] = buf_load<T, 0>(b, off[k][r]);
  }
  template <int AUX>
  __device__ void load_halo(const T* a, Halo& h, HaloZ& z) const {
    const Rsrc b = vec(a);
#pragma unroll
    for (int k = 0; k < Z; ++k) h[k] = buf_load<T, AUX>(b, hoff[k]);
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int r = 0; r < RY; ++r) z[e][r] = buf_load<T, AUX>(b, zoff[e][r]);
  }
  __device__ bool halo_empty(const Halo& h, const HaloZ& z) const {
    bool none = false;
#pragma unroll
    for (int k = 0; k < Z; ++k) none = none | is_empty(h[k]);
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int r = 0; r < RY; ++r) none = none | is_empty(z[e][r]);
    return none;
  }
  __device__ void store_own(T* a, const Own& o) const {
    const Rsrc b = vec(a);
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int r = 0; r < RY; ++r) buf_store<0>(b, off[k][r], o[k][r]);
  }
  __device__ void put_boundary(T* a, const Own& o) const {
    const Rsrc b = vec(a);
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int r = 0; r < RY; ++r) put_value(b, boff[k][r], o[k][r]);
  }
  __device__ void empty_boundary(T* a) const {
    const Rsrc b = vec(a);
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int r = 0; r < RY; ++r) put_empty<T>(b, boff[k][r]);
  }

  // A u of the own cells (0 elsewhere), u staged with its halo.
  __device__ void apply(const Own& u, const Halo& h, const HaloZ& z, Own& Au) {
#pragma clang fp contract(off)
#pragma unroll
    for (int k = 0; k < Z; ++k) {
#pragma unroll
      for (int r = 0; r < RY; ++r) sh.u[k][lidx[r]] = u[k][r];
      sh.u[k][hl] = h[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int r = 0; r < RY; ++r) {
        const T* L = &sh.u[k][lidx[r]];
        const T lo = k > 0 ? u[k > 0 ? k - 1 : 0][r] : z[0][r];
        const T hi = k + 1 >= nzt ? z[1][r] : u[k + 1 < Z ? k + 1 : k][r];
        const T nb[6] = {L[-1], L[1], L[-LW], L[LW], lo, hi};
        T D[6], dg;
        if constexpr (CELL) {
#pragma unroll
          for (int f = 0; f < 6; ++f) D[f] = sh.coef[f][k * RY + r][threadIdx.x];
          dg = sh.coef[6][k * RY + r][threadIdx.x];
        } else {
          const uint32_t in = inside(k, r);
#pragma unroll
          for (int f = 0; f < 6; ++f) D[f] = in & (1u << f) ? op.cD + op.in[f] : T(0);
          dg = diag[k][r];
        }
        T y = apply_coefs(D, dg, u[k][r], nb);
        if (op.jac) y = y * pos_rcp(dg);
        Au[k][r] = off[k][r] != kNowhere ? y : T(0);
      }
  }
};

// Every store of this thread so far is complete (the cells and slots it has
// emptied, before it arrives at the exchange).
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

template <int NV>
__device__ __forceinline__ void wave_sums(double (&v)[NV], double* red) {
#pragma unroll
  for (int q = 0; q < NV; ++q) v[q] = wave_sum(v[q]);
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int q = 0; q < NV; ++q) red[(threadIdx.x >> 6) * NV + q] = v[q];
  }
}
template <int NV>
__device__ __forceinline__ double sum_waves(const double* red, int q) {
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) s += red[w * NV + q];
  return s;
}

// The slots of the partial sums.  Every workgroup reads all of them, and
// hundreds of readers of one line queue up at its home; a tile therefore
// writes its sums to several copies of the ring, and workgroups that fall to
// different XCDs read different ones.
struct Ring {
  Rsrc slots;
  int copies, nt, read;   // read: first slot of the copy this workgroup reads
  __device__ Ring(double* p, int copies_, int nt_)
      : slots(rsrc(p, (size_t)copies_ * kRing * kMaxReduce * nt_ * 8)), copies(copies_), nt(nt_),
        read(((int)blockIdx.x % copies_) * kRing * kMaxReduce * nt_) {}
};

// Exchange number `seq` of the solve: publishes this tile's sums, waits for
// every tile's sums and this tile's halo cells (`poll` loads them and says
// whether one is empty), and leaves the grid's sums in v, in thread 0 (the
// order of publish_and_finalize).  False once a wait has given up.
template <int NV, class Poll>
__device__ __forceinline__ bool exchange(double (&v)[NV], const Ring& ring, int tile, int seq,
                                         double (&red)[2][kWaves * kMaxReduce], int* bad,
                                         Poll poll) {
  const int nt = ring.nt;
  const int set = (seq % kRing) * kMaxReduce * nt;
  const int was = ((seq + kRing - 1) % kRing) * kMaxReduce * nt;
  const int t = threadIdx.x;
  const int tq = t % kMaxReduce, tc = t / kMaxReduce;   // slot and copy of a storing thread
  const int mine = (tc * kRing * kMaxReduce + tq) * nt + tile;
  wave_sums<NV>(v, red[0]);
  __syncthreads();
  if (tq < NV && tc < ring.copies)
    put_value(ring.slots, (set + mine) * 8, sum_waves<NV>(red[0], tq));
  double got[NV];
  bool wait;
  int spins = 0;
  do {
    asm volatile("" ::: "memory");
#pragma unroll
    for (int q = 0; q < NV; ++q)
      got[q] = buf_load<double, kAgent>(
          ring.slots, t < nt ? (ring.read + set + q * nt + t) * 8 : kNowhere);
    wait = poll();
#pragma unroll
    for (int q = 0; q < NV; ++q) wait = wait | is_empty(got[q]);
  } while (wait && ++spins < kSpinLimit);
  if (wait) *bad = 1;
  // the per-pass form adds a thread's partials to zero
#pragma unroll
  for (int q = 0; q < NV; ++q) v[q] = 0.0 + got[q];
  wave_sums<NV>(v, red[1]);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NV; ++q) v[q] = sum_waves<NV>(red[1], q);
  // every workgroup has read the slots before: empty this tile's
  if (tc < ring.copies) put_empty<double>(ring.slots, (was + mine) * 8);
  return *bad == 0;
}

// The finalizer on registers: its loads at once, its stores at once.
template <class Fin, int NV>
__device__ __forceinline__ void finalize(Scalars& sc, const double (&v)[NV]) {
  if (threadIdx.x == 0) {
    Scalars l = sc;
    Fin{&l}(v);
    sc = l;
  }
}

// Before the first exchange of a launch: once every workgroup has loaded its
// cells, the exchange vectors' boundary cells are emptied (the first vector,
// which nobody loads, before).  One exchange without values.
template <typename T, class Tile>
__device__ __forceinline__ bool open_sets(const ResArgs<T>& a, const Tile& tl, const Ring& ring,
                                          int tile, int& seq,
                                          double (&red)[2][kWaves * kMaxReduce], int* bad) {
  tl.empty_boundary(a.set[0]);
  stores_done();
  double none[1] = {0.0};
  if (!exchange<1>(none, ring, tile, seq++, red, bad, [] { return false; }))
    return false;
  tl.empty_boundary(a.set[1]);
  tl.empty_boundary(a.set[2]);
  return true;
}

// The exchange vectors in turn: this exchange's, the next one's and the one
// before's (which needs no emptying after the launch's first exchange).
template <typename T>
struct Sets {
  T *cur, *after, *prev;
  bool fresh = true;
  __device__ void next() {
    T* const c = cur;
    cur = after;
    after = prev;
    prev = c;
    fresh = false;
  }
};

// The scalars go back without the timeout word, which any workgroup may set.
template <class Sh>
__device__ __forceinline__ void leave(Sh& sh, Scalars* sc, bool first_tile, int seq) {
  constexpr int kWords = sizeof(Scalars) / 4;
  constexpr int kTimeout = offsetof(Scalars, timeout) / 4;
  if (threadIdx.x == 0) sh.sc.seq = seq;
  __syncthreads();
  if (sh.bad) {
    if (threadIdx.x == 0)
      __hip_atomic_store(&sc->timeout, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else if (first_tile && threadIdx.x < kWords && threadIdx.x != kTimeout) {
    ((uint32_t*)sc)[threadIdx.x] = ((const uint32_t*)&sh.sc)[threadIdx.x];
  }
}

#define WFA_OWN_CELLS(k, q)             \
  _Pragma("unroll") for (int k = 0; k < Z; ++k) _Pragma("unroll") for (int q = 0; q < 2; ++q)
#define WFA_HALO_Z(e, q)                \
  _Pragma("unroll") for (int e = 0; e < 2; ++e) _Pragma("unroll") for (int q = 0; q < 2; ++q)

// Two-reduction BiCGStab: passes AC and B2 (PhAC, PhB2) on resident tiles.
template <typename T, bool CELL, int Z>
__global__ void __launch_bounds__(kThreads) k_resident_bicgstab2(ResArgs<T> a) {
  using Tile = ResTile<T, CELL, Z>;
  __shared__ ResShared<T, CELL, Z> sh;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  if (threadIdx.x == 0) {
    sh.sc = *a.sc;
    sh.bad = 0;
  }
  __syncthreads();
  if (sh.sc.status != ST_RUN || sh.sc.restart) return;
  Tile tl(a.geo, a.op, sh, tile, a.kappa);
  const Ring ring(a.ring, a.copies, a.geo.ntiles);
  int par = a.parity;
  int seq = sh.sc.seq;
  typename Tile::Own r, p, v, t, x, rh, u;
  typename Tile::Halo hr, hp, hv, ht, hu;
  typename Tile::HaloZ zr, zp, zv, zt, zu;
  const bool first0 = sh.sc.first != 0;
  tl.load_own(pick(a.r, par), r);
  tl.template load_halo<0>(pick(a.r, par), hr, zr);
  if (!first0) {
    tl.load_own(pick(a.p, par), p);
    tl.load_own(pick(a.v, par), v);
    tl.load_own(a.t, t);
    tl.template load_halo<0>(pick(a.p, par), hp, zp);
    tl.template load_halo<0>(pick(a.v, par), hv, zv);
    tl.template load_halo<0>(a.t, ht, zt);
  } else {
    WFA_OWN_CELLS(k, q) p[k][q] = v[k][q] = t[k][q] = T(0);
#pragma unroll
    for (int k = 0; k < Z; ++k) hp[k] = hv[k] = ht[k] = T(0);
    WFA_HALO_Z(e, q) zp[e][q] = zv[e][q] = zt[e][q] = T(0);
  }
  if (!sh.sc.x_zero) {
    tl.load_own(a.x, x);
  } else {
    WFA_OWN_CELLS(k, q) x[k][q] = T(0);
  }
  if (a.hashed) {
    WFA_OWN_CELLS(k, q) {
      rh[k][q] = tl.off[k][q] != kNowhere
                     ? hashed_shadow<T>((size_t)(tl.cell0[q] + k * tl.plane)) : T(0);
    }
  } else {
    tl.load_own(a.rh, rh);
  }

  bool ok = open_sets(a, tl, ring, tile, seq, sh.red, &sh.bad);
  Sets<T> sets{a.set[0], a.set[1], a.set[2]};
  for (int it = 0; ok && it < a.iters; ++it) {
    // ---- pass AC: the update of the iteration before, v' = A p'
    double s3[3] = {0.0, 0.0, 0.0};
    if (sh.sc.first) {
      WFA_OWN_CELLS(k, q) p[k][q] = r[k][q];
#pragma unroll
      for (int k = 0; k < Z; ++k) hp[k] = hr[k];
      WFA_HALO_Z(z, q) zp[z][q] = zr[z][q];
    } else {
      const T alpha = (T)sh.sc.alpha, omega = (T)sh.sc.omega, beta = (T)sh.sc.beta;
      WFA_OWN_CELLS(k, q) {
        const T s = minus_ax(r[k][q], alpha, v[k][q]);
        const T rn = minus_ax(s, omega, t[k][q]);
        x[k][q] = next_x(x[k][q], p[k][q], s, alpha, omega);
        p[k][q] = next_p(rn, p[k][q], v[k][q], beta, omega);
        r[k][q] = rn;
      }
      auto update = [&](T& r_, T& p_, T v_, T t_) {
        r_ = minus_ax(minus_ax(r_, alpha, v_), omega, t_);
        p_ = next_p(r_, p_, v_, beta, omega);
      };
#pragma unroll
      for (int k = 0; k < Z; ++k) update(hr[k], hp[k], hv[k], ht[k]);
      WFA_HALO_Z(z, q) update(zr[z][q], zp[z][q], zv[z][q], zt[z][q]);
    }
    par ^= 1;
    tl.apply(p, hp, zp, v);
    stores_done();
    tl.put_boundary(sets.cur, v);
    WFA_OWN_CELLS(k, q) {
      dot_acc(s3[0], (double)rh[k][q], (double)v[k][q]);
      dot_acc(s3[1], (double)rh[k][q], (double)r[k][q]);
      dot_acc(s3[2], (double)r[k][q], (double)r[k][q]);
    }
    ok = exchange<3>(s3, ring, tile, seq++, sh.red, &sh.bad, [&] {
      tl.template load_halo<kAgent>(sets.cur, hv, zv);
      return tl.halo_empty(hv, zv);
    });
    if (!ok) break;
    finalize<FinAC>(sh.sc, s3);
    if (!sets.fresh) tl.empty_boundary(sets.prev);
    sets.next();
    tl.store_own(pick(a.p, par), p);
    tl.store_own(pick(a.v, par), v);
    __syncthreads();
    if (sh.sc.status != ST_RUN || sh.sc.restart) break;

    // ---- pass B2: t = A s
    double s4[4] = {0.0, 0.0, 0.0, 0.0};
    {
      const T alpha = (T)sh.sc.alpha;
      WFA_OWN_CELLS(k, q) u[k][q] = minus_ax(r[k][q], alpha, v[k][q]);
#pragma unroll
      for (int k = 0; k < Z; ++k) hu[k] = minus_ax(hr[k], alpha, hv[k]);
      WFA_HALO_Z(z, q) zu[z][q] = minus_ax(zr[z][q], alpha, zv[z][q]);
    }
    tl.apply(u, hu, zu, t);
    stores_done();
    tl.put_boundary(sets.cur, t);
    WFA_OWN_CELLS(k, q) {
      dot_acc(s4[0], (double)t[k][q], (double)u[k][q]);
      dot_acc(s4[1], (double)t[k][q], (double)t[k][q]);
      dot_acc(s4[2], (double)rh[k][q], (double)u[k][q]);
      dot_acc(s4[3], (double)rh[k][q], (double)t[k][q]);
    }
    ok = exchange<4>(s4, ring, tile, seq++, sh.red, &sh.bad, [&] {
      tl.template load_halo<kAgent>(sets.cur, ht, zt);
      return tl.halo_empty(ht, zt);
    });
    if (!ok) break;
    finalize<FinB2>(sh.sc, s4);
    if (!sets.fresh) tl.empty_boundary(sets.prev);
    sets.next();
    __syncthreads();
    if (sh.sc.status != ST_RUN || sh.sc.restart) break;
  }
  // r and t live in the exchange vectors' memory: a neighbour still reading
  // halo cells of the last exchange leaves as this workgroup does, whatever
  // value it finds
  tl.store_own(pick(a.r, par), r);
  tl.store_own(a.t, t);
  if (!sh.sc.x_zero) tl.store_own(a.x, x);
  leave(sh, a.sc, tile == 0, seq);
}

// CG with one reduction per iteration (PhCg1): w = A r exchanged, one
// exchange an iteration.  a.v holds w, a.p holds s (double-buffered), a.t
// holds p.
template <typename T, bool CELL, int Z>
__global__ void __launch_bounds__(kThreads) k_resident_cg1(ResArgs<T> a) {
  using Tile = ResTile<T, CELL, Z>;
  __shared__ ResShared<T, CELL, Z> sh;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  if (threadIdx.x == 0) {
    sh.sc = *a.sc;
    sh.bad = 0;
  }
  __syncthreads();
  if (sh.sc.status != ST_RUN || sh.sc.restart) return;
  Tile tl(a.geo, a.op, sh, tile, a.kappa);
  const Ring ring(a.ring, a.copies, a.geo.ntiles);
  int par = a.parity;
  int seq = sh.sc.seq;
  typename Tile::Own r, w, s, p, x;
  typename Tile::Halo hr, hw, hs;
  typename Tile::HaloZ zr, zw, zs;
  int stage = sh.sc.stage;
  tl.load_own(pick(a.r, par), r);
  tl.template load_halo<0>(pick(a.r, par), hr, zr);
  if (stage > 0) {
    tl.load_own(pick(a.v, par), w);
    tl.template load_halo<0>(pick(a.v, par), hw, zw);
  } else {
    WFA_OWN_CELLS(k, q) w[k][q] = T(0);
#pragma unroll
    for (int k = 0; k < Z; ++k) hw[k] = T(0);
    WFA_HALO_Z(e, q) zw[e][q] = T(0);
  }
  if (stage > 1) {
    tl.load_own(pick(a.p, par), s);
    tl.template load_halo<0>(pick(a.p, par), hs, zs);
    tl.load_own(a.t, p);
  } else {
    WFA_OWN_CELLS(k, q) s[k][q] = p[k][q] = T(0);
#pragma unroll
    for (int k = 0; k < Z; ++k) hs[k] = T(0);
    WFA_HALO_Z(e, q) zs[e][q] = T(0);
  }
  if (!sh.sc.x_zero) {
    tl.load_own(a.x, x);
  } else {
    WFA_OWN_CELLS(k, q) x[k][q] = T(0);
  }

  bool ok = open_sets(a, tl, ring, tile, seq, sh.red, &sh.bad);
  Sets<T> sets{a.set[0], a.set[1], a.set[2]};
  for (int it = 0; ok && it < a.iters; ++it) {
    double s2[2] = {0.0, 0.0};
    stage = sh.sc.stage;
    if (stage != 0) {
      const T alpha = (T)sh.sc.alpha, beta = (T)sh.sc.beta;
      const bool start = stage == 1;   // p = r, s = w
      WFA_OWN_CELLS(k, q) {
        s[k][q] = start ? w[k][q] : fma_t(beta, s[k][q], w[k][q]);
        p[k][q] = start ? r[k][q] : fma_t(beta, p[k][q], r[k][q]);
        x[k][q] = fma_t(alpha, p[k][q], x[k][q]);
        r[k][q] = fma_t(-alpha, s[k][q], r[k][q]);
      }
      auto update = [&](T& r_, T w_, T& s_) {
        s_ = start ? w_ : fma_t(beta, s_, w_);
        r_ = fma_t(-alpha, s_, r_);
      };
#pragma unroll
      for (int k = 0; k < Z; ++k) update(hr[k], hw[k], hs[k]);
      WFA_HALO_Z(z, q) update(zr[z][q], zw[z][q], zs[z][q]);
    }
    par ^= 1;
    tl.apply(r, hr, zr, w);
    stores_done();
    tl.put_boundary(sets.cur, w);
    WFA_OWN_CELLS(k, q) {
      dot_acc(s2[0], (double)r[k][q], (double)r[k][q]);
      dot_acc(s2[1], (double)w[k][q], (double)r[k][q]);
    }
    ok = exchange<2>(s2, ring, tile, seq++, sh.red, &sh.bad, [&] {
      tl.template load_halo<kAgent>(sets.cur, hw, zw);
      return tl.halo_empty(hw, zw);
    });
    if (!ok) break;
    finalize<FinCg1>(sh.sc, s2);
    if (!sets.fresh) tl.empty_boundary(sets.prev);
    sets.next();
    tl.store_own(pick(a.r, par), r);
    tl.store_own(pick(a.v, par), w);
    __syncthreads();
    if (sh.sc.status != ST_RUN || sh.sc.restart) break;
  }
  if (stage != 0) {   // s and p: in the exchange vectors' memory, as above
    tl.store_own(pick(a.p, par), s);
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
  if (!L.tl.tile_order || g.ntiles > kResidentTiles) return false;
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
  if (kind == kResidentCg1) {
    a.set[0] = p[parity ^ 1]; a.set[1] = t; a.set[2] = p[parity];
  } else {
    a.set[0] = r[parity ^ 1]; a.set[1] = t; a.set[2] = r[parity];
  }
  a.ring = L.ring;
  a.copies = L.ring_copies;
  a.sc = L.sc;
  a.iters = iters;
  a.parity = parity;
  a.hashed = L.shadow;
  void* args[] = {(void*)&a};
  return hipLaunchCooperativeKernel((const void*)entry_for<T>(L, kind).kernel, dim3(a.geo.ntiles),
                                    dim3(kThreads), args, 0, L.stream);
}

// The solve's scalars, with every slot of the ring empty.
__global__ void __launch_bounds__(1024)
k_set_resident(Scalars* __restrict__ dst, Scalars v, uint64_t* __restrict__ ring, int slots) {
  if (threadIdx.x == 0) *dst = v;
  for (int e = threadIdx.x; e < slots; e += 1024) ring[e] = Empty<double>::value;
}

void launch_set_resident(Scalars* dst, const Scalars& v, double* ring, int copies, int ntiles,
                         hipStream_t s) {
  hipLaunchKernelGGL(k_set_resident, dim3(1), dim3(1024), 0, s, dst, v, (uint64_t*)ring,
                     copies * kRing * kMaxReduce * ntiles);
}

// Copies of the ring that fit in `doubles` (a power of two, one per XCD at most).
int ring_copies(size_t doubles, int ntiles) {
  int c = 8;
  while (c > 1 && (size_t)c * kRing * kMaxReduce * ntiles > doubles) c /= 2;
  return c;
}

#define WFA_RES(T)                                                                             \
  template bool resident_fits<T>(const Launch<T>&, int);                                      \
  template hipError_t launch_resident<T>(const Launch<T>&, int, T*, T* const (&)[2], const T*, \
                                         T* const (&)[2], T* const (&)[2], T*, int, int);
WFA_RES(float)
WFA_RES(double)
#undef WFA_RES

}  // namespace wfa
