// Resident Krylov iterations of small grids: one launch runs a
// whole chunk of iterations of one solve with its vectors held in registers.
//
// A small grid's iteration is latency, not traffic: at 32^3 each pass was a
// launch of 8-11 us, of which the 64 workgroups spent most in dependent trips
// to memory (plane loads, partial store, arrival counter, the last
// workgroup's reduction) and the kernel boundary.  Here every workgroup keeps
// one tile -- the tile a per-pass launch gives it -- with the solve's vectors
// in registers from the first iteration of the chunk to the last, and a
// reduction costs one exchange between the workgroups:
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
// The launch is an ordinary one.  Cooperative launches of a process pass
// through one queue, so that solves of several threads took turns, and waited
// for the streams' queues at each change.  Small heat steps a second from 1, 4
// and 16 threads, one launch per pass / resident, cooperative / ordinary with
// turns: 16^3 CG with one reduction 3046, 6309, 10027 / 7451, 10640, 8840 /
// 8670, 19050, 19090; 32^3 BiCGStab 1249, 4237, 4461 / 3560, 4380, 4060 / 3850,
// 11320, 5450; 64^3 refined 509, 1494, 1349 / 1310, 1630, 1340 / 1460, 2470, 1880.
//
// Measured (us an iteration, one launch per pass -> resident; FP64 constant
// diffusivity, then FP32 per cell):
//   textbook BiCGStab       32^3 24.8 -> 6.6   64^3 32.7 -> 10.9
//                           57x82x90 50.2 -> 13.5   128^3 91.8 -> 45.3
//   two-reduction BiCGStab  32^3 19.9 -> 6.2   64^3 26.3 -> 9.7
//                           57x82x90 38.6 -> 12.4   128^3 63.3 -> 42.7
//   classic CG              32^3 14.3 -> 3.9   64^3 18.4 -> 5.6
//                           57x82x90 24.9 -> 7.0    128^3 41.2 -> 18.7
//   CG with one reduction   32^3 10.5 -> 3.0   64^3 14.7 -> 4.9
//                           57x82x90 23.4 -> 5.8    128^3 47.1 -> 16.9
// (Two-reduction 32^3 and 64^3: 6.6 / 10.6 with one copy of the slots, 8.9 /
// 15.1 where a pass moreover waited for its stores before it published its
// sums and branched around the cells outside the grid.)
//
// Tiles, per-thread order of the dot products, reduction order and
// finalizers are those of the per-pass kernels, so the iterates are bitwise
// theirs.
//
// A wait needs every workgroup of the launch on a CU.  The launches of one
// process see to that among themselves (ResidentTurn), but other kernels may
// prevent it for as long as they like; waits are therefore bounded.  A
// workgroup that gives up sets the scalar block's `timeout` and leaves, and so
// does every other at its next wait, each with x as it has it; the solve goes
// on from that x with one launch per pass.  Once the launch's first exchange
// has passed, every workgroup holds its CU and later waits end.
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
// Polls of one wait: 0.07 s (measured, on 16 to 256 tiles), well under a
// persistent launch's: of two that keep each other out the resident one gives up.
constexpr int kSpinLimit = 1 << 19;

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
// off: the lane's byte offset; soff: one of the whole workgroup, added to it.
template <typename V, int AUX>
__device__ __forceinline__ V buf_load(Rsrc r, int off, int soff = 0) {
  if constexpr (sizeof(V) == 8)
    return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, AUX));
  else
    return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b32(r, off, soff, AUX));
}
template <int AUX, typename V>
__device__ __forceinline__ void buf_store(Rsrc r, int off, V v, int soff = 0) {
  if constexpr (sizeof(V) == 8) {
    using B = decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0, 0, 0));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(B, v), r, off, soff, AUX);
  } else {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, off, soff, AUX);
  }
}
// Exchanged values: stored past the caches, the empty one never among them.
template <typename T>
__device__ __forceinline__ void put_value(Rsrc r, int off, T v, int soff = 0) {
  using E = Empty<T>;
  const auto bits = __builtin_bit_cast(typename E::Bits, v);
  buf_store<kAgent>(r, off, bits == E::value ? E::nan : bits, soff);
}
template <typename T>
__device__ __forceinline__ void put_empty(Rsrc r, int off, int soff = 0) {
  buf_store<kAgent>(r, off, Empty<T>::value, soff);
}
template <typename T>
__device__ __forceinline__ bool is_empty(T v) {
  return __builtin_bit_cast(typename Empty<T>::Bits, v) == Empty<T>::value;
}

template <typename T>
__device__ __forceinline__ T* pick(T* const (&pair)[2], int par) {
  return par ? pair[1] : pair[0];
}

// A Krylov vector on a tile: the own cells of a thread (2 rows of up to Z
// planes), the x-y halo cell it keeps of each plane, and the z-halo cells
// below and above its rows.
template <typename T, int Z>
struct Cells {
  T o[Z][2];
  T h[Z];
  T z[2][2];
  __device__ void clear() {
#pragma unroll
    for (int k = 0; k < Z; ++k) o[k][0] = o[k][1] = h[k] = T(0);
    z[0][0] = z[0][1] = z[1][0] = z[1][1] = T(0);
  }
};
// f on the corresponding cells of some vectors: own cells, all, halo cells.
template <int Z, class F, class... C>
__device__ __forceinline__ void each_own(F f, C&... c) {
#pragma unroll
  for (int k = 0; k < Z; ++k)
#pragma unroll
    for (int r = 0; r < 2; ++r) f(c.o[k][r]...);
}
template <int Z, class F, class... C>
__device__ __forceinline__ void each_halo(F f, C&... c) {
#pragma unroll
  for (int k = 0; k < Z; ++k) f(c.h[k]...);
#pragma unroll
  for (int e = 0; e < 2; ++e)
#pragma unroll
    for (int r = 0; r < 2; ++r) f(c.z[e][r]...);
}

// How a workgroup keeps the operator of a per-cell diffusivity in LDS: its
// rows (the six couplings and the diagonal of each own cell) where they fit,
// else the faces' harmonic means, shared by the two cells of a face.
enum Rows : int { kRowsConst, kRowsFull, kRowsFaces };
template <typename T, bool CELL, int Z>
constexpr Rows rows_of() {
  return !CELL ? kRowsConst
               : (size_t)7 * 2 * Z * kThreads * sizeof(T) <= 120 * 1024 ? kRowsFull : kRowsFaces;
}
template <typename T, int Z, Rows R>
struct OperatorStore {};
template <typename T, int Z>
struct OperatorStore<T, Z, kRowsFull> {
  T coef[7][Z * 2][kThreads];
};
template <typename T, int Z>
struct OperatorStore<T, Z, kRowsFaces> {
  // slot of the face below the cell of that index on its axis
  T x[Z][2 * kWaves][kTX + 1], y[Z][2 * kWaves + 1][kTX], z[Z + 1][2 * kWaves][kTX];
};

// What one workgroup shares in LDS.
template <typename T, bool CELL, int Z>
struct ResShared {
  using TS = TileShape<2>;
  static constexpr int kPlane = TS::LH * TS::LW + 2;   // the last slot: threads without a halo cell
  T u[Z][kPlane];                                      // staged vector, with its x-y halo
  OperatorStore<T, Z, rows_of<T, CELL, Z>()> op;
  double red[2][kWaves * kMaxReduce];
  Scalars sc;
  int bad;
};

// One tile as a thread sees it.
template <typename T, bool CELL, int Z>
struct ResTile {
  using TS = TileShape<2>;
  static constexpr int LW = TS::LW, LH = TS::LH, TY = TS::TY;
  static constexpr int RY = 2, W = sizeof(T);
  static constexpr Rows R = rows_of<T, CELL, Z>();
  using C = Cells<T, Z>;
  const Op<T>& op;
  ResShared<T, CELL, Z>& sh;
  size_t bytes;                  // of one vector
  int row_off[RY], edge_off[RY]; // byte offsets on the first plane: the own cells, those that
  int halo_off, zoff[2][RY];     // a tile beside reads, the halo cell; of the z-halo cells
  int step;                      // bytes of a plane
  int cell0[RY];                 // index of the own cells of the first plane
  int lidx[RY], hl;
  int nzt;                       // planes of this tile
  bool zlo, zhi;                 // the z neighbours exist
  uint32_t ins[RY];              // x and y faces inside
  T diag[R == kRowsConst ? Z : 1][RY];   // constant diffusivity: the diagonal

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
    zlo = k0 > 0;
    zhi = k0 + nzt < g.nz;
    const int i = x0 + lane, nx = g.nx, ny = g.ny;
    const int plane = (int)g.plane;
    step = plane * W;
    bytes = (size_t)g.plane * g.nz * W;
    const int base = k0 * plane;
#pragma unroll
    for (int r = 0; r < RY; ++r) {
      const int j = y0 + wave * RY + r;
      const bool own = i < nx && j < ny;
      cell0[r] = base + (own ? i + nx * j : 0);
      lidx[r] = (wave * RY + r + 1) * LW + lane + 1;
      ins[r] = (i > 0 ? 1u : 0u) | (i < nx - 1 ? 2u : 0u) | (j > 0 ? 4u : 0u) |
               (j < ny - 1 ? 8u : 0u);
      const bool edge = (lane == 0 && x0 > 0) || (lane == kTX - 1 && i < nx - 1) ||
                        (j == y0 && y0 > 0) || (j == y0 + TY - 1 && j < ny - 1);
      row_off[r] = own ? cell0[r] * W : kNowhere;
      edge_off[r] = edge ? row_off[r] : kNowhere;
      zoff[0][r] = own && zlo ? (cell0[r] - plane) * W : kNowhere;
      zoff[1][r] = own && zhi ? (cell0[r] + nzt * plane) * W : kNowhere;
    }
    const int hs = threadIdx.x;
    int hi = -1, hj = 0;
    hl = LH * LW;
    if (hs < kTX) { hi = x0 + hs; hj = y0 - 1; hl = hs + 1; }
    else if (hs < 2 * kTX) { hi = x0 + hs - kTX; hj = y0 + TY; hl = (LH - 1) * LW + hs - kTX + 1; }
    else if (hs < 2 * kTX + TY) { hi = x0 - 1; hj = y0 + hs - 2 * kTX; hl = (hs - 2 * kTX + 1) * LW; }
    else if (hs < TS::NHALO) { hi = x0 + kTX; hj = y0 + hs - 2 * kTX - TY; hl = (hs - 2 * kTX - TY + 1) * LW + LW - 1; }
    const bool hval = hi >= 0 && hi < nx && hj >= 0 && hj < ny;
    halo_off = hval ? (base + hi + nx * hj) * W : kNowhere;
    operator_rows(kappa);
  }

  // Offset of plane k for all lanes, and a lane's: past the end where the tile
  // has no such plane (the scalar offset stays inside the vector: the bounds
  // check subtracts it from the vector's size).
  __device__ int plane_off(int k) const { return k < nzt ? k * step : 0; }
  __device__ int lane_off(int off, int k) const { return k < nzt ? off : kNowhere; }
  __device__ bool own(int k, int r) const { return k < nzt && row_off[r] != kNowhere; }
  __device__ uint32_t inside(int k, int r) const {
    return ins[r] | (k > 0 || zlo ? 16u : 0u) | (k < nzt - 1 || zhi ? 32u : 0u);
  }

  // The operator's row of an own cell: the couplings D of the six faces (0
  // where there is no neighbour) and the diagonal, formed as cell_apply forms
  // them from the faces' harmonic means kf (a Dirichlet face: the cell's own
  // diffusivity).
  __device__ T row(uint32_t in, const T (&kf)[6], T (&D)[6]) const {
#pragma clang fp contract(off)
    T dg = T(1);
#pragma unroll
    for (int f = 0; f < 6; ++f) {
      const T out = CELL ? fma_t(op.cD, kf[f], op.out[f]) : op.cD + op.out[f];
      const T inn = CELL ? fma_t(op.cD, kf[f], op.in[f]) : op.cD + op.in[f];
      if ((in | op.dir) & (1u << f)) dg += out;
      D[f] = in & (1u << f) ? inn : T(0);
    }
    return dg;
  }
  __device__ void operator_rows(const float* __restrict__ kappa) {
    if constexpr (R == kRowsConst) {
      const T none[6] = {};
      T D[6];
#pragma unroll
      for (int k = 0; k < Z; ++k)
#pragma unroll
        for (int r = 0; r < RY; ++r) diag[k][r] = row(inside(k, r), none, D);
    } else {
      const Rsrc kr = rsrc(kappa, bytes / W * 4);
      auto ld = [&](int off, int soff) {
        const float v = buf_load<float, 0>(kr, off == kNowhere ? kNowhere : off / W * 4, soff / W * 4);
        return off == kNowhere ? 1.f : v;
      };
      float kc[Z][RY], kz[2][RY];
      float* Lk = (float*)&sh.u[0][0];   // the diffusivity in the staged vector's place
      constexpr int LP = ResShared<T, CELL, Z>::kPlane;
#pragma unroll
      for (int k = 0; k < Z; ++k) {
        const int so = k < nzt ? k * step : 0;   // (planes past the tile's are not used)
#pragma unroll
        for (int r = 0; r < RY; ++r) {
          kc[k][r] = ld(row_off[r], so);
          Lk[k * LP + lidx[r]] = kc[k][r];
        }
        Lk[k * LP + hl] = ld(halo_off, so);
      }
#pragma unroll
      for (int r = 0; r < RY; ++r)
#pragma unroll
        for (int e = 0; e < 2; ++e) kz[e][r] = ld(zoff[e][r], 0);
      __syncthreads();
      const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
      for (int k = 0; k < Z; ++k)
#pragma unroll
        for (int r = 0; r < RY; ++r) {
          const float* L = Lk + k * LP + lidx[r];
          const float lo = k > 0 ? kc[k > 0 ? k - 1 : 0][r] : kz[0][r];
          const float hi = k + 1 >= nzt ? kz[1][r] : kc[k + 1 < Z ? k + 1 : k][r];
          const T kP = (T)kc[k][r];
          const T kN[6] = {(T)L[-1], (T)L[1], (T)L[-LW], (T)L[LW], (T)lo, (T)hi};
          const uint32_t in = inside(k, r);
          T kf[6];
#pragma unroll
          for (int f = 0; f < 6; ++f)
            kf[f] = in & (1u << f) ? T(2) * kP * kN[f] * pos_rcp(kP + kN[f]) : kP;
          if constexpr (R == kRowsFull) {
            T D[6];
            const T dg = row(in, kf, D);
#pragma unroll
            for (int f = 0; f < 6; ++f) sh.op.coef[f][k * RY + r][threadIdx.x] = D[f];
            sh.op.coef[6][k * RY + r][threadIdx.x] = dg;
          } else if (own(k, r)) {
            const int j = wave * RY + r;
            sh.op.x[k][j][lane] = kf[0];
            sh.op.x[k][j][lane + 1] = kf[1];
            sh.op.y[k][j][lane] = kf[2];
            sh.op.y[k][j + 1][lane] = kf[3];
            sh.op.z[k][j][lane] = kf[4];
            sh.op.z[k + 1][j][lane] = kf[5];
          }
        }
      __syncthreads();
    }
  }
  __device__ T own_row(int k, int r, T (&D)[6]) const {
    if constexpr (R == kRowsConst) {
      const uint32_t in = inside(k, r);
#pragma unroll
      for (int f = 0; f < 6; ++f) D[f] = in & (1u << f) ? op.cD + op.in[f] : T(0);
      return diag[k][r];
    } else if constexpr (R == kRowsFull) {
#pragma unroll
      for (int f = 0; f < 6; ++f) D[f] = sh.op.coef[f][k * RY + r][threadIdx.x];
      return sh.op.coef[6][k * RY + r][threadIdx.x];
    } else {
      const int lane = threadIdx.x & 63, j = (threadIdx.x >> 6) * RY + r;
      const T kf[6] = {sh.op.x[k][j][lane], sh.op.x[k][j][lane + 1], sh.op.y[k][j][lane],
                       sh.op.y[k][j + 1][lane], sh.op.z[k][j][lane], sh.op.z[k + 1][j][lane]};
      return row(inside(k, r), kf, D);
    }
  }

  __device__ Rsrc vec(const T* a) const { return rsrc(a, bytes); }
  __device__ void load_own(const T* a, C& c) const {
    const Rsrc b = vec(a);
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int r = 0; r < RY; ++r)
        c.o[k][r] = buf_load<T, 0>(b, lane_off(row_off[r], k), plane_off(k));
  }
  template <int AUX>
  __device__ void load_halo(const T* a, C& c) const {
    const Rsrc b = vec(a);
#pragma unroll
    for (int k = 0; k < Z; ++k)
      c.h[k] = buf_load<T, AUX>(b, lane_off(halo_off, k), plane_off(k));
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int r = 0; r < RY; ++r) c.z[e][r] = buf_load<T, AUX>(b, zoff[e][r]);
  }
  __device__ void load(const T* a, C& c) const {
    load_own(a, c);
    load_halo<0>(a, c);
  }
  // Loads the halo cells of an exchange vector; true while one is empty.
  __device__ bool poll(const T* a, C& c) const {
    load_halo<kAgent>(a, c);
    bool none = false;
    each_halo<Z>([&](T v) { none = none | is_empty(v); }, c);
    return none;
  }
  __device__ void store_own(T* a, const C& c) const {
    const Rsrc b = vec(a);
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int r = 0; r < RY; ++r)
        buf_store<0>(b, lane_off(row_off[r], k), c.o[k][r], plane_off(k));
  }
  // lane offset of the own cell of plane k, row r, if another tile reads it
  __device__ int boundary_off(int k, int r) const {
    const bool face = (k == 0 && zlo) || (k == nzt - 1 && zhi);
    return lane_off(face ? row_off[r] : edge_off[r], k);
  }
  __device__ void put_boundary(T* a, const C& c) const {
    const Rsrc b = vec(a);
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int r = 0; r < RY; ++r) put_value(b, boundary_off(k, r), c.o[k][r], plane_off(k));
  }
  __device__ void empty_boundary(T* a) const {
    const Rsrc b = vec(a);
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int r = 0; r < RY; ++r) put_empty<T>(b, boundary_off(k, r), plane_off(k));
  }

  // Au.o = A u of the own cells (0 elsewhere), u staged with its halo.
  __device__ void apply(const C& u, C& Au) {
#pragma clang fp contract(off)
#pragma unroll
    for (int k = 0; k < Z; ++k) {
#pragma unroll
      for (int r = 0; r < RY; ++r) sh.u[k][lidx[r]] = u.o[k][r];
      sh.u[k][hl] = u.h[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int r = 0; r < RY; ++r) {
        const T* L = &sh.u[k][lidx[r]];
        const T lo = k > 0 ? u.o[k > 0 ? k - 1 : 0][r] : u.z[0][r];
        const T hi = k + 1 >= nzt ? u.z[1][r] : u.o[k + 1 < Z ? k + 1 : k][r];
        const T nb[6] = {L[-1], L[1], L[-LW], L[LW], lo, hi};
        T D[6];
        const T dg = own_row(k, r, D);
        T y = apply_coefs(D, dg, u.o[k][r], nb);
        if (op.jac) y = y * pos_rcp(dg);
        Au.o[k][r] = own(k, r) ? y : T(0);
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

// What every resident kernel begins with.
#define WFA_RESIDENT_BEGIN                                           \
  using Tile = ResTile<T, CELL, Z>;                                  \
  using C = Cells<T, Z>;                                             \
  __shared__ ResShared<T, CELL, Z> sh;                               \
  const int tile = xcd_tile(blockIdx.x, gridDim.x);                  \
  if (threadIdx.x == 0) {                                            \
    sh.sc = *a.sc;                                                   \
    sh.bad = 0;                                                      \
  }                                                                  \
  __syncthreads();                                                   \
  if (sh.sc.status != ST_RUN || sh.sc.restart) return;               \
  Tile tl(a.geo, a.op, sh, tile, a.kappa);                           \
  const Ring ring(a.ring, a.copies, a.geo.ntiles);                   \
  Sets<T> sets{a.set[0], a.set[1], a.set[2]};                        \
  int par = a.parity, seq = sh.sc.seq;                               \
  bool ok

// One exchange of w's boundary cells and the sums s, with the finalizer;
// false when the solve leaves the loop.  `more` runs behind the finalizer
// (stores nobody waits for).
template <class Fin, typename T, class Tile, class C, int NV, class Sh, class More>
__device__ __forceinline__ bool exchange_cells(const Tile& tl, Sets<T>& sets, const Ring& ring,
                                               Sh& sh, int tile, int& seq, C& w, double (&s)[NV],
                                               bool& ok, More more) {
  ok = exchange<NV>(s, ring, tile, seq++, sh.red, &sh.bad, [&] { return tl.poll(sets.cur, w); });
  if (!ok) return false;
  finalize<Fin>(sh.sc, s);
  if (!sets.fresh) tl.empty_boundary(sets.prev);
  sets.next();
  more();
  __syncthreads();
  return sh.sc.status == ST_RUN && !sh.sc.restart;
}

// Textbook BiCGStab: passes A, B and C (PhA, PhB, phase_c_tile).
template <typename T, bool CELL, int Z>
__global__ void __launch_bounds__(kThreads) k_resident_bicgstab(ResArgs<T> a) {
  WFA_RESIDENT_BEGIN;
  C r, p, v, t, x, rh, u;
  tl.load(a.r[0], r);
  if (sh.sc.first) {
    p.clear();
    v.clear();
  } else {
    tl.load(pick(a.p, par), p);
    tl.load(pick(a.v, par), v);
  }
  if (sh.sc.x_zero) x.clear();
  else tl.load_own(a.x, x);
  tl.load_own(a.rh, rh);
  ok = open_sets(a, tl, ring, tile, seq, sh.red, &sh.bad);
  for (int it = 0; ok && it < a.iters; ++it) {
    // ---- A: p' = r + beta (p - omega v), v' = A p'
    double s1[1] = {0.0};
    if (sh.sc.first) {
      auto copy = [](T r_, T& p_) { p_ = r_; };
      each_own<Z>(copy, r, p);
      each_halo<Z>(copy, r, p);
    } else {
      const T beta = (T)sh.sc.beta, omega = (T)sh.sc.omega;
      auto next = [&](T r_, T& p_, T v_) { p_ = next_p(r_, p_, v_, beta, omega); };
      each_own<Z>(next, r, p, v);
      each_halo<Z>(next, r, p, v);
    }
    par ^= 1;
    tl.apply(p, v);
    stores_done();
    tl.put_boundary(sets.cur, v);
    each_own<Z>([&](T h, T w) { dot_acc(s1[0], (double)h, (double)w); }, rh, v);
    if (!exchange_cells<FinA>(tl, sets, ring, sh, tile, seq, v, s1, ok, [&] {
          tl.store_own(pick(a.p, par), p);
          tl.store_own(pick(a.v, par), v);
        }))
      break;

    // ---- B: s = r - alpha v', t = A s
    double s2[2] = {0.0, 0.0};
    {
      const T alpha = (T)sh.sc.alpha;
      auto stage = [&](T r_, T v_, T& u_) { u_ = minus_ax(r_, alpha, v_); };
      each_own<Z>(stage, r, v, u);
      each_halo<Z>(stage, r, v, u);
    }
    tl.apply(u, t);
    stores_done();
    tl.put_boundary(sets.cur, t);
    each_own<Z>([&](T t_, T u_) {
      dot_acc(s2[0], (double)t_, (double)u_);
      dot_acc(s2[1], (double)t_, (double)t_);
    }, t, u);
    if (!exchange_cells<FinB>(tl, sets, ring, sh, tile, seq, t, s2, ok, [] {})) break;

    // ---- C: x += alpha p' + omega s, r = s - omega t
    double s3[2] = {0.0, 0.0};
    {
      const T alpha = (T)sh.sc.alpha, omega = (T)sh.sc.omega;
      each_own<Z>([&](T& r_, T p_, T u_, T t_, T& x_, T h) {
        x_ = next_x(x_, p_, u_, alpha, omega);
        r_ = minus_ax(u_, omega, t_);
        dot_acc(s3[0], (double)h, (double)r_);
        dot_acc(s3[1], (double)r_, (double)r_);
      }, r, p, u, t, x, rh);
      each_halo<Z>([&](T& r_, T u_, T t_) { r_ = minus_ax(u_, omega, t_); }, r, u, t);
    }
    stores_done();
    ok = exchange<2>(s3, ring, tile, seq++, sh.red, &sh.bad, [] { return false; });
    if (!ok) break;
    finalize<FinC>(sh.sc, s3);
    __syncthreads();
    if (sh.sc.status != ST_RUN || sh.sc.restart) break;
  }
  // r and t live in the exchange vectors' memory: a neighbour still reading
  // halo cells of the last exchange leaves as this workgroup does, whatever
  // value it finds
  tl.store_own(a.r[0], r);
  if (!sh.sc.x_zero) tl.store_own(a.x, x);
  leave(sh, a.sc, tile == 0, seq);
}

// Two-reduction BiCGStab: passes AC and B2 (PhAC, PhB2).
template <typename T, bool CELL, int Z>
__global__ void __launch_bounds__(kThreads) k_resident_bicgstab2(ResArgs<T> a) {
  WFA_RESIDENT_BEGIN;
  C r, p, v, t, x, rh, u;
  tl.load(pick(a.r, par), r);
  if (sh.sc.first) {
    p.clear();
    v.clear();
    t.clear();
  } else {
    tl.load(pick(a.p, par), p);
    tl.load(pick(a.v, par), v);
    tl.load(a.t, t);
  }
  if (sh.sc.x_zero) x.clear();
  else tl.load_own(a.x, x);
  if (a.hashed) {
#pragma unroll
    for (int k = 0; k < Z; ++k)
#pragma unroll
      for (int q = 0; q < 2; ++q)
        rh.o[k][q] = tl.own(k, q) ? hashed_shadow<T>((size_t)(tl.cell0[q] + k * (int)a.geo.plane)) : T(0);
  } else {
    tl.load_own(a.rh, rh);
  }
  ok = open_sets(a, tl, ring, tile, seq, sh.red, &sh.bad);
  for (int it = 0; ok && it < a.iters; ++it) {
    // ---- pass AC: the update of the iteration before, v' = A p'
    double s3[3] = {0.0, 0.0, 0.0};
    if (sh.sc.first) {
      auto copy = [](T r_, T& p_) { p_ = r_; };
      each_own<Z>(copy, r, p);
      each_halo<Z>(copy, r, p);
    } else {
      const T alpha = (T)sh.sc.alpha, omega = (T)sh.sc.omega, beta = (T)sh.sc.beta;
      each_own<Z>([&](T& r_, T& p_, T v_, T t_, T& x_) {
        const T s = minus_ax(r_, alpha, v_);
        r_ = minus_ax(s, omega, t_);
        x_ = next_x(x_, p_, s, alpha, omega);
        p_ = next_p(r_, p_, v_, beta, omega);
      }, r, p, v, t, x);
      each_halo<Z>([&](T& r_, T& p_, T v_, T t_) {
        r_ = minus_ax(minus_ax(r_, alpha, v_), omega, t_);
        p_ = next_p(r_, p_, v_, beta, omega);
      }, r, p, v, t);
    }
    par ^= 1;
    tl.apply(p, v);
    stores_done();
    tl.put_boundary(sets.cur, v);
    each_own<Z>([&](T h, T v_, T r_) {
      dot_acc(s3[0], (double)h, (double)v_);
      dot_acc(s3[1], (double)h, (double)r_);
      dot_acc(s3[2], (double)r_, (double)r_);
    }, rh, v, r);
    if (!exchange_cells<FinAC>(tl, sets, ring, sh, tile, seq, v, s3, ok, [&] {
          tl.store_own(pick(a.p, par), p);
          tl.store_own(pick(a.v, par), v);
        }))
      break;

    // ---- pass B2: t = A s
    double s4[4] = {0.0, 0.0, 0.0, 0.0};
    {
      const T alpha = (T)sh.sc.alpha;
      auto stage = [&](T r_, T v_, T& u_) { u_ = minus_ax(r_, alpha, v_); };
      each_own<Z>(stage, r, v, u);
      each_halo<Z>(stage, r, v, u);
    }
    tl.apply(u, t);
    stores_done();
    tl.put_boundary(sets.cur, t);
    each_own<Z>([&](T t_, T u_, T h) {
      dot_acc(s4[0], (double)t_, (double)u_);
      dot_acc(s4[1], (double)t_, (double)t_);
      dot_acc(s4[2], (double)h, (double)u_);
      dot_acc(s4[3], (double)h, (double)t_);
    }, t, u, rh);
    if (!exchange_cells<FinB2>(tl, sets, ring, sh, tile, seq, t, s4, ok, [] {})) break;
  }
  // in the exchange vectors' memory, as in k_resident_bicgstab
  tl.store_own(pick(a.r, par), r);
  tl.store_own(a.t, t);
  if (!sh.sc.x_zero) tl.store_own(a.x, x);
  leave(sh, a.sc, tile == 0, seq);
}

// Classic CG: passes A and B (PhCgA, cg_b_tile).  a.p holds the directions.
template <typename T, bool CELL, int Z>
__global__ void __launch_bounds__(kThreads) k_resident_cg(ResArgs<T> a) {
  WFA_RESIDENT_BEGIN;
  C r, d, q, x;
  tl.load(a.r[0], r);
  if (sh.sc.first) d.clear();
  else tl.load(pick(a.p, par), d);
  tl.load_own(a.x, x);
  ok = open_sets(a, tl, ring, tile, seq, sh.red, &sh.bad);
  for (int it = 0; ok && it < a.iters; ++it) {
    // ---- A: d' = r + beta d, q = A d'
    double s1[1] = {0.0};
    {
      const T beta = (T)sh.sc.beta;
      const bool first = sh.sc.first;
      auto next = [&](T r_, T& d_) { d_ = first ? r_ : fma_t(beta, d_, r_); };
      each_own<Z>(next, r, d);
      each_halo<Z>(next, r, d);
    }
    par ^= 1;
    tl.apply(d, q);
    stores_done();
    tl.put_boundary(sets.cur, q);
    each_own<Z>([&](T d_, T q_) { dot_acc(s1[0], (double)d_, (double)q_); }, d, q);
    if (!exchange_cells<FinCgA>(tl, sets, ring, sh, tile, seq, q, s1, ok, [] {})) break;

    // ---- B: x += alpha d', r -= alpha q
    double s2[1] = {0.0};
    {
      const T alpha = (T)sh.sc.alpha;
      each_own<Z>([&](T& x_, T d_, T& r_, T q_) { cg_b_elem<T>(x_, d_, r_, q_, alpha, s2); },
                  x, d, r, q);
      each_halo<Z>([&](T& r_, T q_) { r_ = minus_ax(r_, alpha, q_); }, r, q);
    }
    stores_done();
    ok = exchange<1>(s2, ring, tile, seq++, sh.red, &sh.bad, [] { return false; });
    if (!ok) break;
    finalize<FinCgB>(sh.sc, s2);
    __syncthreads();
    if (sh.sc.status != ST_RUN) break;
  }
  tl.store_own(a.r[0], r);
  tl.store_own(pick(a.p, par), d);
  tl.store_own(a.x, x);
  leave(sh, a.sc, tile == 0, seq);
}

// CG with one reduction per iteration (PhCg1): w = A r exchanged, one
// exchange an iteration.  a.v holds w, a.p holds s (double-buffered), a.t
// holds p.
template <typename T, bool CELL, int Z>
__global__ void __launch_bounds__(kThreads) k_resident_cg1(ResArgs<T> a) {
  WFA_RESIDENT_BEGIN;
  C r, w, s, p, x;
  int stage = sh.sc.stage;
  tl.load(pick(a.r, par), r);
  if (stage > 0) tl.load(pick(a.v, par), w);
  else w.clear();
  if (stage > 1) {
    tl.load(pick(a.p, par), s);
    tl.load_own(a.t, p);
  } else {
    s.clear();
    p.clear();
  }
  if (sh.sc.x_zero) x.clear();
  else tl.load_own(a.x, x);
  ok = open_sets(a, tl, ring, tile, seq, sh.red, &sh.bad);
  for (int it = 0; ok && it < a.iters; ++it) {
    double s2[2] = {0.0, 0.0};
    stage = sh.sc.stage;
    if (stage != 0) {
      const T alpha = (T)sh.sc.alpha, beta = (T)sh.sc.beta;
      const bool start = stage == 1;   // p = r, s = w
      each_own<Z>([&](T& r_, T w_, T& s_, T& p_, T& x_) {
        s_ = start ? w_ : fma_t(beta, s_, w_);
        p_ = start ? r_ : fma_t(beta, p_, r_);
        x_ = fma_t(alpha, p_, x_);
        r_ = fma_t(-alpha, s_, r_);
      }, r, w, s, p, x);
      each_halo<Z>([&](T& r_, T w_, T& s_) {
        s_ = start ? w_ : fma_t(beta, s_, w_);
        r_ = fma_t(-alpha, s_, r_);
      }, r, w, s);
    }
    par ^= 1;
    tl.apply(r, w);
    stores_done();
    tl.put_boundary(sets.cur, w);
    each_own<Z>([&](T r_, T w_) {
      dot_acc(s2[0], (double)r_, (double)r_);
      dot_acc(s2[1], (double)w_, (double)r_);
    }, r, w);
    if (!exchange_cells<FinCg1>(tl, sets, ring, sh, tile, seq, w, s2, ok, [&] {
          tl.store_own(pick(a.r, par), r);
          tl.store_own(pick(a.v, par), w);
        }))
      break;
  }
  if (stage != 0) {   // s and p: in the exchange vectors' memory, as above
    tl.store_own(pick(a.p, par), s);
    tl.store_own(a.t, p);
    tl.store_own(a.x, x);
  }
  leave(sh, a.sc, tile == 0, seq);
}
#undef WFA_RESIDENT_BEGIN

// The current device and its CUs (looked up once), or false.
constexpr int kDevices = 16;
bool this_device(int& dev, int& cus) {
  static std::atomic<int> known[kDevices];
  dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevices) return false;
  cus = known[dev].load(std::memory_order_relaxed);
  if (cus > 0) return true;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus < 1)
    return false;
  known[dev].store(cus, std::memory_order_relaxed);
  return true;
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
  static std::atomic<int> known[kDevices];
  int dev, cus;
  if (!this_device(dev, cus)) return {};
  int fit = known[dev].load(std::memory_order_relaxed);
  if (fit == 0) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)K, kThreads, 0) !=
        hipSuccess)
      return {};
    fit = per_cu * cus;
    known[dev].store(fit, std::memory_order_relaxed);
  }
  return {K, fit};
}

template <typename T, bool CELL, int Z>
Entry<T> entry_of(int kind) {
  switch (kind) {
    case kResidentBicgstab: return entry<T, k_resident_bicgstab<T, CELL, Z>>();
    case kResidentBicgstab2: return entry<T, k_resident_bicgstab2<T, CELL, Z>>();
    case kResidentCg: return entry<T, k_resident_cg<T, CELL, Z>>();
    default: return entry<T, k_resident_cg1<T, CELL, Z>>();
  }
}

template <typename T>
Entry<T> entry_for(const Launch<T>& L, int kind) {
  const int zc = L.tl.geo.zc;
  if (zc <= 2) return L.cell ? entry_of<T, true, 2>(kind) : entry_of<T, false, 2>(kind);
  if (zc <= 4) return L.cell ? entry_of<T, true, 4>(kind) : entry_of<T, false, 4>(kind);
  if (zc <= 8) return L.cell ? entry_of<T, true, 8>(kind) : entry_of<T, false, 8>(kind);
  if constexpr (sizeof(T) == 4)
    if (zc <= 16) return L.cell ? entry_of<T, true, 16>(kind) : entry_of<T, false, 16>(kind);
  return {};
}

}  // namespace

// Tiles of the solves that have a turn, by device.
static std::atomic<int> g_tiles[kDevices];

bool ResidentTurn::take(int tiles) {
  int dev, cus;
  if (!this_device(dev, cus)) return false;
  const int others = g_tiles[dev].fetch_add(tiles, std::memory_order_relaxed);
  if (others > 0 && others + tiles > cus) {
    g_tiles[dev].fetch_sub(tiles, std::memory_order_relaxed);
    return false;
  }
  dev_ = dev;
  tiles_ = tiles;
  return true;
}

ResidentTurn::~ResidentTurn() {
  if (tiles_) g_tiles[dev_].fetch_sub(tiles_, std::memory_order_relaxed);
}

template <typename T>
bool resident_fits(const Launch<T>& L, int kind) {
  const Geo& g = L.tl.geo;
  if (!L.ring || !L.tl.tile_order || g.ntiles > kResidentTiles || g.zc > resident_planes(sizeof(T)))
    return false;
  return entry_for<T>(L, kind).fit >= g.ntiles;
}

template <typename T>
hipError_t launch_resident(const Launch<T>& L, int kind, const ResidentVectors<T>& v, int iters,
                           int parity, bool absent) {
  ResArgs<T> a{};
  a.geo = L.tl.geo;
  a.op = L.op;
  a.kappa = L.kappa;
  a.x = v.x; a.rh = v.rh; a.t = v.t;
  for (int q = 0; q < 2; ++q) { a.r[q] = v.r[q]; a.p[q] = v.p[q]; a.v[q] = v.v[q]; }
  // exchange vectors: ones whose values are in registers or not kept
  switch (kind) {
    case kResidentBicgstab: a.set[0] = v.r[1]; a.set[1] = v.t; a.set[2] = v.r[0]; break;
    case kResidentBicgstab2:
      a.set[0] = v.r[parity ^ 1]; a.set[1] = v.t; a.set[2] = v.r[parity];
      break;
    case kResidentCg: a.set[0] = v.v[0]; a.set[1] = v.v[1]; a.set[2] = v.t; break;
    default: a.set[0] = v.p[parity ^ 1]; a.set[1] = v.t; a.set[2] = v.p[parity]; break;
  }
  a.ring = L.ring;
  a.copies = L.ring_copies;
  a.sc = L.sc;
  a.iters = iters;
  a.parity = parity;
  a.hashed = L.shadow;
  void* args[] = {(void*)&a};
  return hipLaunchKernel((const void*)entry_for<T>(L, kind).kernel,
                         dim3(a.geo.ntiles - (absent ? 1 : 0)), dim3(kThreads), args, 0, L.stream);
}

// The solve's scalars, with every slot of the ring empty.
__global__ void __launch_bounds__(1024)
k_set_resident(Scalars* __restrict__ dst, Scalars v, Scalars* __restrict__ dst2, Scalars v2,
               uint64_t* __restrict__ ring, int slots) {
  if (threadIdx.x == 0) *dst = v;
  if (threadIdx.x == 1 && dst2) *dst2 = v2;
  for (int e = threadIdx.x; e < slots; e += 1024) ring[e] = Empty<double>::value;
}

void launch_set_resident(Scalars* dst, const Scalars& v, double* ring, int copies, int ntiles,
                         hipStream_t s, Scalars* dst2, const Scalars* v2) {
  hipLaunchKernelGGL(k_set_resident, dim3(1), dim3(1024), 0, s, dst, v, v2 ? dst2 : nullptr,
                     v2 ? *v2 : v, (uint64_t*)ring, copies * kRing * kMaxReduce * ntiles);
}

// Copies of the ring that fit in `doubles` (a power of two, one per XCD at most).
int ring_copies(size_t doubles, int ntiles) {
  int c = 8;
  while (c > 1 && (size_t)c * kRing * kMaxReduce * ntiles > doubles) c /= 2;
  return c;
}

#define WFA_RES(T)                                       \
  template bool resident_fits<T>(const Launch<T>&, int); \
  template hipError_t launch_resident<T>(const Launch<T>&, int, const ResidentVectors<T>&, int, int, bool);
WFA_RES(float)
WFA_RES(double)
#undef WFA_RES

}  // namespace wfa
