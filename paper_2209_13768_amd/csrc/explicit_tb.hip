// Explicit forward-time steps with temporal blocking: S steps of
//   T' = T - (A T - T) + boundary terms
// (the paper's explicit scheme, Eq. 2, with the operator's general faces)
// per pass over HBM.  The paper's wafer keeps the whole field in SRAM next
// to the processors, so each step costs no memory traffic at all (section
// 3.1); on a GPU a one-step pass reads and writes the field once, which
// bounds it at 2w bytes per cell-step.  Fusing S steps into one pass cuts
// that to about 2w / S plus the redundant halo reads below.
//
// A workgroup owns a column of 64 x TY cells (TY = 4 waves x RY rows; lane =
// x, so each row is one contiguous load) and marches it along z.  Step level
// s (s = 1..S) of a plane m needs level s-1 on the planes m-1, m, m+1 and on
// the x/y neighbours, so the levels run as a pipeline behind the loads: when
// level 0 (the input) of plane j arrives, level s is computed on plane
// j - s.  Each thread keeps the last three planes of every level for its
// own cells in registers (the z neighbours).  The x neighbours are the
// adjacent lanes of the same wave, read with DPP lane shifts; the y
// neighbours are the thread's own rows, except across the boundary between
// two waves, whose first and last rows of every level go through a small
// double-buffered LDS exchange (one barrier per plane).  Level s is correct on the
// column shrunk by s cells on each side, so a tile's output is the inner
// (64 - 2S) x (TY - 2S) cells; neighbouring tiles overlap by 2S cells and
// recompute the overlap.  Along z a tile covers zc output planes and reads
// S more on each side.
//
// Each level applies exactly the arithmetic of a one-step pass to the same
// values, so the result is bitwise that of S one-step passes.
#include "device.hpp"
#include "internal.hpp"

namespace wfa {

struct TbGeo {
  int nx, ny, nz;
  int tiles_x, tiles_y, zchunks, zc;
  int ntiles;
  long long plane;
};

// Value of lane - 1 (from_left) or lane + 1 (from_right) of the wave; 0 at
// the wave's ends, which hold the column's halo, outside every level's
// valid region.
__device__ __forceinline__ int dpp_left(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xF, 0xF, true);   // wave_shr:1
}
__device__ __forceinline__ int dpp_right(int v) {
  return __builtin_amdgcn_update_dpp(0, v, 0x130, 0xF, 0xF, true);   // wave_shl:1
}
__device__ __forceinline__ float from_left(float v) { return __int_as_float(dpp_left(__float_as_int(v))); }
__device__ __forceinline__ float from_right(float v) { return __int_as_float(dpp_right(__float_as_int(v))); }
__device__ __forceinline__ double from_left(double v) {
  return __hiloint2double(dpp_left(__double2hiint(v)), dpp_left(__double2loint(v)));
}
__device__ __forceinline__ double from_right(double v) {
  return __hiloint2double(dpp_right(__double2hiint(v)), dpp_right(__double2loint(v)));
}

// x terms of a row's cells, d(x-) from_left(c) + d(x+) from_right(c), the
// first product alone in its rounding as fma(d, nb, 0) is.  FP32: the lane
// shifts ride on the multiply and the multiply-add (the leading wait states
// cover a source written just before; the assembler's block is opaque to the
// compiler's own check for that).
__device__ __forceinline__ float x_terms(float c, float dm, float dp) {
  float acc;
  asm("s_nop 1\n\t"
      "v_mul_f32_dpp %0, %1, %2 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n\t"
      "v_fmac_f32_dpp %0, %1, %3 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:0"
      : "=&v"(acc)
      : "v"(c), "v"(dm), "v"(dp));
  return acc;
}
__device__ __forceinline__ double x_terms(double c, double dm, double dp) {
#pragma clang fp contract(off)
  return fma_t(dp, from_right(c), dm * from_left(c));
}

// Buffer access with a lane offset and a workgroup-uniform one: no address
// arithmetic per lane, and lanes at kNowhere read 0 and write nothing.
constexpr int kNowhere = 0x7ffff000;
constexpr int kNontemporal = 2;
__device__ __forceinline__ float buf_load_t(__amdgpu_buffer_rsrc_t r, int off, int soff, float) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, soff, 0));
}
__device__ __forceinline__ double buf_load_t(__amdgpu_buffer_rsrc_t r, int off, int soff, double) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, 0));
}
__device__ __forceinline__ void buf_store_t(__amdgpu_buffer_rsrc_t r, int off, int soff, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, off, soff, kNontemporal);
}
__device__ __forceinline__ void buf_store_t(__amdgpu_buffer_rsrc_t r, int off, int soff, double v) {
  using B = decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0, 0, 0));
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(B, v), r, off, soff, kNontemporal);
}

// Instruction issue bounds the fused pass (it moves 2.9 TB/s at S = 4, FP32):
// 12 vector instructions a cell and level in the interior, with the cells of
// the column's overlap and the planes above and below a tile computed again.
// Measured, us a step, before the face tests left the interior, the planes
// stopped moving between registers and the lane shifts joined the arithmetic
// -> now: 512x512x1024 FP32, S = 3: 368 -> 243, S = 4: 505 -> 234; 512^3 FP64,
// S = 2: 342 -> 259, S = 3: 399 -> 222.  Columns of 8 waves, which compute less
// overlap, ran slower (FP32 S = 4: 321); the waves a SIMD is compiled for
// keep S = 3 in FP64 at four (20 bytes spilled; at three 239) and S = 3 and 4
// in FP32 at three without spills (S = 3 at four: 318).
template <typename T, int S, int RY>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(S == 2 || (S == 3 && sizeof(T) == 8) ? 4 : 3)))
k_explicit_tb(TbGeo g, Op<T> op, const T* __restrict__ x, T* __restrict__ y) {
  constexpr int TY = kWaves * RY;
  constexpr int OW = kTX - 2 * S;
  constexpr int OH = TY - 2 * S;
  constexpr int WB = sizeof(T);
  static_assert(OW > 0 && OH > 0, "tile too small for the number of fused steps");
  static_assert(RY >= 2, "a wave's first and last rows must differ");
  // [parity][level][wave][lane]: each wave's first (top) and last (bottom)
  // row of the middle plane of every level below S
  __shared__ T top[2][S][kWaves][kTX];
  __shared__ T bot[2][S][kWaves][kTX];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int tx = tile % g.tiles_x;
  const int rest = tile / g.tiles_x;
  const int ty = rest % g.tiles_y;
  const int tz = rest / g.tiles_y;
  const int i = tx * OW - S + lane;      // this lane's column
  const int j0 = ty * OH - S + wave * RY;  // the wave's first row (uniform)
  const int zs = tz * g.zc;
  const int ze = min(zs + g.zc, g.nz);
  const bool col_in = i >= 0 && i < g.nx;
  const bool col_out = lane >= S && lane < kTX - S && i < g.nx;
  const uint32_t ins_x = (i > 0 ? 1u : 0u) | (i < g.nx - 1 ? 2u : 0u);
  // The wave's rows all have both y neighbours: where the plane has its z
  // neighbours too, a level is computed without a face test, from the
  // coefficients below.
  const bool inner = j0 > 0 && j0 + RY < g.ny;
  // Rows so long that a wave's span passes the buffer offsets' range are
  // addressed by pointers.
  const bool wide = g.nx > (1 << 24) / RY;
  // the neighbouring waves' rows (the tile's outermost waves read a row of
  // their own instead: it lies in the halo, outside every valid region)
  const int wup = wave > 0 ? wave - 1 : wave;
  const int wdn = wave < kWaves - 1 ? wave + 1 : wave;
  // first and last output row of the wave
  const int r_lo = max(0, S - wave * RY), r_hi = min(RY, min(TY - S - wave * RY, g.ny - j0));

  // The operator's row of this lane's cells where y and z neighbours exist:
  // couplings in x (0 where there is no neighbour), the diagonal in face
  // order, and the x faces' boundary terms, as cell_apply and cell_bterm
  // form them.
  T dxm = T(0), dxp = T(0), diag = T(1), diag_x = T(1), bx = T(0);
  {
#pragma clang fp contract(off)
#pragma unroll
    for (int f = 0; f < 6; ++f) {
      const bool in = f > 1 || (ins_x & (1u << f));
      if (in || (op.dir & (1u << f))) diag += op.cD + op.out[f];
      if (f == 1) diag_x = diag;
    }
    if (ins_x & 1u) dxm = op.cD + op.in[0];
    else if (op.dir & 1u) bx = fma_t(op.cD + op.in[0], op.bval[0], bx);
    if (ins_x & 2u) dxp = op.cD + op.in[1];
    else if (op.dir & 2u) bx = fma_t(op.cD + op.in[1], op.bval[1], bx);
  }
  const T dym = op.cD + op.in[2], dyp = op.cD + op.in[3];
  const T dzm = op.cD + op.in[4], dzp = op.cD + op.in[5];

  // W[q][0..2]: level q on three successive planes.  The newest plane's slot
  // is the step's phase (its number modulo 3), so that no plane moves from
  // one register to another.
  T W[S][3][RY];
#pragma unroll
  for (int q = 0; q < S; ++q)
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int r = 0; r < RY; ++r) W[q][a][r] = T(0);

  const int jb = zs - S > 0 ? zs - S : 0;
  const int row_bytes = wide ? 0 : g.nx * WB;
  const int lin = col_in ? i * WB : kNowhere, lout = col_out ? i * WB : kNowhere;
  auto rows_at = [&](const T* p, int k) {
    return __builtin_amdgcn_make_buffer_rsrc(
        const_cast<T*>(p) + (size_t)k * g.plane + (long long)j0 * g.nx, 0, RY * row_bytes, 0x00020000);
  };
  // input plane k (0 past the grid)
  T pre[RY];
  auto load = [&](int k) {
    if (k >= g.nz) {
#pragma unroll
      for (int r = 0; r < RY; ++r) pre[r] = T(0);
    } else if (!wide) {
      const auto p = rows_at(x, k);
#pragma unroll
      for (int r = 0; r < RY; ++r)
        pre[r] = buf_load_t(p, inner || (j0 + r >= 0 && j0 + r < g.ny) ? lin : kNowhere,
                            r * row_bytes, T(0));
    } else {
#pragma unroll
      for (int r = 0; r < RY; ++r) {
        int j = j0 + r;
        asm volatile("" : "+s"(j));   // opaque: no row pointers held over the loop
        const T* row = x + (size_t)k * g.plane + (long long)j * g.nx;
        pre[r] = (col_in && j >= 0 && j < g.ny) ? row[i] : T(0);
      }
    }
  };
  load(jb);

  int par = 0;
  // One step: input plane k arrives, level s is computed on plane k - s.
  // N: the slot of the newest planes.
  auto step = [&](int k, auto phase) {
    constexpr int N = decltype(phase)::value, M = (N + 2) % 3, O = (N + 1) % 3;
#pragma unroll
    for (int r = 0; r < RY; ++r) W[0][N][r] = pre[r];
    load(k + 1);
    // every level's middle plane: the wave's boundary rows into LDS (the
    // buffer of this parity was last read two steps ago, before the
    // previous step's barrier)
#pragma unroll
    for (int q = 0; q < S; ++q) {
      top[par][q][wave][lane] = W[q][M][0];
      bot[par][q][wave][lane] = W[q][M][RY - 1];
    }
    __syncthreads();
#pragma unroll
    for (int s = 1; s <= S; ++s) {
      const int m = k - s;  // plane of level s computed in this step
      const T above = bot[par][s - 1][wup][lane];  // row j0 - 1
      const T below = top[par][s - 1][wdn][lane];  // row j0 + RY
      T v[RY];
      if (inner && m > 0 && m < g.nz - 1) {
#pragma clang fp contract(off)
#pragma unroll
        for (int r = 0; r < RY; ++r) {
          const T c = W[s - 1][M][r];
          T acc = x_terms(c, dxm, dxp);
          acc = fma_t(dym, r > 0 ? W[s - 1][M][r > 0 ? r - 1 : 0] : above, acc);
          acc = fma_t(dyp, r < RY - 1 ? W[s - 1][M][r < RY - 1 ? r + 1 : r] : below, acc);
          acc = fma_t(dzm, W[s - 1][O][r], acc);
          acc = fma_t(dzp, W[s - 1][N][r], acc);
          v[r] = explicit_update(c, fma_t(diag, c, -acc), bx);
        }
      } else {
        // rows or a plane on a face: the couplings, diagonal and boundary
        // terms of the y and z faces by row and plane, all uniform (adding 0
        // to a diagonal and coupling a cell outside with 0 change nothing)
#pragma clang fp contract(off)
        const bool plane_ok = m >= 0 && m < g.nz;
        int jr = j0, mm = m;   // opaque: formed here every time, not hoisted
        asm volatile("" : "+s"(jr), "+s"(mm));
        const bool in_z[2] = {mm > 0, mm < g.nz - 1};
#pragma unroll
        for (int r = 0; r < RY; ++r) {
          const T c = W[s - 1][M][r];
          const T nb[4] = {r > 0 ? W[s - 1][M][r > 0 ? r - 1 : 0] : above,
                           r < RY - 1 ? W[s - 1][M][r < RY - 1 ? r + 1 : r] : below,
                           W[s - 1][O][r], W[s - 1][N][r]};
          T dg = diag_x, bt = bx, acc = x_terms(c, dxm, dxp);
#pragma unroll
          for (int f = 2; f < 6; ++f) {
            const bool in = f == 2 ? jr + r > 0 : f == 3 ? jr + r < g.ny - 1 : in_z[f - 4];
            const bool dir = op.dir & (1u << f);
            const T din = op.cD + op.in[f];
            dg += in || dir ? op.cD + op.out[f] : T(0);
            acc = fma_t(in ? din : T(0), nb[f - 2], acc);
            bt = fma_t(!in && dir ? din : T(0), op.bval[f], bt);
          }
          const T u = explicit_update(c, fma_t(dg, c, -acc), bt);
          v[r] = plane_ok ? u : T(0);
        }
      }
      if (s < S) {
#pragma unroll
        for (int r = 0; r < RY; ++r) W[s < S ? s : 0][N][r] = v[r];
      } else if (m >= zs && m < g.nz) {
        if (!wide) {
          const auto p = rows_at(y, m);
#pragma unroll
          for (int r = 0; r < RY; ++r)
            if (r >= r_lo && r < r_hi) buf_store_t(p, lout, r * row_bytes, v[r]);
        } else if (col_out) {
#pragma unroll
          for (int r = 0; r < RY; ++r) {
            int j = j0 + r;
            asm volatile("" : "+s"(j));
            if (r >= r_lo && r < r_hi)
              __builtin_nontemporal_store(v[r], y + (size_t)m * g.plane + (long long)j * g.nx + i);
          }
        }
      }
    }
    par ^= 1;
  };
  const int end = ze + S;
  for (int k = jb; k < end; k += 3) {
    step(k, std::integral_constant<int, 0>{});
    if (k + 1 < end) step(k + 1, std::integral_constant<int, 1>{});
    if (k + 2 < end) step(k + 2, std::integral_constant<int, 2>{});
  }
}

template <typename T, int S, int RY>
static void launch_tb(const Launch<T>& L, const T* x, T* y, int zc_override) {
  constexpr int TY = kWaves * RY;
  const Geo& G = L.tl.geo;
  TbGeo g{};
  g.nx = G.nx; g.ny = G.ny; g.nz = G.nz;
  g.plane = (long long)G.nx * G.ny;
  g.tiles_x = (G.nx + (kTX - 2 * S) - 1) / (kTX - 2 * S);
  g.tiles_y = (G.ny + (TY - 2 * S) - 1) / (TY - 2 * S);
  const long long txy = (long long)g.tiles_x * g.tiles_y;
  int zc = zc_override > 0 ? zc_override : pass_planes(txy, G.nz, 2 * S, 32);
  if (zc > G.nz) zc = G.nz;
  g.zc = zc;
  g.zchunks = (G.nz + zc - 1) / zc;
  g.ntiles = (int)(txy * g.zchunks);
  hipLaunchKernelGGL((k_explicit_tb<T, S, RY>), dim3(g.ntiles), dim3(kThreads), 0, L.stream, g,
                     L.op, x, y);
}

template <typename T>
void launch_explicit_fused(const Launch<T>& L, const T* x, T* y, int steps, int zc_override) {
  // FP32 columns of 32 rows, FP64 of 16 (registers hold 3 planes per level)
  constexpr int RY = sizeof(T) == 4 ? 8 : 4;
  switch (steps) {
    case 2: launch_tb<T, 2, RY>(L, x, y, zc_override); break;
    case 3: launch_tb<T, 3, RY>(L, x, y, zc_override); break;
    default: launch_tb<T, 4, RY>(L, x, y, zc_override); break;
  }
}

template void launch_explicit_fused<float>(const Launch<float>&, const float*, float*, int, int);
template void launch_explicit_fused<double>(const Launch<double>&, const double*, double*, int,
                                            int);

}  // namespace wfa
