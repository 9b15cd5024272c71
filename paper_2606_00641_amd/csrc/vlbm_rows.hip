// Several steps of a 2D periodic lattice in one pass over memory (gfx950).
//
// The sweep (vlbm_sweep.hip) reads and writes every population once per step and is bound
// by that traffic.  Here a wavefront walks up a strip of 64 x columns and carries T time
// levels at once: level 1 collides row r, level 2 row r - 1 of the next step, ..., level T
// row r - T + 1.  What a level streams within its row passes between lanes (DPP), what it
// streams to the rows above and below stays in the lane's registers, so no LDS, no barrier
// and no memory lie between the levels; the pass reads the populations of T steps ago and
// writes those after T steps.  The outermost lanes and rows of a strip lack their
// neighbours at the next level, so each level is one column and row narrower on each side:
// 64 - 2 (T - 1) columns and `rows` rows of a strip's end result are whole, and the strips
// overlap.  Populations are in natural layout (slot i of cell x holds f_i(x)) before and
// after; a pass goes from one buffer to the other, so neighbouring strips may still read
// what another has already advanced.
// The collision is the sweep's, per cell.
//
// Bound by one wavefront per SIMD working through its levels (293 VGPRs for 8 variables in
// FP32 and 4 levels; held to 256 they spill, and a step took 105 us instead of 28 on
// 1024^2).  Per step, the in-place sweep against passes: 8 variables FP32 1024^2 61.2 ->
// 27.5 us, 2000^2 232 -> 82 us (4 levels; 3 levels at two wavefronts per SIMD 39 and 175);
// FP64 1024^2 124 -> 87 us; 13 variables FP32 2000^2 405 -> 293 us (2 levels).
#include "vlbm_device.h"

namespace vlbm {
namespace {

template <typename R>
__device__ __forceinline__ R from_left(R v) {  // lane l gets the v of lane l - 1 (lane 0 its own)
  return lane_shift<true>(v, v);
}
template <typename R>
__device__ __forceinline__ R from_right(R v) {  // lane l gets the v of lane l + 1 (lane 63 its own)
  return lane_shift<false>(v, v);
}

template <typename R>
__device__ __forceinline__ R get(void* base, size_t plane_bytes, int plane, unsigned off) {
  return *(const VLBM_GLOBAL R*)(plane_base(base, plane_bytes, plane) + off);
}

// T levels, one wavefront per strip; workgroups are numbered so that each XCD gets
// consecutive ones (neighbouring strips share the lines at their edges).  The next row's
// populations are loaded while the levels of this one collide.
template <int ST, int MODEL, int T, int COLL>
__global__ __launch_bounds__(256) void k_rows(const Grid g, void* const out, const Phys ph, int rows) {
  using R = typename Store<ST>::R;
  static_assert(sizeof(R) == sizeof(typename Store<ST>::T), "FP64 or FP32 storage");
  constexpr int NQ = 5, K = kNVars<MODEL>, V = 64 - 2 * (T - 1);
  constexpr unsigned ES = sizeof(R);
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int nx = g.nx, ny = g.ny;
  const int strips = (nx + V - 1) / V, chunks = (ny + rows - 1) / rows;
  const unsigned nb = gridDim.x, L = blockIdx.x, q = nb / 8, rem = nb % 8, xcd = L % 8;
  const long long task = (long long)(xcd * q + min(xcd, rem) + L / 8) * 4 + wv;
  if (task >= (long long)strips * chunks * g.nz) return;
  const int s = (int)(task % strips), ch = (int)((task / strips) % chunks), z = (int)(task / ((long long)strips * chunks));
  const int y0 = ch * rows, nr = min(rows, ny - y0), nj = nr + 2 * (T - 1);
  int x = (s * V - (T - 1) + lane) % nx;
  x = x < 0 ? x + nx : x;
  const bool mine = lane >= T - 1 && lane <= 64 - T && lane - (T - 1) < nx - s * V;
  const unsigned slice = (unsigned)z * (unsigned)nx * (unsigned)ny;
  const unsigned xo = (unsigned)x, xp = x + 1 == nx ? 0u : xo + 1u, xm = x == 0 ? (unsigned)nx - 1u : xo - 1u;
  const size_t pb = (size_t)g.stride * ES;
  void* const F = g.f;
  auto wrap = [&](int y) { return (y % ny + ny) % ny; };

  R f[K][NQ], nf[K][NQ];
  // level t's row below the one in flight: f_0, f_{+x}, f_{-x} as they arrive in it, the
  // f_{+y} that arrives in it, and the f_{+y} it sends up
  R C[T - 1][K][5];
#pragma unroll
  for (int t = 0; t < T - 1; ++t)
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int i = 0; i < 5; ++i) C[t][k][i] = R(0);
  int yr = wrap(y0 - (T - 1));
  auto load = [&](R (&d)[K][NQ], int y) __attribute__((always_inline)) {
    const unsigned off = (slice + (unsigned)y * (unsigned)nx + xo) * ES;
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int i = 0; i < NQ; ++i) d[k][i] = get<R>(F, pb, k * NQ + i, off);
  };
  load(f, yr);
  int yw = wrap(y0);  // the row level T completes next
#pragma unroll 1
  for (int j = 0; j < nj; ++j) {
    yr = yr + 1 == ny ? 0 : yr + 1;
    if (j + 1 < nj) load(nf, yr);
    R dl;
    collide<R, 2, MODEL, COLL>(f, ph, dl);
#pragma unroll
    for (int t = 0; t < T - 1; ++t) {
      R h[K][NQ];
#pragma unroll
      for (int k = 0; k < K; ++k) {
        h[k][0] = C[t][k][0];
        h[k][1] = C[t][k][1];
        h[k][2] = C[t][k][2];
        h[k][3] = C[t][k][3];
        h[k][4] = f[k][4];
        C[t][k][0] = f[k][0];
        C[t][k][1] = from_left(f[k][1]);
        C[t][k][2] = from_right(f[k][2]);
        C[t][k][3] = C[t][k][4];
        C[t][k][4] = f[k][3];
      }
      // level t + 2 begins with the row whose neighbours have both passed level t + 1
      if (j >= 2 * (t + 1)) collide<R, 2, MODEL, COLL>(h, ph, dl);
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int i = 0; i < NQ; ++i) f[k][i] = h[k][i];
    }
    if (j >= 2 * (T - 1)) {
      const unsigned row = slice + (unsigned)yw * (unsigned)nx;
      const unsigned up = slice + (unsigned)(yw + 1 == ny ? 0 : yw + 1) * (unsigned)nx;
      const unsigned dn = slice + (unsigned)(yw == 0 ? ny - 1 : yw - 1) * (unsigned)nx;
      const unsigned dst[NQ] = {(row + xo) * ES, (row + xp) * ES, (row + xm) * ES, (up + xo) * ES, (dn + xo) * ES};
      if (mine) {
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
          for (int i = 0; i < NQ; ++i) st_shifted<R>(out, pb, k * NQ + i, dst[i], f[k][i]);
      }
      yw = yw + 1 == ny ? 0 : yw + 1;
    }
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int i = 0; i < NQ; ++i) f[k][i] = nf[k][i];
  }
}

template <int ST, int MODEL, int T>
hipError_t rows_t(const Launch& L, const Grid& g, void* out, const Phys& ph, int rows) {
  constexpr int V = 64 - 2 * (T - 1);
  const long long tasks = (long long)((g.nx + V - 1) / V) * ((g.ny + rows - 1) / rows) * g.nz;
  const dim3 grd((unsigned)((tasks + 3) / 4)), blk(256);
  if (ph.collision)
    hipLaunchKernelGGL((k_rows<ST, MODEL, T, 1>), grd, blk, 0, L.stream, g, out, ph, rows);
  else
    hipLaunchKernelGGL((k_rows<ST, MODEL, T, 0>), grd, blk, 0, L.stream, g, out, ph, rows);
  return hipGetLastError();
}

// Rows per strip: so many that the strips of the lattice fill the chip once, one wavefront
// per SIMD (1024), and never a few of them a second time; at least 8 (a strip reads and
// partly collides 2 (T - 1) rows more than it completes).
int rows_for(const Grid& g, int T) {
  const int V = 64 - 2 * (T - 1);
  const long long strips = (long long)((g.nx + V - 1) / V) * g.nz, per = std::max<long long>(1, 1024 / strips);
  return (int)std::min<long long>(g.ny, std::max<long long>(8, (g.ny + per - 1) / per));
}

}  // namespace

int rows_levels(const Launch& L, const Grid& g, const Phys& ph) {
  if (L.dim != 2 || (L.storage != ST_F32 && L.storage != ST_F64) || ph.source != 0 || g.mask) return 0;
  if (L.storage == ST_F64 && L.model == 4) return 0;  // its levels do not fit the registers
  const int T = L.storage == ST_F64 || L.model == 4 ? 2 : 4;
  // from 512^2 on (below, the populations sit in the L2s and the sweep is faster: 384^2 FP32
  // 7.7 us a step against 11.6), and where the strips waste at most a quarter of their lanes
  const int V = 64 - 2 * (T - 1), strips = (g.nx + V - 1) / V;
  if ((long long)g.nx * g.ny * g.nz < 512 * 512 || 4LL * g.nx < 3LL * strips * V) return 0;
  return T;
}

hipError_t launch_rows(const Launch& L, const Grid& g, void* out, const Phys& ph, int levels) {
  const int rows = rows_for(g, levels);
#define ROWS_CASE(S, M, T) \
  if (L.storage == S && L.model == M && levels == T) return rows_t<S, M, T>(L, g, out, ph, rows);
  ROWS_CASE(ST_F32, 0, 4) ROWS_CASE(ST_F32, 2, 4) ROWS_CASE(ST_F32, 3, 4)
  ROWS_CASE(ST_F32, 0, 2) ROWS_CASE(ST_F32, 2, 2) ROWS_CASE(ST_F32, 3, 2) ROWS_CASE(ST_F32, 4, 2)
  ROWS_CASE(ST_F64, 0, 2) ROWS_CASE(ST_F64, 2, 2) ROWS_CASE(ST_F64, 3, 2)
#undef ROWS_CASE
  return hipErrorInvalidValue;
}

}  // namespace vlbm
