// Several steps of a periodic lattice in one pass over memory (gfx950): large 2D lattices in
// FP32 (k_rows, described here), other 2D lattices (k_tiles), 3D lattices in FP32 (k_cols).
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
// The collision is the sweep's, per cell and bit for bit (vlbm_fixed.h).
//
// Bound by one wavefront per SIMD working through its levels (293 VGPRs for 8 variables in
// FP32 and 4 levels; held to 256 they spill, and a step took 105 us instead of 28 on
// 1024^2).  Per step, the in-place sweep against passes: 8 variables FP32 1024^2 57.8 ->
// 26.4 us, 1400^2 115 -> 43.3, 2000^2 240 -> 81.1 (4 levels; 3 levels at two wavefronts per SIMD 39 and 175).
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
template <int MODEL, int T, int COLL>
__global__ __launch_bounds__(256) void k_rows(const Grid g, void* const out, const Phys ph, int rows) {
  using R = float;
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
    collide_cell<true, R, 2, MODEL, COLL>(f, ph, dl);
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
      if (j >= 2 * (t + 1)) collide_cell<true, R, 2, MODEL, COLL>(h, ph, dl);
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

// Rows per strip: so many that the strips of the lattice fill the chip once, one wavefront
// per SIMD (1024), and never a few of them a second time; at least 8 (a strip reads and
// partly collides 2 (T - 1) rows more than it completes).
int rows_for(const Grid& g, int T) {
  const int V = 64 - 2 * (T - 1);
  const long long strips = (long long)((g.nx + V - 1) / V) * g.nz, per = std::max<long long>(1, 1024 / strips);
  return (int)std::min<long long>(g.ny, std::max<long long>(8, (g.ny + per - 1) / per));
}

template <int MODEL, int T>
hipError_t rows_t(const Launch& L, const Grid& g, void* out, const Phys& ph) {
  constexpr int V = 64 - 2 * (T - 1);
  const int rows = rows_for(g, T);
  const long long tasks = (long long)((g.nx + V - 1) / V) * ((g.ny + rows - 1) / rows) * g.nz;
  const dim3 grd((unsigned)((tasks + 3) / 4)), blk(256);
  if (ph.collision)
    hipLaunchKernelGGL((k_rows<MODEL, T, 1>), grd, blk, 0, L.stream, g, out, ph, rows);
  else
    hipLaunchKernelGGL((k_rows<MODEL, T, 0>), grd, blk, 0, L.stream, g, out, ph, rows);
  return hipGetLastError();
}

// T steps of a 2D lattice in one pass, one cell per thread: a tile of TX x TY cells, those
// whose result is whole, (TX - 2 (T - 1)) x (TY - 2 (T - 1)), and T - 1 around them; between
// the levels what moves passes through LDS.  For lattices on which k_rows' long strips leave
// the chip idle, and in FP64, where k_rows' registers hold two levels only.
// Bound on small lattices by the launch and the levels' latency (64^2: about 5 us a launch and
// 1.2 us a level in FP64, 0.8 in FP32), on large ones by the overlap: 512 threads complete 260
// cells, 256 threads 100.  Neighbouring tiles go to one XCD, whose L2 then holds what they
// share (512^2 FP32 10.3 -> 7.1 us).  Per step, the in-place sweep against passes of 4: 8
// variables FP64 64^2 4.7 -> 2.4 us, 256^2 7.9 -> 5.1, 1024^2 116 -> 73 (k_rows 86); FP32
// 64^2 5.5 -> 1.9, 512^2 18.0 -> 6.9 (k_rows 12.3), 800^2 37 -> 13.1; 13 variables FP64 64^2
// 5.7 -> 3.7, 2000^2 822 -> 677, FP32 256^2 7.5 -> 5.6, 2000^2 414 -> 258 (k_rows, 2 levels, 294).
// 5 variables in FP64 are held to 128 VGPRs, four wavefronts per SIMD, for which their LDS leaves
// room (at 130: 2000^2 114 -> 147 us a step).
template <int ST, int MODEL, int T, int TX, int TY, int COLL>
__global__ __launch_bounds__(TX* TY, ST == ST_F64 && MODEL == 2 ? 4 : 1) void k_tiles(const Grid g, void* const out,
                                                                                      const Phys ph) {
  using R = typename Store<ST>::R;
  constexpr int NQ = 5, K = kNVars<MODEL>, B = TX * TY, H = T - 1, IX = TX - 2 * H, IY = TY - 2 * H;
  constexpr unsigned ES = sizeof(R);
  __shared__ R e[4][K][B];
  const int t = threadIdx.x, col = t % TX, row = t / TX;
  const int nx = g.nx, ny = g.ny, nbx = (nx + IX - 1) / IX, nby = (ny + IY - 1) / IY;
  const unsigned nb = gridDim.x, L = blockIdx.x, q = nb / 8, rem = nb % 8, xcd = L % 8;
  const int task = (int)(xcd * q + min(xcd, rem) + L / 8);  // neighbouring tiles on one XCD
  const int x0 = task % nbx * IX, y0 = task / nbx % nby * IY;
  const bool mine = col >= H && col < TX - H && row >= H && row < TY - H && x0 + col - H < nx && y0 + row - H < ny;
  int x = (x0 + col - H) % nx, y = (y0 + row - H) % ny;
  x = x < 0 ? x + nx : x;
  y = y < 0 ? y + ny : y;
  const unsigned slice = (unsigned)(task / (nbx * nby)) * (unsigned)nx * (unsigned)ny;
  auto at = [&](int xx, int yy) { return (slice + (unsigned)yy * (unsigned)nx + (unsigned)xx) * ES; };
  const unsigned o = at(x, y);
  const size_t pb = (size_t)g.stride * ES;
  R f[K][NQ], dl;
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int i = 0; i < NQ; ++i) f[k][i] = get<R>(g.f, pb, k * NQ + i, o);
  const int tl = max(t - 1, 0), tr = min(t + 1, B - 1), td = max(t - TX, 0), tu = min(t + TX, B - 1);
  // one copy of the collision's code for all levels
#pragma unroll 1
  for (int lv = 0;;) {
    collide_cell<true, R, 2, MODEL, COLL>(f, ph, dl);
    if (++lv == T) break;
    if (lv > 1) __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int d = 0; d < 4; ++d) e[d][k][t] = f[k][1 + d];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      f[k][1] = e[0][k][tl];
      f[k][2] = e[1][k][tr];
      f[k][3] = e[2][k][td];
      f[k][4] = e[3][k][tu];
    }
  }
  if (!mine) return;
  const unsigned dst[NQ] = {o, at(x + 1 == nx ? 0 : x + 1, y), at(x == 0 ? nx - 1 : x - 1, y),
                            at(x, y + 1 == ny ? 0 : y + 1), at(x, y == 0 ? ny - 1 : y - 1)};
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int i = 0; i < NQ; ++i) st_shifted<R>(out, pb, k * NQ + i, dst[i], f[k][i]);
}

long long tiles_of(const Grid& g, int TX, int TY, int T) {
  const int IX = TX - 2 * (T - 1), IY = TY - 2 * (T - 1);
  return (long long)((g.nx + IX - 1) / IX) * ((g.ny + IY - 1) / IY) * g.nz;
}

template <int ST, int MODEL, int T, int TX, int TY>
hipError_t tiles_s(const Launch& L, const Grid& g, void* out, const Phys& ph) {
  const dim3 grd((unsigned)tiles_of(g, TX, TY, T)), blk(TX * TY);
  if (ph.collision)
    hipLaunchKernelGGL((k_tiles<ST, MODEL, T, TX, TY, 1>), grd, blk, 0, L.stream, g, out, ph);
  else
    hipLaunchKernelGGL((k_tiles<ST, MODEL, T, TX, TY, 0>), grd, blk, 0, L.stream, g, out, ph);
  return hipGetLastError();
}

// The tiles' width, 16 or 32, or 0: no tiles.  32 x 16 tiles once there are cells enough that
// the smaller overlap counts (8 variables FP32 100^2 x 4 3.2 us a step in 16 x 16 tiles, 3.0
// in 32 x 16; FP64, 256^2 6.3 and 7.3, 384^2 12.2 and 11.9), where they are the fewer
// threads (8 x 4000 2.7 and 3.8), and where their exchange fits the LDS (not 13 variables in
// FP64).  No tiles where they fill the chip with overlap and empty lanes: 1400^2 FP32 in 16 x
// 16 tiles, 2.6 threads a cell, 111 us a step like the sweep (32 x 16, 2.0: 49); FP64 158 in 16
// x 16 against 234; 13 variables FP64 2 x 4000, 400 tiles, 6.7 against 5.8.
int tile_width(const Launch& L, const Grid& g) {
  const bool heavy = L.storage == ST_F64 || L.model == 4, fits = !(L.storage == ST_F64 && L.model == 4);
  const long long N = (long long)g.nx * g.ny * g.nz, n16 = tiles_of(g, 16, 16, 4), n32 = tiles_of(g, 32, 16, 4);
  const bool wide = fits && N > (heavy ? 1 << 16 : 1 << 14) && 2 * n32 < n16;
  const long long threads = wide ? 512 * n32 : 256 * n16;
  if (threads > (fits ? 1 << 17 : 1 << 16) && 10 * threads > (heavy ? 27 : 24) * N) return 0;
  return wide ? 32 : 16;
}

template <int ST, int MODEL, int T>
hipError_t tiles_t(const Launch& L, const Grid& g, void* out, const Phys& ph) {
  if constexpr (!(ST == ST_F64 && MODEL == 4))
    if (tile_width(L, g) == 32) return tiles_s<ST, MODEL, T, 32, 16>(L, g, out, ph);
  return tiles_s<ST, MODEL, T, 16, 16>(L, g, out, ph);
}

// Two steps of a 3D lattice in one pass: a workgroup of eight wavefronts holds eight x rows,
// consecutive in y, of a strip of up to 62 columns and the one on each side of it, and walks
// up in z.  Level 1 collides plane z in all eight rows; along x it streams between lanes,
// along y through LDS, along z over the lane's own planes; level 2 collides plane z - 1 of
// the next step in the inner six rows.  The strip's columns of these rows are whole; a
// workgroup stages two planes more than it completes.  The exchange has two LDS buffers, so
// that one barrier per plane is enough: a plane's is written again only after the next
// plane's barrier, which every reader has passed by then.
// Bound by the memory path of one workgroup per CU (256 VGPRs): a wavefront's loads and
// stores of a plane, 56 each, pass one after the other; without its collisions the kernel
// takes as long.  The next plane is therefore asked for after level 1's collision, during
// which the stores of the plane before drain (120^3 110 -> 103 us a step), and the columns
// are shared evenly among as few strips as hold them (190^3 570 -> 420 us: four strips of 48
// columns instead of three of 62 and one of 4), in multiples of eight, whole 32-byte sectors.
// Per step, the in-place sweep against passes, 8 variables: 64^3 23.5 -> 18.8 us, 120^3
// 146 -> 100, 160^3 351 -> 226, 190^3 656 -> 402, 256^3 1351 -> 1217; 5 variables 90^3 38.5 ->
// 23.7, 210^3 576 -> 367; 9 variables 110^3 150 -> 112, 230^3 1373 -> 940 to 1070 (lattices over
// about 4 GB vary by a tenth with where their memory lies).  A tile of any width with both
// exchanges through LDS, and strips that run on over the rows' ends, fill the lanes better
// but need per-lane row addresses and spill: 190^3 474 and 698 us, 240^3 1010 and 1263
// against 873 (strips as they are).  Twelve wavefronts in 168 VGPRs spill more (160^3 415 us).
constexpr int kColWaves = 8, kColRows = kColWaves - 2, kColV = 62;
template <int MODEL, int COLL>
__global__ __launch_bounds__(64 * kColWaves, 2) void k_cols(const Grid g, void* const out, const Phys ph, int V, int planes) {
  using R = float;
  constexpr int NQ = 7, K = kNVars<MODEL>;
  constexpr unsigned ES = sizeof(R);
  __shared__ R xch[2][kColWaves][2][K][64];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int nx = g.nx, ny = g.ny, nz = g.nz;
  const int strips = (nx + V - 1) / V, tiles = (ny + kColRows - 1) / kColRows;
  const unsigned nb = gridDim.x, L = blockIdx.x, q = nb / 8, rem = nb % 8, xcd = L % 8;
  const int task = (int)(xcd * q + min(xcd, rem) + L / 8);
  const int s = task % strips, yt = (task / strips) % tiles, ch = task / (strips * tiles);
  const int z0 = ch * planes, nj = min(planes, nz - z0) + 2;
  // lanes past the strip's last neighbour read that one's address again, not memory of their own
  int x = (s * V - 1 + min(lane, nx - s * V + 1)) % nx;
  x = x < 0 ? x + nx : x;
  const int yi = yt * kColRows + wv - 1;  // this wavefront's row
  const int y = (yi % ny + ny) % ny;
  const bool inner = wv >= 1 && wv <= kColRows && yi < ny;
  const bool mine = inner && lane >= 1 && lane <= V && lane - 1 < nx - s * V;
  const unsigned pl = (unsigned)nx * (unsigned)ny;
  const unsigned xo = (unsigned)x, xp = x + 1 == nx ? 0u : xo + 1u, xm = x == 0 ? (unsigned)nx - 1u : xo - 1u;
  const unsigned ro = (unsigned)y * (unsigned)nx;
  const unsigned rp = (unsigned)(y + 1 == ny ? 0 : y + 1) * (unsigned)nx, rm = (unsigned)(y == 0 ? ny - 1 : y - 1) * (unsigned)nx;
  const size_t pb = (size_t)g.stride * ES;
  void* const F = g.f;

  R f[K][NQ], nf[K][NQ];
  // the plane below the one in flight after level 1: f_0, f_{+-x}, f_{+-y}, f_{+z} as they
  // arrive in it, and the f_{+z} it sends up
  R C[K][7];
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int i = 0; i < 7; ++i) C[k][i] = R(0);
  auto load = [&](R (&d)[K][NQ], int z) __attribute__((always_inline)) {
    const unsigned off = ((unsigned)z * pl + ro + xo) * ES;
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int i = 0; i < NQ; ++i) d[k][i] = get<R>(F, pb, k * NQ + i, off);
  };
  int zr = z0 == 0 ? nz - 1 : z0 - 1, zw = z0;
  load(f, zr);
#pragma unroll 1
  for (int j = 0; j < nj; ++j) {
    zr = zr + 1 == nz ? 0 : zr + 1;
    R dl;
    collide_cell<true, R, 3, MODEL, COLL>(f, ph, dl);
    if (j + 1 < nj) load(nf, zr);
    auto& e = xch[j & 1];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      e[wv][0][k][lane] = f[k][3];
      e[wv][1][k][lane] = f[k][4];
    }
    __syncthreads();
    R h[K][NQ];
    const int below = wv == 0 ? 0 : wv - 1, above = wv == kColWaves - 1 ? wv : wv + 1;
#pragma unroll
    for (int k = 0; k < K; ++k) {
#pragma unroll
      for (int i = 0; i < 6; ++i) h[k][i] = C[k][i];
      h[k][6] = f[k][6];
      C[k][0] = f[k][0];
      C[k][1] = from_left(f[k][1]);
      C[k][2] = from_right(f[k][2]);
      C[k][3] = e[below][0][k][lane];
      C[k][4] = e[above][1][k][lane];
      C[k][5] = C[k][6];
      C[k][6] = f[k][5];
    }
    if (j >= 2) {
      if (inner) {
        collide_cell<true, R, 3, MODEL, COLL>(h, ph, dl);
        const unsigned zo = (unsigned)zw * pl, zp = (unsigned)(zw + 1 == nz ? 0 : zw + 1) * pl,
                       zm = (unsigned)(zw == 0 ? nz - 1 : zw - 1) * pl;
        const unsigned dst[NQ] = {(zo + ro + xo) * ES, (zo + ro + xp) * ES, (zo + ro + xm) * ES, (zo + rp + xo) * ES,
                                  (zo + rm + xo) * ES, (zp + ro + xo) * ES, (zm + ro + xo) * ES};
        if (mine) {
#pragma unroll
          for (int k = 0; k < K; ++k)
#pragma unroll
            for (int i = 0; i < NQ; ++i) st_shifted<R>(out, pb, k * NQ + i, dst[i], h[k][i]);
        }
      }
      ++zw;
    }
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int i = 0; i < NQ; ++i) f[k][i] = nf[k][i];
  }
}

// Models whose two-rate collisions k_cols takes (those of 8 and 9 variables spill: 110^3 135 us
// a step in place, 238 in passes).
constexpr bool cols_two_rate(int model) { return model == 2; }

template <int MODEL>
hipError_t cols_t(const Launch& L, const Grid& g, void* out, const Phys& ph) {
  const int strips = (g.nx + kColV - 1) / kColV, V = std::min(kColV, ((g.nx + strips - 1) / strips + 7) / 8 * 8);
  const long long cols = (long long)((g.nx + V - 1) / V) * ((g.ny + kColRows - 1) / kColRows);
  // planes per workgroup: the share of z for which the rounds of workgroups over 256 CUs
  // times a workgroup's planes, the two it stages beyond them and its start is least
  long long best = -1;
  int planes = g.nz;
  for (int n = 1; n <= g.nz && n <= 256; ++n) {
    const int p = (g.nz + n - 1) / n;
    const long long cost = (cols * ((g.nz + p - 1) / p) + 255) / 256 * (p + 3);
    if (best < 0 || cost < best) best = cost, planes = p;
  }
  const dim3 grd((unsigned)(cols * ((g.nz + planes - 1) / planes))), blk(64 * kColWaves);
  if (ph.collision) {
    if constexpr (cols_two_rate(MODEL)) {
      hipLaunchKernelGGL((k_cols<MODEL, 1>), grd, blk, 0, L.stream, g, out, ph, V, planes);
      return hipGetLastError();
    }
    return hipErrorInvalidValue;
  }
  hipLaunchKernelGGL((k_cols<MODEL, 0>), grd, blk, 0, L.stream, g, out, ph, V, planes);
  return hipGetLastError();
}

// 2D passes of 4 steps by rows (k_rows) instead of tiles: FP32, up to 9 variables, where the
// populations exceed 190 MB and leave the last-level cache (8 variables 800^2 15.7 us a step
// against 13.3, 1024^2 27.3 and 26.9, 1400^2 44.4 and 49.0, 2000^2 81.9 and 97.0; 9 variables
// 1024^2 29.5 and 31.3; 5 variables 1024^2 14.1 and 11.3, 1400^2 28.3 and 29.2), and where the
// strips waste at most a quarter of their lanes and are no flatter than the rows they add.
bool by_rows(const Launch& L, const Grid& g) {
  constexpr int V = 64 - 2 * 3;
  const int K = L.model == 0 ? 8 : L.model == 2 ? 5 : 9, strips = (g.nx + V - 1) / V;
  return L.storage == ST_F32 && L.model != 4 && (long long)g.nx * g.ny * g.nz * K >= 9 << 20 && g.ny >= 16 &&
         4LL * g.nx >= 3LL * strips * V;
}

}  // namespace

int rows_levels(const Launch& L, const Grid& g, const Phys& ph) {
  if ((L.storage != ST_F32 && L.storage != ST_F64) || ph.source != 0 || g.mask) return 0;
  if (L.dim == 3) {
    if (L.storage != ST_F32 || L.model == 1 || (ph.collision && !cols_two_rate(L.model))) return 0;
    // From 2^18 cells on (48^3 stays in the caches: 9.4 us a step against 11.6), with planes,
    // rows and columns enough for the two planes, two of eight rows and two columns a tile
    // reads beyond its own (200^2 x 4 14.7 us against 15.9, 200 x 7 x 200 25.1 against 23.4,
    // 32 x 200^2 105 against 109), where the last of three and more strips is not nearly empty (130^3, 5
    // variables, 108 us against 114).  With 9 variables, more of whose registers spill, only
    // where the strips are three quarters full and the in-place rows not all aligned lines
    // (90^3 67.5 us against 68.8, 256^2 x 128 742 against 806).
    const int strips = (g.nx + kColV - 1) / kColV, tiles = (g.ny + kColRows - 1) / kColRows;
    const double fill = (double)g.nx / (strips * kColV);
    if ((long long)g.nx * g.ny * g.nz < 1 << 18 || g.nx < 56 || g.nz < 48 || 4 * g.ny < 3 * tiles * kColRows) return 0;
    if ((strips > 2 && fill < 0.71) || (L.model == 3 && (fill < 0.75 || g.nx % 64 == 0))) return 0;
    return 2;
  }
  return by_rows(L, g) || tile_width(L, g) ? 4 : 0;
}

hipError_t launch_rows(const Launch& L, const Grid& g, void* out, const Phys& ph, int levels) {
  if (L.dim == 3) {
    switch (L.model) {
      case 0: return cols_t<0>(L, g, out, ph);
      case 2: return cols_t<2>(L, g, out, ph);
      case 3: return cols_t<3>(L, g, out, ph);
      default: return hipErrorInvalidValue;
    }
  }
  if (by_rows(L, g) && levels == 4) {
    switch (L.model) {
      case 0: return rows_t<0, 4>(L, g, out, ph);
      case 2: return rows_t<2, 4>(L, g, out, ph);
      case 3: return rows_t<3, 4>(L, g, out, ph);
      default: return hipErrorInvalidValue;
    }
  }
#define TILES_CASE(S, M) \
  if (L.storage == S && L.model == M) return levels == 4 ? tiles_t<S, M, 4>(L, g, out, ph) : tiles_t<S, M, 2>(L, g, out, ph);
  TILES_CASE(ST_F32, 0) TILES_CASE(ST_F32, 2) TILES_CASE(ST_F32, 3) TILES_CASE(ST_F32, 4)
  TILES_CASE(ST_F64, 0) TILES_CASE(ST_F64, 2) TILES_CASE(ST_F64, 3) TILES_CASE(ST_F64, 4)
#undef TILES_CASE
  return hipErrorInvalidValue;
}

}  // namespace vlbm
