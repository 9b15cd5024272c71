// HIP kernels (gfx950) around the sweep: static faces, the body's mask and refill,
// init, moments and FP64 diagnostics, gather, conversions and the streaming copy.
// Population placement follows the sweep's in-place AA pattern (vlbm_sweep.hip):
// after an even number of steps f_i(x) sits at slot i of cell x, after an odd number
// at slot opposite(i) of cell x - e_i.
#include "vlbm_device.h"

namespace vlbm {
namespace {

// Population f_i of cell c in the layout of the given parity: its slot and the byte
// offset of the cell that holds it.
template <int D>
__device__ __forceinline__ void pop_place(int parity, int i, unsigned c, const unsigned (&np)[3],
                                          const unsigned (&nm)[3], int& slot, unsigned& cell) {
  slot = (parity == 0) ? i : opposite(i);
  cell = (parity == 0 || i == 0) ? c : ((i & 1) ? nm[(i - 1) >> 1] : np[(i - 1) >> 1]);
}

template <int ST>
__device__ inline void cell_moments3(const Grid& g, const Codec& cd, int parity, unsigned c,
                                     typename Store<ST>::R (&Q)[8]) {
  using S = Store<ST>;
  using T = typename S::T;
  using R = typename S::R;
  const int x = (int)(c % (unsigned)g.nx), y = (int)((c / (unsigned)g.nx) % (unsigned)g.ny);
  const int z = (int)(c / ((unsigned)g.nx * (unsigned)g.ny));
  unsigned np[3], nm[3];
  neighbours<3>(g, x, y, z, c, np, nm);
  const T* F = static_cast<const T*>(g.f);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    R q = R(0);
#pragma unroll
    for (int i = 0; i < 7; ++i) {
      int slot;
      unsigned src;
      pop_place<3>(parity, i, c, np, nm, slot, src);
      q += S::dec(F[(size_t)(k * 7 + slot) * g.stride + src], cd, k * 7 + i);
    }
    Q[k] = q;
  }
}

// f := f^eq(Q) for cell c in the layout of the given parity (D3Q7 ideal).
template <int ST>
__device__ inline void write_feq3(const Grid& g, const Phys& ph, const Codec& cd, int parity, unsigned c,
                                  const typename Store<ST>::R (&Q)[8]) {
  using S = Store<ST>;
  using T = typename S::T;
  using R = typename S::R;
  const int x = (int)(c % (unsigned)g.nx), y = (int)((c / (unsigned)g.nx) % (unsigned)g.ny);
  const int z = (int)(c / ((unsigned)g.nx * (unsigned)g.ny));
  unsigned np[3], nm[3];
  neighbours<3>(g, x, y, z, c, np, nm);
  R Jb[3] = {R(0), R(0), R(0)};
  R P[8][3], Sv[8], dl;
  flux_source<R, 3, 0>(Q, Jb, ph, P, Sv, dl);
  const R wi = R(ph.wi);
  const R w0 = rest_weight<R, 3>(wi);
  T* F = static_cast<T*>(g.f);
#pragma unroll
  for (int k = 0; k < 8; ++k)
#pragma unroll
    for (int i = 0; i < 7; ++i) {
      int slot;
      unsigned dst;
      pop_place<3>(parity, i, c, np, nm, slot, dst);
      F[(size_t)(k * 7 + slot) * g.stride + dst] = S::enc(feq_dir<R, 3>(Q[k], P[k], i, w0, wi), cd, k * 7 + i);
    }
}

// Static faces.  blockIdx.z is the face (2a + side); a thread per node of it.  A node
// on several non-periodic faces is handled by each of them with identical values (the
// x faces by the sweep itself where it can, see fuse_x_faces; their edges with the y
// and z faces still here);
// the cells read (no non-periodic face) and the populations written (face nodes
// only) are disjoint.
template <int ST>
__global__ __launch_bounds__(256) void k_faces(const Grid g, const Phys ph, const Codec cd, int parity,
                                               const Inflow in) {
  using R = typename Store<ST>::R;
  const int f = blockIdx.z, a = f >> 1;
  if (g.bc[f] == 0) return;
  if (a == 0 && fuse_x_faces(g)) return;  // the sweep re-sets these nodes
  const int n[3] = {g.nx, g.ny, g.nz};
  // the two other axes in increasing order, so that consecutive threads walk along x
  // (consecutive addresses) on the y and z faces
  const int a1 = a == 0 ? 1 : 0, a2 = a == 2 ? 1 : 2;
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (long long)n[a1] * n[a2]) return;
  int cc[3];
  cc[a] = (f & 1) ? n[a] - 1 : 0;
  cc[a1] = (int)(t % n[a1]);
  cc[a2] = (int)(t / n[a1]);
  bool inflow = false;
  int ic[3] = {cc[0], cc[1], cc[2]};
  for (int b = 0; b < 3; ++b) {
    if (g.bc[2 * b] == 0) continue;
    if ((cc[b] == 0 && g.bc[2 * b] == 1) || (cc[b] == n[b] - 1 && g.bc[2 * b + 1] == 1)) inflow = true;
    ic[b] = min(max(cc[b], 1), n[b] - 2);
  }
  R Q[8];
  if (inflow) {
#pragma unroll
    for (int k = 0; k < 8; ++k) Q[k] = R(in.q[k]);
  } else {
    cell_moments3<ST>(g, cd, parity, (unsigned)ic[0] + (unsigned)g.nx * ((unsigned)ic[1] + (unsigned)g.ny * ic[2]), Q);
  }
  write_feq3<ST>(g, ph, cd, parity, (unsigned)cc[0] + (unsigned)g.nx * ((unsigned)cc[1] + (unsigned)g.ny * cc[2]),
                 Q);
}

__device__ __forceinline__ bool box_cell(const Body& b, int& x, int& y, int& z) {
  const long long bx = b.box[1] - b.box[0], by = b.box[3] - b.box[2], bz = b.box[5] - b.box[4];
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= bx * by * bz) return false;
  x = b.box[0] + (int)(t % bx);
  y = b.box[2] + (int)((t / bx) % by);
  z = b.box[4] + (int)(t / (bx * by));
  return true;
}

// Mask pass 0 (solid bit at time b.t; the previous solid bit kept as kWasSolid unless
// fresh) and pass 1 (link bits from the neighbours' solid bits; only bits 1..6 of the
// own byte change, so concurrent reads of bit 7 are unaffected).
__global__ __launch_bounds__(256) void k_mask(const Grid g, const Body b, int pass, int fresh) {
  int x, y, z;
  if (!box_cell(b, x, y, z)) return;
  const unsigned c = (unsigned)x + (unsigned)g.nx * ((unsigned)y + (unsigned)g.ny * (unsigned)z);
  const unsigned old = g.mask[c];
  if (pass == 0) {
    unsigned v = body_solid(b, x, y, z, b.t) ? kSolid : 0u;
    if (!fresh && (old & kSolid)) v |= kWasSolid;
    g.mask[c] = (unsigned char)v;
  } else {
    unsigned np[3], nm[3];
    neighbours<3>(g, x, y, z, c, np, nm);
    unsigned v = old & (kSolid | kWasSolid);
#pragma unroll
    for (int i = 1; i < 7; ++i) {
      const unsigned nb = (i & 1) ? np[(i - 1) >> 1] : nm[(i - 1) >> 1];
      if (g.mask[nb] & kSolid) v |= link_bit(i);
    }
    g.mask[c] = (unsigned char)v;
  }
}

// Refill of uncovered cells.  The neighbours read are fluid before and after the
// move, so no cell that is read is also written.
template <int ST>
__global__ __launch_bounds__(256) void k_refill(const Grid g, const Phys ph, const Codec cd, int parity,
                                                const Body b, const Inflow in) {
  using R = typename Store<ST>::R;
  int x, y, z;
  if (!box_cell(b, x, y, z)) return;
  const unsigned c = (unsigned)x + (unsigned)g.nx * ((unsigned)y + (unsigned)g.ny * (unsigned)z);
  const unsigned m = g.mask[c];
  if (!(m & kWasSolid) || (m & kSolid)) return;
  unsigned np[3], nm[3];
  neighbours<3>(g, x, y, z, c, np, nm);
  R Qm[8], Qn[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) Qm[k] = R(0);
  int cnt = 0;
  for (int i = 1; i < 7; ++i) {
    const unsigned nb = (i & 1) ? np[(i - 1) >> 1] : nm[(i - 1) >> 1];
    if (g.mask[nb] & (kSolid | kWasSolid)) continue;
    cell_moments3<ST>(g, cd, parity, nb, Qn);
#pragma unroll
    for (int k = 0; k < 8; ++k) Qm[k] += Qn[k];
    ++cnt;
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) Qm[k] = cnt ? Qm[k] / R(cnt) : R(in.q[k]);
  write_feq3<ST>(g, ph, cd, parity, c, Qm);
}

// ---------------------------------------------------------------------------
// init: f := f^eq(Q), natural layout
// ---------------------------------------------------------------------------
// Every cell by itself, so threads take consecutive cells of the whole lattice (row
// workgroups left lanes idle on rows they do not tile: 190 x 113 x 77 in FP32 113 us, flat
// 74 us).  Two cells per thread in 16-bit storage gained nothing (4.1 ms on 512^3 either way).
template <int ST, int D, int MODEL, typename QT>
__global__ __launch_bounds__(256) void k_init(const Grid g, const Phys ph, const Codec cd,
                                              const QT* __restrict__ Qin) {
  using S = Store<ST>;
  using T = typename S::T;
  using R = typename S::R;
  constexpr int NQ = 2 * D + 1;
  constexpr int K = kNVars<MODEL>;
  const unsigned n = (unsigned)g.nx * (unsigned)g.ny * (unsigned)g.nz;
  const unsigned c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n) return;
  const size_t N = n;
  T* __restrict__ F = static_cast<T*>(g.f);
  R Q[K];
#pragma unroll
  for (int k = 0; k < K; ++k) Q[k] = (R)Qin[(size_t)k * N + c];
  R Jb[3] = {R(0), R(0), R(0)};
  R P[K][3], Sv[K], dl;
  flux_source<R, D, MODEL>(Q, Jb, ph, P, Sv, dl);
  const R wi = R(ph.wi);
  const R w0 = rest_weight<R, D>(wi);
  // Guo's source: the populations' sum is the state minus half its source (the inverse
  // of the sweep's half-source shift); Chai's: the previous source starts as S~(Q)
  const R gs = ph.source == 1 ? R(0.5) : R(0);
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int i = 0; i < NQ; ++i)
      F[pop_index(g, NQ, k, i, c)] =
          S::enc(feq_dir<R, D>(Q[k], P[k], i, w0, wi) - gs * (i == 0 ? w0 : wi) * Sv[k], cd, k * NQ + i);
  if (ph.source == 2 && g.sprev) {
#pragma unroll
    for (int k = 0; k < K; ++k) static_cast<R*>(g.sprev)[(size_t)k * N + c] = Sv[k];
  }
}

// ---------------------------------------------------------------------------
// reductions (FP64)
// ---------------------------------------------------------------------------
// Reduce v[0..n) over the block (slots in maxmask take the max, others the sum) and
// let thread j < n write the block result of slot j to out[j].  All threads call it.
template <int NMAX>
__device__ void block_reduce(double (&v)[NMAX], int n, unsigned maxmask, double* out) {
  __shared__ double sh[kReduceThreads / 64][NMAX];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int j = 0; j < n; ++j) {
    const bool mx = (maxmask >> j) & 1u;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const double o = __shfl_xor(v[j], off);
      v[j] = mx ? fmax(v[j], o) : v[j] + o;
    }
    if (lane == 0) sh[wv][j] = v[j];
  }
  __syncthreads();
  if ((int)threadIdx.x < n) {
    const int j = threadIdx.x;
    const bool mx = (maxmask >> j) & 1u;
    double r = sh[0][j];
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) r = mx ? fmax(r, sh[w][j]) : r + sh[w][j];
    out[j] = r;
  }
}

// Moments and FP64 diagnostics.  out names what is written: the FP64 field, the FP32 field,
// and the FP64 field of B alone for the central divergence where the whole FP64 field is
// not asked for (writing it all and converting it in a second pass took 2.9 ms more on
// 512^3 in FP32 storage).  Bound by HBM: the populations once and the fields written.
// 32-bit cell arithmetic: the 64-bit divisions held 512^3 in FP16 at 8.9 ms (now 4.6 ms,
// 4.9 TB/s) and 256^3 x 26 in FP32 at 6.1 (now 2.9 ms, 5.3 TB/s).  Two cells per thread in
// 16-bit storage took 25 ms (356 VGPRs).
template <int ST, int D, int MODEL>
__global__ __launch_bounds__(kReduceThreads) void k_moments(const Grid g, const Phys ph,
                                                            const Codec cd, int parity, const FieldsOut out,
                                                            double* __restrict__ partial) {
  using S = Store<ST>;
  using T = typename S::T;
  constexpr int NQ = 2 * D + 1;
  constexpr int K = kNVars<MODEL>;
  constexpr int NT = K + 5;
  constexpr bool PK = MODEL == 1 && sizeof(T) == 2;
  constexpr int bx = kBx<MODEL>;
  const T* __restrict__ F = static_cast<const T*>(g.f);
  const unsigned N = (unsigned)g.nx * (unsigned)g.ny * (unsigned)g.nz;
  double acc[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) acc[j] = 0.0;
  for (unsigned c = blockIdx.x * blockDim.x + threadIdx.x; c < N; c += gridDim.x * blockDim.x) {
    auto write = [&](int k, double q) {
      if (out.q64) out.q64[(size_t)k * N + c] = q;
      if (out.q32) out.q32[(size_t)k * N + c] = (float)q;
      if (out.b64 && k >= bx && k < bx + D) out.b64[(size_t)(k - bx) * N + c] = q;
    };
    if (g.mask && (g.mask[c] & kSolid)) {  // inside the body: no fluid state
#pragma unroll
      for (int k = 0; k < K; ++k) write(k, 0.0);
      continue;
    }
    const unsigned row = c / (unsigned)g.nx, x = c - row * (unsigned)g.nx;
    const unsigned z = row / (unsigned)g.ny, y = row - z * (unsigned)g.ny;
    unsigned np[3], nm[3];
    neighbours<D>(g, (int)x, (int)y, (int)z, c, np, nm);
    auto cell_of = [&](int i) {
      return (parity == 0 || i == 0) ? c : ((i & 1) ? nm[(i - 1) >> 1] : np[(i - 1) >> 1]);
    };
    auto slot_of = [&](int i) { return parity == 0 ? i : opposite(i); };
    double Q[K];
    double Jb[3] = {0.0, 0.0, 0.0};
    auto add = [&](int k, int i, double v) {
      Q[k] += v;
      if (k >= bx && k < bx + D && i > 0 && ((i - 1) >> 1) == k - bx) Jb[k - bx] += (i & 1) ? v : -v;
    };
#pragma unroll
    for (int k = 0; k < K; ++k) Q[k] = 0.0;
    if constexpr (PK) {
#pragma unroll
      for (int p = 0; p < K / 2; ++p)
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
          const unsigned v = static_cast<const unsigned*>(g.f)[(size_t)(p * NQ + slot_of(i)) * g.stride + cell_of(i)];
          add(2 * p, i, S::dec64((T)(v & 0xffffu), cd, 2 * p * NQ + i));
          add(2 * p + 1, i, S::dec64((T)(v >> 16), cd, (2 * p + 1) * NQ + i));
        }
    } else {
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int i = 0; i < NQ; ++i)
          add(k, i, S::dec64(F[(size_t)(k * NQ + slot_of(i)) * g.stride + cell_of(i)], cd, k * NQ + i));
    }
    double P[K][3], Sv[K], dl;
    if (ph.source == 1) {
      // Guo's state: sum f + S~/2 by the sweep's two fixed-point iterations
      double q[K];
      flux_source<double, D, MODEL>(Q, Jb, ph, P, Sv, dl);
#pragma unroll
      for (int k = 0; k < K; ++k) q[k] = Q[k] + 0.5 * Sv[k];
      flux_source<double, D, MODEL>(q, Jb, ph, P, Sv, dl);
#pragma unroll
      for (int k = 0; k < K; ++k) Q[k] += 0.5 * Sv[k];
    }
#pragma unroll
    for (int k = 0; k < K; ++k) write(k, Q[k]);
    const bool bad = flux_source<double, D, MODEL>(Q, Jb, ph, P, Sv, dl);
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] += Q[k];
    acc[K] += dl;
    acc[K + 1] += dl * dl;
    acc[K + 2] = fmax(acc[K + 2], fabs(dl));
    acc[K + 4] += bad ? 1.0 : 0.0;
  }
  block_reduce<NT>(acc, NT, 1u << (K + 2), partial + (size_t)blockIdx.x * NT);
}

// Network input of the learned correction (8-variable ideal model): the moments of
// each cell in the storage's compute type, summed over i in order, then as FP32 and
// standardised BF16 (round to nearest even), one cell per thread.
template <int ST, int D>
__global__ __launch_bounds__(256) void k_net_input(const Grid g, const Codec cd, int parity, const MomentsOut mo) {
  using S = Store<ST>;
  using T = typename S::T;
  using R = typename S::R;
  constexpr int NQ = 2 * D + 1, K = 8;
  const T* __restrict__ F = static_cast<const T*>(g.f);
  const size_t N = (size_t)g.nx * g.ny * g.nz;
  const size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= N) return;
  const int x = (int)(c % g.nx), y = (int)((c / g.nx) % g.ny), z = (int)(c / ((size_t)g.nx * g.ny));
  unsigned np[3], nm[3];
  neighbours<D>(g, x, y, z, (unsigned)c, np, nm);
  unsigned h[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    R q = R(0);
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const unsigned src = (parity == 0 || i == 0) ? (unsigned)c : ((i & 1) ? nm[(i - 1) >> 1] : np[(i - 1) >> 1]);
      const int slot = parity == 0 ? i : opposite(i);
      q += S::dec(F[(size_t)(k * NQ + slot) * g.stride + src], cd, k * NQ + i);
    }
    const float xq = (float)q;
    mo.x[(size_t)k * N + c] = xq;
    const unsigned u = __float_as_uint((xq - mo.mean[k]) * mo.istd[k]);
    h[k] = (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
  }
  *reinterpret_cast<uint4*>(mo.act + c * K) =
      make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
}

// Per-step loads on the homogenized body at time b.t (cells of b.box): what the
// homogenized collision moves from the fluid to the body -- force (momentum), torque
// about the body's centre, energy -- and the magnetic flux through its surface,
// 1/2 sum |B . r/|r|| over the one-cell porosity ramp.  The cell's moments change by
// omega_k (Q^_k - Q_k) in the collision; omega_k = 1/tau_k (BGK), the symmetric rate
// (two-rate collisions carry the zeroth moment in the symmetric halves), 1 (RLB).
// partial[block][8] = (F, T, W, flux).
template <int ST>
__global__ __launch_bounds__(kReduceThreads) void k_body_loads(const Grid g, const Phys ph, const Codec cd,
                                                               int parity, const Body b,
                                                               double* __restrict__ partial) {
  using R = typename Store<ST>::R;
  double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  const long long bx = b.box[1] - b.box[0], by = b.box[3] - b.box[2], bz = b.box[5] - b.box[4];
  const long long nb = bx * by * bz;
  for (long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x; t < nb; t += (long long)gridDim.x * blockDim.x) {
    const int x = b.box[0] + (int)(t % bx), y = b.box[2] + (int)((t / bx) % by), z = b.box[4] + (int)(t / (bx * by));
    const HlbmTarget tg{&b, x, y, z, HlbmTarget::near_body(b, x, y, z), ph.s, ph.gm1};
    if (!tg.near) continue;
    double r[3], rr;
    const double phi = tg.rr_minus_R(r, rr);
    if (phi >= 0.5) continue;  // porosity 1: fluid, no exchange
    const unsigned c = (unsigned)x + (unsigned)g.nx * ((unsigned)y + (unsigned)g.ny * (unsigned)z);
    R Qr[8];
    cell_moments3<ST>(g, cd, parity, c, Qr);
    double Q[8], Qh[8];
    for (int k = 0; k < 8; ++k) Q[k] = Qh[k] = (double)Qr[k];
    tg(Qh);
    double om[5];
    for (int k = 1; k < 5; ++k) om[k] = ph.collision == 0 ? ph.omega[k] : (ph.collision == 1 ? ph.omega_s[k] : 1.0);
    const double dM[3] = {om[1] * (Qh[1] - Q[1]), om[2] * (Qh[2] - Q[2]), om[3] * (Qh[3] - Q[3])};
    acc[0] -= dM[0];
    acc[1] -= dM[1];
    acc[2] -= dM[2];
    acc[3] -= r[1] * dM[2] - r[2] * dM[1];
    acc[4] -= r[2] * dM[0] - r[0] * dM[2];
    acc[5] -= r[0] * dM[1] - r[1] * dM[0];
    acc[6] -= om[4] * (Qh[4] - Q[4]);
    if (phi > -0.5 && rr > 0.0) acc[7] += 0.5 * fabs(Q[5] * r[0] + Q[6] * r[1] + Q[7] * r[2]) / rr;
  }
  block_reduce<8>(acc, 8, 0u, partial + (size_t)blockIdx.x * 8);
}

// Bf: the FP64 field of B, [D][N]
template <int D>
__global__ __launch_bounds__(kReduceThreads) void k_divc(const Grid g, const double* __restrict__ Bf,
                                                         double* __restrict__ partial) {
  const unsigned N = (unsigned)g.nx * (unsigned)g.ny * (unsigned)g.nz;
  double acc[1] = {0.0};
  for (unsigned c = blockIdx.x * blockDim.x + threadIdx.x; c < N; c += gridDim.x * blockDim.x) {
    const unsigned row = c / (unsigned)g.nx, x = c - row * (unsigned)g.nx;
    const unsigned z = row / (unsigned)g.ny, y = row - z * (unsigned)g.ny;
    unsigned np[3], nm[3];
    neighbours<D>(g, (int)x, (int)y, (int)z, c, np, nm);
    double dv = 0.0;
#pragma unroll
    for (int a = 0; a < D; ++a) dv += 0.5 * (Bf[(size_t)a * N + np[a]] - Bf[(size_t)a * N + nm[a]]);
    acc[0] += dv * dv;
  }
  block_reduce<1>(acc, 1, 0u, partial + blockIdx.x);
}

// One workgroup per slot: slot j < n reduces partial[.][j] into out[j] (thread t takes
// workgroups t, t + 256, ... in that order); slot n, if partial2 is given, the sums
// partial2[.] into *out2, which may be one of out's places.  (All slots in one workgroup, their accumulators indexed at run time, took
// 8-20 us.)
__global__ __launch_bounds__(kReduceThreads) void k_reduce(int n, const double* __restrict__ partial,
                                                           int nblk, MaxMask maxmask, double* __restrict__ out,
                                                           const double* __restrict__ partial2,
                                                           double* __restrict__ out2) {
  const int j = blockIdx.x;
  if (partial2 && out + j == out2) return;  // the other sums' place
  const bool second = j == n, mx = !second && maxmask.has(j);
  const double* p = second ? partial2 : partial + j;
  const size_t stride = second ? 1 : (size_t)n;
  double acc[1] = {mx ? -INFINITY : 0.0};
  for (int b = threadIdx.x; b < nblk; b += blockDim.x) {
    const double v = p[(size_t)b * stride];
    acc[0] = mx ? fmax(acc[0], v) : acc[0] + v;
  }
  block_reduce<1>(acc, 1, mx ? 1u : 0u, second ? out2 : out + j);
}

// Statistics of a field Q [K][N]: per variable k (blockIdx.y) and workgroup the sum, the
// largest value and the largest negated value, partial[(b K + k) 3 + 0..2].  One variable
// per workgroup, so that the accumulators stay in registers (all K in every thread, indexed
// at run time, read 4.3 GB in 3.4 ms).
template <typename QT>
__global__ __launch_bounds__(kReduceThreads) void k_field_stats(const QT* __restrict__ Q, unsigned N,
                                                                double* __restrict__ partial) {
  const int k = blockIdx.y, K = gridDim.y;
  const QT* __restrict__ q = Q + (size_t)k * N;
  double sum = 0.0, hi = -INFINITY, lo = -INFINITY;
#pragma unroll 4
  for (unsigned c = blockIdx.x * blockDim.x + threadIdx.x; c < N; c += gridDim.x * blockDim.x) {
    const double v = (double)q[c];
    sum += v;
    hi = fmax(hi, v);
    lo = fmax(lo, -v);
  }
  double acc[3] = {sum, hi, lo};
  block_reduce<3>(acc, 3, 6u, partial + ((size_t)blockIdx.x * K + k) * 3);
}

template <int ST, int D>
__global__ void k_gather(const Grid g, const Codec cd, int parity, int K,
                         const long long* __restrict__ cells, long long n, double* __restrict__ out) {
  using S = Store<ST>;
  using T = typename S::T;
  constexpr int NQ = 2 * D + 1;
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * K * NQ) return;
  const int i = (int)(t % NQ);
  const int k = (int)((t / NQ) % K);
  const long long c = cells[t / ((long long)NQ * K)];
  const int x = (int)(c % g.nx);
  const int y = (int)((c / g.nx) % g.ny);
  const int z = (int)(c / ((long long)g.nx * g.ny));
  unsigned np[3], nm[3];
  neighbours<D>(g, x, y, z, (unsigned)c, np, nm);
  const unsigned src = (parity == 0 || i == 0) ? (unsigned)c : ((i & 1) ? nm[(i - 1) >> 1] : np[(i - 1) >> 1]);
  const int slot = parity == 0 ? i : opposite(i);
  const T* F = static_cast<const T*>(g.f);
  out[t] = S::dec64(F[pop_index(g, NQ, k, slot, src)], cd, k * NQ + i);
}

// One 16-byte element per thread and no grid-stride loop: the fastest plain copy
// form measured on gfx950 (a grid-stride loop over 8192 blocks reaches ~77 % of it).
__global__ __launch_bounds__(256) void k_copy(uint4* __restrict__ dst, const uint4* __restrict__ src,
                                              size_t n) {
  const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) dst[t] = src[t];
}

// ---------------------------------------------------------------------------
// launch helpers
// ---------------------------------------------------------------------------

template <int ST>
hipError_t boundary_t(const Launch& L, const Grid& g, const Phys& ph, const Codec& cd, int parity,
                      const Body* b, const Inflow* in, int what) {
  if (what == 0) {  // faces
    const long long area = std::max({(long long)g.ny * g.nz, (long long)g.nx * g.nz, (long long)g.nx * g.ny});
    hipLaunchKernelGGL((k_faces<ST>), dim3((unsigned)((area + 255) / 256), 1, 6), dim3(256), 0, L.stream, g, ph,
                       cd, parity, *in);
  } else {  // refill
    const long long n = (long long)(b->box[1] - b->box[0]) * (b->box[3] - b->box[2]) * (b->box[5] - b->box[4]);
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL((k_refill<ST>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, L.stream, g, ph, cd,
                       parity, *b, *in);
  }
  return hipGetLastError();
}

hipError_t boundary(const Launch& L, const Grid& g, const Phys& ph, const Codec& cd, int parity, const Body* b,
                    const Inflow* in, int what) {
  if (L.dim != 3 || L.model != 0) return hipErrorInvalidValue;
  switch (L.storage) {
    case ST_F64: return boundary_t<ST_F64>(L, g, ph, cd, parity, b, in, what);
    case ST_F32: return boundary_t<ST_F32>(L, g, ph, cd, parity, b, in, what);
    case ST_F16: return boundary_t<ST_F16>(L, g, ph, cd, parity, b, in, what);
    case ST_BF16: return boundary_t<ST_BF16>(L, g, ph, cd, parity, b, in, what);
    default: return hipErrorInvalidValue;
  }
}

template <int ST, int D, int MODEL>
hipError_t init_t(const Launch& L, const Grid& g, const Phys& ph, const Codec& cd, const void* Q,
                  int f32) {
  const long long n = (long long)g.nx * g.ny * g.nz;
  const dim3 grd((unsigned)((n + 255) / 256)), blk(256);
  if (f32)
    hipLaunchKernelGGL((k_init<ST, D, MODEL, float>), grd, blk, 0, L.stream, g, ph, cd,
                       static_cast<const float*>(Q));
  else
    hipLaunchKernelGGL((k_init<ST, D, MODEL, double>), grd, blk, 0, L.stream, g, ph, cd,
                       static_cast<const double*>(Q));
  return hipGetLastError();
}

template <int ST, int D, int MODEL>
hipError_t moments_t(const Launch& L, const Grid& g, const Phys& ph, const Codec& cd, int parity,
                     const FieldsOut& out, double* partial, int nblk) {
  hipLaunchKernelGGL((k_moments<ST, D, MODEL>), dim3(nblk), dim3(kReduceThreads), 0, L.stream, g,
                     ph, cd, parity, out, partial);
  return hipGetLastError();
}

template <int ST>
hipError_t gather_t(const Launch& L, const Grid& g, const Codec& cd, int parity, int K,
                    const long long* cells, long long n, double* out) {
  const long long tot = n * K * (2 * L.dim + 1);
  const dim3 grd((unsigned)((tot + 255) / 256)), blk(256);
  if (L.dim == 2)
    hipLaunchKernelGGL((k_gather<ST, 2>), grd, blk, 0, L.stream, g, cd, parity, K, cells, n, out);
  else
    hipLaunchKernelGGL((k_gather<ST, 3>), grd, blk, 0, L.stream, g, cd, parity, K, cells, n, out);
  return hipGetLastError();
}

template <int ST, int D, int M>
struct InitFn {
  static hipError_t run(const Launch& L, const Grid& g, const Phys& ph, const Codec& cd,
                        const void* Q, int f32) {
    return init_t<ST, D, M>(L, g, ph, cd, Q, f32);
  }
};
template <int ST, int D, int M>
struct MomentsFn {
  static hipError_t run(const Launch& L, const Grid& g, const Phys& ph, const Codec& cd, int par,
                        const FieldsOut& out, double* partial, int nblk) {
    return moments_t<ST, D, M>(L, g, ph, cd, par, out, partial, nblk);
  }
};

}  // namespace

hipError_t launch_net_input(const Launch& L, const Grid& g, const Codec& cd, int parity, const MomentsOut& mo) {
  const size_t N = (size_t)g.nx * g.ny * g.nz;
  const dim3 grd((unsigned)((N + 255) / 256)), blk(256);
  switch (L.storage * 2 + (L.dim - 2)) {
#define NI_CASE(ST, D)                                                                               \
  case ST * 2 + (D - 2):                                                                             \
    hipLaunchKernelGGL((k_net_input<ST, D>), grd, blk, 0, L.stream, g, cd, parity, mo);              \
    return hipGetLastError();
    NI_CASE(ST_F64, 2) NI_CASE(ST_F64, 3) NI_CASE(ST_F32, 2) NI_CASE(ST_F32, 3)
    NI_CASE(ST_F16, 2) NI_CASE(ST_F16, 3) NI_CASE(ST_BF16, 2) NI_CASE(ST_BF16, 3)
#undef NI_CASE
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_init(const Launch& L, const Grid& g, const Phys& ph, const Codec& cd,
                       const void* Q, int q_is_f32) {
  return dispatch<InitFn>(L, g, ph, cd, Q, q_is_f32);
}

hipError_t launch_faces(const Launch& L, const Grid& g, const Phys& ph, const Codec& cd, int parity,
                        const Inflow& in) {
  return boundary(L, g, ph, cd, parity, nullptr, &in, 0);
}

hipError_t launch_refill(const Launch& L, const Grid& g, const Phys& ph, const Codec& cd, int parity,
                         const Body& b, const Inflow& in) {
  if (!g.mask) return hipErrorInvalidValue;
  return boundary(L, g, ph, cd, parity, &b, &in, 2);
}

hipError_t launch_mask(const Launch& L, const Grid& g, const Body& b, int pass, int fresh) {
  if (!g.mask) return hipErrorInvalidValue;
  const long long n = (long long)(b.box[1] - b.box[0]) * (b.box[3] - b.box[2]) * (b.box[5] - b.box[4]);
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_mask, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, L.stream, g, b, pass, fresh);
  return hipGetLastError();
}

hipError_t launch_moments(const Launch& L, const Grid& g, const Phys& ph, const Codec& cd,
                          int parity, const FieldsOut& out, double* partial, int nblk) {
  return dispatch<MomentsFn>(L, g, ph, cd, parity, out, partial, nblk);
}

hipError_t launch_divc(const Launch& L, const Grid& g, const double* B, double* partial, int nblk) {
  if (L.dim == 2)
    hipLaunchKernelGGL((k_divc<2>), dim3(nblk), dim3(kReduceThreads), 0, L.stream, g, B, partial);
  else
    hipLaunchKernelGGL((k_divc<3>), dim3(nblk), dim3(kReduceThreads), 0, L.stream, g, B, partial);
  return hipGetLastError();
}

hipError_t launch_body_loads(const Launch& L, const Grid& g, const Phys& ph, const Codec& cd, int parity,
                             const Body& b, double* partial, int nblk) {
  if (L.dim != 3 || L.model != 0) return hipErrorInvalidValue;
  const dim3 grd(nblk), blk(kReduceThreads);
  switch (L.storage) {
    case ST_F64: hipLaunchKernelGGL(k_body_loads<ST_F64>, grd, blk, 0, L.stream, g, ph, cd, parity, b, partial); break;
    case ST_F32: hipLaunchKernelGGL(k_body_loads<ST_F32>, grd, blk, 0, L.stream, g, ph, cd, parity, b, partial); break;
    case ST_F16: hipLaunchKernelGGL(k_body_loads<ST_F16>, grd, blk, 0, L.stream, g, ph, cd, parity, b, partial); break;
    case ST_BF16: hipLaunchKernelGGL(k_body_loads<ST_BF16>, grd, blk, 0, L.stream, g, ph, cd, parity, b, partial); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_reduce(const Launch& L, int n, const double* partial, int nblk, MaxMask maxmask,
                         double* out, const double* partial2, double* out2) {
  if (n > 128) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_reduce, dim3((unsigned)(n + (partial2 ? 1 : 0))), dim3(kReduceThreads), 0, L.stream, n, partial,
                     nblk, maxmask, out, partial2, out2);
  return hipGetLastError();
}

hipError_t launch_gather(const Launch& L, const Grid& g, const Codec& cd, int parity, int K,
                         const long long* cells, long long n, double* out) {
  switch (L.storage) {
    case ST_F64: return gather_t<ST_F64>(L, g, cd, parity, K, cells, n, out);
    case ST_F32: return gather_t<ST_F32>(L, g, cd, parity, K, cells, n, out);
    case ST_F16: return gather_t<ST_F16>(L, g, cd, parity, K, cells, n, out);
    case ST_BF16: return gather_t<ST_BF16>(L, g, cd, parity, K, cells, n, out);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_field_stats(const Launch& L, long long N, int K, const void* Q, int q_is_f32, double* partial,
                              int nblk, double* out) {
  const dim3 grd((unsigned)nblk, (unsigned)K);
  if (q_is_f32)
    hipLaunchKernelGGL((k_field_stats<float>), grd, dim3(kReduceThreads), 0, L.stream, static_cast<const float*>(Q),
                       (unsigned)N, partial);
  else
    hipLaunchKernelGGL((k_field_stats<double>), grd, dim3(kReduceThreads), 0, L.stream, static_cast<const double*>(Q),
                       (unsigned)N, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  MaxMask m;
  for (int k = 0; k < K; ++k) m.add(3 * k + 1), m.add(3 * k + 2);
  return launch_reduce(L, 3 * K, partial, nblk, m, out);
}

hipError_t launch_copy(hipStream_t s, void* dst, const void* src, size_t bytes) {
  const size_t n = bytes / 16;
  const size_t blocks = (n + 255) / 256;
  if (blocks == 0) return hipSuccess;
  if (blocks > 0x7fffffffULL) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_copy, dim3((unsigned)blocks), dim3(256), 0, s, static_cast<uint4*>(dst),
                     static_cast<const uint4*>(src), n);
  return hipGetLastError();
}

}  // namespace vlbm
