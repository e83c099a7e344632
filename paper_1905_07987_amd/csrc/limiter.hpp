// A-posteriori subcell limiter for the Euler equations (ExaHyPE paper,
// Sec. 3.5; the FV, limiter and projection kernels of Table 1; the hybrid
// ADER-DG/FV status stencil of Fig. 2).  A limited step on the device:
//   prepare   u^n copied, the previous status kept, the range of each
//             cell's subcell averages at t^n (FV cells: their own FV data);
//   (the unlimited ADER-DG step in place: the candidate)
//   detect    physical admissibility at every node and subcell average of
//             the candidate, then the relaxed discrete maximum principle;
//   classify  troubled (3), FV as a neighbour of a troubled cell (2), DG
//             with an FV face (1), DG (0); FV cells and DG cells with an FV
//             face are appended to two lists;
//   fv        MUSCL-Hancock with minmod on the (2N+1)^d subcells of each FV
//             cell from the subcell averages at t^n, projected back to the
//             DG space; the fluxes through the cell's faces are kept as
//             face-node values for the DG neighbours;
//   faces     a DG cell with an FV face exchanges the Rusanov flux of that
//             face in its update for the FV one (what leaves one cell
//             enters the other).
// Readings where the paper gives no formula: subcell averages are exact
// averages of the nodal polynomial; the way back is their least-squares
// inverse; the DMP range is the cell's and its face neighbours' subcell
// averages at t^n widened by max(1e-4, 1e-3 (max - min)); a subcell whose
// extrapolated or half-step values are not admissible uses its average on
// all faces; ghost subcells beyond a wall or outflow face mirror the inside
// ones (the wall reverses the normal momentum); FV cells keep their subcell
// averages from step to step and a cell returns to DG once its candidate
// passes both tests.
#pragma once

namespace adg {

template <class PDE>
struct LimiterPDE {
  static constexpr bool value = false;
};
template <int D>
struct LimiterPDE<Euler<D>> {
  static constexpr bool value = true;
};

template <class PDE, int N>
struct GeoLim {
  static constexpr int DIM = PDE::DIM, NV = PDE::NV, n = N + 1, m = 2 * N + 1;
  static constexpr int S = ipow(n, DIM), F = ipow(n, DIM - 1);
  static constexpr int NS = ipow(m, DIM);
  static constexpr int EB = m + 4, NB = ipow(EB, DIM);  // subcells of the cell and two ghost layers
  static constexpr int EC = m + 2, NC = ipow(EC, DIM);  // subcells whose face values are moved
  // threads of the FV kernel: its phases in one round each where that fits
  // (3-D N = 3: 720 lines along x, 729 subcells with moved faces)
  static constexpr int BLOCK = DIM == 2 ? 256 : (N == 3 ? 768 : (N == 2 ? 512 : 256));
  static constexpr int VPT = (NS + BLOCK - 1) / BLOCK;  // subcells per thread in the update
  static constexpr int PPT = (NB + BLOCK - 1) / BLOCK;  // box positions per thread
  static constexpr int NOFF = ipow(3, DIM);             // offsets of the cell and its neighbours
  static constexpr int NFC = ipow(m, DIM - 1) * (m + 1);  // subfaces normal to one axis
  // LDS of the FV kernel (doubles).  REG_A: the projection along x, then the
  // subcell box, then the fit's first stages.  REG_B: (3-D) the projection
  // along y, then the half-step corrections and every subface's flux.
  static constexpr int T1 = NV * ipow(3, DIM - 1) * ipow(n, DIM - 1) * EB;
  static constexpr int T2 = DIM == 3 ? NV * 3 * n * EB * EB : 0;
  static constexpr int FIT = NV * (NS + ipow(m, DIM - 1) * n) + 2 * DIM * NV * ipow(m, DIM - 2) * n;
  static constexpr int REG_A = cmax(T1, cmax(NV * NB, FIT));
  static constexpr int REG_B = cmax(T2, NV * (NC + DIM * NFC));
  static constexpr int FV_D = REG_A + REG_B;
  static constexpr bool built = LimiterPDE<PDE>::value && N <= (DIM == 2 ? 7 : 3);
  // waves per SIMD of the register budget, blocks of the FV kernel per
  // compute unit, and its persistent grid
  static constexpr int FV_WAVES = DIM == 3 && N >= 2 ? (N == 3 ? 3 : 2) : 3;
  static constexpr int FV_BPC = cmax(1, cmin(FV_WAVES * 256 / BLOCK, (160 * 1024) / (FV_D * 8 + NC + 1024)));
  static constexpr int FV_GRID = 256 * FV_BPC;
};

template <int DIM>
__device__ __forceinline__ void lim_multi(int idx, int e, int (&x)[3]) {
  x[0] = idx % e;
  x[1] = (idx / e) % e;
  x[2] = DIM == 3 ? idx / (e * e) : 0;
}

// face neighbour along d on side s (-1, +1); -1 on a non-periodic boundary
template <int DIM>
__device__ __forceinline__ long long lim_neighbour(const KArgs& a, long long c, int d, int s) {
  const int C0 = a.cells[0], C1 = a.cells[1];
  int cc[3] = {(int)(c % C0), (int)((c / C0) % C1), DIM == 3 ? (int)(c / ((long long)C0 * C1)) : 0};
  int to = cc[d] + s;
  if (to < 0 || to >= a.cells[d]) {
    if (a.bc[2 * d + (s > 0)] != ADG_BC_PERIODIC) return -1;
    to = (to + a.cells[d]) % a.cells[d];
  }
  cc[d] = to;
  return cc[0] + (long long)C0 * (cc[1] + (long long)C1 * cc[2]);
}

__device__ __forceinline__ void lim_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Per-wave LDS of the prepare and detect kernels: one group of variables'
// nodal values and the contraction stages of the projection onto the
// subcells (the last stage is evaluated in registers, one column of subcells
// per lane).  Region A holds the nodal values, later the second stage
// (3-D); region B the first stage.  The variables go in two groups, so a
// wave needs half the LDS and more waves share a CU.  The subcell averages
// of the basis, LimConst<n>::A, are compile-time constants.
template <class PDE, int N>
struct GeoLimW {
  using GL = GeoLim<PDE, N>;
  static constexpr int WPB = 4;                   // cells (waves) per block
  static constexpr int VG = (GL::NV + 1) / 2;     // variables of the first group
  static constexpr int P1 = VG * GL::m * ipow(GL::n, GL::DIM - 1);
  static constexpr int P2 = GL::DIM == 3 ? VG * GL::m * GL::m * GL::n : 0;
  static constexpr int RA = cmax(VG * GL::S, P2), RB = P1;
  static constexpr int RN = (GL::NV - VG) * GL::S;  // nodal values of the second group
  static constexpr int PW = RA + RB + RN;
  // columns of subcells along the last axis: one per lane
  static constexpr int LAST = ipow(GL::m, GL::DIM - 1);
  static_assert(LAST <= 64, "one column of subcells per lane");
};

// The leading stages for NVS variables, one line per lane and step: along x
// (nodal values in A, [v][kz][ky][kx], to B, [v][kz][ky][sx]); in 3-D then
// along y (B to A, [v][kz][sy][sx]).
template <class PDE, int N, int NVS>
__device__ __forceinline__ void lim_stages_wave(const double* src, double* ra, double* rb, int lane) {
  using GL = GeoLim<PDE, N>;
  using LC = LimConst<GL::n>;
  constexpr int n = GL::n, m = GL::m;
  constexpr int L1 = NVS * ipow(n, GL::DIM - 1);
  for (int line = lane; line < L1; line += 64) {
    double in[n];
#pragma unroll
    for (int k = 0; k < n; ++k) in[k] = src[line * n + k];
#pragma unroll
    for (int s = 0; s < m; ++s) {
      double acc = 0.0;
#pragma unroll
      for (int k = 0; k < n; ++k) acc += LC::A[s][k] * in[k];
      rb[line * m + s] = acc;
    }
  }
  lim_wave_sync();
  if constexpr (GL::DIM == 3) {
    constexpr int L2 = NVS * n * m;
    for (int line = lane; line < L2; line += 64) {
      const int sx = line % m, vk = line / m;  // vk = v n + kz
      double in[n];
#pragma unroll
      for (int k = 0; k < n; ++k) in[k] = rb[(vk * n + k) * m + sx];
#pragma unroll
      for (int s = 0; s < m; ++s) {
        double acc = 0.0;
#pragma unroll
        for (int k = 0; k < n; ++k) acc += LC::A[s][k] * in[k];
        ra[(vk * m + s) * m + sx] = acc;
      }
    }
    lim_wave_sync();
  }
}

// Variables V0 .. V0 + NVS - 1 of a cell through the projection, from
// their nodal values at src (LDS, [v][S]): out[V0 + v][j] = the average of
// variable V0 + v over the j-th subcell of this lane's column (subcell index
// lane + j m^(dim-1)), for lanes below the column count.
template <class PDE, int N, int V0, int NVS>
__device__ __forceinline__ void lim_group_wave(const double* src, double* ra, double* rb, int lane,
                                               double (&out)[PDE::NV][2 * N + 1]) {
  using GL = GeoLim<PDE, N>;
  using LC = LimConst<GL::n>;
  constexpr int n = GL::n, m = GL::m;
  lim_stages_wave<PDE, N, NVS>(src, ra, rb, lane);
  if (lane < GeoLimW<PDE, N>::LAST) {
#pragma unroll
    for (int v = 0; v < NVS; ++v) {
      double in[n];
#pragma unroll
      for (int k = 0; k < n; ++k)
        in[k] = GL::DIM == 2 ? rb[(v * n + k) * m + lane] : ra[(v * n + k) * m * m + lane];
#pragma unroll
      for (int j = 0; j < m; ++j) {
        double acc = 0.0;
#pragma unroll
        for (int k = 0; k < n; ++k) acc += LC::A[j][k] * in[k];
        out[V0 + v][j] = acc;
      }
    }
  }
  lim_wave_sync();  // the next group overwrites the stages
}

// The cell's nodal values from registers (lane k < S: node k) to the wave's
// LDS: the first group where the projection's first stage reads it, the
// second group in a region of its own.
template <class PDE, int N>
__device__ __forceinline__ void lim_stage_nodes(const double (&x)[PDE::NV], double* ra, double* rn, int lane) {
  constexpr int S = GeoLim<PDE, N>::S, VG = GeoLimW<PDE, N>::VG;
  if (lane < S) {
#pragma unroll
    for (int v = 0; v < PDE::NV; ++v) (v < VG ? ra + v * S : rn + (v - VG) * S)[lane] = x[v];
  }
  lim_wave_sync();
}

__device__ __forceinline__ double lim_wave_min(double x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x = fmin(x, __shfl_xor(x, off, 64));
  return x;
}
__device__ __forceinline__ double lim_wave_max(double x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x = fmax(x, __shfl_xor(x, off, 64));
  return x;
}

// PDE::admissible without its division where the sign of the pressure is
// clear from rho E - |j|^2 / 2 (the same answer: the two differ by rounding).
// FIN: with the test for finite values; without it the answer for values that
// are not finite is open.
template <class PDE, bool FIN = true>
__device__ __forceinline__ bool lim_admissible(const double* q, const PdeConsts& pc) {
  constexpr int NV = PDE::NV, DIM = PDE::DIM;
  bool fin = true;
  if constexpr (FIN) {
#pragma unroll
    for (int v = 0; v < NV; ++v) fin = fin && finite_val(q[v]);
  }
  double jj = 0.0;
#pragma unroll
  for (int a = 0; a < DIM; ++a) jj += q[1 + a] * q[1 + a];
  const double rE = q[0] * q[NV - 1], t = rE - 0.5 * jj;
  if (fin && q[0] > 0.0 && !(fabs(t) > 1e-12 * fabs(rE))) return PDE::admissible(q, q, pc);
  return fin && q[0] > 0.0 && t > 0.0;
}

// The prepare and detect kernels issue every global load of a cell at once
// (all nodal values into registers, and in detect the DMP ranges, one
// (variable, cell) per lane) before the chain of dependent LDS stages of
// the projection, so that a cell waits for one HBM round trip instead of
// one per variable group and neighbour.
template <class PDE, int N>
struct GeoLimSeq {
  static unsigned grid(long long ncells) {
    return (unsigned)((ncells + GeoLimW<PDE, N>::WPB - 1) / GeoLimW<PDE, N>::WPB);
  }
};

// nodal values of cell c (lane k < S: node k), zero past the grid
template <class PDE, int N>
__device__ __forceinline__ void lim_load_nodes(const double* __restrict__ Q, long long c, long long ncells, int lane,
                                               double (&x)[PDE::NV]) {
  constexpr int NV = PDE::NV, S = GeoLim<PDE, N>::S;
  const bool ok = c < ncells && lane < S;
  const long long cl = ok ? c : 0;
#pragma unroll
  for (int v = 0; v < NV; ++v) x[v] = ok ? Q[(cl * NV + v) * S + lane] : 0.0;
}

// The range of the subcell averages at t^n of every cell, the status kept and
// (w.copy) u^n copied, a wave per cell.  With w.reuse the cells of status 0
// have theirs from the previous step's detect, and a wave looks through
// lim_cells_per_wave cells for others.  (96^3 cells, N = 3: 0.16 ms; 0.92 ms
// with a wave per cell and the copy of u^n, which the predictor, reading u^n
// anyway, now writes at no cost that shows.)  Block 0 clears the counters of the step.

// Cells a wave looks through where most need nothing: 16, fewer on meshes
// that leave the chip idle then (81^2 cells, N = 5: 39 us with 16, the FV
// cells of a wave one after the other).  The wave of index i takes cells i,
// i + W, i + 2 W, ... of the W waves, since FV cells lie in clusters.
inline int lim_cells_per_wave(long long ncells) {
  const long long p = ncells / 16384;
  return p < 1 ? 1 : (p > 16 ? 16 : (int)p);
}

// What prepare does for cell c, of status st at t^n, on one wave: u^n copied
// (w.copy), the range of its subcell averages into lohi.
template <class PDE, int N>
__device__ __forceinline__ void lim_prepare_cell(const KArgs& a, const double* __restrict__ Q,
                                                 const double* __restrict__ sub_in, const LimWork& w, double* lohi,
                                                 long long c, int st, double* ra, int lane) {
  using GL = GeoLim<PDE, N>;
  using GW = GeoLimW<PDE, N>;
  constexpr int NV = GL::NV, S = GL::S, NS = GL::NS, m = GL::m;
  double* rb = ra + GW::RA;
  double* rn = rb + GW::RB;
  double x[NV];
  lim_load_nodes<PDE, N>(Q, c, a.ncells, lane, x);
  if (w.copy && lane < S)
#pragma unroll
    for (int v = 0; v < NV; ++v) w.Qold[(c * NV + v) * S + lane] = x[v];
  if (w.reuse && st == 0) return;
  double lo[NV], hi[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    lo[v] = INFINITY;
    hi[v] = -INFINITY;
  }
  if (st >= 2) {
    for (int s = lane; s < NS; s += 64)
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const double y = sub_in[(c * NV + v) * NS + s];
        lo[v] = fmin(lo[v], y);
        hi[v] = fmax(hi[v], y);
      }
  } else {
    lim_stage_nodes<PDE, N>(x, ra, rn, lane);
    double q[NV][m];
    lim_group_wave<PDE, N, 0, GW::VG>(ra, ra, rb, lane, q);
    lim_group_wave<PDE, N, GW::VG, NV - GW::VG>(rn, ra, rb, lane, q);
    if (lane < GW::LAST)
#pragma unroll
      for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int j = 0; j < m; ++j) {
          lo[v] = fmin(lo[v], q[v][j]);
          hi[v] = fmax(hi[v], q[v][j]);
        }
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const double l = lim_wave_min(lo[v]), h = lim_wave_max(hi[v]);
    if (lane == 0) {
      lohi[(c * NV + v) * 2] = l;
      lohi[(c * NV + v) * 2 + 1] = h;
    }
  }
}

// ONE: a wave per cell (per == 1), without the loop, out of which the
// projection's constants are moved into scalar registers and spilled (2-D N =
// 7, 256 cells: 7.6 us, 12.1 us with the loop).
template <class PDE, int N, bool ONE>
__global__ void __launch_bounds__(256)
lim_prepare_kernel(const KArgs a, const double* __restrict__ Q, const double* __restrict__ sub_in,
                   const uint8_t* __restrict__ status, const LimWork w, int per) {
  using GW = GeoLimW<PDE, N>;
  constexpr int NV = GeoLim<PDE, N>::NV;
  __shared__ double buf[GW::WPB][GW::PW];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if (blockIdx.x == 0 && tid < 4) w.counters[tid] = 0;
  const long long first = (long long)blockIdx.x * GW::WPB + wv;
  double* const lohi = w.lohi2 + *w.parity * (a.ncells * (NV * 2));
  if constexpr (ONE) {
    if (first >= a.ncells) return;
    const uint8_t st = status[first];
    if (lane == 0) w.st_prev[first] = st;
    if (!w.reuse || w.copy || st != 0)
      lim_prepare_cell<PDE, N>(a, Q, sub_in, w, lohi, first, st, buf[wv], lane);
  } else {
    const long long waves = (a.ncells + per - 1) / per;
    if (first >= waves) return;
    uint8_t mine = 0;  // lane i: status of the wave's cell i
    const long long mc = first + lane * waves;
    if (lane < per && mc < a.ncells) {
      mine = status[mc];
      w.st_prev[mc] = mine;
    }
    unsigned long long todo = __ballot(lane < per && mc < a.ncells && (!w.reuse || w.copy || mine != 0));
    while (todo) {
      const int i = __ffsll(todo) - 1;
      todo &= todo - 1;
      lim_prepare_cell<PDE, N>(a, Q, sub_in, w, lohi, first + i * waves, __shfl((int)mine, i, 64), buf[wv], lane);
    }
  }
}

// The DMP ranges of cell c and its face neighbours, one (cell, variable)
// per lane: lane v 8 + j holds (lo, hi) of variable v of cell j (j = 0 the
// cell itself, 1 .. 2 dim its face neighbours; an empty range past a
// non-periodic boundary and on the spare lanes).
template <class PDE, int N>
__device__ __forceinline__ void lim_load_ranges(const KArgs& a, const double* lohi, long long c, int lane,
                                                double& lo, double& hi) {
  constexpr int DIM = PDE::DIM, NV = PDE::NV;
  static_assert(NV * 8 <= 64 && 2 * DIM + 1 <= 8, "one lane per (variable, cell)");
  const int v = lane >> 3, j = lane & 7;
  long long o = -1;
  if (c < a.ncells && v < NV && j <= 2 * DIM)
    o = j == 0 ? c : lim_neighbour<DIM>(a, c, (j - 1) >> 1, ((j - 1) & 1) ? 1 : -1);
  lo = INFINITY;
  hi = -INFINITY;
  if (o >= 0) {
    lo = lohi[(o * NV + v) * 2];
    hi = lohi[(o * NV + v) * 2 + 1];
  }
}

// Tests of a lane's column of subcell averages qv[NV][m]: their range (l, h)
// per quantity, and whether every one is admissible.  The sign of the pressure
// is that of rho E - |j|^2 / 2 where that is clear, else PDE::admissible
// decides, subcell by subcell.  Finite values are the nodes' test: averages
// of finite nodes are finite.
template <class PDE, int m>
__device__ __forceinline__ bool lim_column(const KArgs& a, const double (&qv)[PDE::NV][m], double (&l)[PDE::NV],
                                           double (&h)[PDE::NV]) {
  constexpr int NV = PDE::NV, DIM = PDE::DIM;
  double clear = INFINITY;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    l[v] = h[v] = qv[v][0];
#pragma unroll
    for (int j = 1; j < m; ++j) {
      l[v] = fmin(l[v], qv[v][j]);
      h[v] = fmax(h[v], qv[v][j]);
    }
  }
#pragma unroll
  for (int j = 0; j < m; ++j) {
    double jj = 0.0;
#pragma unroll
    for (int d = 0; d < DIM; ++d) jj += qv[1 + d][j] * qv[1 + d][j];
    const double rE = qv[0][j] * qv[NV - 1][j];
    clear = fmin(clear, (rE - 0.5 * jj) - 1e-12 * rE);
  }
  if (l[0] > 0.0 && l[NV - 1] > 0.0 && clear > 0.0) return true;
  bool ok = true;
#pragma unroll
  for (int j = 0; j < m; ++j) {
    double q[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) q[v] = qv[v][j];
    ok = ok && PDE::admissible(q, q, a.pde);
  }
  return ok;
}

// One wave per cell: is the candidate troubled?  (w.store_next: also the
// range of the candidate's subcell averages, as prepare computes it, for
// the next step's prepare.)  (96^3 cells, N = 3: 1.80 ms, 1.3 TB/s of states,
// bound by the projection's LDS passes.)
template <class PDE, int N>
__global__ void __launch_bounds__(256)
lim_detect_kernel(const KArgs a, const double* __restrict__ Q, const LimWork w) {
  using GL = GeoLim<PDE, N>;
  using GW = GeoLimW<PDE, N>;
  constexpr int NV = GL::NV, S = GL::S, m = GL::m;
  __shared__ double buf[GW::WPB][GW::PW];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const long long c = (long long)blockIdx.x * GW::WPB + wv;
  if (c >= a.ncells) return;
  const int par = *w.parity;
  const double* const lohi = w.lohi2 + par * (a.ncells * (NV * 2));
  double* const lohi_next = w.lohi2 + (par ^ 1) * (a.ncells * (NV * 2));
  double* ra = buf[wv];
  double* rb = ra + GW::RA;
  double* rn = rb + GW::RB;
  double x[NV], rlo, rhi;
  lim_load_nodes<PDE, N>(Q, c, a.ncells, lane, x);
  lim_load_ranges<PDE, N>(a, lohi, c, lane, rlo, rhi);
  bool bad = lane < S && !lim_admissible<PDE>(x, a.pde);
  lim_stage_nodes<PDE, N>(x, ra, rn, lane);
  // DMP range: the cell's and its face neighbours' subcell averages at t^n
#pragma unroll
  for (int off = 1; off < 8; off <<= 1) {
    rlo = fmin(rlo, __shfl_xor(rlo, off, 64));
    rhi = fmax(rhi, __shfl_xor(rhi, off, 64));
  }
  {
    // widened
    const double delta = fmax(1e-4, 1e-3 * (rhi - rlo));
    rlo -= delta;
    rhi += delta;
  }
  double qv[NV][m], l2[NV], h2[NV];
  lim_group_wave<PDE, N, 0, GW::VG>(ra, ra, rb, lane, qv);
  lim_group_wave<PDE, N, GW::VG, NV - GW::VG>(rn, ra, rb, lane, qv);
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    l2[v] = INFINITY;
    h2[v] = -INFINITY;
  }
  if (lane < GW::LAST) bad = !lim_column<PDE, m>(a, qv, l2, h2) || bad;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const double lo = __shfl(rlo, v * 8, 64), hi = __shfl(rhi, v * 8, 64);
    bad = bad || (lane < GW::LAST && !(l2[v] >= lo && h2[v] <= hi));
  }
  if (w.store_next) {
    if constexpr (2 * NV * 71 <= GW::PW) {
      // the lanes' partial ranges through the wave's stage buffer (free once
      // the projection is done; rows 65 apart, so the folding lanes take
      // distinct banks), then one lane per (variable, bound) folds the 64
      // (the minima stored negated: one max loop)
      lim_wave_sync();
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        ra[(2 * v) * 65 + lane] = -l2[v];
        ra[(2 * v + 1) * 65 + lane] = h2[v];
      }
      lim_wave_sync();
      if (lane < 2 * NV * 6) {  // six lanes per (variable, bound), 11 values each
        const int slot = lane / 6, part = lane - slot * 6;
        const double* col = ra + slot * 65 + part * 11;
        double r = -INFINITY;
#pragma unroll
        for (int i = 0; i < 11; ++i)
          if (part * 11 + i < 64) r = fmax(r, col[i]);
        ra[2 * NV * 65 + lane] = r;
      }
      lim_wave_sync();
      if (lane < 2 * NV) {
        const double* pr = ra + 2 * NV * 65 + lane * 6;
        double r = pr[0];
#pragma unroll
        for (int i = 1; i < 6; ++i) r = fmax(r, pr[i]);
        lohi_next[c * NV * 2 + lane] = (lane & 1) ? r : -r;
      }
    } else {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const double l = lim_wave_min(l2[v]), h = lim_wave_max(h2[v]);
        if (lane == 0) {
          lohi_next[(c * NV + v) * 2] = l;
          lohi_next[(c * NV + v) * 2 + 1] = h;
        }
      }
    }
  }
  bad = __ballot(bad) != 0;
  if (lane == 0) {
    w.trb[c] = bad ? 1 : 0;
    if (bad) atomicAdd(&w.counters[0], 1);
  }
}

// The same in 2-D, several cells per wave: a cell has only m = 2N+1 columns
// of subcells, one per lane (N = 5: 11 of 64 lanes with a wave per cell).  A
// lane contracts the nodes with its column's row of A along x (nodes in LDS,
// the same for all lanes of a cell), then along y in registers.  (81^2 cells,
// N = 5: 13.8 us, 26 us with a wave per cell.)  On meshes that leave the chip
// idle a cell's chain counts, which is shorter on a wave of its own where the
// cells are large (N = 5, 6, 7: 256 cells 13.4, 14.0 and 16.1 us, a wave per
// cell 11.2, 11.9 and 13.3; 1600 cells 12.5, 13.6 and 15.9, 11.8, 13.3 and
// 15.0): kAlone.
template <class PDE, int N>
struct GeoDet2 {
  using GL = GeoLim<PDE, N>;
  static constexpr int n = GL::n, m = GL::m, S = GL::S, NV = GL::NV;
  static constexpr int CPW = cmin(64 / m, 64 / (2 * NV));  // cells per wave
  static constexpr int WPB = 4;
  // doubles of LDS per cell: the nodes (an odd stride), then the columns' ranges
  static constexpr int CELL = cmax(NV * S, 2 * NV * m) | 1;
  static constexpr long long kAlone = N >= 5 ? 2000 : 0;  // a wave per cell below this many cells
  static unsigned grid(long long ncells) { return (unsigned)((ncells + CPW * WPB - 1) / (CPW * WPB)); }
};

template <class PDE, int N>
__global__ void __launch_bounds__(256)
lim_detect2_kernel(const KArgs a, const double* __restrict__ Q, const LimWork w) {
  using GD = GeoDet2<PDE, N>;
  constexpr int n = GD::n, m = GD::m, S = GD::S, NV = GD::NV, CPW = GD::CPW, CELL = GD::CELL;
  __shared__ double buf[GD::WPB][CPW * CELL];
  __shared__ double bnd[GD::WPB][CPW][2 * NV];  // the widened DMP range of each cell
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const long long c0 = ((long long)blockIdx.x * GD::WPB + wv) * CPW;
  if (c0 >= a.ncells) return;
  const int here = (int)(a.ncells - c0 < CPW ? a.ncells - c0 : CPW);
  const int par = *w.parity;
  const double* const lohi = w.lohi2 + par * (a.ncells * (NV * 2));
  double* const lohi_next = w.lohi2 + (par ^ 1) * (a.ncells * (NV * 2));
  double* const my = buf[wv];
  // nodes (contiguous in memory over the wave's cells) and their test
  for (int i = lane; i < here * NV * S; i += 64) my[i / (NV * S) * CELL + i % (NV * S)] = Q[c0 * (NV * S) + i];
  if (lane < here * NV) {
    const int ci = lane / NV, v = lane - ci * NV;
    double lo = lohi[((c0 + ci) * NV + v) * 2], hi = lohi[((c0 + ci) * NV + v) * 2 + 1];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const long long o = lim_neighbour<2>(a, c0 + ci, j >> 1, (j & 1) ? 1 : -1);
      if (o < 0) continue;
      lo = fmin(lo, lohi[(o * NV + v) * 2]);
      hi = fmax(hi, lohi[(o * NV + v) * 2 + 1]);
    }
    const double delta = fmax(1e-4, 1e-3 * (hi - lo));
    bnd[wv][ci][2 * v] = lo - delta;
    bnd[wv][ci][2 * v + 1] = hi + delta;
  }
  lim_wave_sync();
  unsigned long long bad = 0;  // bit ci: cell ci is troubled
  for (int i0 = 0; i0 < here * S; i0 += 64) {
    const int i = i0 + lane, ci = i / S;
    double x[NV];
    bool b = false;
    if (i < here * S) {
#pragma unroll
      for (int v = 0; v < NV; ++v) x[v] = my[ci * CELL + v * S + i % S];
      b = !lim_admissible<PDE>(x, a.pde);
    }
    for (unsigned long long t = __ballot(b); t; t &= t - 1) bad |= 1ull << ((i0 + __ffsll(t) - 1) / S);
  }
  const int ci = lane / m, sx = lane - ci * m;
  const bool col = ci < here;
  double l2[NV], h2[NV];
  bool b = false;
  if (col) {
    double A[n], qv[NV][m];
#pragma unroll
    for (int k = 0; k < n; ++k) A[k] = w.tab[sx * n + k];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      double t[n];
#pragma unroll
      for (int ky = 0; ky < n; ++ky) {
        double acc = 0.0;
#pragma unroll
        for (int kx = 0; kx < n; ++kx) acc += A[kx] * my[ci * CELL + v * S + ky * n + kx];
        t[ky] = acc;
      }
#pragma unroll
      for (int j = 0; j < m; ++j) {
        double acc = 0.0;
#pragma unroll
        for (int k = 0; k < n; ++k) acc += LimConst<n>::A[j][k] * t[k];
        qv[v][j] = acc;
      }
    }
    b = !lim_column<PDE, m>(a, qv, l2, h2);
#pragma unroll
    for (int v = 0; v < NV; ++v) b = b || !(l2[v] >= bnd[wv][ci][2 * v] && h2[v] <= bnd[wv][ci][2 * v + 1]);
  }
  for (unsigned long long t = __ballot(b); t; t &= t - 1) bad |= 1ull << ((__ffsll(t) - 1) / m);
  if (w.store_next) {
    lim_wave_sync();  // the nodes are read
    if (col) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        my[ci * CELL + (2 * v) * m + sx] = -l2[v];
        my[ci * CELL + (2 * v + 1) * m + sx] = h2[v];
      }
    }
    lim_wave_sync();
    if (lane < here * 2 * NV) {
      const int cj = lane / (2 * NV), slot = lane - cj * (2 * NV);
      const double* p = my + cj * CELL + slot * m;
      double r = p[0];
#pragma unroll
      for (int i = 1; i < m; ++i) r = fmax(r, p[i]);
      lohi_next[c0 * (2 * NV) + lane] = (slot & 1) ? r : -r;
    }
  }
  if (lane < here) w.trb[c0 + lane] = (bad >> lane) & 1;
  if (lane == 0 && bad) atomicAdd(&w.counters[0], __popcll(bad));
}

// One thread per cell: status of the step and the two cell lists (appended a
// wave at a time).  Every troubled flag a cell's status depends on, those at
// most two faces away, is loaded at once (81^2 cells: 6.4 us, bound by
// latency; 8.5 us with a search that stops at the first).
template <int DIM>
__global__ void __launch_bounds__(256) lim_classify_kernel(const KArgs a, uint8_t* __restrict__ status, const LimWork w) {
  const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (c == 0 && w.store_next) *w.parity ^= 1;  // (the ranges' last reader was detect)
  const int lane = threadIdx.x & 63;
  const bool in = c < a.ncells;
  const long long cl = in ? c : a.ncells - 1;
  // one and two faces away along each axis (-1: past a non-periodic boundary)
  int at[DIM][5];
  long long stride[DIM];
  {
    long long rest = cl, st = 1;
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      const int x = (int)(rest % a.cells[d]);
      rest /= a.cells[d];
      stride[d] = st;
      st *= a.cells[d];
      const bool per_lo = a.bc[2 * d] == ADG_BC_PERIODIC, per_hi = a.bc[2 * d + 1] == ADG_BC_PERIODIC;
#pragma unroll
      for (int s = -2; s <= 2; ++s) {
        int y = x + s;
        if (y < 0) y = per_lo ? ((y % a.cells[d]) + a.cells[d]) % a.cells[d] : -1;
        else if (y >= a.cells[d]) y = per_hi ? y % a.cells[d] : -1;
        at[d][s + 2] = y;
      }
    }
  }
  auto flag = [&](int s0, int s1, int s2) -> int {
    const int y0 = at[0][s0 + 2], y1 = at[1][s1 + 2], y2 = DIM == 3 ? at[DIM - 1][s2 + 2] : 0;
    const bool ok = y0 >= 0 && y1 >= 0 && y2 >= 0;
    const long long o = ok ? y0 * stride[0] + y1 * stride[1] + (DIM == 3 ? y2 * stride[DIM - 1] : 0) : cl;
    const int t = w.trb[o];
    return ok ? t : 0;
  };
  const int self = w.trb[cl];
  int one = 0, two = 0;
#pragma unroll
  for (int s2 = DIM == 3 ? -2 : 0; s2 <= (DIM == 3 ? 2 : 0); ++s2)
#pragma unroll
    for (int s1 = -2; s1 <= 2; ++s1)
#pragma unroll
      for (int s0 = -2; s0 <= 2; ++s0) {
        const int dist = (s0 < 0 ? -s0 : s0) + (s1 < 0 ? -s1 : s1) + (s2 < 0 ? -s2 : s2);
        if (dist == 1) one |= flag(s0, s1, s2);
        if (dist == 2) two |= flag(s0, s1, s2);
      }
  const uint8_t s = !in ? 0 : (self ? 3 : (one ? 2 : (two ? 1 : 0)));
  if (in) status[c] = s;
  const unsigned long long fv = __ballot(s >= 2), dg = __ballot(s == 1);
  int base_fv = 0, base_dg = 0;
  if (lane == 0) {
    if (fv) base_fv = atomicAdd(&w.counters[1], __popcll(fv));
    if (dg) base_dg = atomicAdd(&w.counters[2], __popcll(dg));
  }
  base_fv = __shfl(base_fv, 0, 64);
  base_dg = __shfl(base_dg, 0, 64);
  const unsigned long long below = (1ull << lane) - 1;
  if (s >= 2) w.fv_list[base_fv + __popcll(fv & below)] = (int)c;
  if (s == 1) w.y_list[base_dg + __popcll(dg & below)] = (int)c;
}

__device__ __forceinline__ double lim_minmod(double x, double y) {
  if (x > 0.0 && y > 0.0) return fmin(x, y);
  if (x < 0.0 && y < 0.0) return fmax(x, y);
  return 0.0;
}

// Rusanov flux along the axis whose momentum is component 1, between the
// states qa (low side) and qb (high side).
template <class PDE>
__device__ __forceinline__ void lim_rusanov(const PdeConsts& pc, const double* qa, const double* qb, double* G) {
  constexpr int NV = PDE::NV, DIM = PDE::DIM;
  double F[2][NV], s[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const double* q = h ? qb : qa;
    const double irho = 1.0 / q[0];
    double jj = 0.0;
#pragma unroll
    for (int a = 0; a < DIM; ++a) jj += q[1 + a] * q[1 + a];
    const double p = (pc.gamma - 1.0) * (q[NV - 1] - 0.5 * jj * irho);
    const double u = q[1] * irho;
    F[h][0] = q[1];
#pragma unroll
    for (int a = 0; a < DIM; ++a) F[h][1 + a] = a == 0 ? u * q[1] + p : u * q[1 + a];
    F[h][NV - 1] = u * (q[NV - 1] + p);
    s[h] = fabs(u) + sqrt(pc.gamma * p * irho);
  }
  const double sm = fmax(s[0], s[1]);
#pragma unroll
  for (int v = 0; v < NV; ++v) G[v] = 0.5 * (F[0][v] + F[1][v]) - 0.5 * sm * (qb[v] - qa[v]);
}

// The values of box position p extrapolated to its face on side `side` of the
// axis with box stride sd and moved half a step (its averages where the
// subcell falls back to first order); component v at cv[v] of the box.
template <class PDE, int N>
__device__ __forceinline__ void lim_moved(const double* box, const double* corr, const uint8_t* okf, int p, int q,
                                          int sd, int side, const int (&cv)[PDE::NV], double (&out)[PDE::NV]) {
  using GL = GeoLim<PDE, N>;
  constexpr int NV = GL::NV, NB = GL::NB, NC = GL::NC;
  const bool ok = okf[q] != 0;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const double* b = box + cv[v] * NB + p;
    const double wv = b[0], slope = lim_minmod(wv - b[-sd], b[sd] - wv), cr = corr[cv[v] * NC + q];
    out[v] = ok ? (side ? wv + 0.5 * slope : wv - 0.5 * slope) + cr : wv;
  }
}

// Subcell averages along one axis of a line of nodes extended by two subcells
// on either side, from the lines of the cell (own) and of its neighbours on
// the low and high side; a mirrored side (w[side]) repeats the own subcells
// in reverse, times sgn[side] (-1: the normal momentum at a wall).
template <int n>
__device__ __forceinline__ void lim_extend(const double (&own)[n], const double (&lo)[n], const double (&hi)[n],
                                           const bool (&w)[2], const double (&sgn)[2], double (&out)[2 * n + 3]) {
  using LC = LimConst<n>;
  constexpr int m = 2 * n - 1;
  auto dot = [&](int s, const double (&x)[n]) {
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < n; ++k) acc += LC::A[s][k] * x[k];
    return acc;
  };
#pragma unroll
  for (int s = 0; s < m; ++s) out[2 + s] = dot(s, own);
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    out[g] = w[0] ? sgn[0] * out[3 - g] : dot(m - 2 + g, lo);
    out[m + 2 + g] = w[1] ? sgn[1] * out[m + 1 - g] : dot(g, hi);
  }
}

// FV cells, a persistent grid over the FV list.  Bound by the latency of its
// phases, each about one round of dependent FP64 work and LDS accesses, with
// one block of twelve waves per compute unit (3-D N = 3: 138 KiB of LDS; per
// cell 54,000 cycles, the slopes and half-step corrections 12,000, the owners'
// data 10,000, the subface fluxes 8,700).  The box of subcell averages is a
// tensor-product projection, an axis at a time over the cell and its
// neighbours together (82 kFMA per cell; every position from the owner's 64
// nodes: 426 kFMA and the LDS reads with it), each subface's flux is computed
// once (1176 Rusanov fluxes instead of 2058), and the next cell's
// neighbourhood is looked up beside the update.  24,000 FV cells of the 96^3
// explosion: 3.32 -> 1.95 ms; 550 cells of 81^2, N = 5: 37 -> 16 us.
template <class PDE, int N>
__global__ void __launch_bounds__((GeoLim<PDE, N>::BLOCK), (GeoLim<PDE, N>::FV_WAVES))
lim_fv_kernel(const KArgs a, const double* __restrict__ clock, const double* __restrict__ sub_in, double* __restrict__ Q,
              double* __restrict__ sub_out, const uint8_t* __restrict__ status, const LimWork w) {
  using GL = GeoLim<PDE, N>;
  using LC = LimConst<GL::n>;
  constexpr int DIM = GL::DIM, NV = GL::NV, S = GL::S, NS = GL::NS, F = GL::F, NOFF = GL::NOFF;
  constexpr int m = GL::m, n = GL::n, EB = GL::EB, NB = GL::NB, EC = GL::EC, NC = GL::NC, BLOCK = GL::BLOCK;
  constexpr int NL = ipow(n, DIM - 1), NOY = ipow(3, DIM - 1);
  __shared__ double lds[GL::FV_D];
  __shared__ uint8_t okf[NC];
  // of this cell and of the block's next: the cell at every offset in
  // {-1,0,1}^dim (-1 beyond a non-periodic face), whether it was FV at t^n
  // (its subcell data is read), and the faces whose neighbour is a DG cell
  // after the step
  __shared__ long long owner2[2][NOFF];
  __shared__ uint8_t fvdata2[2][NOFF], dgface2[2][2 * DIM];
  double* const ra = lds;
  double* const rb = ra + GL::REG_A;
  double* const box = ra;
  double* const corr = rb;
  double* const ff = rb + NV * NC;  // subface fluxes [d][t][i][v], i = 0..m along d
  const int tid = threadIdx.x;
  const double dt = clock[1];
  double ihs[3] = {1.0, 1.0, 1.0};  // 1 / subcell size
#pragma unroll
  for (int d = 0; d < DIM; ++d) ihs[d] = m * a.inv_h[d];
  const int count = w.counters[1];
  const int C0 = a.cells[0], C1 = a.cells[1];
  // the neighbourhood of list entry it, by threads t0 .. t0 + NOFF - 1: one
  // offset k in {-1,0,1}^dim with at most two nonzero entries each
  auto neighbourhood = [&](int it, int t0) {
    const int k = tid - t0;
    if (it >= count || k < 0 || k >= NOFF) return;
    const long long c = w.fv_list[it];
    const int off[3] = {k % 3 - 1, (k / 3) % 3 - 1, DIM == 3 ? k / 9 - 1 : 0};
    int oc[3] = {(int)(c % C0), (int)((c / C0) % C1), DIM == 3 ? (int)(c / ((long long)C0 * C1)) : 0};
    bool exists = (off[0] != 0) + (off[1] != 0) + (off[2] != 0) <= 2;
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      oc[d] += off[d];
      if (oc[d] < 0 || oc[d] >= a.cells[d]) {
        if (a.bc[2 * d + (off[d] > 0)] != ADG_BC_PERIODIC) exists = false;
        oc[d] = (oc[d] + a.cells[d]) % a.cells[d];
      }
    }
    const long long o = exists ? oc[0] + (long long)C0 * (oc[1] + (long long)C1 * oc[2]) : -1;
    const uint8_t was = exists ? w.st_prev[o] : 0, is = exists ? status[o] : 3;
    const int par = (it / (int)gridDim.x) & 1;
    owner2[par][k] = o;
    fvdata2[par][k] = was >= 2 ? 1 : 0;
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      const int one = d == 0 ? 1 : (d == 1 ? 3 : 9), mid = NOFF / 2;
      if (k == mid - one) dgface2[par][2 * d] = is < 2;
      if (k == mid + one) dgface2[par][2 * d + 1] = is < 2;
    }
  };
  neighbourhood(blockIdx.x, 0);
  for (int it = blockIdx.x; it < count; it += gridDim.x) {
    const long long c = w.fv_list[it];
    const int cc[3] = {(int)(c % C0), (int)((c / C0) % C1), DIM == 3 ? (int)(c / ((long long)C0 * C1)) : 0};
    // sides beyond which the box mirrors this cell's subcells, and whether
    // the mirror reverses the normal momentum
    bool mir[DIM][2], wall[DIM][2];
#pragma unroll
    for (int d = 0; d < DIM; ++d)
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        mir[d][g] = (g ? cc[d] == a.cells[d] - 1 : cc[d] == 0) && a.bc[2 * d + g] != ADG_BC_PERIODIC;
        wall[d][g] = mir[d][g] && a.bc[2 * d + g] == ADG_BC_WALL;
      }
    const int par = (it / (int)gridDim.x) & 1;
    const long long* const owner = owner2[par];
    const uint8_t *const fvdata = fvdata2[par], *const dgface = dgface2[par];
    __syncthreads();  // the neighbourhood is there, the previous cell's LDS reads are done
    // 1. the subcell box: the cell, two ghost layers across each face, one
    //    across each edge (corners are never read).  A position belongs to
    //    the cell or to a face or edge neighbour (beyond a non-periodic face
    //    it mirrors a subcell of the cell on this side).  First the
    //    positions whose owner has FV data, kept in registers until the box
    //    is free; then the projections of the owners' polynomials.
    double pre[GL::PPT][NV];
    int sgn_of[GL::PPT];  // -1: not from FV data, else bit d: component 1 + d reversed
#pragma unroll
    for (int j = 0; j < GL::PPT; ++j) {
      const int p = tid + j * BLOCK < NB ? tid + j * BLOCK : 0;
      int x[3];
      lim_multi<DIM>(p, EB, x);
      int outside = 0, far = 0, k = 0, si = 0, sg = 0;
#pragma unroll
      for (int d = DIM - 1; d >= 0; --d) {
        const int r = x[d] - 2;
        int po = 0, ss = r;
        if (r < 0 || r >= m) {
          ++outside;
          const int g = r >= m;
          const bool mg = g ? mir[d][1] : mir[d][0], wg = g ? wall[d][1] : wall[d][0];
          ss = mg ? (g ? 2 * m - 1 - r : -1 - r) : (g ? r - m : r + m);
          po = mg ? 0 : (g ? 1 : -1);
          if (wg) sg |= 1 << d;
        }
        if (r < -1 || r > m) ++far;
        k = 3 * k + po + 1;
        si = m * si + ss;
      }
      const bool skip = tid + j * BLOCK >= NB || outside > 2 || (outside == 2 && far > 0) || !fvdata[k];
      sgn_of[j] = skip ? -1 : sg;
      const double* src = sub_in + (skip ? c : owner[k]) * (long long)(NV * NS) + si;
      if (!skip) {
#pragma unroll
        for (int v = 0; v < NV; ++v) pre[j][v] = src[v * NS];
      }
    }
    // along x: one task per (quantity, y (and z) offset, line of nodes)
    for (int t = tid; t < NV * NOY * NL; t += BLOCK) {
      const int line = t % NL, ky = (t / NL) % NOY, v = t / (NL * NOY);
      // the three owners along x: offset index ky * 3 + (0, 1, 2)
      double x[3][n];
#pragma unroll
      for (int g = 0; g < 3; ++g) {
        const long long o = owner[ky * 3 + g];
        const double* src = w.Qold + (o >= 0 ? o : c) * (long long)(NV * S) + v * S + line * n;
#pragma unroll
        for (int k = 0; k < n; ++k) x[g][k] = src[k];
      }
      const double sgn[2] = {v == 1 && wall[0][0] ? -1.0 : 1.0, v == 1 && wall[0][1] ? -1.0 : 1.0};
      double out[EB];
      lim_extend<n>(x[1], x[0], x[2], mir[0], sgn, out);
#pragma unroll
      for (int i = 0; i < EB; ++i) ra[t * EB + i] = out[i];
    }
    __syncthreads();
    if constexpr (DIM == 3) {
      // along y: one task per (quantity, z offset, kz, x)
      for (int t = tid; t < NV * 3 * n * EB; t += BLOCK) {
        const int i = t % EB, kz = (t / EB) % n, oz = (t / (EB * n)) % 3, v = t / (EB * n * 3);
        double x[3][n];
#pragma unroll
        for (int g = 0; g < 3; ++g)
#pragma unroll
          for (int k = 0; k < n; ++k) x[g][k] = ra[(((v * NOY + oz * 3 + g) * n + kz) * n + k) * EB + i];
        const double sgn[2] = {v == 2 && wall[1][0] ? -1.0 : 1.0, v == 2 && wall[1][1] ? -1.0 : 1.0};
        double out[EB];
        lim_extend<n>(x[1], x[0], x[2], mir[1], sgn, out);
        double* o = rb + ((v * 3 + oz) * n + kz) * EB * EB + i;
#pragma unroll
        for (int y = 0; y < EB; ++y) o[y * EB] = out[y];
      }
      __syncthreads();
      // along z, into the box: one task per (quantity, y, x)
      for (int t = tid; t < NV * EB * EB; t += BLOCK) {
        const int i = t % EB, y = (t / EB) % EB, v = t / (EB * EB);
        double x[3][n];
#pragma unroll
        for (int g = 0; g < 3; ++g)
#pragma unroll
          for (int k = 0; k < n; ++k) x[g][k] = rb[((v * 3 + g) * n + k) * EB * EB + y * EB + i];
        const double sgn[2] = {v == 3 && wall[2][0] ? -1.0 : 1.0, v == 3 && wall[2][1] ? -1.0 : 1.0};
        double out[EB];
        lim_extend<n>(x[1], x[0], x[2], mir[2], sgn, out);
#pragma unroll
        for (int z = 0; z < EB; ++z) box[v * NB + (z * EB + y) * EB + i] = out[z];
      }
    } else {
      // along y, into registers (the box takes the place of the projection
      // along x), then the box: one task per (quantity, x)
      double out[EB];
      const int t = tid, i = t % EB, v = t / EB;
      static_assert(NV * EB <= BLOCK || DIM == 3, "one task per thread");
      if (t < NV * EB) {
        double x[3][n];
#pragma unroll
        for (int g = 0; g < 3; ++g)
#pragma unroll
          for (int k = 0; k < n; ++k) x[g][k] = ra[((v * NOY + g) * n + k) * EB + i];
        const double sgn[2] = {v == 2 && wall[1][0] ? -1.0 : 1.0, v == 2 && wall[1][1] ? -1.0 : 1.0};
        lim_extend<n>(x[1], x[0], x[2], mir[1], sgn, out);
      }
      __syncthreads();
      if (t < NV * EB) {
#pragma unroll
        for (int y = 0; y < EB; ++y) box[v * NB + y * EB + i] = out[y];
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < GL::PPT; ++j)
      if (sgn_of[j] >= 0) {
#pragma unroll
        for (int v = 0; v < NV; ++v)
          box[v * NB + tid + j * BLOCK] = v >= 1 && v <= DIM && ((sgn_of[j] >> (v - 1)) & 1) ? -pre[j][v] : pre[j][v];
      }
    __syncthreads();
    // 2. minmod slopes, extrapolated values and their half-step correction
    //    for the cell's subcells and the first ghost layer across each face
    for (int q = tid; q < NC; q += BLOCK) {
      int x[3];
      lim_multi<DIM>(q, EC, x);
      int outside = 0, p = 0, mul = 1;
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        const int r = x[d] - 1;
        if (r < 0 || r >= m) ++outside;
        p += (r + 2) * mul;
        mul *= EB;
      }
      if (outside > 1) continue;
      double ext[DIM][2][NV], cv[NV];
      bool ok = true;
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        const int sd = d == 0 ? 1 : (d == 1 ? EB : EB * EB);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const double wv = box[v * NB + p];
          const double slope = lim_minmod(wv - box[v * NB + p - sd], box[v * NB + p + sd] - wv);
          ext[d][0][v] = wv - 0.5 * slope;
          ext[d][1][v] = wv + 0.5 * slope;
        }
        // (finite values: tested below, a moved value is finite only if its extrapolated one is)
        ok = ok && lim_admissible<PDE, false>(ext[d][0], a.pde) && lim_admissible<PDE, false>(ext[d][1], a.pde);
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) cv[v] = 0.0;
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        double Fl[NV], Fr[NV];
        PDE::flux_dir(ext[d][0], ext[d][0], a.pde, d, Fl);
        PDE::flux_dir(ext[d][1], ext[d][1], a.pde, d, Fr);
        const double s = 0.5 * dt * ihs[d];
#pragma unroll
        for (int v = 0; v < NV; ++v) cv[v] += s * (Fl[v] - Fr[v]);
      }
#pragma unroll
      for (int d = 0; d < DIM; ++d)
#pragma unroll
        for (int side = 0; side < 2; ++side) {
          double mv[NV];
#pragma unroll
          for (int v = 0; v < NV; ++v) mv[v] = ext[d][side][v] + cv[v];
          ok = ok && lim_admissible<PDE>(mv, a.pde);
        }
#pragma unroll
      for (int v = 0; v < NV; ++v) corr[v * NC + q] = cv[v];
      okf[q] = ok ? 1 : 0;
    }
    __syncthreads();
    // 3. Rusanov at every subface (components rotated so that the normal
    //    momentum is component 1), then the update of the cell's subcells
    for (int f = tid; f < DIM * GL::NFC; f += BLOCK) {
      const int d = f / GL::NFC, fd = f - d * GL::NFC;
      const int i = fd % (m + 1), t = fd / (m + 1), t0 = t % m, t1 = t / m;
      // the subcell above the face (index i along d), its box and correction
      // positions; t: the other axes, lower first
      const int x[3] = {d == 0 ? i : t0, d == 0 ? t0 : (d == 1 ? i : t1), d == 2 ? i : t1};
      const int p = (x[0] + 2) + EB * ((x[1] + 2) + (DIM == 3 ? EB * (x[2] + 2) : 0));
      const int q = (x[0] + 1) + EC * ((x[1] + 1) + (DIM == 3 ? EC * (x[2] + 1) : 0));
      const int sd = d == 0 ? 1 : (d == 1 ? EB : EB * EB), cd = d == 0 ? 1 : (d == 1 ? EC : EC * EC);
      int cv[NV];
      cv[0] = 0;
      cv[NV - 1] = NV - 1;
#pragma unroll
      for (int e = 0; e < DIM; ++e) cv[1 + e] = 1 + (d + e < DIM ? d + e : d + e - DIM);
      double e0[NV], e1[NV], G[NV];
      lim_moved<PDE, N>(box, corr, okf, p - sd, q - cd, sd, 1, cv, e0);
      lim_moved<PDE, N>(box, corr, okf, p, q, sd, 0, cv, e1);
      lim_rusanov<PDE>(a.pde, e0, e1, G);
#pragma unroll
      for (int v = 0; v < NV; ++v) ff[f * NV + cv[v]] = G[v];
    }
    __syncthreads();
    // (the threads past the subcells: the next cell's neighbourhood)
    neighbourhood(it + gridDim.x, BLOCK - 64);
    double vnew[GL::VPT][NV];
#pragma unroll
    for (int j = 0; j < GL::VPT; ++j) {
      const int s = tid + j * BLOCK;
      if (s >= NS) break;
      int x[3];
      lim_multi<DIM>(s, m, x);
      const int p = (x[0] + 2) + EB * ((x[1] + 2) + (DIM == 3 ? EB * (x[2] + 2) : 0));
      double acc[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) acc[v] = 0.0;
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        const int t = DIM == 2 ? x[1 - d] : (d == 0 ? x[1] + m * x[2] : (d == 1 ? x[0] + m * x[2] : x[0] + m * x[1]));
        const double* g = ff + (d * GL::NFC + t * (m + 1) + x[d]) * NV;
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[v] += (g[NV + v] - g[v]) * ihs[d];
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        vnew[j][v] = box[v * NB + p] - dt * acc[v];
        sub_out[(c * NV + v) * NS + s] = vnew[j][v];
      }
    }
    __syncthreads();
    // 4. back to the DG space, and the face-node fluxes for DG neighbours
    double* const vn = ra;                  // [v][subcell]
    double* const r1 = ra + NV * NS;        // fit: [v][(sz)][sy][kx]
    double* const r2 = corr;                // fit, 3-D: [v][sz][ky][kx]
    double* const g1 = r1 + NV * ipow(m, DIM - 1) * n;  // face fluxes, 3-D: [face][v][t1][f0]
#pragma unroll
    for (int j = 0; j < GL::VPT; ++j) {
      const int s = tid + j * BLOCK;
      if (s < NS)
#pragma unroll
        for (int v = 0; v < NV; ++v) vn[v * NS + s] = vnew[j][v];
    }
    // subfaces of the cell's face (side i = 0 or m), along their first axis:
    // one task per (face, quantity, t1), all n face nodes
    constexpr int NT1 = DIM == 3 ? m : 1;
    for (int t = tid; t < 2 * DIM * NV * NT1; t += BLOCK) {
      const int t1 = t % NT1, v = (t / NT1) % NV, face = t / (NT1 * NV);
      if (!dgface[face]) continue;
      const double* g = ff + ((face >> 1) * GL::NFC + t1 * m * (m + 1) + (face & 1) * m) * NV + v;
      double in[m];
#pragma unroll
      for (int j = 0; j < m; ++j) in[j] = g[j * (m + 1) * NV];
#pragma unroll
      for (int k = 0; k < n; ++k) {
        double acc = 0.0;
#pragma unroll
        for (int j = 0; j < m; ++j) acc += LC::Qf[k][j] * in[j];
        if constexpr (DIM == 3) g1[t * n + k] = acc;
        else w.gfv[((c * 2 * DIM + face) * NV + v) * F + k] = acc;
      }
    }
    __syncthreads();
    // least-squares fit, one axis at a time: x (vn -> r1), y (r1 -> r2,
    // 3-D), the last axis into Q
    {
      constexpr int L1 = NV * ipow(m, DIM - 1);
      for (int line = tid; line < L1; line += BLOCK) {
        double in[m];
#pragma unroll
        for (int j = 0; j < m; ++j) in[j] = vn[line * m + j];
#pragma unroll
        for (int k = 0; k < n; ++k) {
          double acc = 0.0;
#pragma unroll
          for (int j = 0; j < m; ++j) acc += LC::B[k][j] * in[j];
          r1[line * n + k] = acc;
        }
      }
      if constexpr (DIM == 3) {
        // (meanwhile) the face fluxes along their second axis
        for (int t = tid; t < 2 * DIM * NV * n; t += BLOCK) {
          const int f0 = t % n, v = (t / n) % NV, face = t / (n * NV);
          if (!dgface[face]) continue;
          double in[m];
#pragma unroll
          for (int j = 0; j < m; ++j) in[j] = g1[((face * NV + v) * m + j) * n + f0];
#pragma unroll
          for (int k = 0; k < n; ++k) {
            double acc = 0.0;
#pragma unroll
            for (int j = 0; j < m; ++j) acc += LC::Qf[k][j] * in[j];
            w.gfv[((c * 2 * DIM + face) * NV + v) * F + k * n + f0] = acc;
          }
        }
      }
      __syncthreads();
      const double* rl = r1;
      if constexpr (DIM == 3) {
        for (int line = tid; line < NV * m * n; line += BLOCK) {
          const int kx = line % n, vz = line / n;  // vz = v m + sz
          double in[m];
#pragma unroll
          for (int j = 0; j < m; ++j) in[j] = r1[(vz * m + j) * n + kx];
#pragma unroll
          for (int k = 0; k < n; ++k) {
            double acc = 0.0;
#pragma unroll
            for (int j = 0; j < m; ++j) acc += LC::B[k][j] * in[j];
            r2[(vz * n + k) * n + kx] = acc;
          }
        }
        __syncthreads();
        rl = r2;
      }
      constexpr int RL = ipow(n, DIM - 1);  // lines per variable of the last stage
      for (int line = tid; line < NV * RL; line += BLOCK) {
        const int v = line / RL, r = line - v * RL;
        double in[m];
#pragma unroll
        for (int j = 0; j < m; ++j) in[j] = rl[(v * m + j) * RL + r];
#pragma unroll
        for (int k = 0; k < n; ++k) {
          double acc = 0.0;
#pragma unroll
          for (int j = 0; j < m; ++j) acc += LC::B[k][j] * in[j];
          Q[c * NV * S + v * S + k * RL + r] = acc;
        }
      }
    }
  }
}

// DG cells with an FV face: the Rusanov flux of that face in the
// candidate's update exchanged for the FV one.  Persistent grid over the
// list.
template <class PDE, int N>
__global__ void __launch_bounds__(256)
lim_faces_kernel(const KArgs a, const double* __restrict__ clock, const double* __restrict__ traces,
                 const uint8_t* __restrict__ status, double* __restrict__ Q, const LimWork w) {
  using GL = GeoLim<PDE, N>;
  constexpr int DIM = GL::DIM, NV = GL::NV, S = GL::S, F = GL::F, n = GL::n, BLOCK = 256;
  const Tables<double>& T = a.t64;
  const double dt = clock[1];
  const int count = w.counters[2];
  for (int it = blockIdx.x; it < count; it += gridDim.x) {
    const long long c = w.y_list[it];
    for (int i = threadIdx.x; i < NV * S; i += BLOCK) {
      const int v = i / S, k = i - v * S;
      const int kk[3] = {k % n, (k / n) % n, DIM == 3 ? k / (n * n) : 0};
      double delta = 0.0;
#pragma unroll
      for (int d = 0; d < DIM; ++d)
#pragma unroll
        for (int side = 0; side < 2; ++side) {
          const long long o = lim_neighbour<DIM>(a, c, d, side ? 1 : -1);
          if (o < 0 || status[o] < 2) continue;
          const int f = DIM == 2 ? kk[1 - d] : (d == 0 ? kk[1] + n * kk[2] : (d == 1 ? kk[0] + n * kk[2] : kk[0] + n * kk[1]));
          const long long cL = side ? c : o, cR = side ? o : c;
          const double* tL = traces + ((cL * (2 * DIM) + 2 * d + 1) * 2) * NV * F;
          const double* tR = traces + ((cR * (2 * DIM) + 2 * d) * 2) * NV * F;
          double qL[NV], qR[NV];
#pragma unroll
          for (int u = 0; u < NV; ++u) {
            qL[u] = tL[u * F + f];
            qR[u] = tR[u * F + f];
          }
          const double s = fmax(PDE::max_eigen(qL, qL, a.pde, d), PDE::max_eigen(qR, qR, a.pde, d));
          const double G = 0.5 * (tL[(NV + v) * F + f] + tR[(NV + v) * F + f]) - 0.5 * s * (qR[v] - qL[v]);
          const double Gfv = w.gfv[((o * 2 * DIM + 2 * d + 1 - side) * NV + v) * F + f];
          const double dG = (Gfv - G) * T.invw[kk[d]] * a.inv_h[d];
          delta += side ? T.l1[kk[d]] * dG : -T.l0[kk[d]] * dG;
        }
      Q[c * NV * S + i] -= dt * delta;
    }
  }
}

// Eq. (7) after a limited step: the largest signal speed over the nodal
// values of DG cells and the subcell averages of FV cells (an FV cell's
// solution; its least-squares polynomial can hold non-physical nodes).  The
// cells of status 0 hold the candidate, whose speeds the corrector stored; a
// wave looks through lim_cells_per_wave cells and evaluates the others.  Block maxima into
// the reduction slots.  (96^3 cells, N = 3:
// 0.11 ms; 0.48 ms with every cell's nodes read again.)
template <class PDE, int N>
__global__ void __launch_bounds__(256)
lim_lambda_kernel(const KArgs a, const double* __restrict__ Q, const double* __restrict__ sub,
                  const uint8_t* __restrict__ status, const double* __restrict__ cell_lam, int per) {
  using GL = GeoLim<PDE, N>;
  constexpr int DIM = GL::DIM, NV = GL::NV, S = GL::S, NS = GL::NS;
  __shared__ double red[4];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const long long first = (long long)blockIdx.x * 4 + wv, waves = (a.ncells + per - 1) / per;
  const long long mc = first + lane * waves;
  double lam = 0.0;
  int st = 0;
  if (first < waves && lane < per && mc < a.ncells) {
    st = status[mc];
    if (st == 0) lam = cell_lam[mc];
  }
  for (unsigned long long todo = __ballot(st != 0); todo; todo &= todo - 1) {
    const int i = __ffsll(todo) - 1;
    const long long c = first + i * waves;
    const bool fv = __shfl(st, i, 64) >= 2;
    const int npts = fv ? NS : S;
    const double* base = fv ? sub + c * NV * NS : Q + c * NV * S;
    for (int k = lane; k < npts; k += 64) {
      double q[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) q[v] = base[v * npts + k];
#pragma unroll
      for (int d = 0; d < DIM; ++d) lam = lam_max(lam, PDE::max_eigen(q, q, a.pde, d));
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) lam = lam_max(lam, __shfl_xor(lam, off, 64));
  if (lane == 0) red[wv] = lam;
  __syncthreads();
  if (tid == 0) slot_max(a.slots, blockIdx.x, lam_max(lam_max(red[0], red[1]), lam_max(red[2], red[3])));
}

template <class PDE, int N>
struct LimLaunch {
  using GL = GeoLim<PDE, N>;
  static constexpr int kFaceGrid = 1024;
  // prepare; the caller's DG step follows
  static hipError_t before(const KArgs& a, const double* Q, const double* sub_in, const uint8_t* status,
                           const LimWork& w, hipStream_t st) {
    const int per = w.reuse && !w.copy ? lim_cells_per_wave(a.ncells) : 1;
    const unsigned grid = GeoLimSeq<PDE, N>::grid((a.ncells + per - 1) / per);
    const auto k = per == 1 ? lim_prepare_kernel<PDE, N, true> : lim_prepare_kernel<PDE, N, false>;
    hipLaunchKernelGGL(k, dim3(grid), dim3(64 * GeoLimW<PDE, N>::WPB), 0, st, a, Q, sub_in, status, w, per);
    return hipGetLastError();
  }
  // detect, classify, FV cells, DG cells with FV faces
  static hipError_t after(const KArgs& a, double* Q, double* clock, const double* traces,
                          const double* sub_in, double* sub_out, uint8_t* status, const LimWork& w,
                          int next_dt, hipStream_t st) {
    bool packed = false;
    if constexpr (GL::DIM == 2) {
      using GD = GeoDet2<PDE, N>;
      packed = a.ncells >= GD::kAlone;
      if (packed)
        hipLaunchKernelGGL((lim_detect2_kernel<PDE, N>), dim3(GD::grid(a.ncells)), dim3(64 * GD::WPB), 0, st, a, Q, w);
    }
    if constexpr (GL::DIM == 3 || N >= 5) {
      if (!packed)
        hipLaunchKernelGGL((lim_detect_kernel<PDE, N>), dim3(GeoLimSeq<PDE, N>::grid(a.ncells)),
                           dim3(64 * GeoLimW<PDE, N>::WPB), 0, st, a, Q, w);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((lim_classify_kernel<GL::DIM>), dim3((unsigned)((a.ncells + 255) / 256)), dim3(256), 0, st,
                       a, status, w);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL((lim_fv_kernel<PDE, N>), dim3(GL::FV_GRID), dim3(GL::BLOCK), 0, st, a, clock, sub_in, Q,
                       sub_out, status, w);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL((lim_faces_kernel<PDE, N>), dim3(kFaceGrid), dim3(256), 0, st, a, clock, traces,
                       status, Q, w);
    if ((e = hipGetLastError()) != hipSuccess || !next_dt) return e;
    const int per = lim_cells_per_wave(a.ncells);
    const unsigned waves = (unsigned)((a.ncells + per - 1) / per);
    hipLaunchKernelGGL((lim_lambda_kernel<PDE, N>), dim3((waves + 3) / 4), dim3(256), 0, st, a, Q, sub_out, status,
                       w.cell_lam, per);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(finalize_kernel, dim3(1), dim3(kSlots), 0, st, a.slots, a.dt_factor, 1, clock);
    return hipGetLastError();
  }
};

}  // namespace adg
