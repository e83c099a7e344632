// FP64 space-time predictor with one lane per line of nodes along the last
// axis (ExaHyPE paper, Sec. 3.3, Eq. (5): q^{r+1}_i = u^n + dt sum_j
// (K1^{-1})_ij w_j R(q^r)_j), for small cells (3-D, n = N + 1 <= 4).
//
// What bounds the one-thread-per-node kernel there is the LDS: a derivative
// value is written, read by the line task, written back and read again, and a
// wave's 8-byte LDS write takes 6.2 cycles of the CU against 2.3 for a read
// (3-D N = 3: LDS busy 80 % of the launch, the vector unit 57 %).  Here a lane
// keeps the n nodes of its line at all n time slices in registers, so neither
// the derivative along the last axis nor the time operator moves data, and
// all lanes of a cell are in one wave, so there is no block barrier.  The
// other two axes need the same node of the other lines:
//  n = 2, 3  the fluxes of a slice go to LDS once (rows of 64 lanes) and every
//            lane reads the n - 1 other values of its line along the axis and
//            contracts them with its own row of D (one write and n - 1 reads
//            instead of two and two);
//  n = 4     no LDS: v_mfma_f64_4x4x4 contracts across lanes (see mfma4).
// Measured, one launch: 3-D Euler N = 3, 96^3 cells 8.29 -> 4.55 ms (LDS
// gather instead of the matrix instructions: 6.0 ms; gather along x only:
// 4.8 ms), 85 % of the FP64 issue slots at the 1.9 GHz that the card holds
// under this load; N = 2, 72^3 cells 1.63 -> 0.89 ms (traces and state alone
// are 2.4 GB, 0.49 ms at the 4.9 TB/s of a large copy).
#pragma once

namespace adg {

template <class PDE, int N>
struct GeoLine {
  using G = Geo<PDE, N>;
  static constexpr int n = G::n, DIM = G::DIM, NV = G::NV, F = G::F, S = G::S;
  // cells per wave, none across the wave's halves (an 8-byte LDS access is
  // served 32 lanes at a time: a cell's lanes then never share a bank)
  static constexpr int CPH = F <= 32 ? 32 / F : 0;
  static constexpr int CPB = 2 * CPH;
  static constexpr bool ALONE = 16 % F != 0;  // see row_read
  static constexpr bool MF = DIM == 3 && n == 4;  // see mfma4
  static constexpr int XL = MF ? 0 : DIM - 1;  // axes whose derivatives go through LDS
  static constexpr int BLOCK = 64;
  static constexpr int XD = DIM - 1;
  // rows of 64 doubles: the fluxes of one slice along the first XD axes; the
  // final phase takes q-bar and F-bar of one axis
  static constexpr int ROWS = cmax(XD, 2) * NV * n;
  static constexpr int NA = n + 3;           // source amplitudes per source
  static constexpr bool fits = (DIM == 3 || n >= 3) && n <= 4 && !PDE::kHasNcp && NV <= 5;
  // waves per SIMD the register allocator aims at (n n NV doubles per lane)
  static constexpr int MIN_WAVES = n * n * NV >= 64 ? 2 : (n * n * NV >= 36 ? 3 : 4);
};

// Zero, opaque to the optimiser: loads at this offset are not moved out of
// the Picard loop (u^n is read again, an L2 hit, where it is used).
__device__ __forceinline__ int opaque_zero() {
  int z = 0;
  asm volatile("" : "+s"(z));
  return z;
}
// A value computed here and not where it is stored: the optimiser would
// otherwise sink the sums into the guarded stores and keep their inputs live.
__device__ __forceinline__ void pin(double& x) { asm volatile("" : "+v"(x)); }
// An element of the shared rows.  Plain accesses of two rows pair up as one
// ds_read2, which is served 16 lanes of either row at a time: where cells
// straddle the 16-lane groups (ALONE) that pairing puts two lanes on a bank
// (4.1 instead of 2.1 cycles per 8-byte read at n = 3), so there every read
// stays an instruction of its own.
template <bool ALONE>
__device__ __forceinline__ double row_read(const double* p) {
  if constexpr (ALONE) return *(const volatile __attribute__((address_space(3))) double*)p;
  return *p;
}
// Instructions are not moved across: left alone, the scheduler starts every
// LDS read of a pass at once and spills.
__device__ __forceinline__ void sched_fence() { __builtin_amdgcn_sched_barrier(0); }

__device__ __forceinline__ void line_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// a value that is the same in every lane, in scalar registers
__device__ __forceinline__ double uniform(double x) {
  // (opaque first: of a value known to be uniform the builtin is folded away,
  // and a table of such values takes vector registers)
  int lo = __double2loint(x), hi = __double2hiint(x);
  asm("" : "+v"(lo), "+v"(hi));
  lo = __builtin_amdgcn_readfirstlane(lo);
  hi = __builtin_amdgcn_readfirstlane(hi);
  return __hiloint2double(hi, lo);
}

// c + A B for four blocks of 4 x 4 matrices (v_mfma_f64_4x4x4_4b_f64): lane
// i + 4 b + 16 k holds A[i][k] and B[k][i] of block b, and element [k][i] of
// the result.  With the lanes of a cell of 4^3 nodes at x + 4 (cell) + 16 y,
// D as A differentiates the operand B along y in place, and an operand A
// comes out with x and y exchanged: the identity, then D as B, differentiates
// along x.
__device__ __forceinline__ double mfma4(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// Kernel variants: no sources and the constant guess, no sources and the CERK
// guess, and any guess with point sources (the code of the cases a run does
// not have costs registers: 344 bytes of spill at N = 3 in one kernel).
enum LineMode { kLinePlain, kLineCerk, kLineSources };

template <class PDE, int N, int MODE>
__global__ void __launch_bounds__(64, (GeoLine<PDE, N>::MIN_WAVES))
predict_kernel_line(const KArgs a, const double* Q, const double* __restrict__ params,
                    const double* __restrict__ clock, double* Qout, double* __restrict__ traces) {
  // Q and Qout may be the same array (in-place step): each element is read
  // by the lane that writes it at the end.
  using GN = GeoLine<PDE, N>;
  using T = CT<double, GN::n>;
  constexpr int n = GN::n, S = GN::S, F = GN::F, NV = GN::NV, NP = PDE::NP, DIM = GN::DIM;
  constexpr int CPB = GN::CPB, XD = GN::XD, LAST = DIM - 1, NA = GN::NA;
  static_assert(GN::fits, "a lane's nodes must fit its registers, a cell's lines one wave");
  __shared__ double rows[GN::ROWS][64];
  __shared__ double src_amp[MODE == kLineSources ? kMaxSources * NA : 1];

  const int lane = threadIdx.x;
  constexpr bool MF = GN::MF;
  const int half = lane >> 5, hl = lane & 31;
  const bool line = MF || hl < GN::CPH * F;
  const int lh = line ? hl / F : 0;  // lanes past the cells' lines repeat line 0
  // of their half's first cell (nothing of theirs is kept)
  const int l = MF ? (lane & 3) + 4 * (lane >> 4) : (line ? hl - lh * F : 0);
  const int lc = MF ? (lane >> 2) & 3 : half * GN::CPH + lh;
  const int base = MF ? lane : half * 32 + lh * F + l;
  constexpr int XL = GN::XL;
  constexpr int STEP1 = MF ? 16 : n;  // lanes between neighbours along the second axis
  const long long cell0 = (long long)xcd_block(blockIdx.x, a.nblocks) * CPB;
  const long long cell = cell0 + lc;
  const bool active = line && cell < a.ncells;
  const long long cl = cell < a.ncells ? cell : a.ncells - 1;  // clamp loads of the ragged tail

  // this line's position along the first XD axes; the lanes of the other
  // lines at the same other coordinates, r places further (cyclic), and the
  // row of -D / h that belongs to this position
  const int pos[2] = {l % n, (l / n) % n};
  int unit[XD][n];
  double coef[XD][n];
#pragma unroll
  for (int d = 0; d < XD; ++d)
#pragma unroll
    for (int r = 0; r < n; ++r) {
      const int p = pos[d] + r < n ? pos[d] + r : pos[d] + r - n;
      unit[d][r] = base + (p - pos[d]) * (d == 0 ? 1 : STEP1);
      coef[d][r] = -a.inv_h[d] * a.t64.D[pos[d]][p];
    }
  const double mih = -a.inv_h[LAST];
  double Dz[n][n];  // -D / h of the last axis
#pragma unroll
  for (int i = 0; i < n; ++i)
#pragma unroll
    for (int z = 0; z < n; ++z) Dz[i][z] = uniform(mih * T::D(i, z));
  // MF: this lane's elements of -D / h and of the identity as matrix operands
  double mx[XD], eye = 0.0;
  if constexpr (MF) {
#pragma unroll
    for (int d = 0; d < XD; ++d) mx[d] = -a.inv_h[d] * a.t64.D[lane & 3][lane >> 4];
    eye = (lane & 3) == (lane >> 4) ? 1.0 : 0.0;
  }
  // x + (-D / h_d) f along axis d on the matrix cores
  auto mfma_div = [&](int d, double f, double x) {
    if (d == 1) return mfma4(mx[XD - 1], f, x);
    return mfma4(mfma4(f, eye, 0.0), mx[0], x);
  };

  const double* const Q0c = Q + cl * (long long)(NV * S) + l;  // node z of quantity v: Qc[v S + z F]
  double P[NP > 0 ? NP : 1];
#pragma unroll
  for (int p = 0; p < NP; ++p) P[p] = params[cl * NP + p];
  const double t_n = clock[0], dt = clock[1];
  double Kt[n][n];  // the time operator, dt K1^{-1} W
#pragma unroll
  for (int i = 0; i < n; ++i)
#pragma unroll
    for (int j = 0; j < n; ++j) Kt[i][j] = uniform(dt * T::KW(i, j));

  // point sources: the Ricker amplitudes at the n time nodes and at the
  // stage times 0, 1/2, 1 of the CERK guess, where the wave has a source cell
  bool src_here = false;
  unsigned src_mine = 0;  // the sources in this lane's cell
  if constexpr (MODE == kLineSources)
    for (int s = 0; s < a.nsrc; ++s) {
      const long long c = a.src[s].cell;
      src_here = src_here || (c >= cell0 && c < cell0 + CPB);
      src_mine |= c == cell && line ? 1u << s : 0u;
    }
  if (src_here) {
    for (int e = lane; e < a.nsrc * NA; e += 64) {
      const int s = e / NA, j = e - s * NA;
      const double tau = j < n ? a.t64.xi[j] : 0.5 * (j - n);
      src_amp[e] = ricker(a.src[s].f0, a.src[s].t0, a.src[s].amp, t_n + tau * dt);
    }
    line_wave_sync();
  }
  // f(source, node z, its weights there) for the sources of the cell
  auto each_source = [&](auto f) {
    if (!src_here) return;
    for (unsigned m = src_mine; m; m &= m - 1) {
      const int s = __builtin_ctz(m);
      const double* ws = a.src_w + ((long long)s * S + l) * NV;
      double w[n][NV];
#pragma unroll
      for (int z = 0; z < n; ++z)
#pragma unroll
        for (int v = 0; v < NV; ++v) w[z][v] = ws[(long long)z * F * NV + v];
#pragma unroll
      for (int z = 0; z < n; ++z) f(s, z, w[z]);
    }
  };

  // R = S - div F of the line's states y, without the point sources
  auto rhs = [&](const double (&y)[n][NV], double (&R)[n][NV]) {
    double Sv[n][NV];
#pragma unroll
    for (int z = 0; z < n; ++z) {
      sched_fence();
      double Fl[DIM][NV];
      PDE::fluxes(y[z], P, a.pde, Fl);
      if constexpr (PDE::kHasSource) PDE::source(y[z], P, a.pde, Sv[z]);
#pragma unroll
      for (int d = 0; d < XL; ++d)
#pragma unroll
        for (int v = 0; v < NV; ++v) rows[(d * NV + v) * n + z][lane] = Fl[d][v];
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const double f = Fl[LAST][v];
#pragma unroll
        for (int i = 0; i < n; ++i) R[i][v] = z == 0 ? Dz[i][z] * f : fma_r(Dz[i][z], f, R[i][v]);
      }
#pragma unroll
      for (int d = 0; d < XD; ++d)
#pragma unroll
        for (int v = 0; v < NV; ++v)
          R[z][v] = d < XL ? fma_r(coef[d][0], Fl[d][v], R[z][v]) : mfma_div(d, Fl[d][v], R[z][v]);
    }
    if constexpr (XL > 0) {
      line_wave_sync();
      // the other lines' fluxes, one (axis, quantity) ahead of its use
      constexpr int NG = XL * NV;
      double x[2][n][n];
      auto fetch = [&](int g, double (&o)[n][n]) {
#pragma unroll
        for (int z = 0; z < n; ++z)
#pragma unroll
          for (int r = 1; r < n; ++r) o[z][r] = row_read<GN::ALONE>(&rows[g * n + z][unit[g / NV][r]]);
      };
      fetch(0, x[0]);
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        sched_fence();
        if (g + 1 < NG) fetch(g + 1, x[(g + 1) & 1]);
#pragma unroll
        for (int z = 0; z < n; ++z)
#pragma unroll
          for (int r = 1; r < n; ++r) R[z][g % NV] = fma_r(coef[g / NV][r], x[g & 1][z][r], R[z][g % NV]);
      }
      sched_fence();
      line_wave_sync();
    }
    if constexpr (PDE::kHasSource) {
#pragma unroll
      for (int z = 0; z < n; ++z)
#pragma unroll
        for (int v = 0; v < NV; ++v) R[z][v] += Sv[z][v];
    }
  };

  double q[n][n][NV];  // [time][node of the line][quantity]: the iterate, then its right-hand sides

  auto load_u = [&](double (&u)[n][NV]) {
    const double* Qc = Q0c + opaque_zero();
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int z = 0; z < n; ++z) u[z][v] = Qc[v * S + z * F];
  };
  // the point sources of every time node, added to the R_j that q holds
  auto add_sources = [&]() {
    each_source([&](int s, int z, const double (&w)[NV]) {
#pragma unroll
      for (int j = 0; j < n; ++j) {
        const double amp = src_amp[s * NA + j];
#pragma unroll
        for (int v = 0; v < NV; ++v) q[j][z][v] += amp * w[v];
      }
    });
  };
  // q_i = u + dt sum_j KW_ij R_j, R_j held in q[j]
  auto update = [&]() {
    double u[n][NV];
    load_u(u);
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int z = 0; z < n; ++z) {
        sched_fence();
        double t[n];
#pragma unroll
        for (int i = 0; i < n; ++i) {
          double s = u[z][v];
#pragma unroll
          for (int j = 0; j < n; ++j) s = fma_r(Kt[i][j], q[j][z][v], s);
          t[i] = s;
        }
#pragma unroll
        for (int i = 0; i < n; ++i) q[i][z][v] = t[i];
      }
  };

  const int I = a.picard_iters;
  int r0 = 0;
  if (MODE == kLineCerk || (MODE == kLineSources && a.guess == ADG_GUESS_CERK)) {
    // the continuous extension of the classical Runge-Kutta method on the
    // cell-local ODE, taken at the time nodes (see predict_kernel_n64)
    double Y[n][NV];
    load_u(Y);
#pragma unroll
    for (int j = 0; j < n; ++j)
#pragma unroll
      for (int z = 0; z < n; ++z)
#pragma unroll
        for (int v = 0; v < NV; ++v) q[j][z][v] = Y[z][v];
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      double kk[n][NV];
      rhs(Y, kk);
      each_source([&](int s, int z, const double (&w)[NV]) {
        const double amp = src_amp[s * NA + n + (st == 0 ? 0 : (st == 3 ? 2 : 1))];
#pragma unroll
        for (int v = 0; v < NV; ++v) kk[z][v] += amp * w[v];
      });
#pragma unroll
      for (int j = 0; j < n; ++j) {
        const double b = dt * T::cerk_b(st, j);
#pragma unroll
        for (int z = 0; z < n; ++z)
#pragma unroll
          for (int v = 0; v < NV; ++v) q[j][z][v] += b * kk[z][v];
      }
      const double as = (st == 2 ? 1.0 : 0.5) * dt;  // Y_{s+1} = u + dt a_{s+1} k_s
      load_u(Y);
#pragma unroll
      for (int z = 0; z < n; ++z)
#pragma unroll
        for (int v = 0; v < NV; ++v) Y[z][v] += as * kk[z][v];
    }
  } else {
    // first Picard step: q^0 = u^n at every time node, so every slice has
    // the same right-hand side apart from point sources
    double u[n][NV], R[n][NV];
    load_u(u);
    rhs(u, R);
#pragma unroll
    for (int j = 0; j < n; ++j)
#pragma unroll
      for (int z = 0; z < n; ++z)
#pragma unroll
        for (int v = 0; v < NV; ++v) q[j][z][v] = R[z][v];
    add_sources();
    update();
    r0 = 1;
  }
  for (int r = r0; r < I; ++r) {
#pragma unroll
    for (int j = 0; j < n; ++j) {
      double R[n][NV];
      rhs(q[j], R);
#pragma unroll
      for (int z = 0; z < n; ++z)
#pragma unroll
        for (int v = 0; v < NV; ++v) q[j][z][v] = R[z][v];
    }
    add_sources();
    update();
  }

  // time averages of the last iterate (READING: the averaged terms use the
  // final iterate), node by node of the line: q-bar and F-bar along the first
  // axis go to LDS, the other F-bar stay in registers in place of the node's
  // slices
  constexpr int QR = 0, FR = NV * n;  // rows of q-bar and of one axis's F-bar
  double vol[n][NV], Fo[XD][n][NV];   // S-bar, then the volume term; F-bar of axes 1 ..
#pragma unroll
  for (int z = 0; z < n; ++z) {
    sched_fence();
    double qb[NV], Fb[DIM][NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      vol[z][v] = 0.0;
      qb[v] = T::w(0) * q[0][z][v];
#pragma unroll
      for (int j = 1; j < n; ++j) qb[v] = fma_r(T::w(j), q[j][z][v], qb[v]);
      rows[QR + v * n + z][lane] = qb[v];
    }
#pragma unroll
    for (int j = 0; j < n; ++j) {
      double Fl[DIM][NV];
      PDE::fluxes(q[j][z], P, a.pde, Fl);
#pragma unroll
      for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int d = 0; d < DIM; ++d) Fb[d][v] = j == 0 ? T::w(0) * Fl[d][v] : fma_r(T::w(j), Fl[d][v], Fb[d][v]);
      if constexpr (PDE::kHasSource) {
        double Sv[NV];
        PDE::source(q[j][z], P, a.pde, Sv);
#pragma unroll
        for (int v = 0; v < NV; ++v) vol[z][v] += T::w(j) * Sv[v];
      }
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      rows[FR + v * n + z][lane] = Fb[0][v];
      if constexpr (MF)
#pragma unroll
        for (int d = 0; d < XD; ++d) vol[z][v] = mfma_div(d, Fb[d][v], vol[z][v]);
#pragma unroll
      for (int d = 1; d < DIM; ++d) {
        Fo[d - 1][z][v] = Fb[d][v];
        pin(Fo[d - 1][z][v]);
      }
    }
  }
  each_source([&](int s, int z, const double (&w)[NV]) {
    double amp = 0.0;
#pragma unroll
    for (int j = 0; j < n; ++j) amp += T::w(j) * src_amp[s * NA + j];
#pragma unroll
    for (int v = 0; v < NV; ++v) vol[z][v] += amp * w[v];
  });

  // Face projection and volume term, an axis at a time.  Along the first XD
  // axes the lane at position p projects the line through node p of the last
  // axis, so that every lane has one line; along the last axis each lane has
  // its own.
  double* const trc = traces + cl * (long long)(2 * DIM * 2 * NV * F);
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    if (d > 0 && d < LAST) {
      sched_fence();
      line_wave_sync();
#pragma unroll
      for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int z = 0; z < n; ++z) rows[FR + v * n + z][lane] = Fo[d - 1][z][v];
    }
    line_wave_sync();
    const int p = d < LAST ? pos[d < XD ? d : 0] : 0;
    const int st = d == 0 ? 1 : STEP1;
    const int first = d < LAST ? base - p * st : lane;
    // face-node index: the other coordinates, lower axis first
    const int f = d == LAST ? l : (DIM == 2 ? p : (d == 0 ? pos[1] : pos[0]) + n * p);
    double* const tr = trc + 2 * d * 2 * NV * F + f;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      sched_fence();
      double e0 = 0.0, e1 = 0.0, f0 = 0.0, f1 = 0.0;
#pragma unroll
      for (int m = 0; m < n; ++m) {
        const double x = d < LAST ? rows[QR + v * n + p][first + m * st] : rows[QR + v * n + m][lane];
        const double g = d < LAST ? rows[FR + v * n + p][first + m * st] : Fo[XD - 1][m][v];
        e0 = m == 0 ? T::l0(m) * x : fma_r(T::l0(m), x, e0);
        e1 = m == 0 ? T::l1(m) * x : fma_r(T::l1(m), x, e1);
        f0 = m == 0 ? T::l0(m) * g : fma_r(T::l0(m), g, f0);
        f1 = m == 0 ? T::l1(m) * g : fma_r(T::l1(m), g, f1);
      }
      if (d == LAST) {
        double x[n], y[n];
#pragma unroll
        for (int m = 0; m < n; ++m) x[m] = Fo[XD - 1][m][v];
        line_deriv<double, n>(x, y, mih);
#pragma unroll
        for (int z = 0; z < n; ++z) vol[z][v] += y[z];
      } else if (!MF) {
        const int dd = d < XD ? d : 0;
#pragma unroll
        for (int z = 0; z < n; ++z)
#pragma unroll
          for (int r = 0; r < n; ++r)
            vol[z][v] = fma_r(coef[dd][r], row_read<GN::ALONE>(&rows[FR + v * n + z][unit[dd][r]]), vol[z][v]);
      }
      pin(e0), pin(e1), pin(f0), pin(f1);
#pragma unroll
      for (int z = 0; z < n; ++z) pin(vol[z][v]);
      if (active) {
        tr[(0 * NV + v) * F] = e0;  // low face, state
        tr[(1 * NV + v) * F] = f0;  // low face, normal flux
        tr[(2 * NV + v) * F] = e1;  // high face, state
        tr[(3 * NV + v) * F] = f1;  // high face, normal flux
      }
    }
  }
  if (active) {
    double un[n][NV];
    load_u(un);
    const long long c0 = cell * (long long)(NV * S) + l;
    if (a.qcopy) {
      // (a limited step's copy of u^n)
#pragma unroll
      for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int z = 0; z < n; ++z) a.qcopy[c0 + v * S + z * F] = un[z][v];
    }
    double* const Qo = Qout + c0;
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int z = 0; z < n; ++z) Qo[v * S + z * F] = fma_r(dt, vol[z][v], un[z][v]);
  }
}

}  // namespace adg
