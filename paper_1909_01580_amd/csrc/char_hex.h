// Reconstruction in characteristic variables on hexahedral grids (Pan & Xu,
// Sec. 4: the option stated after the limiting procedure), static or moving.
//
// For face fs = 2 D + s of a cell (s = 0 the face on the cell's low side
// along index axis D, s = 1 the high one) the stencil data are projected to
// U = L Q, L = R^-1, R the right eigenvectors of the Euler Jacobian along
// the frame of Sec. 3 at the face's centre (n along X_a x X_b, the shear
// fields along X_b x n and X_b), taken at the mean of the two cell averages
// that share the face.  The least squares of Sec. 2 are linear, so the 25
// polynomials of U are L times those of Q; indicators and nonlinear weights
// belong to each characteristic field.  As on box grids, each cell gets six
// reconstructions stored as six coefficient arrays (array fs): row 10 v the
// conservative cell mean of variable v, rows 10 f + 1 .. 10 f + 9 the nine
// coefficients of characteristic field f in the cell's scaled basis.  The
// face flux forms R from the two cells' means and the same frame and
// projects back at its Gauss points: value Q_c + R dU(x), gradient
// R grad U(x).  The positivity fallback stays on the conservative
// polynomials (the mask of the component-wise reconstruction).
#pragma once

#include "char_basis.h"
#include "hex_kernels.h"

namespace hgks {

// One workgroup of twelve waves per tile of 128 cells: of each 64 cells six
// waves, wave = face, reconstruct the six faces.  What does not depend on the
// face is formed once per cell and shared through LDS: the sums of the big
// stencil's normal equations (15 of the 90 per wave), its solution (one
// variable per wave), and the 24 sub-stencil fits (one per wave and round,
// four rounds; every wave then projects the round's six).  One lane per cell
// repeated the 24 fits for every face, 48,600 vector instructions per cell
// in one serial chain at two waves per SIMD; here a lane runs 6,930, six of
// them per cell, at three waves per SIMD: 463 -> 254 us per launch on
// 56x41x36 cells (mixed).  Twelve waves fill a compute unit evenly; of
// workgroups of six only one fitted (310 us).
constexpr int kQX = 8, kQY = 4, kQZ = 4, kQCells = kQX * kQY * kQZ, kQLanes = 6 * kQCells;
using CharTile = HexTileOf<kQX, kQY, kQZ>;
constexpr int kQBuf = 90;  // doubles per cell of the exchange buffer: 6 fits of 15, or 45 + 45 sums

// Rows of L (characteristic projection) along a frame, in the combinations
// that need fewest products: with s = (b2 rho - b1 V.M + b1 E)/2 and t =
// (u_n rho - n.M)/(2 c) the fields are s + t, rho - 2 s, M.t1 - v1 rho,
// M.t2 - v2 rho, s - t.
struct CharRows {
  double s[5], t[4], u1[4], u2[4];
};

HGKS_FN void char_rows(const CharFrame& B, CharRows& R) {
  R.s[0] = 0.5 * B.b2;
  R.s[4] = 0.5 * B.b1;
  R.t[0] = 0.5 * B.ic * B.un;
  R.u1[0] = -B.v1;
  R.u2[0] = -B.v2;
  for (int e = 0; e < 3; ++e) {
    R.s[1 + e] = -0.5 * B.b1 * B.V[e];
    R.t[1 + e] = -0.5 * B.ic * B.n[e];
    R.u1[1 + e] = B.t1[e];
    R.u2[1 + e] = B.t2[e];
  }
}

HGKS_FN void char_project(const CharRows& R, double q0, double q1, double q2, double q3, double q4, double (&f)[5]) {
  const double s = R.s[0] * q0 + R.s[1] * q1 + R.s[2] * q2 + R.s[3] * q3 + R.s[4] * q4;
  const double t = R.t[0] * q0 + R.t[1] * q1 + R.t[2] * q2 + R.t[3] * q3;
  f[0] = s + t;
  f[1] = q0 - 2.0 * s;
  f[2] = R.u1[0] * q0 + R.u1[1] * q1 + R.u1[2] * q2 + R.u1[3] * q3;
  f[3] = R.u2[0] * q0 + R.u2[1] * q1 + R.u2[2] * q2 + R.u2[3] * q3;
  f[4] = s - t;
}

// Sums 15 W .. 15 W + 14 of the big stencil's normal equations (the lower
// triangle of the 9 x 9 matrix, then the right-hand sides 9 v + e) of the
// cell of nb, written to buf (kQCells apart).
template <int W, typename NB>
__device__ __forceinline__ void char_normal_sums(const NB& nb, const HexCell& Ci, const double (&qc)[5],
                                                 double* buf) {
  double acc[15];
#pragma unroll
  for (int k = 0; k < 15; ++k) acc[k] = 0.0;
#pragma unroll 1
  for (int s = 0; s < 27; ++s) {
    const int ox = s % 3 - 1, oy = (s / 3) % 3 - 1, oz = s / 9 - 1;
    const int nz = (ox != 0) + (oy != 0) + (oz != 0);
    if (nz == 0 || nz == 3) continue;
    double d[3], mo[6], dq[5], r[9];
    nb.template get<true>(ox, oy, oz, Ci, qc, d, mo, dq);
    big_row(d, mo, Ci, r);
#pragma unroll
    for (int k = 0; k < 15; ++k) {
      constexpr int tri[9] = {0, 1, 3, 6, 10, 15, 21, 28, 36};
      const int m = 15 * W + k;
      if (m < 45) {
        int p = 0;
        while (p < 8 && tri[p + 1] <= m) ++p;
        acc[k] += r[p] * r[m - tri[p]];
      } else {
        acc[k] += r[(m - 45) % 9] * dq[(m - 45) / 9];
      }
    }
  }
#pragma unroll
  for (int k = 0; k < 15; ++k) buf[(15 * W + k) * kQCells] = acc[k];
}

// Linear fit of sub-stencil m (uniform over the wave) of tile cell `base`,
// all five variables, written to out (kQCells apart, 3 v + e): sub_fit with
// the inverse first and then one variable at a time, which holds few
// registers beside the caller's sums.
__device__ __forceinline__ void char_sub_fit(const CharTile& T, int base, double ih, int m, double* out) {
  int o[4][3];
  sub_offsets(m, o);
  int at[4];
  double d[4][3], A[6];
#pragma unroll
  for (int e = 0; e < 6; ++e) A[e] = 0.0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    at[r] = base + (o[r][2] * CharTile::HY + o[r][1]) * CharTile::HX + o[r][0];
#pragma unroll
    for (int e = 0; e < 3; ++e) d[r][e] = (T.c[e][at[r]] - T.c[e][base]) * ih;
    A[0] += d[r][0] * d[r][0];
    A[1] += d[r][1] * d[r][1];
    A[2] += d[r][2] * d[r][2];
    A[3] += d[r][0] * d[r][1];
    A[4] += d[r][1] * d[r][2];
    A[5] += d[r][0] * d[r][2];
  }
  double I[6] = {A[1] * A[2] - A[4] * A[4], A[0] * A[2] - A[5] * A[5], A[0] * A[1] - A[3] * A[3],
                 A[5] * A[4] - A[3] * A[2], A[3] * A[5] - A[0] * A[4], A[3] * A[4] - A[1] * A[5]};
  const double idet = d_rcp(A[0] * I[0] + A[3] * I[3] + A[5] * I[5]);
#pragma unroll
  for (int e = 0; e < 6; ++e) I[e] *= idet;
  asm volatile("" ::: "memory");
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    double r[3] = {0.0, 0.0, 0.0};
    const double qv = T.q[v][base];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double dq = T.q[v][at[k]] - qv;
#pragma unroll
      for (int e = 0; e < 3; ++e) r[e] += d[k][e] * dq;
    }
    out[(3 * v + 0) * kQCells] = I[0] * r[0] + I[3] * r[1] + I[5] * r[2];
    out[(3 * v + 1) * kQCells] = I[3] * r[0] + I[1] * r[1] + I[4] * r[2];
    out[(3 * v + 2) * kQCells] = I[5] * r[0] + I[4] * r[1] + I[2] * r[2];
    asm volatile("" ::: "memory");
  }
}

template <typename TS>
__global__ void __launch_bounds__(kQLanes) __attribute__((amdgpu_waves_per_eu(3)))
    k_char_recon_hex(HexGrid H, const double* __restrict__ geo, const double* __restrict__ q, TS* __restrict__ faces,
                     size_t fs_stride, WenoParams<double> P, double gamma, size_t N, unsigned ntx, unsigned nty,
                     unsigned ntiles) {
  __shared__ CharTile T;
  __shared__ double buf[kQBuf][kQCells];
  const unsigned b = xcd_block(blockIdx.x, gridDim.x);
  if (b >= ntiles) return;
  const int tx = (int)(b % ntx), ty = (int)((b / ntx) % nty), tz = (int)(b / (ntx * nty));
  const int o0 = tx * kQX, o1 = ty * kQY, o2 = tz * kQZ;
  stage_hex_tile<kQLanes>(H, geo, q, N, o0, o1, o2, T);
  __syncthreads();
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int fs = wave % 6;  // wave = face of 64 of the cells
  const int lane = wave / 6 * 64 + (int)(threadIdx.x & 63u);
  const int lx = lane % kQX, ly = (lane / kQX) % kQY, lz = lane / (kQX * kQY);
  // lanes of cells beyond the grid work on the tile's (wrapped) cells and
  // write nothing; every lane reaches every barrier
  const int i = o0 + lx, j = o1 + ly, k = o2 + lz;
  const bool live = i < H.n[0] && j < H.n[1] && k < H.n[2];
  const int base = ((lz + 1) * CharTile::HY + (ly + 1)) * CharTile::HX + (lx + 1);
  const NbrTile<CharTile> nb{T, base};
  // the cell itself, all from the tile but h
  const int ci = live ? i : 0, cj = live ? j : 0, ck = live ? k : 0;
  const size_t idx = ((size_t)ck * H.n[1] + cj) * H.n[0] + ci;
  HexCell Ci;
  Ci.h = geo[10 * N + idx];
  Ci.ih = geo[11 * N + idx];
#pragma unroll
  for (int e = 0; e < 3; ++e) Ci.c[e] = T.c[e][base];
#pragma unroll
  for (int e = 0; e < 6; ++e) Ci.m[e] = T.m[e][base] * (Ci.ih * Ci.ih);
  double qc[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) qc[v] = T.q[v][base];
  double* const col = &buf[0][lane];
  switch (fs) {
    case 0: char_normal_sums<0>(nb, Ci, qc, col); break;
    case 1: char_normal_sums<1>(nb, Ci, qc, col); break;
    case 2: char_normal_sums<2>(nb, Ci, qc, col); break;
    case 3: char_normal_sums<3>(nb, Ci, qc, col); break;
    case 4: char_normal_sums<4>(nb, Ci, qc, col); break;
    default: char_normal_sums<5>(nb, Ci, qc, col); break;
  }
  __syncthreads();
  if (fs < 5) {
    // variable fs of P_0, in place of its right-hand side
    double L[45], a[9];
#pragma unroll
    for (int e = 0; e < 45; ++e) L[e] = col[e * kQCells];
    chol9(L);
#pragma unroll
    for (int e = 0; e < 9; ++e) a[e] = col[(45 + 9 * fs + e) * kQCells];
    chol9_solve(L, a);
#pragma unroll
    for (int e = 0; e < 9; ++e) col[(45 + 9 * fs + e) * kQCells] = a[e];
  }
  __syncthreads();
  // the face's projection; P_0 projected waits in the cell's rows of the
  // face array (read back below by the lane that wrote it)
  constexpr int CB = kCB<TS>;
  TS* const out = faces + (size_t)fs * fs_stride + coef_cell<TS>(idx);
  CharRows R;
  {
    const int D = fs >> 1, side = fs & 1;
    const int step = D == 0 ? 1 : (D == 1 ? CharTile::HX : CharTile::HX * CharTile::HY);
    const int nbr = base + (side ? step : -step);
    double Qb[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) Qb[v] = 0.5 * (T.q[v][base] + T.q[v][nbr]);
    double n[3], t1[3], t2[3];
    face_centre_frame(H, D, ci + (D == 0 ? side : 0), cj + (D == 1 ? side : 0), ck + (D == 2 ? side : 0), n, t1, t2);
    CharFrame B;
    char_frame(Qb, n, t1, t2, gamma, B);
    char_rows(B, R);
  }
  double beta0[5], r0[5];
  {
    // a field's nine coefficients at a time (all 45 and the rows of L would
    // pass the register budget)
    auto field = [&](int f, const double (&c)[9]) {
      double cr[9];
#pragma unroll
      for (int e = 0; e < 9; ++e) {
        const TS stored = TS(c[e]);
        if (live) out[(10 * f + 1 + e) * CB] = stored;
        cr[e] = (double)stored;
      }
      beta0[f] = hex_beta0(cr, Ci);
      r0[f] = d_rcp(beta0[f] + P.eps);
      asm volatile("" : "+v"(beta0[f])::"memory");
    };
    double c[9], s[9], t[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) {
      const double* a = col + (45 + e) * kQCells;
      s[e] = R.s[0] * a[0] + R.s[1] * a[9 * kQCells] + R.s[2] * a[18 * kQCells] + R.s[3] * a[27 * kQCells] +
             R.s[4] * a[36 * kQCells];
      t[e] = R.t[0] * a[0] + R.t[1] * a[9 * kQCells] + R.t[2] * a[18 * kQCells] + R.t[3] * a[27 * kQCells];
    }
#pragma unroll
    for (int e = 0; e < 9; ++e) c[e] = s[e] + t[e];
    field(0, c);
#pragma unroll
    for (int e = 0; e < 9; ++e) c[e] = s[e] - t[e];
    field(4, c);
#pragma unroll
    for (int e = 0; e < 9; ++e) c[e] = col[(45 + e) * kQCells] - 2.0 * s[e];
    field(1, c);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const double(&w)[4] = u ? R.u2 : R.u1;
#pragma unroll
      for (int e = 0; e < 9; ++e) {
        const double* a = col + (45 + e) * kQCells;
        c[e] = w[0] * a[0] + w[1] * a[9 * kQCells] + w[2] * a[18 * kQCells] + w[3] * a[27 * kQCells];
      }
      field(2 + u, c);
    }
  }
  // weights affine in tau, as in the component-wise reconstruction
  double tsum[5], rsum[5], db[5][3];
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    tsum[f] = rsum[f] = 0.0;
    db[f][0] = db[f][1] = db[f][2] = 0.0;
  }
#pragma unroll 1
  for (int round = 0; round < 4; ++round) {
    __syncthreads();  // the previous contents of buf are consumed
    char_sub_fit(T, base, Ci.ih, 6 * round + fs, col + 15 * fs * kQCells);
    __syncthreads();
#pragma unroll 1
    for (int m = 0; m < 6; ++m) {
      const double* bq = col + 15 * m * kQCells;
      double bu[5][3];
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        double f[5];
        char_project(R, bq[e * kQCells], bq[(3 + e) * kQCells], bq[(6 + e) * kQCells], bq[(9 + e) * kQCells],
                     bq[(12 + e) * kQCells], f);
#pragma unroll
        for (int v = 0; v < 5; ++v) bu[v][e] = f[v];
      }
#pragma unroll
      for (int f = 0; f < 5; ++f) {
        const double bm = bu[f][0] * bu[f][0] + bu[f][1] * bu[f][1] + bu[f][2] * bu[f][2];
        tsum[f] += fabs(beta0[f] - bm);
        const double rm = d_rcp(bm + P.eps);
        rsum[f] += rm;
        const double dr = rm - r0[f];
#pragma unroll
        for (int e = 0; e < 3; ++e) db[f][e] += dr * bu[f][e];
      }
    }
  }
  if (!live) return;
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    const double tau = tsum[f] * (1.0 / 24.0);
    const double w0r = 1.0 + tau * r0[f];
    const double iS = d_rcp(P.gamma0 * w0r + P.Gamma * (24.0 + tau * rsum[f]));
    const double w0g = w0r * iS;  // wbar_0 / gamma_0
    TS* cv = out + 10 * f * CB;
#pragma unroll
    for (int e = 0; e < 9; ++e) {
      const double au = (double)cv[(1 + e) * CB];
      cv[(1 + e) * CB] = TS(e < 3 ? w0g * au + iS * P.Gamma * tau * db[f][e] : w0g * au);
    }
    cv[0] = TS(T.q[f][base]);  // the conservative mean of variable f
  }
}

}  // namespace hgks
