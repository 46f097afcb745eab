// DSOLVE of the EXCMG cascade (the exact solve of the two coarsest grids, Algorithm 1) for gfx950, grids of at most
// kDstMax cells per axis.
//
// With zero Dirichlet data M is diagonalised by the products of DST-I vectors s_p(i) = sin(pi p i / N): M S = S Lambda
// with lambda = c0 + 2 sum c_d C_d + 4 sum c_de C_d C_e, C_d = cos(pi p_d / N_d), and S^2 = (Nx Ny Nz / 8) I, so
// M^-1 b = (8 / (Nx Ny Nz)) S Lambda^-1 S b: three dense sine transforms, a division, three more.  The boundary values of
// u, the record of the solve's residual and the outcome that the host reads at the cascade's end go along.
//   - up to 1024 unknowns: one workgroup, one unknown per thread, everything in LDS (8^3 cells: 17 us,
//     where boundary, solve through memory and copy took 2.5 + 21 + 3 us, with a gap of 4 us before each);
//   - above: four launches over the planes and columns of the grid (x and y transforms of a plane; z transform,
//     division and z transform of 64 columns; y and x transforms of a plane; the residual).  52 x 44 x 36 cells in one
//     workgroup took 2.7 ms, its 20 M multiply-adds fed from memory by one CU; in four launches 96 us.
#include <math.h>

#include "cg_device.h"
#include "excmg_internal.h"

namespace excmg {

namespace {

constexpr int kDirectSmall = 1024;  // unknowns of the one-workgroup form
constexpr int DP = 512;             // threads of a plane workgroup
constexpr int kDpk = (kDstMax - 1) * (kDstMax - 1) / DP + 1;  // unknowns of a plane per thread at most

// tab[(p-1) L + (q-1)] = sin(pi p q / N), p, q = 1 .. L = N - 1; half: LDS of 2 N doubles
__device__ __forceinline__ void sine_table(double *tab, double *half, int N, int nt) {
  const int L = N - 1;
  for (int m = threadIdx.x; m < 2 * N; m += nt) half[m] = sinpi((double)m / N);
  __syncthreads();
  for (int e = threadIdx.x; e < L * L; e += nt) tab[e] = half[((e / L + 1) * (e % L + 1)) % (2 * N)];
  __syncthreads();
}

__device__ __forceinline__ double eigenvalue(const Stencil &s, double Cx, double Cy, double Cz) {
  return s.c0 + 2.0 * (s.cx * Cx + s.cy * Cy + s.cz * Cz) +
         4.0 * (s.cxy * Cx * Cy + s.cxz * Cx * Cz + s.cyz * Cy * Cz);
}

// the outcome of the solve, in the CG state and for the host
__device__ void direct_outcome(const Direct &a, double rho, double bb) {
  CgState *cs = a.cs;
  const double bnorm2 = bb + cs->gbnd2;
  cs->iter = 0;
  cs->rho = rho;
  cs->rho0 = rho;
  cs->bnorm2 = bnorm2;
  cs->status = (isfinite(rho) && isfinite(bnorm2)) ? 0 : EXCMG_ERR_BREAKDOWN;
  cs->done = 1;
  if (a.out) {
    set_outcome(cs, a.out, rho, rho, bnorm2, 0, cs->status);
    a.out->abort = 0;
  }
}

__device__ __forceinline__ double dirichlet(const Direct &a, int i, int j, int k) {
  return a.gdat ? a.gdat[a.rs.gf.at(i * a.rs.s, j * a.rs.s, k * a.rs.s)] : 0.0;
}

__device__ __forceinline__ void direct_small_body(const Direct &a) {
  extern __shared__ double lds[];
  __shared__ double sh[2][kDirectSmall / 64];
  const Grid g = a.g;
  const int nt = blockDim.x, m = threadIdx.x;
  if (a.mark && m == 0) *a.mark = (long long)wall_clock64();
  const int Lx = g.nx - 1, Ly = g.ny - 1, Lz = g.nz - 1, n = Lx * Ly * Lz;
  double *P = lds, *Sx = P + n, *Sy = Sx + Lx * Lx, *Sz = Sy + Ly * Ly, *half = Sz + Lz * Lz;
  const bool own = m < n;
  const int i = m % Lx, j = (m / Lx) % Ly, k = own ? m / (Lx * Ly) : 0;
  double b = 0.0, b2 = 0.0;
  if (own) {
    double rf;
    b = rhs_at(a.rs, g.nx, g.ny, g.nz, i + 1, j + 1, k + 1, rf);
    b2 = stop_norm_term(a.rs, b, rf);
    P[m] = b;
  }
  const int nodes = (g.nx + 1) * (g.ny + 1) * (g.nz + 1);
  for (int e = m; e < nodes; e += nt) {
    const int x = e % (g.nx + 1), yz = e / (g.nx + 1), y = yz % (g.ny + 1), z = yz / (g.ny + 1);
    if (x == 0 || y == 0 || z == 0 || x == g.nx || y == g.ny || z == g.nz) a.u[g.at(x, y, z)] = dirichlet(a, x, y, z);
  }
  sine_table(Sx, half, g.nx, nt);
  sine_table(Sy, half, g.ny, nt);
  sine_table(Sz, half, g.nz, nt);
  // v = sum over the line of tab[q][t] * src, t: the unknown's place on the line
  auto transform = [&](const double *tab, int L, int t, int stride) {
    const double *src = P + m - t * stride;
    double v = 0.0;
    if (own)
      for (int q = 0; q < L; ++q) v += tab[q * L + t] * src[q * stride];
    __syncthreads();
    return v;
  };
  auto store = [&](double v) {
    if (own) P[m] = v;
    __syncthreads();
  };
  store(transform(Sx, Lx, i, 1));
  store(transform(Sy, Ly, j, Lx));
  const double lam = eigenvalue(a.st, cospi((double)(i + 1) / g.nx), cospi((double)(j + 1) / g.ny),
                                cospi((double)(k + 1) / g.nz));
  store(transform(Sz, Lz, k, Lx * Ly) * (8.0 / ((double)g.nx * g.ny * g.nz) / lam));
  store(transform(Sx, Lx, i, 1));
  store(transform(Sy, Ly, j, Lx));
  const double u = transform(Sz, Lz, k, Lx * Ly);
  store(u);
  double r2 = 0.0;
  if (own) {
    a.u[g.at(i + 1, j + 1, k + 1)] = u;
    auto X = [&](int di, int dj, int dk) {
      const int x = i + di, y = j + dj, z = k + dk;
      return x < 0 || y < 0 || z < 0 || x >= Lx || y >= Ly || z >= Lz ? 0.0 : P[(z * Ly + y) * Lx + x];
    };
    const Stencil &s = a.st;
    double v = s.c0 * u + s.cx * (X(1, 0, 0) + X(-1, 0, 0)) + s.cy * (X(0, 1, 0) + X(0, -1, 0)) +
               s.cz * (X(0, 0, 1) + X(0, 0, -1));
    v += s.cxy * ((X(1, 1, 0) + X(-1, 1, 0)) + (X(1, -1, 0) + X(-1, -1, 0)));
    v += s.cxz * ((X(1, 0, 1) + X(-1, 0, 1)) + (X(1, 0, -1) + X(-1, 0, -1)));
    v += s.cyz * ((X(0, 1, 1) + X(0, -1, 1)) + (X(0, 1, -1) + X(0, -1, -1)));
    r2 = (b - v) * (b - v);
  }
  r2 = wave_sum(r2);
  b2 = wave_sum(b2);
  if ((m & 63) == 0) {
    sh[0][m >> 6] = r2;
    sh[1][m >> 6] = b2;
  }
  __syncthreads();
  if (m == 0) {
    double rho = 0.0, bb = 0.0;
    for (int q = 0; q < nt / 64; ++q) {
      rho += sh[0][q];
      bb += sh[1][q];
    }
    direct_outcome(a, rho, bb);
  }
}

// The transforms of one plane (P: LDS, Ly rows of Lx): along x and along y, in place; each thread keeps its results
// in registers until all have read.
__device__ __forceinline__ void plane_transform(double *P, const double *tab, int L, int Lx, int np, bool along_y) {
  double v[kDpk];
#pragma unroll
  for (int q = 0; q < kDpk; ++q) {
    const int e = threadIdx.x + q * DP;
    v[q] = 0.0;
    if (e < np) {
      const int i = e % Lx, j = e / Lx, t = along_y ? j : i;
      const double *src = along_y ? P + i : P + j * Lx;
      const int stride = along_y ? Lx : 1;
      double x = 0.0;
      for (int p = 0; p < L; ++p) x += tab[p * L + t] * src[p * stride];
      v[q] = x;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kDpk; ++q)
    if (threadIdx.x + q * DP < np) P[threadIdx.x + q * DP] = v[q];
  __syncthreads();
}

__device__ __forceinline__ double plane_sum(double v, double *sh) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double t = 0.0;
  for (int q = 0; q < DP / 64; ++q) t += sh[q];
  return t;
}

// plane k: u's boundary values, b (kept in B), its transforms along x and y into A, and the plane's part of the
// stopping norm
__device__ __forceinline__ void direct_forward_body(const Direct &a, int bid) {
  extern __shared__ double lds[];
  __shared__ double sh[DP / 64];
  const Grid g = a.g;
  const int k = bid, Lx = g.nx - 1, Ly = g.ny - 1, np = Lx * Ly;
  const bool end = k == 0 || k == g.nz;
  if (a.mark && k == 0 && threadIdx.x == 0) *a.mark = (long long)wall_clock64();
  for (int e = threadIdx.x; e < (g.nx + 1) * (g.ny + 1); e += DP) {
    const int x = e % (g.nx + 1), y = e / (g.nx + 1);
    if (end || x == 0 || y == 0 || x == g.nx || y == g.ny) a.u[g.at(x, y, k)] = dirichlet(a, x, y, k);
  }
  if (end) return;
  double *P = lds, *S = P + np, *half = S + max(Lx * Lx, Ly * Ly);
  double b2 = 0.0;
  for (int e = threadIdx.x; e < np; e += DP) {
    const int i = 1 + e % Lx, j = 1 + e / Lx;
    double rf;
    const double b = rhs_at(a.rs, g.nx, g.ny, g.nz, i, j, k, rf);
    b2 += stop_norm_term(a.rs, b, rf);
    a.B[g.at(i, j, k)] = b;
    P[e] = b;
  }
  const double t = plane_sum(b2, sh);
  if (threadIdx.x == 0) a.parts[2 * (g.nz - 1) + k - 1] = t;
  sine_table(S, half, g.nx, DP);
  plane_transform(P, S, Lx, Lx, np, false);
  sine_table(S, half, g.ny, DP);
  plane_transform(P, S, Ly, Lx, np, true);
  for (int e = threadIdx.x; e < np; e += DP) a.A[g.at(1 + e % Lx, 1 + e / Lx, k)] = P[e];
}

constexpr int DC = 64, DCT = 512;  // columns and threads of a column workgroup
constexpr int kDck = ((kDstMax - 1) * DC + DCT - 1) / DCT;

// 64 columns: the transform along z, the division by the eigenvalues, the transform back
__device__ __forceinline__ void direct_columns_body(const Direct &a, int bid) {
  extern __shared__ double lds[];
  const Grid g = a.g;
  const int Lx = g.nx - 1, Ly = g.ny - 1, Lz = g.nz - 1, nc = Lx * Ly;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int c = min(bid * DC + lane, nc - 1), i = 1 + c % Lx, j = 1 + c / Lx;  // lanes past the last repeat it
  double *P = lds, *S = P + Lz * DC, *half = S + Lz * Lz;
  for (int k = w; k < Lz; k += DCT / 64) P[k * DC + lane] = a.A[g.at(i, j, k + 1)];
  sine_table(S, half, g.nz, DCT);
  const double Cx = cospi((double)i / g.nx), Cy = cospi((double)j / g.ny);
  const double scale = 8.0 / ((double)g.nx * g.ny * g.nz);
  for (int back = 0; back < 2; ++back) {
    double v[kDck];
#pragma unroll
    for (int q = 0; q < kDck; ++q) {
      const int k = w + q * (DCT / 64);
      double x = 0.0;
      if (k < Lz) {
        for (int p = 0; p < Lz; ++p) x += S[p * Lz + k] * P[p * DC + lane];
        if (back == 0) x *= scale / eigenvalue(a.st, Cx, Cy, cospi((double)(k + 1) / g.nz));
      }
      v[q] = x;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kDck; ++q) {
      const int k = w + q * (DCT / 64);
      if (k < Lz) P[k * DC + lane] = v[q];
    }
    __syncthreads();
  }
  if (bid * DC + lane < nc)
    for (int k = w; k < Lz; k += DCT / 64) a.A[g.at(i, j, k + 1)] = P[k * DC + lane];
}

// plane k: the transforms along y and x back, into u
__device__ __forceinline__ void direct_backward_body(const Direct &a, int bid) {
  extern __shared__ double lds[];
  const Grid g = a.g;
  const int k = 1 + bid, Lx = g.nx - 1, Ly = g.ny - 1, np = Lx * Ly;
  double *P = lds, *S = P + np, *half = S + max(Lx * Lx, Ly * Ly);
  for (int e = threadIdx.x; e < np; e += DP) P[e] = a.A[g.at(1 + e % Lx, 1 + e / Lx, k)];
  sine_table(S, half, g.ny, DP);
  plane_transform(P, S, Ly, Lx, np, true);
  sine_table(S, half, g.nx, DP);
  plane_transform(P, S, Lx, Lx, np, false);
  for (int e = threadIdx.x; e < np; e += DP) a.u[g.at(1 + e % Lx, 1 + e / Lx, k)] = P[e];
}

// the residual b - M u of plane k; the last workgroup records the outcome
__device__ __forceinline__ void direct_residual_body(const Direct &a, int bid) {
  const Grid g = a.g;
  const int k = 1 + bid, Lx = g.nx - 1, np = Lx * (g.ny - 1);
  const Stencil &s = a.st;
  double v[2] = {0.0, threadIdx.x == 0 ? a.parts[2 * (g.nz - 1) + k - 1] : 0.0}, tot[2];
  for (int e = threadIdx.x; e < np; e += DP) {
    const int i = 1 + e % Lx, j = 1 + e / Lx;
    auto X = [&](int di, int dj, int dk) {
      const int x = i + di, y = j + dj, z = k + dk;
      return x <= 0 || y <= 0 || z <= 0 || x >= g.nx || y >= g.ny || z >= g.nz ? 0.0 : a.u[g.at(x, y, z)];
    };
    double m = s.c0 * X(0, 0, 0) + s.cx * (X(1, 0, 0) + X(-1, 0, 0)) + s.cy * (X(0, 1, 0) + X(0, -1, 0)) +
               s.cz * (X(0, 0, 1) + X(0, 0, -1));
    m += s.cxy * ((X(1, 1, 0) + X(-1, 1, 0)) + (X(1, -1, 0) + X(-1, -1, 0)));
    m += s.cxz * ((X(1, 0, 1) + X(-1, 0, 1)) + (X(1, 0, -1) + X(-1, 0, -1)));
    m += s.cyz * ((X(0, 1, 1) + X(0, -1, 1)) + (X(0, 1, -1) + X(0, -1, -1)));
    const double r = a.B[g.at(i, j, k)] - m;
    v[0] += r * r;
  }
  if (last_sums<2, DP>(v, a.parts, &a.cs->count, bid, g.nz - 1, tot) && threadIdx.x == 0)
    direct_outcome(a, tot[0], tot[1]);
}

// entry e of a batch
__device__ __forceinline__ Direct direct_of(const BatchList &L, int e) {
  const BatchEntry &E = entry_at(L, e);
  Direct a;
  a.g = E.g;
  a.u = as_global(E.u);
  a.rs = E.rs;
  a.rs.f = as_global(E.rs.f);
  a.rs.g = as_global(E.rs.g);
  a.gdat = as_global(E.gb);
  a.st = E.st;
  a.cs = as_global(E.cs);
  a.out = nullptr;
  a.mark = nullptr;
  a.A = as_global(E.r);
  a.B = as_global(E.p0);
  a.parts = as_global(E.parts);
  return a;
}

__global__ __launch_bounds__(kDirectSmall) void direct_small_kernel(Direct a) { direct_small_body(a); }
__global__ __launch_bounds__(DP) void direct_forward_kernel(Direct a) { direct_forward_body(a, blockIdx.x); }
__global__ __launch_bounds__(DCT) void direct_columns_kernel(Direct a) { direct_columns_body(a, blockIdx.x); }
__global__ __launch_bounds__(DP) void direct_backward_kernel(Direct a) { direct_backward_body(a, blockIdx.x); }
__global__ __launch_bounds__(DP) void direct_residual_kernel(Direct a) { direct_residual_body(a, blockIdx.x); }

// one grid to a y of the launch; x covers the largest grid
__global__ __launch_bounds__(kDirectSmall) void b_direct_small_kernel(BatchList L) {
  direct_small_body(direct_of(L, blockIdx.x));
}
__global__ __launch_bounds__(DP) void b_direct_forward_kernel(BatchList L) {
  const Direct a = direct_of(L, blockIdx.y);
  if ((int)blockIdx.x <= a.g.nz) direct_forward_body(a, blockIdx.x);
}
__global__ __launch_bounds__(DCT) void b_direct_columns_kernel(BatchList L) {
  const Direct a = direct_of(L, blockIdx.y);
  if ((int)blockIdx.x * DC < (a.g.nx - 1) * (a.g.ny - 1)) direct_columns_body(a, blockIdx.x);
}
__global__ __launch_bounds__(DP) void b_direct_backward_kernel(BatchList L) {
  const Direct a = direct_of(L, blockIdx.y);
  if ((int)blockIdx.x < a.g.nz - 1) direct_backward_body(a, blockIdx.x);
}
__global__ __launch_bounds__(DP) void b_direct_residual_kernel(BatchList L) {
  const Direct a = direct_of(L, blockIdx.y);
  if ((int)blockIdx.x < a.g.nz - 1) direct_residual_body(a, blockIdx.x);
}

// LDS of the kernels for grids of at most the given unknowns and cells
size_t small_lds(int n, int nx, int ny, int nz) {
  const int Lx = nx - 1, Ly = ny - 1, Lz = nz - 1;
  return (size_t)(n + Lx * Lx + Ly * Ly + Lz * Lz + 2 * std::max(nx, std::max(ny, nz))) * sizeof(double);
}
size_t plane_lds(int nx, int ny) {
  const int Lx = nx - 1, Ly = ny - 1;
  return (size_t)(Lx * Ly + std::max(Lx * Lx, Ly * Ly) + 2 * std::max(nx, ny)) * sizeof(double);
}
size_t column_lds(int nz) { return (size_t)((nz - 1) * DC + (nz - 1) * (nz - 1) + 2 * nz) * sizeof(double); }

}  // namespace

bool direct_small(const Grid &g) { return g.interior() <= kDirectSmall; }

void launch_direct(const Direct &a, hipStream_t st) {
  const Grid &g = a.g;
  const int nc = (g.nx - 1) * (g.ny - 1), Lz = g.nz - 1;
  if (direct_small(g)) {
    direct_small_kernel<<<1, (nc * Lz + 63) / 64 * 64, small_lds(nc * Lz, g.nx, g.ny, g.nz), st>>>(a);
    return;
  }
  const size_t plane = plane_lds(g.nx, g.ny);
  direct_forward_kernel<<<g.nz + 1, DP, plane, st>>>(a);
  direct_columns_kernel<<<(nc + DC - 1) / DC, DCT, column_lds(g.nz), st>>>(a);
  direct_backward_kernel<<<Lz, DP, plane, st>>>(a);
  direct_residual_kernel<<<Lz, DP, 0, st>>>(a);
}

void launch_b_direct_small(const BatchList &L, int unknowns, const int cells[3], BatchStatus *stat, hipStream_t st) {
  if (L.n == 0) return;
  const size_t lds = small_lds(unknowns, cells[0], cells[1], cells[2]);
  b_direct_small_kernel<<<L.n, (unknowns + 63) / 64 * 64, lds, st>>>(L);
  launch_b_mirror(L, stat, st);
}

void launch_b_direct(const BatchList &L, const int cells[3], BatchStatus *stat, hipStream_t st) {
  const int nc = (cells[0] - 1) * (cells[1] - 1), Lz = cells[2] - 1;
  const size_t plane = plane_lds(cells[0], cells[1]);
  for (int e = 0; e < L.n; e += 65535) {  // (the limit of y)
    BatchList part = L;
    part.ent += e;
    part.n = std::min(L.n - e, 65535);
    b_direct_forward_kernel<<<dim3(Lz + 2, part.n), DP, plane, st>>>(part);
    b_direct_columns_kernel<<<dim3((nc + DC - 1) / DC, part.n), DCT, column_lds(cells[2]), st>>>(part);
    b_direct_backward_kernel<<<dim3(Lz, part.n), DP, plane, st>>>(part);
    b_direct_residual_kernel<<<dim3(Lz, part.n), DP, 0, st>>>(part);
  }
  launch_b_mirror(L, stat, st);
}

}  // namespace excmg
