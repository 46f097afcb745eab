// Two-step CG sweeps of the EXCMG relaxation for gfx950: two iterations of Algorithm 1's CG in two passes over the grid.
#include <math.h>

#include "cg_device.h"
#include "excmg_internal.h"

namespace excmg {

namespace {

// ------------------------------------------------------------------------------------------------ two-step sweeps
//
// Two CG iterations (k, k + 1) in two sweeps over the grid, each bound by HBM bytes:
//   pass G:  p = r + beta p_old, q = M p, t = M q; partial sums of p.q, r.q, q.q, q.t, r.t     reads r, p_old
//   pass U:  p, q again; r1 = r - alpha q, p1 = r1 + beta0 p, q1 = M p1,
//            u += alpha p + alpha1 p1, r2 = r1 - alpha1 q1; partial sums for the next step      reads r, p_old, u;
//                                                                                              writes r2, p1, u
// 64 bytes per unknown and two iterations (16 + 48; 48 in a grid's first pair, where p = r) where two sweeps an
// iteration move 128.  The coefficients of the second iteration come from pass G's sums (two_after_g), which are
// exact consequences of r1 = r - alpha q and p1 = r1 + beta0 p, so the iterates are CG's; the residual norms that the
// stopping test and beta use are summed directly in pass U.
// Measured at 511^3 unknowns in FP64: pass G 0.57 ms, pass U 1.39 ms (4.6 TB/s of its 48 bytes), 1.97 ms a pair, where
// two iterations of the two-pass form take 3.1 ms; in FP32 1.13 against 2.0 ms; at 255^3 0.26 against 0.38 ms.  Pass G is
// bound by its LDS reads and vector instructions (half of each unit's time in a step, with a barrier between), pass U by
// HBM.  What does not depend on the data is kept out of the vector instructions for that: masks that a whole wave shares
// are branches, nodes outside the grid are zeroed once and their threads write to a spare row, and offsets stay 32 bits
// (98 vector instructions a step and wave instead of 138: pass G 0.63 -> 0.57 ms at 511^3, 106 -> 89 us at 255^3, in
// FP32 427 -> 355 us).
//
// Tile: a wavefront covers one 64-node row segment, each lane two rows (12 LDS reads for two nodes instead of 18),
// MW such waves the rows of the region where q (or p1) is needed (2 MW rows: the output rows and one more on each
// side), one more wave the region's two outer columns; output 64 x (2 MW - 2).  Every thread loads its own two nodes
// of r and p_old (whole cache lines) and at most one node of the outer ring that p needs besides (2 nodes out).  One
// barrier per plane: step s stages plane s of p and the q of plane s - 2 (kept in registers by the threads that
// formed it), then forms q of plane s - 1 and the second product of plane s - 3.
template <int TY>
struct Two {
  static constexpr int MW = TY == 16 ? 15 : (TY == 8 ? 7 : 3);  // waves over rows
  static constexpr int RP = TY == 16 ? 1 : 2;    // rows per lane
  static constexpr int NT = 64 * (MW + 1);
  static constexpr int QH = RP * MW, QW = TX + 2;  // region of q
  static constexpr int PH = QH + 2, PW = TX + 4;  // region of p
  static constexpr int OH = QH - 2;               // output rows
  static constexpr int Ring = 2 * PW + 2 * QH;    // nodes of p's region outside q's
  static_assert(Ring <= NT, "one ring node per thread at most");
};

// plane k >= 0 of an array in layout g (a plane is under 2^32 bytes: two scalar multiplications)
template <typename T>
__device__ __forceinline__ T *plane_of(T *a, const Grid &g, int k) {
  return at_plane(a + g.off, (unsigned)(g.sz * (long long)sizeof(T)), (unsigned)k);
}

// T: precision; D: planes of loads in flight; FIRST: p = r (no p_old).  P: the policy of the pass: mid(m, row, off, k, r,
// p, q) at q's plane k (row: the tile puts out row m of plane k; returns the staged second operand), fin(m, row, off, k,
// c, t) two planes behind (c: the second operand there, t: M of it); center<S>() for the pass's own loads, place(m, ...)
// once for the node's place in the pass's other arrays, lane: whether the thread's column lies in the grid.
template <typename T, int D, int TY, bool FIRST, typename P>
__device__ __forceinline__ void march2(const Sweep &sw, const T *rin, const T *pin, const Grid &gp, T beta, P &pol,
                                       T (*tp)[Two<TY>::PH + 1][Two<TY>::PW],
                                       T (*tq)[Two<TY>::QH + 2][Two<TY>::QW], int bid,
                                       int nb, bool remap) {
  using W = Two<TY>;
  constexpr int U = D % 2 == 0 ? D : 2 * D;
  constexpr int RP = W::RP, NL = RP + 1;  // own rows; loads per array and plane
  const Grid &g = sw.g;
  const int t = remap ? xcd_remap(bid, nb) : bid;
  const int bx = t % sw.ntx;
  const int rest = t / sw.ntx;
  const int by = rest % sw.nty, bz = rest / sw.nty;
  const int i0 = 1 + bx * TX, j0 = 1 + by * W::OH, k0 = 1 + bz * sw.zc;
  const int k1 = min(k0 + sw.zc, g.nz);
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool side = w == W::MW;
  const int sl = min(lane, 2 * W::MW - 1);  // side wave: lanes past its nodes repeat the last one
  const int d = side ? ((sl & 1) ? W::QW - 1 : 0) : lane + 1;
  const int b0 = RP * (side ? sl >> 1 : w);
  const int i = i0 - 1 + d, j = j0 - 1 + b0;
  // rows of the tile that are output nodes of the grid: the same for a whole wave
  bool in[RP], row[RP];
  unsigned offR[NL], offP[NL];
  int wp[RP], wq[RP];
  const bool xin = i >= 1 && i < g.nx;
  const unsigned ci = clampi(i, 1, g.nx - 1);
#pragma unroll
  for (int m = 0; m < RP; ++m) {
    in[m] = xin && j + m >= 1 && j + m < g.ny;
    const int b = RP * w + m;
    row[m] = !side && b >= 1 && b <= W::QH - 2 && j0 - 1 + b < g.ny;
    const unsigned cj = clampi(j + m, 1, g.ny - 1);
    offR[m] = (cj * (unsigned)g.sy + ci) * (unsigned)sizeof(T);
    offP[m] = (cj * (unsigned)gp.sy + ci) * (unsigned)sizeof(T);
    pol.place(m, ci, cj);
    // a node outside the grid is 0 in both buffers for good, and its thread writes to the spare row
    wp[m] = in[m] ? b0 + 1 + m : W::PH;
    wq[m] = in[m] ? b0 + 1 + m : W::QH + 1;
  }
  pol.lane = xin;
  // ring node of p's region
  int ra, rc;
  {
    const int e = min(tid, W::Ring - 1);
    if (e < 2 * W::PW) {
      ra = e < W::PW ? 0 : W::PH - 1;
      rc = e < W::PW ? e : e - W::PW;
    } else {
      const int f = e - 2 * W::PW;
      ra = 1 + (f >> 1);
      rc = (f & 1) ? W::PW - 1 : 0;
    }
  }
  const int gi = i0 - 2 + rc, gj = j0 - 2 + ra;
  if (!(gi >= 1 && gi < g.nx && gj >= 1 && gj < g.ny)) ra = W::PH;
  for (int e = tid; e < 2 * (W::PH + 1) * W::PW; e += W::NT) (&tp[0][0][0])[e] = T(0);
  for (int e = tid; e < 2 * (W::QH + 2) * W::QW; e += W::NT) (&tq[0][0][0])[e] = T(0);
  __syncthreads();
  {
    const unsigned cj = clampi(gj, 1, g.ny - 1), cx = clampi(gi, 1, g.nx - 1);
    offR[RP] = (cj * (unsigned)g.sy + cx) * (unsigned)sizeof(T);
    offP[RP] = (cj * (unsigned)gp.sy + cx) * (unsigned)sizeof(T);
  }
  T rr[D][NL], pp[D][NL];
  auto fetch = [&](T(&r)[NL], T(&p)[NL], int kk) {
    const int kc = clampi(kk, 1, g.nz - 1);
    const T *rb = plane_of(rin, g, kc);
#pragma unroll
    for (int m = 0; m < NL; ++m) r[m] = *at_byte(rb, offR[m]);
    if constexpr (!FIRST) {
      const T *pb = plane_of(pin, gp, kc);
#pragma unroll
      for (int m = 0; m < NL; ++m) p[m] = *at_byte(pb, offP[m]);
    }
  };
  auto val = [&](T r, T p) { return FIRST ? r : r + beta * p; };
  const Stencil &st = sw.st;
  const T c0 = (T)st.c0, cx = (T)st.cx, cy = (T)st.cy, cz = (T)st.cz;
  const T cxy = (T)st.cxy, cxz = (T)st.cxz, cyz = (T)st.cyz;
  // column sums of one product: S = cz C + cxz X + cyz Y of the last plane, A = its in-plane part plus the S before it
  T S1[RP] = {}, A1[RP] = {}, S2[RP] = {}, A2[RP] = {};
  T rown[RP] = {}, pown[RP] = {}, qreg[RP] = {}, cprev[RP] = {};
  const int ns = k1 - k0 + 5;
#pragma unroll
  for (int q = 0; q < D; ++q) fetch(rr[q], pp[q], k0 - 2 + q);
  static_for<D>([&](auto qc) {  // step q's own loads are of plane k0 - 3 + q
    constexpr int q = decltype(qc)::value;
    pol.template center<q>(offR, clampi(k0 - 3 + q, k0, k1 - 1));
  });
  auto body = [&](auto pb, auto pr, int s) {
    const int PB = pb;  // LDS buffer of the step
    constexpr int PR = decltype(pr)::value;  // register set of the step
    const int kp = k0 - 2 + s;
    const bool kin = kp >= 1 && kp < g.nz;
    // the offsets are new to the compiler in every step (and block of it): it would else keep them widened to 64 bits and
    // add them to the planes' bases in vector registers
#pragma unroll
    for (int m = 0; m < NL; ++m) {
      __asm__ volatile("" : "+v"(offR[m]));
      if constexpr (!FIRST) __asm__ volatile("" : "+v"(offP[m]));
    }
    T rnew[RP], pnew[NL] = {};
    if (kin) {
      __asm__ volatile("");  // a branch, not selects
#pragma unroll
      for (int m = 0; m < NL; ++m) pnew[m] = val(rr[PR][m], pp[PR][m]);
    }
#pragma unroll
    for (int m = 0; m < RP; ++m) {
      rnew[m] = rr[PR][m];
      tp[PB][wp[m]][d + 1] = pnew[m];
      tq[PB][wq[m]][d] = qreg[m];
    }
    tp[PB][ra][rc] = pnew[RP];
    __syncthreads();
    fetch(rr[PR], pp[PR], kp + D);
    {  // q = M p of plane kp - 1 at the own nodes
      T c[RP + 2], x[RP + 2];
#pragma unroll
      for (int a = 0; a < RP + 2; ++a) {
        const T *row = &tp[PB][b0 + a][d];
        c[a] = row[1];
        x[a] = row[0] + row[2];
      }
      const int k = kp - 1;
      const bool kq = k >= 1 && k < g.nz, ko = k >= k0 && k < k1;
#pragma unroll
      for (int m = 0; m < RP; ++m) {
        const T y = c[m] + c[m + 2];
        const T S = cz * c[m + 1] + cxz * x[m + 1] + cyz * y;
        const T q = A1[m] + S;
        A1[m] = S1[m] + (c0 * c[m + 1] + cx * x[m + 1] + cy * y + cxy * (x[m] + x[m + 2]));
        S1[m] = S;
        qreg[m] = pol.template mid<PR>(m, ko && row[m], offR[m], k, rown[m], pown[m], q);
        if (!kq) {
          __asm__ volatile("");
          qreg[m] = T(0);
        }
        rown[m] = rnew[m];
        pown[m] = c[m + 1];
      }
      pol.template center<PR>(offR, clampi(k + D, k0, k1 - 1));
    }
    __builtin_amdgcn_sched_barrier(0);  // the second product's LDS reads stay behind the first's (registers)
    if (!side) {  // the second product of plane kp - 3
      T c[RP + 2], x[RP + 2];
#pragma unroll
      for (int a = 0; a < RP + 2; ++a) {
        const T *row = &tq[PB][b0 + a][d - 1];
        c[a] = row[1];
        x[a] = row[0] + row[2];
      }
      const int k = kp - 3;
      const bool ko = k >= k0 && k < k1;
#pragma unroll
      for (int m = 0; m < RP; ++m) {
        const T y = c[m] + c[m + 2];
        const T S = cz * c[m + 1] + cxz * x[m + 1] + cyz * y;
        const T o = A2[m] + S;
        A2[m] = S2[m] + (c0 * c[m + 1] + cx * x[m + 1] + cy * y + cxy * (x[m] + x[m + 2]));
        S2[m] = S;
        pol.fin(m, ko && row[m], offR[m], k, cprev[m], o);
        cprev[m] = c[m + 1];
      }
    }
  };
  if constexpr (D == 1) {
#pragma unroll 1
    for (int s = 0; s < ns; s += 2) {
      body(0, std::integral_constant<int, 0>{}, s);
      if (s + 1 < ns) body(1, std::integral_constant<int, 0>{}, s + 1);
    }
  } else {
    int s = 0;
    for (; s + U <= ns; s += U) {
      static_for<U>([&](auto sc) {
        constexpr int q = decltype(sc)::value;
        body(std::integral_constant<int, q % 2>{}, std::integral_constant<int, q % D>{}, s + q);
      });
    }
    static_for<U>([&](auto sc) {
      constexpr int q = decltype(sc)::value;
      if (s + q < ns) body(std::integral_constant<int, q % 2>{}, std::integral_constant<int, q % D>{}, s + q);
    });
  }
}

template <typename T, int RP>
struct PolG {
  T r2[RP] = {}, r3[RP] = {};  // r of the two planes behind rown's
  // (of all lanes, whether their nodes lie in the grid or not: those of the others are left out at the end)
  double pq = 0, rq = 0, qq = 0, qt = 0, rt = 0;
  bool lane;
  __device__ __forceinline__ void place(int, unsigned, unsigned) {}
  template <int S>
  __device__ __forceinline__ void center(const unsigned (&)[RP + 1], int) {}
  template <int S>
  __device__ __forceinline__ T mid(int m, bool row, unsigned &, int, T r, T p, T q) {
    if (row) {
      __asm__ volatile("");
      pq += (double)p * (double)q;
      rq += (double)r * (double)q;
      qq += (double)q * (double)q;
    }
    rcur[m] = r;
    return q;
  }
  T rcur[RP];
  __device__ __forceinline__ void fin(int m, bool row, unsigned &, int, T c, T t) {
    if (row) {
      __asm__ volatile("");
      qt += (double)c * (double)t;
      rt += (double)r3[m] * (double)t;
    }
    r3[m] = r2[m];
    r2[m] = rcur[m];
  }
};

template <typename T, int D, bool NTP, int RP>
struct PolU {
  T *u, *rout, *pout;
  Grid gu, gpo;  // layouts of u and r, and of pout
  unsigned offo[RP];
  T alpha, alpha1, beta0;
  bool single, lane;
  T uu[D][RP];
  T s2[RP] = {}, s3[RP] = {}, scur[RP];  // r1 of this plane and the two behind
  double rho1 = 0, rho2 = 0, cs = 0, cd = 0;
  __device__ __forceinline__ void place(int m, unsigned ci, unsigned cj) {
    offo[m] = (cj * (unsigned)gpo.sy + ci) * (unsigned)sizeof(T);
  }
  template <int S>
  __device__ __forceinline__ void center(const unsigned (&own)[RP + 1], int k) {
    const T *ub = plane_of(u, gu, k);
#pragma unroll
    for (int m = 0; m < RP; ++m) uu[S][m] = ld1<NTP>(at_byte(ub, own[m]));
  }
  template <int S>
  __device__ __forceinline__ T mid(int m, bool row, unsigned &own, int k, T r, T p, T q) {
    const T r1 = r - alpha * q;
    const T v = single ? p : r1 + beta0 * p;
    if (row && lane) {
      __asm__ volatile("" : "+v"(own), "+v"(offo[m]));
      st1<NTP>(uu[S][m] + alpha * p + alpha1 * v, at_byte(plane_of(u, gu, k), own));
      st1<NTP>(v, at_byte(plane_of(pout, gpo, k), offo[m]));
      rho1 += (double)r1 * (double)r1;
      cs += (double)r1 * (double)r;
    }
    scur[m] = r1;
    return v;
  }
  __device__ __forceinline__ void fin(int m, bool row, unsigned &own, int k, T, T t) {
    if (row && lane) {
      __asm__ volatile("" : "+v"(own));
      const T r1 = s3[m];
      const T r2 = r1 - alpha1 * t;
      st1<NTP>(r2, at_byte(plane_of(rout, gu, k), own));
      rho2 += (double)r2 * (double)r2;
      cd += (double)r2 * (double)r1;
    }
    s3[m] = s2[m];
    s2[m] = scur[m];
  }
};

// After pass G: alpha, and the second iteration's beta0 and alpha1.  With r1 = r - alpha q and p1 = r1 + beta0 p,
//   r1.r1 = r.r - 2 alpha r.q + alpha^2 q.q,
//   p1.M p1 = r.Mr + alpha^2 q.t + beta0^2 p.q - 2 alpha r.t + 2 beta0 r.q - 2 alpha beta0 q.q,
// and r.Mr = r.q - beta r.M p_old, where alpha_old M p_old = r_old - r (cross = r.r_old was summed in the last pass U).
// Only one iteration is taken (single) where the first already ends the solve, or where r1.r1 is so far below r.r that
// the difference above has lost its digits.
template <typename T>
__device__ void two_after_g(CgState *cs, const double (&v)[5]) {
  const double pq = v[0], rq = v[1], qq = v[2], qt = v[3], rt = v[4];
  cs->pq = pq;
  if (!(pq > 0.0) || !isfinite(pq)) {
    cs->status = EXCMG_ERR_BREAKDOWN;
    cs->done = 1;
    return;
  }
  const double rho = cs->rho, a = rho / pq;
  cs->alpha = a;
  cs->alpha1 = 0.0;
  cs->beta0 = 0.0;
  cs->single = 1;
  const double rho1 = rho - 2.0 * a * rq + a * a * qq;
  const double least = sizeof(T) == 8 ? 1e-6 : 1e-4;
  if (!(rho1 > least * rho) || rho1 <= cs->stop2 || cs->iter + 1 >= cs->max_iters) return;
  const double b = rho1 / rho;
  const double rmr = cs->pairs == 0 ? pq : rq - cs->beta * (cs->cross - rho) / cs->alast;
  const double pq1 = rmr + a * a * qt + b * b * pq - 2.0 * a * rt + 2.0 * b * rq - 2.0 * a * b * qq;
  if (!(pq1 > 0.0) || !isfinite(pq1)) return;
  cs->beta0 = b;
  cs->alpha1 = rho1 / pq1;
  cs->single = 0;
}

// After pass U: the one or two iterations it made are counted, and the stopping test taken (Algorithm 1).
__device__ void two_after_u(CgState *cs, const double (&v)[4]) {
  const double rho1 = v[0], rho2 = v[1];
  const bool single = cs->single != 0;
  const double before = single ? cs->rho : rho1, rho = single ? rho1 : rho2;
  int it = cs->iter + 1;
  auto record = [&](double x) {
    if (cs->hist_on && it < EXCMG_MAX_HISTORY) cs->hist[it] = cs->bnorm2 > 0.0 ? sqrt(x / cs->bnorm2) : 0.0;
  };
  record(rho1);
  if (!single) {
    ++it;
    record(rho2);
  }
  cs->rho_old = before;
  cs->rho = rho;
  cs->beta = rho / before;
  cs->cross = single ? v[2] : v[3];
  cs->alast = single ? cs->alpha : cs->alpha1;
  cs->iter = it;
  cs->pairs += 1;
  if (!isfinite(rho)) {
    cs->status = EXCMG_ERR_BREAKDOWN;
    cs->done = 1;
  } else if (rho <= cs->stop2) {
    cs->done = 1;
  } else if (it >= cs->max_iters) {
    cs->status = EXCMG_ERR_NOCONV;
    cs->done = 1;
  }
}

// Buffers of pair n: (r, p) go from R (p = r) to (P0, P1), then alternate between (P0, P1) and (R, X).
template <typename T>
struct TwoBufs {
  const T *r, *p;
  T *ro, *po;
  Grid gp, gpo;
};
template <typename T>
__device__ __forceinline__ TwoBufs<T> two_bufs(int n, const TwoVecs<T> &v, const Grid &g) {
  TwoBufs<T> b;
  const bool odd = n & 1;
  b.r = odd ? v.p0 : v.r;
  b.p = odd ? v.p1 : v.x;
  b.gp = odd ? g : v.gx;
  b.ro = odd ? v.r : v.p0;
  b.po = odd ? v.x : v.p1;
  b.gpo = odd ? v.gx : g;
  return b;
}

template <typename T, int D, int TY>
__device__ __forceinline__ bool two_g(const Sweep &sw, const TwoVecs<T> &vec, CgState *cs, double *parts, int bid,
                                      int nb, bool remap) {
  using W = Two<TY>;
  __shared__ T tp[2][W::PH + 1][W::PW];
  __shared__ T tq[2][W::QH + 2][W::QW];
  const int n = cs->pairs;
  const TwoBufs<T> b = two_bufs(n, vec, sw.g);
  PolG<T, W::RP> pol;
  if (n == 0) march2<T, D, TY, true>(sw, b.r, b.r, sw.g, T(0), pol, tp, tq, bid, nb, remap);
  else march2<T, D, TY, false>(sw, b.r, b.p, b.gp, (T)cs->beta, pol, tp, tq, bid, nb, remap);
  double v[5] = {pol.pq, pol.rq, pol.qq, pol.qt, pol.rt}, tot[5];
#pragma unroll
  for (int k = 0; k < 5; ++k) v[k] = pol.lane ? v[k] : 0.0;
  if (!last_sums<5, W::NT>(v, parts, &cs->count, bid, nb, tot)) return false;
  if (threadIdx.x == 0 && !cs->tune) two_after_g<T>(cs, tot);
  return true;
}

template <typename T, int D, bool NTP, int TY>
__device__ __forceinline__ bool two_u(const Sweep &sw, const TwoVecs<T> &vec, CgState *cs, double *parts, int bid,
                                      int nb, bool remap) {
  using W = Two<TY>;
  __shared__ T tp[2][W::PH + 1][W::PW];
  __shared__ T tq[2][W::QH + 2][W::QW];
  const int n = cs->pairs;
  const TwoBufs<T> b = two_bufs(n, vec, sw.g);
  PolU<T, D, NTP, W::RP> pol;
  pol.u = vec.u;
  pol.rout = b.ro;
  pol.pout = b.po;
  pol.gu = sw.g;
  pol.gpo = b.gpo;
  pol.alpha = (T)cs->alpha;
  pol.alpha1 = (T)cs->alpha1;
  pol.beta0 = (T)cs->beta0;
  pol.single = cs->single != 0;
  if (n == 0) march2<T, D, TY, true>(sw, b.r, b.r, sw.g, T(0), pol, tp, tq, bid, nb, remap);
  else march2<T, D, TY, false>(sw, b.r, b.p, b.gp, (T)cs->beta, pol, tp, tq, bid, nb, remap);
  double v[4] = {pol.rho1, pol.rho2, pol.cs, pol.cd}, tot[4];
  if (!last_sums<4, W::NT>(v, parts, &cs->count, bid, nb, tot)) return false;
  if (threadIdx.x == 0 && !cs->tune) two_after_u(cs, tot);
  return true;
}

// waves per SIMD that pass U is built for: its FP64 form with two rows per lane needs 170 registers
template <typename T, int TY>
constexpr int two_u_waves() { return sizeof(T) == 8 && TY != 16 ? 3 : 4; }

template <typename T, int D, int TY>
__global__ __launch_bounds__(Two<TY>::NT) __attribute__((amdgpu_waves_per_eu(4))) void two_g_kernel(Sweep sw, TwoVecs<T> vec, CgState *cs, double *parts) {
  if (cs->done) return;
  two_g<T, D, TY>(sw, vec, cs, parts, blockIdx.x, gridDim.x, true);
}

template <typename T, int D, bool NTP, int TY>
__global__ __launch_bounds__(Two<TY>::NT) __attribute__((amdgpu_waves_per_eu(two_u_waves<T, TY>()))) void two_u_kernel(Sweep sw, TwoVecs<T> vec, CgState *cs, double *parts) {
  if (cs->done) return;
  two_u<T, D, NTP, TY>(sw, vec, cs, parts, blockIdx.x, gridDim.x, true);
}

}  // namespace

// f(height) for the tile height of a sweep
template <typename F>
static void with_two_height(const Sweep &sw, F &&f) {
  switch (sw.ty) {
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 16: f(std::integral_constant<int, 16>{}); break;
    default: f(std::integral_constant<int, 4>{}); break;
  }
}

// Planes of loads in flight (DEEP: the sweep's depth is over 2).  FP64 takes what its registers allow: one plane in
// pass G with two rows per lane (at 128 registers, so that two workgroups share a CU: 635 us at 511^3 unknowns against
// 745 us with two planes at 184 registers), else two.  FP32 with one row per lane has room for
// three.
template <typename T, int TY, bool DEEP>
constexpr int two_depth_g() { return sizeof(T) == 8 ? (TY == 16 ? 2 : 1) : (DEEP && TY == 16 ? 3 : 2); }
template <typename T, int TY, bool DEEP>
constexpr int two_depth_u() { return sizeof(T) == 4 && DEEP && TY == 16 ? 3 : 2; }

Sweep two_sweep(const Sweep &sw) {
  Sweep t = sw;
  const int oh = sw.ty == 16 ? Two<16>::OH : (sw.ty == 8 ? Two<8>::OH : Two<4>::OH);
  t.nty = (sw.g.ny - 1 + oh - 1) / oh;
  return t;
}

// The shape of a two-step sweep that was neither tuned nor set.  A workgroup steps through zc planes and about ten
// more (five of halo and pipeline, the rest its start and its sums), and the launch takes as many rounds as its
// workgroups need of the slots that are resident at once, so the time is rounds x (zc + 10) x the time of a step.  The
// slots follow from the registers; the steps' times are measured at 511^3 unknowns (the model gives 256^3's and
// 128^3's best chunks too: pass G, 16 rows, chunks of 64 / 86 / 128 planes at 255^3: 148 / 96 / 138 us predicted,
// 143 / 97 / 132 measured).
Sweep two_default(const Grid &g, const Stencil &st, bool fp32, bool pass_u, int nt) {
  struct Kind {
    int ty, slots;
    double step;
  };
  static const Kind kinds[2][2][3] = {
      {{{4, 1024, 1.35}, {8, 512, 1.48}, {16, 256, 1.0}}, {{4, 768, 1.92}, {8, 256, 1.75}, {16, 256, 2.0}}},
      {{{4, 1024, 0.85}, {8, 512, 0.88}, {16, 256, 0.73}}, {{4, 1024, 1.63}, {8, 512, 1.76}, {16, 256, 1.11}}}};
  Sweep best = make_sweep(g, st, 0, 3, nt, 4);
  double least = 1e300;
  for (const Kind &k : kinds[fp32][pass_u]) {
    for (int parts = 1; parts <= (g.nz - 1 + 1) / 2 && parts <= 512; ++parts) {
      const int zc = ((g.nz - 1 + parts - 1) / parts + 1) & ~1;
      const Sweep sw = make_sweep(g, st, zc, 3, nt, k.ty);
      const long long nb = sweep_blocks(two_sweep(sw));
      const double cost = (double)((nb + k.slots - 1) / k.slots) * (sw.zc + 10) * k.step;
      if (cost < least) {
        least = cost;
        best = sw;
      }
      if (nb > 64LL * k.slots) break;  // shorter chunks only add halo planes
    }
  }
  return best;
}

template <typename T>
void launch_two_g(const Sweep &swA, const TwoVecs<T> &v, CgState *cs, double *parts, hipStream_t st) {
  const Sweep sw = two_sweep(swA);
  with_two_height(sw, [&](auto ty) {
    constexpr int TY = decltype(ty)::value;
    const int nb = sweep_blocks(sw);
    if (sw.depth > 2) two_g_kernel<T, two_depth_g<T, TY, true>(), TY><<<nb, Two<TY>::NT, 0, st>>>(sw, v, cs, parts);
    else two_g_kernel<T, two_depth_g<T, TY, false>(), TY><<<nb, Two<TY>::NT, 0, st>>>(sw, v, cs, parts);
  });
}

template <typename T>
void launch_two_u(const Sweep &swB, const TwoVecs<T> &v, CgState *cs, double *parts, hipStream_t st) {
  const Sweep sw = two_sweep(swB);
  with_two_height(sw, [&](auto ty) {
    constexpr int TY = decltype(ty)::value;
    const int nb = sweep_blocks(sw);
    auto go = [&](auto nt) {
      constexpr bool NTP = decltype(nt)::value;
      if (sw.depth > 2)
        two_u_kernel<T, two_depth_u<T, TY, true>(), NTP, TY><<<nb, Two<TY>::NT, 0, st>>>(sw, v, cs, parts);
      else
        two_u_kernel<T, two_depth_u<T, TY, false>(), NTP, TY><<<nb, Two<TY>::NT, 0, st>>>(sw, v, cs, parts);
    };
    if (sw.nt) go(std::true_type{});
    else go(std::false_type{});
  });
}

template void launch_two_g<double>(const Sweep &, const TwoVecs<double> &, CgState *, double *, hipStream_t);
template void launch_two_g<float>(const Sweep &, const TwoVecs<float> &, CgState *, double *, hipStream_t);
template void launch_two_u<double>(const Sweep &, const TwoVecs<double> &, CgState *, double *, hipStream_t);
template void launch_two_u<float>(const Sweep &, const TwoVecs<float> &, CgState *, double *, hipStream_t);

}  // namespace excmg
