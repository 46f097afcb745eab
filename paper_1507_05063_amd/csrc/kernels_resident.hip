// Resident CG of the EXCMG relaxation for gfx950: the whole CG of a grid in one launch, with the grid's vectors held on
// the chip (at most 8192 unknowns on each of 256 CUs: grids up to 128^3 cells).
//
// Such a grid is bound by latency, not by bytes: as sweeps, an iteration costs one or two launches and, in each, the
// chain from the partial sums through the staged planes to the stores (10 us on 32^3 and 64^3, 31 us on 128^3).  Here a
// workgroup owns a brick of the grid.  u, p, s = M p and w = M r are in registers (ZR nodes of a z column per thread),
// r in LDS with one layer of its neighbours' nodes.  The iteration is Chronopoulos and Gear's form of CG, the same
// Krylov iterates as Algorithm 1's in exact arithmetic, because it takes both inner products from one reduction:
//   gamma = r.r, delta = w.r;  beta = gamma / gamma_old, alpha = gamma / (delta - beta gamma / alpha_old);
//   p = r + beta p, s = w + beta s, u += alpha p, r -= alpha s, w = M r      (p = r, s = w, alpha = gamma / delta first)
// so the grid meets once an iteration.  r of the neighbours' layer is not exchanged but updated here too, from w there,
// which the owners publish before the meeting; every workgroup that holds a node forms the same bits.
//
// The meeting: a workgroup stores its published w and then its two partial sums past its XCD's L2 (agent-scope
// stores, each waited for), and reads the partial sums of all workgroups the same way until none is missing, so that
// there is no counter, no fence (one writes back the whole L2) and one store-to-load latency.  All workgroups add the
// partial sums in one order: the scalars, and so every decision, are the same bits everywhere.  A slot that has not
// been written holds a NaN that no sum produces; slots rotate through three sets, and a workgroup clears its own slot
// of the set after next once all have arrived.  There are no more workgroups than CUs and the host lets such launches
// run at once only where they have room together, so all workgroups of a launch come to run; the wait is bounded
// nevertheless (another process may hold CUs), and a workgroup that gives up says so in the CG state: the host then takes the grid up again
// from its initial guess with the sweeps.  (Others may have got through the same meeting and, if it was the last, have
// written their part of the solution and the outcome: only the give-up counts then.)  Until the host has seen it, later
// launches of the same call end at their first meeting (CgState::looks), instead of waiting once more each.  (A
// cooperative launch would keep launches apart too, but costs about 190 us on this runtime.)
// Measured per iteration (per-grid times of solves capped at 24 and at 4 iterations): 128^3 41 -> 11.5 us (operator and
// updates 4 us, meeting 3, publishing and the layer 4), 64^3 12.3 -> 5.1 us, 32^3 16.8 -> 4.1 us, 16^3 5.0 -> 3.6 us.  A
// launch spends another 113, 32, 26 and 38 us (kernel trace) before its first iteration: u's loads, the right-hand side
// node by node, two operators and the first meeting.
#include <math.h>

#include "cg_device.h"
#include "excmg_internal.h"

namespace excmg {

namespace {

constexpr unsigned long long kMissing = kMissingSlot;

__device__ __forceinline__ void put(double *p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double get(const double *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// a value that is the same in every lane, as a scalar
__device__ __forceinline__ double uniform(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b), hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__global__ void resident_init_kernel(ResidentInit i) { resident_init_block(i); }

__global__ void outcome_kernel(CgState *cs, Outcome *out) {
  set_outcome(cs, out, cs->rho, cs->rho0, cs->bnorm2, cs->iter, cs->status);
  out->abort = 0;
}

// v of another lane of the wave by a DPP move (0 where the move has no source, or in rows outside the mask)
template <int Ctrl, int Rows = 0xf>
__device__ __forceinline__ double dpp(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, Ctrl, Rows, 0xf, true);
  const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), Ctrl, Rows, 0xf, true);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// Sums by DPP moves (a shuffle through LDS takes ten times as long): of the 16 lanes of a row, in its last lane, and of
// the wave, in lane 63.
__device__ __forceinline__ double row_sum(double v) {
  v += dpp<0x111>(v);  // row_shr 1, 2, 4, 8
  v += dpp<0x112>(v);
  v += dpp<0x114>(v);
  v += dpp<0x118>(v);
  return v;
}
__device__ __forceinline__ double wave_sum63(double v) {
  v = row_sum(v);
  v += dpp<0x142, 0xa>(v);  // the row before's last lane, into rows 1 and 3
  v += dpp<0x143, 0xc>(v);  // lane 31, into rows 2 and 3
  return v;
}

// LDS of the meetings of a workgroup of NW waves
template <int NW>
struct Meeting {
  double mine[2][NW];  // the waves' sums of the workgroup's own values
  double sum[2];       // the sums over all workgroups
  int there;           // whether all have arrived
  int looks;           // at the slots before this workgroup gives up
};

// A set of slots: per group of 32 workgroups 32 slots of a and 32 of b, then one line of the groups' sums.
constexpr int kGroup = 32, kGroups = 8;
__host__ __device__ constexpr int set_slots(int groups) { return 2 * kGroup * groups + 2 * kGroups; }
// the three sets of nb workgroups
__host__ __device__ constexpr int slots_of(int nb) { return 3 * set_slots((nb + kGroup - 1) / kGroup); }

// Reads slot p of every lane that has one until none is missing (0 in the other lanes), at most `looks` times; there:
// whether that happened.
__device__ __forceinline__ double await(const double *p, bool mine, int looks, bool &there) {
  double v = 0.0;
  there = false;
  for (int look = 0; !there && look < looks; ++look) {
    if (mine) v = get(p);
    there = __all((unsigned long long)__double_as_longlong(v) != kMissing);
  }
  return v;
}

// a and b summed over all workgroups (the same bits in every one); seq numbers the meetings of the launch.  False: gave
// up waiting.  Up to 32 workgroups read one another's slots; more of them meet by way of the first of every 32, which
// adds up its group, and read the groups' sums (256 workgroups that all read 512 slots get in one another's way: 3.6 us
// a meeting, against 1.2 us among four).
template <int NW>
__device__ __forceinline__ bool meet(double &a, double &b, double *slots, int seq, int bid, int nb, Meeting<NW> &m) {
  const int groups = (nb + kGroup - 1) / kGroup;
  __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");  // what this thread has published has arrived
  a = wave_sum63(a);
  b = wave_sum63(b);
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (lane == 63) {
    m.mine[0][w] = a;
    m.mine[1][w] = b;
  }
  __syncthreads();
  if (w == 0) {
    const int now = (seq % 3) * set_slots(groups), before = ((seq + 2) % 3) * set_slots(groups);
    const int group = bid / kGroup, line = 2 * kGroup * groups;
    const bool writer = lane == 15 || lane == 31, leader = groups == 1 || bid % kGroup == 0;
    const int own = 2 * kGroup * group + (lane >> 4) * kGroup + bid % kGroup;
    double x = row_sum(lane < 32 && (lane & 15) < NW ? m.mine[lane >> 4][lane & 15] : 0.0);
    if (!(x == x)) x = __longlong_as_double(0x7ff8000000000000ll);  // any NaN is the plain one
    if (writer) put(&slots[now + own], x);
    bool there = true;
    if (leader) {
      const bool mine = kGroup * group + (lane & 31) < nb;
      x = row_sum(await(&slots[now + 2 * kGroup * group + lane], mine, m.looks, there));
      x += dpp<0x142, 0xa>(x);  // lane 31: the group's a, lane 63: its b
      if (groups > 1 && there && (lane & 31) == 31) {
        if (!(x == x)) x = __longlong_as_double(0x7ff8000000000000ll);
        put(&slots[now + line + (lane >> 5) * kGroups + group], x);
      }
    }
    if (groups > 1) {
      x = await(&slots[now + line + (lane & 15)], lane < 16 && (lane & 7) < groups, m.looks, there);
      // lanes 7 and 15: the sums of eight
      x += dpp<0x111>(x);
      x += dpp<0x112>(x);
      x += dpp<0x114>(x);
    }
    const int at = groups > 1 ? 7 : 31, step = groups > 1 ? 8 : 32;
    if (lane == at) m.sum[0] = x;
    if (lane == at + step) m.sum[1] = x;
    if (lane == 0) m.there = there;
    // every workgroup has arrived here, so all have left the meeting before: its slots are free
    const double missing = __longlong_as_double((long long)kMissing);
    if (writer) put(&slots[before + own], missing);
    if (groups > 1 && leader && (lane & 31) == 31) put(&slots[before + line + (lane >> 5) * kGroups + group], missing);
  }
  __syncthreads();
  a = uniform(m.sum[0]);
  b = uniform(m.sum[1]);
  return __builtin_amdgcn_readfirstlane(m.there) != 0;
}

// Brick: BX x BY x (ZS ZR) nodes, ZR nodes along z to a thread.
template <int BX, int BY, int ZS, int ZR>
struct Brick {
  static constexpr int BZ = ZS * ZR, NT = BX * BY * ZS;
  static constexpr int PX = BX + 2, PY = BY + 2, Plane = PX * PY, Nodes = Plane * (BZ + 2);
  static constexpr int Layer = 2 * (BX * BY + BX * BZ + BY * BZ) + 4 * (BX + BY + BZ);
  static constexpr int HM = (Layer + NT - 1) / NT;  // layer nodes per thread
  // u beside r in LDS where p, s and w are all that the registers hold
  static constexpr bool ULds = ZR == 16;
  static constexpr int Xf = 2 * BY * BZ;  // nodes of the two x faces
  static constexpr size_t Lds = (size_t)(Nodes + Xf + (ULds ? NT * ZR : 0)) * sizeof(double);
};

template <int BX, int BY, int ZS, int ZR>
__device__ __forceinline__ void resident_cg(const Resident &a, double *u_, double *W0, double *W1, double *WX,
                                            double *slots, CgState *cs, int gx, int gy, int bid, int nb) {
  using B = Brick<BX, BY, ZS, ZR>;
  constexpr int BZ = B::BZ, PX = B::PX, PY = B::PY, plane = B::Plane, HM = B::HM, nt = B::NT, XF = B::Xf;
  extern __shared__ double R[];  // r on the brick and its neighbours' layer
  double *const FX = R + B::Nodes;  // w on the two x faces
  __shared__ Meeting<nt / 64> meeting;
  const Grid g = a.g;
  const int tid = threadIdx.x;
  const int wx = bid % gx, wr = bid / gx;
  const int i0 = 1 + wx * BX, j0 = 1 + (wr % gy) * BY, k0 = 1 + (wr / gy) * BZ;
  auto interior = [&](int i, int j, int k) {
    return i >= 1 && j >= 1 && k >= 1 && i < g.nx && j < g.ny && k < g.nz;
  };
  const int lx = tid % BX, lr = tid / BX, ly = lr % BY, lz = (lr / BY) * ZR;
  const int i = i0 + lx, j = j0 + ly;
  const int o = ((lz + 1) * PY + ly + 1) * PX + lx + 1;
  const bool col = i < g.nx && j < g.ny;
  const bool side = ly == 0 || ly == BY - 1;
  bool act[ZR], face[ZR];
#pragma unroll
  for (int q = 0; q < ZR; ++q) {
    act[q] = col && k0 + lz + q < g.nz;
    face[q] = act[q] && (side || lz + q == 0 || lz + q == BZ - 1);
  }
  // byte offset of the thread's first node in an array of the grid (used where act only); the launcher refuses grids of
  // more than 2^29 elements
  const unsigned own = (unsigned)(g.at(i, j, k0 + lz) * (long long)sizeof(double));
  auto node = [&](auto *base, int q) { return at_byte(base + q * g.sz, own); };
  if (tid == 0) meeting.looks = cs->looks;
  // u of the brick and its layer (0 outside the interior)
  for (int e = tid; e < plane * (BZ + 2); e += nt) {
    const int x = e % PX, yz = e / PX, y = yz % PY, z = yz / PY;
    const int gi = i0 - 1 + x, gj = j0 - 1 + y, gk = k0 - 1 + z;
    R[e] = interior(gi, gj, gk) ? u_[g.at(gi, gj, gk)] : 0.0;
  }
  // the layer's nodes of this thread: six faces, then twelve edges (the operator reads no corner)
  // hg: where the owner publishes the node, an element of W, or of WX for those of the x faces (hx)
  int hl[HM], hg[HM];
  bool hx[HM];
  {
    const int fz = BX * BY, fy = BX * BZ, fx = BY * BZ;
#pragma unroll
    for (int m = 0; m < HM; ++m) {
      int e = tid + m * nt, x, y, z;
      bool have = true;
      int wx = -1;
      if (e < 2 * fz) {
        z = e < fz ? -1 : BZ;
        e %= fz;
        x = e % BX; y = e / BX;
      } else if ((e -= 2 * fz) < 2 * fy) {
        y = e < fy ? -1 : BY;
        e %= fy;
        x = e % BX; z = e / BX;
      } else if ((e -= 2 * fy) < 2 * fx) {
        x = e < fx ? -1 : BX;
        wx = (bid + (e < fx ? -1 : 1)) * XF + (e < fx ? fx : -fx) + e;
        e %= fx;
        y = e % BY; z = e / BY;
      } else if ((e -= 2 * fx) < 4 * BX) {
        x = e >> 2;
        y = (e & 1) ? BY : -1; z = (e & 2) ? BZ : -1;
      } else if ((e -= 4 * BX) < 4 * BY) {
        y = e >> 2;
        x = (e & 1) ? BX : -1; z = (e & 2) ? BZ : -1;
      } else {
        e -= 4 * BY;
        have = e < 4 * BZ;
        z = e >> 2;
        x = (e & 1) ? BX : -1; y = (e & 2) ? BY : -1;
      }
      have = have && interior(i0 + x, j0 + y, k0 + z);
      hl[m] = have ? ((z + 1) * PY + y + 1) * PX + x + 1 : -1;
      hx[m] = wx >= 0;
      hg[m] = !have ? 0 : (hx[m] ? wx : (int)g.at(i0 + x, j0 + y, k0 + z));
    }
  }
  const double c0 = a.st.c0, cx = a.st.cx, cy = a.st.cy, cz = a.st.cz;
  const double cxy = a.st.cxy, cxz = a.st.cxz, cyz = a.st.cyz;
  double w[ZR];
  double gam = 0.0, del = 0.0;
  // w = M of what R holds, at the thread's nodes (0 outside the grid); gam and del: the thread's parts of r.r and w.r
  auto apply = [&]() {
    double A = 0.0, S1 = 0.0, c1 = 0.0;
    gam = del = 0.0;
#pragma unroll
    for (int q = -1; q <= ZR; ++q) {
      const double *x = &R[o + q * plane];
      const double c = x[0], X = x[1] + x[-1], Y = x[PX] + x[-PX];
      const double S = cz * c + cxz * X + cyz * Y;
      if (q >= 1) {
        w[q - 1] = act[q - 1] ? A + S : 0.0;
        gam += c1 * c1;
        del += w[q - 1] * c1;
        __asm__ volatile("" : "+v"(w[q - 1]));  // formed here: not sunk to its uses, with all planes' reads kept
      }
      if (q >= 0 && q < ZR) {
        const double D = (x[PX + 1] + x[PX - 1]) + (x[1 - PX] + x[-1 - PX]);
        A = S1 + (c0 * c + cx * X + cy * Y + cxy * D);
      }
      S1 = S;
      c1 = c;
      __builtin_amdgcn_sched_barrier(0);  // one plane's reads at a time (registers)
    }
  };
  // The outer nodes of the brick for its neighbours: rows of the y and z faces in place, the x faces packed by way of
  // LDS (stored one by one they took 4 us at 128^3).
  auto publish = [&](int odd, const double (&v)[ZR]) {
    double *const W = odd ? W1 : W0;
#pragma unroll
    for (int q = 0; q < ZR; ++q) {
      if (face[q]) put(node(W, q), v[q]);
      if (lx == 0 || lx == BX - 1) FX[(lx != 0 ? XF / 2 : 0) + (lz + q) * BY + ly] = v[q];
    }
    __syncthreads();
    double *const X = WX + ((odd ? nb : 0) + bid) * XF;
    for (int e = tid; e < XF; e += nt) put(&X[e], FX[e]);
  };
  auto layer = [&](int odd, int m) {
    return get((hx[m] ? WX + (odd ? nb * XF : 0) : (odd ? W1 : W0)) + hg[m]);
  };
  // the right-hand side at the thread's nodes, by way of W0 (not unrolled: it would take the loop's registers)
  double bsum = 0.0;
#pragma unroll 1
  for (int q = 0; q < ZR; ++q) {
    if (!(col && k0 + lz + q < g.nz)) continue;
    double rf;
    const double bv = rhs_at(a.rs, g.nx, g.ny, g.nz, i, j, k0 + lz + q, rf);
    put(node(W0, q), bv);
    bsum += stop_norm_term(a.rs, bv, rf);
  }
  __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  double u[B::ULds ? 1 : ZR], p[ZR], s[ZR], hs[HM];
  double *const ul = FX + XF + tid;  // (u of node q: ul[q * nt])
  apply();
  gam = 0.0;
#pragma unroll
  for (int q = 0; q < ZR; ++q) {
    if constexpr (B::ULds) ul[q * nt] = R[o + q * plane];
    else u[q] = R[o + q * plane];
    p[q] = s[q] = 0.0;
    w[q] = act[q] ? get(node(W0, q)) - w[q] : 0.0;  // r
    gam += w[q] * w[q];
  }
  __syncthreads();  // every read of u is done
#pragma unroll
  for (int q = 0; q < ZR; ++q) R[o + q * plane] = w[q];
  publish(1, w);
  const double gbnd2 = uniform(cs->gbnd2);
  int seq = 0;
  bool here = meet(gam, bsum, slots, seq++, bid, nb, meeting);
  const double rho0 = gam, bb = bsum + gbnd2;
  const double stop2 = a.tol * a.tol * bb;
#pragma unroll
  for (int m = 0; m < HM; ++m) {
    hs[m] = 0.0;
    if (here && hl[m] >= 0) R[hl[m]] = layer(1, m);
  }
  __syncthreads();
  apply();
  publish(0, w);
  double gold = 1.0, aold = 1.0, gamma = rho0;
  int k = 0, status = 0;
  while (here) {
    here = meet(gam, del, slots, seq++, bid, nb, meeting);
    if (!here) break;
    gamma = gam;
    const double delta = del;
    if (a.hist_on && bid == 0 && tid == 0 && k < EXCMG_MAX_HISTORY)
      cs->hist[k] = bb > 0.0 ? sqrt(gamma / bb) : 0.0;
    if (!isfinite(gamma) || !isfinite(bb)) {
      status = EXCMG_ERR_BREAKDOWN;
      break;
    }
    if (gamma <= stop2) break;
    if (k >= a.cap) {
      status = EXCMG_ERR_NOCONV;
      break;
    }
    const double beta = k == 0 ? 0.0 : gamma / gold;
    const double alpha = k == 0 ? gamma / delta : gamma / (delta - beta * gamma / aold);
    if (!(alpha > 0.0) || !isfinite(alpha)) {
      status = EXCMG_ERR_BREAKDOWN;
      break;
    }
    gold = gamma;
    aold = alpha;
    double hw[HM];
#pragma unroll
    for (int m = 0; m < HM; ++m) hw[m] = hl[m] >= 0 ? layer(k & 1, m) : 0.0;
#pragma unroll
    for (int q = 0; q < ZR; ++q) {
      const double r = R[o + q * plane];
      p[q] = r + beta * p[q];
      s[q] = w[q] + beta * s[q];
      R[o + q * plane] = r - alpha * s[q];
      if constexpr (B::ULds) {
        ul[q * nt] += alpha * p[q];
      } else {
        u[q] += alpha * p[q];
        __asm__ volatile("" : "+v"(u[q]));
      }
      __asm__ volatile("" : "+v"(p[q]), "+v"(s[q]));
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int m = 0; m < HM; ++m) {
      if (hl[m] >= 0) {
        hs[m] = hw[m] + beta * hs[m];
        R[hl[m]] -= alpha * hs[m];
      }
    }
    ++k;
    __syncthreads();
    apply();
    publish(k & 1, w);
  }
  if (!here) {
    if (tid == 0) {
      __hip_atomic_store(&cs->abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (a.out) a.out->abort = 1;
    }
    return;
  }
#pragma unroll
  for (int q = 0; q < ZR; ++q)
    if (act[q]) *node(u_, q) = B::ULds ? ul[q * nt] : u[B::ULds ? 0 : q];
  if (bid == 0 && tid == 0) {
    cs->iter = k;
    cs->rho = gamma;
    cs->rho0 = rho0;
    cs->bnorm2 = bb;
    cs->stop2 = stop2;
    cs->status = status;
    cs->done = 1;
    if (a.out) set_outcome(cs, a.out, gamma, rho0, bb, k, status);
  }
}

template <int BX, int BY, int ZS, int ZR>
__global__ __launch_bounds__(BX * BY * ZS) void resident_cg_kernel(Resident a, double *u, double *W0, double *W1,
                                                                    double *WX, double *slots, CgState *cs) {
  resident_cg<BX, BY, ZS, ZR>(a, u, W0, W1, WX, slots, cs, a.plan.gx, a.plan.gy, blockIdx.x, gridDim.x);
}

// Several grids of a batch in one launch, each on a range of the workgroups.  Their meetings are apart; the launch lasts
// as long as the grid with the most iterations.  (A full launch takes 6.5 us an
// iteration in bricks of 32 x 16 x 8, 11.6 us in the largest.)
template <int BX, int BY, int ZS, int ZR>
__global__ __launch_bounds__(BX * BY * ZS) void b_resident_cg_kernel(BatchList L) {
  const int first = L.pre[0], e = find_entry(L.pre, L.n, first + blockIdx.x);
  const int start = L.pre[e], nb = L.pre[e + 1] - start;
  const BatchEntry &E = entry_at(L, e);
  Resident a;
  a.g = E.g;
  a.rs = E.rs;
  a.rs.f = as_global(E.rs.f);
  a.rs.g = as_global(E.rs.g);
  a.st = E.st;
  a.tol = E.tol;
  a.cap = E.cap;
  a.hist_on = 0;
  a.out = nullptr;
  double *const scratch = as_global(E.p1);
  const int gx = (E.g.nx - 1 + BX - 1) / BX, gy = (E.g.ny - 1 + BY - 1) / BY;
  resident_cg<BX, BY, ZS, ZR>(a, as_global(E.u), as_global(E.r), as_global(E.p0), scratch + slots_of(nb), scratch,
                              as_global(E.cs), gx, gy, first + blockIdx.x - start, nb);
}

__global__ void b_resident_init_kernel(BatchList L) {
  const BatchEntry &E = entry_at(L, blockIdx.x);
  resident_init_block({E.p1, slots_of(L.pre[blockIdx.x + 1] - L.pre[blockIdx.x]), E.looks, E.cs, nullptr, nullptr});
}

__global__ void b_mirror_kernel(BatchList L, BatchStatus *stat) {
  const BatchEntry &E = entry_at(L, blockIdx.x);
  if (threadIdx.x == 0) mirror(E, E.cs, stat, 0, true);
}

// f(Brick, its kernel, its batched kernel) for brick number b
template <typename F>
void with_brick(int b, F &&f) {
  auto go = [&](auto br, auto *kernel, auto *batched) { f(br, kernel, batched); };
  switch (b) {
    case 0: go(Brick<16, 8, 4, 2>{}, resident_cg_kernel<16, 8, 4, 2>, b_resident_cg_kernel<16, 8, 4, 2>); break;
    case 1: go(Brick<16, 16, 2, 4>{}, resident_cg_kernel<16, 16, 2, 4>, b_resident_cg_kernel<16, 16, 2, 4>); break;
    case 2: go(Brick<32, 16, 1, 8>{}, resident_cg_kernel<32, 16, 1, 8>, b_resident_cg_kernel<32, 16, 1, 8>); break;
    default: go(Brick<32, 16, 1, 16>{}, resident_cg_kernel<32, 16, 1, 16>, b_resident_cg_kernel<32, 16, 1, 16>); break;
  }
}

// the bricks of grid g; none where g's work arrays do not hold the slots and the packed x faces
template <typename B>
ResidentPlan bricks_of(const Grid &g, int b) {
  const int gx = (g.nx - 1 + B::PX - 3) / (B::PX - 2), gy = (g.ny - 1 + B::PY - 3) / (B::PY - 2);
  const int gz = (g.nz - 1 + B::BZ - 1) / B::BZ;
  const long long nb = (long long)gx * gy * gz;
  if (nb > kGroup * kGroups || slots_of((int)nb) + 2 * nb * B::Xf > g.elems) return {};
  return {b, gx, gy, gz, B::NT, B::Lds};
}

}  // namespace

// The bricks of a grid, of those that need no more than `blocks` workgroups (one per CU): the work of an iteration
// grows with the brick (1.0, 1.4, 2.1 and 4.1 us), the meeting with the workgroups (about 0.4 us with every doubling).
ResidentPlan resident_plan(const Grid &g, int blocks) {
  static const double work[kResidentBricks] = {1.0, 1.4, 2.1, 4.1};
  ResidentPlan best = {};
  double least = 1e300;
  if (g.elems >= (1ll << 29)) return best;
  for (int b = 0; b < kResidentBricks; ++b)
    with_brick(b, [&](auto br, auto, auto) {
      const ResidentPlan p = bricks_of<decltype(br)>(g, b);
      const int nb = p.gx * p.gy * p.gz;
      const double t = work[b] + 0.4 * log2((double)nb);
      if (nb == 0 || nb > blocks || t >= least) return;
      least = t;
      best = p;
    });
  return best;
}

ResidentInit resident_init(const Resident &a) {
  return {a.scratch, slots_of(a.plan.gx * a.plan.gy * a.plan.gz), a.looks, a.cs, a.out, nullptr};
}

void launch_resident_init(const ResidentInit &i, hipStream_t st) { resident_init_kernel<<<1, 256, 0, st>>>(i); }

void launch_outcome(CgState *cs, Outcome *out, hipStream_t st) { outcome_kernel<<<1, 1, 0, st>>>(cs, out); }

void launch_resident(const Resident &a, hipStream_t st) {
  const ResidentPlan &p = a.plan;
  const int nb = p.gx * p.gy * p.gz;
  with_brick(p.brick, [&](auto, auto *kernel, auto) {
    kernel<<<nb, p.threads, p.lds, st>>>(a, a.u, a.W0, a.W1, a.scratch + resident_init(a).n, a.scratch, a.cs);
  });
}

int brick_blocks(const Grid &g, int brick) {
  int n = 0;
  with_brick(brick, [&](auto br, auto, auto) {
    const ResidentPlan p = bricks_of<decltype(br)>(g, brick);
    n = p.gx * p.gy * p.gz;
  });
  return n;
}

double brick_time(int brick) {
  static const double t[kResidentBricks] = {4.5, 5.1, 6.5, 11.1};
  return t[brick];
}

void launch_b_resident_init(const BatchList &L, hipStream_t st) {
  if (L.n > 0) b_resident_init_kernel<<<L.n, 256, 0, st>>>(L);
}

void launch_b_resident(int brick, const BatchList &L, hipStream_t st) {
  with_brick(brick, [&](auto br, auto, auto *kernel) {
    using B = decltype(br);
    kernel<<<L.total, B::NT, B::Lds, st>>>(L);
  });
}

void launch_b_mirror(const BatchList &L, BatchStatus *stat, hipStream_t st) {
  if (L.n > 0) b_mirror_kernel<<<L.n, 64, 0, st>>>(L, stat);
}

}  // namespace excmg
