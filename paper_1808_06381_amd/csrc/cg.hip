// cg.hip -- the sparse solve of Eq. 9 (Method section) on gfx950:
// (A (x) I3) v = b, A = gamma0*I + alpha*L(w), three right-hand sides sharing
// one scalar matrix, Jacobi-preconditioned conjugate gradients in the
// single-reduction form of Chronopoulos & Gear (J. Comput. Appl. Math. 25,
// 1989), which in exact arithmetic produces the iterates of standard PCG:
//
//   u_k = M^-1 r_k, w_k = A u_k; gamma_k = (r_k, u_k), delta_k = (u_k, w_k)
//   beta_k = gamma_k / gamma_{k-1}
//   alpha_k = gamma_k / (delta_k - beta_k gamma_k / alpha_{k-1})
//
// The direction p_k = u_k + beta_k p_{k-1} and its product A p_k are not
// kept: A p_{k-1} = (r_{k-1} - r_k) / alpha_{k-1}, so the residual follows from
// its own last two values (the three-term form of the same iterates),
//   r_{k+1} = r_k + theta_k (r_k - r_{k-1}) - alpha_k w_k,
//   theta_k = alpha_k beta_k / alpha_{k-1},
// and x = sum_k alpha_k p_k is a combination of the u_k.  The last `ring` of
// them stay where they were written (a ring of slots), and k_cg_flush adds
// them to x (and forms the direction that later terms build on) in one pass
// every ring - 1 iterations and before a true-residual check.  Per row and
// iteration the vector work moves 96 bytes (r twice, w, the new r; with
// Jacobi 32 more for 1/diag and u) and 30 for x, against 192 and 24 with p, s
// and x kept: at N = 8e6 k_cg_vec 266 -> 131 us (learned).
//
// Per iteration three launches (four with the learned M^-1 product,
// k_cg_apply), none with a cache write-back fence:
//   k_cg_vec   the scalar recurrences and the convergence state (every block
//              alike, from k_cg_groups' sums), then the new residual (and u
//              with Jacobi), element-parallel (fully coalesced), and the
//              partial sums of (r, u) and (r, r) per sub-tile of 256 rows;
//   k_cg_spmv  w = A u, by default entry-parallel (the sub-tile's entries
//              striped over its threads, the products summed per row from
//              LDS), or with a group of 1, 2, 4 or 8 lanes per CSR row (the
//              tuning variants); partial sums of (w, u);
//   k_cg_groups the partials of at most 64 groups of sub-tiles per replica, in
//              a fixed order.
// Starts, checks, passes over the ring, IC(0) and solves under the timing probe
// use k_cg_finish (the same sums, then the recurrences) instead; small handles
// run an iteration as one launch, k_cg_fused.
// Sums are deterministic (fixed trees, no floating-point atomics).
#include "sim_dev.h"
#include "launch.h"

#include <hip/hip_ext.h>

#define VEC_ELEMS (3 * SUB_ROWS)  // elements (row, component) per sub-tile

// sum over the LANES lanes of a row's group, on registers (DPP): lanes
// exchange with lane ^ 1, then lane ^ 2 (quad permutes), then, for 8 lanes,
// with the mirrored lane of the other quad, which after the quad steps holds
// that quad's sum.  Every lane ends with the same bits, since each step adds
// the same two operands.
template <int LANES>
__device__ __forceinline__ void lane_group_sum(double (&a)[3]) {
  static_assert(LANES == 1 || LANES == 2 || LANES == 4 || LANES == 8, "lanes per row");
  if constexpr (LANES >= 2) {
#pragma unroll
    for (int k = 0; k < 3; ++k) a[k] += dpp_move<DPP_XOR1>(a[k]);
  }
  if constexpr (LANES >= 4) {
#pragma unroll
    for (int k = 0; k < 3; ++k) a[k] += dpp_move<DPP_XOR2>(a[k]);
  }
  if constexpr (LANES >= 8) {
#pragma unroll
    for (int k = 0; k < 3; ++k) a[k] += dpp_move<DPP_HALF_MIRROR>(a[k]);
  }
}

// Components per row are finished by lanes 0..2 of the row's group; with
// LANES < 3 a lane takes TURNS turns (component t * LANES + lane in turn t).
// Register arrays are only indexed with compile-time indices here.
// The entry-parallel form (LANES == 0) gives each thread one whole row: three
// turns, turn k being component k.
template <int LANES>
constexpr int TURNS = LANES == 0 ? 3 : (LANES >= 3 ? 1 : (3 + LANES - 1) / LANES);

__device__ __forceinline__ double pick3(const double (&a)[3], int k) {
  return k == 0 ? a[0] : (k == 1 ? a[1] : a[2]);
}
__device__ __forceinline__ bool on_k(const bool (&on)[3], int k) {
  return k == 0 ? on[0] : (k == 1 ? on[1] : on[2]);
}
// v[k] = the turn sum that belongs to component k (0 where this lane has none)
template <int LANES>
__device__ __forceinline__ void turns_to_components(const double (&vt)[TURNS<LANES>], int lane,
                                                    double (&v)[3]) {
  if constexpr (LANES == 0) {
    v[0] = vt[0];
    v[1] = vt[1];
    v[2] = vt[2];
    return;
  }
#pragma unroll
  for (int t = 0; t < TURNS<LANES>; ++t) {
    const int k = t * LANES + lane;
    v[0] = k == 0 ? vt[t] : v[0];
    v[1] = k == 1 ? vt[t] : v[1];
    v[2] = k == 2 ? vt[t] : v[2];
  }
}

// sub-tile partial sums: [gamma0..2, delta0..2, rr0..2]; `first`..`first+n`
// written (blocks of SUB_THREADS threads).  With d.qper an array per sum, of one
// slot per sub-tile or per wave (k_cg_fused's layout).
template <int N>
__device__ __forceinline__ void write_partials(const DevPtrs& d, int sub, int first,
                                               double (&v)[N]) {
  __shared__ double lds[SUB_THREADS / 64][9];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = wave_sum(v[k]);
  if (d.qper == 4) {
    if (lane == 0) {
#pragma unroll
      for (int k = 0; k < N; ++k)
        d.partial[(int64_t)(first + k) * d.qstride + 4 * sub + wave] = v[k];
    }
    return;
  }
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < N; ++k) lds[wave][k] = v[k];
  }
  __syncthreads();
  if (threadIdx.x < N) {
    double s = 0.0;
    for (int w = 0; w < SUB_THREADS / 64; ++w) s += lds[w][threadIdx.x];
    if (d.qper) d.partial[(int64_t)(first + threadIdx.x) * d.qstride + sub] = s;
    else d.partial[(int64_t)sub * NPART + first + threadIdx.x] = s;
  }
}

// XCD-contiguous sub-tile of this block (or -1 past the end).  With d.rev
// each XCD takes its range from the last sub-tile down: a kernel launched
// right after one that walked forward starts on the rows that one touched
// last, the most likely to be still in the Infinity Cache.  Partials go to
// their sub-tile's slot either way, so the order changes no bits.
__device__ __forceinline__ int sub_of_block(const DevPtrs& d) {
  const int nsub = SUBS_PER_TILE * d.nblk;
  const int per = (nsub + 7) >> 3;
  const int hw = blockIdx.x;
  const int sub = d.rev ? (hw & 7) * per + (per - 1 - (hw >> 3)) : xcd_block(hw, nsub);
  return sub < nsub ? sub : -1;
}

__global__ void k_cg_reset(DevPtrs d, double tol_override) {
  for (int r = threadIdx.x; r < d.nrep; r += blockDim.x) {
    CgRep& c = d.cg[r];
    for (int k = 0; k < 3; ++k) {
      c.bb[k] = c.rr[k] = c.gamma[k] = c.alpha[k] = c.theta[k] = 0.0;
      c.pend[k] = c.cbase[k] = 0;
      c.state[k] = 0;
      c.it[k] = 0;
    }
    c.tol2 = tol_override > 0.0 ? tol_override * tol_override : d.rep[r].tol2;
    c.run = 1;
    c.check = 0;
    c.restart = 0;
    c.restarts = 0;
    c.breakdown = 0;
  }
  if (threadIdx.x == 0) {
    d.ctrl->n_notdone = 3 * d.nrep;
    d.ctrl->breakdown = 0;
  }
}

// nontemporal (streaming) loads and stores, or ordinary ones
template <bool NT, class T>
__device__ __forceinline__ T ldv(const T* p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool NT, class T>
__device__ __forceinline__ void stv(T* p, T v) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// The ring's pending terms u_0 .. u_{m-1} (slots cbase ..) of a component
// into x and into the direction p that the later terms build on.  With
// p_j = u_j + beta_j p_{j-1} and x += sum_j alpha_j p_j, the beta are ratios of
// the gamma (beta_{j+1} = gamma_{j+1} / gamma_j), so
//   x += sum_j c_j u_j + beta_0 c_0 p,  c_j = (sum_{k>=j} alpha_k gamma_k) / gamma_j,
//   p  = sum_j d_j u_j + beta_0 d_0 p,  d_j = gamma_{m-1} / gamma_j
// (every term positive), the sums by a suffix scan, one wave per component;
// every u is read once.  forced = 1 (the ring is full): replicas that iterate,
// every component with pending terms; forced = 0: before a check, the
// components whose check is pending (p is not needed after it).  The
// finisher that follows marks the terms as added.
// NE elements per thread, NT threads: 3 and 256 stream a sub-tile; small
// handles, whose few blocks would each wait for the ring's slots in rounds, use
// 1 and 192 (64 rows; limit and times beside FLUSH_SPLIT_SUBS).  An element's
// terms are added in the same order.
template <int NE, int NT>
__global__ __launch_bounds__(NT) void k_cg_flush(DevPtrs d, int forced) {
  constexpr int PARTS = VEC_ELEMS / (NE * NT);  // blocks per sub-tile
  const int per = PARTS * ((SUBS_PER_TILE * d.nblk + 7) >> 3);
  const int part = (blockIdx.x & 7) * per + (blockIdx.x >> 3), sub = part / PARTS;
  if (sub >= SUBS_PER_TILE * d.nblk) return;
  const int rid = d.blk_rep[sub / SUBS_PER_TILE];
  const CgRep& cr = d.cg[rid];
  if (forced ? !cr.run : !cr.check) return;
  static_assert(U_RING <= 64 && NT >= 192 && NT % 3 == (NE > 1 ? 1 : 0), "one lane per term, one wave per component");
  __shared__ double h[U_RING][3][2];       // c, d
  __shared__ double hp[3][2];              // the factors of p
  __shared__ int cnt[3], off[3];
  const int t = threadIdx.x;
  if (t < 192) {
    const int k = t >> 6, j = t & 63;
    const int m = cr.state[k] == 1 || (forced && cr.state[k] == 0) ? cr.pend[k] : 0;
    int slot = cr.cbase[k] + j;
    slot = slot >= d.ring ? slot - d.ring : slot;
    const double* hs = d.hist + (((int64_t)rid * U_RING + slot) * 3 + k) * 3;
    const double ga = j < m ? hs[2] : 1.0;
    double s = j < m ? hs[0] * ga : 0.0;  // alpha_j gamma_j
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const double up = __shfl_down(s, o, 64);
      s += j + o < 64 ? up : 0.0;
    }
    const double last = __shfl(ga, m > 0 ? m - 1 : 0, 64);
    if (j < m) {
      h[j][k][0] = s / ga;
      h[j][k][1] = last / ga;
    }
    if (j == 0) {
      cnt[k] = m;
      off[k] = cr.cbase[k];
      hp[k][0] = m > 0 ? hs[1] * (s / ga) : 0.0;
      hp[k][1] = m > 0 ? hs[1] * (last / ga) : 0.0;
    }
  }
  __syncthreads();
  const int64_t base = (int64_t)part * (NE * NT), ring = 3 * d.rows;
  double ax[NE] = {}, ap[NE] = {};
  const int m = max(cnt[0], max(cnt[1], cnt[2]));
#pragma unroll NE == 1 ? 16 : 8
  for (int j = 0; j < m; ++j) {  // independent loads
#pragma unroll
    for (int q = 0; q < NE; ++q) {
      const int le = q * NT + t;
      const int k = le % 3;
      if (j >= cnt[k]) continue;
      int slot = off[k] + j;
      slot = slot >= d.ring ? slot - d.ring : slot;
      const double uj = __builtin_nontemporal_load(d.u + slot * ring + base + le);
      ax[q] += h[j][k][0] * uj;
      ap[q] += h[j][k][1] * uj;
    }
  }
#pragma unroll
  for (int q = 0; q < NE; ++q) {
    const int le = q * NT + t;
    const int k = le % 3;
    if (cnt[k] == 0) continue;
    const int64_t e = base + le;
    if (hp[k][1] != 0.0) {  // a direction from before the ring's first term
      const double p0 = d.p[e];
      ax[q] += hp[k][0] * p0;
      ap[q] += hp[k][1] * p0;
    }
    d.x[e] += ax[q];
    if (forced) d.p[e] = ap[q];
  }
}

// Partials (r, u) per sub-tile after an external preconditioner pass (IC(0)),
// component selection as k_cg_vec's mode.
__global__ __launch_bounds__(SUB_THREADS) void k_cg_dot_ru(DevPtrs d, int mode) {
  const int sub = sub_of_block(d);
  if (sub < 0) return;
  const CgRep& cr = d.cg[d.blk_rep[sub / SUBS_PER_TILE]];
  if ((mode == 1 && !cr.restart) || (mode == 2 && !cr.run)) return;
  bool on[3];
#pragma unroll
  for (int k = 0; k < 3; ++k)
    on[k] = mode == 0 ? true : (mode == 1 ? cr.state[k] == 3 : cr.state[k] == 0);
  double v[3] = {0, 0, 0};
  const int64_t base = (int64_t)sub * VEC_ELEMS;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int le = q * SUB_THREADS + threadIdx.x;
    const int k = le % 3;
    if (!on_k(on, k)) continue;
    const double add = d.r[base + le] * d.u[base + le];
    v[0] += k == 0 ? add : 0.0;
    v[1] += k == 1 ? add : 0.0;
    v[2] += k == 2 ? add : 0.0;
  }
  write_partials<3>(d, sub, 0, v);
}

// Entry-parallel product over a sub-tile (the (0, EPT) variants).  The
// sub-tile's off-diagonal entries are one contiguous CSR range [E0, E1); it is
// striped over the block's threads in passes of SUB_THREADS * EPT entries
// (entry E0 + c0 + t + k * SUB_THREADS to thread t), so the column and value
// loads are coalesced, all of a thread's are in flight together, and none
// waits on the row pointers of its own row; the next pass's are loaded while
// this pass's gathers are summed.  Each thread gathers its entries' rows of
// src and leaves the three products in LDS; after a barrier the thread of row
// i adds its row's products in entry order (the same order for every EPT: the
// variants give the same bits, and those of the one-lane loop form).  A row
// that spans passes continues its sum in the next one.  The sub-tile's own
// rows of src come in, and its results go out, through LDS as contiguous runs
// of 3 * SUB_ROWS doubles.  Measured at N = 8e6 (brick order, k = 5.5): the
// product 227 against 304 us for four lanes per row (learned CG iterations of
// the evolved box), the loads no longer waiting on a row-pointer load of
// their own and every lane carrying an entry.
template <int EPT, class Val, class Fin>
__device__ __forceinline__ void ep_tile(const DevPtrs& d, int sub, const double* __restrict__ src,
                                        const double* __restrict__ dg, Val val, const bool (&on)[3],
                                        double* __restrict__ out, Fin fin) {
  static_assert(SUB_THREADS == SUB_ROWS, "one thread per row of the sub-tile");
  static_assert(SUB_THREADS % 3 == 1, "component of an io element");
  constexpr int CAP = SUB_THREADS * EPT;
  __shared__ double prod[3][CAP];
  __shared__ double io[3 * SUB_ROWS];
  const int cap = (int)d.nnz_cap;  // clamped as in lane_tile
  const int t = threadIdx.x;
  const int64_t base = (int64_t)sub * SUB_ROWS;
  const int E0 = min(d.rowptr[base], cap);
  const int ne = min(d.rowptr[base + SUB_ROWS], cap) - E0;
  const int64_t i = base + t;
  const int r0 = min(d.rowptr[i], cap) - E0, r1 = min(d.rowptr[i + 1], cap) - E0;
  const double dgi = dg[i];
#pragma unroll
  for (int q = 0; q < 3; ++q) io[t + q * SUB_THREADS] = src[3 * base + t + q * SUB_THREADS];
  // values kept in their stored type until the multiply: a conversion next
  // to the load would wait for it, and with it for every gather in flight
  using VT = decltype(val(0));
  int c[EPT];
  VT m[EPT];
  auto load = [&](int c0, int (&cl)[EPT], VT (&ml)[EPT]) {
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      const int e = c0 + t + k * SUB_THREADS;
      cl[k] = -1;
      ml[k] = VT(0);
      if (e < ne) {
        cl[k] = d.col[E0 + e];
        ml[k] = val(E0 + e);
      }
    }
  };
  load(0, c, m);
  double a[3] = {0.0, 0.0, 0.0};
  for (int c0 = 0; c0 < ne; c0 += CAP) {
    double g[EPT][3];
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      g[k][0] = g[k][1] = g[k][2] = 0.0;
      if (c[k] >= 0) {
        const double* gp = src + 3 * (int64_t)c[k];
        g[k][0] = gp[0];
        g[k][1] = gp[1];
        g[k][2] = gp[2];
      }
    }
    int cn[EPT];
    VT mn[EPT];
    if (c0 + CAP < ne) {
      load(c0 + CAP, cn, mn);
    } else {
#pragma unroll
      for (int k = 0; k < EPT; ++k) {
        cn[k] = -1;
        mn[k] = VT(0);
      }
    }
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      if (c[k] >= 0) {
        const int slot = t + k * SUB_THREADS;
        const double mk = m[k];
        prod[0][slot] = mk * g[k][0];
        prod[1][slot] = mk * g[k][1];
        prod[2][slot] = mk * g[k][2];
      }
    }
    __syncthreads();
    const int lo = r0 > c0 ? r0 : c0, hi = r1 < c0 + CAP ? r1 : c0 + CAP;
    for (int e = lo; e < hi; ++e) {
      a[0] += prod[0][e - c0];
      a[1] += prod[1][e - c0];
      a[2] += prod[2][e - c0];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
      c[k] = cn[k];
      m[k] = mn[k];
    }
  }
  if (ne == 0) __syncthreads();  // the own rows in io, as after a pass
  double v[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double sk = io[3 * t + k];
    v[k] = on_k(on, k) ? fin(i, k, k, sk, dgi * sk + a[k]) : 0.0;
  }
  __syncthreads();  // every own row read
#pragma unroll
  for (int k = 0; k < 3; ++k) io[3 * t + k] = v[k];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    int k = t % 3 + q;  // component of element t + q * SUB_THREADS (SUB_THREADS = 1 mod 3)
    k = k >= 3 ? k - 3 : k;
    if (on_k(on, k)) out[3 * base + t + q * SUB_THREADS] = io[t + q * SUB_THREADS];
  }
}

// Products sum_j M_ij src_j (three components) of the sub-tile's 256 rows
// with a group of LANES lanes per row, LANES passes over 256 / LANES rows
// each.
// Lane l of a group takes the row's entries l, l + LANES, l + 2 LANES, ...,
// adds them in that order, then the group adds its lanes; both forms below
// therefore give the same bits.
//   ENT = 0: each lane walks its entries, loading column, value and the
//            gathered row in turn.
//   ENT > 0: software-pipelined over the passes.  The row pointers and the
//            diagonal terms of every pass load first; then the columns and
//            values of the first ENT entries per lane of pass p + 1 load
//            while pass p gathers, so each pass waits for one gather instead
//            of a column load followed by a gather.  Entries past LANES * ENT
//            in a row follow in the loop form.  Loads of missing entries are
//            masked, not issued.  (Loading further ahead was measured slower:
//            the extra data in flight no longer fits the L1 cache.)
// val(e) is the off-diagonal value of CSR entry e (in its stored type, FP32
// or FP64; the products are formed in FP64), dg the diagonal; for the
// components finished by this lane (component k = t * LANES + lane, turn t)
// that are on, out[3i+k] = fin(i, k, t, src_ik, own) with
// own = dg_i src_ik + sum_j M_ij src_jk.
template <int LANES, int ENT, class Val, class Fin>
__device__ __forceinline__ void lane_tile(const DevPtrs& d, int sub, const double* __restrict__ src,
                                          const double* __restrict__ dg, Val val, const bool (&on)[3],
                                          double* __restrict__ out, Fin fin) {
  constexpr int GROUPS = SUB_THREADS / LANES;
  constexpr int PASSES = SUB_ROWS / GROUPS;
  constexpr int T = TURNS<LANES>;
  const int lane = threadIdx.x & (LANES - 1);
  const int grp = threadIdx.x / LANES;
  // clamped: after an overflowing fill the row pointers may pass the
  // capacity (the host discards that solve; the reads stay in bounds)
  const int cap = (int)d.nnz_cap;
  if constexpr (ENT == 0) {
    for (int pass = 0; pass < PASSES; ++pass) {
      const int64_t i = (int64_t)sub * SUB_ROWS + pass * GROUPS + grp;
      const int e0 = min(d.rowptr[i], cap), e1 = min(d.rowptr[i + 1], cap);
      double a[3] = {0.0, 0.0, 0.0};
      for (int e = e0 + lane; e < e1; e += LANES) {
        const int64_t j = d.col[e];
        const double m = val(e);
        a[0] += m * src[3 * j];
        a[1] += m * src[3 * j + 1];
        a[2] += m * src[3 * j + 2];
      }
      lane_group_sum<LANES>(a);
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int k = t * LANES + lane;
        if (k >= 3) continue;
        if (!on_k(on, k)) continue;
        const double sk = src[3 * i + k];
        out[3 * i + k] = fin(i, k, t, sk, dg[i] * sk + pick3(a, k));
      }
    }
  } else {
    int e0[PASSES], e1[PASSES];
    double dv[PASSES], sv[PASSES][T];
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int64_t i = (int64_t)sub * SUB_ROWS + p * GROUPS + grp;
      e0[p] = min(d.rowptr[i], cap);
      e1[p] = min(d.rowptr[i + 1], cap);
      dv[p] = lane < 3 ? dg[i] : 0.0;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int k = t * LANES + lane;
        sv[p][t] = k < 3 ? src[3 * i + k] : 0.0;
      }
    }
    int c[2][ENT];      // columns of the current / next pass (-1: no entry)
    decltype(val(0)) m[2][ENT];  // values in their stored type (as in ep_tile)
    auto load_entries = [&](int p, int buf) {
#pragma unroll
      for (int q = 0; q < ENT; ++q) {
        const int e = e0[p] + lane + q * LANES;
        c[buf][q] = -1;
        m[buf][q] = 0;
        if (e < e1[p]) {
          c[buf][q] = d.col[e];
          m[buf][q] = val(e);
        }
      }
    };
    load_entries(0, 0);
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
      const int cur = p & 1;
      if (p + 1 < PASSES) load_entries(p + 1, cur ^ 1);
      double g[ENT][3];
#pragma unroll
      for (int q = 0; q < ENT; ++q) {
        g[q][0] = g[q][1] = g[q][2] = 0.0;
        const int64_t j = c[cur][q];
        if (j >= 0) {
          g[q][0] = src[3 * j];
          g[q][1] = src[3 * j + 1];
          g[q][2] = src[3 * j + 2];
        }
      }
      double a[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        a[k] = 0.0;
#pragma unroll
        for (int q = 0; q < ENT; ++q) {
          const double prod = (double)m[cur][q] * g[q][k];
          a[k] += c[cur][q] >= 0 ? prod : 0.0;  // adding +0 leaves the bits
        }
      }
      for (int e = e0[p] + lane + ENT * LANES; e < e1[p]; e += LANES) {
        const int64_t j = d.col[e];
        const double mv = val(e);
        a[0] += mv * src[3 * j];
        a[1] += mv * src[3 * j + 1];
        a[2] += mv * src[3 * j + 2];
      }
      lane_group_sum<LANES>(a);
      const int64_t i = (int64_t)sub * SUB_ROWS + p * GROUPS + grp;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int k = t * LANES + lane;
        if (k >= 3 || !on_k(on, k)) continue;
        out[3 * i + k] = fin(i, k, t, sv[p][t], dv[p] * sv[p][t] + pick3(a, k));
      }
    }
  }
}

// The product of one sub-tile in the form of variant (LANES, ENT): for every
// row i and component k with on[k], out[3i+k] = fin(i, k, t, src_ik, own)
// with own = dg_i src_ik + sum_j M_ij src_jk (fin also takes the partial sums;
// t is the turn of the calling lane)
template <int LANES, int ENT, class Val, class Fin>
__device__ __forceinline__ void csr_tile(const DevPtrs& d, int sub, const double* __restrict__ src,
                                         const double* __restrict__ dg, Val val, const bool (&on)[3],
                                         double* __restrict__ out, Fin fin) {
  if constexpr (LANES == 0)
    ep_tile<ENT>(d, sub, src, dg, val, on, out, fin);
  else
    lane_tile<LANES, ENT>(d, sub, src, dg, val, on, out, fin);
}

// Learned preconditioner: u = M^-1 r with M^-1 in A's pattern, partial
// (r, u).  Same component selection as k_cg_vec's mode.
template <int LANES, int ENT>
__global__ __launch_bounds__(SUB_THREADS) void k_cg_apply(DevPtrs d, int mode) {
  const int sub = sub_of_block(d);
  if (sub < 0) return;
  const int rid = d.blk_rep[sub / SUBS_PER_TILE];
  const CgRep& cr = d.cg[rid];
  if ((mode == 1 && !cr.restart) || (mode == 2 && !cr.run)) return;
  bool on[3];
#pragma unroll
  for (int k = 0; k < 3; ++k)
    on[k] = mode == 0 ? true : (mode == 1 ? cr.state[k] == 3 : cr.state[k] == 0);
  const float* __restrict__ moff = d.moff;
  double vt[TURNS<LANES>] = {};  // this lane's sums, one per turn
  csr_tile<LANES, ENT>(
      d, sub, d.r, d.mdiag, [&](int e) { return moff[e]; }, on, d.u,
      [&](int64_t, int, int t, double rk, double uk) {
        vt[t] += rk * uk;
        return uk;
      });
  double v[3] = {0, 0, 0};
  turns_to_components<LANES>(vt, threadIdx.x & (LANES - 1), v);
  write_partials<3>(d, sub, 0, v);
}

// Advance the recurrences of one replica from its totals
// tot = [gamma0..2, delta0..2, rr0..2] (in LDS), called by the first wave:
// lane k < 3 takes component k.  mode 0: after a fresh start, 1: after a
// restart, 2: after an iteration, 3: after a true-residual check, 4: after
// the residual of a warm-start guess.  `slot` is the ring slot of the u just
// multiplied, whose alpha, beta and gamma go to the history; `flushed`
// (mode 2): the terms before the last one were added to x in this iteration.
// c may be a copy in LDS that several blocks advance alike; one of them,
// `leader`, also writes the history and the control words.
__device__ __forceinline__ void cg_advance(const DevPtrs& d, int rid, CgRep& c, int mode,
                                           const double* tot, int slot, int flushed,
                                           bool leader) {
  const int k = threadIdx.x;
  int state = -1;
  bool finished = false, broke = false, restarted = false;
  if (k < 3) {
    const double gam = tot[k], del = tot[3 + k], rr = tot[6 + k];
    double* hs = d.hist + (((int64_t)rid * U_RING + slot) * 3 + k) * 3;
    const double bb = mode == 0 ? rr : c.bb[k], lim = c.tol2 * bb;
    state = c.state[k];
    if (mode == 0 || (mode == 1 && state == 3)) {
      if (mode == 0) c.bb[k] = rr;
      c.rr[k] = rr;
      if (bb == 0.0) {  // b = 0: x = 0 is exact
        state = 2;
        finished = true;
      } else if (rr <= lim) {
        state = 1;
      } else if (!(del > 0.0)) {
        state = 2;
        broke = finished = true;
      } else {
        state = 0;
        const double al = gam / del;
        c.gamma[k] = gam;
        c.alpha[k] = al;
        c.theta[k] = 0.0;
        c.pend[k] = 0;
        c.cbase[k] = slot;
        if (leader) {
          hs[0] = al;
          hs[1] = 0.0;
          hs[2] = gam;
        }
      }
    } else if (mode == 2) {
      int pend = c.pend[k];
      if (flushed) {
        pend = 0;
        c.cbase[k] = slot > 0 ? slot - 1 : d.ring - 1;
      }
      if (state == 0) {
        c.it[k] += 1;
        pend += 1;
        c.rr[k] = rr;
        if (rr <= lim) {
          state = 1;
        } else {
          const double beta = gam / c.gamma[k];
          const double bal = beta / c.alpha[k];
          const double den = del - bal * gam;
          if (!(den > 0.0)) {
            state = 2;
            broke = finished = true;
          } else {
            const double al = gam / den;
            c.theta[k] = al * bal;
            c.alpha[k] = al;
            c.gamma[k] = gam;
            if (leader) {
              hs[0] = al;
              hs[1] = beta;
              hs[2] = gam;
            }
          }
        }
      }
      c.pend[k] = pend;
    } else if (mode == 4 && state == 0) {
      // residual of the warm-start guess: done if it passes, else restart
      // from it (no restart is counted)
      c.rr[k] = rr;
      state = rr <= lim ? 1 : 3;
    } else if (mode == 3 && state == 1) {
      c.rr[k] = rr;
      c.pend[k] = 0;  // added before the check
      if (rr <= lim) {
        state = 2;
        finished = true;
      } else {
        state = 3;
        restarted = true;
      }
    }
    c.state[k] = state;
  }
  const uint64_t run = __ballot(state == 0), pending = __ballot(state == 1);
  const uint64_t rst = __ballot(state == 3), nf = __ballot(finished), nb = __ballot(broke);
  const uint64_t nr = __ballot(restarted);
  if (k == 0) {
    c.run = run != 0;
    c.check = run == 0 && pending != 0;
    c.restart = rst != 0;
    if (nr) c.restarts += __popcll(nr);
    if (nb) {
      c.breakdown = 1;
      if (leader) atomicOr(&d.ctrl->breakdown, 1);
    }
    if (nf && leader) atomicSub(&d.ctrl->n_notdone, (int)__popcll(nf));
  }
}

// acc of FINISH_THREADS threads summed over the block (wave trees, then the
// waves in order) into tot (LDS), valid for every thread
__device__ __forceinline__ void block_sums(double (&acc)[9], double* tot) {
  __shared__ double lds[FINISH_THREADS / 64][9];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 9; ++k) acc[k] = wave_sum(acc[k]);
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < 9; ++k) lds[wave][k] = acc[k];
  }
  __syncthreads();
  if (threadIdx.x < 9) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < FINISH_THREADS / 64; ++w) s += lds[w][threadIdx.x];
    tot[threadIdx.x] = s;
  }
  __syncthreads();
}

// This thread's share (sub-tiles t, t + FINISH_THREADS, ...) of the sums of
// `count` sub-tiles from sub-tile `first`, in the layout of k_cg_fused: QPER
// neighbouring slots per sub-tile
template <int QPER>
__device__ __forceinline__ void slot_sums(const double* __restrict__ part, int qstride, int first,
                                          int count, double (&acc)[9]) {
#pragma unroll
  for (int k = 0; k < 9; ++k) acc[k] = 0.0;
  for (int q = threadIdx.x; q < count; q += FINISH_THREADS) {
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const double* p = part + (int64_t)k * qstride + (int64_t)QPER * (first + q);
      if constexpr (QPER == 4) {
        const double4 w = *reinterpret_cast<const double4*>(p);
        acc[k] += ((w.x + w.y) + w.z) + w.w;
      } else {
        acc[k] += *p;
      }
    }
  }
}

// ... and of `count` slots of NPART doubles.  SHARED: slots that other blocks
// of this launch wrote.
template <bool SHARED = false>
__device__ __forceinline__ void slot_sums(const double* first, int count, double (&acc)[9]) {
#pragma unroll
  for (int k = 0; k < 9; ++k) acc[k] = 0.0;
  for (int t = threadIdx.x; t < count; t += FINISH_THREADS) {
    const double* src = first + (int64_t)t * NPART;
#pragma unroll
    for (int k = 0; k < 9; ++k) acc[k] += SHARED ? load_shared(src + k) : src[k];
  }
}

// CSR product over the sub-tile's 256 rows.
//   mode 0: w = A u, partial (w, u)  (components iterating / restarting / fresh)
//   mode 1: r = b - A x, partial (r, r)  (components whose check is pending)
//   mode 2: r = b - A x, partial (r, r)  (iterating components: the residual
//           of a warm-start guess)
// Lane k of a row's group finishes component k (coalesced stores); with
// fewer than three lanes, lane l takes components l, l + LANES, ...
template <bool FP32, int LANES, int ENT>
__global__ __launch_bounds__(SUB_THREADS) void k_cg_spmv(DevPtrs d, int mode, int start_mode) {
  const int sub = sub_of_block(d);
  if (sub < 0) return;
  const int rid = d.blk_rep[sub / SUBS_PER_TILE];
  const CgRep& cr = d.cg[rid];
  bool on[3];
  if (mode == 0) {
    // start_mode: 0 fresh start, 1 restart, 2 iteration (as in k_cg_vec)
    if ((start_mode == 1 && !cr.restart) || (start_mode == 2 && !cr.run)) return;
#pragma unroll
    for (int k = 0; k < 3; ++k)
      on[k] = start_mode == 0 ? true : (start_mode == 1 ? cr.state[k] == 3 : cr.state[k] == 0);
  } else if (mode == 1) {
    if (!cr.check) return;
#pragma unroll
    for (int k = 0; k < 3; ++k) on[k] = cr.state[k] == 1;
  } else {
    if (!cr.run) return;
#pragma unroll
    for (int k = 0; k < 3; ++k) on[k] = cr.state[k] == 0;
  }
  const double* __restrict__ src = mode == 0 ? d.u : d.x;
  const double* __restrict__ val = d.val;
  const float* __restrict__ valf = d.valf;
  double vt[TURNS<LANES>] = {};  // this lane's sums, one per turn
  csr_tile<LANES, ENT>(
      d, sub, src, d.diag, [&](int e) {
        if constexpr (FP32)
          return valf[e];
        else
          return val[e];
      }, on,
      mode == 0 ? d.w : d.r,
      [&](int64_t i, int k, int t, double sk, double own) {
        if (mode == 0) {
          vt[t] += own * sk;
          return own;
        }
        const double rk = d.b[3 * i + k] - own;
        vt[t] += rk * rk;
        return rk;
      });
  double v[3] = {0, 0, 0};
  turns_to_components<LANES>(vt, threadIdx.x & (LANES - 1), v);
  write_partials<3>(d, sub, mode == 0 ? 3 : 6, v);
}

// Warm start: x = the previous step's velocity of each row's particle (kept
// in original order) for the components still iterating after the fresh
// start, which has set ||b||^2 and finished the components with b = 0.
__global__ __launch_bounds__(BLOCK_THREADS) void k_cg_warm(DevPtrs d, const int64_t* __restrict__ id_off) {
  const int tile = xcd_block(blockIdx.x, d.nblk);
  if (tile >= d.nblk) return;
  const int rid = d.blk_rep[tile];
  const CgRep& cr = d.cg[rid];
  if (!cr.run) return;
  const RepDev& R = d.rep[rid];
  const int64_t i = (int64_t)tile * ROWS_PER_BLOCK + threadIdx.x;
  if (i - R.row_off >= R.n) return;  // padding rows keep x = 0
  const int64_t g = id_off[rid] + (int64_t)d.pos[i].w;
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (cr.state[k] == 0) d.x[3 * i + k] = d.vel_orig[3 * g + k];
}

__device__ __forceinline__ bool finish_work(const CgRep& c, int mode) {
  return (mode == 0) || (mode == 1 && c.restart) || (mode == 2 && c.run) ||
         (mode == 3 && c.check) || (mode == 4 && c.run);
}

// words of the per-replica state, as copied between memory and LDS
constexpr int CG_WORDS = sizeof(CgRep) / 8;
__device__ __forceinline__ void copy_state(CgRep* dst, const CgRep* src) {
  if (threadIdx.x < CG_WORDS)
    reinterpret_cast<uint64_t*>(dst)[threadIdx.x] =
        reinterpret_cast<const uint64_t*>(src)[threadIdx.x];
}

// k_cg_vec with MERGE: the same elements, operands and sums as below
template <bool NT>
__device__ __forceinline__ void vec_merged(const DevPtrs& d, int sub, const int4 info,
                                           const CgFused& f) {
  const int rid = info.x, t = threadIdx.x;
  const bool leader = sub == info.y;
  __shared__ CgRep c;
  __shared__ double tot[9];
  if (!f.cg_in[rid].run) {
    if (leader) copy_state(f.cg_out + rid, f.cg_in + rid);
    return;
  }
  const bool ext = d.learned;
  double r0[3], rm[3], w[3], di[3];
  const int64_t base = (int64_t)sub * VEC_ELEMS;
  const int le0 = 192 * (t >> 6) + (t & 63);
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int64_t e = base + le0 + 64 * q;
    r0[q] = ldv<NT>(d.r + e);
    rm[q] = ldv<NT>(d.s + e);
    w[q] = ldv<NT>(d.w + e);
    di[q] = (ext || d.pc_none) ? 1.0 : ldv<NT>(d.dinv + (int64_t)sub * SUB_ROWS + (le0 + 64 * q) / 3);
  }
  copy_state(&c, f.cg_in + rid);
  if (f.first) {
    __syncthreads();
  } else {
    double acc[9];
    slot_sums(d.partial2 + (int64_t)info.w * NPART, info.z, acc);
    block_sums(acc, tot);
    if (t < 64) cg_advance(d, rid, c, 2, tot, f.slot, f.flushed, leader);
    __syncthreads();
  }
  if (leader) copy_state(f.cg_out + rid, &c);
  if (!c.run) return;
  double g[3] = {0, 0, 0}, rr[3] = {0, 0, 0};
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int le = le0 + 64 * q, k = le % 3;
    if (c.state[k] != 0) continue;
    const double th = c.theta[k], old = th != 0.0 ? rm[q] : r0[q];
    const double rk = (r0[q] + th * (r0[q] - old)) - c.alpha[k] * w[q];
    stv<NT>(d.s + base + le, rk);
    if (!ext) {
      const double uk = di[q] * rk;
      d.u[base + le] = uk;
#pragma unroll
      for (int j = 0; j < 3; ++j) g[j] += j == k ? rk * uk : 0.0;
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) rr[j] += j == k ? rk * rk : 0.0;
  }
  if (!ext) {
    write_partials<3>(d, sub, 0, g);
    __syncthreads();
  }
  write_partials<3>(d, sub, 6, rr);
}

// Element-parallel vector work of one sub-tile (3 * 256 consecutive doubles
// of the AoS arrays; element e is row e/3, component e%3).  NT: the streams
// that are not read again within the iteration (r twice, w, 1/diag) are
// loaded and stored as nontemporal, u (gathered by the product next) as
// usual: on a working set larger than the last-level cache this streams
// faster (measured at N = 8e6), below it the ordinary form keeps the
// vectors cached; the autotuner picks.  Same bits either way.
//   mode 0 (fresh start):   x = 0, r = b, u = M^-1 r
//   mode 1 (restart, r already = b - A x):   u = M^-1 r
//   mode 2 (iteration):     d.s = r + theta (r - d.s) - alpha w, u = M^-1 (new r)
// In mode 2 the new residual overwrites the one before r; the host swaps the
// two for the launches that follow, and points d.u at the next ring slot.
// With theta = 0 (a first iteration) the old d.s is not read.
// Partials (r, u) and (r, r) of the components touched.
// MERGE (mode 2): the scalars are advanced here, from the sums of at most
// L1_MAX_GROUPS groups of sub-tiles (k_cg_groups), by every block alike; the
// replica's first block stores them (f.cg_out).  The block's own elements load
// meanwhile, so the pass takes as long as without; the launch before it is 2 us
// shorter than the finisher: a solve at N = 2.5e5 2.21 -> 2.03 ms, the step at
// N = 1e6 (Jacobi) 4.81 -> 4.57.  (The groups' sums by the product's last blocks
// instead of a launch: every block waited for its stores, product 10.5 -> 20.6
// us at N = 2.5e5, 27 -> 35 at 1e6.)
template <bool NT, bool MERGE>
__global__ __launch_bounds__(SUB_THREADS) void k_cg_vec(DevPtrs d, int mode, CgFused f) {
  const int sub = sub_of_block(d);
  if (sub < 0) return;
  if constexpr (MERGE) {
    const int4 info = d.blk_info[sub / SUBS_PER_TILE];
    vec_merged<NT>(d, sub, info, f);
    return;
  }
  const int rid = d.blk_rep[sub / SUBS_PER_TILE];
  const CgRep& cr = d.cg[rid];
  if ((mode == 1 && !cr.restart) || (mode == 2 && !cr.run)) return;
  bool on[3];
  double al[3], th[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    on[k] = mode == 0 ? true : (mode == 1 ? cr.state[k] == 3 : cr.state[k] == 0);
    al[k] = cr.alpha[k];
    th[k] = cr.theta[k];
  }
  double v[6] = {0, 0, 0, 0, 0, 0};  // (r,u)[3], (r,r)[3]
  const int64_t base = (int64_t)sub * VEC_ELEMS;
  const bool ext = d.learned || d.ic0;  // u = M^-1 r comes from a separate pass
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    // a wave takes the elements of its 64 rows (as in k_cg_fused)
    const int le = 192 * (threadIdx.x >> 6) + 64 * q + (threadIdx.x & 63);
    const int k = le % 3;
    if (!on_k(on, k)) continue;
    const int64_t e = base + le;
    // 1/diag only where this kernel applies Jacobi itself
    const double di =
        (ext || d.pc_none) ? 1.0 : ldv<NT>(d.dinv + (int64_t)sub * SUB_ROWS + le / 3);
    double rk;
    if (mode == 0) {
      rk = d.b[e];
      d.x[e] = 0.0;
      d.r[e] = rk;
    } else if (mode == 1) {
      rk = d.r[e];
    } else {
      const double r0 = ldv<NT>(d.r + e), t = pick3(th, k);
      const double rm = t != 0.0 ? ldv<NT>(d.s + e) : r0;
      rk = (r0 + t * (r0 - rm)) - pick3(al, k) * ldv<NT>(d.w + e);
      stv<NT>(d.s + e, rk);
    }
    if (!ext) {
      const double uk = di * rk;
      d.u[e] = uk;
      v[k] += rk * uk;
    }
    v[3 + k] += rk * rk;
  }
  double g[3] = {v[0], v[1], v[2]}, rr[3] = {v[3], v[4], v[5]};
  if (!ext) {
    write_partials<3>(d, sub, 0, g);
    __syncthreads();
  }
  write_partials<3>(d, sub, 6, rr);
}

// Sub-tile partials in a fixed order, then the recurrences.  A replica of few
// sub-tiles is one block's work.  Of a larger one, block b sums L1_SUBS
// sub-tiles into partial2[b], and the last block to finish (last_block) adds
// those sums in order and advances: one launch where two were (9.3 us at
// N = 1e6, now 5.6 traced, early returns included).  `from`: the state to advance into
// d.cg (d.cg itself, or the other copy after an odd number of fused or merged
// iterations; the block that advances moves it).
__global__ __launch_bounds__(FINISH_THREADS) void k_cg_finish(DevPtrs d, int mode, int slot,
                                                              int flushed, const CgRep* from) {
  const FinBlock F = d.fin[blockIdx.x];
  const int rid = F.rep;
  CgRep& c = d.cg[rid];
  __shared__ double tot[9];
  // summed before the state says whether they are needed: the two loads are
  // the launch's longest waits, and neither waits for the other
  const bool work = finish_work(from[rid], mode), moved = from != d.cg;
  double acc[9];
  if (d.qper == 4) slot_sums<4>(d.partial, d.qstride, F.sub0, F.nsub, acc);
  else if (d.qper) slot_sums<1>(d.partial, d.qstride, F.sub0, F.nsub, acc);
  else slot_sums(d.partial + (int64_t)F.sub0 * NPART, F.nsub, acc);
  block_sums(acc, tot);
  if (!work) {
    if (moved && (int)blockIdx.x == F.off) copy_state(&c, from + rid);
    return;
  }
  if (F.cnt > 1) {
    double* out = d.partial2 + (int64_t)blockIdx.x * NPART;
    if (threadIdx.x < 9) store_shared(out + threadIdx.x, tot[threadIdx.x]);
    if (!last_block(d.fin_ticket + rid, F.cnt)) return;
    slot_sums<true>(d.partial2 + (int64_t)F.off * NPART, F.cnt, acc);
    block_sums(acc, tot);
  }
  if (moved) {
    copy_state(&c, from + rid);
    __syncthreads();
  }
  if (threadIdx.x < 64) cg_advance(d, rid, c, mode, tot, slot, flushed, true);
}

// The first level alone, for a vector pass that advances the scalars itself
// (merged iterations): every finishing block's sums into partial2.
__global__ __launch_bounds__(FINISH_THREADS) void k_cg_groups(DevPtrs d) {
  const FinBlock F = d.fin[blockIdx.x];
  double* out = d.partial2 + (int64_t)blockIdx.x * NPART;
  double acc[9];
  if (F.nsub <= 64) {  // one wave's work (the others would add zeros)
    if (threadIdx.x >= 64) return;
    slot_sums(d.partial + (int64_t)F.sub0 * NPART, F.nsub, acc);
#pragma unroll
    for (int k = 0; k < 9; ++k) acc[k] = wave_sum(acc[k]);
    if (threadIdx.x == 0) {
#pragma unroll
      for (int k = 0; k < 9; ++k) out[k] = acc[k];
    }
    return;
  }
  __shared__ double tot[9];
  slot_sums(d.partial + (int64_t)F.sub0 * NPART, F.nsub, acc);
  block_sums(acc, tot);
  if (threadIdx.x < 9) out[threadIdx.x] = tot[threadIdx.x];
}

// ---------------------------------------------------------------------------
// One launch for finisher, vector pass and the product that follows, for
// handles whose iterations are a few microseconds of work each, where every
// launch costs about as much again.  Each block forms the replica's new
// scalars itself from the last launch's sub-tile partials (the same sums in
// the same order in every block; the replica's first block stores them), and
// takes the new residual of a gathered row j from the three vectors that
// define it, r_j, s_j and w_j, instead of waiting for a pass that stores it:
//   Jacobi:   u_j = (1/diag_j) r'_j, w' = A u        one launch per iteration
//   learned:  u = M^-1 r'                            then k_cg_spmv: w = A u
// What is read here by other blocks is not written here: the new residual
// goes to a third buffer, w', the partials and the scalars to second ones.
// Every sum has the operands and the order of the separate kernels (product
// in entry order), so both forms give the same bits.  Three gathers per entry
// in place of one: for large handles the separate passes are faster.
// Bound by launch and memory latency: the longest chain of loads is row pointer
// -> column -> gathered rows, and everything else that the scalars need (the
// partials, the state, the block's table entry) loads beside it.  A block has
// 64 * W rows and T threads: all threads take entries, W waves the elements
// (r', u and their sums), the next ones add up the rows' products.  Small
// handles use W = 1, which spreads their entries over four times as many units
// (N = 1000, ten steps: 7.4 -> 5.5 ms); every block of it writes one slot per
// sum and reads four per sub-tile of its replica, in the order in which a
// 256-row block adds its waves, so both forms give the same bits.
// A 256-row block (W = 4) takes two entries per thread and pass: a pass is a
// barrier, a chain of a row's additions and another barrier, and with one entry
// per thread the paper's box (15 entries per row) had 7.5 of them in 23 us; the
// additions' operands are read four at a time.  4 x 20060 rows, ten steps: 16.8
// -> 15.4 -> 14.8 ms, N = 1e5 learned 1.91 -> 1.80 (three entries per thread: 19.4
// and 1.88, three waves per SIMD; eight operands: 15.7).
// The times and the limits are beside FUSED_ROWS.
// ---------------------------------------------------------------------------
template <int T, int W, bool LEARNED, bool FP32>
__global__ __launch_bounds__(T) void k_cg_fused(DevPtrs d, CgFused f) {
  constexpr int ROWS = 64 * W, QPER = 4 / W;
  constexpr int RC = T >= 256 * W ? 1 : 3;      // components per row thread
  constexpr int EPT = W == 4 ? 2 : 1, CAP = EPT * T;  // entries per thread and pass
  constexpr int RWAVES = W * (3 / RC);          // waves W .. W + RWAVES - 1
  static_assert(T >= FINISH_THREADS && T >= 64 * (W + RWAVES) && CG_WORDS <= 64, "roles of waves");
  const int per = QPER * ((SUBS_PER_TILE * d.nblk + 7) >> 3);  // blocks per XCD, whole sub-tiles
  const int qb = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (qb >= QPER * SUBS_PER_TILE * d.nblk) return;
  __shared__ CgRep c;
  __shared__ double prod[3][CAP];
  __shared__ double io[3 * ROWS];     // the source's own rows
  __shared__ double res[3 * ROWS];    // the results
  __shared__ double lds[FINISH_THREADS / 64][9];
  __shared__ double tot[9];
  __shared__ double own[W][9];        // this block's sums
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t base = (int64_t)qb * ROWS;
  // everything that does not depend on the scalars is loaded first: the
  // entries with the rows they gather, the last launch's partials, the state
  const int4 info = d.blk_info[qb / (QPER * SUBS_PER_TILE)];
  const int rid = info.x;
  const int cap = (int)d.nnz_cap;     // clamped as in lane_tile
  const int E0 = min(d.rowptr[base], cap);
  const int ne = min(d.rowptr[base + ROWS], cap) - E0;
  // waves 0 .. W - 1: the elements of 64 rows each; the next RWAVES: the sums
  // of 64 rows' products, of one component or of all three
  const bool elems = wave < W, sums = wave >= W && wave < W + RWAVES;
  const int comp = RC == 1 ? (wave - W) / W : 0;
  const int group = elems ? wave : (wave - W) % W, row = 64 * group + lane;
  int r0 = 0, r1 = 0;
  double dgi = 0.0, er[3], es[3], ew[3], ed[3];
  if (elems) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int le = 192 * wave + 64 * q + lane;
      er[q] = d.r[3 * base + le];
      es[q] = d.s[3 * base + le];
      ew[q] = d.w[3 * base + le];
      ed[q] = LEARNED || d.pc_none ? 1.0 : d.dinv[base + le / 3];
    }
  } else if (sums) {
    r0 = min(d.rowptr[base + row], cap) - E0;
    r1 = min(d.rowptr[base + row + 1], cap) - E0;
    dgi = LEARNED ? d.mdiag[base + row] : d.diag[base + row];
  }
  auto value = [&](int e) {
    if constexpr (LEARNED) return d.moff[e];
    else if constexpr (FP32) return d.valf[e];
    else return d.val[e];
  };
  using VT = decltype(value(0));
  VT m[EPT];
  double gr[EPT][3], gs[EPT][3], gw[EPT][3], gd[EPT];
  auto load = [&](int c0) {   // entries of the pass at c0 and the rows they gather
    int j[EPT];
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
      const int e = c0 + q * T + t;
      j[q] = -1;
      if (e < ne) {
        j[q] = d.col[E0 + e];
        m[q] = value(E0 + e);
      }
    }
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
      if (j[q] < 0) continue;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        gr[q][k] = d.r[3 * (int64_t)j[q] + k];
        gs[q][k] = d.s[3 * (int64_t)j[q] + k];
        gw[q][k] = d.w[3 * (int64_t)j[q] + k];
      }
      gd[q] = LEARNED || d.pc_none ? 1.0 : d.dinv[j[q]];
    }
  };
  if (t < CG_WORDS)
    reinterpret_cast<uint64_t*>(&c)[t] = reinterpret_cast<const uint64_t*>(f.cg_in + rid)[t];
  load(0);
  double acc[9];
  if (!f.first && t < FINISH_THREADS) {
    slot_sums<QPER>(f.part_in, d.qstride, info.y, info.z, acc);
#pragma unroll
    for (int k = 0; k < 9; ++k) acc[k] = wave_sum(acc[k]);
    if (lane == 0) {
#pragma unroll
      for (int k = 0; k < 9; ++k) lds[wave][k] = acc[k];
    }
  }
  __syncthreads();
  const bool leader = qb == QPER * info.y;
  // the state is advanced unless the last launch left it advanced
  if (!f.first && c.run) {
    if (t < 9) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < FINISH_THREADS / 64; ++w) s += lds[w][t];
      tot[t] = s;
    }
    __syncthreads();
    if (t < 64) cg_advance(d, rid, c, 2, tot, f.slot, f.flushed, leader);
    __syncthreads();
  }
  if (leader) copy_state(f.cg_out + rid, &c);
  if (!c.run) return;
  bool on[3];
  double al[3], th[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    on[k] = c.state[k] == 0;
    al[k] = c.alpha[k];
    th[k] = c.theta[k];
  }
  // r' as k_cg_vec forms it
  auto next = [](double r, double s, double w, double a, double tk) {
    const double rm = tk != 0.0 ? s : r;
    return (r + tk * (r - rm)) - a * w;
  };
  double v[6] = {0, 0, 0, 0, 0, 0};  // (r,u), (r,r) of the elements
  if (elems) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int le = 192 * wave + 64 * q + lane, k = le % 3;
      double src = 0.0;
      if (on_k(on, k)) {
        const double rk = next(er[q], es[q], ew[q], pick3(al, k), pick3(th, k));
        f.rnew[3 * base + le] = rk;
        src = rk;
        if constexpr (!LEARNED) {
          src = ed[q] * rk;
          d.u[3 * base + le] = src;
          v[k] += rk * src;
        }
        v[3 + k] += rk * rk;
      }
      io[le] = src;
    }
  }
  double a[RC] = {};
  for (int c0 = 0; c0 < ne; c0 += CAP) {
#pragma unroll
    for (int q = 0; q < EPT; ++q) {
      if (c0 + q * T + t >= ne) continue;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        double src = next(gr[q][k], gs[q][k], gw[q][k], al[k], th[k]);
        if constexpr (!LEARNED) src = gd[q] * src;
        prod[k][q * T + t] = (double)m[q] * src;
      }
    }
    if (c0 + CAP < ne) load(c0 + CAP);
    __syncthreads();
    if (sums) {
      const int lo = r0 > c0 ? r0 : c0, hi = r1 < c0 + CAP ? r1 : c0 + CAP;
#pragma unroll 4
      for (int e = lo; e < hi; ++e) {
#pragma unroll
        for (int k = 0; k < RC; ++k) a[k] += prod[comp + k][e - c0];
      }
    }
    if (c0 + CAP < ne) __syncthreads();
  }
  if (ne == 0) __syncthreads();
  if (elems) {
#pragma unroll
    for (int k = LEARNED ? 3 : 0; k < 6; ++k) {
      const double s = wave_sum(v[k]);
      if (lane == 0) own[wave][k < 3 ? k : k + 3] = s;
    }
  } else if (sums) {
#pragma unroll
    for (int k = 0; k < RC; ++k) {
      const double sk = io[3 * row + comp + k];
      const double out = dgi * sk + a[k];
      res[3 * row + comp + k] = out;
      // learned: (r, u), u the result (k_cg_spmv adds (w, u)); Jacobi: (w, u)
      const double s = wave_sum(on_k(on, comp + k) ? out * sk : 0.0);
      if (lane == 0) own[group][(LEARNED ? 0 : 3) + comp + k] = s;
    }
  }
  __syncthreads();
  if (t < 3 * ROWS) {
    double* __restrict__ dst = LEARNED ? d.u : f.wnew;
    for (int le = t; le < 3 * ROWS; le += T)
      if (on_k(on, le % 3)) dst[3 * base + le] = res[le];
  }
  if (t < 9 && !(LEARNED && t / 3 == 1)) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) s += own[w][t];
    d.partial[(int64_t)t * d.qstride + qb] = s;
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// With events, the extended launch records the kernel's own start and end;
// without, a plain launch (the form that stream capture records).
#define LAUNCH_EV(K, G, B, S, E0, E1, ...)                              \
  do {                                                                  \
    if ((E0) || (E1))                                                   \
      hipExtLaunchKernelGGL(K, G, B, 0, S, E0, E1, 0, __VA_ARGS__);     \
    else                                                                \
      hipLaunchKernelGGL(K, G, B, 0, S, __VA_ARGS__);                   \
  } while (0)

hipError_t launch_cg_reset(const DevPtrs& d, double tol_override, hipStream_t s) {
  hipLaunchKernelGGL(k_cg_reset, dim3(1), dim3(256), 0, s, d, tol_override);
  return hipGetLastError();
}

// ev0/ev1 (optional) take the kernel's own start and end timestamps
hipError_t launch_cg_vec(const DevPtrs& d, int mode, hipStream_t s, hipEvent_t ev0,
                         hipEvent_t ev1) {
  const dim3 g(xcd_grid(SUBS_PER_TILE * d.nblk)), b(SUB_THREADS);
  if (d.vec_nt && mode == 2)
    LAUNCH_EV((k_cg_vec<true, false>), g, b, s, ev0, ev1, d, mode, CgFused{});
  else
    LAUNCH_EV((k_cg_vec<false, false>), g, b, s, ev0, ev1, d, mode, CgFused{});
  return hipGetLastError();
}

hipError_t launch_cg_groups(const DevPtrs& d, hipStream_t s) {
  hipLaunchKernelGGL(k_cg_groups, dim3(d.fin_total), dim3(FINISH_THREADS), 0, s, d);
  return hipGetLastError();
}

hipError_t launch_cg_vec_merged(const DevPtrs& d, const CgFused& f, hipStream_t s) {
  const dim3 g(xcd_grid(SUBS_PER_TILE * d.nblk)), b(SUB_THREADS);
  if (d.vec_nt)
    hipLaunchKernelGGL((k_cg_vec<true, true>), g, b, 0, s, d, 2, f);
  else
    hipLaunchKernelGGL((k_cg_vec<false, true>), g, b, 0, s, d, 2, f);
  return hipGetLastError();
}

hipError_t launch_cg_spmv(const DevPtrs& d, int mode, int start_mode, hipStream_t s,
                          hipEvent_t ev0, hipEvent_t ev1) {
  const dim3 g(xcd_grid(SUBS_PER_TILE * d.nblk)), b(SUB_THREADS);
  const bool f32 = d.spmv_fp32 && mode == 0;
  switch (d.spmv_var * 2 + (f32 ? 1 : 0)) {
#define SPMV_CASE(V, L, E)                                                                  \
    case 2 * V:                                                                            \
      LAUNCH_EV((k_cg_spmv<false, L, E>), g, b, s, ev0, ev1, d, mode, start_mode);          \
      break;                                                                               \
    case 2 * V + 1:                                                                        \
      LAUNCH_EV((k_cg_spmv<true, L, E>), g, b, s, ev0, ev1, d, mode, start_mode);           \
      break;
    CSR_VARIANT_LIST(SPMV_CASE)
#undef SPMV_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_cg_dot_ru(const DevPtrs& d, int mode, hipStream_t s) {
  hipLaunchKernelGGL(k_cg_dot_ru, dim3(xcd_grid(SUBS_PER_TILE * d.nblk)), dim3(SUB_THREADS), 0, s,
                     d, mode);
  return hipGetLastError();
}

hipError_t launch_cg_apply(const DevPtrs& d, int mode, hipStream_t s, hipEvent_t ev0,
                           hipEvent_t ev1) {
  const dim3 g(xcd_grid(SUBS_PER_TILE * d.nblk)), b(SUB_THREADS);
  switch (d.apply_var) {
#define APPLY_CASE(V, L, E) \
    case V: LAUNCH_EV((k_cg_apply<L, E>), g, b, s, ev0, ev1, d, mode); break;
    CSR_VARIANT_LIST(APPLY_CASE)
#undef APPLY_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_cg_warm(const DevPtrs& d, const int64_t* id_off, hipStream_t s) {
  hipLaunchKernelGGL(k_cg_warm, dim3(xcd_grid(d.nblk)), dim3(BLOCK_THREADS), 0, s, d, id_off);
  return hipGetLastError();
}

// d.u: the first ring slot
hipError_t launch_cg_flush(const DevPtrs& d, int forced, hipStream_t s) {
  const int g = xcd_grid(SUBS_PER_TILE * d.nblk);
  if (SUBS_PER_TILE * d.nblk <= FLUSH_SPLIT_SUBS)
    hipLaunchKernelGGL((k_cg_flush<1, 192>), dim3(4 * g), dim3(192), 0, s, d, forced);
  else
    hipLaunchKernelGGL((k_cg_flush<3, 256>), dim3(g), dim3(256), 0, s, d, forced);
  return hipGetLastError();
}

template <int T, int W>
static void launch_fused_t(const DevPtrs& d, const CgFused& f, hipStream_t s) {
  const dim3 g(4 / W * xcd_grid(SUBS_PER_TILE * d.nblk)), b(T);
  if (d.learned)
    hipLaunchKernelGGL((k_cg_fused<T, W, true, false>), g, b, 0, s, d, f);
  else if (d.spmv_fp32)
    hipLaunchKernelGGL((k_cg_fused<T, W, false, true>), g, b, 0, s, d, f);
  else
    hipLaunchKernelGGL((k_cg_fused<T, W, false, false>), g, b, 0, s, d, f);
}

hipError_t launch_cg_fused(const DevPtrs& d, const CgFused& f, hipStream_t s) {
  if (d.qper == 4) launch_fused_t<512, 1>(d, f, s);
  else launch_fused_t<512, 4>(d, f, s);
  return hipGetLastError();
}

hipError_t launch_cg_finish(const DevPtrs& d, int mode, int slot, int flushed, hipStream_t s,
                            const CgRep* from) {
  hipLaunchKernelGGL(k_cg_finish, dim3(d.fin_total), dim3(FINISH_THREADS), 0, s, d, mode, slot, flushed,
                     from ? from : d.cg);
  return hipGetLastError();
}
