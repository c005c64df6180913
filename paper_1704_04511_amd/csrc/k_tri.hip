// Householder reduction of the Hermitian Gram matrix to real symmetric
// tridiagonal form, R = Q T Q^H (FP64), first stage of the eigen-decomposition
// in the weight update (Sec. III.B, Algorithm 1 step 1).
//
// Column k needs a global matrix-vector product with the trailing block, and so
// a grid-wide exchange.  Sizes whose matrix fits the registers of 256 workgroups
// (129 to 1280) are reduced in one launch (k_tri_res, below); other sizes, calls
// on a stream that is being captured or kept to some of the CUs, and runs repeated
// after a resident launch gave up use one launch per column, the launch boundary
// being the exchange.  A launch for column k:
//   * in every workgroup (redundantly, identical arithmetic): finishes the
//     previous reflector's w = tau p - |tau|^2/2 (p^H v) v from the previous
//     launch's p = A v, corrects row k with the pending rank-2 update
//     A <- A - v w^H - w v^H, and forms reflector k, H = I - tau v v^H with
//     H^H x = (beta, 0, ..)^T, beta real (the elementary reflector convention
//     of LAPACK's zlarfg);
//   * on its rows i > k: applies the pending rank-2 update and accumulates
//     p_i = sum_j A_ij v_j for the next launch.
// Where the trailing block is small the time of a launch is the serial chain of
// the reflector, not the traffic of the block, so the chain is kept short: thread t holds the
// entries j = k + t + 256 u of every vector in registers (the same entries of
// every row it updates), and a launch makes exactly three block reductions
// (p^H v, the norm of the column, the row products), each a fixed DPP tree in
// every wave plus the four wave sums added in order, with the scalars other
// threads need (p_k, v_k, the subdiagonal entry, the rows' own coefficients)
// passed through the same exchange.  Results are bit-reproducible and do not
// depend on how many workgroups run or which rows a workgroup takes.
// The last 96 columns, whose trailing block fits in the registers of one
// workgroup, are reduced in a single launch (k_tri_tail).
// The working matrix Aw is full (both triangles) and row-major; reflectors are
// stored as LAPACK's zhetrd (lower) stores them: v(k+2:n) in column k of the
// column-major matrix Vst below the subdiagonal, tau(k), diagonal D, real
// subdiagonal E.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <mutex>
#include <thread>
#include <type_traits>
#include <vector>

#include "common.h"
#include "kernels.h"
#include "../../include/slrx.h"

namespace slrx {

constexpr int kTriNT = 256;
constexpr int kTriRB = 4;      // rows of a workgroup whose elements are loaded at kernel entry
// Rows held in registers at a time for U vector entries per thread: fewer for the
// long columns of Gram matrices above 2048 (their register arrays otherwise need
// about 500 registers per lane, and the U = 12 instance holding four rows gave wrong
// eigenvalues for n > 2560 while U = 9 and 10 were exact).
template <int U> constexpr int tri_rb() { return U > 10 ? 1 : (U > 8 ? 2 : kTriRB); }
constexpr int kTriRMax = 32;   // rows per workgroup at most

SLRX_DEV double2 dsub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
// Trailing-block rows are read and written once per column launch.  STREAM
// marks those accesses nontemporal (the nt cache-policy bit of the load and
// store instructions); the values are the same either way.
typedef double d2v __attribute__((ext_vector_type(2)));
template <bool STREAM> SLRX_DEV double2 row_load(const double2* p) {
  if constexpr (STREAM) {
    const d2v v = __builtin_nontemporal_load((const d2v*)p);
    return make_double2(v.x, v.y);
  } else {
    return *p;
  }
}
template <bool STREAM> SLRX_DEV void row_store(double2* p, double2 e) {
  if constexpr (STREAM) {
    const d2v v = {e.x, e.y};
    __builtin_nontemporal_store(v, (d2v*)p);
  } else {
    *p = e;
  }
}
SLRX_DEV double2 dscale(double2 a, double s) { return make_double2(a.x * s, a.y * s); }

// Copy of v from the lane selected by a DPP control (rows masked by RM keep 0).
template <int CTRL, int RM>
SLRX_DEV double dpp_mov(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, RM, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, RM, 0xf, false);
  return __hiloint2double(hi, lo);
}
// The same for a control that gives every lane a source (no previous value to keep).
template <int CTRL>
SLRX_DEV double dpp_all(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// The two values of lanes 16 apart within a half-wave, added: the even row of 16
// lanes gets the sums of x over both rows, the odd row those of y
// (v_permlane16_swap exchanges the odd row of its first operand with the even row
// of the second).
SLRX_DEV double pair_rows(double x, double y) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(x), __double2loint(y), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(x), __double2hiint(y), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
// The same for lanes 32 apart: lanes 0-31 get the sums of x over both halves of the wave,
// lanes 32-63 those of y.
SLRX_DEV double pair_halves(double x, double y) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(x), __double2loint(y), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(x), __double2hiint(y), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
// Sum over each row of 16 lanes (a fixed tree); every lane of the row gets it.
SLRX_DEV double row_total(double v) {
  v += dpp_all<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_all<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_all<0x141>(v);  // row_half_mirror
  v += dpp_all<0x140>(v);  // row_mirror
  return v;
}
// Sum over the 64 lanes of a wave in a fixed tree; every lane gets the total.
// Call with all 64 lanes active.
SLRX_DEV double wave_total(double v) {
  v = pair_halves(v, v);
  return row_total(pair_rows(v, v));
}
SLRX_DEV double2 wave_total2(double2 v) { return make_double2(wave_total(v.x), wave_total(v.y)); }
// The four wave sums of an exchange slot, added in wave order.
SLRX_DEV double2 sum4(const double2* s, int stride) {
  double2 r = s[0];
  r = dadd(r, s[stride]);
  r = dadd(r, s[2 * stride]);
  return dadd(r, s[3 * stride]);
}

// One column of the reduction.  U: vector entries per thread (n - k <= 256 U);
// rows: rows of the trailing block per workgroup (blockIdx.x * rows + k + 1 ..);
// STREAM: nontemporal row accesses.
template <int U, bool STREAM>
__global__ __launch_bounds__(kTriNT) void k_tri_col(TriArgs a, int rows) {
  // exchange slots: [wave][item] for the three reductions
  __shared__ double2 xa[4][3];
  __shared__ double2 xb[4][3];
  __shared__ double2 xc[4][kTriRMax];
  __shared__ double2 coef[kTriRMax][2];  // v_{k-1}(i), w_{k-1}(i) of the workgroup's rows
  const int n = a.n, k = a.k;
  const int b = blockIdx.y;  // problem in a batch
  double2* Aw = a.Aw + (size_t)b * a.strideA;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool pending = k > 0;
  const double2 zero = make_double2(0.0, 0.0);
  const int row0 = k + 1 + blockIdx.x * rows;
  const int nrow = min(rows, n - row0);  // >= 1 by the grid size

  // 0. every independent load first: row k, v_{k-1}, p_{k-1}, the first rows of the block
  const double2 t = pending ? a.tau[(size_t)b * n + (k - 1)] : zero;
  const double2* rowk = Aw + (size_t)k * n;
  const double2* vprev = a.vbuf[(k + 1) & 1] + (size_t)b * n;  // written by launch k-1
  const double2* pprev = a.pbuf[(k + 1) & 1] + (size_t)b * n;
  double2 rk[U], vp[U], pp[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int j = k + tid + kTriNT * u;
    rk[u] = vp[u] = pp[u] = zero;
    if (j < n) {
      rk[u] = rowk[j];
      if (pending) {
        vp[u] = vprev[j];
        pp[u] = pprev[j];
      }
    }
  }
  constexpr int RB = tri_rb<U>();
  double2 xr[RB][U];
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = k + tid + kTriNT * u;
      xr[r][u] = (r < nrow && j > k && j < n) ? row_load<STREAM>(&Aw[(size_t)(row0 + r) * n + j]) : zero;
    }

  // 1. d = p^H v of the pending reflector; p_{k-1}(k), v_{k-1}(k) ride along
  double2 d = zero;
#pragma unroll
  for (int u = 0; u < U; ++u) d = dadd(d, dcmul(pp[u], vp[u]));
  d = wave_total2(d);
  if (lane == 0) xa[wave][0] = d;
  if (tid == 0) {
    xa[0][1] = pp[0];  // entry j = k
    xa[0][2] = vp[0];
  }
  __syncthreads();
  d = sum4(&xa[0][0], 3);
  const double2 pk = xa[0][1], vk = xa[0][2];

  // 2. w = tau p + c d v, c = -|tau|^2 / 2; column k with the pending update; its norm below k+1
  const double c = -0.5 * (t.x * t.x + t.y * t.y);
  const double2 cd = dscale(d, c);
  const double2 wk = dadd(dmul(t, pk), dmul(cd, vk));
  double2 w[U], col[U];
  double xn = 0.0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int j = k + tid + kTriNT * u;
    w[u] = dadd(dmul(t, pp[u]), dmul(cd, vp[u]));
    double2 x = dconj(rk[u]);  // A(j, k) = conj(A(k, j))
    if (pending) x = dsub(x, dadd(dmul(vp[u], dconj(wk)), dmul(w[u], dconj(vk))));
    col[u] = x;
    if (j >= k + 2 && j < n) xn += x.x * x.x + x.y * x.y;
  }
  xn = wave_total(xn);
  if (lane == 0) xb[wave][0] = make_double2(xn, 0.0);
  if (tid == 1) xb[0][1] = col[0];  // alpha = column entry k + 1
  if (tid == 0) xb[0][2] = col[0];  // diagonal entry k
  // coefficients of the workgroup's rows i: held by the thread with i = k + t + 256 u
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int j = k + tid + kTriNT * u;
    const int r = j - row0;
    if (r >= 0 && r < nrow) {
      coef[r][0] = vp[u];
      coef[r][1] = w[u];
    }
  }
  __syncthreads();
  const double xn2 = sum4(&xb[0][0], 3).x;
  const double2 alpha = xb[0][1];
  const double dk = xb[0][2].x;

  // 3. reflector k on x = column k rows k+1 .. n-1
  double beta;
  double2 tau, scale;
  if (xn2 == 0.0 && alpha.y == 0.0) {
    tau = zero;
    beta = alpha.x;
    scale = zero;
  } else {
    const double nrm = sqrt(alpha.x * alpha.x + alpha.y * alpha.y + xn2);
    beta = alpha.x >= 0.0 ? -nrm : nrm;
    tau = make_double2((beta - alpha.x) / beta, -alpha.y / beta);
    const double2 den = make_double2(alpha.x - beta, alpha.y);  // scale = 1 / (alpha - beta)
    const double dd = den.x * den.x + den.y * den.y;
    scale = make_double2(den.x / dd, -den.y / dd);
  }
  double2 v[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int j = k + tid + kTriNT * u;
    v[u] = j == k + 1 ? make_double2(1.0, 0.0) : (j >= k + 2 && j < n ? dmul(col[u], scale) : zero);
  }
  if (blockIdx.x == 0) {
    double2* vout = a.vbuf[k & 1] + (size_t)b * n;
    double2* Vst = a.Vst + (size_t)b * a.strideA;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = k + tid + kTriNT * u;
      if (j > k && j < n) {
        vout[j] = v[u];
        Vst[(size_t)k * n + j] = j == k + 1 ? make_double2(beta, 0.0) : v[u];
      }
    }
    if (tid == 0) {
      a.D[(size_t)b * n + k] = dk;
      a.E[(size_t)b * n + k] = beta;
      a.tau[(size_t)b * n + k] = tau;
    }
  }

  // 4. the workgroup's rows: pending update (written back), p_i = sum_j A_ij v_j,
  //    each row's partials summed over the wave at once (nrow is uniform)
  double2* pout = a.pbuf[k & 1] + (size_t)b * n;
  auto row_work = [&](int r, const double2 (&x)[U]) {
    const int i = row0 + r;
    const double2 vi = coef[r][0], wi = coef[r][1];
    double2 acc = zero;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = k + tid + kTriNT * u;
      if (j > k && j < n) {
        double2 e = x[u];
        if (pending) {
          e = dsub(e, dadd(dmul(vi, dconj(w[u])), dmul(wi, dconj(vp[u]))));
          row_store<STREAM>(&Aw[(size_t)i * n + j], e);
        }
        acc = dadd(acc, dmul(e, v[u]));
      }
    }
    acc = wave_total2(acc);
    if (lane == 0) xc[wave][r] = acc;
  };
#pragma unroll
  for (int r = 0; r < RB; ++r)
    if (r < nrow) row_work(r, xr[r]);
  for (int r0 = RB; r0 < nrow; r0 += RB) {  // rows beyond the prefetched ones
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = k + tid + kTriNT * u;
        xr[r][u] = (r0 + r < nrow && j > k && j < n) ? row_load<STREAM>(&Aw[(size_t)(row0 + r0 + r) * n + j])
                                                     : zero;
      }
#pragma unroll
    for (int r = 0; r < RB; ++r)
      if (r0 + r < nrow) row_work(r0 + r, xr[r]);
  }
  __syncthreads();
  if (tid < nrow) pout[row0 + tid] = sum4(&xc[0][tid], kTriRMax);
}

// The last columns (a trailing block of at most kTriTail rows) in one launch, one
// workgroup of kTailNT threads per problem with the block in registers.  A column
// is a serial chain (the reflector's norm, square root and divisions, then the row
// products), so the layout is chosen to shorten it: the workgroup is 8 half-waves
// of 32 lanes; half-wave h holds the rows h + 8 r (dealt out so that the work
// stays balanced as the block shrinks), lane l of it the columns l + 32 c.  Every
// half-wave forms the reflector redundantly from p and row k in LDS, with the same
// arithmetic and so the same bits: its two sums stay within 32 lanes and the only
// barrier of a column is the one that publishes p and the next row.  The operands
// of the rank-2 update are in registers, one per column slot.  Per column:
//   1. d = Re p^H v of the pending reflector (real for a Hermitian block),
//      w = tau p + c d v, c = -|tau|^2 / 2, column k = conj(row k) - v conj(w_k) - w conj(v_k);
//   2. reflector k from it as in k_tri_col;
//   3. the rows: the pending rank-2 update, p_i = sum_j A_ij v_j.
// v and p are zero outside the trailing block, so the update needs no masks; rows
// and column slots left of it are skipped.  The outputs stay in LDS until the end
// (a barrier would otherwise wait for each column's global stores).
// What bounds it is the issue of its instructions on one CU (about 1100, 770 and 480
// per wave and column with three, two and one live column slots; four waves, one per
// SIMD, since every wave repeats the reflector): 75 columns take 160 us and 96 take
// 185 us, against 229 and 281 us for four lanes per row reading v and p from LDS for
// every entry, with two barriers per column; with eight waves 179 and 212 us.
constexpr int kTriTail = 96;
constexpr int kTailNT = 256;
constexpr int kTailH = kTailNT / 32;  // half-waves
// packed reflectors of the block: column kk's entries kk+1..L-1 at voff(kk)
__host__ __device__ inline int tail_voff(int L, int kk) { return kk * (2 * L - kk - 1) / 2; }
inline size_t tail_lds(int L) { return (size_t)tail_voff(L, L - 1) * sizeof(double2); }

// Sum over each half-wave of 32 lanes; every lane of it gets the total.
SLRX_DEV double half_total(double v) { return row_total(pair_rows(v, v)); }

// e - x conj(y) and e + x y, in fused steps.
SLRX_DEV double2 sub_conj(double2 e, double2 x, double2 y) {
  return make_double2(fma(-x.y, y.y, fma(-x.x, y.x, e.x)), fma(x.x, y.y, fma(-x.y, y.x, e.y)));
}
SLRX_DEV double2 add_mul(double2 e, double2 x, double2 y) {
  return make_double2(fma(-x.y, y.y, fma(x.x, y.x, e.x)), fma(x.y, y.x, fma(x.x, y.y, e.y)));
}

// State of the last-columns kernel that lives across columns (registers) and its LDS.
template <int C>
struct TailState {
  double2 A[4 * C][C], v[C], tau;
};
struct TailLds {
  // by column parity: v and p of the pending reflector, the row of the next column
  double2 vs[2][kTriTail], ps[2][kTriTail], rows[2][kTriTail];
  double2 tl[kTriTail];
  double Dl[kTriTail], El[kTriTail];
};

// Columns kk0 .. kk1-1 of the block, all with their first live column slot CS
// ((kk + 1) / 32 == CS), so that dead slots and rows cost no registers or branches.
template <int C, int CS>
SLRX_DEV void tail_columns(TailState<C>& st, TailLds& q, double2* vl, int L, int kk0, int kk1) {
  constexpr int R = 4 * C, R0 = CS > 0 ? 4 * CS - 1 : 0;  // rows before R0 are finished and cleared
  const int tid = threadIdx.x, lane = tid & 31, h = tid >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const double2 zero = make_double2(0.0, 0.0);
  for (int kk = kk0; kk < kk1; ++kk) {
    const int s = kk & 1;
    // 1. the pending w, column kk, its norm below kk + 1
    double2 p[C], w[C], col[C];
#pragma unroll
    for (int c = CS; c < C; ++c) {
      p[c] = q.ps[s][lane + 32 * c];
      col[c] = q.rows[s][lane + 32 * c];
    }
    const double2 pk = q.ps[s][kk], vk = q.vs[s][kk], pk1 = q.ps[s][kk + 1], vk1 = q.vs[s][kk + 1];
    const double2 rk1 = q.rows[s][kk + 1];
    const double rk = q.rows[s][kk].x;
    // v and p of the pending reflector at kk itself, which slot CS may no longer hold
    double d = (kk & 31) == 31 && lane == 0 ? pk.x * vk.x + pk.y * vk.y : 0.0;
#pragma unroll
    for (int c = CS; c < C; ++c) d = fma(p[c].x, st.v[c].x, fma(p[c].y, st.v[c].y, d));
    d = half_total(d);
    const double2 tau = st.tau;
    const double cd = -0.5 * (tau.x * tau.x + tau.y * tau.y) * d;
    const double2 wk = dadd(dmul(tau, pk), dscale(vk, cd));
    double xn = 0.0;
#pragma unroll
    for (int c = CS; c < C; ++c) {
      const int j = lane + 32 * c;
      w[c] = dadd(dmul(tau, p[c]), dscale(st.v[c], cd));
      col[c] = sub_conj(sub_conj(dconj(col[c]), st.v[c], wk), w[c], vk);
      if (j >= kk + 2) xn += col[c].x * col[c].x + col[c].y * col[c].y;
    }
    const double2 wk1 = dadd(dmul(tau, pk1), dscale(vk1, cd));
    const double2 alpha = sub_conj(sub_conj(dconj(rk1), vk1, wk), wk1, vk);
    xn = half_total(xn);
    // 2. reflector kk
    double beta;
    double2 taun, scale;
    if (xn == 0.0 && alpha.y == 0.0) {
      taun = zero;
      beta = alpha.x;
      scale = zero;
    } else {
      const double nrm = sqrt(alpha.x * alpha.x + alpha.y * alpha.y + xn);
      beta = alpha.x >= 0.0 ? -nrm : nrm;
      const double ib = 1.0 / beta;
      taun = make_double2((beta - alpha.x) * ib, -alpha.y * ib);
      const double2 den = make_double2(alpha.x - beta, alpha.y);  // scale = 1 / (alpha - beta)
      const double id = 1.0 / (den.x * den.x + den.y * den.y);
      scale = make_double2(den.x * id, -den.y * id);
    }
    double2 vn[C];
#pragma unroll
    for (int c = CS; c < C; ++c) {
      const int j = lane + 32 * c;
      double2 x = dmul(col[c], scale);  // 0 beyond the block
      if (j < kk + 2) x = make_double2(j == kk + 1 ? 1.0 : 0.0, 0.0);
      vn[c] = x;
    }
    if (wv == 0 && h == 0) {
      const int vo = tail_voff(L, kk) - kk - 1;
#pragma unroll
      for (int c = CS; c < C; ++c) {
        const int j = lane + 32 * c;
        q.vs[s ^ 1][j] = vn[c];
        if (j > kk && j < L) vl[vo + j] = j == kk + 1 ? make_double2(beta, 0.0) : vn[c];
      }
      if (lane == 0) {
        q.Dl[kk] = rk - 2.0 * (vk.x * wk.x + vk.y * wk.y);
        q.El[kk] = beta;
        q.tl[kk] = taun;
      }
    }
    // 3. the rows: the pending rank-2 update and p_i = sum_j A_ij v_j, all rows in one
    //    block of code so that their loads and sums overlap
    double t[R];
#pragma unroll
    for (int r = R0; r < R; ++r) {
      const int i = h + kTailH * r;
      const double2 vi = q.vs[s][i], wi = dadd(dmul(tau, q.ps[s][i]), dscale(vi, cd));
      double2 acc = zero;
#pragma unroll
      for (int c = CS; c < C; ++c) {
        const double2 e = sub_conj(sub_conj(st.A[r][c], vi, w[c]), wi, st.v[c]);
        st.A[r][c] = e;
        acc = add_mul(acc, e, vn[c]);
      }
      t[r] = pair_rows(acc.x, acc.y);  // even rows of 16 lanes: the real part, odd rows: the imaginary part
    }
#pragma unroll
    for (int r = R0; r < R; ++r) t[r] = row_total(t[r]);
#pragma unroll
    for (int r = R0; r < R; ++r) {
      const int i = h + kTailH * r;
      if (i == kk + 1) {  // the next column's row
#pragma unroll
        for (int c = CS; c < C; ++c) q.rows[s ^ 1][lane + 32 * c] = st.A[r][c];
      }
    }
    if ((lane & 15) == 0) {  // p, cleared for finished rows
#pragma unroll
      for (int r = R0; r < R; ++r) {
        const int i = h + kTailH * r;
        ((double*)&q.ps[s ^ 1][i])[lane >> 4] = i > kk && i < L ? t[r] : 0.0;
      }
    }
    __syncthreads();
#pragma unroll
    for (int c = CS; c < C; ++c) st.v[c] = vn[c];
    st.tau = taun;
  }
}

// C: column slots per lane (L <= 32 C); 4 C rows per half-wave.
template <int C>
__global__ __launch_bounds__(kTailNT) void k_tri_tail(TriArgs a, int k0, const double2* vpend, const double2* ppend,
                                                      const int* stall) {
  constexpr int R = 4 * C;
  extern __shared__ double2 vl[];  // reflectors, packed (tail_voff)
  __shared__ TailLds q;
  const int n = a.n, L = n - k0;
  const int b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 31, h = tid >> 5;
  if (stall && *stall) {  // the resident launch gave up: a finite result that is not used
    for (int i = tid; i < n; i += kTailNT) {
      a.D[(size_t)b * n + i] = a.E[(size_t)b * n + i] = 0.0;
      a.tau[(size_t)b * n + i] = make_double2(0.0, 0.0);
    }
    return;
  }
  const double2* Aw = a.Aw + (size_t)b * a.strideA;
  const double2 zero = make_double2(0.0, 0.0);
  TailState<C> st;
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int i = h + kTailH * r, j = lane + 32 * c;
      double2 x = zero;
      if (i < L && j < L) x = Aw[(size_t)(k0 + i) * n + k0 + j];
      st.A[r][c] = x;
    }
  // pending reflector k0-1 (v, p from the last column launch; none: zeros)
  st.tau = zero;
  if (k0 > 0) st.tau = a.tau[(size_t)b * n + k0 - 1];
  if (tid < kTriTail) {
    const double2* vprev = vpend + (size_t)b * n + k0;
    const double2* pprev = ppend + (size_t)b * n + k0;
    double2 x = zero, y = zero;
    if (k0 > 0 && tid < L) {
      x = vprev[tid];
      y = pprev[tid];
    }
    q.vs[0][tid] = x;
    q.ps[0][tid] = y;
    q.vs[1][tid] = q.ps[1][tid] = zero;
  }
  if (h == 0) {
#pragma unroll
    for (int c = 0; c < C; ++c) q.rows[0][lane + 32 * c] = st.A[0][c];
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < C; ++c) st.v[c] = q.vs[0][lane + 32 * c];
  tail_columns<C, 0>(st, q, vl, L, 0, min(L - 1, 31));
  if constexpr (C > 1) tail_columns<C, 1>(st, q, vl, L, 31, min(L - 1, 63));
  if constexpr (C > 2) tail_columns<C, 2>(st, q, vl, L, 63, min(L - 1, 95));
  if (tid == 0) {  // the last diagonal entry: v of reflector L-2 is 1 there and 0 elsewhere
    const int s = (L - 1) & 1;
    const double2 pk = q.ps[s][L - 1], vk = q.vs[s][L - 1];
    const double2 tau = st.tau;
    const double cd = -0.5 * (tau.x * tau.x + tau.y * tau.y) * (pk.x * vk.x + pk.y * vk.y);
    const double2 wk = dadd(dmul(tau, pk), dscale(vk, cd));
    q.Dl[L - 1] = q.rows[s][L - 1].x - 2.0 * (vk.x * wk.x + vk.y * wk.y);
  }
  __syncthreads();
  double2* Vst = a.Vst + (size_t)b * a.strideA;
  for (int kk = h; kk < L - 1; kk += kTailH) {
    const int vo = tail_voff(L, kk) - kk - 1;
    for (int j = kk + 1 + lane; j < L; j += 32) Vst[(size_t)(k0 + kk) * n + k0 + j] = vl[vo + j];
  }
  if (tid < L) {
    a.D[(size_t)b * n + k0 + tid] = q.Dl[tid];
    if (tid < L - 1) {
      a.E[(size_t)b * n + k0 + tid] = q.El[tid];
      a.tau[(size_t)b * n + k0 + tid] = q.tl[tid];
    }
  }
}

// ------------------------------------------------------- resident reduction
// The columns before the last ones in ONE launch, for n in (kTriResMin, 1280]: the
// trailing block stays in registers (n = 1125: 20 MB over 225 workgroups), so a column
// costs no pass over it and no launch, only an exchange: p = A v of every row and the
// next column have to reach every workgroup.
//   Workgroup g of G holds the rows g + G r, thread t of it their columns t + 256 u (the
// dealt-out rows keep the workgroups balanced as the block shrinks).  Every workgroup
// repeats the reflector, as in k_tri_col, from the vectors of the exchange.
//   The exchange has one hop: a workgroup stores the entries of its rows, and everybody
// polls the vector itself.  Each column has its own vectors (P: p, C: the next column,
// write-once, column k at k n), filled with a bit pattern that no arithmetic produces (all
// ones), so an entry that differs has arrived; entries are read and written as atomic words
// of 8 bytes at device scope.  No counter, no second round trip for a flag: an exchange
// through an agent-scope counter costs 6.2 us over 256 workgroups, this one 0.7 us (n = 140)
// to 1.2 us (n = 1125).
//   What bounds it: the chain of a column.  Measured in cycles per column at n = 405 (135
// workgroups) and n = 1125 (225): exchange 1680 and 2430, d 360 and 420, norm 710 and 820,
// reflector 760 and 880, rows 980 and 1490, publishing 330 and 330 (about 2 GHz).  Whole
// reductions with the last columns: 905 us (n = 405) and 3350 us (n = 1125), where the
// column launches take 1503 and 6970 us (4.4 to 11.6 us each, the longer ones bound by
// reading and writing the trailing block).
//   Every wait ends: a thread that has polled for `wait` ticks, or sees that another has,
// gives up, raises `stall`, and its workgroup leaves the kernel at the next barrier.  The
// last-columns kernel then writes zeros for the problem, the launches of the run's later
// decompositions give up at their first miss, and the host, which finds the flag, repeats
// the run by column launches.  This only happens where workgroups of the launch are kept
// from running (the launches of this process that may run at a time are limited to what
// fits the chip, res_admit).
constexpr int kTriResMin = 128;   // largest n left to the column launches
constexpr unsigned long long kResEmpty = ~0ull;

// An element of a column's vector as two words.
struct ResWords {
  unsigned long long re, im;
};
SLRX_DEV ResWords res_load(const double2* p) {
  const unsigned long long* w = (const unsigned long long*)p;
  return ResWords{__hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                  __hip_atomic_load(w + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)};
}
SLRX_DEV void res_store(double2* p, double2 v) {
  unsigned long long* w = (unsigned long long*)p;
  __hip_atomic_store(w, (unsigned long long)__double_as_longlong(v.x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(w + 1, (unsigned long long)__double_as_longlong(v.y), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// One of two values (by value: a select of their addresses would put them in memory).
SLRX_DEV double2 pick(bool c, double2 a, double2 b) {
  double x = b.x, y = b.y;
  if (c) {
    x = a.x;
    y = a.y;
  }
  return make_double2(x, y);
}
SLRX_DEV bool res_missing(ResWords w) { return w.re == kResEmpty || w.im == kResEmpty; }
SLRX_DEV double2 res_value(ResWords w) {
  return make_double2(__longlong_as_double((long long)w.re), __longlong_as_double((long long)w.im));
}

__global__ __launch_bounds__(256) void k_tri_res_fill(TriResArgs x, long n2, int nb) {
  const long stride = (long)gridDim.x * 256, i0 = (long)blockIdx.x * 256 + threadIdx.x;
  const unsigned long long e = kResEmpty;
  for (int b = 0; b < nb; ++b) {
    ulonglong2* P = (ulonglong2*)(x.P + b * x.sP);
    ulonglong2* C = (ulonglong2*)(x.C + b * x.sC);
    for (long i = i0; i < n2; i += stride) P[i] = C[i] = make_ulonglong2(e, e);
  }
  if (i0 == 0) {
    if (x.clear) x.stall[0] = 0;
    if (x.stall[0] == 0) x.stall[1] = x.id;  // the first launch of the run that gives up stays named
  }
}

// Rows per workgroup by column slots U.  One problem (or few) is split finely: a column
// costs its serial chain, and fewer rows shorten it until the exchange among more
// workgroups costs as much (n = 405: 2, 3, 4, 6, 12 rows take 929, 949, 1005, 1086, 1349
// us).  Batches take as many rows as fit 256 registers per thread, so that more problems run
// at a time.
__host__ __device__ constexpr int res_rows(int U, bool many) {
  return many ? (U == 1 ? 12 : U == 2 ? 14 : U == 3 ? 10 : U == 4 ? 7 : 5) : (U == 1 ? 2 : U == 2 ? 3 : U);
}
template <int U, int R>
struct ResState {
  double2 A[R][U], v[U], tau;
};
template <int U, int R>
struct ResLds {
  double2 v[2][256 * U];         // v by column parity
  double2 pown[R];               // p of this workgroup's rows
  double2 xcol[R];               // the next column's entries in them
  double xc[4][R + 1][2];        // row sums by wave (rows in pairs)
  double xa[4], xb[4];           // wave sums of d and of the norm
  double2 pk, vk, ck, alpha;     // entries k and k + 1
  int dead;
};

// Columns kk0 .. kk1-1, kk / 256 == US.  false: the workgroup gave up.
template <int U, int R, int US>
SLRX_DEV bool res_columns(ResState<U, R>& st, ResLds<U, R>& q, const TriArgs& a, const TriResArgs& x, int g, int G, int b,
                          int kk0, int kk1) {
  constexpr int R0 = US * 256 / ((256 * U + R - 1) / R);  // rows before R0 are finished (G <= ceil(256 U / R))
  const int n = a.n, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double2 zero = make_double2(0.0, 0.0);
  for (int k = kk0; k < kk1; ++k) {
    const int par = k & 1;
    // 0. p of the pending reflector and column k, once every entry has arrived
    double2 p[U], col[U];
    if (k == 0) {
#pragma unroll
      for (int u = US; u < U; ++u) {
        const int j = tid + 256 * u;
        p[u] = col[u] = zero;
        if (j < n) col[u] = dconj(a.Aw[(size_t)b * a.strideA + j]);
      }
    } else {
      const double2* vp = x.P + b * x.sP + (size_t)(k - 1) * n;
      const double2* vc = x.C + b * x.sC + (size_t)(k - 1) * n;
      ResWords wp[U], wc[U];
      bool miss = false;
#pragma unroll
      for (int u = US; u < U; ++u) {
        const int j = tid + 256 * u;
        const bool need = j >= k && j < n;
        wp[u] = wc[u] = ResWords{need ? kResEmpty : 0, 0};
      }
      // The first look comes when the entries are due.  A look that finds them missing
      // costs the whole vector once more, from every workgroup, and delays the stores it
      // waits for: n = 1125 took 4780 us without a delay and 3440 us with it.
      // Due: about 450 cycles after the own entries, and the time that the vectors of all
      // workgroups take; where two workgroups share a CU the others' rows come first (as far
      // as this launch shows: those of other streams on the same CUs are not counted; 15
      // problems of n = 405: 2060 us with 7 units of 64 cycles, 1660 with 24, 1510 with 32,
      // 1570 with 50; 6 of n = 605: 3640, 2590, 2260, 2410; 32 of n = 140: 195, 173, 179, 190).
      const int wgs = (int)(gridDim.x * gridDim.y);
      for (int i = (wgs > 256 ? 28 : 7) + ((n - k) * wgs >> 15); i > 0; --i) __builtin_amdgcn_s_sleep(1);
      unsigned long long t0 = 0;
      for (int spin = 0;; ++spin) {
        miss = false;
#pragma unroll
        for (int u = US; u < U; ++u) {
          const int j = tid + 256 * u;
          if (res_missing(wp[u])) wp[u] = res_load(vp + j);
          if (res_missing(wc[u])) wc[u] = res_load(vc + j);
        }
#pragma unroll
        for (int u = US; u < U; ++u) miss = miss || res_missing(wp[u]) || res_missing(wc[u]);
        if (__ballot(miss) == 0) break;
        if ((spin & 63) == 63) {  // give up after `wait` ticks, or if anybody has
          const unsigned long long t = wall_clock64();
          if (t0 == 0) t0 = t;
          if (t - t0 > x.wait || __hip_atomic_load(x.stall, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
            if (lane == 0) {
              __hip_atomic_store(x.stall, x.stall[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              q.dead = 1;
            }
            break;
          }
        }
      }
#pragma unroll
      for (int u = US; u < U; ++u) {
        p[u] = res_value(wp[u]);
        col[u] = res_value(wc[u]);
      }
    }
    // 1. d = Re p^H v; the entries at k
    double d = 0.0;
#pragma unroll
    for (int u = US; u < U; ++u) d = fma(p[u].x, st.v[u].x, fma(p[u].y, st.v[u].y, d));
    d = wave_total(d);
    if (lane == 0) q.xa[wave] = d;
    if (tid == (k & 255)) {
      q.pk = p[US];
      q.vk = st.v[US];
      q.ck = col[US];
    }
    __syncthreads();
    if (q.dead) return false;
    const double2 tau = st.tau, pk = q.pk, vk = q.vk;
    const double cd = -0.5 * (tau.x * tau.x + tau.y * tau.y) * (((q.xa[0] + q.xa[1]) + q.xa[2]) + q.xa[3]);
    const double2 wk = dadd(dmul(tau, pk), dscale(vk, cd));
    const double dk = q.ck.x - 2.0 * (vk.x * wk.x + vk.y * wk.y);
    // 2. w, column k with the pending update, its norm below k + 1
    double2 w[U];
    double xn = 0.0;
#pragma unroll
    for (int u = US; u < U; ++u) {
      w[u] = dadd(dmul(tau, p[u]), dscale(st.v[u], cd));
      col[u] = sub_conj(sub_conj(col[u], st.v[u], wk), w[u], vk);
      if (tid + 256 * u >= k + 2) xn = fma(col[u].x, col[u].x, fma(col[u].y, col[u].y, xn));
    }
    xn = wave_total(xn);
    if (lane == 0) q.xb[wave] = xn;
    // entry k + 1: thread (k + 1) mod 256, whose slot is the next one at the end of a slot
    const bool wrap = (k & 255) == 255;
    constexpr int UN = US + 1 < U ? US + 1 : US;
    if (tid == ((k + 1) & 255)) q.alpha = pick(wrap, col[UN], col[US]);
    __syncthreads();
    const double xn2 = ((q.xb[0] + q.xb[1]) + q.xb[2]) + q.xb[3];
    const double2 alpha = q.alpha;
    // 3. reflector k
    double beta;
    double2 taun, scale;
    if (xn2 == 0.0 && alpha.y == 0.0) {
      taun = zero;
      beta = alpha.x;
      scale = zero;
    } else {
      const double nrm = sqrt(alpha.x * alpha.x + alpha.y * alpha.y + xn2);
      beta = alpha.x >= 0.0 ? -nrm : nrm;
      const double ib = 1.0 / beta;
      taun = make_double2((beta - alpha.x) * ib, -alpha.y * ib);
      const double2 den = make_double2(alpha.x - beta, alpha.y);  // scale = 1 / (alpha - beta)
      const double id = 1.0 / (den.x * den.x + den.y * den.y);
      scale = make_double2(den.x * id, -den.y * id);
    }
    double2 vn[U];
#pragma unroll
    for (int u = US; u < U; ++u) {
      const int j = tid + 256 * u;
      double2 y = dmul(col[u], scale);  // 0 beyond the matrix
      if (j < k + 2) y = make_double2(j == k + 1 ? 1.0 : 0.0, 0.0);
      vn[u] = y;
      q.v[par][j] = y;
    }
    if (g == k % G) {  // its row k is finished
      double2* Vst = a.Vst + (size_t)b * a.strideA;
#pragma unroll
      for (int u = US; u < U; ++u) {
        const int j = tid + 256 * u;
        if (j > k && j < n) Vst[(size_t)k * n + j] = j == k + 1 ? make_double2(beta, 0.0) : vn[u];
      }
      if (tid == 0) {
        a.D[(size_t)b * n + k] = dk;
        a.E[(size_t)b * n + k] = beta;
        a.tau[(size_t)b * n + k] = taun;
      }
    }
    // 4. the rows: pending update, p_i = sum_j A_ij v_j, the entries of column k + 1.
    //    p and v of the pending reflector at the rows are in LDS (own p, v of all).
    double t[R + 1];
#pragma unroll
    for (int r = R0; r < R; ++r) {
      const int i = min(g + G * r, n - 1);
      const double2 vi = q.v[par ^ 1][i], wi = dadd(dmul(tau, q.pown[r]), dscale(vi, cd));
      double2 acc = zero;
#pragma unroll
      for (int u = US; u < U; ++u) {
        const double2 e = sub_conj(sub_conj(st.A[r][u], vi, w[u]), wi, st.v[u]);
        st.A[r][u] = e;
        acc = add_mul(acc, e, vn[u]);
      }
      t[r] = pair_halves(acc.x, acc.y);
    }
    t[R] = 0.0;
    if (tid == ((k + 1) & 255)) {
#pragma unroll
      for (int r = R0; r < R; ++r) q.xcol[r] = pick(wrap, st.A[r][UN], st.A[r][US]);
    }
    // rows of 16 lanes: re of row r, re of row r + 1, im of row r, im of row r + 1
#pragma unroll
    for (int r = R0; r < R; r += 2) t[r] = row_total(pair_rows(t[r], t[r + 1]));
    if ((lane & 15) == 0) {
#pragma unroll
      for (int r = R0; r < R; r += 2) q.xc[wave][r + (lane >> 4 & 1)][lane >> 5] = t[r];
    }
    __syncthreads();
    {
      const int r = R0 + (tid & 63), i = g + G * r;
      if (r < R) {
        if (wave == 0) {
          const double2 s = make_double2(((q.xc[0][r][0] + q.xc[1][r][0]) + q.xc[2][r][0]) + q.xc[3][r][0],
                                         ((q.xc[0][r][1] + q.xc[1][r][1]) + q.xc[2][r][1]) + q.xc[3][r][1]);
          q.pown[r] = s;
          if (i > k && i < n) res_store(x.P + b * x.sP + (size_t)k * n + i, s);
        } else if (wave == 1) {
          if (i > k && i < n) res_store(x.C + b * x.sC + (size_t)k * n + i, q.xcol[r]);
        }
      }
    }
#pragma unroll
    for (int u = US; u < U; ++u) st.v[u] = vn[u];
    st.tau = taun;
  }
  return true;
}

// U: column slots per thread (n <= 256 U); workgroup (g, problem b) = (blockIdx.x, blockIdx.y);
// columns 0 .. k0-1, k0 = n - kTriTail.
// Two workgroups have to fit a CU (res_capacity): 256 registers a thread, of which the largest
// instance takes 251. Asking the compiler for it (two waves per SIMD in the launch bounds) made
// 256 x 256 x 20 with s = 1125 0.7% slower, so a test reads the counts instead.
template <int U, int R>
__global__ __launch_bounds__(256) void k_tri_res(TriArgs a, TriResArgs x, int k0) {
  __shared__ ResLds<U, R> q;
  const int n = a.n, g = blockIdx.x, G = gridDim.x, b = blockIdx.y, tid = threadIdx.x;
  double2* Aw = a.Aw + (size_t)b * a.strideA;
  const double2 zero = make_double2(0.0, 0.0);
  ResState<U, R> st;
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = g + G * r, j = tid + 256 * u;
      double2 e = zero;
      if (i < n && j < n) e = Aw[(size_t)i * n + j];
      st.A[r][u] = e;
    }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    st.v[u] = zero;
    q.v[1][tid + 256 * u] = zero;
  }
  st.tau = zero;
  if (tid < R) q.pown[tid] = zero;
  if (tid == 0) q.dead = x.missing && g == G - 1;
  __syncthreads();
  if (q.dead) {  // the missing one (tests)
    if (tid == 0 && x.wait == 0) __hip_atomic_store(x.stall, x.stall[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  if (!res_columns<U, R, 0>(st, q, a, x, g, G, b, 0, min(k0, 256))) return;
  if constexpr (U > 1)
    if (!res_columns<U, R, 1>(st, q, a, x, g, G, b, 256, min(k0, 512))) return;
  if constexpr (U > 2)
    if (!res_columns<U, R, 2>(st, q, a, x, g, G, b, 512, min(k0, 768))) return;
  if constexpr (U > 3)
    if (!res_columns<U, R, 3>(st, q, a, x, g, G, b, 768, min(k0, 1024))) return;
  if constexpr (U > 4)
    if (!res_columns<U, R, 4>(st, q, a, x, g, G, b, 1024, min(k0, 1280))) return;
  // the trailing block and the pending reflector for the last-columns kernel
  __syncthreads();
  const size_t o = (size_t)b * n;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int i = g + G * r;
    if (i < k0 || i >= n) continue;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = tid + 256 * u;
      if (j >= k0 && j < n) Aw[(size_t)i * n + j] = st.A[r][u];
    }
    if (tid == 0) a.pbuf[0][o + i] = q.pown[r];
  }
  if (g == 0)
    for (int j = k0 + tid; j < n; j += 256) a.vbuf[0][o + j] = q.v[(k0 - 1) & 1][j];
}

template <int C>
static hipError_t launch_tail_c(const TriArgs& a, int nbatch, int k0, int par, const int* stall, hipStream_t s) {
  static LdsLimit lim;
  const hipError_t e = lim.ensure((const void*)k_tri_tail<C>, tail_lds(32 * C));
  if (e != hipSuccess) return e;
  k_tri_tail<C><<<dim3(1, nbatch), kTailNT, tail_lds(a.n - k0), s>>>(a, k0, a.vbuf[par], a.pbuf[par], stall);
  return hipGetLastError();
}
// Columns k0.. of every problem; v and p of the pending reflector in buffer `par`.
static hipError_t launch_tail(const TriArgs& a, int nbatch, int k0, int par, const int* stall, hipStream_t s) {
  const int L = a.n - k0;
  if (L <= 32) return launch_tail_c<1>(a, nbatch, k0, par, stall, s);
  if (L <= 64) return launch_tail_c<2>(a, nbatch, k0, par, stall, s);
  return launch_tail_c<3>(a, nbatch, k0, par, stall, s);
}

int tri_max_n() { return 3000; }

template <int U>
static void launch_col(const TriArgs& a, int nbatch, int rows, bool stream, hipStream_t s) {
  const int nr = a.n - a.k - 1;
  const dim3 grid((nr + rows - 1) / rows, nbatch);
  if (stream) k_tri_col<U, true><<<grid, kTriNT, 0, s>>>(a, rows);
  else k_tri_col<U, false><<<grid, kTriNT, 0, s>>>(a, rows);
}

// Workgroup budgets per column launch (all problems of a batch together) the
// tuner chooses from: each workgroup recomputes the reflector, so many small
// problems want more rows per workgroup than one large one.
// (Timings at 1125 are from when that size used column launches.)
// One problem also tries 256 with long columns split so that every row of a
// workgroup is loaded at kernel entry (kTriRB rows each, up to 320 workgroups):
// 8.03 against 8.13 ms per 1125 x 1125 decomposition when measured.  The row
// access policy is tuned afterwards for the chosen budget: nontemporal rows took
// 7.15 against 8.04 ms for one 1125 x 1125 problem, but made a batch of 32
// problems of 405 about 6% slower.
static const int kTriBudget1[] = {128, 256, 256};
static const int kTriBudgetN[] = {256, 512, 1024, 2048, 4096};
int tri_budget_candidates(int nbatch) { return nbatch > 1 ? 5 : 3; }
int tri_budget(int nbatch, int cand) { return nbatch > 1 ? kTriBudgetN[cand] : kTriBudget1[cand]; }

hipError_t launch_tridiag(const TriArgs& base, int nbatch, hipStream_t s, int cand, bool stream) {
  const int budget = tri_budget(nbatch, cand);
  const bool fit = nbatch == 1 && cand == 2;
  const int n = base.n;
  if (n > tri_max_n()) return hipErrorInvalidValue;
  const int k0 = n > kTriTail ? n - kTriTail : 0;  // columns k0.. in one launch
  TriArgs a = base;
  for (int k = 0; k < k0; ++k) {
    a.k = k;
    const int nr = n - k - 1;                        // trailing rows
    // rows per workgroup: at most 256 workgroups per problem and about `budget` in all
    int rows = (nr + kTriNT - 1) / kTriNT;
    const int rb = (int)(((long)nr * nbatch + budget - 1) / budget);
    if (rb > rows) rows = rb < kTriRMax ? rb : kTriRMax;
    const int u = (n - k + kTriNT - 1) / kTriNT;      // vector entries per thread
    const int rbu = u > 10 ? 1 : (u > 8 ? 2 : kTriRB); // rows loaded at entry (tri_rb<U>)
    if (fit && rows > rbu && (nr + rbu - 1) / rbu <= 320) rows = rbu;
    if (u <= 1) launch_col<1>(a, nbatch, rows, stream, s);
    else if (u <= 2) launch_col<2>(a, nbatch, rows, stream, s);
    else if (u <= 3) launch_col<3>(a, nbatch, rows, stream, s);
    else if (u <= 4) launch_col<4>(a, nbatch, rows, stream, s);
    else if (u <= 5) launch_col<5>(a, nbatch, rows, stream, s);
    else if (u <= 6) launch_col<6>(a, nbatch, rows, stream, s);
    else if (u <= 8) launch_col<8>(a, nbatch, rows, stream, s);
    else if (u <= 9) launch_col<9>(a, nbatch, rows, stream, s);
    else if (u <= 10) launch_col<10>(a, nbatch, rows, stream, s);
    else launch_col<12>(a, nbatch, rows, stream, s);
  }
  return launch_tail(a, nbatch, k0, (k0 + 1) & 1, nullptr, s);
}

// Workgroups of a resident launch wait for each other, so all of them have to fit the
// chip together with those of the other resident launches that may run.  256 threads of
// at most 256 registers leave room for two workgroups per CU (512 on 256 CUs).  The
// dispatcher deals the workgroups of a launch to the XCDs in turn, whatever they already
// hold, so a launch counts as a multiple of their number: what the fullest XCD gets.
// (Seven launches of 73 are 511 workgroups, but 70 on one XCD, which holds 64.)  Per stream
// (its launches run one after another) the last launch is kept; a new one waits, on the
// device, for the streams whose launches would not fit beside it, the ones used longest ago
// first.  So of launches that may run together the one admitted last has left room for all
// the others.  Ordinary kernels only delay a resident launch.
constexpr int kXcds = 8;
namespace {
struct ResStream {
  hipStream_t s;
  std::thread::id by;  // of hipStreamPerThread, one handle for a stream of every thread
  hipEvent_t done;  // its last launch
  int wgs;          // its largest launch that may not have run yet
};
struct ResHeld {  // a stream whose launches gave up
  hipStream_t s;
  std::thread::id by;
  int stall;  // the last launch that did
  std::chrono::steady_clock::time_point last, until;
};
constexpr std::chrono::seconds kResHold(60);
constexpr size_t kResHeldMax = 64;  // streams remembered
struct ResDevice {
  std::mutex mu;
  std::vector<ResHeld> held;
  std::vector<ResStream> streams;  // in order of their last launch; those that have run are dropped
  std::vector<hipEvent_t> spare;
};
ResDevice g_res[32];
std::atomic<int> g_res_id{0};
std::atomic<int> g_res_stall{0};       // tests: resident launches that miss a workgroup
std::atomic<int> g_res_stall_wait{0};  // and how long they wait for it in ms

// The fewest workgroups per CU over the kernels of U column slots and fewer.
template <int U>
hipError_t res_per_cu(int& per) {
  int a = 0, b = 0;
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&a, k_tri_res<U, res_rows(U, true)>, 256, 0);
  if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, k_tri_res<U, res_rows(U, false)>, 256, 0);
  if (e != hipSuccess) return e;
  per = std::min(per, std::min(a, b));
  if constexpr (U > 1) return res_per_cu<U - 1>(per);
  return hipSuccess;
}

// Workgroups of resident launches that the current device holds at a time (0: unknown),
// whichever kernels they are of; at most two per CU are counted.
int res_capacity() {
  static std::atomic<int> known[32];  // capacity + 1
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  std::atomic<int>& c = known[dev & 31];
  if (c.load() == 0) {
    int cus = 0, per = 2;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        res_per_cu<5>(per) != hipSuccess) {
      (void)hipGetLastError();
      return 0;
    }
    c.store(cus / kXcds * kXcds * per + 1);
  }
  return c.load() - 1;
}

// The thread that tells the streams behind one handle apart.
std::thread::id res_thread(hipStream_t s) {
  return s == hipStreamPerThread ? std::this_thread::get_id() : std::thread::id();
}
ResDevice* res_device() {
  int dev = 0;
  return hipGetDevice(&dev) == hipSuccess ? &g_res[dev & 31] : nullptr;
}
std::vector<ResHeld>::iterator res_held(ResDevice& d, hipStream_t s) {
  const std::thread::id by = res_thread(s);
  return std::find_if(d.held.begin(), d.held.end(), [&](const ResHeld& h) { return h.s == s && h.by == by; });
}

// Room for wgs workgroups on stream s (d.mu held); the stream's entry is the last one then.
hipError_t res_admit(ResDevice& d, int wgs, hipStream_t s) {
  wgs = (wgs + kXcds - 1) / kXcds * kXcds;
  const std::thread::id by = res_thread(s);
  ResStream mine{s, by, nullptr, wgs};
  const RelaxedCapture relaxed;
  std::vector<ResStream> keep;
  for (const ResStream& t : d.streams) {
    // an event of a stream that is gone gives an error: its work has run
    const bool ran = hipEventQuery(t.done) != hipErrorNotReady;
    (void)hipGetLastError();
    if (t.s == s && t.by == by) {
      mine.done = t.done;
      if (!ran && t.wgs > mine.wgs) mine.wgs = t.wgs;
    } else if (ran) {
      d.spare.push_back(t.done);
    } else {
      keep.push_back(t);
    }
  }
  hipError_t e = hipSuccess;
  int sum = wgs;
  for (size_t i = keep.size(); i-- > 0 && e == hipSuccess;) {
    if (sum + keep[i].wgs <= res_capacity()) sum += keep[i].wgs;
    else e = hipStreamWaitEvent(s, keep[i].done, 0);
  }
  if (!mine.done) {
    if (d.spare.empty()) {
      const hipError_t ec = hipEventCreateWithFlags(&mine.done, hipEventDisableTiming);
      if (ec != hipSuccess) {
        d.streams.swap(keep);
        return ec;
      }
    } else {
      mine.done = d.spare.back();
      d.spare.pop_back();
    }
  }
  keep.push_back(mine);
  d.streams.swap(keep);
  return e;
}

int res_groups(int n, bool many) {
  const int R = res_rows((n + 255) / 256, many);
  return (n + R - 1) / R;
}
// The split of a batch: fine while all problems then run at a time on a workgroup per CU,
// else coarse, as many problems at a time as fit, in launches of about equal size.
struct ResShape {
  bool many;
  int G, per;  // workgroups per problem, problems per launch
};
ResShape res_shape(int n, int nbatch) {
  const bool many = nbatch * res_groups(n, false) > 256;
  const int G = res_groups(n, many), most = res_capacity() / G;
  const int launches = (nbatch + most - 1) / most;
  return ResShape{many, G, (nbatch + launches - 1) / launches};
}
}  // namespace

void tri_resident_gave_up(hipStream_t s, int stall) {
  ResDevice* d = res_device();
  if (!d) return;
  std::lock_guard<std::mutex> lk(d->mu);
  const auto now = std::chrono::steady_clock::now();
  const auto it = res_held(*d, s);
  if (it == d->held.end()) {
    if (d->held.size() >= kResHeldMax) d->held.erase(d->held.begin());
    d->held.push_back(ResHeld{s, res_thread(s), stall, now, now});
  } else if (it->stall != stall) {  // several runs may report one launch
    if (now - it->last < 2 * kResHold) it->until = now + kResHold;
    it->stall = stall;
    it->last = now;
  }
}
bool tri_resident_on(hipStream_t s) {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return false;
  uint32_t mask[32] = {};  // without a mask: ones (0.5 us)
  const int words = std::min((cus + 31) / 32, 32);
  if (hipExtStreamGetCUMask(s, words, mask) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  int in = 0;
  for (uint32_t w : mask) in += __builtin_popcount(w);
  if (in < cus) return false;
  ResDevice& d = g_res[dev & 31];
  std::lock_guard<std::mutex> lk(d.mu);
  const auto it = res_held(d, s);
  return it == d.held.end() || std::chrono::steady_clock::now() >= it->until;
}
void tri_resident_forget(hipStream_t s) {
  ResDevice* d = res_device();
  if (!d) return;
  std::lock_guard<std::mutex> lk(d->mu);
  const auto it = res_held(*d, s);
  if (it != d->held.end()) d->held.erase(it);
}

// Sizes with more columns than the last-columns kernel takes plus a few (each is worth an
// exchange then), whose rows fit the registers of 256 workgroups.
bool tri_resident(int n) { return n > kTriResMin && n <= 256 * 5 && res_capacity() >= 256; }
int tri_resident_workgroups(int n, int nbatch) {
  const ResShape r = res_shape(n, nbatch);
  return r.G * r.per;
}

template <int U>
static void res_launch(const TriArgs& a, const TriResArgs& x, const ResShape& r, int nb, int k0, hipStream_t s) {
  const dim3 grid(r.G, nb);
  if (r.many) k_tri_res<U, res_rows(U, true)><<<grid, 256, 0, s>>>(a, x, k0);
  else k_tri_res<U, res_rows(U, false)><<<grid, 256, 0, s>>>(a, x, k0);
}

hipError_t launch_tridiag_resident(const TriArgs& base, const TriResArgs& xbase, int nbatch, hipStream_t s) {
  const int n = base.n, U = (n + 255) / 256, k0 = n - kTriTail;
  if (!tri_resident(n)) return hipErrorInvalidValue;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  ResDevice& d = g_res[dev & 31];
  const ResShape r = res_shape(n, nbatch);
  TriResArgs x = xbase;
  x.wait = kTriResWait;
  do x.id = g_res_id.fetch_add(1) + 1;
  while (x.id == 0);
  x.missing = g_res_stall.load() > 0 && g_res_stall.fetch_sub(1) > 0;
  if (x.missing) x.wait = (unsigned long long)g_res_stall_wait.load() * 100000;
  k_tri_res_fill<<<512, 256, 0, s>>>(x, (long)n * n, nbatch);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  for (int b = 0; b < nbatch; b += r.per) {
    const int nb = nbatch - b < r.per ? nbatch - b : r.per;
    TriArgs a = base;
    a.Aw += b * base.strideA;
    a.Vst += b * base.strideA;
    a.D += (long)b * n;
    a.E += (long)b * n;
    a.tau += (long)b * n;
    a.vbuf[0] += (long)b * n;
    a.pbuf[0] += (long)b * n;
    TriResArgs y = x;
    y.P += b * x.sP;
    y.C += b * x.sC;
    std::lock_guard<std::mutex> lk(d.mu);  // launches are made in the order of their admission
    if ((e = res_admit(d, r.G * nb, s)) != hipSuccess) return e;
    if (U == 1) res_launch<1>(a, y, r, nb, k0, s);
    else if (U == 2) res_launch<2>(a, y, r, nb, k0, s);
    else if (U == 3) res_launch<3>(a, y, r, nb, k0, s);
    else if (U == 4) res_launch<4>(a, y, r, nb, k0, s);
    else res_launch<5>(a, y, r, nb, k0, s);
    e = hipGetLastError();
    const hipError_t er = hipEventRecord(d.streams.back().done, s);
    if (e != hipSuccess) return e;
    if (er != hipSuccess) return er;
  }
  return launch_tail(base, nbatch, k0, 0, x.stall, s);
}

}  // namespace slrx

extern "C" void slrx_fault_stall(int32_t n) { slrx::g_res_stall.store(n < 0 ? 0 : n); }
extern "C" void slrx_fault_stall_wait(int32_t ms) {
  slrx::g_res_stall_wait.store(ms < 0 ? 0 : ms > 2000 ? 2000 : ms);
}
