// Back-transformation of the tridiagonal eigenvectors, U = Q Z (FP64), last
// stage of the Gram eigen-decomposition in the weight update (Sec. III.B,
// Algorithm 1 step 1).
//
// The Householder reduction leaves Q = H_0 H_1 ... H_{n-2}, H_k = I - tau_k v_k
// v_k^H, v_k zero above row k+1 and one at row k+1.  Reflectors are grouped in
// blocks of kBtNb; a block is I - V T V^H with V (n x kBtNb) its reflectors and
// T upper triangular (the forward, column-wise compact WY form, T(i,i) = tau_i,
// T(0:i, i) = -tau_i T(0:i, 0:i) V(:, 0:i)^H v_i).  With Y = V T the block acts
// on Z as Z <- Z - Y (V^H Z), and Q Z applies the blocks from the last to the
// first.  Every product is a complex FP64 matrix product on the f64 16x16x4
// MFMA.  k_bt_apply applies every block to eight columns of Z held in LDS; the
// products within the blocks, and sizes whose columns do not fit, take output tiles of
// 64 x 16 (one 16 x 16 tile per wave), K staged through LDS in chunks of 16; long
// reductions are split over workgroups into partial results that the consumer sums
// in a fixed order (results are reproducible bit for bit).
#include "common.h"
#include "kernels.h"

namespace slrx {

typedef double v4d __attribute__((ext_vector_type(4)));

namespace {

constexpr int kBtNb = 64;  // reflectors per block
constexpr int kTM = 64, kTN = 16, kKC = 16;
constexpr int kBtSplitG = 4;  // split-K of the block Gram matrices
constexpr int kBtSplitW = 8;  // split-K of V^H Z

enum BtKind { BT_GRAM = 0, BT_YMAT = 1, BT_APPLY_W = 2, BT_APPLY_Z = 3 };

// One product of the back-transformation for reflector block g.  For
//   r0 = nb g + 1 (first row the block touches), m = n - r0, nr = reflectors in the block,
//   GRAM:    G_g = V_g^H V_g        (nr x nr, K = m), partial z -> Gp[(z * ng + g) nb^2]
//   YMAT:    Y_g = V_g T_g          (m x nr, K = nr)  -> Yx, column-major n x n, rows r0..
//   APPLY_W: W   = V_g^H Z(r0:, :)  (nr x n, K = m),  partial z -> Wp[z nb n]
//   APPLY_Z: Z(r0:, :) -= Y_g W     (m x n, K = nr),  W = the partials summed (k_bt_wsum).
struct BtArgs {
  int n, ng, nsplit, g;
  const double2* Vx;  // reflectors, column-major n x n, explicit zeros and unit entries
  double2* Yx;        // Y blocks, column-major n x n
  double2* Z;         // eigenvectors, column-major n x n
  double2* Gp;        // Gram partials of the blocks
  double2* Tb;        // T of the blocks, column-major nb x nb each
  double2* Wp;        // V^H Z partials, column-major nb x n each
  const double2* tau; // reflector scalars, n
  long sV, sY, sZ, sW;  // strides between the problems of a batch (sW: scratch)
};

// The arguments of problem b of a batch.
SLRX_DEV BtArgs bt_at(BtArgs a, int b) {
  a.Vx += b * a.sV;
  a.Yx += b * a.sY;
  a.Z += b * a.sZ;
  a.Gp += b * a.sW;
  a.Tb += b * a.sW;
  a.Wp += b * a.sW;
  a.tau += (long)b * a.n;
  return a;
}

template <int KIND>
__global__ __launch_bounds__(256) void k_bt_gemm(BtArgs a0, int zper) {
  // blockIdx.z = problem * zper + (split / block index within the problem)
  const BtArgs a = bt_at(a0, blockIdx.z / zper);
  const int bz = blockIdx.z % zper;
  __shared__ double Lar[kKC][kTM + 1], Lai[kKC][kTM + 1];  // padded against bank conflicts
  __shared__ double Lbr[kKC][kTN + 1], Lbi[kKC][kTN + 1];
  const int n = a.n;
  int g, z;
  if (KIND == BT_GRAM) {
    g = bz / a.nsplit;
    z = bz % a.nsplit;
  } else if (KIND == BT_YMAT) {
    g = bz;
    z = 0;
  } else {
    g = a.g;
    z = bz;
  }
  const int k0 = kBtNb * g, r0 = k0 + 1, m = n - r0;
  const int nr = min(kBtNb, n - 1 - k0);
  int M, N, K;
  if (KIND == BT_GRAM) { M = nr; N = nr; K = m; }
  else if (KIND == BT_YMAT) { M = m; N = nr; K = nr; }
  else if (KIND == BT_APPLY_W) { M = nr; N = n; K = m; }
  else { M = m; N = n; K = nr; }
  const int i0 = blockIdx.y * kTM, j0 = blockIdx.x * kTN;
  if (i0 >= M || j0 >= N) return;
  // split-K range of this workgroup (whole chunks)
  int kb = 0, ke = K;
  if (KIND == BT_GRAM || KIND == BT_APPLY_W) {
    const int per = ((K + a.nsplit - 1) / a.nsplit + kKC - 1) / kKC * kKC;
    kb = z * per;
    ke = min(K, kb + per);
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  v4d accR = v4d{0.0, 0.0, 0.0, 0.0}, accI = v4d{0.0, 0.0, 0.0, 0.0};
  // global loads of one K chunk into registers (4 A elements and 1 B element per thread)
  constexpr int kAE = kTM * kKC / 256;
  double2 ra[kAE], rb;
  auto load_chunk = [&](int kc) {
#pragma unroll
    for (int u = 0; u < kAE; ++u) {
      const int e = tid + 256 * u;
      double2 v = make_double2(0.0, 0.0);
      if (KIND == BT_GRAM || KIND == BT_APPLY_W) {  // A(i, r) = conj(V(r0 + r, k0 + i))
        const int i = e / kKC, r = kc + e % kKC;
        if (i0 + i < M && r < ke) {
          v = a.Vx[(long)(r0 + r) + (long)(k0 + i0 + i) * n];
          v.y = -v.y;
        }
      } else {  // A(r, l) column-major: V for YMAT, Y for APPLY_Z
        const int i = e % kTM, l = kc + e / kTM;
        if (i0 + i < M && l < ke) {
          const double2* src = KIND == BT_YMAT ? a.Vx : a.Yx;
          v = src[(long)(r0 + i0 + i) + (long)(k0 + l) * n];
        }
      }
      ra[u] = v;
    }
    const int j = tid / kKC, k = kc + tid % kKC, c = j0 + j;
    rb = make_double2(0.0, 0.0);
    if (k < ke && c < N) {
      if (KIND == BT_GRAM) rb = a.Vx[(long)(r0 + k) + (long)(k0 + c) * n];
      else if (KIND == BT_YMAT) rb = a.Tb[(long)g * kBtNb * kBtNb + k + (long)c * kBtNb];
      else if (KIND == BT_APPLY_W) rb = a.Z[(long)(r0 + k) + (long)c * n];
      else rb = a.Wp[(long)a.nsplit * kBtNb * n + k + (long)c * kBtNb];  // summed W
    }
  };
  // APPLY_Z: this lane's Z elements, loaded before the product
  double2 zold[4];
  if (KIND == BT_APPLY_Z) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = i0 + wave * 16 + (lane >> 4) + 4 * v;
      const int c = j0 + (lane & 15);
      zold[v] = (i < M && c < N) ? a.Z[(long)(r0 + i) + (long)c * n] : make_double2(0.0, 0.0);
    }
  }
  if (kb < ke) load_chunk(kb);
  for (int kc = kb; kc < ke; kc += kKC) {
#pragma unroll
    for (int u = 0; u < kAE; ++u) {
      const int e = tid + 256 * u;
      int i, kk;
      if (KIND == BT_GRAM || KIND == BT_APPLY_W) {
        i = e / kKC;
        kk = e % kKC;
      } else {
        kk = e / kTM;
        i = e % kTM;
      }
      Lar[kk][i] = ra[u].x;
      Lai[kk][i] = ra[u].y;
    }
    Lbr[tid % kKC][tid / kKC] = rb.x;
    Lbi[tid % kKC][tid / kKC] = rb.y;
    __syncthreads();
    if (kc + kKC < ke) load_chunk(kc + kKC);  // next chunk in flight during the products
#pragma unroll
    for (int kq = 0; kq < kKC; kq += 4) {
      const int kl = kq + (lane >> 4);
      const double ar = Lar[kl][wave * 16 + (lane & 15)];
      const double ai = Lai[kl][wave * 16 + (lane & 15)];
      const double br = Lbr[kl][lane & 15];
      const double bi = Lbi[kl][lane & 15];
      accR = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, br, accR, 0, 0, 0);
      accR = __builtin_amdgcn_mfma_f64_16x16x4f64(-ai, bi, accR, 0, 0, 0);
      accI = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, bi, accI, 0, 0, 0);
      accI = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, br, accI, 0, 0, 0);
    }
    __syncthreads();
  }
  // D layout of the f64 16x16x4 MFMA: item v of lane l is row l/16 + 4v, column l%16.
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = i0 + wave * 16 + (lane >> 4) + 4 * v;
    const int c = j0 + (lane & 15);
    if (i >= M || c >= N) continue;
    const double2 r = make_double2(accR[v], accI[v]);
    if (KIND == BT_GRAM) {
      a.Gp[((long)z * a.ng + g) * kBtNb * kBtNb + i + (long)c * kBtNb] = r;
    } else if (KIND == BT_YMAT) {
      a.Yx[(long)(r0 + i) + (long)(k0 + c) * n] = r;
    } else if (KIND == BT_APPLY_W) {
      a.Wp[(long)z * kBtNb * n + i + (long)c * kBtNb] = r;
    } else {
      a.Z[(long)(r0 + i) + (long)c * n] = make_double2(zold[v].x - r.x, zold[v].y - r.y);
    }
  }
}

// W = sum of the split-K partials of V^H Z, in a fixed order, into the slot
// after the partials.
__global__ void k_bt_wsum(BtArgs a0) {
  const BtArgs a = bt_at(a0, blockIdx.y);
  const long o = (long)blockIdx.x * 256 + threadIdx.x;
  const long len = (long)kBtNb * a.n;
  if (o >= len) return;
  double2 v = make_double2(0.0, 0.0);
  for (int p = 0; p < a.nsplit; ++p) {
    const double2 w = a.Wp[(long)p * len + o];
    v.x += w.x;
    v.y += w.y;
  }
  a.Wp[(long)a.nsplit * len + o] = v;
}

// Reflectors in explicit form, in place: column k of the n x n column-major
// matrix becomes v_k (zero above row k+1, one at row k+1; the last column is zero).
__global__ void k_bt_explicit(int n, double2* V0, long sV) {
  double2* V = V0 + blockIdx.y * sV;
  const long o = (long)blockIdx.x * 256 + threadIdx.x;
  if (o >= (long)n * n) return;
  const int R = (int)(o % n), k = (int)(o / n);
  if (R < k + 1) V[o] = make_double2(0.0, 0.0);
  else if (R == k + 1) V[o] = make_double2(1.0, 0.0);
}

// T of each block by recursive doubling: for adjacent index blocks A, B (B after
// A), the product of their block reflectors has T = [T_A, -T_A G_AB T_B; 0, T_B]
// with G_AB = V_A^H V_B; blocks of 1, 2, 4, .., 32 are joined level by level,
// every entry of a level in parallel.  T is packed by columns (T(l, q) at
// q(q+1)/2 + l, l <= q); G's strict upper triangle likewise (l < i at
// i(i-1)/2 + l) and is overwritten level by level with X = G_AB T_B.  Indices
// beyond the block's reflectors get tau = 0 and G = 0, so their rows and
// columns of T are zero.  A serial chain of 2 x 6 levels in one workgroup per block, bound
// by LDS latency: a thread per entry of the widest level, and all of a thread's split sums
// of G in flight together (51 us with 256 threads and one load at a time, 19 us so).
constexpr int kTmatThreads = 1024;

__global__ __launch_bounds__(kTmatThreads) void k_bt_tmat(BtArgs a0) {
  const BtArgs a = bt_at(a0, blockIdx.y);
  const double2* tau = a.tau;
  __shared__ double2 T[kBtNb * (kBtNb + 1) / 2];
  __shared__ double2 G[kBtNb * (kBtNb - 1) / 2];
  const int g = blockIdx.x, tid = threadIdx.x;
  const int k0 = kBtNb * g, nr = min(kBtNb, a.n - 1 - k0);
  auto tix = [](int l, int q) { return q * (q + 1) / 2 + l; };
  auto gix = [](int l, int i) { return i * (i - 1) / 2 + l; };
  double2 gs[kBtNb * kBtNb / kTmatThreads];  // entry (l, i), l = e % 64, i = e / 64
#pragma unroll
  for (int u = 0; u < kBtNb * kBtNb / kTmatThreads; ++u) gs[u] = make_double2(0.0, 0.0);
#pragma unroll 4
  for (int p = 0; p < a.nsplit; ++p)
#pragma unroll
    for (int u = 0; u < kBtNb * kBtNb / kTmatThreads; ++u) {
      const int e = tid + kTmatThreads * u, l = e % kBtNb, i = e / kBtNb;
      if (l < i && i < nr) gs[u] = dadd(gs[u], a.Gp[((long)p * a.ng + g) * kBtNb * kBtNb + e]);
    }
#pragma unroll
  for (int u = 0; u < kBtNb * kBtNb / kTmatThreads; ++u) {
    const int e = tid + kTmatThreads * u, l = e % kBtNb, i = e / kBtNb;
    if (l < i) G[gix(l, i)] = gs[u];
  }
  for (int e = tid; e < kBtNb * (kBtNb + 1) / 2; e += kTmatThreads) T[e] = make_double2(0.0, 0.0);
  __syncthreads();
  if (tid < nr) T[tix(tid, tid)] = tau[k0 + tid];
  __syncthreads();
  for (int bs = 1; bs < kBtNb; bs *= 2) {
    const int per_pair = bs * bs, total = (kBtNb / (2 * bs)) * per_pair;  // = 32 bs <= kTmatThreads
    const int pr = tid / per_pair, rr = tid % per_pair;
    const int a0 = 2 * bs * pr, b0 = a0 + bs;
    const int r = a0 + rr / bs, c = b0 + rr % bs;
    // X(r, c) = sum_{q in B, q <= c} G(r, q) T(q, c), r in A, c in B
    double2 x = make_double2(0.0, 0.0);
    if (tid < total)
      for (int q = b0; q <= c; ++q) x = dadd(x, dmul(G[gix(r, q)], T[tix(q, c)]));
    __syncthreads();
    if (tid < total) G[gix(r, c)] = x;
    __syncthreads();
    // T(r, c) = -sum_{p in A, p >= r} T(r, p) X(p, c), r in A, c in B
    if (tid < total) {
      double2 acc = make_double2(0.0, 0.0);
      for (int p = r; p < b0; ++p) acc = dadd(acc, dmul(T[tix(r, p)], G[gix(p, c)]));
      T[tix(r, c)] = make_double2(-acc.x, -acc.y);
    }
    __syncthreads();
  }
  double2* out = a.Tb + (long)g * kBtNb * kBtNb;
  for (int e = tid; e < kBtNb * kBtNb; e += kTmatThreads) {
    const int r = e % kBtNb, c = e / kBtNb;
    out[e] = r <= c ? T[tix(r, c)] : make_double2(0.0, 0.0);
  }
}

// Every block applied to eight columns of Z by one workgroup: Z(:, c0 .. c0+7) stays in
// LDS as rows [re of 8 | im of 8], the 16 columns of a real operand, so a complex product is
// two MFMAs, [Vr^T Z | Vi^T Z], whose halves are combined across lanes.  The columns of Z
// are independent, so one launch does what took three per block of 64 reflectors (54 at
// n = 1125), each with too little work for the chip.
// Per block: W = V^H Z, a wave per 16 reflectors and half of the rows; then Z -= Y W, a wave
// per 16 rows in turn.  Bound by the FP64 matrix cores of the ceil(n / 8) CUs at work (280 us
// of its 468 at n = 1125), the panels' loads running ahead of them: the whole
// back-transformation takes 717 -> 542 us at n = 1125, 183 -> 132 at 405, 63 -> 49 at 75.
constexpr int kApNT = 512;
constexpr int kApCols = 8;
static size_t bt_apply_lds(int n) { return ((size_t)(n + 1) * 16 + 2 * kBtNb * 16) * sizeof(double); }
constexpr size_t kApLds = 160 * 1024;

// The value of lane ^ 8 (within rows of 16 lanes).
SLRX_DEV double swap8(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x128, 0xf, 0xf, false);  // row_ror:8
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x128, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__global__ __launch_bounds__(kApNT) void k_bt_apply(BtArgs a0) {
  extern __shared__ double zl[];  // [n + 1][16], row n zero, then W [2][kBtNb][16]
  const BtArgs a = bt_at(a0, blockIdx.y);
  const int n = a.n, c0 = kApCols * blockIdx.x, nc = min(kApCols, n - c0);
  double* W = zl + (size_t)(n + 1) * 16;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j = lane & 15, q = lane >> 4;  // column (or row) and k of the MFMA operands
  const double2 zero = make_double2(0.0, 0.0);
  const v4d vzero = v4d{0.0, 0.0, 0.0, 0.0};
  for (int e = tid; e < kApCols * (n + 8); e += kApNT) {  // 8 rows of 8 columns per wave
    const int c = e / 8 % kApCols, r = e / 64 * 8 + e % 8;
    const double2 v = c < nc && r < n ? a.Z[(long)(c0 + c) * n + r] : zero;
    if (r <= n) {
      zl[r * 16 + c] = v.x;
      zl[r * 16 + kApCols + c] = v.y;
    }
  }
  __syncthreads();
  for (int g = a.ng - 1; g >= 0; --g) {
    const int k0 = kBtNb * g, r0 = k0 + 1, m = n - r0, nr = min(kBtNb, n - 1 - k0);
    // Loads are clamped instead of masked (no branch between a load and its use): rows from
    // m on meet the zero row of Z or results that are not stored, columns from nr on zero rows of W.
    {  // W = V^H Z: reflectors 16 tile + j, rows kb .. ke-1 of the block
      const int tile = wave & 3, half = wave >> 2;
      const int mh = (m + 95) / 96 * 48, kb = half * mh, ke = min(m, kb + mh);
      const double2* vc = a.Vx + (long)(k0 + min(16 * tile + j, nr - 1)) * n + r0;
      auto fetch = [&](double2 (&x)[4], int kc) {
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = vc[min(kc + 4 * u + q, m - 1)];
      };
      v4d P1 = vzero, P2 = vzero;
      auto product = [&](const double2 (&x)[4], int kc) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const double b = zl[min(r0 + kc + 4 * u + q, n) * 16 + j];
          P1 = __builtin_amdgcn_mfma_f64_16x16x4f64(x[u].x, b, P1, 0, 0, 0);
          P2 = __builtin_amdgcn_mfma_f64_16x16x4f64(x[u].y, b, P2, 0, 0, 0);
        }
      };
      double2 x0[4], x1[4], x2[4];
      fetch(x0, kb);
      fetch(x1, kb + 16);
      for (int kc = kb; kc < ke; kc += 48) {
        fetch(x2, kc + 32);
        product(x0, kc);
        fetch(x0, kc + 48);
        product(x1, kc + 16);
        fetch(x1, kc + 64);
        product(x2, kc + 32);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {  // Re: Vr Zr + Vi Zi, Im: Vr Zi - Vi Zr
        const double o = swap8(P2[v]);
        W[(half * kBtNb + 16 * tile + q + 4 * v) * 16 + j] = j < kApCols ? P1[v] + o : P1[v] - o;
      }
    }
    // Z -= Y W: rows i0 .. i0+15, columns 4 u + q of Y, u in halves H
    constexpr int kH = kBtNb / 8, kStep = 16 * (kApNT / 64);
    auto fetch = [&](double2 (&y)[kH], int i0, int h) {
      const double2* yr = a.Yx + (long)k0 * n + r0 + min(i0 + j, m - 1);
#pragma unroll
      for (int u = 0; u < kH; ++u) y[u] = yr[min(4 * (kH * h + u) + q, nr - 1) * n];
    };
    double2 y0[kH], y1[kH];
    fetch(y0, 16 * wave, 0);
    __syncthreads();
    double w[kBtNb / 4];
#pragma unroll
    for (int u = 0; u < kBtNb / 4; ++u)
      w[u] = W[(4 * u + q) * 16 + j] + W[(kBtNb + 4 * u + q) * 16 + j];
    if (nr < kBtNb) {
#pragma unroll
      for (int u = 0; u < kBtNb / 4; ++u)
        if (4 * u + q >= nr) w[u] = 0.0;
    }
    for (int i0 = 16 * wave; i0 < m; i0 += kStep) {
      v4d P1 = vzero, P2 = vzero;
      auto product = [&](const double2 (&y)[kH], int h) {
#pragma unroll
        for (int u = 0; u < kH; ++u) {
          P1 = __builtin_amdgcn_mfma_f64_16x16x4f64(y[u].x, w[kH * h + u], P1, 0, 0, 0);
          P2 = __builtin_amdgcn_mfma_f64_16x16x4f64(y[u].y, w[kH * h + u], P2, 0, 0, 0);
        }
      };
      fetch(y1, i0, 1);
      product(y0, 0);
      fetch(y0, i0 + kStep, 0);
      product(y1, 1);
#pragma unroll
      for (int v = 0; v < 4; ++v) {  // Re: Yr Wr - Yi Wi, Im: Yr Wi + Yi Wr
        const double o = swap8(P2[v]);
        if (i0 + q + 4 * v < m) zl[(r0 + i0 + q + 4 * v) * 16 + j] -= j < kApCols ? P1[v] - o : P1[v] + o;
      }
    }
    __syncthreads();
  }
  for (int e = tid; e < kApCols * (n + 7); e += kApNT) {
    const int c = e / 8 % kApCols, r = e / 64 * 8 + e % 8;
    if (c < nc && r < n) a.Z[(long)(c0 + c) * n + r] = make_double2(zl[r * 16 + c], zl[r * 16 + kApCols + c]);
  }
}

}  // namespace

static int bt_nblocks(int n) { return n > 1 ? (n - 2) / kBtNb + 1 : 0; }

size_t bt_scratch_elems(int n) {
  const int ng = bt_nblocks(n);
  return (size_t)ng * kBtNb * kBtNb * (1 + kBtSplitG) + (size_t)(kBtSplitW + 1) * kBtNb * n;
}

hipError_t launch_backtransform(const BackTrArgs& b, hipStream_t s) {
  const int n = b.n, nb = b.nb;
  if (n < 2) return hipSuccess;  // Q = I
  const int ng = bt_nblocks(n);
  BtArgs a{};
  a.n = n;
  a.ng = ng;
  a.Vx = b.V;
  a.Yx = b.Y;
  a.Z = b.Z;
  a.tau = b.tau;
  a.Tb = b.scratch;
  a.Gp = b.scratch + (size_t)ng * kBtNb * kBtNb;
  a.Wp = a.Gp + (size_t)ng * kBtNb * kBtNb * kBtSplitG;
  a.sV = b.sV;
  a.sY = b.sY;
  a.sZ = b.sZ;
  a.sW = b.s_scratch;
  k_bt_explicit<<<dim3((unsigned)(((long)n * n + 255) / 256), nb), 256, 0, s>>>(n, b.V, b.sV);
  const int mt = (n - 1 + kTM - 1) / kTM;  // row tiles of the largest block (m = n - 1)
  a.nsplit = kBtSplitG;
  k_bt_gemm<BT_GRAM><<<dim3(kBtNb / kTN, 1, nb * ng * kBtSplitG), 256, 0, s>>>(a, ng * kBtSplitG);
  k_bt_tmat<<<dim3(ng, nb), kTmatThreads, 0, s>>>(a);
  a.nsplit = 1;
  k_bt_gemm<BT_YMAT><<<dim3(kBtNb / kTN, mt, nb * ng), 256, 0, s>>>(a, ng);
  if (bt_apply_lds(n) <= kApLds) {  // n <= 1151: the columns of Z fit a workgroup's LDS
    static LdsLimit lim;
    const hipError_t e = lim.ensure((const void*)k_bt_apply, kApLds);
    if (e != hipSuccess) return e;
    k_bt_apply<<<dim3((n + kApCols - 1) / kApCols, nb), kApNT, bt_apply_lds(n), s>>>(a);
    return hipGetLastError();
  }
  const int nt = (n + kTN - 1) / kTN;
  a.nsplit = kBtSplitW;
  for (int g = ng - 1; g >= 0; --g) {
    a.g = g;
    const int m = n - (kBtNb * g + 1);
    k_bt_gemm<BT_APPLY_W><<<dim3(nt, 1, nb * kBtSplitW), 256, 0, s>>>(a, kBtSplitW);
    k_bt_wsum<<<dim3((unsigned)(((long)kBtNb * n + 255) / 256), nb), 256, 0, s>>>(a);
    k_bt_gemm<BT_APPLY_Z><<<dim3(nt, (m + kTM - 1) / kTM, nb), 256, 0, s>>>(a, 1);
  }
  return hipGetLastError();
}

}  // namespace slrx
