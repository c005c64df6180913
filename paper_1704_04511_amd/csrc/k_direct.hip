// IRLS-direct (SLRX_FLAG_DIRECT): the method without the FFT-based
// approximations, which the paper compares with (Sec. IV, Fig. 2).  The lifting
// is linear in all three dimensions: k-space in centred order (DC at
// (P/2, Q/2)), rows (n, w) for n = M-1..T-1 and the valid shifts w (the
// N1 x N2 support w - a inside the grid, (P-N1+1)(Q-N2+1) of them), columns
// (m, a) with a the filter offsets in row-major order; entry xc[n-m][w-a].
// Both sub-problems run on the explicit matrix:
//   * R = X^H X with X the lifted matrix of the iterate, on FP64 MFMA with the
//     entries gathered from the iterate as they are multiplied (k_dgram), then the
//     library's own eigen-decomposition chain;
//   * the least-squares operator A v = S o v + lam T^*(T(v) H): T(v) gathered
//     in complex64, times H (a plain library GEMM), and the adjoint T^* as a
//     gather per k-space sample (every entry of T(v) H that was read from that
//     sample, in a fixed order, accumulated in FP64), fused with S o v and the CG
//     dot product.
// T(v) and T(v) H are stored column by column (ld = rows): consecutive rows are
// consecutive k-space samples of one shift, so both gathers are coalesced.  With
// row-major matrices the adjoint's reads were a row (8 s bytes) apart: 35.4 against
// 24.5 us at 64 x 64 x 8 with 5 x 5 x 3 (21600 x 75), the lifting 12.2 against 9.9 us.
// This file holds the gathers and the CG glue; the operator's GEMM is a rocBLAS call.
#include <hip/hip_runtime.h>

#include "common.h"
#include "kernels.h"

namespace slrx {
namespace {

constexpr int kDirNT = 256;

// Column j of the lifted matrix: the frame offset and the k-space shifts it reads, in
// DFT order (to be wrapped once, w + o < 2 P).
struct LiftCol {
  int m, o1, o2;
};
SLRX_DEV LiftCol lift_col(const DirectArgs& a, int j) {
  const int NN = a.N1 * a.N2;
  const int m = j / NN, ia = j - m * NN;
  const int a1 = ia / a.N2 + a.a1min, a2 = ia % a.N2 + a.a2min;
  return LiftCol{m, a.a1max - a1 + a.P / 2, a.a2max - a2 + a.Q / 2};
}
// Row r of the lifted matrix: echo shift n and the valid shifts (w1, w2), row-major.
struct LiftRow {
  int n, w1, w2;
};
SLRX_DEV LiftRow lift_row(const DirectArgs& a, int r) {
  const int rq = r / a.nw2;
  const int n = rq / a.nw1;
  return LiftRow{n + a.M - 1, rq - n * a.nw1, r - rq * a.nw2};
}
SLRX_DEV int lift_src(const DirectArgs& a, const LiftRow& r, const LiftCol& c) {
  int k1 = r.w1 + c.o1, k2 = r.w2 + c.o2;
  if (k1 >= a.P) k1 -= a.P;
  if (k2 >= a.Q) k2 -= a.Q;
  return ((r.n - c.m) * a.P + k1) * a.Q + k2;
}

// X = T(x), column j at j * rows; block (x: rows, y: columns).
constexpr int kLiftCols = 8;  // columns per thread
__global__ __launch_bounds__(kDirNT) void k_dlift(DirectArgs a, const float2* __restrict__ x, float2* __restrict__ X) {
  const int s = a.N1 * a.N2 * a.M;
  const long r = (long)blockIdx.x * kDirNT + threadIdx.x;
  if (r >= a.rows) return;
  const LiftRow lr = lift_row(a, (int)r);
  const int j0 = blockIdx.y * kLiftCols;
#pragma unroll
  for (int u = 0; u < kLiftCols; ++u)
    if (j0 + u < s) X[(long)(j0 + u) * a.rows + r] = x[lift_src(a, lr, lift_col(a, j0 + u))];
}

// R = X^H X of the lifting X (rows x s) in FP64: 64 x 64 tiles on or above the
// diagonal, the rows split over nsplit workgroups per tile so that the chip is filled
// whatever s is; the tile's partial sums are added in split order by k_dgram_sum.
// X is never stored: a chunk of 16 rows of the tile's columns is gathered from the
// iterate (L2 resident, 16 consecutive samples per column) into registers while the
// chunk before it is multiplied from LDS.  Four waves of 32 x 32, f64 16x16x4 MFMA,
// which bounds it: 8 * 64^2 flop per row and tile, 2.1 GFlop at 21600 x 75.  The
// library's zgemm ran that shape in four workgroups: 2336 us, against 57 us here
// and 8 us for the sum of the partials.
constexpr int kGrTB = 64, kGrKC = 16;
typedef double v4d __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void k_dgram(DirectArgs a, const float2* __restrict__ x, double2* __restrict__ part,
                                               int nsplit, int per) {
  __shared__ double Lar[kGrKC][kGrTB + 1], Lai[kGrKC][kGrTB + 1], Lbr[kGrKC][kGrTB + 1], Lbi[kGrKC][kGrTB + 1];
  const int s = a.N1 * a.N2 * a.M, nt = (s + kGrTB - 1) / kGrTB;
  const int tile = blockIdx.x / nsplit, split = blockIdx.x % nsplit;
  int bi = 0, rem = tile;
  while (rem >= nt - bi) {
    rem -= nt - bi;
    ++bi;
  }
  const int i0 = bi * kGrTB, j0 = (bi + rem) * kGrTB;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wi = (wave >> 1) * 32, wj = (wave & 1) * 32;
  const int kk = tid & (kGrKC - 1), c0 = tid / kGrKC;  // this thread's row of a chunk, its columns c0 + 16 u
  constexpr int U = kGrTB / (256 / kGrKC);
  LiftCol ca[U], cb[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    ca[u] = lift_col(a, min(i0 + c0 + 16 * u, s - 1));  // columns beyond s only feed entries that are not used
    cb[u] = lift_col(a, min(j0 + c0 + 16 * u, s - 1));
  }
  v4d accR[2][2], accI[2][2];
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int q = 0; q < 2; ++q) accR[p][q] = accI[p][q] = v4d{0.0, 0.0, 0.0, 0.0};
  const long r0 = (long)split * per;
  const int nr = (int)max(0L, min((long)per, a.rows - r0));
  float2 pa[U], pb[U];
  auto load = [&](int k) {
    const bool in = k + kk < nr;
    const LiftRow lr = lift_row(a, (int)(in ? r0 + k + kk : 0));
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float2 va = x[lift_src(a, lr, ca[u])], vb = x[lift_src(a, lr, cb[u])];
      pa[u] = in ? va : make_float2(0.f, 0.f);
      pb[u] = in ? vb : make_float2(0.f, 0.f);
    }
  };
  if (nr > 0) load(0);
  for (int k = 0; k < nr; k += kGrKC) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      Lar[kk][c0 + 16 * u] = pa[u].x;
      Lai[kk][c0 + 16 * u] = pa[u].y;
      Lbr[kk][c0 + 16 * u] = pb[u].x;
      Lbi[kk][c0 + 16 * u] = pb[u].y;
    }
    __syncthreads();
    if (k + kGrKC < nr) load(k + kGrKC);
#pragma unroll
    for (int kq = 0; kq < kGrKC; kq += 4) {
      const int kl = kq + (lane >> 4);
      double ar[2], ai[2], an[2], br[2], bm[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        ar[t] = Lar[kl][wi + 16 * t + (lane & 15)];
        ai[t] = Lai[kl][wi + 16 * t + (lane & 15)];
        an[t] = -ai[t];
        br[t] = Lbr[kl][wj + 16 * t + (lane & 15)];
        bm[t] = Lbi[kl][wj + 16 * t + (lane & 15)];
      }
      // conj(a) b = (ar br + ai bi) + i (ar bi - ai br)
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          accR[p][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[p], br[q], accR[p][q], 0, 0, 0);
          accI[p][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[p], bm[q], accI[p][q], 0, 0, 0);
          accR[p][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(ai[p], bm[q], accR[p][q], 0, 0, 0);
          accI[p][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(an[p], br[q], accI[p][q], 0, 0, 0);
        }
    }
    __syncthreads();
  }
  // item v of lane l is row l / 16 + 4 v, column l % 16
  double2* out = part + (long)blockIdx.x * (kGrTB * kGrTB);
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = wi + 16 * p + (lane >> 4) + 4 * v, j = wj + 16 * q + (lane & 15);
        out[i * kGrTB + j] = make_double2(accR[p][q][v], accI[p][q][v]);
      }
}

// The splits' partial tiles added in order, R row-major with both triangles; a
// non-finite entry raises the flag and is written as 0, as in k_gram_assemble.
__global__ __launch_bounds__(256) void k_dgram_sum(int s, const double2* __restrict__ part, int nsplit, double2* R,
                                                   int* bad) {
  const int nt = (s + kGrTB - 1) / kGrTB;
  const int tile = blockIdx.x / (kGrTB * kGrTB / 256), e = blockIdx.x % (kGrTB * kGrTB / 256) * 256 + threadIdx.x;
  int bi = 0, rem = tile;
  while (rem >= nt - bi) {
    rem -= nt - bi;
    ++bi;
  }
  const int i = bi * kGrTB + e / kGrTB, j = (bi + rem) * kGrTB + e % kGrTB;
  if (i > j || j >= s) return;
  const double2* p = part + (long)tile * nsplit * (kGrTB * kGrTB) + e;
  double2 v = make_double2(0.0, 0.0);
  int q = 0;
  for (; q + 8 <= nsplit; q += 8) {  // eight loads in flight
    double2 t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = p[(long)(q + u) * (kGrTB * kGrTB)];
#pragma unroll
    for (int u = 0; u < 8; ++u) v = dadd(v, t[u]);
  }
  for (; q < nsplit; ++q) v = dadd(v, p[(long)q * (kGrTB * kGrTB)]);
  if (i == j) v.y = 0.0;
  if (!isfinite(v.x) || !isfinite(v.y)) {
    *bad = 1;
    v = make_double2(0.0, 0.0);
  }
  R[(long)i * s + j] = v;
  if (i != j) R[(long)j * s + i] = dconj(v);
}

// out = S o v + lam T^*(Y) (init: out = y - that), partial dot products per block.
// One wave per block: a sample's up to s terms are a serial sum, so the samples are
// spread over as many CUs as there are (512 blocks at 64 x 64 x 8), and the taps are
// walked in their valid ranges with several loads in flight.
constexpr int kAdjNT = 64;
__global__ __launch_bounds__(kAdjNT) void k_dadj(DirectArgs a, const float2* __restrict__ Y,
                                                 const float2* __restrict__ v, const uint8_t* __restrict__ S,
                                                 const float2* __restrict__ y, float2* __restrict__ out, int init,
                                                 double* part, int* flag) {
  __shared__ double red[1];
  const int P = a.P, Q = a.Q, N1 = a.N1, N2 = a.N2;
  const int V = a.T * P * Q;
  double dot = 0.0;
  for (int g = (int)blockIdx.x * kAdjNT + threadIdx.x; g < V; g += (int)gridDim.x * kAdjNT) {
    const int gq = g / Q, k2 = g - gq * Q;
    const int f = gq / P, k1 = gq - f * P;
    const int c1 = k1 >= P / 2 ? k1 - P / 2 : k1 + P / 2, c2 = k2 >= Q / 2 ? k2 - Q / 2 : k2 + Q / 2;  // centred
    double ax = 0.0, ay = 0.0;
    // tap (u1, u2) reads row (c1 + u1 - (N1 - 1), c2 + u2 - (N2 - 1)) of the valid shifts
    const int u1a = max(0, N1 - 1 - c1), u1b = min(N1, P - c1);
    const int u2a = max(0, N2 - 1 - c2), u2b = min(N2, Q - c2);
    const int ma = max(0, a.M - 1 - f), mb = min(a.M, a.T - f);
    for (int m = ma; m < mb; ++m)
      for (int u1 = u1a; u1 < u1b; ++u1) {
        const long r = ((long)(f + m - a.M + 1) * a.nw1 + (c1 + u1 - (N1 - 1))) * a.nw2 + (c2 + u2a - (N2 - 1));
        const float2* q = Y + ((long)(m * N1 + u1) * N2 + u2a) * a.rows + r;
#pragma unroll 8
        for (int u2 = u2a; u2 < u2b; ++u2) {
          const float2 t = *q;
          ax += t.x;
          ay += t.y;
          q += a.rows + 1;
        }
      }
    const float2 vv = v[g];
    const float sv = S[g] ? 1.f : 0.f;
    float2 av = make_float2(sv * vv.x + (float)(a.lam * ax), sv * vv.y + (float)(a.lam * ay));
    if (init) {
      const float2 yv = y[g];
      av = make_float2(yv.x - av.x, yv.y - av.y);
      dot += (double)av.x * av.x + (double)av.y * av.y;
    } else {
      dot += (double)vv.x * av.x + (double)vv.y * av.y;
    }
    out[g] = av;
  }
  dot = block_sum<kAdjNT>(dot, red);
  if (threadIdx.x == 0) {
    part[blockIdx.x] = dot;
    if (init && blockIdx.x == 0) *flag = 0;
  }
}

// p = r + beta p, beta = rr_k / rr_{k-1} from the partials of rr_k (rr_hist[k] recorded).
__global__ __launch_bounds__(kDirNT) void k_dpupdate(long n, const float2* __restrict__ r, float2* __restrict__ p,
                                                     const double* part, int npart, double* rr_hist, int k) {
  __shared__ double red[kDirNT / 64];
  const double rr = reduce_partials<kDirNT>(part, npart, red);
  double beta = 0.0;
  if (k > 0) {
    const double prev = rr_hist[k - 1];
    beta = prev > 0.0 ? rr / prev : 0.0;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) rr_hist[k] = rr;
  const float fb = (float)beta;
  for (long i = (long)blockIdx.x * kDirNT + threadIdx.x; i < n; i += (long)gridDim.x * kDirNT) {
    const float2 rv = r[i];
    const float2 po = k > 0 ? p[i] : make_float2(0.f, 0.f);
    p[i] = make_float2(rv.x + fb * po.x, rv.y + fb * po.y);
  }
}

__global__ void k_hf(long n, const double* __restrict__ re, const double* __restrict__ im, float2* __restrict__ out) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = make_float2((float)re[i], (float)im[i]);
}

unsigned grid_for(long n, int nt = kDirNT) {
  const long b = (n + nt - 1) / nt;
  return (unsigned)(b < 1 ? 1 : (b > 1024 ? 1024 : b));
}

}  // namespace

DirectArgs direct_args(int P, int Q, int T, int N1, int N2, int M, double lam) {
  DirectArgs a{};
  a.P = P; a.Q = Q; a.T = T; a.N1 = N1; a.N2 = N2; a.M = M;
  a.a1min = -(N1 / 2);
  a.a2min = -(N2 / 2);
  a.a1max = N1 - 1 - N1 / 2;
  a.a2max = N2 - 1 - N2 / 2;
  a.nw1 = P - N1 + 1;
  a.nw2 = Q - N2 + 1;
  a.rows = (long)(T - M + 1) * a.nw1 * a.nw2;
  a.lam = lam;
  return a;
}

int direct_blocks(long V) { return (int)grid_for(V, kAdjNT); }

hipError_t launch_dlift32(const DirectArgs& a, const float2* x, float2* X, hipStream_t s) {
  const int cols = a.N1 * a.N2 * a.M;
  const dim3 grid((unsigned)((a.rows + kDirNT - 1) / kDirNT), (cols + kLiftCols - 1) / kLiftCols);
  k_dlift<<<grid, kDirNT, 0, s>>>(a, x, X);
  return hipGetLastError();
}

// Row splits per tile: about one workgroup per CU over all tiles (more would only add
// partial tiles of 64 KB to write and read back), each with at least 64 rows.
static int dgram_tiles(const DirectArgs& a) {
  const int nt = (a.N1 * a.N2 * a.M + kGrTB - 1) / kGrTB;
  return nt * (nt + 1) / 2;
}
static int dgram_splits(const DirectArgs& a) {
  const long by_chip = (256 + dgram_tiles(a) - 1) / dgram_tiles(a), by_rows = (a.rows + 63) / 64;
  const long n = by_chip < by_rows ? by_chip : by_rows;
  return (int)(n < 1 ? 1 : n);
}
size_t dgram_part_elems(const DirectArgs& a) { return (size_t)dgram_tiles(a) * dgram_splits(a) * kGrTB * kGrTB; }

hipError_t launch_dgram(const DirectArgs& a, const float2* x, double2* part, double2* R, int* bad, hipStream_t s) {
  const int tiles = dgram_tiles(a), nsplit = dgram_splits(a);
  // whole chunks per split, so that only the last split ends in a partial one
  const int per = (int)(((a.rows + nsplit - 1) / nsplit + kGrKC - 1) / kGrKC * kGrKC);
  k_dgram<<<tiles * nsplit, 256, 0, s>>>(a, x, part, nsplit, per);
  k_dgram_sum<<<tiles * (kGrTB * kGrTB / 256), 256, 0, s>>>(a.N1 * a.N2 * a.M, part, nsplit, R, bad);
  return hipGetLastError();
}

hipError_t launch_dadj(const DirectArgs& a, const float2* Y, const float2* v, const uint8_t* S, const float2* y,
                       float2* out, int init, double* part, int* flag, hipStream_t s) {
  const long V = (long)a.T * a.P * a.Q;
  k_dadj<<<grid_for(V, kAdjNT), kAdjNT, 0, s>>>(a, Y, v, S, y, out, init, part, flag);
  return hipGetLastError();
}

hipError_t launch_dpupdate(long n, const float2* r, float2* p, const double* part, int npart, double* rr_hist, int k,
                           hipStream_t s) {
  k_dpupdate<<<grid_for(n), kDirNT, 0, s>>>(n, r, p, part, npart, rr_hist, k);
  return hipGetLastError();
}

hipError_t launch_hf(long n, const double* re, const double* im, float2* out, hipStream_t s) {
  k_hf<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(n, re, im, out);
  return hipGetLastError();
}

}  // namespace slrx
