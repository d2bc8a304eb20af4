// Induced vector potential (App. D): the zero-padded FFT correlation and the
// separable, eigen-truncated kernel; the magnetic moment of Sec. V.A
// (Eq. magnetic_moment_def).
//
// Eigen-truncated: with G = V Lambda V^T kept to N* modes, A = -kappa^-2 sum_k lambda_k
// T_k J' T_k, where T_k[a][b] = V_k[|a - b|] is a symmetric Toeplitz
// matrix.  Two FP64 MFMA contractions per component:
//   Y_k = J' T_k        (one N x N x N product per mode; T_k generated from V_k),
//   A   = s sum_k lambda_k T_k Y_k   (one N x (N* N) x N product; lambda_k T_k
//                        generated from V_k, Y stacked mode by mode).
// The Toeplitz operands are formed from the N-vector of each mode as they
// are loaded, so no N x N x N* table is stored.
#include <algorithm>

#include "kernels.hpp"
#include "sweep.hpp"

namespace qc {

typedef double v4d __attribute__((ext_vector_type(4)));

// MFMA f64 16x16x4 operands: lane l holds A[l % 16][l / 16] and
// B[l / 16][l % 16]; the result D[l / 16 + 4 v][l % 16] in element v of its
// four accumulators (checked on the device).  The contraction index runs in
// chunks of 16: step s of a chunk takes its indices 4 (l / 16) + s.
//   MODE 1: C = Y[c][k] (N x N), A = J'[c] (row-major), B[a][b] = V[k][|a - b|];
//           a wave per 16 x 32 tile, blockIdx.z = c * nmodes + k.
//   MODE 2: C = A_out[c], A[r][(k, a)] = lambda_k V[k][|r - a|],
//           B = Y[c] as an (N* N) x N row-major matrix; a block per 32 x 16
//           tile, its waves share the contraction, blockIdx.z = c.
// The Toeplitz operand of the tile's second half is that of its first half one
// chunk before, so a chunk costs four loads of it and four of the dense
// operand for eight MFMAs (512 cycles): both go to registers, one chunk
// ahead, with no LDS and no barrier.  Bound by the matrix cores' FP64 rate and
// the shortage of tiles.  A wave per 32 x 32 tile with the whole contraction
// and staging through LDS took 49 + 242 us on 200 x 200 with 5 modes (98 waves
// on 1024 SIMDs in the second product); 15 + 11 us now (5 us at the rate a
// large FP64 product reaches).
constexpr int kEigWaves1 = 4, kEigWaves2 = 8;
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));
template <int MODE>
__global__ void __launch_bounds__(64 * (MODE == 1 ? kEigWaves1 : kEigWaves2))
    eig_gemm_kernel(int n, int nmodes, const double* __restrict__ jp, const double* __restrict__ vk,
                    const double* __restrict__ lam, double* __restrict__ y, double* __restrict__ aout, double alpha) {
  const int l = threadIdx.x & 63, m = l & 15, g = l >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
  const int z = blockIdx.z;
  const int64_t nn = static_cast<int64_t>(n) * n;
  const int r0 = MODE == 1 ? (static_cast<int>(blockIdx.y) * kEigWaves1 + wv) * 16 : static_cast<int>(blockIdx.y) * 32;
  const int c0 = static_cast<int>(blockIdx.x) * (MODE == 1 ? 32 : 16);
  if (MODE == 1 && r0 >= n) return;  // (no barrier in this product)
  // Toeplitz tile origin and the dense operand's fixed index (clamped: what
  // lies outside is not stored)
  const int t0 = (MODE == 1 ? c0 : r0) + m;
  const int fixed = min(MODE == 1 ? r0 + m : c0 + m, n - 1);
  // the wave's chunks [q0, q1) of the contraction
  const int per = (n + 15) / 16;
  const int64_t total = MODE == 1 ? per : static_cast<int64_t>(per) * nmodes;
  const int64_t q0 = MODE == 1 ? 0 : total * wv / kEigWaves2, q1 = MODE == 1 ? total : total * (wv + 1) / kEigWaves2;
  v4d acc[2] = {v4d{0.0, 0.0, 0.0, 0.0}, v4d{0.0, 0.0, 0.0, 0.0}};
  for (int64_t q = q0; q < q1;) {
    const int k = MODE == 1 ? z % nmodes : static_cast<int>(q / per);
    const int b0 = MODE == 1 ? 0 : static_cast<int>(q - static_cast<int64_t>(k) * per);
    const int b1 = static_cast<int>(min(static_cast<int64_t>(per), b0 + (q1 - q)));
    q += b1 - b0;
    const double* const v = vk + static_cast<int64_t>(k) * n;
    const double scale = MODE == 1 ? 1.0 : lam[k];
    const double* const dense = MODE == 1 ? jp + (z / nmodes) * nn + static_cast<int64_t>(fixed) * n
                                          : y + (static_cast<int64_t>(z) * nmodes + k) * nn + fixed;
    auto toeplitz = [&](int b, double* t) {
      for (int s = 0; s < 4; ++s) t[s] = scale * v[min(abs(16 * b + 4 * g + s - t0), n - 1)];
    };
    auto load = [&](int b, double* d) {
      const int a = 16 * b + 4 * g;
      if (16 * b + 16 <= n) {
        if (MODE == 1) {
          const d2u lo = *reinterpret_cast<const d2u*>(dense + a), hi = *reinterpret_cast<const d2u*>(dense + a + 2);
          d[0] = lo.x;
          d[1] = lo.y;
          d[2] = hi.x;
          d[3] = hi.y;
        } else {
          for (int s = 0; s < 4; ++s) d[s] = dense[static_cast<int64_t>(a + s) * n];
        }
      } else {  // the last chunk: zero beyond n
        for (int s = 0; s < 4; ++s) {
          const int e = min(a + s, n - 1);
          const double x = dense[MODE == 1 ? e : static_cast<int64_t>(e) * n];
          d[s] = a + s < n ? x : 0.0;
        }
      }
    };
    double tp[4], tc[4], d[4];
    toeplitz(b0 - 1, tp);
    toeplitz(b0, tc);
    load(b0, d);
    for (int b = b0; b < b1; ++b) {
      double tn[4], dn[4];
      const int nb = min(b + 1, b1 - 1);
      toeplitz(nb, tn);
      load(nb, dn);
      for (int s = 0; s < 4; ++s) {
        if (MODE == 1) {
          acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(d[s], tc[s], acc[0], 0, 0, 0);
          acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(d[s], tp[s], acc[1], 0, 0, 0);
        } else {
          acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(tc[s], d[s], acc[0], 0, 0, 0);
          acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(tp[s], d[s], acc[1], 0, 0, 0);
        }
      }
      for (int s = 0; s < 4; ++s) {
        tp[s] = tc[s];
        tc[s] = tn[s];
        d[s] = dn[s];
      }
    }
  }
  if (MODE == 1) {
    double* const out = y + static_cast<int64_t>(z) * nn;
    for (int j = 0; j < 2; ++j)
      for (int e = 0; e < 4; ++e) {
        const int r = r0 + g + 4 * e, c = c0 + 16 * j + m;
        if (r < n && c < n) out[static_cast<int64_t>(r) * n + c] = acc[j][e];
      }
  } else {
    __shared__ double part[kEigWaves2][8][64];
    for (int e = 0; e < 8; ++e) part[wv][e][l] = acc[e >> 2][e & 3];
    __syncthreads();
    // thread (wv, l) sums element wv of lane l over the waves
    double sum = 0.0;
    for (int w = 0; w < kEigWaves2; ++w) sum += part[w][wv][l];
    const int r = r0 + 16 * (wv >> 2) + g + 4 * (wv & 3), c = c0 + m;
    if (r < n && c < n) aout[z * nn + static_cast<int64_t>(r) * n + c] = alpha * sum;
  }
}
static_assert(kEigWaves2 == 8, "a thread of the second product sums one of a lane's eight elements");

// sum of component c's partials over a wave, in an order of its own
__device__ __forceinline__ double sum_parts(const double* part, int nparts, int c, int l) {
  double v = 0.0;
  for (int i = l; i < nparts; i += 64) v += part[c * nparts + i];
  return group_sum(v, 64);
}

// j' = (j - grain mean) on grain cells, zero elsewhere, both components; the
// means from the block partials of the two sums (each block forms them: a
// launch less)
__global__ void __launch_bounds__(256) masked_current_kernel(const double* __restrict__ j,
                                                             const uint8_t* __restrict__ mask, int64_t ncell,
                                                             const double* __restrict__ part, int nparts,
                                                             double inv_n, double* __restrict__ jp) {
  __shared__ double mean[2];
  if (threadIdx.x < 128) {
    const int c = threadIdx.x >> 6, l = threadIdx.x & 63;
    const double v = sum_parts(part, nparts, c, l);
    if (l == 0) mean[c] = v * inv_n;
  }
  __syncthreads();
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= ncell) return;
  const bool in = mask[i] != 0;
  jp[i] = in ? j[i] - mean[0] : 0.0;
  jp[ncell + i] = in ? j[ncell + i] - mean[1] : 0.0;
}

// (x - cx) j_y - (y - cy) j_x at every grain cell (grain-cell order)
__global__ void __launch_bounds__(256) torque_kernel(const double* __restrict__ j,
                                                     const int32_t* __restrict__ grain_cells, int64_t ncg,
                                                     int64_t ncell, int nx, double x0, double y0, double h,
                                                     double cx, double cy, double* __restrict__ out) {
  const int64_t c = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (c >= ncg) return;
  const int cell = grain_cells[c];
  const double x = x0 + ((cell % nx) + 0.5) * h - cx, y = y0 + ((cell / nx) + 0.5) * h - cy;
  out[c] = x * j[ncell + cell] - y * j[cell];
}

static inline unsigned nb256(int64_t n) { return static_cast<unsigned>((n + 255) / 256); }

void launch_eig_vecpot(int n, int nmodes, const double* jp, const double* vk, const double* lam, double* y,
                       double* aout, double alpha, hipStream_t st) {
  const unsigned t16 = static_cast<unsigned>((n + 15) / 16), t32 = static_cast<unsigned>((n + 31) / 32);
  hipLaunchKernelGGL(eig_gemm_kernel<1>, dim3(t32, (t16 + kEigWaves1 - 1) / kEigWaves1, 2 * nmodes),
                     dim3(64 * kEigWaves1), 0, st, n, nmodes, jp, vk, lam, y, aout, 1.0);
  hipLaunchKernelGGL(eig_gemm_kernel<2>, dim3(t16, t32, 2), dim3(64 * kEigWaves2), 0, st, n, nmodes, jp, vk, lam, y,
                     aout, alpha);
}
void launch_masked_current(const double* j, const uint8_t* mask, int64_t ncell, const double* part, int nparts,
                           double inv_n, double* jp, hipStream_t st) {
  if (ncell > 0)
    hipLaunchKernelGGL(masked_current_kernel, dim3(nb256(ncell)), dim3(256), 0, st, j, mask, ncell, part, nparts, inv_n,
                       jp);
}
void launch_torque(const double* j, const int32_t* grain_cells, int64_t ncg, int64_t ncell, int nx, double x0,
                   double y0, double h, double cx, double cy, double* out, hipStream_t st) {
  if (ncg > 0)
    hipLaunchKernelGGL(torque_kernel, dim3(nb256(ncg)), dim3(256), 0, st, j, grain_cells, ncg, ncell, nx, x0, y0, h,
                       cx, cy, out);
}

// --------------------------------------------------------------------------
// FFT A-solve (App. D): zero-padded correlation of the current with the
// cell-averaged Green's function, the two components as one complex field.
//
// Three launches: rows forward, columns (forward, product, inverse), rows
// inverse.  Lengths are R 2^k (R = 1, 3 or 5).  A transform is one radix-R
// pass and radix-4 passes in LDS (a radix-2 pass where k is odd), decimation
// in frequency forward and in time backward, so the transformed data stay in
// the order the forward passes leave them in: the kernel's transform is
// tabulated through the same passes, and neither a bit reversal nor a
// transpose runs.  Only the ny rows that hold current (and the ny that are
// kept) exist in memory; the rest of the padding is zeros in LDS.  The column
// pass takes C columns at a time, C * 16 B contiguous per row.  Bound: the
// LDS exchange of the passes (each moves every element out and in) and, at
// small grids, launch and load latency.  Measured against padding, four row
// transforms, two transposes and unpadding as launches of their own, with
// power-of-two lengths: 512 x 512 cells 73 -> 47 us, 600 x 600 197 -> 60 us,
// 200 x 200 41 -> 27 us, 40 x 40 41 -> 23 us per solve.
// --------------------------------------------------------------------------
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
// a w, or a conj(w) when BACK
template <bool BACK>
__device__ __forceinline__ double2 ctw(double2 a, double2 w) {
  return BACK ? make_double2(a.x * w.x + a.y * w.y, a.y * w.x - a.x * w.y)
              : make_double2(a.x * w.x - a.y * w.y, a.x * w.y + a.y * w.x);
}
// -i a forward, i a back
template <bool BACK>
__device__ __forceinline__ double2 crot(double2 a) {
  return BACK ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}
// y_q = sum_m x_m exp(-+ 2 pi i m q / 3 or 5)
template <bool BACK>
__device__ __forceinline__ void dft3(double2* x) {
  const double s = 0.86602540378443864676;  // sin(2 pi / 3)
  const double2 t = cadd(x[1], x[2]), d = csub(x[1], x[2]);
  const double2 m = make_double2(x[0].x - 0.5 * t.x, x[0].y - 0.5 * t.y);
  const double2 r = crot<BACK>(make_double2(s * d.x, s * d.y));
  x[0] = cadd(x[0], t);
  x[1] = cadd(m, r);
  x[2] = csub(m, r);
}
template <bool BACK>
__device__ __forceinline__ void dft5(double2* x) {
  const double c1 = 0.30901699437494742410, s1 = 0.95105651629515357212;   // cos, sin of 2 pi / 5
  const double c2 = -0.80901699437494742410, s2 = 0.58778525229247312917;  // of 4 pi / 5
  const double2 t1 = cadd(x[1], x[4]), d1 = csub(x[1], x[4]), t2 = cadd(x[2], x[3]), d2 = csub(x[2], x[3]);
  const double2 m1 = make_double2(x[0].x + c1 * t1.x + c2 * t2.x, x[0].y + c1 * t1.y + c2 * t2.y);
  const double2 m2 = make_double2(x[0].x + c2 * t1.x + c1 * t2.x, x[0].y + c2 * t1.y + c1 * t2.y);
  const double2 r1 = crot<BACK>(make_double2(s1 * d1.x + s2 * d2.x, s1 * d1.y + s2 * d2.y));
  const double2 r2 = crot<BACK>(make_double2(s2 * d1.x - s1 * d2.x, s2 * d1.y - s1 * d2.y));
  x[0] = cadd(x[0], cadd(t1, t2));
  x[1] = cadd(m1, r1);
  x[4] = csub(m1, r1);
  x[2] = cadd(m2, r2);
  x[3] = csub(m2, r2);
}

// Place of element i of a sequence in LDS: the 2^k blocks one after the
// other, and inside a block lanes that touch elements 1, 4 or 16 apart land
// on different banks (16 B elements, 16 of them per 256 B of banks).
__device__ __forceinline__ int fft_at(int i, int k) {
  const int low = i & ((1 << k) - 1);
  return (i - low) + (low ^ (((low >> 4) & 3) * 5));
}

// The radix-R pass over `count` sequences of length n = R 2^k (nothing for
// R = 1): forward before the power-of-two passes, back after them
template <bool BACK, int R>
__device__ __forceinline__ void fft_pass_r(double2* buf, int count, int k, const double2* tw) {
  const int K = 1 << k, n = R << k;
  for (int t = threadIdx.x; t < (count << k); t += blockDim.x) {
    const int r = t >> k, pos = t & (K - 1);
    double2* s = buf + r * n;
    double2 x[R];
    for (int m = 0; m < R; ++m) {
      x[m] = s[fft_at(pos + (m << k), k)];
      if (BACK && m > 0) x[m] = ctw<true>(x[m], tw[m * pos]);
    }
    if (R == 3)
      dft3<BACK>(x);
    else
      dft5<BACK>(x);
    for (int m = 0; m < R; ++m) {
      if (!BACK && m > 0) x[m] = ctw<false>(x[m], tw[m * pos]);
      s[fft_at(pos + (m << k), k)] = x[m];
    }
  }
  __syncthreads();
}

// A radix-4 pass on blocks of 4 h = 2^(LH+2) elements inside every 2^k
// sequence (seqs of them, one after the other); LH is a constant, so that the
// LDS places reduce to a base and constant offsets.
template <bool BACK, int LH>
__device__ __forceinline__ void fft_pass4(double2* buf, int seqs, int k, int R, const double2* tw) {
  constexpr int h = 1 << LH;
  const int ws = k - LH - 2;
  for (int t = threadIdx.x; t < (seqs << (k - 2)); t += blockDim.x) {
    const int b = t & ((1 << (k - 2)) - 1);
    const int pos = b & (h - 1), g = b >> LH;
    double2* s = buf + ((t >> (k - 2)) << k);
    // places of i0 + m h, i0 = 4 h g + pos (see fft_at)
    int at[4];
    for (int m = 0; m < 4; ++m) {
      if (LH >= 6)
        at[m] = (((g << (LH + 2)) + pos) ^ (((pos >> 4) & 3) * 5)) + m * h;
      else if (LH == 4)
        at[m] = (g << 6) + 16 * m + (pos ^ (5 * m));
      else if (LH == 2)
        at[m] = (g << 4) + ((4 * m + pos) ^ ((g & 3) * 5));
      else
        at[m] = ((g << 2) ^ (((g >> 2) & 3) * 5)) ^ m;
    }
    const int w = (pos << ws) * R;
    double2 x0 = s[at[0]], x1 = s[at[1]], x2 = s[at[2]], x3 = s[at[3]];
    double2 w1 = make_double2(1.0, 0.0), w2 = w1, w3 = w1;
    if (LH > 0) {
      w1 = tw[w];
      w2 = tw[2 * w];
      w3 = tw[3 * w];
    }
    if (BACK && LH > 0) {
      x1 = ctw<true>(x1, w1);
      x2 = ctw<true>(x2, w2);
      x3 = ctw<true>(x3, w3);
    }
    const double2 a = cadd(x0, x2), e = csub(x0, x2), c = cadd(x1, x3), d = crot<BACK>(csub(x1, x3));
    x0 = cadd(a, c);
    x1 = cadd(e, d);
    x2 = csub(a, c);
    x3 = csub(e, d);
    if (!BACK && LH > 0) {
      x1 = ctw<false>(x1, w1);
      x2 = ctw<false>(x2, w2);
      x3 = ctw<false>(x3, w3);
    }
    s[at[0]] = x0;
    s[at[1]] = x1;
    s[at[2]] = x2;
    s[at[3]] = x3;
  }
  __syncthreads();
}
template <bool BACK>
__device__ __forceinline__ void fft_pass4_at(int lh, double2* buf, int seqs, int k, int R,
                                             const double2* tw) {
  switch (lh) {
    case 0: fft_pass4<BACK, 0>(buf, seqs, k, R, tw); break;
    case 2: fft_pass4<BACK, 2>(buf, seqs, k, R, tw); break;
    case 4: fft_pass4<BACK, 4>(buf, seqs, k, R, tw); break;
    case 6: fft_pass4<BACK, 6>(buf, seqs, k, R, tw); break;
    case 8: fft_pass4<BACK, 8>(buf, seqs, k, R, tw); break;
    default: fft_pass4<BACK, 10>(buf, seqs, k, R, tw); break;
  }
}
// the radix-2 pass over the halves of a 2^k sequence (odd k)
template <bool BACK>
__device__ __forceinline__ void fft_pass2(double2* buf, int seqs, int k, int R, const double2* tw) {
  const int h = 1 << (k - 1);
  for (int t = threadIdx.x; t < (seqs << (k - 1)); t += blockDim.x) {
    const int pos = t & (h - 1);
    double2* s = buf + ((t >> (k - 1)) << k);
    const double2 a = s[fft_at(pos, k)], v = s[fft_at(pos + h, k)], f = tw[pos * R];
    const double2 b = BACK ? ctw<true>(v, f) : v;
    s[fft_at(pos, k)] = cadd(a, b);
    s[fft_at(pos + h, k)] = BACK ? csub(a, b) : ctw<false>(csub(a, b), f);
  }
  __syncthreads();
}

// Forward transform (exp(-2 pi i jk/n)) of `count` sequences of n = R 2^k
// elements (R = 1, 3, 5; k <= 12), sequence r at buf + r n; tw[j] =
// exp(-2 pi i j / n), j < n, in LDS.  Every thread of the block takes part; buf
// is ready on entry and on exit.
__device__ __forceinline__ void fft_forward(double2* buf, int count, int k, int R, const double2* tw) {
  if (R == 3) fft_pass_r<false, 3>(buf, count, k, tw);
  if (R == 5) fft_pass_r<false, 5>(buf, count, k, tw);
  const int odd = k & 1;
  if (odd) fft_pass2<false>(buf, count * R, k, R, tw);
  for (int lh = k - odd - 2; lh >= 0; lh -= 2) fft_pass4_at<false>(lh, buf, count * R, k, R, tw);
}

// the passes of fft_forward undone one by one, last first: n times the
// inverse transform, from the order fft_forward leaves to natural order
__device__ __forceinline__ void fft_backward(double2* buf, int count, int k, int R, const double2* tw) {
  const int odd = k & 1;
  for (int lh = 0; lh <= k - odd - 2; lh += 2) fft_pass4_at<true>(lh, buf, count * R, k, R, tw);
  if (odd) fft_pass2<true>(buf, count * R, k, R, tw);
  if (R == 3) fft_pass_r<true, 3>(buf, count, k, tw);
  if (R == 5) fft_pass_r<true, 5>(buf, count, k, tw);
}

// The twiddle table of a length into LDS: read from memory pass by pass, each
// pass of a block waits for L2 anew (24 x 900 cells: 47 us per solve, 37 with
// the table in LDS)
__device__ __forceinline__ void load_twiddles(double2* tws, int n, const double2* __restrict__ tw) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) tws[i] = tw[i];
}

// Rows forward.  The input is the current of the grain cells minus its grain
// mean (from the block partials of the two sums), zero elsewhere; a block of
// 256 takes rpb rows.  LDS: the rows, then the twiddles.  pitch: elements
// from row to row of w (more than px: with the power of two alone a column's
// elements meet in one memory channel).
__global__ void __launch_bounds__(256) vecpot_rows_kernel(const double* __restrict__ j, const uint8_t* __restrict__ mask,
                                                          int nx, int ny, FftLen lx, int pitch, int rpb,
                                                          const double* __restrict__ part, int nparts, double inv_n,
                                                          const double2* __restrict__ tw, double2* __restrict__ w) {
  extern __shared__ double2 buf[];
  __shared__ double mean[2];
  const int px = lx.n(), y0 = blockIdx.x * rpb, rows = min(rpb, ny - y0);
  const int64_t ncell = static_cast<int64_t>(nx) * ny, c0 = static_cast<int64_t>(y0) * nx;
  double2* tws = buf + rpb * px;
  load_twiddles(tws, px, tw);
  // the masked current first, its mean off it afterwards: the loads of both
  // overlap
  for (int t = threadIdx.x; t < rpb * px; t += blockDim.x) buf[t] = make_double2(0.0, 0.0);
  if (threadIdx.x < 128) {
    const int c = threadIdx.x >> 6, l = threadIdx.x & 63;
    const double v = sum_parts(part, nparts, c, l);
    if (l == 0) mean[c] = v * inv_n;
  }
  // (up to kHold elements per thread held over the barrier; the rest after it)
  constexpr int kHold = 4;
  double2 hold[kHold];
  bool in[kHold];
  for (int q = 0; q < kHold; ++q) {
    const int t = threadIdx.x + q * 256;
    in[q] = t < rows * nx && mask[c0 + t];
    if (t < rows * nx) hold[q] = make_double2(j[c0 + t], j[ncell + c0 + t]);
  }
  __syncthreads();
  auto put = [&](int t, double2 v) {
    const int r = t / nx, x = t - r * nx;
    buf[r * px + fft_at(x, lx.k)] = make_double2(v.x - mean[0], v.y - mean[1]);
  };
  for (int q = 0; q < kHold; ++q)
    if (in[q]) put(threadIdx.x + q * 256, hold[q]);
  for (int t = threadIdx.x + kHold * 256; t < rows * nx; t += 256)
    if (mask[c0 + t]) put(t, make_double2(j[c0 + t], j[ncell + c0 + t]));
  __syncthreads();
  fft_forward(buf, rpb, lx.k, lx.r, tws);
  for (int r = 0; r < rows; ++r)
    for (int x = threadIdx.x; x < px; x += blockDim.x)
      w[static_cast<int64_t>(y0 + r) * pitch + x] = buf[r * px + fft_at(x, lx.k)];
}

// Columns, C = 2^lc of them per block: forward, times the transform of the
// kernel, back; rows >= ny are zero on the way in and dropped on the way out.
// TABLE: the rows hold the kernel itself; its transform (real, since the
// kernel is even in both directions) goes to ghat[column][place].
// A block has one thread per four elements; blocks of neighbouring columns
// run on one XCD, whose L2 then holds the lines they share.
template <bool TABLE>
__global__ void __launch_bounds__(1024) vecpot_cols_kernel(double2* __restrict__ w, int ny, int pitch, FftLen ly, int lc,
                                                           const double2* __restrict__ tw, double* __restrict__ ghat) {
  extern __shared__ double2 buf[];
  const int py = ly.n(), C = 1 << lc;
  const int64_t x0 = xcd_block(blockIdx.x, gridDim.x) << lc;
  double2* tws = buf + (py << lc);
  load_twiddles(tws, py, tw);
  // the kernel's transform is loaded here, so that the product does not wait
  constexpr int kHold = 5;
  double gh[kHold];
  for (int q = 0; q < kHold; ++q) {
    const int t = threadIdx.x + q * blockDim.x;
    if (!TABLE && t < (py << lc)) gh[q] = ghat[x0 * py + t];
  }
  for (int t = threadIdx.x; t < (py << lc); t += blockDim.x) {
    const int c = t & (C - 1), y = t >> lc;
    buf[c * py + fft_at(y, ly.k)] = y < ny ? w[static_cast<int64_t>(y) * pitch + x0 + c] : make_double2(0.0, 0.0);
  }
  __syncthreads();
  fft_forward(buf, C, ly.k, ly.r, tws);
  // (the columns of buf follow each other, so element t of the block is place
  // t of ghat's columns)
  auto times = [&](int t, double g) {
    double2& v = buf[fft_at(t, ly.k)];
    v = make_double2(g * v.x, g * v.y);
  };
  if (TABLE) {
    for (int t = threadIdx.x; t < (py << lc); t += blockDim.x) ghat[x0 * py + t] = buf[fft_at(t, ly.k)].x;
    return;
  }
  for (int q = 0; q < kHold; ++q) {
    const int t = threadIdx.x + q * blockDim.x;
    if (t < (py << lc)) times(t, gh[q]);
  }
  for (int t = threadIdx.x + kHold * blockDim.x; t < (py << lc); t += blockDim.x) times(t, ghat[x0 * py + t]);
  __syncthreads();
  fft_backward(buf, C, ly.k, ly.r, tws);
  for (int t = threadIdx.x; t < (ny << lc); t += blockDim.x) {
    const int c = t & (C - 1), y = t >> lc;
    w[static_cast<int64_t>(y) * pitch + x0 + c] = buf[c * py + fft_at(y, ly.k)];
  }
}

// Rows backward: the nx values kept of each row, scaled, to A
__global__ void __launch_bounds__(256) vecpot_rows_back_kernel(const double2* __restrict__ w, int nx, int ny, FftLen lx,
                                                               int pitch, int rpb, const double2* __restrict__ tw,
                                                               double scale, double* __restrict__ A) {
  extern __shared__ double2 buf[];
  const int px = lx.n(), y0 = blockIdx.x * rpb, rows = min(rpb, ny - y0);
  double2* tws = buf + rpb * px;
  load_twiddles(tws, px, tw);
  for (int r = 0; r < rows; ++r)
    for (int x = threadIdx.x; x < px; x += blockDim.x)
      buf[r * px + fft_at(x, lx.k)] = w[static_cast<int64_t>(y0 + r) * pitch + x];
  __syncthreads();
  fft_backward(buf, rows, lx.k, lx.r, tws);
  const int64_t ncell = static_cast<int64_t>(nx) * ny, c0 = static_cast<int64_t>(y0) * nx;
  for (int r = 0; r < rows; ++r)
    for (int x = threadIdx.x; x < nx; x += blockDim.x) {
      const double2 v = buf[r * px + fft_at(x, lx.k)];
      A[c0 + r * nx + x] = scale * v.x;
      A[ncell + c0 + r * nx + x] = scale * v.y;
    }
}

// rows of the kernel itself, for the table: all py of them
__global__ void __launch_bounds__(256) vecpot_kernel_rows_kernel(const double* __restrict__ g, FftLen lx, int pitch,
                                                                 const double2* __restrict__ tw,
                                                                 double2* __restrict__ w) {
  extern __shared__ double2 buf[];
  const int px = lx.n();
  double2* tws = buf + px;
  load_twiddles(tws, px, tw);
  for (int x = threadIdx.x; x < px; x += blockDim.x)
    buf[fft_at(x, lx.k)] = make_double2(g[static_cast<int64_t>(blockIdx.x) * px + x], 0.0);
  __syncthreads();
  fft_forward(buf, 1, lx.k, lx.r, tws);
  for (int x = threadIdx.x; x < px; x += blockDim.x)
    w[static_cast<int64_t>(blockIdx.x) * pitch + x] = buf[fft_at(x, lx.k)];
}

// The smallest length of at least m of the forms 2^k, 3 2^k and 5 2^k (the
// last two from k = 4 on, where the LDS order keeps inside a block): padding
// to the next power of two makes 2.6 times the area at 600 x 600 cells (2048
// for 1200, here 1280; 114 us per solve against 61)
FftLen fft_length(int m) {
  FftLen best{1, 0};
  while (best.n() < m) ++best.k;
  for (int r : {3, 5})
    for (int k = 4; k < 12; ++k) {
      const FftLen c{r, k};
      if (c.n() >= m && c.n() < best.n()) best = c;
    }
  return best;
}

// elements from row to row of the work array
static int fft_pitch(FftLen lx) { return lx.n() + 8; }
int64_t vecpot_work_elems(FftLen lx, FftLen ly) { return static_cast<int64_t>(fft_pitch(lx)) * ly.n(); }
// rows per block (about 1024 elements, at least one row)
static int fft_rpb(FftLen lx) { return lx.n() >= 1024 ? 1 : 1024 / lx.n(); }
// log2 of the columns per block: four (64 B of every row), fewer where they
// would take more than 3072 elements of LDS beside the twiddles (64 KB in all
// up to lengths of 1024) or the row is shorter
static int fft_lc(FftLen ly, FftLen lx) {
  int lc = 0;
  while (lc < 2 && (ly.n() << (lc + 1)) <= 3072 && lx.n() % (2 << lc) == 0) ++lc;
  return lc;
}
static dim3 fft_cols_block(FftLen ly, int lc) {
  return dim3(static_cast<unsigned>(std::min(std::max(((ly.n() << lc) / 4 + 63) / 64 * 64, 64), 1024)));
}
static size_t fft_lds(int elems, int tw) { return sizeof(double2) * static_cast<size_t>(elems + tw); }
// A kernel has to ask for more than 64 KB of LDS, dynamic and static together
// (the rows forward hold their two means beside the rows): rows from length
// 2048 on, columns beyond it.  The limit belongs to the function, not to the
// grain, so every grain that needs one asks for the largest that any length
// needs (4096: one sequence and its twiddles), and none lowers another's.
constexpr size_t kFftLdsMax = sizeof(double2) * 2 * 4096;
hipError_t vecpot_prepare(FftLen lx, FftLen ly) {
  const int px = lx.n(), py = ly.n();
  hipError_t e = hipSuccess;
  auto ask = [&](const void* f, size_t dynamic, size_t fixed) {
    if (dynamic > kFftLdsMax) e = hipErrorInvalidValue;
    if (e == hipSuccess && dynamic + fixed > 65536)
      e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(kFftLdsMax));
  };
  const size_t rows = fft_lds(fft_rpb(lx) * px, px), cols = fft_lds(py << fft_lc(ly, lx), py);
  ask(reinterpret_cast<const void*>(vecpot_rows_kernel), rows, 2 * sizeof(double));
  ask(reinterpret_cast<const void*>(vecpot_rows_back_kernel), rows, 0);
  ask(reinterpret_cast<const void*>(vecpot_kernel_rows_kernel), fft_lds(px, px), 0);
  ask(reinterpret_cast<const void*>(vecpot_cols_kernel<true>), cols, 0);
  ask(reinterpret_cast<const void*>(vecpot_cols_kernel<false>), cols, 0);
  return e;
}

void launch_vecpot_table(const double* g, FftLen lx, FftLen ly, const double2* twx, const double2* twy, double2* w,
                         double* ghat, hipStream_t st) {
  const int px = lx.n(), py = ly.n(), lc = fft_lc(ly, lx);
  hipLaunchKernelGGL(vecpot_kernel_rows_kernel, dim3(py), dim3(256), fft_lds(px, px), st, g, lx, fft_pitch(lx), twx, w);
  hipLaunchKernelGGL(vecpot_cols_kernel<true>, dim3(px >> lc), fft_cols_block(ly, lc), fft_lds(py << lc, py), st, w, py,
                     fft_pitch(lx), ly, lc, twy, ghat);
}
void launch_vecpot_fft(const double* j, const uint8_t* mask, int nx, int ny, FftLen lx, FftLen ly, const double* part,
                       int nparts, double inv_n, const double2* twx, const double2* twy, double2* w, double* ghat,
                       double scale, double* A, hipStream_t st) {
  const int px = lx.n(), py = ly.n(), rpb = fft_rpb(lx), lc = fft_lc(ly, lx), pitch = fft_pitch(lx);
  const unsigned rows = static_cast<unsigned>((ny + rpb - 1) / rpb);
  hipLaunchKernelGGL(vecpot_rows_kernel, dim3(rows), dim3(256), fft_lds(rpb * px, px), st, j, mask, nx, ny, lx, pitch,
                     rpb, part, nparts, inv_n, twx, w);
  hipLaunchKernelGGL(vecpot_cols_kernel<false>, dim3(px >> lc), fft_cols_block(ly, lc), fft_lds(py << lc, py), st, w, ny,
                     pitch, ly, lc, twy, ghat);
  hipLaunchKernelGGL(vecpot_rows_back_kernel, dim3(rows), dim3(256), fft_lds(rpb * px, px), st, w, nx, ny, lx, pitch,
                     rpb, twx, scale, A);
}

}  // namespace qc
