// Offline spectra of the scored weight matrices (fp64): the Gram matrix of the short side, a
// Householder reduction of that symmetric matrix to tridiagonal form and the largest eigenvalues
// of that form, the squared singular values the spectral concentration ratio needs.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace sgd {

// ---------------------------------------------------------------------------- Gram
// G[i][j] = sum_t E(t, i) E(t, j) with E(t, i) = X[t][i] (trans = 0) or X[i][t] (trans = 1), for
// every matrix of a batch in one launch.  64 x 64 output tiles on and below the diagonal; each is
// mirrored on store, rows are lda = n rounded up to even apart, and the padding column is zero.
template <typename T>
__device__ __forceinline__ double ld64(const T* p) { return (double)ElemIO<T>::load(p); }

template <typename T>
__device__ __forceinline__ void gram_tile(const SpectralJob& jb, double* G, int idx, double (*si)[65], double (*sj)[65],
                                          double (&acc)[4][4], int& i0, int& j0) {
    constexpr int TB = 64, KB = 16;
    const T* X = (const T*)jb.X;
    int ti = 0;  // lower-triangle tile index -> (ti, tj), tj <= ti
    while (idx >= ti + 1) { idx -= ti + 1; ++ti; }
    i0 = ti * TB;
    j0 = idx * TB;
    const long cols = jb.cols, tlen = jb.trans ? cols : jb.rows;
    const int n = jb.n, trans = jb.trans;
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
    for (long t0 = 0; t0 < tlen; t0 += KB) {
        __syncthreads();
        for (int e = tid; e < KB * TB; e += 256) {
            int kk, c;
            if (trans) { c = e / KB; kk = e % KB; }  // consecutive threads walk t (contiguous in X)
            else { kk = e / TB; c = e % TB; }       // consecutive threads walk i (contiguous in X)
            const long t = t0 + kk;
            const int gi = i0 + c, gj = j0 + c;
            double vi = 0.0, vj = 0.0;
            if (t < tlen) {
                if (gi < n) vi = trans ? ld64(X + (long)gi * cols + t) : ld64(X + t * cols + gi);
                if (gj < n) vj = trans ? ld64(X + (long)gj * cols + t) : ld64(X + t * cols + gj);
            }
            si[kk][c] = vi;
            sj[kk][c] = vj;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < KB; ++kk) {
            double a[4], b[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) a[r] = si[kk][ty + 16 * r];
#pragma unroll
            for (int c = 0; c < 4; ++c) b[c] = sj[kk][tx + 16 * c];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[r][c] = fma(a[r], b[c], acc[r][c]);
        }
    }
}

__global__ __launch_bounds__(256) void gram_kernel(SpectralBatch sb) {
    __shared__ double si[16][65];
    __shared__ double sj[16][65];
    const int bi = blockIdx.x, tid = threadIdx.x;
    int b = 0;
    while (b + 1 < sb.count && sb.jobs[b + 1].tile0 <= bi) ++b;
    const SpectralJob jb = sb.jobs[b];
    double* G = sb.gram(b);
    double acc[4][4] = {};
    int i0, j0;
    if (jb.dtype == 1) gram_tile<bf16>(jb, G, bi - jb.tile0, si, sj, acc, i0, j0);
    else gram_tile<float>(jb, G, bi - jb.tile0, si, sj, acc, i0, j0);
    const int n = jb.n, lda = spectral_lda(n), tx = tid & 15, ty = tid >> 4;
    double* trace = sb.out(b) + 2 * (long)sb.nmax;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int gi = i0 + ty + 16 * r, gj = j0 + tx + 16 * c;
            if (gi < n && gj < n) {
                G[(long)gi * lda + gj] = acc[r][c];
                G[(long)gj * lda + gi] = acc[r][c];
                if (gi == gj) {
                    trace[gi] = acc[r][c];
                    if (lda > n) G[(long)gi * lda + n] = 0.0;
                }
            }
        }
}

// ---------------------------------------------------------------------------- tridiagonal
// Householder reduction A = Q T Q^T (Golub & Van Loan, Sec. 8.3.1).  Step j reflects the
// column x = A[j+1:, j] onto beta e_1 with H = I - tau v v^T (v_0 = 1), using the trailing
// block A22 = A[j+1:, j+1:]:  p = tau A22 v,  w = p - (tau/2)(p.v) v,  A22 -= v w^T + w v^T.
//
// One launch per step for a whole batch of matrices.  Every workgroup forms w, the next column and
// its reflector v' by itself (O(n) values out of L2 and two block sums), then applies the rank-2
// update to its rows and, in the same pass over them, forms its part of the next p.  The reduction
// is a chain of n dependent steps, so a step's fixed cost counts as much as its bytes: a kernel of
// one workgroup for the vectors and one for the rows, per matrix and on a stream and host thread
// of its own, took 4-5 us each and were bound by the launches (24 matrices of 256 x 256 to
// 1024 x 256: 21.3 ms; 4 of 1152 x 1152 and 2 of 4608 x 1152: 62.9 ms, both with the host's QR).

// sum over the workgroup through red (one double per wave, used once per call)
__device__ __forceinline__ double block_sum_d(double v, double* red) {
    v = warp_sum(v);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) red[w] = v;
    __syncthreads();
    double t = 0.0;
    const int nw = blockDim.x >> 6;
    for (int i = 0; i < nw; ++i) t += red[i];
    return t;
}

constexpr int kTriThreads = 256, kTriRows = 16;  // rows per workgroup pass: four per wave

// FIRST: the reflector of column 0 and its p (no update).  Otherwise step j: consumes v_j, p_j,
// tau_j and leaves v_{j+1}, p_{j+1}, tau_{j+1} (ping-pong buffers: other workgroups of the launch
// still read the old ones).
template <bool FIRST>
__global__ __launch_bounds__(kTriThreads) void tri_step_kernel(SpectralBatch sb, int j) {
    extern __shared__ __attribute__((aligned(16))) double sh[];
    __shared__ double red[2 * (kTriThreads / 64)];
    const int b = blockIdx.y, n = sb.jobs[b].n, tid = threadIdx.x;
    if (n < 3) {
        if (FIRST && blockIdx.x == 0 && tid == 0) {  // already tridiagonal
            double *diag = sb.out(b), *offd = diag + sb.nmax, *A = sb.gram(b);
            diag[0] = A[0];
            if (n == 2) { diag[1] = A[spectral_lda(2) + 1]; offd[0] = A[1]; }
        }
        return;
    }
    if (!FIRST && j > n - 3) return;
    const int lda = spectral_lda(n);
    double* A = sb.gram(b);
    double *diag = sb.out(b), *offd = diag + sb.nmax;
    double* work = sb.work(b);  // v[2], p[2], tau[2]
    const int r0 = FIRST ? 0 : j + 1;  // row and column 0 of the block
    const int m = n - r0;              // its size
    if ((int)blockIdx.x * kTriRows + 1 >= m && blockIdx.x > 0) return;
    // vectors by column c - c0, c0 the even column at or before r0 + 1 (16-byte row accesses);
    // entries outside the block are zero
    const int c0 = (r0 + 1) & ~1, len = ((n + 1) & ~1) - c0, sp = r0 + 1 - c0;
    double *sv = sh, *sw = sh + len, *sx = sh + 2 * len;
    const double* arow = A + (long)r0 * lda + r0;  // row 0 of the block (== column 0)
    const int nx = j + 1;                          // index of the reflector formed here (FIRST: j = -1)
    double* const vn = work + (long)(nx & 1) * sb.nmax;
    double* const pn = work + (long)(2 + (nx & 1)) * sb.nmax;
    double* const taus = work + 4 * (long)sb.nmax;
    // rows 1 .. m - 1 of the block, four per wave at once (the LDS vectors are read once for four).
    // The first PRE column chunks of the first pass are loaded here, before the vectors are formed:
    // the step is a chain of memory round trips and block sums, and the rows depend on none of them.
    const int lane = tid & 63, wave = tid >> 6;
    constexpr int PRE = 2;
    double2 pre[PRE][4];
    {
        const int i0 = 1 + blockIdx.x * kTriRows + wave * 4;
#pragma unroll
        for (int u = 0; u < PRE; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int c = lane * 2 + u * 128;
                pre[u][r] = c < len ? *(const double2*)(A + (long)(r0 + min(i0 + r, m - 1)) * lda + c0 + c)
                                    : make_double2(0.0, 0.0);
            }
    }
    if (tid == 0) {
        if (sp) { sv[0] = 0.0; sw[0] = 0.0; sx[0] = 0.0; }
        if (n & 1) { sv[len - 1] = 0.0; sw[len - 1] = 0.0; sx[len - 1] = 0.0; }
    }
    // a thread handles the same entries in every pass over the vectors, so only the sums need barriers
    double v0 = 0.0, w0 = 0.0, k = 0.0;
    double alpha = arow[1];
    if (!FIRST) {
        const double* v = work + (long)(j & 1) * sb.nmax;
        const double* p = work + (long)(2 + (j & 1)) * sb.nmax;
        const double tau = taus[j & 1], p0 = p[0], v1 = v[1], p1 = p[1];
        double s = 0.0;
        v0 = 1.0;
        for (int i = tid; i < m - 1; i += kTriThreads) {
            const double vi = v[i + 1], pi = p[i + 1];
            s += pi * vi;
            sv[i + sp] = vi;
            sw[i + sp] = pi;
            sx[i + sp] = arow[i + 1];
        }
        k = 0.5 * tau * (block_sum_d(s, red) + p0);
        w0 = p0 - k;
        alpha = alpha - v1 * w0 - (p1 - k * v1);
        if (m == 2) {
            // last step: the trailing 2 x 2 block after its update is the end of T
            if (blockIdx.x == 0 && tid == 0) {
                diag[j + 1] = arow[0] - 2.0 * w0;
                offd[j + 1] = alpha;
                diag[j + 2] = A[(long)(j + 2) * lda + (j + 2)] - 2.0 * v1 * (p1 - k * v1);
            }
            return;
        }
    }
    // w, the updated column 0 below the diagonal, x[i] = A22[1+i][0] - v[1+i] w[0] - w[1+i] v[0], and its
    // reflector (x[0] is alpha)
    double s = 0.0;
    for (int i = tid; i < m - 1; i += kTriThreads) {
        double x = FIRST ? arow[1 + i] : sx[i + sp];
        if (FIRST) {
            sv[i + sp] = 0.0;
            sw[i + sp] = 0.0;
        } else {
            const double w = sw[i + sp] - k * sv[i + sp];
            sw[i + sp] = w;
            x = x - sv[i + sp] * w0 - w;
        }
        sx[i + sp] = x;
        if (i > 0) s += x * x;
    }
    const double sigma = block_sum_d(s, red + kTriThreads / 64);
    double taun = 0.0, beta = alpha, scale = 0.0;
    if (sigma != 0.0) {
        const double mu = sqrt(alpha * alpha + sigma);
        beta = alpha <= 0.0 ? mu : -mu;
        taun = (beta - alpha) / beta;
        scale = 1.0 / (alpha - beta);
    }
    for (int i = tid; i < m - 1; i += kTriThreads) {
        const double y = i == 0 ? 1.0 : sx[i + sp] * scale;
        sx[i + sp] = y;
        if (blockIdx.x == 0) vn[i] = y;
    }
    if (blockIdx.x == 0 && tid == 0) {
        diag[nx] = FIRST ? A[0] : arow[0] - 2.0 * w0;
        offd[nx] = beta;
        taus[nx & 1] = taun;
    }
    __syncthreads();
    for (int base = 1 + blockIdx.x * kTriRows; base < m; base += gridDim.x * kTriRows) {
        const int i0 = base + wave * 4;
        const bool first = base == 1 + (int)blockIdx.x * kTriRows;
        double vi[4], wi[4], acc[4] = {};
        double* ar[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = min(i0 + r, m - 1);  // past the last row: the last one again, not stored
            vi[r] = sv[i - 1 + sp];
            wi[r] = sw[i - 1 + sp];
            ar[r] = A + (long)(r0 + i) * lda + c0;
        }
        auto chunk = [&](int c, double2 (&a)[4]) {
            const double2 w2 = *(const double2*)(sw + c), v2 = *(const double2*)(sv + c), x2 = *(const double2*)(sx + c);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (!FIRST) {
                    a[r].x -= vi[r] * w2.x + wi[r] * v2.x;
                    a[r].y -= vi[r] * w2.y + wi[r] * v2.y;
                    if (i0 + r < m) *(double2*)(ar[r] + c) = a[r];
                }
                acc[r] += a[r].x * x2.x;
                acc[r] += a[r].y * x2.y;
            }
        };
        auto load = [&](int c, double2 (&a)[4]) {
#pragma unroll
            for (int r = 0; r < 4; ++r) a[r] = *(const double2*)(ar[r] + c);
        };
        int c = lane * 2;
        if (first) {
#pragma unroll
            for (int u = 0; u < PRE; ++u, c += 128)
                if (c < len) chunk(c, pre[u]);
        }
        for (; c + 128 < len; c += 256) {
            double2 a[2][4];
            load(c, a[0]);
            load(c + 128, a[1]);
            chunk(c, a[0]);
            chunk(c + 128, a[1]);
        }
        if (c < len) {
            double2 a[4];
            load(c, a);
            chunk(c, a);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const double t = warp_sum(acc[r]);
            if (lane == 0 && i0 + r < m) pn[i0 + r - 1] = taun * t;
        }
    }
}

// Short sides past kSpectralMax (three vectors no longer fit the LDS): the same steps as two kernels,
// one workgroup for the vectors (w, the next column, the next reflector) and a wide one that applies
// the rank-2 update and forms the next p, one matrix at a time.
// work layout (doubles): v[2][nmax], p[nmax], w[nmax], xbuf[nmax], tau[2]

constexpr int kHouseThreads = 1024;

// Reflector of x[0..len-1] (len >= 1) into vout (vout[0] = 1); returns tau, writes beta.
__device__ double house(const double* x, int len, double* vout, double* beta_out, double* red) {
    double s = 0.0;
    for (int i = 1 + threadIdx.x; i < len; i += blockDim.x) s += x[i] * x[i];
    __syncthreads();  // red is free
    const double sigma = block_sum_d(s, red);
    const double alpha = x[0];
    double tau, beta, scale;
    if (sigma == 0.0) {
        tau = 0.0;
        beta = alpha;
        scale = 0.0;
    } else {
        const double mu = sqrt(alpha * alpha + sigma);
        beta = alpha <= 0.0 ? mu : -mu;
        tau = (beta - alpha) / beta;
        scale = 1.0 / (alpha - beta);
    }
    for (int i = threadIdx.x; i < len; i += blockDim.x) vout[i] = i == 0 ? 1.0 : x[i] * scale;
    *beta_out = beta;
    return tau;
}

// first reflector (step 0): x = A[0][1..n-1] (row 0 == column 0)
__global__ __launch_bounds__(kHouseThreads) void tri_init_kernel(const double* A, int n, double* v0,
                                                                 double* scal, double* diag, double* offd) {
    __shared__ double red[16];
    double beta;
    const double tau = house(A + 1, n - 1, v0, &beta, red);
    if (threadIdx.x == 0) {
        scal[0] = tau;
        diag[0] = A[0];
        offd[0] = beta;
    }
}

// p = tau A22 v for step 0 (A22 = A[1:, 1:]); one wave per row
__global__ __launch_bounds__(256) void tri_symv0_kernel(const double* A, int n, const double* v,
                                                        const double* scal, double* p) {
    const int m = n - 1;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= m) return;
    const double* ar = A + (long)(1 + row) * spectral_lda(n) + 1;
    double acc = 0.0;
    for (int c = lane; c < m; c += 64) acc += ar[c] * v[c];
    acc = warp_sum(acc);
    if (lane == 0) p[row] = scal[0] * acc;
}

// Step j: w = p - (tau/2)(p.v) v; the updated column j+1; the next reflector.
__global__ __launch_bounds__(kHouseThreads) void tri_w_house_kernel(const double* A, int n, int j,
                                                                    const double* v, double* vnext,
                                                                    const double* p, double* w, double* xbuf,
                                                                    double* scal, double* diag, double* offd) {
    __shared__ double red[16];
    const int m = n - j - 1;  // size of A22
    const double tau = scal[j & 1];
    double s = 0.0;
    for (int i = threadIdx.x; i < m; i += blockDim.x) s += p[i] * v[i];
    const double pv = block_sum_d(s, red);
    const double k = 0.5 * tau * pv;
    for (int i = threadIdx.x; i < m; i += blockDim.x) w[i] = p[i] - k * v[i];
    __syncthreads();
    const double* arow = A + (long)(j + 1) * spectral_lda(n) + (j + 1);  // row 0 of A22 (== column 0)
    if (m == 2) {
        // last step: the trailing 2 x 2 block after its update is the end of T
        if (threadIdx.x == 0) {
            diag[j + 1] = arow[0] - 2.0 * v[0] * w[0];
            offd[j + 1] = arow[1] - v[1] * w[0] - w[1] * v[0];
            diag[j + 2] = A[(long)(j + 2) * spectral_lda(n) + (j + 2)] - 2.0 * v[1] * w[1];
        }
        return;
    }
    // updated column 0 of A22 below the diagonal: x'[i] = A22[1+i][0] - v[1+i] w[0] - w[1+i] v[0]
    for (int i = threadIdx.x; i < m - 1; i += blockDim.x) xbuf[i] = arow[1 + i] - v[1 + i] * w[0] - w[1 + i] * v[0];
    __syncthreads();
    double beta;
    const double taun = house(xbuf, m - 1, vnext, &beta, red);
    if (threadIdx.x == 0) {
        diag[j + 1] = arow[0] - 2.0 * v[0] * w[0];
        offd[j + 1] = beta;
        scal[(j + 1) & 1] = taun;
    }
}

// Step j: A22[i][c] -= v[i] w[c] + w[i] v[c] for i, c >= 1, and the next p:
// pnext[i-1] = tau' sum_{c >= 1} A22[i][c] vnext[c-1].  One wave per row.
__global__ __launch_bounds__(256) void tri_update_kernel(double* A, int n, int j, const double* v,
                                                         const double* w, const double* vnext, const double* scal,
                                                         double* pnext) {
    const int m = n - j - 1;
    const int i = 1 + blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (i >= m) return;
    double* ar = A + (long)(j + 1 + i) * spectral_lda(n) + (j + 1);
    const double vi = v[i], wi = w[i];
    double acc = 0.0;
    for (int c = 1 + lane; c < m; c += 64) {
        const double a = ar[c] - (vi * w[c] + wi * v[c]);
        ar[c] = a;
        acc += a * vnext[c - 1];
    }
    acc = warp_sum(acc);
    if (lane == 0) pnext[i - 1] = scal[(j + 1) & 1] * acc;
}

static void tridiagonalize_large(const SpectralBatch& sb, int b, int n, hipStream_t st) {
    double *A = sb.gram(b), *diag = sb.out(b), *offd = diag + sb.nmax, *work = sb.work(b);
    const long ld = sb.nmax;
    double* v[2] = {work, work + ld};
    double *p = work + 2 * ld, *w = work + 3 * ld, *xbuf = work + 4 * ld, *scal = work + 5 * ld;
    hipLaunchKernelGGL(tri_init_kernel, dim3(1), dim3(kHouseThreads), 0, st, A, n, v[0], scal, diag, offd);
    hipLaunchKernelGGL(tri_symv0_kernel, dim3((n - 1 + 3) / 4), dim3(256), 0, st, A, n, v[0], scal, p);
    for (int j = 0; j <= n - 3; ++j) {
        const int m = n - j - 1;
        hipLaunchKernelGGL(tri_w_house_kernel, dim3(1), dim3(kHouseThreads), 0, st, A, n, j, v[j & 1],
                           v[(j + 1) & 1], p, w, xbuf, scal, diag, offd);
        if (m > 2)
            hipLaunchKernelGGL(tri_update_kernel, dim3((m - 1 + 3) / 4), dim3(256), 0, st, A, n, j, v[j & 1], w,
                               v[(j + 1) & 1], scal, p);
    }
}

// The largest eigenvalues of each tridiagonal matrix, by bisection on the count of negative pivots
// of T - x I (Golub & Van Loan, Sec. 8.4.1): eigenvalue i < k_b of matrix b per wave.  The 64 lanes
// evaluate 64 points of the current interval at once, so ten passes shrink it by 65^10 > 2^60.
// Only the top k = n / 10 are needed (the tail is the trace minus them); the host's QR over all of
// them took longer than the reduction.
constexpr int kSturmChunk = 1024;
__global__ __launch_bounds__(256) void sturm_kernel(SpectralBatch sb) {
    __shared__ __attribute__((aligned(16))) double2 de[kSturmChunk];  // diagonal, squared off-diagonal above it
    __shared__ double red[8];
    const int b = blockIdx.y, n = sb.jobs[b].n, kb = sb.jobs[b].k, tid = threadIdx.x, lane = tid & 63;
    if ((int)blockIdx.x * 4 >= kb) return;
    const int i = blockIdx.x * 4 + (tid >> 6);  // i-th largest (past kb: computed, not stored)
    const double *d = sb.out(b), *e = d + sb.nmax;
    // Gershgorin bounds and the smallest pivot magnitude allowed
    double lo = 1e308, hi = -1e308, emax = 0.0;
    for (int c = tid; c < n; c += 256) {
        const double r = (c > 0 ? fabs(e[c - 1]) : 0.0) + (c + 1 < n ? fabs(e[c]) : 0.0);
        lo = fmin(lo, d[c] - r);
        hi = fmax(hi, d[c] + r);
        if (c + 1 < n) emax = fmax(emax, e[c] * e[c]);
    }
    auto block = [&](double v, bool mx) {
        for (int o = 32; o > 0; o >>= 1) { const double u = __shfl_xor(v, o, 64); v = mx ? fmax(v, u) : fmin(v, u); }
        __syncthreads();
        if (lane == 0) red[tid >> 6] = v;
        __syncthreads();
        for (int w = 0; w < 4; ++w) v = mx ? fmax(v, red[w]) : fmin(v, red[w]);
        return v;
    };
    lo = block(lo, false);
    hi = block(hi, true);
    emax = block(emax, true);
    const double pivmin = 2.2250738585072014e-308 * fmax(1.0, emax) * 4.0;
    const double pad = 4.4408920985006262e-16 * fmax(fabs(lo), fabs(hi)) * n + pivmin;
    lo -= pad;
    hi += pad;
    const int want = n - i;  // count(x) >= want: at least n - i eigenvalues below x, so x > lambda_i
    for (int pass = 0; pass < 10; ++pass) {
        const double step = (hi - lo) * (1.0 / 65.0);
        const double x = lo + step * (lane + 1);
        int cnt = 0;
        double q = 1.0;
        for (int c0 = 0; c0 < n; c0 += kSturmChunk) {
            const int cn = min(kSturmChunk, n - c0);
            __syncthreads();
            for (int c = tid; c < cn; c += 256) {
                const double u = c0 + c > 0 ? e[c0 + c - 1] : 0.0;
                de[c] = make_double2(d[c0 + c], u * u);
            }
            __syncthreads();
#pragma unroll 4
            for (int c = 0; c < cn; ++c) {
                // 1 / q to full precision: the hardware estimate and two Newton steps
                double r = __builtin_amdgcn_rcp(q);
                r = fma(fma(-q, r, 1.0), r, r);
                r = fma(fma(-q, r, 1.0), r, r);
                q = fma(-de[c].y, r, de[c].x - x);
                if (fabs(q) <= pivmin) q = -pivmin;
                cnt += q < 0.0;
            }
        }
        const unsigned long long above = __ballot(cnt >= want);
        const int f = above ? __ffsll((long long)above) - 1 : 64;  // first point above lambda_i
        const double nlo = f == 0 ? lo : lo + step * f, nhi = f == 64 ? hi : lo + step * (f + 1);
        lo = nlo;
        hi = nhi;
    }
    if (lane == 0 && i < kb) sb.out(b)[3 * (long)sb.nmax + i] = 0.5 * (lo + hi);
}

hipError_t launch_spectra(const SpectralBatch& sb, const SpectralJob* host_jobs, hipStream_t st) {
    int tiles = 0, nb = 1, kmax = 1;
    for (int b = 0; b < sb.count; ++b) {
        const int nt = (host_jobs[b].n + 63) / 64;
        tiles = host_jobs[b].tile0 + nt * (nt + 1) / 2;
        nb = std::max(nb, (int)host_jobs[b].n);
        kmax = std::max(kmax, (int)host_jobs[b].k);
    }
    hipLaunchKernelGGL(gram_kernel, dim3(tiles), dim3(256), 0, st, sb);
    if (nb > kSpectralMax) {
        for (int b = 0; b < sb.count; ++b) tridiagonalize_large(sb, b, host_jobs[b].n, st);
    } else {
        if (3 * (size_t)(nb + 2) * sizeof(double) > 64 * 1024)
            for (auto f : {(const void*)tri_step_kernel<true>, (const void*)tri_step_kernel<false>}) {
                const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 256);
                if (e != hipSuccess) return e;
            }
        for (int j = -1; j == -1 || j <= nb - 3; ++j) {
            // workgroups per matrix: one pass of 16 rows each while that stays near 2048 in all
            // (eight per CU); beyond, a workgroup loops over its rows and the O(n) vectors are
            // formed fewer times
            const int m = nb - j - 1;
            const int wgs = std::max(1, std::min((m - 1 + kTriRows - 1) / kTriRows, std::max(1, 2048 / sb.count)));
            const size_t bytes = 3 * (size_t)(m + 2) * sizeof(double);
            if (j < 0)
                hipLaunchKernelGGL(tri_step_kernel<true>, dim3(wgs, sb.count), dim3(kTriThreads), bytes, st, sb, j);
            else
                hipLaunchKernelGGL(tri_step_kernel<false>, dim3(wgs, sb.count), dim3(kTriThreads), bytes, st, sb, j);
        }
    }
    hipLaunchKernelGGL(sturm_kernel, dim3((kmax + 3) / 4, sb.count), dim3(256), 0, st, sb);
    return hipGetLastError();
}

}  // namespace sgd
