// Offline spectra of the scored weight matrices (fp64): the Gram matrix of the short side, a
// Householder reduction of that symmetric matrix to tridiagonal form and the eigenvalues of that
// form, the squared singular values the spectral concentration ratio needs.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace sgd {

// ---------------------------------------------------------------------------- Gram
// G[i][j] = sum_t E(t, i) E(t, j) with E(t, i) = X[t][i] (trans = 0) or X[i][t] (trans = 1), for
// every matrix of a batch in one launch.  64 x 64 output tiles on and below the diagonal; each is
// mirrored on store, rows are lda = n rounded up to even apart, and the padding column is zero.
//
// On the matrix cores (v_mfma_f64_16x16x4_f64: lane l holds row l % 16 and k = l / 16 of either operand,
// and of the product column l % 16 and row 4 r + l / 16 in register r): the same fp64 products and
// sums at the same peak rate as vector FMAs, but a wave's 32 x 32 tile reads 4 values a lane from the
// LDS for 4096 FMAs; a 4 x 4 patch a thread read 8 for 1024 and was bound by the LDS.  The next k chunk
// is on its way while one is multiplied.  24 fp32 matrices of 256 x 256 to 1024 x 256 264 -> 85 us; bf16
// 4 of 1152 x 1152 and 2 of 4608 x 1152 1401 -> 681 us.
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kGramKB = 16, kGramLD = 66;  // k depth of a chunk; LDS row pitch (rows 16 bytes apart in the banks)

template <typename T>
__device__ __forceinline__ void gram_tile(const SpectralJob& jb, int idx, double (*si)[kGramLD], double (*sj)[kGramLD],
                                          f64x4 (&acc)[2][2], int& i0, int& j0) {
    constexpr int TB = 64, KB = kGramKB, E = KB * TB / 256;
    const T* X = (const T*)jb.X;
    int ti = 0;  // lower-triangle tile index -> (ti, tj), tj <= ti
    while (idx >= ti + 1) { idx -= ti + 1; ++ti; }
    i0 = ti * TB;
    j0 = idx * TB;
    const long cols = jb.cols, tlen = jb.trans ? cols : jb.rows;
    const int n = jb.n, trans = jb.trans;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wi = (wave >> 1) * 32, wj = (wave & 1) * 32, fr = lane & 15, fk = lane >> 4;
    // consecutive threads walk X's contiguous dimension
    auto place = [&](int u, int& kk, int& c) {
        const int e = tid + u * 256;
        if (trans) { c = e / KB; kk = e % KB; }
        else { kk = e / TB; c = e % TB; }
    };
    T ri[E], rj[E];
    auto load = [&](long t0) {
#pragma unroll
        for (int u = 0; u < E; ++u) {
            int kk, c;
            place(u, kk, c);
            const long t = t0 + kk;
            const int gi = i0 + c, gj = j0 + c;
            ri[u] = t < tlen && gi < n ? X[trans ? (long)gi * cols + t : t * cols + gi] : T(0.f);
            rj[u] = t < tlen && gj < n ? X[trans ? (long)gj * cols + t : t * cols + gj] : T(0.f);
        }
    };
    load(0);
    for (long t0 = 0; t0 < tlen; t0 += KB) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < E; ++u) {
            int kk, c;
            place(u, kk, c);
            si[kk][c] = (double)ElemIO<T>::load(&ri[u]);
            sj[kk][c] = (double)ElemIO<T>::load(&rj[u]);
        }
        __syncthreads();
        if (t0 + KB < tlen) load(t0 + KB);
#pragma unroll
        for (int k = 0; k < KB; k += 4) {
            double a[2], b[2];
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                a[x] = si[k + fk][wi + x * 16 + fr];
                b[x] = sj[k + fk][wj + x * 16 + fr];
            }
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int y = 0; y < 2; ++y) acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[x], b[y], acc[x][y], 0, 0, 0);
        }
    }
}

__global__ __launch_bounds__(256) void gram_kernel(SpectralBatch sb) {
    __shared__ double si[kGramKB][kGramLD];
    __shared__ double sj[kGramKB][kGramLD];
    const int bi = blockIdx.x, tid = threadIdx.x;
    int b = 0;
    while (b + 1 < sb.count && sb.jobs[b + 1].tile0 <= bi) ++b;
    const SpectralJob jb = sb.jobs[b];
    double* G = sb.gram(b);
    f64x4 acc[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = f64x4{0.0, 0.0, 0.0, 0.0};
    int i0, j0;
    if (jb.dtype == 1) gram_tile<bf16>(jb, bi - jb.tile0, si, sj, acc, i0, j0);
    else gram_tile<float>(jb, bi - jb.tile0, si, sj, acc, i0, j0);
    const int n = jb.n, lda = spectral_lda(n), lane = tid & 63, wave = tid >> 6;
    double* trace = sb.out(b) + 2 * (long)sb.nmax;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int gi = i0 + (wave >> 1) * 32 + x * 16 + 4 * r + (lane >> 4);
                const int gj = j0 + (wave & 1) * 32 + y * 16 + (lane & 15);
                // a diagonal tile stores its lower half both ways, so that the matrix is symmetric
                if (gi >= n || gj >= n || gj > gi) continue;
                const double v = acc[x][y][r];
                G[(long)gi * lda + gj] = v;
                G[(long)gj * lda + gi] = v;
                if (gi == gj) {
                    trace[gi] = v;
                    if (lda > n) G[(long)gi * lda + n] = 0.0;
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

// x of the lane that the DPP control CTRL names
template <int CTRL>
__device__ __forceinline__ double dpp_d(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = __builtin_amdgcn_mov_dpp((uint32_t)u, CTRL, 0xF, 0xF, true);
    const uint32_t hi = __builtin_amdgcn_mov_dpp((uint32_t)(u >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
// x + x of lane ^ 16 / ^ 32 (register swaps between rows of 16 and halves of the wave)
__device__ __forceinline__ double add_xor16(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const auto a = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto b = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    return __builtin_bit_cast(double, (uint64_t)b[0] << 32 | a[0]) + __builtin_bit_cast(double, (uint64_t)b[1] << 32 | a[1]);
}
__device__ __forceinline__ double add_xor32(double x) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const auto a = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)u, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    return __builtin_bit_cast(double, (uint64_t)b[0] << 32 | a[0]) + __builtin_bit_cast(double, (uint64_t)b[1] << 32 | a[1]);
}
// sum over the wave in every lane, without the LDS round trips of a shuffle (a step is a chain of sums)
__device__ __forceinline__ double wave_sum_d(double x) {
    x += dpp_d<0xB1>(x);   // lane ^ 1
    x += dpp_d<0x4E>(x);   // lane ^ 2
    x += dpp_d<0x141>(x);  // the other quad of eight lanes
    x += dpp_d<0x140>(x);  // the other eight lanes of sixteen
    return add_xor32(add_xor16(x));
}

// sum over the workgroup through red (one double per wave, used once per call)
__device__ __forceinline__ double block_sum_d(double v, double* red) {
    v = wave_sum_d(v);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) red[w] = v;
    __syncthreads();
    double t = 0.0;
    const int nw = blockDim.x >> 6;
    for (int i = 0; i < nw; ++i) t += red[i];
    return t;
}

constexpr int kTriThreads = 256, kTriRows = 16;  // rows per workgroup pass: four per wave
// The last trailing block, of up to kTail rows, fits one CU's registers and is reduced by tri_tail_kernel:
// from step tail_step(n) on
constexpr int kTail = 192;
__host__ __device__ inline int tail_step(int n) { return n - 1 > kTail ? n - 1 - kTail : 0; }

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
    if (!FIRST && j >= tail_step(n)) return;
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
            const double t = wave_sum_d(acc[r]);
            if (lane == 0 && i0 + r < m) pn[i0 + r - 1] = taun * t;
        }
    }
}

// The last steps, from tail_step(n) on: the trailing block stays in the registers of one workgroup
// (thread (ty, tx) of 16 x 32 owns rows ty + 16 a and columns tx + 32 c, so work shrinks evenly as rows
// and columns are finished) and the vectors in LDS, two barriers a step.  A step takes 2.8 us (two wave
// sums, a square root and two divisions in sequence) instead of the 5.4-6 us that a launch and its round
// trips through L2 take at these sizes: the last 192 of 256 steps 1100 -> 540 us.
constexpr int kTailTY = 16, kTailTX = 32, kTailA = kTail / kTailTY, kTailC = kTail / kTailTX;
__global__ __launch_bounds__(kTailTY * kTailTX) void tri_tail_kernel(SpectralBatch sb) {
    __shared__ double sv[kTail], sp[kTail], sx[kTail], sy[kTail];
    static_assert(kTail % 64 == 0 && kTailA % 4 == 0, "tail shape");
    const int b = blockIdx.x, n = sb.jobs[b].n, tid = threadIdx.x, lane = tid & 63;
    if (n < 3) return;  // the first launch has written T
    const int tx = tid & (kTailTX - 1), ty = tid / kTailTX;
    const int js = tail_step(n), m0 = n - js - 1, lda = spectral_lda(n);
    const double* A = sb.gram(b) + (long)(js + 1) * lda + (js + 1);
    double *diag = sb.out(b) + js + 1, *offd = diag + sb.nmax;
    const double* work = sb.work(b);
    // rows, columns and vector entries past the block are zero and stay zero
    double acc[kTailA][kTailC];
#pragma unroll
    for (int a = 0; a < kTailA; ++a)
#pragma unroll
        for (int c = 0; c < kTailC; ++c) {
            const int i = ty + kTailTY * a, k = tx + kTailTX * c;
            const double x = A[(long)min(i, m0 - 1) * lda + min(k, m0 - 1)];
            acc[a][c] = max(i, k) < m0 ? x : 0.0;
        }
    for (int i = tid; i < kTail; i += kTailTY * kTailTX) {
        sv[i] = i < m0 ? work[(long)(js & 1) * sb.nmax + i] : 0.0;
        sp[i] = i < m0 ? work[(long)(2 + (js & 1)) * sb.nmax + i] : 0.0;
    }
    double tau = work[4 * (long)sb.nmax + (js & 1)];
    __syncthreads();
    for (int o = 0;; ++o) {  // the block's first row; v, p are zero before it
        // w = p - (tau / 2) (p . v) v and A -= v w^T + w v^T
        double s = 0.0;
#pragma unroll
        for (int u = 0; u < kTail / 64; ++u) s += sp[lane + 64 * u] * sv[lane + 64 * u];
        const double k = 0.5 * tau * wave_sum_d(s);
        {
            double vc[kTailC], wc[kTailC];
#pragma unroll
            for (int c = 0; c < kTailC; ++c) {
                vc[c] = sv[tx + kTailTX * c];
                wc[c] = sp[tx + kTailTX * c] - k * vc[c];
            }
#pragma unroll
            for (int a = 0; a < kTailA; ++a) {
                if (kTailTY * (a + 1) <= o || kTailTY * a >= m0) continue;  // finished or past the block
                const double vr = sv[ty + kTailTY * a], wr = sp[ty + kTailTY * a] - k * vr;
#pragma unroll
                for (int c = 0; c < kTailC; ++c) acc[a][c] -= vr * wc[c] + wr * vc[c];
            }
        }
        // column o
#pragma unroll
        for (int c = 0; c < kTailC; ++c)
            if (c == o / kTailTX && tx == o % kTailTX)
#pragma unroll
                for (int a = 0; a < kTailA; ++a) sx[ty + kTailTY * a] = acc[a][c];
        const bool last = m0 - o == 2;  // the trailing 2 x 2 block is the end of T
        if (last) {
#pragma unroll
            for (int c = 0; c < kTailC; ++c)
                if (c == (o + 1) / kTailTX && tx == (o + 1) % kTailTX)
#pragma unroll
                    for (int a = 0; a < kTailA; ++a) sy[ty + kTailTY * a] = acc[a][c];
        }
        __syncthreads();
        const double alpha = sx[o + 1];
        if (last) {
            if (tid == 0) {
                diag[o] = sx[o];
                offd[o] = alpha;
                diag[o + 1] = sy[o + 1];
            }
            return;
        }
        // the reflector of column o below the diagonal
        s = 0.0;
#pragma unroll
        for (int u = 0; u < kTail / 64; ++u) {
            const int i = lane + 64 * u;
            const double x = sx[i];
            if (i > o + 1) s += x * x;
        }
        const double sigma = wave_sum_d(s);
        double beta = alpha, scale = 0.0;
        tau = 0.0;
        if (sigma != 0.0) {
            const double mu = sqrt(alpha * alpha + sigma);
            beta = alpha <= 0.0 ? mu : -mu;
            tau = (beta - alpha) / beta;
            scale = 1.0 / (alpha - beta);
        }
        auto v_at = [&](int i) { return i > o + 1 ? sx[i] * scale : i == o + 1 ? 1.0 : 0.0; };
        if (tid == 0) {
            diag[o] = sx[o];
            offd[o] = beta;
        }
        if (tid < kTail) sv[tid] = v_at(tid);
        // p = tau A v
        double p[kTailA];
        {
            double vc[kTailC];
#pragma unroll
            for (int c = 0; c < kTailC; ++c) vc[c] = v_at(tx + kTailTX * c);
#pragma unroll
            for (int a = 0; a < kTailA; ++a) {
                p[a] = 0.0;
                if (kTailTY * (a + 1) <= o || kTailTY * a >= m0) continue;
#pragma unroll
                for (int c = 0; c < kTailC; ++c) p[a] += acc[a][c] * vc[c];
            }
        }
        // row sums over the 32 lanes of a row: lanes exchange halves of their rows twice, after which
        // lane tx holds the quad's sums of rows 4 g + tx % 4, then add over the eight quads
        const bool o1 = tx & 1, o2 = tx & 2;
#pragma unroll
        for (int g = 0; g < kTailA / 4; ++g) {
            double u0 = o1 ? p[4 * g + 1] : p[4 * g], u1 = o1 ? p[4 * g + 3] : p[4 * g + 2];
            u0 += dpp_d<0xB1>(o1 ? p[4 * g] : p[4 * g + 1]);
            u1 += dpp_d<0xB1>(o1 ? p[4 * g + 2] : p[4 * g + 3]);
            double t = o2 ? u1 : u0;
            t += dpp_d<0x4E>(o2 ? u0 : u1);
            t += dpp_d<0x128>(t);  // eight lanes on
            t += dpp_d<0x124>(t);  // four lanes on
            t = add_xor16(t);
            const int i = ty + kTailTY * (4 * g + tx);
            if (tx < 4) sp[i] = i > o ? tau * t : 0.0;
        }
        __syncthreads();
    }
}

// Short sides past kSpectralMax (three vectors no longer fit the LDS): the same steps as two kernels,
// one workgroup a matrix for the vectors (w, the next column, the next reflector) and a wide one that
// applies the rank-2 update and forms the next p, each launched once per step for the whole batch: the
// vector kernels of all matrices run side by side (24 matrices of 6656 x 6656: 10.7 s, one matrix after
// another 11.7).
// work layout (doubles): v[2][nmax], p[nmax], w[nmax], xbuf[nmax], tau[2]
struct LargeWork {
    double *A, *diag, *offd, *vs, *p, *w, *xbuf, *scal;
    long ld;
    __device__ __forceinline__ double* v(int j) const { return vs + (j & 1) * ld; }
    __device__ __forceinline__ LargeWork(const SpectralBatch& sb, int b) {
        double* work = sb.work(b);
        ld = sb.nmax;
        A = sb.gram(b);
        diag = sb.out(b);
        offd = diag + ld;
        vs = work;
        p = work + 2 * ld;
        w = work + 3 * ld;
        xbuf = work + 4 * ld;
        scal = work + 5 * ld;
    }
};

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
__global__ __launch_bounds__(kHouseThreads) void tri_init_kernel(SpectralBatch sb) {
    __shared__ double red[16];
    const LargeWork W(sb, blockIdx.x);
    double beta;
    const double tau = house(W.A + 1, sb.jobs[blockIdx.x].n - 1, W.v(0), &beta, red);
    if (threadIdx.x == 0) {
        W.scal[0] = tau;
        W.diag[0] = W.A[0];
        W.offd[0] = beta;
    }
}

// p = tau A22 v for step 0 (A22 = A[1:, 1:]); one wave per row
__global__ __launch_bounds__(256) void tri_symv0_kernel(SpectralBatch sb) {
    const LargeWork W(sb, blockIdx.y);
    const int n = sb.jobs[blockIdx.y].n, m = n - 1;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= m) return;
    const double* ar = W.A + (long)(1 + row) * spectral_lda(n) + 1;
    double acc = 0.0;
    for (int c = lane; c < m; c += 64) acc += ar[c] * W.v(0)[c];
    acc = warp_sum(acc);
    if (lane == 0) W.p[row] = W.scal[0] * acc;
}

// Step j: w = p - (tau/2)(p.v) v; the updated column j+1; the next reflector.
__global__ __launch_bounds__(kHouseThreads) void tri_w_house_kernel(SpectralBatch sb, int j) {
    __shared__ double red[16];
    const LargeWork W(sb, blockIdx.x);
    const int n = sb.jobs[blockIdx.x].n;
    const int m = n - j - 1;  // size of A22
    if (m < 2) return;        // this matrix is done
    const double *v = W.v(j), *p = W.p;
    double* const w = W.w;
    const double tau = W.scal[j & 1];
    double s = 0.0;
    for (int i = threadIdx.x; i < m; i += blockDim.x) s += p[i] * v[i];
    const double pv = block_sum_d(s, red);
    const double k = 0.5 * tau * pv;
    for (int i = threadIdx.x; i < m; i += blockDim.x) w[i] = p[i] - k * v[i];
    __syncthreads();
    const double* arow = W.A + (long)(j + 1) * spectral_lda(n) + (j + 1);  // row 0 of A22 (== column 0)
    if (m == 2) {
        // last step: the trailing 2 x 2 block after its update is the end of T
        if (threadIdx.x == 0) {
            W.diag[j + 1] = arow[0] - 2.0 * v[0] * w[0];
            W.offd[j + 1] = arow[1] - v[1] * w[0] - w[1] * v[0];
            W.diag[j + 2] = W.A[(long)(j + 2) * spectral_lda(n) + (j + 2)] - 2.0 * v[1] * w[1];
        }
        return;
    }
    // updated column 0 of A22 below the diagonal: x'[i] = A22[1+i][0] - v[1+i] w[0] - w[1+i] v[0]
    for (int i = threadIdx.x; i < m - 1; i += blockDim.x) W.xbuf[i] = arow[1 + i] - v[1 + i] * w[0] - w[1 + i] * v[0];
    __syncthreads();
    double beta;
    const double taun = house(W.xbuf, m - 1, W.v(j + 1), &beta, red);
    if (threadIdx.x == 0) {
        W.diag[j + 1] = arow[0] - 2.0 * v[0] * w[0];
        W.offd[j + 1] = beta;
        W.scal[(j + 1) & 1] = taun;
    }
}

// Step j: A22[i][c] -= v[i] w[c] + w[i] v[c] for i, c >= 1, and the next p:
// pnext[i-1] = tau' sum_{c >= 1} A22[i][c] vnext[c-1].  One wave per row.
__global__ __launch_bounds__(256) void tri_update_kernel(SpectralBatch sb, int j) {
    const LargeWork W(sb, blockIdx.y);
    const int n = sb.jobs[blockIdx.y].n, m = n - j - 1;
    const int i = 1 + blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (i >= m || m < 3) return;
    const double *v = W.v(j), *w = W.w, *vnext = W.v(j + 1);
    double* ar = W.A + (long)(j + 1 + i) * spectral_lda(n) + (j + 1);
    const double vi = v[i], wi = w[i];
    double acc = 0.0;
    for (int c = 1 + lane; c < m; c += 64) {
        const double a = ar[c] - (vi * w[c] + wi * v[c]);
        ar[c] = a;
        acc += a * vnext[c - 1];
    }
    acc = warp_sum(acc);
    if (lane == 0) W.p[i - 1] = W.scal[(j + 1) & 1] * acc;
}

// every matrix of the batch past kSpectralMax, nb the largest short side
static void tridiagonalize_large(const SpectralBatch& sb, int nb, hipStream_t st) {
    hipLaunchKernelGGL(tri_init_kernel, dim3(sb.count), dim3(kHouseThreads), 0, st, sb);
    hipLaunchKernelGGL(tri_symv0_kernel, dim3((nb - 1 + 3) / 4, sb.count), dim3(256), 0, st, sb);
    for (int j = 0; j <= nb - 3; ++j) {
        const int m = nb - j - 1;
        hipLaunchKernelGGL(tri_w_house_kernel, dim3(sb.count), dim3(kHouseThreads), 0, st, sb, j);
        if (m > 2) hipLaunchKernelGGL(tri_update_kernel, dim3((m - 1 + 3) / 4, sb.count), dim3(256), 0, st, sb, j);
    }
}

// The eigenvalues of each tridiagonal matrix, by bisection on the number of sign changes in the
// sequence of leading principal minors of T - x I (Golub & Van Loan, Sec. 8.4.1), p_i = (d_i - x) p_{i-1} -
// e_{i-1}^2 p_{i-2}: sixteen lanes per eigenvalue evaluate sixteen points of its interval at once, so sixteen
// passes shrink it by 17^16 > 2^65.  All of them are found, not the largest k alone: the tail energy is
// then a sum of small values, where the trace minus the k largest leaves their roundings behind.
// A step of the sequence is one dependent fma (the quotient of neighbouring minors instead, with its
// reciprocal, took 115 cycles); the pair is scaled back every eight steps, T is scaled to norm one by a
// power of two.
constexpr int kSturmChunk = 1024;
__global__ __launch_bounds__(256) void sturm_kernel(SpectralBatch sb) {
    __shared__ __attribute__((aligned(16))) double2 de[kSturmChunk];  // diagonal, squared off-diagonal above it
    __shared__ double red[8];
    const int b = blockIdx.y, n = sb.jobs[b].n, tid = threadIdx.x, lane = tid & 63;
    if ((int)blockIdx.x * 16 >= n) return;
    const int i = blockIdx.x * 16 + (tid >> 4);  // i-th largest (past n: computed, not stored)
    const double *d = sb.out(b), *e = d + sb.nmax;
    // Gershgorin bounds
    double lo = 1e308, hi = -1e308;
    for (int c = tid; c < n; c += 256) {
        const double r = (c > 0 ? fabs(e[c - 1]) : 0.0) + (c + 1 < n ? fabs(e[c]) : 0.0);
        lo = fmin(lo, d[c] - r);
        hi = fmax(hi, d[c] + r);
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
    const double norm = fmax(fabs(lo), fabs(hi));
    int ex = 0;
    if (norm > 0.0 && norm < 1e308) frexp(norm, &ex);
    const double pad = 4.4408920985006262e-16 * n;
    lo = ldexp(lo, -ex) - pad;
    hi = ldexp(hi, -ex) + pad;
    const int want = n - i;  // count(x) >= want: at least n - i eigenvalues below x, so x > lambda_i
    for (int pass = 0; pass < 16; ++pass) {
        const double step = (hi - lo) * (1.0 / 17.0);
        const double x = lo + step * ((lane & 15) + 1);
        int cnt = 0;
        double p0 = 0.0, p1 = 1.0;
        for (int c0 = 0; c0 < n; c0 += kSturmChunk) {
            const int cn = min(kSturmChunk, n - c0);
            __syncthreads();
            for (int c = tid; c < kSturmChunk; c += 256) {
                // past n: positive multiples of the last minor (no sign change)
                const double u = c0 + c > 0 && c < cn ? ldexp(e[c0 + c - 1], -ex) : 0.0;
                de[c] = make_double2(c < cn ? ldexp(d[c0 + c], -ex) : 4.0, u * u);
            }
            __syncthreads();
            for (int c = 0; c < cn; c += 8) {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const double2 t = de[c + u];
                    double q = fma(t.x - x, p1, -(t.y * p0));
                    // a zero minor takes the sign that makes the step a change
                    if (q == 0.0) q = -1e-30 * p1;
                    cnt += (int)((__builtin_bit_cast(uint64_t, q) ^ __builtin_bit_cast(uint64_t, p1)) >> 63);
                    p0 = p1;
                    p1 = q;
                }
                const int s = -__builtin_amdgcn_frexp_exp(fmax(fabs(p0), fabs(p1)));
                p0 = ldexp(p0, s);
                p1 = ldexp(p1, s);
            }
        }
        const unsigned above = (unsigned)(__ballot(cnt >= want) >> (lane & 48)) & 0xFFFFu;
        const int f = above ? __ffs(above) - 1 : 16;  // first point above lambda_i
        const double nlo = f == 0 ? lo : lo + step * f, nhi = f == 16 ? hi : lo + step * (f + 1);
        lo = nlo;
        hi = nhi;
    }
    if ((lane & 15) == 0 && i < n) sb.out(b)[3 * (long)sb.nmax + i] = norm == 0.0 ? 0.0 : ldexp(0.5 * (lo + hi), ex);
}

hipError_t launch_spectra(const SpectralBatch& sb, const SpectralJob* host_jobs, hipStream_t st) {
    int tiles = 0, nb = 1;
    for (int b = 0; b < sb.count; ++b) {
        const int nt = (host_jobs[b].n + 63) / 64;
        tiles = host_jobs[b].tile0 + nt * (nt + 1) / 2;
        nb = std::max(nb, (int)host_jobs[b].n);
    }
    hipLaunchKernelGGL(gram_kernel, dim3(tiles), dim3(256), 0, st, sb);
    if (nb > kSpectralMax) {
        tridiagonalize_large(sb, nb, st);
    } else {
        if (3 * (size_t)(nb + 2) * sizeof(double) > 64 * 1024)
            for (auto f : {(const void*)tri_step_kernel<true>, (const void*)tri_step_kernel<false>}) {
                const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 256);
                if (e != hipSuccess) return e;
            }
        for (int j = -1; j < tail_step(nb); ++j) {
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
        hipLaunchKernelGGL(tri_tail_kernel, dim3(sb.count), dim3(kTailTY * kTailTX), 0, st, sb);
    }
    hipLaunchKernelGGL(sturm_kernel, dim3((nb + 15) / 16, sb.count), dim3(256), 0, st, sb);
    return hipGetLastError();
}

}  // namespace sgd
