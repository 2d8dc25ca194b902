// Branch GEMMs of the active units in fp32: C = A . B^T with fused epilogues, and the
// dtype dispatch (the bf16 path is in gemm_bf16.hip).
//
// fp32 path: matrix-core kernels (32 x 32 and 16 x 16 tiles) with K split across the waves of a
// workgroup (the fp32 workload is small and latency-bound); gated and rotary epilogues are
// bf16 only.
#include "common.h"
#include "kernels.h"

namespace sgd {

// ---------------------------------------------------------------------------- epilogue

template <typename OutT>
struct Epi {
    EpiParams p;

    int tw = 0;  // EP_HEADS: projection of this tile (0 q, 1 k, 2 v^T); tiles never straddle two

    // bias and (EP_RESID) stream value of an element, loaded ahead of its single() or single_vt()
    bool pre = false;
    float pre_bias = 0.f, pre_h = 0.f;
    __device__ __forceinline__ void preload(int row, int n) {
        pre = true;
        if (p.bias) pre_bias = p.bias[n];
        if (p.kind == EP_RESID) pre_h = (p.hin ? p.hin : p.h)[(long)row * p.d + n];
    }
    __device__ __forceinline__ float bias_at(int n) const { return pre ? pre_bias : p.bias[n]; }

    __device__ __forceinline__ void store_qk(int row, int nn, float v) const {
        const int b = row / p.ntok, tok = row - b * p.ntok;
        const int hh = nn / p.dh, j = nn - hh * p.dh;
        OutT* base = (OutT*)(tw == 0 ? p.q : p.k);
        ElemIO<OutT>::store(base + (((long)b * p.H + hh) * p.np + tok) * p.dh + j, v);
    }
    __device__ __forceinline__ void store_vt(int row, int nn, float v) const {
        const int b = row / p.ntok, tok = row - b * p.ntok;
        const int hh = nn / p.dh, j = nn - hh * p.dh;
        ElemIO<OutT>::store((OutT*)p.vt + (((long)b * p.H + hh) * p.dh + j) * p.np + tok, v);
    }
    // V^T columns of a tile (tw == 2): their own store loop
    __device__ __forceinline__ void single_vt(int row, int n, float v) const {
        if (p.bias) v += bias_at(n);
        store_vt(row, n - (tw - p.which0) * p.d, v);
    }

    // one element at product column n
    __device__ __forceinline__ void single(int row, int n, float v) const {
        switch (p.kind) {
            case EP_HEADS: {
                if (p.bias) v += bias_at(n);
                store_qk(row, n - (tw - p.which0) * p.d, v);
                break;
            }
            case EP_ACT: {
                if (p.bias) v += bias_at(n);
                ElemIO<OutT>::store((OutT*)p.out + (long)row * p.ldo + n, apply_act(p.act, v));
                break;
            }
            case EP_RESID: {
                if (p.bias) v += bias_at(n);
                if (p.gate) v *= p.gate[(long)(row / p.ntok) * p.gate_ld + n];
                const long idx = (long)row * p.d + n;
                const float hn = (pre ? pre_h : (p.hin ? p.hin : p.h)[idx]) + v;
                if (!p.z) p.h[idx] = hn;
                else {
                    const int tok = row % p.ntok;
                    if (tok >= p.r0 && tok < p.r1) p.z[idx] = p.alpha * p.z[idx] - p.beta * hn;
                }
                if (p.delta_mode == 1) p.delta[idx] = v;
                else if (p.delta_mode == 2) p.delta[idx] = p.delta[idx] + v;
                if (p.hcopy) ElemIO<OutT>::store((OutT*)p.hcopy + idx, hn);
                break;
            }
            case EP_SKIP: {
                if (p.bias) v += bias_at(n);
                const long idx = (long)row * p.d + n;
                if (p.delta_mode == 1) v = v + p.delta[idx];
                p.h[idx] = v;
                if (p.hcopy) ElemIO<OutT>::store((OutT*)p.hcopy + idx, v);
                break;
            }
            default: break;
        }
    }
};

// ---------------------------------------------------------------------------- fp32 MFMA

// 32 x 32 output tile per workgroup on v_mfma_f32_32x32x2_f32 (fp32 products, fp32
// accumulation).  The NW waves split K: k unit u (8 values) goes to wave u % NW, and in a unit
// lanes 0-31 contract k = 8u .. 8u+3 and lanes 32-63 k = 8u+4 .. 8u+7 (four MFMA steps), so each
// lane reads one float4 of its A row and one of its B row per unit, straight from global
// memory.  The partial tiles meet in LDS and are summed in wave order (deterministic); every
// thread then applies the epilogue to its elements. 
constexpr int kF32Chunk = 4;  // k units per wave per pass (loads issued together)
template <int NW>
__global__ __launch_bounds__(NW * 64) void gemm_f32_kernel(GemmArgs g, EpiParams ep) {
    __shared__ float red[NW][32 * 33];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 31, half = lane >> 5;
    const int nt_m = (g.M + 31) / 32;
    const int tm = blockIdx.x % nt_m, tn = blockIdx.x / nt_m;
    const int m0 = tm * 32;
    // operand rows of this lane: A row m0 + col (clamped; rows past M are never stored), B row
    // of product column col of the tile
    const int ar = min(m0 + col, g.M - 1);
    const long br = (long)tn * 32 + col;
    const float* bp = (const float*)g.B + br * g.ldb + half * 4;
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    const int units = g.K / 8;
    for (int u0 = wave; u0 < units; u0 += NW * kF32Chunk) {
        f32x4 av[kF32Chunk], bv[kF32Chunk];
#pragma unroll
        for (int c = 0; c < kF32Chunk; ++c) {
            const int u = u0 + c * NW;
            const int k = u * 8 + half * 4;
            if (u < units) {
                const bool second = g.A1 && k >= g.K0;
                const float* ap = second ? (const float*)g.A1 + (long)ar * g.lda1 + (k - g.K0)
                                         : (const float*)g.A0 + (long)ar * g.lda0 + k;
                av[c] = *(const f32x4*)ap;
                bv[c] = *(const f32x4*)(bp + u * 8);
            } else {
                av[c] = f32x4{0.f, 0.f, 0.f, 0.f};
                bv[c] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
#pragma unroll
        for (int c = 0; c < kF32Chunk; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av[c][e], bv[c][e], acc, 0, 0, 0);
    }
    // lane l holds tile column l % 32 and, for register r, row (r / 4) * 8 + (l / 32) * 4 + r % 4
#pragma unroll
    for (int r = 0; r < 16; ++r) red[wave][((r >> 2) * 8 + half * 4 + (r & 3)) * 33 + col] = acc[r];
    __syncthreads();
    auto tile_at = [&](int row, int c) {
        float v = red[0][row * 33 + c];
#pragma unroll
        for (int w = 1; w < NW; ++w) v += red[w][row * 33 + c];
        return v;
    };
    Epi<float> e{ep};
    if (ep.kind == EP_HEADS) e.tw = ep.which0 + (tn * 32) / ep.d;
#pragma unroll
    for (int idx = tid; idx < 1024; idx += NW * 64) {
        const int row = idx >> 5, c = idx & 31;
        if (m0 + row >= g.M) continue;
        const float v = tile_at(row, c);
        if (ep.kind == EP_HEADS && e.tw == 2) e.single_vt(m0 + row, tn * 32 + c, v);
        else e.single(m0 + row, tn * 32 + c, v);
    }
}

// 16 x 16 output tile per workgroup on v_mfma_f32_16x16x4_f32, for products with few tiles, which are
// bound by round trips of loads: four times the workgroups of the 32 x 32 kernel, so a wave's K range is
// one or two round trips (256 x 256 outputs: K = 256 5.9 -> 3.5 us, K = 1024 11.6 -> 6.3).  The NW waves split K in units of 16 (unit u goes to wave u % NW; in a unit lane
// group l / 16 contracts k = 16 u + 4 (l / 16) .. + 3, one float4 of its A row and one of its B row,
// over four MFMA steps).  The partial tiles meet in LDS and are summed in wave order; thread t < 256
// finishes element t, whose bias and stream value it loads before the K loop.
template <int NW>
__global__ __launch_bounds__(NW * 64) void gemm_f32_small_kernel(GemmArgs g, EpiParams ep) {
    __shared__ float red[NW][16 * 17];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 15, grp = lane >> 4;
    const int nt_m = (g.M + 15) / 16;
    const int tm = blockIdx.x % nt_m, tn = blockIdx.x / nt_m;
    const int m0 = tm * 16;
    const int ar = min(m0 + col, g.M - 1);  // rows past M are never stored
    const long br = (long)tn * 16 + col;
    const float* bp = (const float*)g.B + br * g.ldb + grp * 4;
    Epi<float> e{ep};
    if (ep.kind == EP_HEADS) e.tw = ep.which0 + (tn * 16) / ep.d;
    // the thread's element: V^T tiles walk tokens, all others columns
    const bool vt = ep.kind == EP_HEADS && e.tw == 2;
    const int er = vt ? tid & 15 : (tid >> 4) & 15, ec = vt ? (tid >> 4) & 15 : tid & 15;
    const bool mine = tid < 256 && m0 + er < g.M;
    if (mine) e.preload(m0 + er, tn * 16 + ec);
    f32x4 acc{0.f, 0.f, 0.f, 0.f};
    const int units = g.K / 16;
    constexpr int CH = 4;
    for (int u0 = wave; u0 < units; u0 += NW * CH) {
        f32x4 av[CH], bv[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int u = u0 + c * NW, k = u * 16 + grp * 4;
            if (u < units) {
                const bool second = g.A1 && k >= g.K0;
                const float* ap = second ? (const float*)g.A1 + (long)ar * g.lda1 + (k - g.K0)
                                         : (const float*)g.A0 + (long)ar * g.lda0 + k;
                av[c] = *(const f32x4*)ap;
                bv[c] = *(const f32x4*)(bp + u * 16);
            } else {
                av[c] = f32x4{0.f, 0.f, 0.f, 0.f};
                bv[c] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[c][i], bv[c][i], acc, 0, 0, 0);
    }
    // lane l holds tile column l % 16 and rows 4 (l / 16) + r
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][(grp * 4 + r) * 17 + col] = acc[r];
    __syncthreads();
    auto tile_at = [&](int row, int c) {
        float v = red[0][row * 17 + c];
#pragma unroll
        for (int w = 1; w < NW; ++w) v += red[w][row * 17 + c];
        return v;
    };
    if (!mine) return;
    const float v = tile_at(er, ec);
    if (vt) e.single_vt(m0 + er, tn * 16 + ec, v);
    else e.single(m0 + er, tn * 16 + ec, v);
}

// ---------------------------------------------------------------------------- dispatch

bool gemm_shape_ok(int dtype, const GemmArgs& g, const EpiParams& e, int tile) {
    if (g.M <= 0 || g.N <= 0 || g.K <= 0) return false;
    if (dtype == 1) return gemm_bf16_shape_ok(g, e, tile);
    if (g.ksplit != 1 || e.kind == EP_PARTIAL) return false;  // split products: bf16 only
    if (g.K % 16 || g.N % 64) return false;
    if (g.A1 && (g.K0 % 16)) return false;
    if (e.kind == EP_GATED || (e.kind == EP_HEADS && (e.rope || e.d % 64))) return false;
    return true;
}

hipError_t launch_gemm(int dtype, const GemmArgs& g, const EpiParams& e, hipStream_t st, int tile) {
    if (dtype == 1) return launch_gemm_bf16(g, e, st, tile);
    if (g.ksplit != 1 || e.kind == EP_PARTIAL) return hipErrorInvalidValue;
    const int nt_m = (g.M + 31) / 32, nt_n = g.N / 32;
    // What a launch takes is a start plus its round trips of loads per CU.  16 x 16 tiles while two
    // of them a CU cover the product (256 x 256 x 1024: 6.4 us against 11.8; 400 x 512 x 512, 208 tiles
    // of 32 x 32: 10.0 against 7.8).  Past that 32 x 32 tiles: eight waves up to one tile a CU (256 x 1024
    // x 256 5.2 us, four waves 6.1), four where K is deep (224 x 640 x 2560 28.2, sixteen 29.4).  With more
    // tiles the waves of several share a CU, and a pass of 32 values of K a wave that K does not fill
    // costs more than more waves give: four (400 x 1536 x 384 15.6, eight 17.0), eight for many tiles
    // whose K is whole passes (1040 x 1536 x 512 37.8, four 40.0), sixteen for many tiles of deep
    // K (912 x 1152 x 4608 215, four 245; but 416 x 1152 x 2304, 468 tiles, 48.2, four 45.9).
    if (nt_m * nt_n <= 128) {
        const dim3 grid(((g.M + 15) / 16) * (g.N / 16));
        if (g.K > 256) hipLaunchKernelGGL(gemm_f32_small_kernel<8>, grid, dim3(512), 0, st, g, e);
        else hipLaunchKernelGGL(gemm_f32_small_kernel<4>, grid, dim3(256), 0, st, g, e);
        return hipGetLastError();
    }
    const int n = nt_m * nt_n;
    const dim3 grid(n);
    const int nw = g.K >= 2048 ? (n >= 512 ? 16 : 4) : n <= 256 || (n >= 1024 && g.K % 256 == 0) ? 8 : 4;
    if (nw == 16) hipLaunchKernelGGL(gemm_f32_kernel<16>, grid, dim3(1024), 0, st, g, e);
    else if (nw == 8) hipLaunchKernelGGL(gemm_f32_kernel<8>, grid, dim3(512), 0, st, g, e);
    else hipLaunchKernelGGL(gemm_f32_kernel<4>, grid, dim3(256), 0, st, g, e);
    return hipGetLastError();
}

}  // namespace sgd
