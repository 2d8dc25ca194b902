// Branch GEMMs of the active units in bf16: C = A . B^T on the CDNA4 matrix cores
// (v_mfma_f32_32x32x16_bf16, fp32 accumulation) with the unit's epilogue fused.
//
// Two kernels share the epilogue, both with operands loaded straight into LDS and two wave groups
// that alternate between reading fragments and MFMAs: gemm_pp_kernel, whose groups share large block
// tiles, and gemm_pk_kernel, small tiles for products that cannot fill the chip with large ones, whose
// groups split K.
//
// Epilogue.  Straight from the accumulators: the loader orders the weight rows so that what a
// store or a pair of columns needs sits in one lane (see the epilogue).
#include <algorithm>
#include <type_traits>
#include <utility>

#include "common.h"
#include "kernels.h"
#include "tile_order.h"

namespace sgd {

// Rotary head projections: the q and k product columns of each head are taken in the order
// (0, dh/2, 1, dh/2 + 1, ...), so the two dims of every rotary pair are adjacent columns and a
// block tile of any even width holds whole pairs.  Column n of the product is weight row (and
// bias entry) rope_row(n); v columns (n >= vstart) keep their order.
__device__ __forceinline__ long rope_row(long n, int dh, long vstart) {
    if (n >= vstart) return n;
    const int hl = (int)(n % dh);
    return n - hl + ((hl & 1) ? dh / 2 + hl / 2 : hl / 2);
}

template <int I> using IntC = std::integral_constant<int, I>;

// f(IntC<0>{}), ..., f(IntC<N - 1>{})
template <class Fn, int... I>
__device__ __forceinline__ void static_for_impl(Fn& f, std::integer_sequence<int, I...>) {
    (f(IntC<I>{}), ...);
}
template <int N, class Fn>
__device__ __forceinline__ void static_for(Fn&& f) {
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// --------------------------------------------------------------------------- epilogue
//
// Straight from the accumulators, without LDS or a barrier.  In the MFMA output layout lane l holds
// column l % 32 of a 32 x 32 block and, in registers 4 q .. 4 q + 3, its rows 8 q + 4 (l / 32) +
// 0..3.  Which product column a block column stands for is the loader's choice (it picks the weight
// row for each LDS row), and it is made so that a lane's values of one row are neighbours
// (tile_col): two blocks side by side give a lane columns 2 l and 2 l + 1.  The pairs of a rotary
// head and the gate and up columns of a gated MLP then meet in one lane, four consecutive tokens of
// a V^T row are four registers, and a transpose of the four rows within a quad of lanes (DPP) leaves
// each lane eight neighbouring columns of one row: 16-byte stores that fill whole 128-byte lines.
//
// Every batch of rows loads its global operands (h, delta, gate) before its first store: a loop
// that alternates them waits for each store (vmcnt counts both).
//
// An epilogue's cost beyond its bytes is what a launch with K = 64 shows (8192 rows, 256 x 256
// tiles): staged through LDS in 128-row chunks 28.9 us plain, 42.7 GELU(erf), 21.5 residual (1024
// columns), 56.5 GEGLU; this one 24.1, 34.8, 19.9 and 48.4.

__device__ __forceinline__ void store_bf16x4(bf16* dst, const float v[4]) {
    bf16x4 s;
    s[0] = f2bf(v[0]); s[1] = f2bf(v[1]); s[2] = f2bf(v[2]); s[3] = f2bf(v[3]);
    *(bf16x4*)dst = s;
}

template <int ACT>
__device__ __forceinline__ float act_fn(float x) {
    if (ACT == ACT_GELU_ERF) return gelu_erf(x);
    if (ACT == ACT_GELU_TANH) return gelu_tanh(x);
    if (ACT == ACT_SILU) return silu(x);
    return x;
}

// calls f(tag) with the activation as a compile-time constant
template <class Fn>
__device__ __forceinline__ void with_act(int act, Fn&& f) {
    switch (act) {
        case ACT_GELU_ERF: f(IntC<ACT_GELU_ERF>{}); break;
        case ACT_GELU_TANH: f(IntC<ACT_GELU_TANH>{}); break;
        case ACT_SILU: f(IntC<ACT_SILU>{}); break;
        default: f(IntC<ACT_NONE>{}); break;
    }
}

// Column (of a wave's TN x 32) of lane column l in MFMA block j: blocks are taken in pairs whose
// columns interleave; a last single block keeps its order.
template <int TN>
__device__ __forceinline__ int tile_col(int j, int l) {
    return j < TN / 2 * 2 ? j / 2 * 64 + 2 * l + (j & 1) : j * 32 + l;
}
// Gated products: hidden column (of a wave's TN x 16) of lane column l in block j, and whether it
// is the up half.  Gate block j pairs with up block j + (TN + 1) / 2; the middle block of an odd TN
// holds 16 gate columns and then their 16 up columns.
template <int TN>
__device__ __forceinline__ int gated_col(int j, int l, bool& up) {
    constexpr int H = TN / 2, UP = (TN + 1) / 2;
    if (TN % 2 && j == H) { up = l >= 16; return H * 32 + (l & 15); }
    up = j >= UP;
    return (up ? j - UP : j) * 32 + l;
}

// Weight row of LDS row r of column tile tn (every kernel's B loader)
template <class C>
__device__ __forceinline__ long weight_row(const EpiParams& ep, int F, int tn, int r) {
    const int w = r / C::WN, x = r - w * C::WN, j = x >> 5, l = x & 31;
    if (ep.kind == EP_GATED) {
        bool up;
        const int c = gated_col<C::TN>(j, l, up);
        return (long)tn * (C::BN / 2) + w * (C::WN / 2) + c + (up ? F : 0);
    }
    const long n = (long)tn * C::BN + w * C::WN + tile_col<C::TN>(j, l);
    if (ep.kind == EP_HEADS && ep.rope) return rope_row(n, ep.dh, (long)(2 - ep.which0) * ep.d);
    return n;
}

// 4 x 4 transpose of 32-bit values within each quad of lanes: v[k] of lane q becomes v[q] of lane k
// (DPP quad permutes; every lane of the quad active).
__device__ __forceinline__ uint32_t quad_xor1(uint32_t x) { return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true); }
__device__ __forceinline__ uint32_t quad_xor2(uint32_t x) { return __builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, true); }
__device__ __forceinline__ void quad_transpose(uint32_t (&v)[4], int l) {
    const bool o1 = l & 1, o2 = l & 2;
    uint32_t a[4];
#pragma unroll
    for (int k = 0; k < 4; k += 2) {
        const uint32_t x = quad_xor1(v[k + 1]), y = quad_xor1(v[k]);
        a[k] = o1 ? x : v[k];
        a[k + 1] = o1 ? v[k + 1] : y;
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const uint32_t x = quad_xor2(a[k + 2]), y = quad_xor2(a[k]);
        v[k] = o2 ? x : a[k];
        v[k + 2] = o2 ? a[k + 2] : y;
    }
}
__device__ __forceinline__ uint32_t pack_bf16(float x, float y) {
    bf16x2 s;
    s[0] = f2bf(x);
    s[1] = f2bf(y);
    return __builtin_bit_cast(uint32_t, s);
}

// two bf16 values at p (4-byte aligned)
__device__ __forceinline__ void put2(bf16* p, const float* v) { *(uint32_t*)p = pack_bf16(v[0], v[1]); }

template <class C>
__device__ __forceinline__ void epilogue(f32x16 (&acc)[C::TM][C::TN], const GemmArgs& g, const EpiParams& ep, int m0,
                                         int tn, int wm, int wn, int split) {
    constexpr int TM = C::TM, TN = C::TN;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // nothing derived from it is computed before the main loop
    const int l = tid & 31, lhalf = (tid >> 5) & 1, lq = l & 3;
    // first of the four rows of registers 4 q .. 4 q + 3 of MFMA block i
    auto row_of = [&](int i, int q) { return m0 + C::block_row(wm, i) + lhalf * 4 + q * 8; };
    // sample of a row: floor((row + 0.5) / ntok) in fp32 is exact while row < 2^21
    const float rntok = 1.0f / (float)ep.ntok;
    auto sample_of = [&](int row) { return (int)(((float)row + 0.5f) * rntok); };
    // bf16 values o[u] of rows row0 + u, u < 4, column c of this lane -> after a quad transpose the
    // lane holds row row0 + l % 4 and four columns of its quad, from c - l % 4 on (dst: that place)
    auto quad_single = [&](const float (&o)[4]) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = __float_as_uint(o[u]);
        quad_transpose(v, l);
        return u32x2{pack_bf16(__uint_as_float(v[0]), __uint_as_float(v[1])),
                     pack_bf16(__uint_as_float(v[2]), __uint_as_float(v[3]))};
    };

    if (ep.kind == EP_GATED) {
        const int F = ep.F, c0 = tn * (C::BN / 2) + wn * (C::WN / 2);
        float b[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            bool up;
            const int c = gated_col<TN>(j, l, up);
            b[j] = ep.bias ? ep.bias[c0 + c + (up ? F : 0)] : 0.f;
        }
        with_act(ep.act, [&](auto actc) {
            constexpr int ACT = decltype(actc)::value;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int row = row_of(i, q) + lq;
                    bf16* const out = (bf16*)ep.out + (long)row * ep.ldo + c0 + (l & ~3);
                    constexpr int H = TN / 2;
                    // gate block j pairs with up block j + (TN + 1) / 2
#pragma unroll
                    for (int j = 0; j < H; ++j) {
                        constexpr int UP = (TN + 1) / 2;
                        float o[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            o[u] = act_fn<ACT>(acc[i][j][q * 4 + u] + b[j]) * (acc[i][UP + j][q * 4 + u] + b[UP + j]);
                        const u32x2 s = quad_single(o);
                        if (row < g.M) *(u32x2*)(out + j * 32) = s;
                    }
                    if constexpr (TN % 2) {
                        // lanes 0..15 of the middle block hold gate columns, 16..31 their up columns
                        float o[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const float x = acc[i][H][q * 4 + u] + b[H];
                            const float y = __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(x), 0x401F));  // l ^ 16
                            o[u] = act_fn<ACT>(x) * y;
                        }
                        const u32x2 s = quad_single(o);
                        if (l < 16 && row < g.M) *(u32x2*)(out + H * 32) = s;
                    }
                }
        });
        return;
    }

    // column groups: a pair of neighbouring columns from blocks j, j + 1 (V = 2), or one column of a
    // last single block (V = 1)
    const int nw = tn * C::BN + wn * C::WN;  // the wave's first product column
    auto groups = [&](auto&& f) {
        if constexpr (TN >= 2) f(IntC<0>{}, IntC<2>{}, nw + 2 * l);
        if constexpr (TN >= 4) f(IntC<2>{}, IntC<2>{}, nw + 64 + 2 * l);
        if constexpr (TN % 2) f(IntC<TN - 1>{}, IntC<1>{}, nw + (TN - 1) * 32 + l);
    };
    // rows row0 .. row0 + 3 of a group's columns n .. n + V - 1 as bf16: one store of the quad's 4 V
    // columns of row row0 + l % 4 at dst (a pointer to column n - V (l % 4) of that row); cols: how
    // many of them exist (a multiple of 4; <= 0: none)
    auto store_quad = [&](auto vc, bf16* dst, const float (*o)[decltype(vc)::value], int cols) {
        constexpr int V = decltype(vc)::value;
        if constexpr (V == 2) {
            uint32_t v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = pack_bf16(o[u][0], o[u][1]);
            quad_transpose(v, l);
            if (cols >= 8) *(u32x4*)dst = u32x4{v[0], v[1], v[2], v[3]};
            else if (cols >= 4) *(u32x2*)dst = u32x2{v[0], v[1]};
        } else {
            const float t[4] = {o[0][0], o[1][0], o[2][0], o[3][0]};
            const u32x2 s = quad_single(t);
            if (cols >= 4) *(u32x2*)dst = s;
        }
    };

    if (ep.kind == EP_ACT) {
        groups([&](auto jc, auto vc, int n) {
            constexpr int J = decltype(jc)::value, V = decltype(vc)::value;
            float b[V];
#pragma unroll
            for (int v = 0; v < V; ++v) b[v] = ep.bias && n < g.N ? ep.bias[n + v] : 0.f;
            const int nq = n - V * lq;
            with_act(ep.act, [&](auto actc) {
                constexpr int ACT = decltype(actc)::value;
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    float rb[V] = {};
                    int bs = -1;  // sample whose row bias rb holds (rows rise: it changes rarely)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int row0 = row_of(i, q);
                        float o[4][V];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            if (ACT == ACT_NONE && ep.rowbias) {
                                const int s = sample_of(min(row0 + u, g.M - 1));
                                if (s != bs && n < g.N)
#pragma unroll
                                    for (int v = 0; v < V; ++v) rb[v] = ep.rowbias[(long)s * ep.rowbias_ld + n + v];
                                bs = s;
                            }
#pragma unroll
                            for (int v = 0; v < V; ++v) o[u][v] = act_fn<ACT>((acc[i][J + v][q * 4 + u] + b[v]) + rb[v]);
                        }
                        const int row = row0 + lq;
                        store_quad(vc, (bf16*)ep.out + (long)row * ep.ldo + nq, o, row < g.M ? g.N - nq : 0);
                    }
                }
            });
        });
    } else if (ep.kind == EP_HEADS) {
        const int vstart = (2 - ep.which0) * ep.d;  // first v^T product column
        bf16* const qptr = (bf16*)ep.q;
        bf16* const kptr = (bf16*)ep.k;
        bf16* const vt = (bf16*)ep.vt;
        groups([&](auto jc, auto vc, int n) {
            constexpr int J = decltype(jc)::value, V = decltype(vc)::value;
            if (n >= g.N) return;
            if (n >= vstart) {
                // V^T: four consecutive tokens of a row per store
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    const int nv = n + v - vstart, vh = nv / ep.dh, vj = nv - vh * ep.dh;
                    const float bv = ep.bias ? ep.bias[n + v] : 0.f;
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const int row0 = row_of(i, q);
                            if (row0 >= g.M) continue;
                            const int bs0 = sample_of(row0), tok0 = row0 - bs0 * ep.ntok;
                            float o[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u) o[u] = acc[i][J + v][q * 4 + u] + bv;
                            if (tok0 % 4 == 0 && tok0 + 3 < ep.ntok && row0 + 3 < g.M) {
                                store_bf16x4(vt + (((long)bs0 * ep.H + vh) * ep.dh + vj) * ep.np + tok0, o);
                            } else {
                                // two tokens at a time where they stay together (an even sample length)
#pragma unroll
                                for (int u = 0; u < 4; u += 2) {
                                    const int row = row0 + u;
                                    if (row >= g.M) break;
                                    const int bs = sample_of(row), tok = row - bs * ep.ntok;
                                    bf16* const dst = vt + (((long)bs * ep.H + vh) * ep.dh + vj) * ep.np + tok;
                                    if (tok % 2 == 0 && tok + 1 < ep.ntok && row + 1 < g.M) {
                                        put2(dst, o + u);
                                        continue;
                                    }
                                    dst[0] = f2bf(o[u]);
                                    if (row + 1 >= g.M) break;
                                    const int bs1 = sample_of(row + 1), tok1 = row + 1 - bs1 * ep.ntok;
                                    vt[(((long)bs1 * ep.H + vh) * ep.dh + vj) * ep.np + tok1] = f2bf(o[u + 1]);
                                }
                            }
                        }
                }
                return;
            }
            // q / k columns.  Quads of lanes share one head: d, vstart and dh are multiples of 8 (or
            // dh of 4 only, whose columns are stored one by one below)
            const int proj = ep.which0 + n / ep.d, nn = n - (proj - ep.which0) * ep.d;
            const int hh = nn / ep.dh, j = nn - hh * ep.dh;
            bf16* const base = (proj == 0 ? qptr : kptr) + (long)hh * ep.np * ep.dh;
            const long bstride = (long)ep.H * ep.np * ep.dh;
            if (!ep.rope) {
                float b[V];
#pragma unroll
                for (int v = 0; v < V; ++v) b[v] = ep.bias ? ep.bias[n + v] : 0.f;
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int row0 = row_of(i, q);
                        float o[4][V];
#pragma unroll
                        for (int u = 0; u < 4; ++u)
#pragma unroll
                            for (int v = 0; v < V; ++v) o[u][v] = acc[i][J + v][q * 4 + u] + b[v];
                        if (ep.dh % 8 == 0) {
                            const int row = row0 + lq, bs = sample_of(row), tok = row - bs * ep.ntok;
                            store_quad(vc, base + bs * bstride + (long)tok * ep.dh + j - V * lq, o, row < g.M ? 8 : 0);
                        } else {
#pragma unroll
                            for (int u = 0; u < 4; ++u) {
                                const int row = row0 + u, bs = sample_of(row), tok = row - bs * ep.ntok;
                                if (row >= g.M) break;
#pragma unroll
                                for (int v = 0; v < V; ++v) base[bs * bstride + (long)tok * ep.dh + j + v] = f2bf(o[u][v]);
                            }
                        }
                    }
                return;
            }
            // rotary columns (pairs adjacent, see rope_row): product columns 2 p and 2 p + 1 of a
            // head hold dims p and p + dh/2.  A group of two is a whole pair; in a single block the
            // pair's other column is in lane l ^ 1.  The angle is the fractional turn of token x
            // inverse frequency (v_sin_f32 / v_cos_f32 take turns); the turn count carries ~1e-4 rad
            // of fp32 rounding at 1024 tokens, far below the bf16 resolution of the output
            const int hd = ep.dh / 2, pj = j / 2;
            float b[V];
#pragma unroll
            for (int v = 0; v < V; ++v) b[v] = ep.bias ? ep.bias[rope_row(n + v, ep.dh, vstart)] : 0.f;
            const float invt = exp2f(-(2.0f * (float)pj / (float)ep.dh) * ep.rope_log2_theta) * 0.159154943091895336f;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int row0 = row_of(i, q);
                    float o1[4], o2[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int bs = sample_of(row0 + u), tok = row0 + u - bs * ep.ntok;
                        const float t = (float)tok * invt;
                        const float f = t - rintf(t);
                        const float sn = __builtin_amdgcn_sinf(f), cs = __builtin_amdgcn_cosf(f);
                        const float x = acc[i][J][q * 4 + u] + b[0];
                        if constexpr (V == 2) {
                            const float x2 = acc[i][J + 1][q * 4 + u] + b[1];
                            o1[u] = x * cs - x2 * sn;
                            o2[u] = x2 * cs + x * sn;
                        } else {
                            const float y = __uint_as_float(quad_xor1(__float_as_uint(x)));
                            o1[u] = (l & 1) ? x * cs + y * sn : x * cs - y * sn;
                        }
                    }
                    if constexpr (V == 2) {
                        // four neighbouring pairs of token row0 + l % 4: dims p .. p + 3 and their partners
                        const u32x2 s1 = quad_single(o1), s2 = quad_single(o2);
                        const int row = row0 + lq, bs = sample_of(row), tok = row - bs * ep.ntok;
                        bf16* const dst = base + bs * bstride + (long)tok * ep.dh + pj - lq;
                        if (row < g.M) {
                            *(u32x2*)dst = s1;
                            *(u32x2*)(dst + hd) = s2;
                        }
                    } else {
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int row = row0 + u, bs = sample_of(row), tok = row - bs * ep.ntok;
                            if (row < g.M) base[bs * bstride + (long)tok * ep.dh + pj + ((l & 1) ? hd : 0)] = f2bf(o1[u]);
                        }
                    }
                }
        });
    } else {
        // EP_RESID: v = (acc + bias) [* gate]; h = hin + v; delta = v | delta += v; hcopy = bf16(h);
        //           the last of a step: z <- alpha z - beta h in place of h's store
        // EP_SKIP:  h = acc + bias [+ cached delta]; hcopy = bf16(h)
        // EP_PARTIAL: part s = acc (+ bias in range 0), as EP_SKIP into h + s * part_stride
        // Lane pairs (V = 2) or quads (V = 1) exchange rows, so a lane handles four neighbouring
        // columns of a row: two rows per lane and register group (V = 2), or one (V = 1).
        const bool resid = ep.kind == EP_RESID;
        const bool rd_delta = resid ? ep.delta_mode == 2 : ep.kind == EP_SKIP && ep.delta_mode == 1;
        float* const hdst = ep.kind == EP_PARTIAL ? ep.h + (long)split * ep.part_stride : ep.h;
        const float* const hsrc = ep.hin ? ep.hin : ep.h;
        groups([&](auto jc, auto vc, int n) {
            constexpr int J = decltype(jc)::value, V = decltype(vc)::value;
            constexpr int RL = V;                     // rows per lane and register group
            constexpr int QB = 2;                     // register groups per load batch
            const int n4 = V == 2 ? n - 2 * (l & 1) : n - lq;  // first of the lane's four columns
            const int nl = min(n4, g.N - 4);          // clamped: every load stays inside
            float b[V];
#pragma unroll
            for (int v = 0; v < V; ++v) b[v] = ep.bias && split == 0 && n < g.N ? ep.bias[n + v] : 0.f;
            // row of the lane's w-th row in register group q of block i
            auto lane_row = [&](int i, int q, int w) { return row_of(i, q) + (V == 2 ? 2 * w + (l & 1) : lq); };
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int q0 = 0; q0 < 4; q0 += QB) {
                    f32x4 hv[QB][RL], dv[QB][RL], gt[QB][RL], zv[QB][RL];
#pragma unroll
                    for (int q = 0; q < QB; ++q)
#pragma unroll
                        for (int w = 0; w < RL; ++w) {
                            const int row = min(lane_row(i, q0 + q, w), g.M - 1);
                            const long idx = (long)row * ep.d + nl;
                            hv[q][w] = resid ? *(const f32x4*)(hsrc + idx) : f32x4{0.f, 0.f, 0.f, 0.f};
                            zv[q][w] = ep.z ? *(const f32x4*)(ep.z + idx) : f32x4{0.f, 0.f, 0.f, 0.f};
                            dv[q][w] = rd_delta ? *(const f32x4*)(ep.delta + idx) : f32x4{0.f, 0.f, 0.f, 0.f};
                            gt[q][w] = ep.gate ? *(const f32x4*)(ep.gate + (long)sample_of(row) * ep.gate_ld + nl)
                                               : f32x4{1.f, 1.f, 1.f, 1.f};
                        }
#pragma unroll
                    for (int q = 0; q < QB; ++q) {
                        f32x4 x[RL];
                        if constexpr (V == 2) {
                            // rows 2 w (even lanes) and 2 w + 1 (odd lanes): own pair and the neighbour's
#pragma unroll
                            for (int w = 0; w < 2; ++w) {
                                const int r = (q0 + q) * 4 + 2 * w;
#pragma unroll
                                for (int v = 0; v < 2; ++v) {
                                    const float e = acc[i][J + v][r] + b[v], o = acc[i][J + v][r + 1] + b[v];
                                    const float pe = __uint_as_float(quad_xor1(__float_as_uint(e)));
                                    const float po = __uint_as_float(quad_xor1(__float_as_uint(o)));
                                    x[w][v] = (l & 1) ? po : e;
                                    x[w][2 + v] = (l & 1) ? o : pe;
                                }
                            }
                        } else {
                            uint32_t t[4];
#pragma unroll
                            for (int u = 0; u < 4; ++u) t[u] = __float_as_uint(acc[i][J][(q0 + q) * 4 + u] + b[0]);
                            quad_transpose(t, l);
#pragma unroll
                            for (int u = 0; u < 4; ++u) x[0][u] = __uint_as_float(t[u]);
                        }
#pragma unroll
                        for (int w = 0; w < RL; ++w) {
                            const int row = lane_row(i, q0 + q, w);
                            if (row >= g.M || n4 >= g.N) continue;
                            const long idx = (long)row * ep.d + n4;
                            f32x4 xx = x[w], hn;
                            if (ep.gate) xx = xx * gt[q][w];
                            const f32x4 dn = dv[q][w] + xx;
                            hn = resid ? hv[q][w] + xx : rd_delta ? dn : xx;
                            if (!ep.z) {
                                *(f32x4*)(hdst + idx) = hn;
                            } else {
                                const int tok = row - sample_of(row) * ep.ntok;
                                if (tok >= ep.r0 && tok < ep.r1) *(f32x4*)(ep.z + idx) = zv[q][w] * ep.alpha - hn * ep.beta;
                            }
                            if (resid && ep.delta_mode == 1) *(f32x4*)(ep.delta + idx) = xx;
                            if (resid && ep.delta_mode == 2) *(f32x4*)(ep.delta + idx) = dn;
                            if (ep.hcopy) {
                                const float t[4] = {hn[0], hn[1], hn[2], hn[3]};
                                store_bf16x4((bf16*)ep.hcopy + idx, t);
                            }
                        }
                    }
                }
        });
    }
}

// --------------------------------------------------------------------------- large tiles
//
// 256 x BN and 128 x 256 block tiles, eight waves, 64-deep k tiles.  Operands go from global memory straight
// into LDS (buffer_load ... lds, 16 bytes a lane: no staging registers, no ds_write issue); the
// XOR swizzle of a row's chunks is applied to the lanes' global addresses, since a wave's LDS
// destination is contiguous.  The waves form two groups (one wave of each per SIMD) that run the
// same phases half a phase apart: while one group issues its MFMAs the other reads its fragments
// and issues loads, so each SIMD always has one wave in the matrix cores.
//
// A k tile is two phases.  Phase 0 reads the fragments of A's first half of rows and of all of B,
// phase 1 those of the second half; a phase's LDS regions are free once both groups have read them, so
// they are refilled two k tiles ahead, one to two tiles before they are read (128 KB of LDS at
// BN = 256 keep ~1.5 tiles in flight).  Each wave waits for its own loads by count (vmcnt), one
// phase before the data is read, and the barrier in between makes that true of every wave.
//
// What bounds it: the matrix cores' power.  On the 8192^3 product the loop runs at 1830 TFLOP/s on
// zero operands and 1350 on Gaussian ones (hipBLASLt: 1440); the register-staged loop it replaced
// reached 1220-1245 there.  Same run, plain bf16 store, 256 x 256 tiles, before -> after:
// 8192 x 10240 x 1280 241 -> 201 us, 1024 x 24576 x 4096 222 -> 182, 8192 x 4608 x 1152 116 -> 90,
// 8192 x 1280 x 5120 121 -> 102.  With the epilogues (one op in a loop, weights cold): GELU(tanh)
// 8192 x 4608 x 1152 107 -> 93 us, GELU(erf) 8256 x 4096 x 1024 104 -> 92, GEGLU 8192 x 10240 x 1280
// 213 -> 196, residual 8192 x 1280 x 5120 106 -> 97, 3 x 3 convolution 8192 x 1280 channels 237 -> 211;
// in a whole step the clock falls with the power drawn and half of that remains.  Two workgroups of 128 x 256 per CU instead (epilogues overlapped)
// ran at 1030 on 8192^3: they move 1.5x the operand bytes.

template <int BM_, int BN_, int WGM_, int WGN_, int ST_ = 2>
struct PPCfg {
    static constexpr int BM = BM_, BN = BN_, WGM = WGM_, WGN = WGN_, ST = ST_, NT = 512, NW = 8;
    static constexpr int BH = BM / 2, HP = BH / 64;      // rows and load parts (64 rows) of each half
    static constexpr int RW = BH / WGM;                  // a wave's rows of each half
    static constexpr int CB = RW / 32, TM = 2 * CB;      // MFMA row blocks per half, per wave
    static constexpr int WN = BN / WGN, TN = WN / 32;
    static constexpr int BP = BN / 64, BL = BP / 2;      // B parts (64 rows) per tile; those loaded in phase 1
    static constexpr int A_HALF = BH * 128, A_STAGE = BM * 128, B_STAGE = BN * 128, B_LDS = ST * A_STAGE;
    static constexpr int LDS_BYTES = B_LDS + ST * B_STAGE;
    __device__ static __forceinline__ int block_row(int wm, int i) { return (i / CB) * BH + wm * RW + (i % CB) * 32; }
    static_assert(WGM * WGN == NW && RW % 32 == 0 && WN % 32 == 0 && BN % 64 == 0 && BH % 64 == 0, "wave tile");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS");
};

// 16 bytes a lane from buffer r at voff + soff to LDS byte address lds + 16 lane (voff out of the
// descriptor's range: zeros).  Counted in vmcnt; the caller waits.  m0 (the LDS address) is used by
// nothing else in these kernels.
__device__ __forceinline__ void dma16(unsigned lds, unsigned voff, u32x4 r, unsigned soff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds), "v"(voff), "s"(r), "s"(__builtin_amdgcn_readfirstlane(soff)) : "memory");
}
template <int N>
__device__ __forceinline__ void vm_wait() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// workgroup barrier without the waits of __syncthreads (outstanding loads stay in flight)
__device__ __forceinline__ void raw_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
// buffer descriptor as four scalars (nothing is in range when bytes = 0)
__device__ __forceinline__ u32x4 buf_desc(const void* base, unsigned bytes) {
    const uint64_t p = (uint64_t)base;
    u32x4 r;
    r[0] = __builtin_amdgcn_readfirstlane((unsigned)p);
    r[1] = __builtin_amdgcn_readfirstlane((unsigned)(p >> 32));
    r[2] = bytes;
    r[3] = 0x00020000;
    return r;
}

template <class C, bool CONV, bool SPLIT>
__global__ __launch_bounds__(C::NT, 2) void gemm_pp_kernel(GemmArgs g, EpiParams ep) {
    __shared__ __attribute__((aligned(1024))) char lds[C::LDS_BYTES];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nt_m = (g.M - g.m_begin + C::BM - 1) / C::BM;
    const int nt_n = (g.N + C::BN - 1) / C::BN;
    // split K: workgroup b takes K range b / T of tile b % T (T tiles)
    const int split = SPLIT ? (int)blockIdx.x / (nt_m * nt_n) : 0;
    int tm, tn;
    tile_at(tile_position((int)blockIdx.x - split * nt_m * nt_n, nt_m * nt_n), nt_m, nt_n, g.band, tm, tn);
    const int m0 = g.m_begin + tm * C::BM;
    const int F = g.N / 2;
    const int KT = (SPLIT ? g.K / g.ksplit : g.K) / 64;
    const int kbase = SPLIT ? split * (g.K / g.ksplit) : 0;
    const unsigned bytesA = (unsigned)((long)g.M * g.lda0 * 2), bytesB = (unsigned)((long)g.N * g.ldb * 2);
    constexpr unsigned OOB = 0xFFFFFF00u;

    // Load part p of an operand tile: rows 64 p + 8 wave + lane / 8, the 16-byte chunk of the row
    // that belongs at LDS position lane % 8.  The first HP A parts are the first half's rows.
    const int prow = wave * 8 + (lane >> 3);
    const int pch = ((lane & 7) ^ ((prow >> 1) & 7)) * 16;  // swizzle key of the row: 64-row parts keep it
    unsigned aoff[2 * C::HP], boff[C::BP];  // both A sources share the row pitch
    int gpos[CONV ? 2 * C::HP : 1];         // convolution: grid position (y << 16 | x) of the A row
#pragma unroll
    for (int p = 0; p < 2 * C::HP; ++p) {
        const int row = m0 + p * 64 + prow;
        aoff[p] = (unsigned)((long)row * g.lda0 * 2 + pch);
        if constexpr (CONV) {
            const int side = g.conv_side, pix = row % (side * side), y = pix / side;
            gpos[p] = (y << 16) | (pix - y * side);
        }
    }
#pragma unroll
    for (int p = 0; p < C::BP; ++p) {
        boff[p] = (unsigned)(weight_row<C>(ep, F, tn, p * 64 + prow) * g.ldb * 2 + pch);
    }
    const unsigned lw = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds + wave * 1024;
    // k tile t's half h of A into stage t % ST (stage and part numbers are compile-time constants
    // at every call); tiles at or past K load nothing but still count
    auto load_a = [&](int t, int stage, int h) {
        const bool in = t < KT;
        const int k0 = t * 64;
        const unsigned l = lw + stage * C::A_STAGE + h * C::A_HALF;
        if constexpr (CONV) {
            // the k tile lies inside one tap (conv_c % 64 == 0): shift the row by the tap's grid
            // offset, or load zeros (an out-of-range offset) where it leaves the grid
            const int tap = k0 / g.conv_c, c0 = k0 - tap * g.conv_c;
            const int ky = tap / 3, dy = ky - 1, dx = tap - ky * 3 - 1;
            const int shift = (dy * g.conv_side + dx) * (int)g.lda0 * 2;
            const u32x4 r = buf_desc(g.A0, bytesA);
#pragma unroll
            for (int i = 0; i < C::HP; ++i) {
                const int yy = (gpos[h * C::HP + i] >> 16) + dy, xx = (gpos[h * C::HP + i] & 0xFFFF) + dx;
                const bool ok = in && (unsigned)yy < (unsigned)g.conv_side && (unsigned)xx < (unsigned)g.conv_side;
                dma16(l + i * 8192, ok ? (unsigned)((int)aoff[h * C::HP + i] + shift) : OOB, r, in ? c0 * 2 : 0);
            }
        } else {
            const bool second = g.A1 && k0 >= g.K0;
            const u32x4 r = buf_desc(second ? g.A1 : g.A0, in ? bytesA : 0);
            const unsigned so = in ? (second ? (k0 - g.K0) * 2 : (kbase + k0) * 2) : 0;
#pragma unroll
            for (int i = 0; i < C::HP; ++i) dma16(l + i * 8192, aoff[h * C::HP + i], r, so);
        }
    };
    auto load_b = [&](int t, int stage, auto from, auto to) {
        const bool in = t < KT;
        const u32x4 r = buf_desc(g.B, in ? bytesB : 0);
#pragma unroll
        for (int p = decltype(from)::value; p < decltype(to)::value; ++p)
            dma16(lw + C::B_LDS + stage * C::B_STAGE + p * 8192, boff[p], r, in ? (kbase + t * 64) * 2 : 0);
    };

    const int wm = wave / C::WGN, wn = wave % C::WGN, wn0 = wn * C::WN;
    const int lrow = lane & 31, lhalf = lane >> 5;
    const char *fa[4], *fb[4];  // fragment addresses of the four 16-deep k steps
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int sw = ((q * 2 + lhalf) ^ ((lrow >> 1) & 7)) << 4;
        fa[q] = lds + (wm * C::RW + lrow) * 128 + sw;
        fb[q] = lds + C::B_LDS + (wn0 + lrow) * 128 + sw;
    }
    f32x16 acc[C::TM][C::TN];
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    bf16x8 af[C::CB][4], bfr[C::TN][4];
    auto read_a = [&](int stage, int h) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < C::CB; ++i)
                af[i][q] = *(const bf16x8*)(fa[q] + stage * C::A_STAGE + h * C::A_HALF + i * 4096);
    };
    auto read_b = [&](int stage) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < C::TN; ++j) bfr[j][q] = *(const bf16x8*)(fb[q] + stage * C::B_STAGE + j * 4096);
    };
    auto mfmas = [&](int h) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < C::CB; ++i)
#pragma unroll
                for (int j = 0; j < C::TN; ++j)
                    acc[h * C::CB + i][j] =
                        __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i][q], bfr[j][q], acc[h * C::CB + i][j], 0, 0, 0);
    };
    // end of a phase's reads: the fragments are in registers before the other group may refill
    auto turn = [&] {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        raw_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr IntC<0> B0{};
    constexpr IntC<C::BL> BLO{};
    constexpr IntC<C::BP> B1{};
    // load order per tile: A half 0 and the first BL B parts (phase 1 of tile t - ST), the other B
    // parts and A half 1 (phase 0 of tile t - ST + 1).  Before phase 1 of tile t is read, at most the
    // loads issued after its A half 1 may be outstanding: ST - 1 tiles' worth; before phase 0 of
    // tile t, those after its B parts: its A half 1, ST - 1 phases 1 and ST - 2 phases 0.
    constexpr int L1 = C::HP + C::BL, L0 = C::BP - C::BL + C::HP;  // loads of phases 1 and 0
    constexpr int W0 = (C::ST - 1) * (L0 + L1), W1 = C::HP + (C::ST - 1) * L1 + (C::ST - 2) * L0;
    static_assert(W0 < 64, "vmcnt");
    static_for<C::ST - 1>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        load_a(s, s, 0);
        load_b(s, s, B0, B1);
        load_a(s, s, 1);
    });
    load_a(C::ST - 1, C::ST - 1, 0);
    load_b(C::ST - 1, C::ST - 1, B0, BLO);
    vm_wait<W1>();
    raw_barrier();
    const bool late = wave >= 4;  // the second group runs half a phase behind
    if (late) raw_barrier();
    auto tile = [&](int t, auto sc) {
        constexpr int s = decltype(sc)::value, prev = (s + C::ST - 1) % C::ST;
        __builtin_amdgcn_sched_barrier(0);
        read_b(s);
        read_a(s, 0);
        load_b(t + C::ST - 1, prev, BLO, B1);
        load_a(t + C::ST - 1, prev, 1);
        vm_wait<W0>();
        turn();
        mfmas(0);
        __builtin_amdgcn_sched_barrier(0);
        raw_barrier();
        __builtin_amdgcn_sched_barrier(0);
        read_a(s, 1);
        load_a(t + C::ST, s, 0);
        load_b(t + C::ST, s, B0, BLO);
        vm_wait<W1>();
        turn();
        mfmas(1);
        __builtin_amdgcn_sched_barrier(0);
        raw_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int t = 0; t < KT; t += C::ST)
        static_for<C::ST>([&](auto sc) {
            if (t + decltype(sc)::value < KT) tile(t + decltype(sc)::value, sc);
        });
    if (!late) raw_barrier();
    vm_wait<0>();
    // the epilogue's arguments are read again here, through an address the compiler cannot see
    // through, instead of holding their scalars (and what follows from them) across the main loop
    const char __attribute__((address_space(4)))* args =
        (const char __attribute__((address_space(4)))*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    constexpr int EP_AT = (sizeof(GemmArgs) + alignof(EpiParams) - 1) / alignof(EpiParams) * alignof(EpiParams);
    epilogue<C>(acc, *(const GemmArgs*)(const char*)args, *(const EpiParams*)(const char*)(args + EP_AT), m0, tn, wm, wn,
                split);
}

// --------------------------------------------------------------------------- K-group kernel
//
// Small tiles (64 x 64 to 128 x 128) for products with too few tiles to fill the chip: what such a
// product takes is its chain of k tiles, so the two wave groups split K instead of the tile.  Group
// g takes k tiles g, g + 2, ..., each with a full set of accumulators (four waves, 2 x 2), and the
// groups run half a step apart as above: while one issues a tile's MFMAs the other reads its
// fragments.  The MFMA slot also issues the loads that refill the stage just read, one between two
// MFMAs.  At the end the groups exchange halves of their sums through LDS and each finishes its own
// half of the rows (64-row tiles: group 0 finishes all).
//
// A step's length is the LDS's: a 128 x 128 tile takes 0.37 us per 64-deep k tile on its own (64 KB
// of fragment reads, 32 KB of loads landing at 64 bytes a cycle), 64 x 64 0.17.  The 128 x 128
// kernel with register-staged loads that it replaced took 0.37-0.46.  Residual products, before ->
// after (weights cold): 200 x 4096 x 12288 100 -> 46 us, 512 x 1152 x 4608 34 -> 19, 625 x 1280 x 5120
// 40 -> 21; 3 x 3 convolution on 625 positions of 1280 channels 100 -> 38.

template <int BM_, int BN_, int S_>
struct PKCfg {
    static constexpr int BM = BM_, BN = BN_, S = S_, NT = 512;
    static constexpr int TMW = BM / 64, TN = BN / 64, WN = BN / 2;  // a wave's MFMA blocks, columns
    static constexpr int TM = 1;                                    // row blocks per wave in the epilogue
    static constexpr int AP = BM / 32, BP = BN / 32, P = AP + BP;   // loads per wave and k tile
    static constexpr int A_BYTES = BM * 128, STAGE = (BM + BN) * 128;
    static constexpr int LDS_BYTES = 2 * S * STAGE;
    // two-block waves: group g finishes row block g of its wave row (row index wm * 2 + g)
    __device__ static __forceinline__ int block_row(int w, int) { return w * 32; }
    static_assert((TMW == 1 || TMW == 2) && P <= 4 * TMW * TN && (S - 1) * P < 64, "k-group tile");
    static_assert(LDS_BYTES <= 160 * 1024 && LDS_BYTES >= BM * BN * 4, "LDS: stages, then the exchange");
};

template <class C, bool CONV, bool SPLIT>
__global__ __launch_bounds__(C::NT, 2) void gemm_pk_kernel(GemmArgs g, EpiParams ep) {
    __shared__ __attribute__((aligned(1024))) char lds[C::LDS_BYTES];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), grp = wave >> 2, gw = wave & 3;
    const int nt_m = (g.M - g.m_begin + C::BM - 1) / C::BM;
    const int nt_n = (g.N + C::BN - 1) / C::BN;
    const int split = SPLIT ? (int)blockIdx.x / (nt_m * nt_n) : 0;
    int tm, tn;
    tile_at(tile_position((int)blockIdx.x - split * nt_m * nt_n, nt_m * nt_n), nt_m, nt_n, g.band, tm, tn);
    const int m0 = g.m_begin + tm * C::BM;
    const int KT = (SPLIT ? g.K / g.ksplit : g.K) / 64;
    const int kbase = SPLIT ? split * (g.K / g.ksplit) : 0;
    const unsigned bytesA = (unsigned)((long)g.M * g.lda0 * 2), bytesB = (unsigned)((long)g.N * g.ldb * 2);
    constexpr unsigned OOB = 0xFFFFFF00u;

    // load part p: rows 32 p + 8 gw + lane / 8 of an operand tile, swizzled chunk as in the large-tile kernel
    const int prow = gw * 8 + (lane >> 3);
    const int pch = ((lane & 7) ^ ((prow >> 1) & 7)) * 16;
    unsigned off[C::P];
    int gpos[CONV ? C::AP : 1];
#pragma unroll
    for (int p = 0; p < C::AP; ++p) {
        const int row = m0 + p * 32 + prow;
        off[p] = (unsigned)((long)row * g.lda0 * 2 + pch);
        if constexpr (CONV) {
            const int side = g.conv_side, pix = row % (side * side), y = pix / side;
            gpos[p] = (y << 16) | (pix - y * side);
        }
    }
#pragma unroll
    for (int p = 0; p < C::BP; ++p)
        off[C::AP + p] = (unsigned)(weight_row<C>(ep, g.N / 2, tn, p * 32 + prow) * g.ldb * 2 + pch);
    const unsigned lw = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds + grp * (C::S * C::STAGE) + gw * 1024;
    // the group's i-th k tile into stage i % S; tiles at or past K load zeros
    struct Src { u32x4 ra, rb; unsigned sa, sb; int dy, dx, shift; bool in; };
    auto source = [&](int i) {
        const int t = 2 * i + grp, k0 = t * 64;
        Src c;
        c.in = t < KT;
        c.sb = c.in ? (kbase + k0) * 2 : 0;
        c.rb = buf_desc(g.B, c.in ? bytesB : 0);
        c.dy = c.dx = c.shift = 0;
        if constexpr (CONV) {
            const int tap = k0 / g.conv_c, ky = tap / 3;
            c.dy = ky - 1;
            c.dx = tap - ky * 3 - 1;
            c.shift = (c.dy * g.conv_side + c.dx) * (int)g.lda0 * 2;
            c.ra = buf_desc(g.A0, c.in ? bytesA : 0);
            c.sa = c.in ? (k0 - tap * g.conv_c) * 2 : 0;
        } else {
            const bool second = g.A1 && k0 >= g.K0;
            c.ra = buf_desc(second ? g.A1 : g.A0, c.in ? bytesA : 0);
            c.sa = c.in ? (second ? (k0 - g.K0) * 2 : (kbase + k0) * 2) : 0;
        }
        return c;
    };
    auto load = [&](const Src& c, unsigned l, int p) {
        if (p < C::AP) {
            unsigned o = off[p];
            if constexpr (CONV) {
                const int yy = (gpos[p] >> 16) + c.dy, xx = (gpos[p] & 0xFFFF) + c.dx;
                const bool ok = (unsigned)yy < (unsigned)g.conv_side && (unsigned)xx < (unsigned)g.conv_side;
                o = ok ? (unsigned)((int)o + c.shift) : OOB;
            }
            dma16(l + p * 4096, o, c.ra, c.sa);
        } else {
            dma16(l + C::A_BYTES + (p - C::AP) * 4096, off[p], c.rb, c.sb);
        }
    };

    const int wm = gw >> 1, wn = gw & 1;
    const int lrow = lane & 31, lhalf = lane >> 5;
    const char *fa[4], *fb[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int sw = ((q * 2 + lhalf) ^ ((lrow >> 1) & 7)) << 4;
        fa[q] = lds + grp * (C::S * C::STAGE) + (wm * (C::BM / 2) + lrow) * 128 + sw;
        fb[q] = lds + grp * (C::S * C::STAGE) + C::A_BYTES + (wn * C::WN + lrow) * 128 + sw;
    }
    f32x16 acc[C::TMW][C::TN];
#pragma unroll
    for (int i = 0; i < C::TMW; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

#pragma unroll
    for (int s = 0; s < C::S; ++s) {
        const Src c = source(s);
#pragma unroll
        for (int p = 0; p < C::P; ++p) load(c, lw + s * C::STAGE, p);
    }
    constexpr int W = (C::S - 1) * C::P;  // the next tile has landed; those after it may be in flight
    vm_wait<W>();
    raw_barrier();
    if (grp) raw_barrier();
    const int steps = (KT + 1) / 2;  // the same for both groups: barriers match
    int stage = 0;
    for (int i = 0; i < steps; ++i) {
        const int so = stage * C::STAGE;
        bf16x8 af[C::TMW][4], bfr[C::TN][4];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int x = 0; x < C::TMW; ++x) af[x][q] = *(const bf16x8*)(fa[q] + so + x * 4096);
#pragma unroll
            for (int x = 0; x < C::TN; ++x) bfr[x][q] = *(const bf16x8*)(fb[q] + so + x * 4096);
        }
        const Src c = source(i + C::S);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        raw_barrier();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int x = 0; x < C::TMW; ++x)
#pragma unroll
                for (int y = 0; y < C::TN; ++y) {
                    acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[x][q], bfr[y][q], acc[x][y], 0, 0, 0);
                    const int slot = (q * C::TMW + x) * C::TN + y;
                    if (slot < C::P) {
                        __builtin_amdgcn_sched_barrier(0);
                        load(c, lw + so, slot);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
        vm_wait<W>();
        __builtin_amdgcn_sched_barrier(0);
        raw_barrier();
        stage = stage + 1 == C::S ? 0 : stage + 1;
    }
    if (!grp) raw_barrier();
    vm_wait<0>();  // the loads past K have written their zeros before LDS is used for the exchange
    raw_barrier();
    // exchange: register group of four of block (x, y), register quad q, of wave gw: 1 KB a wave
    f32x4* const ex = (f32x4*)lds;
    auto slot_of = [&](int y, int q, int half) { return (((half * 4 + gw) * C::TN + y) * 4 + q) * 64 + lane; };
    f32x16 sum[1][C::TN];
    if constexpr (C::TMW == 2) {
#pragma unroll
        for (int y = 0; y < C::TN; ++y)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f32x4 o;  // the other group's row block
#pragma unroll
                for (int u = 0; u < 4; ++u) o[u] = grp ? acc[0][y][q * 4 + u] : acc[1][y][q * 4 + u];
                ex[slot_of(y, q, grp)] = o;
            }
        __syncthreads();
#pragma unroll
        for (int y = 0; y < C::TN; ++y)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 o = ex[slot_of(y, q, grp ^ 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u) sum[0][y][q * 4 + u] = (grp ? acc[1][y][q * 4 + u] : acc[0][y][q * 4 + u]) + o[u];
            }
    } else {
        if (grp) {
#pragma unroll
            for (int y = 0; y < C::TN; ++y)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    f32x4 o;
#pragma unroll
                    for (int u = 0; u < 4; ++u) o[u] = acc[0][y][q * 4 + u];
                    ex[slot_of(y, q, 0)] = o;
                }
        }
        __syncthreads();
        if (grp) return;
#pragma unroll
        for (int y = 0; y < C::TN; ++y)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 o = ex[slot_of(y, q, 0)];
#pragma unroll
                for (int u = 0; u < 4; ++u) sum[0][y][q * 4 + u] = acc[0][y][q * 4 + u] + o[u];
            }
    }
    const char __attribute__((address_space(4)))* args =
        (const char __attribute__((address_space(4)))*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    constexpr int EP_AT = (sizeof(GemmArgs) + alignof(EpiParams) - 1) / alignof(EpiParams) * alignof(EpiParams);
    epilogue<C>(sum, *(const GemmArgs*)(const char*)args, *(const EpiParams*)(const char*)(args + EP_AT), m0, tn,
                wm * C::TMW + (C::TMW == 2 ? grp : 0), wn, split);
}

// --------------------------------------------------------------------------- dispatch

namespace {
using T256x256 = PPCfg<256, 256, 2, 4>;  // 128 x 64 wave tiles
using T256x192 = PPCfg<256, 192, 4, 2>;  // 64 x 96
using T256x128 = PPCfg<256, 128, 4, 2, 3>;  // 64 x 64
using T128x256 = PPCfg<128, 256, 2, 4, 3>;  // 64 x 64
using T128x128 = PKCfg<128, 128, 2>;
using T128x64 = PKCfg<128, 64, 3>;
using T64x64 = PKCfg<64, 64, 4>;

// tile id -> block shape and what a tile takes: us per 64-deep k tile with the chip nearly empty and
// with every CU busy, and us for its start and epilogue.  Fitted to 690 products (1 to 8300 rows, 256 to
// 49152 columns, K 256 to 12288, weights cold) timed with every tile, where the choice made from them is
// within 0.3 % of the fastest tile on average and 20 % at worst (6572 x 1280 x 256, gated: 16.3 us, 13.7);
// fitted to either half of them, within 0.6 % on the other's average.  The values before them, from 62
// products, chose 1.5 % slower on average (6592 x 4096 x 512, gated: 45 us, now 37.5; 896 x 384 x 384: 8.1,
// now 6.8).  They rank tiles and are no model of a launch's time: small cold products take up to twice the
// cost (2 x 2048 x 8192 on 64 x 64 tiles 28.6 us, cost 15.2), and t0 of two small tiles is below what one
// takes on its own (0.37 us for 128 x 128, 0.17 for 64 x 64, bound by the LDS).
struct Shape { int bm, bn; double t0, t1, fix; };
Shape tile_shape(int tile) {
    switch (tile) {
        case 1: return {256, 256, 0.74, 1.5, 7.5};
        case 2: return {256, 128, 0.58, 0.89, 2.7};
        case 3: return {128, 256, 0.73, 0.97, 1.9};
        case 4: return {128, 128, 0.29, 0.59, 2.1};
        case 5: return {256, 192, 0.61, 1.3, 4.9};
        case 6: return {128, 64, 0.30, 0.41, 1.9};
        case 7: return {64, 64, 0.10, 0.245, 2.4};
        default: return {0, 0, 0.0, 0.0, 0.0};
    }
}
// a second launch for the tail rows
constexpr double kTailLaunch = 5.5;
}  // namespace

static bool conv_tile(int tile) { return tile == 2 || (tile >= 4 && tile <= 7); }

// Time (us) of one launch of `tile` over `rows` rows: one workgroup per CU, so n tiles take n / 256
// full rounds and a last one whose k tiles are faster the emptier it is.  Infinite when the epilogue
// cannot use the tile.  Past one round, one or two row tiles are bound by the weights, read once from HBM at
// kHbm in all and kCuHbm a CU (64 x 24576 x 4096: 384 tiles of 64 x 64 52 us, 192 of 128 x 128 45); one
// round, even a whole one, has its rate in t1 (64 x 32768 x 3072: 256 tiles of 128 x 128 40 us, 128 of 128 x
// 256 51; 64 x 16384 x 3072: 256 tiles of 64 x 64 21 us, 128 of 128 x 64 23).
// And a grid that the XCDs do not divide keeps no neighbouring tiles on one XCD (tile_order.h): where the
// activations are past two L2s, tiles of up to 128 columns, which read the most operand bytes, pay for it (2560 x
// 2560 weights, 256 x 128 tiles: 7680 rows, 600 tiles, 123 us, 7936, 620 tiles, 162).
constexpr double kHbm = 5e6, kCuHbm = 25e3;  // bytes a us
constexpr double kUneven = 1.2;
static double tile_cost(int tile, long rows, const GemmArgs& g, const EpiParams& e, int ks = 1) {
    const Shape s = tile_shape(tile);
    if (!s.bm) return 1e300;
    if (g.conv_side > 0 && !conv_tile(tile)) return 1e300;
    if (e.kind == EP_GATED && g.N % s.bn) return 1e300;
    const long nm = (rows + s.bm - 1) / s.bm, nn = (g.N + s.bn - 1) / s.bn, tiles = nm * nn * ks;
    const long full = tiles / 256, rem = tiles % 256;
    const double kt = g.K / (64.0 * ks);
    auto round = [&](long n) {  // n workgroups side by side
        double t = s.t0 + (s.t1 - s.t0) * (double)n / 256.0;
        if (tiles > 256 && nm <= 2) t = std::max(t, s.bn * 128.0 / nm / std::min(kCuHbm, kHbm / (double)n));
        return kt * t + s.fix;
    };
    double t = full * round(256);
    if (rem) t += round(rem);
    return (nm * nn) % kXcds && s.bn <= 128 && rows * g.K * 2 > (8L << 20) ? t * kUneven : t;
}

// Automatic choice: the tile with the least cost (200 x 4096 x 12288: 64 x 64 tiles, 256 of them, 45 us
// against 99 with 64 of 128 x 128; 1024 x 4096 x 4096: one round of 128 x 128).  When the rows leave a
// short tail past the last whole 256-row tile (U-ViT: 32 x 258 = 8256 = 32 x 256 + 64 rows), the tail
// can go to a second launch of small tiles, so the main launch fills whole rounds instead of starting
// a third one for 64 rows (8256 x 4096 x 1024: 90 us against 100).  The tail reads the weights once more
// (545 x 15360 x 2560: 62 us split, 52 on 256 x 192 tiles; 1088 x 7680 x 2560 64 and 59; but 1298 x 12288
// x 4096 135 and 166).
GemmPlan gemm_bf16_plan(const GemmArgs& g, const EpiParams& e) {
    GemmPlan best{1, g.M, 0};
    double best_t = 1e300;
    for (int tile = 1; tile <= kGemmTiles; ++tile) {
        const double t = tile_cost(tile, g.M, g, e);
        if (t < best_t) { best_t = t; best = GemmPlan{tile, g.M, 0}; }
    }
    const int tail = g.M % 256;
    if (g.M > 512 && tail > 0 && tail <= 128 && g.conv_side == 0) {
        for (int tile = 1; tile <= kGemmTiles; ++tile) {
            if (tile_shape(tile).bm != 256) continue;
            const double tm = tile_cost(tile, g.M - tail, g, e);
            for (int tt = 1; tt <= kGemmTiles; ++tt) {
                if (tile_shape(tt).bm > 128) continue;
                const double t = tm + std::max(tile_cost(tt, tail, g, e), 2.0 * g.N * g.K / kHbm) + kTailLaunch;
                if (t < best_t * 0.99) { best_t = t; best = GemmPlan{tile, g.M - tail, tt}; }
            }
        }
    }
    return best;
}

// Tiles of a product in K ranges (EP_PARTIAL)
static bool split_tile(int tile) { return tile == 2 || tile == 4 || tile == 6 || tile == 7; }
static int partial_tile(const GemmArgs& g, const EpiParams& e) {
    int best = 2;
    double best_t = 1e300;
    for (int tile = 1; tile <= kGemmTiles; ++tile) {
        if (!split_tile(tile)) continue;
        const double t = tile_cost(tile, g.M, g, e, g.ksplit);
        if (t < best_t) { best_t = t; best = tile; }
    }
    return best;
}

// Two K ranges where they shorten a residual product by more than their fp32 partials cost: the
// pre-norm that adds them to the stream itself reads and writes 12 bytes a value more than the
// residual epilogue moves (at ~4 TB/s) and is charged 1 us.  Large products gain from larger tiles that
// still fill the chip (LLaDA's 1024 x 4096 x 12288: 256 x 128 tiles over half of K, 100 us against
// 120), small ones from a chain of k tiles half as long (200 x 256 x 8192).
int gemm_bf16_ksplit(const GemmArgs& g) {
    if (g.A1 || g.conv_side > 0 || g.K % 128) return 1;
    EpiParams e;
    e.kind = EP_RESID;
    e.d = g.N;
    const GemmPlan p = gemm_bf16_plan(g, e);
    if (p.tail_tile) return 1;
    GemmArgs gs = g;
    gs.ksplit = 2;
    const double extra = 12.0 * g.M * g.N / 4e6 + 1.0;
    return tile_cost(partial_tile(gs, e), g.M, gs, e, 2) + extra < 0.95 * tile_cost(p.tile, g.M, g, e) ? 2 : 1;
}

static bool aligned(const void* p, unsigned a) { return ((uintptr_t)p % a) == 0; }

bool gemm_bf16_shape_ok(const GemmArgs& g, const EpiParams& e, int tile) {
    if (tile == 0 && e.kind == EP_PARTIAL) tile = partial_tile(g, e);
    if (tile == 0) {
        const GemmPlan p = gemm_bf16_plan(g, e);
        if (p.tail_tile && !gemm_bf16_shape_ok(g, e, p.tail_tile)) return false;
        tile = p.tile;
    }
    if (g.m_begin != 0) return false;  // set by the dispatcher only
    // vector accesses of the loader and the epilogue: 16-byte operand rows and fp32 vectors,
    // 8-byte bf16 output groups
    if (!aligned(g.A0, 16) || !aligned(g.A1, 16) || !aligned(g.B, 16) || !aligned(e.bias, 16) ||
        !aligned(e.gate, 16) || e.gate_ld % 4 || !aligned(e.h, 16) || !aligned(e.hin, 16) || !aligned(e.z, 16) || !aligned(e.delta, 16) ||
        !aligned(e.out, 8) || !aligned(e.hcopy, 8) || !aligned(e.q, 8) || !aligned(e.k, 8) || !aligned(e.vt, 2))
        return false;
    const Shape s = tile_shape(tile);
    if (!s.bm) return false;
    if (g.M >= (1 << 21)) return false;  // the epilogue's fp32 row -> sample split is exact below
    if (g.conv_side > 0) {
        const long area = (long)g.conv_side * g.conv_side;
        if (!conv_tile(tile) || g.A1 || g.conv_c % 64 || g.K != 9 * g.conv_c || g.lda0 != g.conv_c ||
            g.M % area || g.conv_side >= (1 << 15))
            return false;
    }
    if (!aligned(e.rowbias, 16) || e.rowbias_ld % 4 || (e.rowbias && e.act != ACT_NONE)) return false;
    if (g.K % 64 || (g.A1 && (g.K0 % 64 || g.lda1 != g.lda0))) return false;
    if (g.N % 4 || g.lda0 % 8 || (g.A1 && g.lda1 % 8) || g.ldb % 8) return false;  // 16-byte rows
    if (e.kind == EP_GATED && (g.N % s.bn || e.ldo % 4)) return false;
    if (e.kind == EP_ACT && e.ldo % 4) return false;
    if ((e.kind == EP_RESID || e.kind == EP_SKIP || e.kind == EP_PARTIAL) && (g.N != e.d)) return false;
    if (g.ksplit < 1 || (g.ksplit > 1) != (e.kind == EP_PARTIAL) || (g.ksplit > 1 && !split_tile(tile))) return false;
    if (e.kind == EP_PARTIAL && (g.A1 || g.conv_side > 0 || g.K % (64 * g.ksplit) || e.gate || e.hcopy ||
                                 e.delta_mode || (long)e.part_stride < (long)g.M * g.N || e.part_stride % 4))
        return false;
    if (e.kind == EP_HEADS) {
        if (e.d % 32 || e.dh % 4) return false;  // V^T from whole 32-column MFMA blocks
        if (e.rope && e.dh % 8) return false;  // eight-column pair groups within one head
    }
    const long lim = 0xFFFFFF00L;  // 32-bit buffer ranges below the loader's out-of-range offset
    if ((long)g.M * g.lda0 * 2 > lim || (g.A1 && (long)g.M * g.lda1 * 2 > lim) || (long)g.N * g.ldb * 2 > lim)
        return false;
    return true;
}

template <class C> struct is_pk : std::false_type {};
template <int BM, int BN, int S> struct is_pk<PKCfg<BM, BN, S>> : std::true_type {};

template <class C, bool CONV = false, bool SPLIT = false>
static hipError_t run_tile(const GemmArgs& g, const EpiParams& e, hipStream_t st) {
    const int nt_m = (g.M - g.m_begin + C::BM - 1) / C::BM, nt_n = (g.N + C::BN - 1) / C::BN;
    GemmArgs ga = g;
    ga.band = tile_band(nt_m, nt_n, C::BM, C::BN);
    const dim3 grid(nt_m * nt_n * (SPLIT ? g.ksplit : 1));
    if constexpr (is_pk<C>::value) hipLaunchKernelGGL((gemm_pk_kernel<C, CONV, SPLIT>), grid, dim3(C::NT), 0, st, ga, e);
    else hipLaunchKernelGGL((gemm_pp_kernel<C, CONV, SPLIT>), grid, dim3(C::NT), 0, st, ga, e);
    return hipGetLastError();
}

static hipError_t launch_tile(const GemmArgs& g, const EpiParams& e, hipStream_t st, int tile) {
    if (g.conv_side > 0) {
        switch (tile) {  // implicit-GEMM convolution: the tiles with registers to spare
            case 2: return run_tile<T256x128, true>(g, e, st);
            case 4: return run_tile<T128x128, true>(g, e, st);
            case 5: return run_tile<T256x192, true>(g, e, st);
            case 6: return run_tile<T128x64, true>(g, e, st);
            case 7: return run_tile<T64x64, true>(g, e, st);
            default: return hipErrorInvalidValue;
        }
    }
    if (g.ksplit > 1) {  // K ranges (EP_PARTIAL)
        switch (tile) {
            case 2: return run_tile<T256x128, false, true>(g, e, st);
            case 4: return run_tile<T128x128, false, true>(g, e, st);
            case 6: return run_tile<T128x64, false, true>(g, e, st);
            case 7: return run_tile<T64x64, false, true>(g, e, st);
            default: return hipErrorInvalidValue;
        }
    }
    switch (tile) {
        case 1: return run_tile<T256x256>(g, e, st);
        case 2: return run_tile<T256x128>(g, e, st);
        case 3: return run_tile<T128x256>(g, e, st);
        case 4: return run_tile<T128x128>(g, e, st);
        case 5: return run_tile<T256x192>(g, e, st);
        case 6: return run_tile<T128x64>(g, e, st);
        case 7: return run_tile<T64x64>(g, e, st);
        default: return hipErrorInvalidValue;
    }
}

// rows [0, m_split) with the plan's tile, then the tail rows [m_split, M) with the tail tile;
// both launches index rows globally (the epilogue's sample / token split needs it)
hipError_t launch_gemm_bf16(const GemmArgs& g, const EpiParams& e, hipStream_t st, int tile) {
    if (e.kind == EP_PARTIAL && tile == 0) tile = partial_tile(g, e);
    if (tile != 0) return launch_tile(g, e, st, tile);
    const GemmPlan p = gemm_bf16_plan(g, e);
    if (!p.tail_tile) return launch_tile(g, e, st, p.tile);
    GemmArgs gm = g;
    gm.M = p.m_split;
    const hipError_t err = launch_tile(gm, e, st, p.tile);
    if (err != hipSuccess) return err;
    GemmArgs gt = g;
    gt.m_begin = p.m_split;
    return launch_tile(gt, e, st, p.tail_tile);
}

}  // namespace sgd
