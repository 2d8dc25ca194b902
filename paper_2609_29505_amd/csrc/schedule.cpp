// Schedule construction (Alg. 1, Sec. 4.1) behind sgd_schedule_build.
//
// Per scored matrix W (m x n, d = min(m, n)), all on the GPU and for many matrices at once: the
// fp64 Gram matrix of the short side, its Householder tridiagonal form and the
// eigenvalues of that form by bisection.  They are squared singular values sigma_i^2, from which
//   E_k = sum_{i<=k} sigma_i^2, k = min(d, max(1, floor(d/10)))
//   SCR_eta = log((E_k + eta F) / (tail + eta F)), F = ||W||_F^2 = trace of the Gram
//   g(W) = sqrt(F) sqrt(rho), rho = (E_k + eta F) / (E_k + tail + 2 eta F)
// (Eq. scr-reg; Eq. app-matrix-score with rho(u) = e^u / (1 + e^u) evaluated at u = SCR).
// Unit scores combine g by Eqs. app-attn-score / app-xattn-score / app-mlp-score /
// app-conv-score, sum per unit (Eq. app-block-score) and normalise with eps = 1e-12
// (Eq. app-score-normalization).  Lifetimes follow Eq. schedule.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <tuple>
#include <vector>

#include "internal.h"
#include "kernels.h"

namespace sgd {

struct MatStats {
    double e_top = 0, e_tail = 0, frob = 0, scr = 0, g = 0, sigma1_sq = 0;
};

static int rank_k(long m, long n) {
    const long d = std::min(m, n);
    return (int)std::min<long>(d, std::max<long>(1, d / 10));
}

// Statistics from the eigenvalues (descending), summed in extended precision.
static MatStats stats_from_eigs(const double* lam, double frob, int k, int n, double eta) {
    MatStats s;
    long double top = 0.0L, tail = 0.0L;
    for (int i = 0; i < k; ++i) top += std::max(lam[i], 0.0);
    for (int i = n - 1; i >= k; --i) tail += std::max(lam[i], 0.0);
    s.e_top = (double)top;
    s.e_tail = (double)tail;
    s.frob = frob;
    const double A = s.e_top + eta * frob, B = s.e_tail + eta * frob;
    s.scr = B > 0 ? std::log(A / B) : std::numeric_limits<double>::infinity();
    const double rho = (A + B) > 0 ? A / (A + B) : 0.0;
    s.g = std::sqrt(frob) * std::sqrt(rho);
    s.sigma1_sq = std::max(lam[0], 0.0);
    return s;
}

// ---------------------------------------------------------------------------- GPU driver

struct MatJob {
    const sgd_matrix* m;
    MatStats out;
};

static int validate_matrix(const sgd_matrix* m) {
    if (!m || !m->ptr) return fail(SGD_E_ARG, "matrix pointer is NULL");
    if (m->rows < 1 || m->cols < 1) return fail(SGD_E_SHAPE, "matrix has an empty dimension");
    if (std::min(m->rows, m->cols) > 16384) return fail(SGD_E_SHAPE, "matrix short side above 16384");
    if (m->dtype != SGD_F32 && m->dtype != SGD_BF16) return fail(SGD_E_DTYPE, "matrix dtype must be F32 or BF16");
    if (m->role < SGD_ROLE_Q || m->role > SGD_ROLE_CONV) return fail(SGD_E_ARG, "unknown matrix role");
    return SGD_OK;
}

static size_t pad256(size_t b) { return (b + 255) & ~(size_t)255; }

// Device bytes of one matrix of a batch whose short sides are at most n: its job record, its results
// (four vectors) and its slot (the Gram matrix, then work vectors).
static size_t slot_bytes(long n) {
    return pad256((size_t)n * spectral_lda((int)n) * 8 + (size_t)(5 * n + 8) * 8);
}
static size_t matrix_bytes(long n) { return pad256(sizeof(SpectralJob)) + pad256((size_t)n * 32) + slot_bytes(n); }

// Device bytes per worker: at least 4 MiB, so that a batch of small matrices, whose chain of steps
// costs the same for one matrix as for all of them, takes several per worker.
static size_t worker_bytes(long n) { return std::max(matrix_bytes(n), (size_t)4 << 20); }

// Score every job on hip_stream, in batches of as many matrices as the workspace holds, largest first
// (a batch's launches cover its largest matrix's steps).
static int run_stats(std::vector<MatJob>& jobs, double eta, char* ws, size_t ws_bytes, hipStream_t st) {
    if (jobs.empty()) return SGD_OK;
    std::vector<size_t> order(jobs.size());
    for (size_t i = 0; i < order.size(); ++i) order[i] = i;
    auto side = [&](size_t i) { return std::min(jobs[i].m->rows, jobs[i].m->cols); };
    std::stable_sort(order.begin(), order.end(), [&](size_t x, size_t y) { return side(x) > side(y); });
    if (!ws || ws_bytes < matrix_bytes(side(order[0]))) return fail(SGD_E_ARG, "schedule workspace smaller than one worker slot");
    if ((uintptr_t)ws % 256) return fail(SGD_E_ARG, "schedule workspace must be 256-byte aligned");
    constexpr size_t kBatchMax = 512;
    for (size_t done = 0; done < order.size();) {
        const long nmax = side(order[done]);
        size_t count = std::min({order.size() - done, ws_bytes / matrix_bytes(nmax), kBatchMax});
        if (nmax > kSpectralMax)  // batches lie on one side of the fused reduction's limit
            while (count > 1 && side(order[done + count - 1]) <= kSpectralMax) --count;
        std::vector<SpectralJob> hj(count);
        int tiles = 0;
        for (size_t b = 0; b < count; ++b) {
            const sgd_matrix* m = jobs[order[done + b]].m;
            SpectralJob& j = hj[b];
            j.X = m->ptr;
            j.rows = m->rows;
            j.cols = m->cols;
            j.trans = m->cols > m->rows ? 1 : 0;  // Gram of the short side
            j.dtype = m->dtype;
            j.n = (int)std::min(m->rows, m->cols);
            j.k = rank_k(m->rows, m->cols);
            j.tile0 = tiles;
            j.pad = 0;
            const int nt = (j.n + 63) / 64;
            tiles += nt * (nt + 1) / 2;
        }
        SpectralBatch sb;
        sb.jobs = (const SpectralJob*)ws;
        sb.outs = (double*)(ws + pad256(count * sizeof(SpectralJob)));
        sb.slots = (double*)((char*)sb.outs + pad256(count * (size_t)nmax * 32));
        sb.slot = (long)(slot_bytes(nmax) / 8);
        sb.nmax = (int)nmax;
        sb.count = (int)count;
        std::vector<double> ho(count * (size_t)nmax * 4);
        hipError_t e = hipMemcpyAsync(ws, hj.data(), count * sizeof(SpectralJob), hipMemcpyHostToDevice, st);
        if (e == hipSuccess) e = launch_spectra(sb, hj.data(), st);
        if (e == hipSuccess) e = hipMemcpyAsync(ho.data(), sb.outs, ho.size() * 8, hipMemcpyDeviceToHost, st);
        // the host vectors live until here on every path
        const hipError_t es = hipStreamSynchronize(st);
        if (e == hipSuccess) e = es;
        if (e != hipSuccess) return fail(SGD_E_HIP, std::string("spectral kernels: ") + hipGetErrorString(e));
        for (size_t b = 0; b < count; ++b) {
            const double* o = ho.data() + b * (size_t)nmax * 4;
            const int n = hj[b].n, k = hj[b].k;
            double frob = 0.0;
            for (int i = 0; i < n; ++i) frob += o[2 * nmax + i];
            bool finite = std::isfinite(frob);
            for (int i = 0; i < n; ++i) finite = finite && std::isfinite(o[i]) && (i + 1 >= n || std::isfinite(o[nmax + i]));
            for (int i = 0; i < n; ++i) finite = finite && std::isfinite(o[3 * nmax + i]);
            if (!finite) return fail(SGD_E_NUMERIC, "non-finite weights in a scored matrix");
            jobs[order[done + b]].out = stats_from_eigs(o + 3 * nmax, frob, k, n, eta);
        }
        done += count;
    }
    return SGD_OK;
}

// ---------------------------------------------------------------------------- lifetimes

// The parameters with the library's defaults applied: S_min <= 0 -> ceil(T / 10); a
// percentage budget -> N* = floor(pct L T / 100).  Validates the result.
static int resolve_params(const sgd_sched_params* p, int L, sgd_sched_params* r) {
    if (!p) return fail(SGD_E_ARG, "params is NULL");
    if (L < 1) return fail(SGD_E_ARG, "L must be >= 1");
    if (p->T < 1) return fail(SGD_E_ARG, "T must be >= 1");
    *r = *p;
    if (r->s_min <= 0) r->s_min = sgd_s_min_default(p->T);
    if (r->s_min > p->T) return fail(SGD_E_ARG, "s_min must lie in 1..T");
    if (r->budget_layer_steps < 0 && r->budget_pct > 0) {
        if (r->budget_pct > 100) return fail(SGD_E_ARG, "budget_pct must lie in 1..100");
        const int64_t n = (int64_t)r->budget_pct * L * p->T / 100;
        if (n > INT32_MAX) return fail(SGD_E_ARG, "budget above 2^31 layer-steps");
        r->budget_layer_steps = (int32_t)n;
    }
    if (r->budget_layer_steps < 0 && !(r->tau > 0)) return fail(SGD_E_ARG, "tau must be > 0 in tau mode");
    if (!(r->eta >= 0) || !std::isfinite(r->eta)) return fail(SGD_E_ARG, "eta must be finite and >= 0");
    if (r->rule < 0 || r->rule >= SGD_RULE_COUNT) return fail(SGD_E_ARG, "unknown ranking rule");
    if (r->budget_layer_steps >= 0) {
        const long lo = (long)L * r->s_min, hi = (long)L * p->T;
        if (r->budget_layer_steps < lo || r->budget_layer_steps > hi)
            return fail(SGD_E_BUDGET, "budget outside [L*s_min, L*T]");
    }
    return SGD_OK;
}

int lifetimes_from_scores(const double* score, int L, const sgd_sched_params* p, sgd_schedule* out) {
    const int T = p->T;
    std::vector<int> S(L, p->s_min);
    double margin = std::numeric_limits<double>::infinity();
    if (p->budget_layer_steps < 0) {
        for (int l = 0; l < L; ++l) {
            const double v = std::ceil((double)T * std::min(1.0, score[l] / p->tau));
            S[l] = std::max(p->s_min, (int)v);
        }
    } else {
        struct Ev { double key; int l, j; };
        std::vector<Ev> ev;
        ev.reserve((size_t)L * (T - p->s_min));
        for (int l = 0; l < L; ++l)
            for (int j = p->s_min; j < T; ++j)
                ev.push_back({score[l] > 0 ? (double)j / score[l] : std::numeric_limits<double>::infinity(), l, j});
        std::sort(ev.begin(), ev.end(), [](const Ev& x, const Ev& y) {
            return std::tie(x.key, x.l, x.j) < std::tie(y.key, y.l, y.j);
        });
        const long grant = (long)p->budget_layer_steps - (long)L * p->s_min;
        for (long i = 0; i < grant; ++i) S[ev[i].l] += 1;
        if (grant > 0 && grant < (long)ev.size()) {
            const double last = ev[grant - 1].key, nxt = ev[grant].key;
            if (std::isfinite(last) && last > 0 && std::isfinite(nxt)) margin = (nxt - last) / last;
        }
    }
    out->L = L;
    out->T = T;
    long total = 0;
    for (int l = 0; l < L; ++l) total += S[l];
    if (out->lifetimes)
        for (int l = 0; l < L; ++l) out->lifetimes[l] = S[l];
    if (out->active)
        for (int s = 1; s <= T; ++s)
            for (int l = 0; l < L; ++l) out->active[(size_t)(s - 1) * L + l] = (uint8_t)(s <= S[l]);
    out->layer_steps = total;
    out->cut_margin = margin;
    out->s_min = p->s_min;
    return SGD_OK;
}

// SplitMix64 (Steele, Lea and Flood, "Fast splittable pseudorandom number generators",
// OOPSLA 2014): output i of the stream seeded with `seed` mixes seed + i * golden gamma.
static uint64_t splitmix64(uint64_t seed, uint64_t i) {
    uint64_t z = seed + i * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Matrix statistic of a ranking rule (g(W) for the method).
static double rule_stat(const MatStats& s, int rule) {
    switch (rule) {
        case SGD_RULE_FROB: return std::sqrt(s.frob);
        case SGD_RULE_SPECTRAL: return std::sqrt(s.sigma1_sq);
        case SGD_RULE_STABLE_RANK: return s.frob > 0 ? s.sigma1_sq / s.frob : 0.0;
        case SGD_RULE_FROB_SRANK: return s.frob > 0 ? std::sqrt(s.frob) * (s.sigma1_sq / s.frob) : 0.0;
        case SGD_RULE_RAW_SCR: {
            const double g = s.g, f = std::sqrt(s.frob);
            return f > 0 ? g / f : 0.0;
        }
        default: return s.g;
    }
}

}  // namespace sgd

using namespace sgd;

// Unit raw scores of the rule from the matrices' statistics (Eqs. app-attn-score,
// app-xattn-score, app-mlp-score, app-conv-score, app-block-score with the rule's statistic
// in place of g), normalised (Eq. app-score-normalization) and mapped to lifetimes.
static int rank_units(const sgd_unit* units, int L, const std::vector<MatStats>& st, const sgd_sched_params& p,
                      sgd_schedule* out) {
    std::vector<double> raw(L, 0.0);
    if (p.rule == SGD_RULE_DEPTH) {
        for (int l = 0; l < L; ++l) raw[l] = (double)(l + 1);
    } else if (p.rule == SGD_RULE_RANDOM) {
        for (int l = 0; l < L; ++l) raw[l] = (double)(splitmix64(p.seed, (uint64_t)l + 1) >> 11) * 0x1.0p-53;
    } else {
        size_t ji = 0;
        for (int l = 0; l < L; ++l) {
            const sgd_unit& u = units[l];
            double g[SGD_ROLE_CONV + 1];
            bool have[SGD_ROLE_CONV + 1] = {};
            double conv = 0.0;
            for (int i = 0; i < u.n_mats; ++i, ++ji) {
                const int r = u.mats[i].role;
                const double v = rule_stat(st[ji], p.rule);
                if (r == SGD_ROLE_CONV) { conv += v; continue; }
                have[r] = true;
                g[r] = v;
            }
            const double sdh = std::sqrt((double)u.head_dim);
            double q = 0.0;
            if (have[SGD_ROLE_Q] && have[SGD_ROLE_K] && have[SGD_ROLE_V] && have[SGD_ROLE_O])
                q += g[SGD_ROLE_O] * g[SGD_ROLE_V] * (1.0 + g[SGD_ROLE_Q] * g[SGD_ROLE_K] / sdh);
            if (have[SGD_ROLE_XQ] && have[SGD_ROLE_XK] && have[SGD_ROLE_XV] && have[SGD_ROLE_XO])
                q += g[SGD_ROLE_XO] * g[SGD_ROLE_XV] * (1.0 + g[SGD_ROLE_XQ] * g[SGD_ROLE_XK] / sdh);
            if (have[SGD_ROLE_W1] && have[SGD_ROLE_W2]) q += g[SGD_ROLE_W2] * g[SGD_ROLE_W1];
            q += conv;
            raw[l] = q;
        }
    }
    double mx = 0.0;
    for (double v : raw) {
        if (!std::isfinite(v)) return fail(SGD_E_NUMERIC, "non-finite unit score");
        mx = std::max(mx, v);
    }
    std::vector<double> score(L);
    for (int l = 0; l < L; ++l) score[l] = raw[l] / (mx + 1e-12);
    int rc = lifetimes_from_scores(score.data(), L, &p, out);
    if (rc) return rc;
    if (out->unit_raw) std::memcpy(out->unit_raw, raw.data(), L * sizeof(double));
    if (out->unit_score) std::memcpy(out->unit_score, score.data(), L * sizeof(double));
    if (out->mat_stats)
        for (size_t i = 0; i < st.size(); ++i) {
            const MatStats& m = st[i];
            double* o = out->mat_stats + 6 * i;
            o[0] = m.e_top; o[1] = m.e_tail; o[2] = m.frob; o[3] = m.scr; o[4] = m.g; o[5] = m.sigma1_sq;
        }
    return SGD_OK;
}

extern "C" int32_t sgd_s_min_default(int32_t T) { return T >= 1 ? (T + 9) / 10 : 0; }

extern "C" int sgd_budget_layer_steps(int32_t pct, int32_t L, int32_t T, int64_t* n_star) {
    if (!n_star) return fail(SGD_E_ARG, "NULL argument");
    if (pct < 0 || pct > 100 || L < 1 || T < 1) return fail(SGD_E_ARG, "need 0 <= pct <= 100, L >= 1, T >= 1");
    *n_star = (int64_t)pct * L * T / 100;
    return SGD_OK;
}

extern "C" int sgd_schedule_from_scores(const double* unit_score, int32_t L, const sgd_sched_params* params,
                                        sgd_schedule* out) {
    if (!unit_score || !out || !out->lifetimes || !out->active) return fail(SGD_E_ARG, "NULL argument");
    sgd_sched_params p;
    int rc = resolve_params(params, L, &p);
    if (rc) return rc;
    for (int l = 0; l < L; ++l)
        if (!std::isfinite(unit_score[l]) || unit_score[l] < 0) return fail(SGD_E_NUMERIC, "scores must be finite and >= 0");
    rc = lifetimes_from_scores(unit_score, L, &p, out);
    if (rc) return rc;
    if (out->unit_score)
        for (int l = 0; l < L; ++l) out->unit_score[l] = unit_score[l];
    return SGD_OK;
}

extern "C" int sgd_schedule_from_lifetimes(int32_t L, int32_t T, const int32_t* lifetimes, sgd_schedule* out) {
    if (!lifetimes || !out || !out->lifetimes || !out->active) return fail(SGD_E_ARG, "NULL argument");
    if (L < 1 || T < 1) return fail(SGD_E_ARG, "L and T must be >= 1");
    long total = 0;
    int smin = T;
    for (int l = 0; l < L; ++l) {
        if (lifetimes[l] < 1 || lifetimes[l] > T) return fail(SGD_E_ARG, "lifetimes must lie in 1..T");
        total += lifetimes[l];
        smin = std::min(smin, (int)lifetimes[l]);
    }
    out->L = L;
    out->T = T;
    for (int l = 0; l < L; ++l) out->lifetimes[l] = lifetimes[l];
    for (int s = 1; s <= T; ++s)
        for (int l = 0; l < L; ++l) out->active[(size_t)(s - 1) * L + l] = (uint8_t)(s <= lifetimes[l]);
    out->layer_steps = total;
    out->cut_margin = std::numeric_limits<double>::infinity();
    out->s_min = smin;
    return SGD_OK;
}

extern "C" int sgd_schedule_workspace_bytes(const sgd_unit* units, int32_t L, int32_t workers, size_t* bytes) {
    if (!bytes || (!units && L > 0)) return fail(SGD_E_ARG, "NULL argument");
    if (workers < 1 || workers > 16) return fail(SGD_E_ARG, "workers must lie in 1..16");
    long nmax = 0;
    for (int l = 0; l < L; ++l) {
        if (units[l].n_mats > 0 && !units[l].mats) return fail(SGD_E_ARG, "unit without matrices");
        for (int i = 0; i < units[l].n_mats; ++i)
            nmax = std::max<long>(nmax, std::min(units[l].mats[i].rows, units[l].mats[i].cols));
    }
    *bytes = nmax > 0 ? (size_t)workers * worker_bytes(nmax) : 0;
    return SGD_OK;
}

extern "C" int sgd_matrix_stats(const sgd_matrix* m, double eta, void* workspace, size_t workspace_bytes,
                                void* hip_stream, double out[6]) {
    if (!out) return fail(SGD_E_ARG, "out is NULL");
    int rc = validate_matrix(m);
    if (rc) return rc;
    if (!(eta >= 0) || !std::isfinite(eta)) return fail(SGD_E_ARG, "eta must be finite and >= 0");
    std::vector<MatJob> jobs{{m, {}}};
    rc = run_stats(jobs, eta, (char*)workspace, workspace_bytes, (hipStream_t)hip_stream);
    if (rc) return rc;
    const MatStats& s = jobs[0].out;
    out[0] = s.e_top; out[1] = s.e_tail; out[2] = s.frob; out[3] = s.scr; out[4] = s.g; out[5] = s.sigma1_sq;
    return SGD_OK;
}

extern "C" int sgd_schedule_build(const sgd_unit* units, int32_t L, const sgd_sched_params* params, void* workspace,
                                  size_t workspace_bytes, void* hip_stream, sgd_schedule* out) {
    if (!out || !out->lifetimes || !out->active) return fail(SGD_E_ARG, "NULL argument");
    sgd_sched_params p;
    int rc = resolve_params(params, L, &p);
    if (rc) return rc;
    const bool unit_rule = p.rule == SGD_RULE_DEPTH || p.rule == SGD_RULE_RANDOM;
    if (!units && !unit_rule) return fail(SGD_E_ARG, "units is NULL");
    std::vector<MatJob> jobs;
    if (units) {
        for (int l = 0; l < L; ++l) {
            const sgd_unit& u = units[l];
            if (u.n_mats < 1 || !u.mats) return fail(SGD_E_ARG, "unit without matrices");
            if (u.head_dim < 1) return fail(SGD_E_ARG, "head_dim must be >= 1");
            bool seen[SGD_ROLE_CONV + 1] = {};
            for (int i = 0; i < u.n_mats; ++i) {
                rc = validate_matrix(&u.mats[i]);
                if (rc) return rc;
                const int r = u.mats[i].role;
                if (r != SGD_ROLE_CONV && seen[r]) return fail(SGD_E_ARG, "a unit lists the same role twice");
                seen[r] = true;
                jobs.push_back({&u.mats[i], {}});
            }
        }
    }
    // unit rules only rank units; spectra are computed when matrices are given (mat_stats)
    if (!unit_rule || (units && out->mat_stats)) {
        rc = run_stats(jobs, p.eta, (char*)workspace, workspace_bytes, (hipStream_t)hip_stream);
        if (rc) return rc;
    }
    std::vector<MatStats> st(jobs.size());
    for (size_t i = 0; i < jobs.size(); ++i) st[i] = jobs[i].out;
    return rank_units(units, L, st, p, out);
}

extern "C" int sgd_schedule_from_stats(const sgd_unit* units, int32_t L, const double* mat_stats,
                                       const sgd_sched_params* params, sgd_schedule* out) {
    if (!units || !mat_stats || !out || !out->lifetimes || !out->active) return fail(SGD_E_ARG, "NULL argument");
    sgd_sched_params p;
    int rc = resolve_params(params, L, &p);
    if (rc) return rc;
    std::vector<MatStats> st;
    for (int l = 0; l < L; ++l) {
        const sgd_unit& u = units[l];
        if (u.n_mats < 1 || !u.mats) return fail(SGD_E_ARG, "unit without matrices");
        if (u.head_dim < 1) return fail(SGD_E_ARG, "head_dim must be >= 1");
        bool seen[SGD_ROLE_CONV + 1] = {};
        for (int i = 0; i < u.n_mats; ++i) {
            const int r = u.mats[i].role;
            if (r < SGD_ROLE_Q || r > SGD_ROLE_CONV) return fail(SGD_E_ARG, "unknown matrix role");
            if (r != SGD_ROLE_CONV && seen[r]) return fail(SGD_E_ARG, "a unit lists the same role twice");
            seen[r] = true;
            const double* o = mat_stats + 6 * st.size();
            MatStats m;
            m.e_top = o[0]; m.e_tail = o[1]; m.frob = o[2]; m.scr = o[3]; m.g = o[4]; m.sigma1_sq = o[5];
            for (int c = 0; c < 6; ++c)
                if (!std::isfinite(o[c]) && c != 3) return fail(SGD_E_NUMERIC, "non-finite matrix statistic");
            st.push_back(m);
        }
    }
    double* keep = out->mat_stats;
    out->mat_stats = nullptr;  // the statistics are inputs here
    rc = rank_units(units, L, st, p, out);
    out->mat_stats = keep;
    return rc;
}
