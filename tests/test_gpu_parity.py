"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the same seeded inputs.

Tolerances: schedules and masks bit-exact; hidden states max|x - y| / max|y| <= 1e-4 (fp32
workloads) and <= 2e-2 (bf16 workloads) at every step.
"""
import numpy as np
import pytest

import synth
from oracle import schedule as osch
from oracle import spectral as osp

from helpers import (FREE_RUNNING_CEIL, TOL, chaos_floor, gpu_teacher_forced, gpu_trajectory, oracle_schedule,
                     oracle_trajectory, rel_err)

pytestmark = pytest.mark.gpu

MINIS = ["tiny_ragged", "llada_mini", "dit_mini", "uvit_mini", "sdxl_mini", "sdxl_unet_mini"]


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_29505_amd as P
    P.lib()
    return P


_cache = {}


def workload(name, **kw):
    key = (name, tuple(sorted(kw.items())))
    if key not in _cache:
        cfg = synth.get_config(name, **kw)
        _cache[key] = (cfg, synth.model_weights(cfg), synth.inputs(cfg))
    return _cache[key]


# ---------------------------------------------------------------- spectra and schedules

def _dev(arr):
    import torch
    if arr.dtype == np.uint16:
        return torch.from_numpy(arr.view(np.int16)).view(torch.bfloat16).cuda()
    return torch.from_numpy(np.ascontiguousarray(arr, np.float32)).cuda()


@pytest.mark.parametrize("shape,dtype", [((100, 37), "f32"), ((37, 100), "f32"), ((256, 256), "bf16"),
                                         ((300, 700), "bf16"), ((1280, 640), "bf16"), ((1, 50), "f32"),
                                         ((5, 3), "f32"), ((130, 129), "f32")])
def test_matrix_stats(P, shape, dtype):
    rng = np.random.default_rng(sum(shape))
    w, _ = synth.planted_matrix(rng, *shape, np.float64)
    stored = synth.store(w, dtype)
    from oracle.numerics import decode
    ref = osp.matrix_stats(decode(stored, dtype), eta=1e-6)
    got = P.matrix_stats(_dev(stored), eta=1e-6)
    F = ref.frob_sq
    assert got[2] == pytest.approx(F, rel=1e-12)
    assert abs(got[0] - ref.energy_top) <= 1e-11 * F
    assert abs(got[1] - ref.energy_tail) <= 1e-11 * F
    assert got[4] == pytest.approx(ref.g, rel=1e-11)
    assert got[3] == pytest.approx(ref.scr, rel=1e-6, abs=1e-7)
    assert got[5] == pytest.approx(ref.sigma1_sq, rel=1e-11)


def test_schedule_build_mixed_sizes(P):
    """One batch of matrices of very different sizes: short sides 1, 2 and 3 (no or one reduction
    step), odd and even ones around a row pass of the reduction (17, 18, 33), both orientations and
    both storage types; each matrix's statistics as from a batch of its own and as the oracle's."""
    from oracle.numerics import decode
    rng = np.random.default_rng(41)
    shapes = [(1, 9), (2, 2), (7, 2), (3, 3), (3, 40), (17, 17), (18, 50), (90, 33), (130, 129)]
    mats = [synth.store(synth.planted_matrix(rng, *sh, np.float64)[0], "bf16" if i % 2 else "f32")
            for i, sh in enumerate(shapes)]
    units = [[("conv", _dev(m)) for m in mats[:4]], [("conv", _dev(m)) for m in mats[4:]]]
    got = P.schedule_build(units, [64, 64], 10, budget_pct=50).mat_stats
    for i, m in enumerate(mats):
        ref = osp.matrix_stats(decode(m, "bf16" if i % 2 else "f32"), eta=1e-6)
        F = ref.frob_sq
        assert np.array_equal(got[i], P.matrix_stats(_dev(m), eta=1e-6)), shapes[i]
        assert abs(got[i, 0] - ref.energy_top) <= 1e-13 * F and abs(got[i, 1] - ref.energy_tail) <= 1e-13 * F
        assert got[i, 2] == pytest.approx(F, rel=1e-13) and got[i, 4] == pytest.approx(ref.g, rel=1e-13)
        assert got[i, 5] == pytest.approx(ref.sigma1_sq, rel=1e-13)


@pytest.mark.parametrize("n", [64, 192, 193, 194, 195, 385])
def test_matrix_stats_tail_block(P, n):
    """Short sides around the block that is reduced in registers (192 rows, all steps up to 193), graded so
    that the tail holds ~1e-4 of the energy: it has to keep its own relative accuracy.  A Gram matrix is
    exact to ~n 2^-53 of its norm and so are its eigenvalues."""
    rng = np.random.default_rng(n)
    w = (rng.standard_normal((n + 70, n)) * np.arange(1, n + 1) ** -1.3).astype(np.float32)
    ref = osp.matrix_stats(w.astype(np.float64), eta=1e-6)
    got = P.matrix_stats(_dev(w), eta=1e-6)
    assert got[0] == pytest.approx(ref.energy_top, rel=n * 2.0 ** -52)
    assert abs(got[1] - ref.energy_tail) <= n * 2.0 ** -52 * ref.sigma1_sq
    assert got[5] == pytest.approx(ref.sigma1_sq, rel=n * 2.0 ** -52)


def test_matrix_stats_decoupled(P):
    """Diagonal weights (every off-diagonal of the tridiagonal form zero), repeated and zero singular values,
    and the zero matrix."""
    s = np.zeros(230, np.float32)
    s[:7], s[7:120] = 2.0, 0.5
    got = P.matrix_stats(_dev(np.diag(s)), eta=1e-6)
    assert got[0] == pytest.approx(7 * 4.0 + 16 * 0.25, rel=1e-14)
    assert got[1] == pytest.approx(97 * 0.25, rel=1e-14)
    got = P.matrix_stats(_dev(np.zeros((30, 200), np.float32)), eta=1e-6)
    assert got[0] == got[1] == got[2] == got[4] == got[5] == 0.0 and np.isinf(got[3])


@pytest.mark.parametrize("n", [6592, 6720])
def test_matrix_stats_large(P, n):
    """The last short sides whose reduction keeps its vectors in LDS and the first that does not:
    W = diag(s) Q with Q block diagonal, 64 x 64 Hadamard blocks over 8 (orthogonal, exact in bf16),
    so the singular values are exactly s (powers of two)."""
    import torch
    h = torch.ones(1, 1)
    while h.shape[0] < 64:
        h = torch.cat([torch.cat([h, h], 1), torch.cat([h, -h], 1)])
    rng = np.random.default_rng(n)
    s = 2.0 ** rng.integers(-6, 3, n)
    w = torch.zeros((n, n), dtype=torch.bfloat16, device="cuda")
    sd = torch.from_numpy(s).cuda()
    for i in range(0, n, 64):
        w[i:i + 64, i:i + 64] = (sd[i:i + 64, None] * (h.double().cuda() / 8)).bfloat16()
    got = P.matrix_stats(w, eta=1e-6)
    lam = np.sort(s * s)[::-1]
    k, F = n // 10, lam.sum()
    assert got[2] == pytest.approx(F, rel=1e-14)
    assert abs(got[0] - lam[:k].sum()) <= 1e-13 * F and abs(got[1] - lam[k:].sum()) <= 1e-13 * F
    assert got[5] == pytest.approx(lam[0], rel=1e-13)


def test_large_matrices_share_a_batch(P):
    """Short sides past the LDS limit are reduced side by side, one launch per step for all: matrices of
    different sizes and storage types in one batch, each with the bits of a batch of its own."""
    import torch
    torch.manual_seed(6656)
    mats = [torch.randn(6720, 6656, device="cuda").bfloat16(), torch.randn(6605, 6700, device="cuda"),
            torch.randn(6720, 6720, device="cuda").bfloat16()]
    got = P.schedule_build([[("conv", m) for m in mats]], [64], 10, budget_pct=50).mat_stats
    for i, m in enumerate(mats):
        assert np.array_equal(got[i], P.matrix_stats(m, eta=1e-6)), i
        assert got[i, 2] == pytest.approx(float((m.double() ** 2).sum()), rel=1e-12)
        assert got[i, 0] + got[i, 1] == pytest.approx(got[i, 2], rel=1e-12)


@pytest.mark.parametrize("name", MINIS + ["tiny"])
def test_schedule_bit_exact(P, name):
    cfg, w, x = workload(name)
    dm = P.DeviceModel(cfg, w, x)
    for pct in cfg.budgets:
        raw, lam, bs = oracle_schedule(cfg, w, pct)
        n = osch.budget_layer_steps(pct, cfg.L, cfg.T)
        got = P.schedule_build(dm.scored_units(), [cfg.dh] * cfg.L, cfg.T, budget=n)
        assert np.allclose(got.unit_raw, raw, rtol=1e-11)
        assert np.allclose(got.unit_score, lam, rtol=1e-11)
        assert bs.cut_margin > 1e-9, "near-tie: the comparison below would be fragile"
        assert np.array_equal(got.lifetimes, bs.lifetimes)
        assert np.array_equal(got.active, osch.active_mask(bs.lifetimes, cfg.T))
        assert got.layer_steps == n
    dm.close()


@pytest.mark.parametrize("name", ["tiny", "llada_mini", "dit_mini", "sdxl_mini"])
def test_rule_schedules_bit_exact(P, name):
    """Every static ranking rule (Sec. "Static ranking comparisons") built on the GPU: unit
    raw scores against the oracle's rule on its own spectra, lifetimes bit for bit."""
    from oracle import rules as ru
    cfg, w, x = workload(name)
    dm = P.DeviceModel(cfg, w, x)
    stats = [osp.unit_score(osp.unit_matrices(u, cfg.d, cfg.dtype), cfg.dh).stats for u in w]
    smin = osch.s_min_default(cfg.T)
    for rule in ru.RULES:
        pct = cfg.budgets[-1]
        n = osch.budget_layer_steps(pct, cfg.L, cfg.T)
        ref = ru.lifetimes(rule, stats, cfg.dh, cfg.T, n, smin, seed=11, L=cfg.L)
        got = P.schedule_build(dm.scored_units(), [cfg.dh] * cfg.L, cfg.T, budget_pct=pct, rule=rule, seed=11)
        assert np.allclose(got.unit_raw, ru.raw_scores(rule, stats, cfg.dh, seed=11, L=cfg.L), rtol=1e-11, atol=0)
        if rule not in ("depth", "random"):
            assert ref.cut_margin > 1e-9, (rule, ref.cut_margin)
        assert np.array_equal(got.lifetimes, ref.lifetimes), rule
        assert got.layer_steps == n
    dm.close()


# ---------------------------------------------------------------- trajectories

@pytest.mark.parametrize("name", MINIS)
def test_step_parity_teacher_forced(P, name):
    """Every step s = 1..T of the scheduled trajectory, fed the oracle's state z_s, matches the
    oracle's z_{s+1}: the per-step bar of 1e-4 (fp32) / 2e-2 (bf16)."""
    cfg, w, x = workload(name)
    dm = P.DeviceModel(cfg, w, x)
    pct = cfg.budgets[-1]
    _, _, bs = oracle_schedule(cfg, w, pct)
    mask = osch.active_mask(bs.lifetimes, cfg.T)
    ref = oracle_trajectory(cfg, w, x, mask)
    n = osch.budget_layer_steps(pct, cfg.L, cfg.T)
    sched = P.schedule_build(dm.scored_units(), [cfg.dh] * cfg.L, cfg.T, budget=n)  # end to end on the GPU
    assert np.array_equal(sched.lifetimes, bs.lifetimes)
    got = gpu_teacher_forced(dm, cfg, ref.z, x["z"], sched)
    errs = [rel_err(g, r) for g, r in zip(got, ref.z)]
    print(name, "teacher-forced per-step error", ["%.2e" % e for e in errs])
    assert max(errs) <= TOL[cfg.dtype], errs
    dm.close()


@pytest.mark.parametrize("name", MINIS)
def test_trajectory_parity(P, name):
    """Free-running scheduled trajectory.  fp32: 1e-4 at every step.  bf16: the bf16-quantised
    map amplifies any rounding difference, so the bound is max(2e-2, twice the largest
    divergence of the oracle from itself under 1e-7 and 1e-5 relative perturbations of its
    initial state, two seeds each), capped at FREE_RUNNING_CEIL; the oracle's own divergence
    must stay below the cap, or the case says nothing."""
    cfg, w, x = workload(name)
    dm = P.DeviceModel(cfg, w, x)
    pct = cfg.budgets[-1]
    _, _, bs = oracle_schedule(cfg, w, pct)
    mask = osch.active_mask(bs.lifetimes, cfg.T)
    n = osch.budget_layer_steps(pct, cfg.L, cfg.T)
    sched = P.schedule_build(dm.scored_units(), [cfg.dh] * cfg.L, cfg.T, budget=n)
    assert np.array_equal(sched.lifetimes, bs.lifetimes)
    got = gpu_trajectory(dm, cfg, x, sched)
    if cfg.dtype == "f32":
        ref = oracle_trajectory(cfg, w, x, mask)
        bounds = [TOL["f32"]] * cfg.T
    else:
        ref, floor = chaos_floor(cfg, w, x, mask)
        print(name, "oracle self-divergence", ["%.2e" % e for e in floor])
        assert max(floor) < FREE_RUNNING_CEIL, floor
        bounds = [min(FREE_RUNNING_CEIL, max(TOL["bf16"], 2 * f)) for f in floor]
    errs = [rel_err(g, r) for g, r in zip(got, ref.z)]
    print(name, "free-running per-step error", ["%.2e" % e for e in errs])
    assert all(e <= b for e, b in zip(errs, bounds)), (errs, bounds)
    dm.close()


@pytest.mark.parametrize("name", MINIS)
def test_all_active_equals_unscheduled_bitwise(P, name):
    cfg, w, x = workload(name)
    dm = P.DeviceModel(cfg, w, x)
    steps = min(cfg.T, 3)
    a = gpu_trajectory(dm, cfg, x, P.schedule_from_lifetimes([cfg.T] * cfg.L, cfg.T), steps)
    b = gpu_trajectory(dm, cfg, x, None, steps)
    c = gpu_trajectory(dm, cfg, x, None, steps)
    for za, zb, zc in zip(a, b, c):
        assert np.array_equal(za, zb)
        assert np.array_equal(zb, zc)  # deterministic
    dm.close()


@pytest.mark.parametrize("name", MINIS)
def test_workspace_contents_do_not_matter(P, name):
    """The step reads no workspace byte it has not written in the same step: a workspace
    full of NaN bit patterns and one full of zeros give bitwise the same trajectory
    (padded query rows, for instance, must not steer the attention's rescaling)."""
    cfg, w, x = workload(name)
    dm = P.DeviceModel(cfg, w, x)
    sched = P.schedule_from_lifetimes([1 + (l * 3) % cfg.T for l in range(cfg.L)], cfg.T)
    outs = []
    for fill in (0x00, 0xFF):
        dm.workspace.fill_(fill)
        outs.append(gpu_trajectory(dm, cfg, x, sched, min(cfg.T, 4)))
    for a, b in zip(*outs):
        assert np.array_equal(a, b)
    dm.close()


@pytest.mark.parametrize("name", ["llada_mini", "uvit_mini", "dit_mini"])
def test_frozen_early(P, name):
    """Lifetimes of 1 freeze units from step 2 on: the frozen path carries most of the trajectory."""
    cfg, w, x = workload(name)
    dm = P.DeviceModel(cfg, w, x)
    S = np.array([1 + (l % 3) for l in range(cfg.L)])
    mask = osch.active_mask(S, cfg.T)
    ref = oracle_trajectory(cfg, w, x, mask)
    got = gpu_trajectory(dm, cfg, x, P.schedule_from_lifetimes(S, cfg.T))
    errs = [rel_err(g, r) for g, r in zip(got, ref.z)]
    print(name, "per-step error", ["%.2e" % e for e in errs])
    assert max(errs) <= TOL[cfg.dtype], errs
    dm.close()


def test_step_errors(P):
    cfg, w, x = workload("llada_mini")
    dm = P.DeviceModel(cfg, w, x)
    import torch
    z = torch.from_numpy(x["z"].copy()).cuda()
    cache = P.Cache(dm)
    a = P.schedule_from_lifetimes([5] * cfg.L, cfg.T)
    b = P.schedule_from_lifetimes([1] * cfg.L, cfg.T)
    with pytest.raises(P.SgdError) as e:
        dm.step(z, 2, a, cache)  # out of order
    assert e.value.code == -5
    dm.step(z, 1, a, cache)
    with pytest.raises(P.SgdError) as e:
        dm.step(z, 2, b, cache)  # frozen, but schedule a never wrote the slot
    assert e.value.code == -6
    with pytest.raises(P.SgdError) as e:
        dm.step(z, cfg.T + 1, None, None)
    assert e.value.code == -5
    torch.cuda.synchronize()
    dm.close()


@pytest.mark.parametrize("name,over", [("tiny_ragged", dict(L=1, T=1)), ("tiny_ragged", dict(B=1, N=1, L=2, T=4)),
                                       ("llada_mini", dict(L=1, T=3)), ("dit_mini", dict(B=1, L=1, T=2)),
                                       ("dit_mini", dict(B=3, N=1, L=2, T=2)), ("sdxl_mini", dict(B=1, L=1, T=2)),
                                       ("uvit_mini", dict(B=1, L=3, T=2)), ("sdxl_unet_mini", dict(B=1, L=1, T=2))])
def test_degenerate_sizes(P, name, over):
    """One unit (U-ViT: its smallest stack, one in-block, the mid block and one out-block), one
    step, one sample, one token per sample (a single key and a one-row GEMM tile); the only unit,
    or every odd-numbered one, frozen after step 1: teacher-forced against the oracle at every
    step, at the per-step bar of the workload's dtype."""
    cfg = synth.get_config(name, **over)
    w, x = synth.model_weights(cfg), synth.inputs(cfg)
    S = np.array([cfg.T if l % 2 == 0 and cfg.L > 1 else (1 if cfg.T > 1 else cfg.T) for l in range(cfg.L)])
    mask = osch.active_mask(S, cfg.T)
    ref = oracle_trajectory(cfg, w, x, mask)
    dm = P.DeviceModel(cfg, w, x)
    got = gpu_teacher_forced(dm, cfg, ref.z, x["z"], P.schedule_from_lifetimes(S, cfg.T))
    errs = [rel_err(g, r) for g, r in zip(got, ref.z)]
    print(name, over, "per-step error", ["%.2e" % e for e in errs])
    assert max(errs) <= TOL[cfg.dtype], errs
    dm.close()
