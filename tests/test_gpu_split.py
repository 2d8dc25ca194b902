"""GPU parity of the split MLP output GEMM: where two K ranges cost less than the whole product by more
than their fp32 partials do, the launcher runs it so and the next unit's pre-norm adds the partials to
the stream, unless the next unit is frozen or the step stores the unit's cached update.  LLaDA-shaped
stacks with an 8192-wide MLP take that path; teacher-forced against the oracle and all-active against
the unscheduled forward bit for bit.  (The LLaDA-8B shape itself, on 256 x 128 tiles, is in
test_gpu_fullsize.py.)"""
import numpy as np
import pytest

import synth
from oracle import schedule as osch

from helpers import TOL, gpu_teacher_forced, gpu_trajectory, oracle_trajectory, rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2609_29505_amd as P
    P.lib()
    return P


@pytest.fixture(scope="module")
def wide():
    # 200 tokens x d = 256: sixteen 64 x 64 tiles with 128 k tiles each, halved by two K ranges
    cfg = synth.get_config("llada_mini", F=8192, T=6)
    return cfg, synth.model_weights(cfg), synth.inputs(cfg)


@pytest.mark.parametrize("granularity", ["block", "branch"])
def test_split_output_gemm_teacher_forced(P, wide, granularity):
    """Every fourth unit lives two steps: before that the units ahead of it take the split
    product, afterwards they do not (a frozen unit follows) and the frozen unit folds into the
    next pre-norm; the stores of cached updates at s = S_l take the unsplit epilogue.  Per-step
    error against the oracle."""
    cfg, w, x = wide
    dm = P.DeviceModel(cfg, w, x, granularity=granularity)
    U = dm.n_units
    S = np.array([cfg.T if j % 4 != 1 else 2 for j in range(U)])
    mask = osch.active_mask(S, cfg.T)
    ref = oracle_trajectory(cfg, w, x, mask, granularity=granularity)
    got = gpu_teacher_forced(dm, cfg, ref.z, x["z"], P.schedule_from_lifetimes(S, cfg.T))
    errs = [rel_err(g, r) for g, r in zip(got, ref.z)]
    print(granularity, "split output GEMM, teacher-forced per-step error", ["%.2e" % e for e in errs])
    assert max(errs) <= TOL["bf16"], errs
    dm.close()


def test_split_output_gemm_large_tiles(P):
    """1030 tokens x d = 1024: 72 tiles of 128 x 128, 144 of them in two K ranges; both steps unscheduled-like
    (no unit stores an update), so the first unit's output is split at each."""
    cfg = synth.get_config("llada_mini", N=1030, d=1024, H=8, F=8192, L=2, T=2, prompt_rows=515)
    w, x = synth.model_weights(cfg), synth.inputs(cfg)
    dm = P.DeviceModel(cfg, w, x)
    S = [cfg.T] * cfg.L
    ref = oracle_trajectory(cfg, w, x, osch.active_mask(np.array(S), cfg.T))
    got = gpu_teacher_forced(dm, cfg, ref.z, x["z"], P.schedule_from_lifetimes(S, cfg.T))
    dm.close()
    errs = [rel_err(g, r) for g, r in zip(got, ref.z)]
    assert max(errs) <= TOL["bf16"], errs


def test_split_output_gemm_all_active_is_unscheduled(P, wide):
    cfg, w, x = wide
    dm = P.DeviceModel(cfg, w, x)
    a = gpu_trajectory(dm, cfg, x, P.schedule_from_lifetimes([cfg.T] * cfg.L, cfg.T), 3)
    b = gpu_trajectory(dm, cfg, x, None, 3)
    dm.close()
    for za, zb in zip(a, b):
        assert np.array_equal(za, zb)


def test_split_output_gemm_graph_replays_equal_eager(P, wide):
    """The split product and its partial-adding pre-norm captured in a whole-trajectory HIP
    graph: two replays, with eager work between them, equal the eager trajectory bit for bit."""
    import torch
    cfg, w, x = wide
    dm = P.DeviceModel(cfg, w, x)
    S = np.array([cfg.T, 2, cfg.T, cfg.T])
    sched = P.schedule_from_lifetimes(S, cfg.T)
    eager = gpu_trajectory(dm, cfg, x, sched)[-1]
    stream = torch.cuda.Stream()
    z0 = torch.from_numpy(x["z"].copy()).cuda()
    z = torch.empty_like(z0)
    cache = P.Cache(dm)
    with torch.cuda.stream(stream):
        g = dm.capture(z, sched, cache, stream)
    other = torch.from_numpy(x["z"].copy()).cuda()
    for rep in range(2):
        with torch.cuda.stream(stream):
            z.copy_(z0)
            g.launch(stream)
        stream.synchronize()
        assert np.array_equal(z.cpu().numpy().astype(np.float64), eager), rep
        c2 = P.Cache(dm)
        c2.reset()
        dm.step(other, 1, sched, c2)
        torch.cuda.synchronize()
    g.close()
    dm.close()


def test_replay_inert_units_where_outputs_split(P, wide):
    """Oracle replay on a shape whose MLP outputs split: the reference evaluation stores every unit's
    update and the candidates store none, yet units whose branches are identically zero freeze at a
    deviation of exactly 0 (tau = 0)."""
    import torch
    from dataclasses import replace
    cfg, w, x = wide
    cfg = replace(cfg, T=3)
    w = [dict(u) for u in w]
    for l in (0, 2):
        for key in ("w_o", "w2"):
            w[l][key] = np.zeros_like(w[l][key])
    dm = P.DeviceModel(cfg, w, x)
    life, _, dlog = dm.replay_search(torch.from_numpy(x["z"].copy()).cuda(), tau_agree=0.0, log=True)
    dm.close()
    assert dlog[1, 0, 0] == 0.0 and dlog[1, 0, 2] == 0.0
    assert dlog[1, 0, 1] > 0 and dlog[1, 0, 3] > 0
    assert life.tolist() == [1, cfg.T, 1, cfg.T]
