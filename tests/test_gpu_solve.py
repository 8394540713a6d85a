"""GPU parity of poisson_solve (plain FP64 and mixed precision) against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import RESID_RTOL, needs_gpu, rel, say

pytestmark = [pytest.mark.gpu, needs_gpu]

# pass lengths forced on the small test grids ("" lets the solver choose:
# two-sweep and single passes there, three-sweep passes on large grids)
STEPS = ["", "1", "3"]

from paper_2409_18824_amd import j3d  # noqa: E402


def test_small_plain_100_sweeps_residual_every_sweep():
    """64^3 FP64, u0 ~ U[0,1), f ~ U[-1,1), h = 1/65: 100 sweeps, residual after each."""
    say("64^3 x 100 sweeps")
    u0, f, h = synth.small_plain(64, seed=1)
    du = j3d.FArray.from_numpy(u0)
    df = j3d.FArray.from_numpy(f)
    res = j3d.poisson_solve(du, df, h, mode=j3d.MODE_FP64, rtol=0.0, max_sweeps=100, check_every=1)
    uo, ro = oracle.solve_plain(u0, f, h, rtol=0.0, check_every=1, max_sweeps=100)
    assert res.sweeps == ro.sweeps == 100 and not res.converged
    assert len(res.history) == len(ro.history) == 101
    worst = max(rel(a, b) for a, b in zip(res.history, ro.history))
    say("worst residual rel err", worst)
    assert worst <= RESID_RTOL
    assert rel(res.norm_f, ro.norm_f) <= RESID_RTOL
    assert np.array_equal(du.to_numpy(), uo)


@pytest.mark.parametrize("max_sweeps,check_every", [(0, 1), (7, 3), (10, 5), (1, 1), (10, 2), (9, 4), (1, 2),
                                                   (3, 2), (0, 2), (23, 10), (8, 3), (5, 9), (17, 8)])
@pytest.mark.parametrize("step", STEPS)
def test_plain_cadence_edges(max_sweeps, check_every, step, monkeypatch):
    monkeypatch.setenv("J3D_SOLVE_SWEEPS_PER_PASS", step)
    n = (9, 11, 6)
    say("cadence", max_sweeps, check_every)
    u0 = synth.uniform_field(*n, 4, 1, 0, 1)
    f = synth.uniform_field(*n, 4, 2, -1, 1)
    h = 0.1
    du, df = j3d.FArray.from_numpy(u0), j3d.FArray.from_numpy(f)
    res = j3d.poisson_solve(du, df, h, rtol=0.0, max_sweeps=max_sweeps, check_every=check_every)
    uo, ro = oracle.solve_plain(u0, f, h, rtol=0.0, check_every=check_every, max_sweeps=max_sweeps)
    assert res.sweeps == ro.sweeps
    assert len(res.history) == len(ro.history)
    assert all(rel(a, b) <= RESID_RTOL for a, b in zip(res.history, ro.history))
    assert rel(res.resid, ro.resid) <= RESID_RTOL
    assert np.array_equal(du.to_numpy(), uo)


def test_plain_early_exit_matches_oracle():
    n = 20
    say("plain early exit")
    h = 1.0 / (n + 1)
    u0 = synth.uniform_field(n, n, n, 2, 1, 0, 1)
    f = synth.manufactured_f(n, n, n, h)
    du, df = j3d.FArray.from_numpy(u0), j3d.FArray.from_numpy(f)
    res = j3d.poisson_solve(du, df, h, rtol=1e-6, max_sweeps=100000, check_every=10)
    uo, ro = oracle.solve_plain(u0, f, h, rtol=1e-6, check_every=10, max_sweeps=100000)
    assert ro.converged and res.converged
    assert res.sweeps == ro.sweeps
    assert rel(res.resid, ro.resid) <= RESID_RTOL and res.resid <= 1e-6 * res.norm_f
    assert np.array_equal(du.to_numpy(), uo)


@pytest.mark.parametrize("n,rtol", [(12, 1e-3), (16, 2e-5), (9, 1e-12)])
def test_plain_early_exit_every_sweep_matches_oracle(n, rtol):
    """A check after every sweep (each check reduced by a workgroup of the
    next pass, which runs before the verdict is known): the solve stops at
    the oracle's sweep with the oracle's iterate, including exits inside a
    replayed chunk."""
    say("plain early exit, check every sweep", n, rtol)
    h = 1.0 / (n + 1)
    u0 = synth.uniform_field(n, n, n, 5, 1, 0, 1)
    f = synth.manufactured_f(n, n, n, h)
    du, df = j3d.FArray.from_numpy(u0), j3d.FArray.from_numpy(f)
    res = j3d.poisson_solve(du, df, h, rtol=rtol, max_sweeps=100000, check_every=1)
    uo, ro = oracle.solve_plain(u0, f, h, rtol=rtol, check_every=1, max_sweeps=100000)
    assert ro.converged and res.converged
    assert res.sweeps == ro.sweeps
    assert len(res.history) == len(ro.history)
    assert all(rel(a, b) <= RESID_RTOL for a, b in zip(res.history, ro.history))
    assert np.array_equal(du.to_numpy(), uo)


@pytest.mark.parametrize("n,S,rtol,tune", [(64, 100, 0.0, None), (9, 1, 0.0, None), (9, 0, 0.0, None),
                                           (11, 1001, 0.0, None), (12, 100000, 1e-3, None), (10, 7, 0.0, None),
                                           (13, 13, 0.0, None),
                                           # one to sixteen wavefronts per workgroup (the reducing workgroup
                                           # stands in for 1024 / T threads), persistent grids, LDS variants
                                           (40, 50, 0.0, (1, 4, 20, 1, 2, 1)), (40, 50, 0.0, (8, 2, 6, 0, 1, 2)),
                                           (40, 50, 0.0, (2, 2, 21, 0, 1, 1)), (40, 50, 0.0, (4, 8, 20, 1, 0, 4)),
                                           (33, 40, 0.0, (1, 16, 4, 0, 2, 1))])
def test_fused_checks_equal_reduction_kernels(n, S, rtol, tune, monkeypatch):
    """The checks reduced inside the next pass give the same bits as the
    schedule with a reduction kernel per check: history, sweeps, iterate."""
    say("fused checks", n, S, rtol, tune)
    if tune is not None:
        j3d.j3d_tune_set_single(j3d.F64, n, n, n, tune)
    h = 1.0 / (n + 1)
    u0 = synth.uniform_field(n, n, n, 7, 1, 0, 1)
    f = synth.manufactured_f(n, n, n, h) if rtol > 0 else synth.uniform_field(n, n, n, 7, 2, -1, 1)
    df = j3d.FArray.from_numpy(f)
    out = []
    for fused in ("1", "0"):
        monkeypatch.setenv("J3D_SOLVE_FUSED_CHECKS", fused)
        du = j3d.FArray.from_numpy(u0)
        r = j3d.poisson_solve(du, df, h, rtol=rtol, max_sweeps=S, check_every=1)
        out.append((r.sweeps, r.converged, list(r.history), r.resid, du.to_numpy()))
    a, b = out
    assert a[0] == b[0] and a[1] == b[1] and a[3] == b[3]
    assert a[2] == b[2], "residual histories differ"
    assert np.array_equal(a[4], b[4])


@pytest.mark.parametrize("n,inner,rtol,cap", [(24, 50, 1e-8, 100000), (13, 7, 1e-10, 100000),
                                              (16, 50, 1e-14, 120), (10, 1, 1e-3, 1000), (11, 2, 1e-9, 100000),
                                              (12, 3, 1e-9, 100000), (9, 4, 1e-9, 100000), (14, 6, 1e-12, 53),
                                              (70, 50, 1e-7, 100000), (15, 5, 1e-9, 100000),
                                              (17, 9, 1e-10, 100000), (19, 10, 1e-9, 100000)])
@pytest.mark.parametrize("step", STEPS)
def test_mixed_matches_oracle(n, inner, rtol, cap, step, monkeypatch):
    monkeypatch.setenv("J3D_SOLVE_SWEEPS_PER_PASS", step)
    say("mixed", n, inner, rtol, cap, step)
    h = 1.0 / (n + 1)
    u0 = synth.uniform_field(n, n, n, 2, 1, 0, 1)
    f = synth.manufactured_f(n, n, n, h)
    du, df = j3d.FArray.from_numpy(u0), j3d.FArray.from_numpy(f)
    res = j3d.poisson_solve(du, df, h, mode=j3d.MODE_MIXED, rtol=rtol, max_sweeps=cap, inner_sweeps=inner)
    uo, ro = oracle.solve_mixed(u0, f, h, rtol=rtol, inner=inner, max_sweeps=cap)
    assert res.converged == ro.converged
    assert res.sweeps == ro.sweeps
    assert len(res.history) == len(ro.history)
    assert all(rel(a, b) <= RESID_RTOL for a, b in zip(res.history, ro.history))
    # FP32 sweeps, FP64 defects, same order on both sides: the fields agree bitwise
    assert np.array_equal(du.to_numpy(), uo)


def test_mixed_and_plain_reach_tolerance_at_same_sweep_count():
    n = 24
    say("mixed vs plain sweep count")
    h = 1.0 / (n + 1)
    u0 = synth.uniform_field(n, n, n, 2, 1, 0, 1)
    f = synth.manufactured_f(n, n, n, h)
    a, b = j3d.FArray.from_numpy(u0), j3d.FArray.from_numpy(u0)
    df = j3d.FArray.from_numpy(f)
    rp = j3d.poisson_solve(a, df, h, mode=j3d.MODE_FP64, rtol=1e-8, max_sweeps=10 ** 6, check_every=50)
    rm = j3d.poisson_solve(b, df, h, mode=j3d.MODE_MIXED, rtol=1e-8, max_sweeps=10 ** 6, inner_sweeps=50)
    assert rp.converged and rm.converged and rp.sweeps == rm.sweeps
    # the converged fields agree to the tolerance's order
    ua, ub = a.to_numpy(), b.to_numpy()
    assert np.max(np.abs(ua - ub)) <= 1e-7 * np.max(np.abs(ua))
    # both residuals verified on the CPU
    assert oracle.residual_l2(ub, f, h) <= 1e-8 * rm.norm_f * (1 + 1e-9)


def test_nonfinite_reported():
    n = 8
    u0 = np.zeros((n + 2,) * 3)
    f = synth.uniform_field(n, n, n, 3, 2, -1, 1)
    f[4, 4, 4] = np.nan
    du, df = j3d.FArray.from_numpy(u0), j3d.FArray.from_numpy(f)
    with pytest.raises(j3d.J3DError) as ei:
        j3d.poisson_solve(du, df, 0.1, rtol=1e-8, max_sweeps=50, check_every=5)
    assert ei.value.code == j3d.ENONFINITE
    r = j3d.poisson_solve(du, df, 0.1, mode=j3d.MODE_MIXED, rtol=1e-8, max_sweeps=50, raise_nonfinite=False)
    assert r.status == j3d.ENONFINITE and not r.converged


def test_warm_start_resume():
    """Solving in two halves from the returned iterate equals one solve."""
    n = 12
    h = 1.0 / 13
    u0 = synth.uniform_field(n, n, n, 6, 1, 0, 1)
    f = synth.uniform_field(n, n, n, 6, 2, -1, 1)
    a, b = j3d.FArray.from_numpy(u0), j3d.FArray.from_numpy(u0)
    df = j3d.FArray.from_numpy(f)
    j3d.poisson_solve(a, df, h, rtol=0.0, max_sweeps=60, check_every=10)
    j3d.poisson_solve(b, df, h, rtol=0.0, max_sweeps=30, check_every=10)
    j3d.poisson_solve(b, df, h, rtol=0.0, max_sweeps=30, check_every=10)
    assert np.array_equal(a.to_numpy(), b.to_numpy())


@pytest.mark.parametrize("S,every", [(1234, 2), (1001, 1), (1200, 3), (999, 4), (1100, 7), (997, 6), (1000, 10)])
@pytest.mark.parametrize("step", STEPS)
def test_plain_graph_replay_and_tail(S, every, step, monkeypatch):
    """Long solves replay a captured chunk graph, then finish directly: same
    iterate and history as the oracle, and again on a second call (cached
    graph)."""
    monkeypatch.setenv("J3D_SOLVE_SWEEPS_PER_PASS", step)
    n = 24
    say("graph replay", S, every, step)
    h = 1.0 / (n + 1)
    u0 = synth.uniform_field(n, n, n, 8, 1, 0, 1)
    f = synth.uniform_field(n, n, n, 8, 2, -1, 1)
    uo, ro = oracle.solve_plain(u0, f, h, rtol=0.0, check_every=every, max_sweeps=S)
    df = j3d.FArray.from_numpy(f)
    for rep in range(2):
        du = j3d.FArray.from_numpy(u0)
        res = j3d.poisson_solve(du, df, h, rtol=0.0, max_sweeps=S, check_every=every)
        assert res.sweeps == S and len(res.history) == len(ro.history)
        assert all(rel(a, b) <= RESID_RTOL for a, b in zip(res.history, ro.history))
        assert np.array_equal(du.to_numpy(), uo), "call %d" % rep


@pytest.mark.parametrize("step", STEPS)
def test_mixed_graph_replay_matches_oracle(step, monkeypatch):
    monkeypatch.setenv("J3D_SOLVE_SWEEPS_PER_PASS", step)
    n = 24
    say("mixed graph replay", step)
    h = 1.0 / (n + 1)
    u0 = synth.uniform_field(n, n, n, 9, 1, 0, 1)
    f = synth.uniform_field(n, n, n, 9, 2, -1, 1)
    uo, ro = oracle.solve_mixed(u0, f, h, rtol=0.0, inner=50, max_sweeps=5030)
    df = j3d.FArray.from_numpy(f)
    for rep in range(2):
        du = j3d.FArray.from_numpy(u0)
        res = j3d.poisson_solve(du, df, h, mode=j3d.MODE_MIXED, rtol=0.0, max_sweeps=5030, inner_sweeps=50)
        assert res.sweeps == ro.sweeps == 5030 and len(res.history) == len(ro.history)
        assert all(rel(a, b) <= RESID_RTOL for a, b in zip(res.history, ro.history))
        assert np.array_equal(du.to_numpy(), uo), "call %d" % rep


@pytest.mark.parametrize("mode,shape,every", [(j3d.MODE_FP64, (320, 300, 230), 5), (j3d.MODE_MIXED, (360, 350, 340), 7)])
def test_large_grids_choose_three_sweep_passes(mode, shape, every, monkeypatch):
    """Grids whose pass arrays overflow the cache (over 512 MB: FP64 u, w, f;
    FP32 r, e0, e1) run three-sweep passes by themselves: same iterate and
    history as the oracle."""
    monkeypatch.delenv("J3D_SOLVE_SWEEPS_PER_PASS", raising=False)
    nx, ny, nz = shape
    say("large solve", mode, shape, every)
    h = 1.0 / (max(shape) + 1)
    u0 = synth.uniform_field(nx, ny, nz, 10, 1, 0, 1)
    f = synth.uniform_field(nx, ny, nz, 10, 2, -1, 1)
    du, df = j3d.FArray.from_numpy(u0), j3d.FArray.from_numpy(f)
    if mode == j3d.MODE_FP64:
        assert 24 * nx * ny * nz > 512e6
        res = j3d.poisson_solve(du, df, h, rtol=0.0, max_sweeps=13, check_every=every)
        uo, ro = oracle.solve_plain(u0, f, h, rtol=0.0, check_every=every, max_sweeps=13)
    else:
        assert 12 * nx * ny * nz > 512e6
        res = j3d.poisson_solve(du, df, h, mode=j3d.MODE_MIXED, rtol=0.0, max_sweeps=2 * every,
                                inner_sweeps=every)
        uo, ro = oracle.solve_mixed(u0, f, h, rtol=0.0, inner=every, max_sweeps=2 * every)
    assert res.sweeps == ro.sweeps and len(res.history) == len(ro.history)
    assert all(rel(a, b) <= RESID_RTOL for a, b in zip(res.history, ro.history))
    assert np.array_equal(du.to_numpy(), uo)


@pytest.mark.parametrize("every", [3, 4, 5, 7])
@pytest.mark.parametrize("rtol", [0.9, 0.5, 0.2, 3e-2, 3e-3])
def test_early_exit_inside_three_sweep_passes(every, rtol):
    """Passes run straight through the checks: whichever stage of a pass forms
    the converged iterate (every position of a check in the passes of three
    occurs), and inside replayed chunks, the solve returns the oracle's
    iterate and history."""
    n = (23, 17, 20)
    say("early exit inside passes", every, rtol)
    h = 1.0 / 24
    u0 = synth.uniform_field(*n, 12, 1, 0, 1)
    f = synth.manufactured_f(*n, h)
    du, df = j3d.FArray.from_numpy(u0), j3d.FArray.from_numpy(f)
    # a first guess far off, so that the relative residual falls from about 10
    res = j3d.poisson_solve(du, df, h, rtol=rtol, max_sweeps=20000, check_every=every)
    uo, ro = oracle.solve_plain(u0, f, h, rtol=rtol, check_every=every, max_sweeps=20000)
    assert res.converged == ro.converged and res.sweeps == ro.sweeps
    assert len(res.history) == len(ro.history)
    assert all(rel(a, b) <= RESID_RTOL for a, b in zip(res.history, ro.history))
    assert rel(res.resid, ro.resid) <= RESID_RTOL
    assert np.array_equal(du.to_numpy(), uo)


# more points than the small grids that check in one-sweep passes: every
# number of sweeps left over, exits at each stage of a pass and in the sweeps
# left over, replayed chunks (S > 78)
@pytest.mark.parametrize("S,rtol", [(0, 0.0), (1, 0.0), (2, 0.0), (3, 0.0), (4, 0.0), (8, 0.0), (83, 0.0),
                                    (84, 2.0), (84, 0.9), (84, 0.6), (84, 0.5), (84, 0.4), (84, 0.05), (5, 0.6),
                                    (5, 0.5), (5, 0.4), (5, 0.32)])
def test_checks_after_every_sweep_in_three_sweep_passes(S, rtol, monkeypatch):
    n = (70, 64, 66)
    say("three checks per pass", S, rtol)
    h = 1.0 / 71
    u0 = synth.uniform_field(*n, 13, 1, 0, 1)
    f = synth.manufactured_f(*n, h) if rtol == 0.0 else synth.uniform_field(*n, 13, 2, -1, 1)
    if rtol > 0.0:  # residuals of about 1.9, 0.84, 0.56, 0.43, 0.36, 0.31, ... times the norm of f
        u0[1:-1, 1:-1, 1:-1] *= 1e-4
    df = j3d.FArray.from_numpy(f)
    uo, ro = oracle.solve_plain(u0, f, h, rtol=rtol, check_every=1, max_sweeps=S)
    for fused in ("1", "0"):
        monkeypatch.setenv("J3D_SOLVE_FUSED_CHECKS", fused)
        du = j3d.FArray.from_numpy(u0)
        res = j3d.poisson_solve(du, df, h, rtol=rtol, max_sweeps=S, check_every=1)
        assert res.converged == ro.converged and res.sweeps == ro.sweeps, fused
        assert len(res.history) == len(ro.history)
        assert all(rel(a, b) <= RESID_RTOL for a, b in zip(res.history, ro.history))
        assert np.array_equal(du.to_numpy(), uo), fused
        if fused == "1":
            first = list(res.history)
        else:
            assert first == list(res.history)


@pytest.mark.parametrize("S,every", [(4094, 1), (4095, 1), (4096, 1), (9000, 2)])
def test_long_histories(S, every):
    """Around the history length that comes back with the control block."""
    say("long history", S, every)
    n = (5, 4, 3)
    u0 = synth.uniform_field(*n, 14, 1, 0, 1)
    f = synth.uniform_field(*n, 14, 2, -1, 1)
    du, df = j3d.FArray.from_numpy(u0), j3d.FArray.from_numpy(f)
    res = j3d.poisson_solve(du, df, 0.1, rtol=0.0, max_sweeps=S, check_every=every)
    uo, ro = oracle.solve_plain(u0, f, 0.1, rtol=0.0, check_every=every, max_sweeps=S)
    assert len(res.history) == len(ro.history) == S // every + 1
    # the first hundred checks; later ones are rounding errors of a converged iterate
    assert all(rel(a, b) <= RESID_RTOL for a, b in zip(list(res.history)[:100], ro.history[:100]))
    assert np.all(np.asarray(res.history)[100:] <= np.asarray(ro.history)[100])
    assert res.resid == res.history[-1]
    assert np.array_equal(du.to_numpy(), uo)


# the iterate that converged lies inside a pass and is formed again into u:
# stages 1 and 2 of a pass of three checks (sweeps 7 and 8: the third pass,
# whose input is in the last of three arrays) and of the straight schedule
# (sweep 10 of the fourth, 5 of the second pass, whose inputs are in the other
# array); sweep 20 is formed into the other array and copied
@pytest.mark.parametrize("every,at", [(1, 7), (1, 8), (10, 10), (5, 5), (10, 20)])
def test_returns_when_the_converged_iterate_is_in_place(every, at):
    """The call blocks until u holds the reported iterate, also where the solve
    queues work after the verdict: its stream is idle at the return, and another
    stream reads the oracle's bits."""
    n = (256, 256, 252) if every == 1 else (300, 300, 200)
    say("returns when done", every, at)
    h = 1.0 / 301
    u0 = synth.uniform_field(*n, 15, 1, 0, 1)
    f = synth.uniform_field(*n, 15, 2, -1, 1)
    uo, ro = oracle.solve_plain(u0, f, h, rtol=0.0, check_every=every, max_sweeps=at)
    before, after = ro.history[at // every - 1], ro.history[at // every]
    assert after < before
    rtol = float(np.sqrt(before * after) / ro.norm_f)
    du, df = j3d.FArray.from_numpy(u0), j3d.FArray.from_numpy(f)
    got = torch.empty_like(du.storage)
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    res = j3d.poisson_solve(du, df, h, rtol=rtol, max_sweeps=1000, check_every=every, stream=side)
    idle = side.query()
    with torch.cuda.stream(other):
        got.copy_(du.storage)
    assert idle
    assert res.converged and res.sweeps == at and len(res.history) == at // every + 1
    torch.cuda.synchronize()
    du.storage.copy_(got)
    assert np.array_equal(du.to_numpy(), uo)


# checks far apart: chunks of whole check groups, with an odd number of passes
# (251: 753 sweeps in 251 passes, so that replays alternate between the arrays;
# 333: 999 in 333) and an even one whose last pass is short (1000 in 334)
@pytest.mark.parametrize("every", [251, 333, 1000])
@pytest.mark.parametrize("at", [0, 1, 2, 3, 7])
def test_checks_far_apart(every, at):
    """Early exits in the first chunks and the end of the solve, in replayed
    chunks and in the rest after them."""
    n = (40, 38, 36)
    say("checks far apart", every, at)
    h = 1.0 / 41
    u0 = synth.uniform_field(*n, 16, 1, 0, 1)
    f = synth.uniform_field(*n, 16, 2, -1, 1)
    S = 3 * every * (at + 1) // 2 + 5 if at else 4 * every + 2
    _, ro = oracle.solve_plain(u0, f, h, rtol=0.0, check_every=every, max_sweeps=S)
    rtol = 0.0
    if at and at < len(ro.history):
        assert ro.history[at] < ro.history[at - 1]
        rtol = float(np.sqrt(ro.history[at] * ro.history[at - 1]) / ro.norm_f)
    du, df = j3d.FArray.from_numpy(u0), j3d.FArray.from_numpy(f)
    res = j3d.poisson_solve(du, df, h, rtol=rtol, max_sweeps=S, check_every=every)
    uo, ro = oracle.solve_plain(u0, f, h, rtol=rtol, check_every=every, max_sweeps=S)
    assert res.converged == ro.converged == (rtol > 0.0) and res.sweeps == ro.sweeps
    assert len(res.history) == len(ro.history)
    assert all(rel(a, b) <= RESID_RTOL for a, b in zip(res.history, ro.history))
    assert rel(res.resid, ro.resid) <= RESID_RTOL
    assert np.array_equal(du.to_numpy(), uo)
