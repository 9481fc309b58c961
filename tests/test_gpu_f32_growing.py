"""FP32 arithmetic with schedules whose polynomials grow on [0, 1] while the
spectrum stays where they are small: a first step (k, 0, 0) or a large quintic
and Newton-Schulz steps behind it, in every form of an FP32 call, against the
oracle at the FP32 path's bars (1e-5 relative, 2e-4 for the fast iteration,
1e-5 + 2e-6 kappa for the spectrum-aware init)."""
import numpy as np
import pytest

import synth
from oracle import fastapply as FA
from oracle import iteration as OI
from oracle import muon as MU
from oracle import spectral_init as SI
from tests.gpu_util import device_input, oracle_same_iteration, relf, to_np

pytestmark = pytest.mark.gpu

NS = (1.875, -1.25, 0.375)


def _abc(k, steps):
    """(k, 0, 0), then Newton-Schulz."""
    return np.array([(k, 0.0, 0.0)] + [NS] * (steps - 1))


@pytest.fixture(scope="module")
def pe():
    import paper_2505_16932_amd as pe
    pe.lib()
    return pe


def _gauss(seed, *shape):
    """Singular values up to 0.06 (17 x 2000) to 0.3 (40 x 40) of the norm."""
    import torch
    return device_input(synth.rng(seed).standard_normal(shape), torch.float32)


@pytest.mark.parametrize("out", ["float32", "bfloat16"])
@pytest.mark.parametrize("shape,k", [((300, 700), 8.0), ((700, 300), 8.0), ((128, 8192), 7.0), ((1024, 1024), 12.0), ((40, 40), 2.0), ((9, 50), 1.2)])
def test_growing_schedule(pe, shape, k, out):
    """(9 x 50 has fewer than 16 rows; 128 x 8192 splits its k.)"""
    import torch
    G, vals = _gauss(9000 + shape[0], *shape)
    abc = _abc(k, 5)
    X = pe.polar(G, T=5, abc=abc, compute="f32", out_dtype=getattr(torch, out))
    torch.cuda.synchronize()
    e = relf(to_np(X), oracle_same_iteration(vals, abc))
    print(f"[grow] {shape} {out} relF={e:.3e}", flush=True)
    assert e <= (1e-5 if out == "float32" else 2.0 ** -8)


def test_large_quintic_and_batch(pe):
    import torch
    abc = np.array([(20.0, -300.0, 900.0), NS, NS, NS])
    items = [_gauss(9100 + i, *sh) for i, sh in enumerate([(1024, 4096), (600, 2000), (4096, 1024), (512, 512)])]
    abc[0] *= 0.5   # 512 x 512 reaches 0.09
    Xs = pe.polar_batched([g for g, _ in items], T=4, abc=abc, compute="f32", out_dtype=torch.float32)
    torch.cuda.synchronize()
    for X, (_, v) in zip(Xs, items):
        assert relf(to_np(X), oracle_same_iteration(v, abc)) <= 1e-5


@pytest.mark.parametrize("wdtype", ["float32", "bfloat16"])
def test_growing_schedule_muon(pe, wdtype):
    import torch
    abc = _abc(8.0, 5)
    G, g = _gauss(9200, 700, 300)
    M = torch.from_numpy((0.5 * synth.rng(9201).standard_normal((700, 300))).astype(np.float32)).cuda()
    W = torch.from_numpy(synth.rng(9202).standard_normal((700, 300)).astype(np.float32)).to(getattr(torch, wdtype)).cuda()
    M0, W0 = to_np(M), to_np(W)
    pe.muon_step([G], [M], [W], lr=0.5, beta=0.9, wd=0.1, T=5, abc=abc, compute="f32")
    torch.cuda.synchronize()
    Mr, Xr, Wr = MU.muon_step(g, M0, W0, abc, lr=0.5, beta=0.9, wd=0.1)
    assert relf(to_np(M), Mr) <= 1e-6
    if wdtype == "float32":
        assert relf((0.95 * W0 - to_np(W)) / 0.5, Xr) <= 1e-5
    else:
        assert np.all(np.abs(to_np(W) - Wr) <= 2.0 ** -8 * np.abs(Wr) + 1e-6)


@pytest.mark.parametrize("force,tau", [(4, 0.0), (0, 1e-3)])
def test_growing_schedule_learned(pe, force, tau):
    """The caller's schedule as class 4, and as the fallback of class 0 (two steps
    of the l = 0.1 schedule, whose estimate is far above tau)."""
    import torch
    abc = _abc(8.0, 5)
    items = [_gauss(9300 + i, *sh) for i, sh in enumerate([(300, 700), (1500, 400)])]
    Xs = pe.polar_batched([g for g, _ in items], T=5, abc=abc, compute="f32", out_dtype=torch.float32,
                          force_class=force, fallback_tau=tau)
    torch.cuda.synchronize()
    for X, (_, v) in zip(Xs, items):
        assert relf(to_np(X), oracle_same_iteration(v, abc)) <= 1e-5


def test_growing_schedule_other_class(pe):
    """A class with fewer steps beside such a schedule: the last step copies X."""
    import torch
    G, v = _gauss(9350, 300, 700)
    X = pe.polar(G, T=5, abc=_abc(8.0, 5), compute="f32", out_dtype=torch.float32, force_class=0)
    torch.cuda.synchronize()
    assert relf(to_np(X), oracle_same_iteration(v, pe.coeffs(0.1, 5).abc[:2])) <= 1e-5


def test_growing_schedule_spectral_init(pe):
    import torch
    abc = _abc(8.0, 5)
    G, v = _gauss(9400, 300, 700)  # no outlier: the init step is the identity
    X = pe.polar(G, T=5, abc=abc, compute="f32", out_dtype=torch.float32, spectral_init=8)
    torch.cuda.synchronize()
    assert relf(to_np(X), oracle_same_iteration(v, abc)) <= 1e-5
    # an outlier, which the init step brings to 1 and the schedule to 70
    abc = np.array([(8.0, 0.0, 0.0), (1.0, -5.0, 0.08)])
    sig = np.r_[1.0, 0.03 / np.arange(2, 301)]
    G, v = device_input(synth.usv(synth.rng(9401), 300, 700, sig).G, torch.float32)
    X = pe.polar(G, T=2, abc=abc, compute="f32", out_dtype=torch.float32, spectral_init=16)
    torch.cuda.synchronize()
    A = OI.normalise(v) @ OI.normalise(v).T
    z = SI.power_lower_bound(A, 16)
    kappa = z * z / (np.trace(A) - z * z)
    e = relf(to_np(X), SI.spectrum_aware_polar_express(v, abc, iters=16))
    print(f"[grow] init relF={e:.3e} kappa={kappa:.0f}", flush=True)
    assert e <= 1e-5 + 2e-6 * kappa


@pytest.mark.parametrize("restart", [2, 3])
@pytest.mark.parametrize("shape,k", [((300, 1100), 9.0), ((1024, 4096), 16.0), ((2000, 500), 10.0)])
def test_growing_schedule_fast(pe, shape, k, restart):
    import torch
    G, v = _gauss(9500 + shape[0], *shape)
    abc = _abc(k, 5)
    X = pe.polar(G, T=5, abc=abc, compute="f32", out_dtype=torch.float32, fast_restart=restart, fast_eps=0.0)
    torch.cuda.synchronize()
    e = relf(to_np(X), FA.fast_polar_express(v, abc, restart=restart, eps=0.0))
    print(f"[grow] fast {shape} restart {restart} relF={e:.3e}", flush=True)
    assert e <= 2e-4


def _fast_segment_f32(vals, abc):
    """One segment of the fast iteration in FP32 on the CPU, in the library's form
    (D = Q - q I, products of rows by rows)."""
    X = OI.normalise(vals).astype(np.float32)
    R = X @ X.T
    D, q = np.zeros_like(R), np.float32(1.0)
    for a, b, c in np.asarray(abc, dtype=np.float32):
        B = b * R + c * (R @ R.T)
        D = a * D + q * B + D @ B.T
        P = R @ B.T
        R = a * a * R + 2 * a * P + P @ B.T
        q = np.float32(q * a)
    return q * X + D @ X


def test_fast_segment_with_a_small_polynomial_at_one(pe):
    """Four steps for [1/16, 1] leave the upper spectrum within 1e-4 of 1, where the
    fifth, (1, 10, -10), has B near 0; on the singular values below 1/16, which are
    still on their way, its B reaches 2.5.  (Segments of five steps cancel by q = 52:
    no further off than four times the same segment in FP32 on the CPU.)"""
    import torch
    abc = np.concatenate([np.asarray(pe.coeffs(1.0 / 16.0, 4).abc).reshape(4, 3), [(1.0, 10.0, -10.0)]])
    G, v = device_input(synth.usv(synth.rng(9700), 64, 200, np.geomspace(1.0, 1e-3, 64)).G, torch.float32)
    X = pe.polar(G, T=5, abc=abc, compute="f32", out_dtype=torch.float32, fast_restart=5, fast_eps=0.0)
    torch.cuda.synchronize()
    ref = FA.fast_polar_express(v, abc, restart=5, eps=0.0)
    e, bar = relf(to_np(X), ref), 4.0 * relf(_fast_segment_f32(v, abc), ref)
    print(f"[grow] small at one relF={e:.3e} bar={bar:.3e}", flush=True)
    assert e <= bar


def test_growing_schedule_plan(pe):
    """Replays of a captured plan, with other work in between."""
    import torch
    abc = _abc(8.0, 5)
    G, v = _gauss(9600, 300, 700)
    plan = pe.Plan([G], T=5, abc=abc, compute="f32", out_dtype=torch.float32)
    ref = oracle_same_iteration(v, abc)
    for _ in range(3):
        plan.outs[0].zero_()
        plan.launch(graph=True)
        torch.cuda.synchronize()
        assert relf(to_np(plan.outs[0]), ref) <= 1e-5
    plan.close()
