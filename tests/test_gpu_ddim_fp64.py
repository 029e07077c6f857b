"""The FP64 likelihood and steps at d = 8 on the matrix cores: the tiles that go by
differences, and the tempering step's buffers."""

import numpy as np
import pytest
import torch

from gpu_common import announce, oracle_model, rel_err
from oracle import gmm as ogmm
from oracle import smc as osmc
from workloads import make_mixture_data, theta_near_posterior

pytestmark = pytest.mark.gpu

FP64_TOL = 1e-12


@pytest.fixture(scope="module")
def smc():
    import paper_0905_2441_amd as smc
    return smc


def _loglik(smc, ctx, g, y, th):
    out = smc.smc_loglik(ctx, g, torch.as_tensor(y).cuda(), torch.as_tensor(th).cuda(), "fp64")
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("k", [1, 2, 4, 8])
@pytest.mark.parametrize("case,n,N,slices", [
    ("all", 1, 17, 0), ("all", 17, 70, 0), ("all", 1025, 65, 1), ("all", 2100, 33, 2),
    ("mixed", 1025, 65, 1), ("mixed", 1040, 16, 1), ("mixed", 2100, 130, 3), ("last", 1025, 64, 1),
    ("first", 130, 1, 1),
])
def test_tiles_by_differences(smc, k, case, n, N, slices):
    """Every tile (means hundreds of standard deviations apart), every fifth one, or
    only the first or last, with one slice of more than 64 tiles (the block after
    which a wave works the tiles off), partial tiles and columns. Plain FP64 terms:
    1e-12 as for every FP64 form."""
    announce(f"ddim fp64 differences k={k} {case} n={n} N={N} slices={slices}")
    rng = np.random.default_rng(65)
    mu = 3.0 * rng.standard_normal((k, 8))
    sigma2 = 0.003 if case == "all" else 1.0
    y = make_mixture_data(n, mu, sigma2, seed=66)
    th = theta_near_posterior(N, mu, seed=67)
    tiles = np.arange(n) // 16
    far = {"all": np.zeros(n, bool), "mixed": tiles % 5 == 3, "last": tiles == tiles[-1],
           "first": tiles == 0}[case]
    y[far, 2] += 500.0
    g = smc.Gmm.equal_weights(k, 8, sigma2)
    ctx = smc.Context(0)
    ctx.set_slices(slices)
    err = rel_err(_loglik(smc, ctx, g, y, th), ogmm.loglik(th, y, oracle_model(g)))
    ctx.check()
    assert err.max() <= FP64_TOL, float(err.max())


@pytest.mark.parametrize("what", ["nan_mean", "inf_mean", "nan_datum", "inf_datum"])
def test_values_that_are_not_finite(smc, what):
    """A NaN mean makes its own particle NaN and no other; an infinite mean is a
    component of zero density; a datum that is not finite makes every particle NaN."""
    announce(f"ddim fp64 {what}")
    rng = np.random.default_rng(68)
    mu = 3.0 * rng.standard_normal((4, 8))
    y = make_mixture_data(300, mu, 1.0, seed=69)
    th = theta_near_posterior(70, mu, seed=70)
    g = smc.Gmm.equal_weights(4, 8, 1.0)
    clean = ogmm.loglik(th, y, oracle_model(g))
    hit = np.zeros(70, bool)
    if what == "nan_mean":
        th[11, 21] = np.nan
        hit[21] = True
    elif what == "inf_mean":
        th[8:16, 21] = np.inf
        with np.errstate(invalid="ignore"):
            clean[21] = ogmm.loglik(th[:, 21:22], y, oracle_model(g))[0]
    else:
        y[37, 3] = np.nan if what == "nan_datum" else np.inf
        hit[:] = True
    ctx = smc.Context(0)
    got = _loglik(smc, ctx, g, y, th)
    assert np.array_equal(np.isnan(got), hit)
    if not hit.all():
        assert rel_err(got[~hit], clean[~hit]).max() <= FP64_TOL
    if hit.any():
        with pytest.raises(Exception, match="NaN"):
            ctx.check()
    else:
        ctx.check()


@pytest.mark.parametrize("k,n,N", [(1, 60, 65), (2, 200, 130), (8, 150, 70)])
@pytest.mark.parametrize("moves,ess_frac,slices,steps_per_call", [
    (1, 0.5, 1, 1), (3, 1.0, 1, 1), (3, 0.0, 3, 1), (1, 1.0, 3, 3), (3, 0.5, 1, 3), (0, 0.5, 0, 1)])
def test_tempering_steps_match_oracle(smc, k, n, N, moves, ess_frac, slices, steps_per_call):
    """smc_step and smc_steps at d = 8: the first move writes its proposals into the
    output population and, with one slice, its partial sums into the output
    log-likelihoods; later moves use the gather's buffers; resampling never, at every
    step (ESS below N) and by its test. Every decision, population, weight and
    count as the oracle's, eager and replayed."""
    announce(f"ddim fp64 steps k={k} n={n} N={N} moves={moves} ess={ess_frac} slices={slices}")
    mu = 3.0 * np.random.default_rng(78).standard_normal((k, 8))
    y = make_mixture_data(n, mu, 1.0, seed=79)
    betas = np.linspace(0.0, 0.01, 7)
    g = smc.Gmm.equal_weights(k, 8, 1.0)
    ref = osmc.smc_run(y, oracle_model(g), betas, N, 0.4, moves, 81, ess_frac=ess_frac,
                       resample=ess_frac > 0.0)
    for graph in (False, True):
        ctx = smc.Context(0)
        ctx.set_slices(slices)
        s = smc.SMCSampler(ctx, g, y, N, betas, 0.4, moves, 81, ess_frac=ess_frac, prec="fp64")
        r = s.run(graph=graph, steps_per_graph=steps_per_call)
        assert r["resamples"] == int(np.sum(ref["trace"]["resampled"]))
        assert r["accepted"] == int(np.sum(ref["trace"]["accepted"]))
        assert abs(r["logZ"] - ref["logZ"]) <= 1e-9 * max(1.0, abs(ref["logZ"]))
        assert np.max(np.abs(r["theta"] - ref["theta"])) <= 1e-9
        assert rel_err(r["l"], ref["l"]).max() <= 1e-10
        assert np.max(np.abs(r["W"] - ref["W"])) <= 1e-12
        assert np.max(np.abs(r["logw"] - ref["logw"])) <= 1e-8


@pytest.mark.parametrize("k,slices", [(1, 1), (4, 1), (8, 1), (8, 2)])
def test_single_move_with_one_slice(smc, k, slices):
    """A standalone move whose partial sums, of one slice, share a scratch array."""
    announce(f"ddim fp64 move k={k} slices={slices}")
    mu = 3.0 * np.random.default_rng(82).standard_normal((k, 8))
    y = make_mixture_data(90, mu, 1.0, seed=83)
    g = smc.Gmm.equal_weights(k, 8, 1.0)
    om = oracle_model(g)
    th = theta_near_posterior(130, mu, seed=84)
    l = ogmm.loglik(th, y, om)
    ctx = smc.Context(0)
    ctx.set_slices(slices)
    t, ll = torch.as_tensor(th).cuda(), torch.as_tensor(l).cuda()
    for move in (0, 1):
        rt, rl, _ = osmc.rwmh_move(th, l, y, om, 0.2, 0.1, 9, 4, move)
        smc.smc_rwmh_move(ctx, g, torch.as_tensor(y).cuda(), t, ll, 0.2, 0.1, 9, 4, move=move,
                          prec="fp64")
        th, l = rt, rl
    ctx.check()
    assert np.max(np.abs(t.cpu().numpy() - th)) <= 1e-11
    assert rel_err(ll.cpu().numpy(), l).max() <= FP64_TOL


@pytest.mark.parametrize("k,n,N", [(1, 31, 70), (1, 32, 70), (2, 63, 8193), (2, 64, 8193),
                                   (4, 63, 8192), (4, 63, 8193), (8, 15, 8193), (8, 16, 8193)])
def test_loglik_on_both_sides_of_the_short_data_rule(smc, k, n, N):
    """The VALU form below, the matrix form from there on, both as exact."""
    announce(f"ddim fp64 short data k={k} n={n} N={N}")
    mu = 3.0 * np.random.default_rng(85).standard_normal((k, 8))
    y = make_mixture_data(n, mu, 1.0, seed=86)
    th = theta_near_posterior(N, mu, seed=87)
    g = smc.Gmm.equal_weights(k, 8, 1.0)
    ctx = smc.Context(0)
    err = rel_err(_loglik(smc, ctx, g, y, th), ogmm.loglik(th, y, oracle_model(g)))
    ctx.check()
    assert err.max() <= FP64_TOL, float(err.max())


@pytest.mark.parametrize("k,n", [(1, 191), (1, 192), (2, 191), (2, 192), (4, 63), (4, 64)])
@pytest.mark.parametrize("moves,steps_per_call", [(1, 1), (3, 4)])
def test_steps_on_both_sides_of_the_short_data_rule(smc, k, n, moves, steps_per_call):
    """Single steps and chains of them, one and several moves, with either form."""
    announce(f"ddim fp64 short data steps k={k} n={n} moves={moves}")
    N = 130
    mu = 3.0 * np.random.default_rng(88).standard_normal((k, 8))
    y = make_mixture_data(n, mu, 1.0, seed=89)
    betas = np.linspace(0.0, 0.01, 9)
    g = smc.Gmm.equal_weights(k, 8, 1.0)
    ref = osmc.smc_run(y, oracle_model(g), betas, N, 0.4, moves, 90)
    s = smc.SMCSampler(smc.Context(0), g, y, N, betas, 0.4, moves, 90, prec="fp64")
    r = s.run(graph=True, steps_per_graph=steps_per_call)
    assert r["accepted"] == int(np.sum(ref["trace"]["accepted"]))
    assert r["resamples"] == int(np.sum(ref["trace"]["resampled"]))
    assert np.max(np.abs(r["theta"] - ref["theta"])) <= 1e-9
    assert rel_err(r["l"], ref["l"]).max() <= 1e-10
