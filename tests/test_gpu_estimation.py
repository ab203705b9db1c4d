"""GPU parity of the estimation path: the reduced-energy matrix u_kn (every
sample at every state, Estimation section) and device MBAR, plus the
whole-pipeline pin on the solvable toy (GPU sampling + u_kn + MBAR must
recover the exact free energies).

Tolerances: |u32 - u64| <= 1e-5 * beta_k * S_n (S_n the magnitude sum of
sample n's energy contributions); MBAR f on identical u_kn: 1e-7 absolute
(both float64, different reduction order); variances 1e-5 relative.
"""
import math

import numpy as np
import pytest

import oracle
import synth
from gpu_util import dev, make_context, print_case, require_gpu, torch
from oracle import estimators

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _samples(lig, rng, N, sigma=0.35):
    x = lig.x0[0][None].astype(np.float64) + rng.normal(
        scale=sigma, size=(N, lig.n_atoms, 3))
    return x.astype(np.float32)


def test_energy_matrix_matches_brute_force_ukn():
    print_case("energy_matrix c1")
    system = synth.make_system(1)
    lig, g = system.ligands[0], system.grid
    rng = np.random.default_rng(1)
    xs = _samples(lig, rng, 300)
    ctx, (lid,) = make_context(g, [lig], seed=1)
    u = ctx.energy_matrix(lid, dev(xs, torch.float32)).cpu().numpy()
    og, ol = oracle.OGrid(g), oracle.OLigand(lig)
    u64 = oracle.ukn(og, ol, xs)
    _, mags = oracle.components(og, ol, xs)
    S = mags.sum(axis=1)
    beta = 1.0 / (oracle.R_GAS * lig.T)
    assert np.all(np.abs(u - u64) <= 1e-5 * beta[:, None] * S[None, :] + 1e-12)
    ctx.close()


@pytest.mark.parametrize("atoms,N", [(31, 1), (32, 2), (32, 3), (32, 67),
                                     (33, 9), (64, 65), (65, 9)])
def test_energy_matrix_wavefront_edges(atoms, N):
    """Ligands around two samples to a wavefront (32 atoms) and one (64), and
    sample counts that leave a half, a wavefront or a group short: against
    brute force (the tolerance above), each column the bits of the sample
    alone."""
    print_case(f"energy_matrix edges {atoms} atoms {N} samples")
    g = synth.make_system(1).grid
    rng = np.random.default_rng([5, atoms, N])
    lig = synth.make_ligand(rng, atoms, 6)
    xs = _samples(lig, rng, N)
    ctx, (lid,) = make_context(g, [lig], seed=1)
    x = dev(xs, torch.float32)
    u = ctx.energy_matrix(lid, x)
    for i in {0, N // 2, N - 1}:
        assert torch.equal(ctx.energy_matrix(lid, x[i:i + 1].clone())[:, 0],
                           u[:, i])
    og, ol = oracle.OGrid(g), oracle.OLigand(lig)
    u64 = oracle.ukn(og, ol, xs)
    _, mags = oracle.components(og, ol, xs)
    beta = 1.0 / (oracle.R_GAS * lig.T)
    assert np.all(np.abs(u.cpu().numpy() - u64) <=
                  1e-5 * beta[:, None] * mags.sum(axis=1)[None, :] + 1e-12)
    ctx.close()


@pytest.mark.parametrize("atoms", [(32, 12, 31), (33, 64, 50), (32, 33, 7),
                                   (33, 32, 64), (30, 34, 70)])
def test_energy_matrix_batch_of_either_and_both_sizes(atoms):
    """Launches whose ligands all take two samples a wavefront, all one, and
    both kinds (with a larger ligand in another launch): each matrix the bits
    of the ligand's own call, which is of one kind."""
    print_case(f"energy_matrix kinds {atoms}")
    g = synth.make_system(1).grid
    rng = np.random.default_rng(atoms[0])
    ligs = [synth.make_ligand(rng, a, 6, box=8.0) for a in atoms]
    xs = [dev(_samples(l, rng, 37 + 5 * i), torch.float32)
          for i, l in enumerate(ligs)]
    ctx, ids = make_context(g, ligs, seed=1)
    for lid, x, u in zip(ids, xs, ctx.energy_matrix_batch(ids, xs)):
        assert torch.equal(u, ctx.energy_matrix(lid, x))
    ctx.close()


def test_energy_matrix_full_size_config2_sampled_entries():
    """64 states x 32000 samples (the production u_kn of the 48-atom
    system), checked on 1000 sampled entries against brute force."""
    print_case("energy_matrix c2 full size")
    system = synth.make_system(2, grid_device="cuda:0")
    lig, g = system.ligands[0], system.grid
    rng = np.random.default_rng(2)
    N = 64 * 500
    xs = _samples(lig, rng, N, sigma=0.5)
    ctx, (lid,) = make_context(g, [lig], seed=2)
    u = ctx.energy_matrix(lid, dev(xs, torch.float32))
    torch.cuda.synchronize()
    assert u.shape == (64, N)
    u = u.cpu().numpy()
    assert np.all(np.isfinite(u))
    pick = rng.choice(N, 250, replace=False)
    og, ol = oracle.OGrid(g), oracle.OLigand(lig)
    u64 = oracle.ukn(og, ol, xs[pick])
    _, mags = oracle.components(og, ol, xs[pick])
    S = mags.sum(axis=1)
    beta = 1.0 / (oracle.R_GAS * lig.T)
    assert np.all(np.abs(u[:, pick] - u64) <=
                  1e-5 * beta[:, None] * S[None, :] + 1e-12)
    ctx.close()


def test_energy_matrix_of_recorded_samples():
    print_case("energy_matrix recorded")
    system = synth.make_system(1)
    lig, g = system.ligands[0], system.grid
    ctx, (lid,) = make_context(g, [lig], seed=4, capacity=20)
    ctx.hmc_sweep(40, 10, exchange_every=1, sample_every=2)
    xs, cs = ctx.get_samples(lid)
    R, K = xs.shape[:2]
    assert R == 20
    u_rec = ctx.energy_matrix(lid, None, n_samples=R * K)
    u_exp = ctx.energy_matrix(lid, dev(xs.reshape(R * K, lig.n_atoms, 3),
                                       torch.float32))
    assert torch.equal(u_rec, u_exp)
    # without n_samples: every recorded sample
    assert ctx.n_records(lid) == R
    assert torch.equal(ctx.energy_matrix(lid), u_rec)
    (u_b,) = ctx.energy_matrix_batch([lid])
    assert torch.equal(u_b, u_rec)
    # the recorded components give the same u_kn through the affine form
    beta = 1.0 / (oracle.R_GAS * lig.T)
    c = cs.reshape(R * K, -1)
    u_aff = beta[:, None] * (c[None, :, 0] + lig.w @ c[:, 1:].T)
    S = np.abs(c).sum(axis=1)
    assert np.all(np.abs(u_rec.cpu().numpy() - u_aff) <=
                  1e-5 * beta[:, None] * S[None, :] + 1e-9)
    ctx.close()


def _mbar_both(ctx, u, Nk):
    f, var, it = ctx.mbar(dev(u, torch.float64), Nk, tol=1e-11, max_iter=200)
    f64, v64, _ = estimators.mbar(u, Nk, tol=1e-12)
    return f, var, it, f64, v64


def test_mbar_matches_oracle_harmonic():
    print_case("mbar harmonic")
    rng = np.random.default_rng(3)
    ks = np.array([1.0, 1.4, 2.0, 2.9, 4.1, 6.0])
    Nk = np.array([300, 250, 400, 350, 300, 500])
    xs = np.concatenate([rng.normal(0, 1 / math.sqrt(k), (n, 3))
                         for k, n in zip(ks, Nk)])
    u = 0.5 * ks[:, None] * (xs ** 2).sum(1)[None, :]
    ctx = __import__("paper_1507_03703_amd").Context(seed=0)
    f, var, it, f64, v64 = _mbar_both(ctx, u, Nk)
    assert np.max(np.abs(f - f64)) < 1e-7
    assert abs(var[-1] / v64 - 1) < 1e-5
    exact = 1.5 * np.log(ks / ks[0])
    assert abs(f[-1] - exact[-1]) < 3 * math.sqrt(var[-1])
    ctx.close()


def test_mbar_matches_oracle_on_sampled_ladder():
    print_case("mbar c1 ladder")
    system = synth.make_system(1)
    lig, g = system.ligands[0], system.grid
    ctx, (lid,) = make_context(g, [lig], seed=5, capacity=100)
    ctx.hmc_sweep(1000, 10, exchange_every=1, sample_every=10)
    R = 100
    K = lig.n_states
    u = ctx.energy_matrix(lid, None, n_samples=R * K)
    Nk = np.full(K, R)
    f, var, it = ctx.mbar(u, Nk, tol=1e-11, max_iter=200)
    f64, v64, _ = estimators.mbar(u.cpu().numpy(), Nk, tol=1e-12)
    assert np.max(np.abs(f - f64)) < 1e-6 * max(1.0, np.abs(f64).max())
    assert np.allclose(var[1:], [estimators.mbar_var(u.cpu().numpy(), Nk, f64,
                                                     k, 0) for k in
                                 range(1, K)], rtol=1e-5)
    ctx.close()


def test_mbar_production_ladder_full_size():
    """The 64-state production ladder (48-atom system): 5000 GPU sweeps,
    u_kn 64 x 32000 recomputed from the recorded samples, device MBAR
    against the oracle's MBAR on the same matrix."""
    print_case("mbar c2 full size")
    system = synth.make_system(2, grid_device="cuda:0")
    lig, g = system.ligands[0], system.grid
    ctx, (lid,) = make_context(g, [lig], seed=system.seed, capacity=500)
    ctx.hmc_sweep(5000, 20, exchange_every=1, sample_every=10)
    K = lig.n_states
    u = ctx.energy_matrix(lid, None, n_samples=500 * K)
    Nk = np.full(K, 500)
    f, var, it = ctx.mbar(u, Nk, tol=1e-10, max_iter=200)
    un = u.cpu().numpy()
    f64, v64, it64 = estimators.mbar(un, Nk, tol=1e-11)
    assert np.max(np.abs(f - f64)) < 1e-6 * max(1.0, np.abs(f64).max())
    assert abs(var[-1] / v64 - 1) < 1e-4
    assert np.all(np.isfinite(var))
    # warm starts (the solution, a perturbed solution, another gauge) reach
    # the same solution; from the solution itself in at most two iterations
    f2, var2, it2 = ctx.mbar(u, Nk, tol=1e-10, max_iter=200, f_init=f)
    assert it2 <= 2 and np.max(np.abs(f2 - f)) < 1e-8 * max(1.0,
                                                            np.abs(f).max())
    rng = np.random.default_rng(0)
    f3, _, it3 = ctx.mbar(u, Nk, tol=1e-10, max_iter=200,
                          f_init=f + 5.0 + rng.normal(scale=2.0, size=K))
    assert np.max(np.abs(f3 - f64)) < 1e-6 * max(1.0, np.abs(f64).max())
    assert np.array_equal(var2 > 0, var > 0)
    ctx.close()


def test_exact_toy_pipeline_gpu():
    """GPU replica-exchange HMC + u_kn + MBAR on the solvable toy recovers
    the exact f_k - f_0 (and the synthetic BPMF f_{K-1} - f_0)."""
    print_case("toy pipeline gpu")
    import sys
    import os
    sys.path.insert(0, os.path.dirname(__file__))
    from test_oracle_pipeline import toy_system, block_estimate
    grid, lig, exact = toy_system()
    ctx, (lid,) = make_context(grid, [lig], seed=2024, capacity=3000)
    K = lig.n_states
    ctx.hmc_sweep(2000, 10, exchange_every=1)
    ctx.hmc_sweep(24000, 10, exchange_every=1, sample_every=8)
    xs, _ = ctx.get_samples(lid)
    S = xs.shape[0]
    lo = grid.origin[0] + grid.spacing
    assert np.all(np.abs(xs) < abs(lo))
    u = ctx.energy_matrix(lid, None, n_samples=S * K)
    f, var, it = ctx.mbar(u, np.full(K, S), tol=1e-11)
    ukn = u.cpu().numpy()
    f_blk, sd = block_estimate(ukn, K, S)
    assert np.max(np.abs(f - f_blk)) < 1e-7
    err = f - exact
    assert np.all(np.abs(err[1:]) < 4 * sd[1:] + 1e-3), (f, exact, sd)
    st = ctx.get_stats(lid)
    assert np.all(st["ex_acc"] / st["ex_try"] > 0.05)
    ctx.close()


def _harmonic_problem(rng, K, n_per, spread):
    """K harmonic states with force constants spread over `spread` decades;
    exact f_k - f_0 = 1.5 ln(k_k / k_0)."""
    ks = np.logspace(0, spread, K)
    Nk = rng.integers(n_per // 2, n_per + 1, K)
    xs = np.concatenate([rng.normal(0, 1 / math.sqrt(k), (n, 3))
                         for k, n in zip(ks, Nk)])
    return 0.5 * ks[:, None] * (xs ** 2).sum(1)[None, :], Nk


def test_mbar_batch_equals_lone_solves():
    """A batch mixing every register-tile class of the accumulation (K = 12,
    24, 40, 70), a one-state problem, a padded leading dimension and a
    problem far from overlap (fixed-point steps first) gives each problem
    bit for bit what a lone solve gives, with or without warm starts, and
    the oracle's MBAR within the float64 tolerance."""
    print_case("mbar batch")
    rng = np.random.default_rng(11)
    probs = [_harmonic_problem(rng, 12, 300, 1.0),
             _harmonic_problem(rng, 24, 200, 1.5),
             _harmonic_problem(rng, 1, 50, 0.0),
             _harmonic_problem(rng, 40, 120, 2.0),
             _harmonic_problem(rng, 70, 60, 2.5),
             _harmonic_problem(rng, 6, 80, 4.0)]
    us = []
    for p, (u, _) in enumerate(probs):
        if p == 1:      # leading dimension larger than N
            buf = torch.zeros((u.shape[0], u.shape[1] + 37),
                              dtype=torch.float64, device="cuda:0")
            buf[:, :u.shape[1]] = dev(u, torch.float64)
            us.append(buf[:, :u.shape[1]])
        else:
            us.append(dev(u, torch.float64))
    Nks = [nk for _, nk in probs]
    ctx = __import__("paper_1507_03703_amd").Context(seed=0)
    batch = ctx.mbar_batch(us, Nks, tol=1e-11, max_iter=200)
    lone = [ctx.mbar(u, nk, tol=1e-11, max_iter=200) for u, nk in
            zip(us, Nks)]
    for p, ((fb, vb, ib), (fl, vl, il)) in enumerate(zip(batch, lone)):
        assert np.array_equal(fb, fl) and np.array_equal(vb, vl), p
        assert ib == il, p
    assert batch[2][2] == 0 and batch[2][0].tolist() == [0.0]
    for p, (u, nk) in enumerate(probs):
        if u.shape[0] == 1:
            continue
        f64, _, _ = estimators.mbar(u, nk, tol=1e-12)
        assert np.max(np.abs(batch[p][0] - f64)) < 1e-7 * max(
            1.0, np.abs(f64).max()), p
    # warm starts for some problems only
    init = [None if p % 2 else batch[p][0] + 0.3 for p in range(len(us))]
    wb = ctx.mbar_batch(us, Nks, tol=1e-11, max_iter=200, f_init=init)
    for p, (u, nk) in enumerate(zip(us, Nks)):
        wl = ctx.mbar(u, nk, tol=1e-11, max_iter=200, f_init=init[p])
        assert np.array_equal(wb[p][0], wl[0]) and wb[p][2] == wl[2], p
        assert np.array_equal(wb[p][1], wl[1]), p
    # argument errors name the problem and compute nothing
    bad = [np.array(n) for n in Nks]
    bad[3] = bad[3] + 1
    with pytest.raises(RuntimeError, match="problem 3"):
        ctx.mbar_batch(us, bad)
    assert ctx.mbar_batch([], []) == []
    ctx.close()


@pytest.mark.parametrize("K,per", [
    (2, 2), (2, 700), (3, 43), (15, 17), (16, 8), (17, 9), (31, 33), (32, 64),
    (33, 31), (47, 11), (48, 12), (49, 13), (63, 16), (64, 17), (65, 9),
    (80, 5), (96, 11), (97, 6), (112, 8), (113, 7), (127, 9), (128, 12)])
def test_mbar_tile_edges(K, per):
    """One state short of, at and past every 16-state tile, both kernels of
    the pass (up to three tiles and more) and every register block of the
    solve, with sample counts that leave partial chunks: the free energies
    and the last state's variance are the oracle's, to the tolerances of the
    solves above (1e-7 kT, 1e-5 relative)."""
    print_case("mbar tiles", K, per)
    rng = np.random.default_rng([K, per])
    u, Nk = _harmonic_problem(rng, K, per, 1.0 + 0.01 * K)
    ctx = __import__("paper_1507_03703_amd").Context(seed=0)
    f, var, it, f64, v64 = _mbar_both(ctx, u, Nk)
    assert np.max(np.abs(f - f64)) < 1e-7 * max(1.0, np.abs(f64).max())
    if np.isfinite(var[-1]):
        assert abs(var[-1] / v64 - 1) < 1e-5
    assert 0 < it < 200
    ctx.close()


@pytest.mark.parametrize("K,per", [
    (2, 40), (3, 43), (15, 17), (16, 20), (17, 19), (31, 33), (33, 31),
    (48, 22), (49, 23), (64, 17), (65, 19), (80, 15), (97, 16), (113, 17),
    (128, 14)])
@pytest.mark.parametrize("infinite", [False, True])
def test_mbar_every_variance_at_tile_edges(K, per, infinite):
    """The whole diagonal of the in-register inverse around its blocks'
    edges, and with infinite energies of some samples in foreign states (a
    clash), in the last state among them, whose energies the lanes past it
    repeat.  The states overlap, so the Hessian at the oracle's solution is
    well conditioned and every variance has to be finite: f to 1e-7 kT and
    the variances to 1e-5 relative, as in the solves above."""
    print_case("mbar variances", K, per, infinite)
    rng = np.random.default_rng([7, K, per])
    u, Nk = _harmonic_problem(rng, K, per, 0.5)
    if infinite:
        own = np.repeat(np.arange(K), Nk)
        hit = rng.random(u.shape) < 0.02
        hit[-1] |= rng.random(u.shape[1]) < 0.3
        hit[own, np.arange(u.shape[1])] = False
        u = np.where(hit, np.inf, u)
    ctx = __import__("paper_1507_03703_amd").Context(seed=0)
    f, var, it = ctx.mbar(dev(u, torch.float64), Nk, tol=1e-11, max_iter=200)
    f64, _, _ = estimators.mbar(u, Nk, tol=1e-12)
    a = (np.log(Nk) + f64)[:, None] - u
    W = np.exp(a - np.logaddexp.reduce(a, axis=0))
    H = (np.diag(W.sum(1)) - W @ W.T)[1:, 1:]
    assert np.linalg.cond(H) < 1e5
    want = np.diag(np.linalg.inv(H)) - 1.0 / Nk[1:] - 1.0 / Nk[0]
    assert np.max(np.abs(f - f64)) < 1e-7 * max(1.0, np.abs(f64).max())
    assert np.all(np.isfinite(var)) and var[0] == 0.0
    assert np.allclose(var[1:], want, rtol=1e-5, atol=1e-12)
    ctx.close()
