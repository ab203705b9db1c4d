"""GPU parity of the intramolecular nonbonded / implicit-solvent terms
(pairs.hip) against the FP64 oracle (oracle/pairs.py): the four energies
per configuration and the forces against the oracle's central differences,
for a 24-atom ligand (one wavefront), a 90-atom ligand (two), and a
three-atom case whose close, large descreening spheres reach every branch of
the descreening integral (an atom inside another's sphere, a sphere inside
an atom's own radius).

Tolerances: each energy within 1e-5 of the magnitude sum of its
contributions (the workload's relative 1e-5 made well-posed under
cancellation, as for the grid and bonded energies); forces within 1e-4 of
the largest component of the oracle's central differences (+2e-3 kJ/mol/A
for the differences' own truncation and rounding)."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import dev, make_context, print_case, require_gpu, torch
from lockstep import lockstep
from oracle import external as Ex
from oracle import pairs as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _oracle_params(p, n):
    ex, o4 = O.masks(n, p["exclusions"], p["pairs14"])
    q = dict(p)
    q.update(excluded=ex, one_four=o4)
    return q


def _check(ctx, lid, xs, p, fd_atoms=None):
    n = xs.shape[1]
    terms, F = ctx.pair_evaluate(lid, dev(xs, torch.float32))
    terms, F = terms.cpu().numpy(), F.cpu().numpy()
    t2, _ = ctx.pair_evaluate(lid, dev(xs, torch.float32), forces=False)
    assert np.array_equal(t2.cpu().numpy(), terms)
    po = _oracle_params(p, n)
    for c in range(len(xs)):
        x = xs[c].astype(np.float64)
        ref, mag = O.energy_terms(x, po, magnitudes=True)
        # |E32 - E64| <= 1e-5 S per energy, S the sum of the magnitudes of
        # its contributions (1e-9 kJ/mol absolute for sums that vanish)
        assert np.all(np.abs(terms[c] - ref) <= 1e-5 * mag + 1e-9), \
            (c, terms[c], ref, np.abs(terms[c] - ref) / mag)
        atoms = range(n) if fd_atoms is None else fd_atoms
        Fr = np.zeros((n, 3))
        for i in atoms:
            for d in range(3):
                h = 1e-5
                xp, xm = x.copy(), x.copy()
                xp[i, d] += h
                xm[i, d] -= h
                Fr[i, d] = -(O.energy_terms(xp, po).sum() -
                             O.energy_terms(xm, po).sum()) / (2 * h)
        idx = list(atoms)
        scale = np.abs(Fr[idx]).max()
        err = np.abs(F[c][idx] - Fr[idx]).max()
        assert err <= 1e-4 * scale + 2e-3, (c, err, scale)


def test_pair_terms_24_atoms():
    print_case("pairs 24 atoms")
    system = synth.make_system(1)
    lig, g = system.ligands[0], system.grid
    ctx, (lid,) = make_context(g, [lig], seed=1)
    p = synth.pair_params(lig, seed=1)
    ctx.pair_setup(lid, p)
    rng = np.random.default_rng(4)
    xs = (lig.x0[:3] + rng.normal(scale=0.15, size=(3, lig.n_atoms, 3))
          ).astype(np.float32)
    _check(ctx, lid, xs, p)
    ctx.close()


def test_pair_terms_90_atoms_two_wavefronts():
    print_case("pairs 90 atoms")
    rng = np.random.default_rng(12)
    lig = synth.make_ligand(rng, 90, 2)
    system = synth.make_system(1)
    ctx, (lid,) = make_context(system.grid, [lig], seed=1)
    p = synth.pair_params(lig, seed=2)
    ctx.pair_setup(lid, p)
    xs = (lig.x0[:2] + rng.normal(scale=0.1, size=(2, 90, 3))
          ).astype(np.float32)
    _check(ctx, lid, xs, p, fd_atoms=[0, 17, 45, 89])
    ctx.close()


@pytest.mark.parametrize("n,N", [(3, 86), (31, 9), (32, 8), (33, 8), (64, 3),
                                 (64, 4), (65, 4), (128, 3)])
def test_pair_terms_packing_edges(n, N):
    """Sizes around a mask word, a wavefront and the largest whose derivatives
    are kept, with the last workgroup full or short: the first and the last
    configuration against the oracle, and each the bits of itself alone."""
    print_case(f"pairs packing {n} atoms {N} configurations")
    rng = np.random.default_rng([6, n])
    lig = synth.make_ligand(rng, n, 2, box=8.0)
    system = synth.make_system(1)
    ctx, (lid,) = make_context(system.grid, [lig], seed=1)
    p = synth.pair_params(lig, seed=3)
    ctx.pair_setup(lid, p)
    xs = (lig.x0[0] + rng.normal(scale=0.1, size=(N, n, 3))).astype(np.float32)
    _check(ctx, lid, xs[[0, N - 1]], p, fd_atoms=[0, n - 1])
    x = dev(xs, torch.float32)
    terms, F = ctx.pair_evaluate(lid, x)
    for c in {0, N // 2, N - 1}:
        t1, F1 = ctx.pair_evaluate(lid, x[c:c + 1].clone())
        assert torch.equal(t1[0], terms[c]) and torch.equal(F1[0], F[c])
    ctx.close()


def test_pair_terms_close_spheres_reach_every_branch():
    print_case("pairs close spheres")
    x = np.array([[0.0, 0.0, 0.0], [0.35, 0.0, 0.0], [0.0, 2.6, 0.3]])
    lig = synth.toy_ligand(x, [[0, 1]], 10.0, np.array([300.0]),
                           np.array([1.0]))
    system = synth.make_system(1)
    ctx, (lid,) = make_context(system.grid, [lig], seed=1)
    p = dict(charge=np.array([0.4, -0.3, 0.2]), sigma=np.array([3.0, 3.2, 3.4]),
             eps=np.array([0.1, 0.2, 0.15]), rho=np.array([1.2, 1.8, 1.5]),
             S=np.array([0.8, 1.9, 0.5]), exclusions=np.array([[0, 1]]),
             pairs14=np.zeros((0, 2), np.int32), lj14=0.5, el14=1 / 1.2,
             eps_solute=1.0, eps_solvent=78.5, gamma=0.0225936, probe=1.4)
    # atom 0 sits inside atom 1's descreening sphere (s = 1.9 x 1.71 > r +
    # rt_0); atom 1 sees atom 0's small sphere partly inside its own radius
    assert 1.9 * (1.8 - 0.09) > 0.35 + (1.2 - 0.09)
    ctx.pair_setup(lid, p)
    rng = np.random.default_rng(5)
    xs = (x[None] + rng.normal(scale=0.02, size=(4, 3, 3))).astype(np.float32)
    _check(ctx, lid, xs, p)
    ctx.close()


def test_pair_setup_replaces_earlier_parameters():
    """A second bpmf_pair_setup replaces the first: evaluations then equal
    those of a context that only ever had the second parameters."""
    print_case("pairs re-setup")
    system = synth.make_system(1)
    lig, g = system.ligands[0], system.grid
    p1 = synth.pair_params(lig, seed=1)
    p2 = synth.pair_params(lig, seed=2)
    p2["eps_solvent"] = 40.0
    xs = dev(lig.x0[:2], torch.float32)
    ca, (la,) = make_context(g, [lig], seed=1)
    ca.pair_setup(la, p1)
    ca.pair_setup(la, p2)
    ta, fa = ca.pair_evaluate(la, xs)
    cb, (lb,) = make_context(g, [lig], seed=1)
    cb.pair_setup(lb, p2)
    tb, fb = cb.pair_evaluate(lb, xs)
    assert torch.equal(ta, tb) and torch.equal(fa, fb)
    ca.close()
    cb.close()


def test_pair_setup_errors():
    print_case("pairs errors")
    import paper_1507_03703_amd as pkg
    system = synth.make_system(1)
    lig = system.ligands[0]
    ctx, (lid,) = make_context(system.grid, [lig], seed=1)
    x = dev(lig.x0[:1], torch.float32)
    with pytest.raises(pkg.BPMFError) as ei:
        ctx.pair_evaluate(lid, x)
    assert ei.value.code == -4
    p = synth.pair_params(lig)
    bad = dict(p)
    bad["rho"] = np.full(lig.n_atoms, 0.05)
    with pytest.raises(pkg.BPMFError):
        ctx.pair_setup(lid, bad)
    bad = dict(p)
    bad["exclusions"] = np.array([[0, lig.n_atoms]])
    with pytest.raises(pkg.BPMFError):
        ctx.pair_setup(lid, bad)
    ctx.close()


# --------------------------------------------------------------------------
# pair terms inside the sampled energy (bpmf_pair_sample): the Full
# pathway's ligand energy in HMC, exchange, u_kn and the rigid moves
# --------------------------------------------------------------------------

def _full_pathway_system(n=24, K=6, seed=31):
    """A ligand grown without nonbonded clashes (atoms three or more bonds
    apart at least 3 A apart, 2.6 A above 32 atoms), its pair parameters,
    and a 64^3 receptor
    grid of 300 point atoms kept 3 A from its atoms."""
    rng = np.random.default_rng(seed)
    box, sep = (10.0, 3.0) if n <= 32 else (12.0, 2.6)
    lig = synth.make_ligand(rng, n, K, box=box, far_sep=sep)
    nn, h = 64, 0.25
    edge = (nn - 1) * h
    pts, q, sig, eps = synth.make_receptor(np.random.default_rng(seed + 1),
                                           300, edge, 0.3 * edge,
                                           avoid_xyz=lig.x0[0])
    nodes = synth.grids_from_points(pts, q, sig, eps, nn, h)
    grid = synth.Grid((nn,) * 3, (-(nn - 1) * h / 2,) * 3, h, (4, 0, 0),
                      nodes)
    return grid, lig, synth.pair_params(lig, seed=seed)


@pytest.mark.parametrize("n,waves", [(24, 0), (24, 2), (70, 0)])
def test_pair_terms_in_the_sampled_energy(n, waves):
    """Components after switching the terms on, lock-step sweeps with them
    (HMC force and energy, exchange, records), u_kn of samples, external
    moves, and switching them off again, each against the oracle with the
    same pair terms in the ligand's energy."""
    print_case("pairs in the energy", n, waves)
    g, lig, p = _full_pathway_system(n)
    og = oracle.OGrid(g)
    on, off = oracle.OLigand(lig, pairs=p), oracle.OLigand(lig)
    ctx, (lid,) = make_context(g, [lig], seed=17)
    ctx.set_waves(waves)
    ctx.pair_setup(lid, p)
    ctx.pair_sample(lid, True)

    def check_comps(ol):
        st = ctx.get_replicas(lid)
        c, m = oracle.components(og, ol, st["x"])
        assert np.all(np.abs(st["comps"] - c) <= 1e-5 * m.sum(1)[:, None] +
                      1e-9)

    check_comps(on)
    n_clear = lockstep(ctx, og, [(lid, lig)], 17, 3, 8, "pairs",
                       pairs={lid: p})
    assert n_clear[lid] >= 1
    # u_kn of perturbed configurations
    rng = np.random.default_rng(3)
    xs = (lig.x0[0][None] + rng.normal(scale=0.15, size=(12, n, 3))
          ).astype(np.float32)
    u = ctx.energy_matrix(lid, dev(xs, torch.float32)).cpu().numpy()
    u64 = oracle.ukn(og, on, xs)
    _, mags = oracle.components(og, on, xs)
    beta = 1.0 / (oracle.R_GAS * lig.T)
    assert np.all(np.abs(u - u64) <= 1e-5 * beta[:, None] *
                  mags.sum(1)[None, :] + 1e-12)
    # external moves (rigid: the pair energy is the cached one)
    st = ctx.get_replicas(lid)
    ctx.external_move(lid, n_moves=3, k_max=lig.n_states, sigma=0.3)
    st2 = ctx.get_replicas(lid)
    checked = 0
    for r in range(lig.n_states):
        k = st["state_of_replica"][r]
        xo, n_acc, lns = Ex.external_moves(og, on, st["x"][r], k, 17, lid, r,
                                           st["counter"], 3, 0.3)
        if min(abs(lu - la) for la, lu in lns) < 5e-2:
            continue
        checked += 1
        assert np.max(np.abs(st2["x"][r] - xo)) < 2e-4, r
    assert checked >= 2
    ctx.pair_sample(lid, False)
    check_comps(off)
    ctx.close()


@pytest.mark.parametrize("n,waves", [(3, 8), (25, 8), (26, 4), (65, 8)])
def test_pair_slices_of_uneven_length(n, waves):
    """Slices of a thread's partners that are shorter than, longer than and no
    multiple of the three taken side by side (down to an empty one): lock-step
    sweeps against the oracle."""
    print_case("pair slices", n, waves)
    g, lig, p = _full_pathway_system(n, K=3)
    og = oracle.OGrid(g)
    ctx, (lid,) = make_context(g, [lig], seed=18)
    ctx.set_waves(waves)
    ctx.pair_setup(lid, p)
    ctx.pair_sample(lid, True)
    lockstep(ctx, og, [(lid, lig)], 18, 2, 5, "pairs", pairs={lid: p})
    ctx.close()


@pytest.mark.parametrize("n,waves", [(3, 8), (4, 2), (5, 2), (8, 4), (9, 4),
                                     (15, 8), (16, 8), (17, 8)])
def test_pair_partners_two_at_a_time(n, waves):
    """Ligands around two partners a thread, which take them two at a time when
    every ligand of the launch does: the replicas are those of the same ligand
    swept beside a larger one, three at a time, bit for bit."""
    print_case("pair partners", n, waves)
    g, lig, p = _full_pathway_system(n, K=4)
    _, large, pl = _full_pathway_system(24, K=2)

    def swept(*others):
        ctx, ids = make_context(g, [lig] + [o for o, _ in others], seed=19)
        ctx.set_waves(waves)
        for lid, q in zip(ids, [p] + [q for _, q in others]):
            ctx.pair_setup(lid, q)
            ctx.pair_sample(lid, True)
        ctx.hmc_sweep(6, 8)
        st = ctx.get_replicas(ids[0])
        ctx.close()
        return st
    a = swept((large, pl))
    for b in (swept(), swept((lig, p))):
        for k in ("x", "state_of_replica", "comps"):
            assert np.array_equal(a[k], b[k]), k


def test_pair_sample_needs_parameters():
    print_case("pair_sample errors")
    g, lig, p = _full_pathway_system(12, K=2)
    ctx, (lid,) = make_context(g, [lig], seed=1)
    with pytest.raises(RuntimeError, match="no pair parameters"):
        ctx.pair_sample(lid, True)
    ctx.pair_sample(lid, False)   # nothing to take out
    ctx.close()
