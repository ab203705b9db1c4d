"""GPU parity of the sampler against the FP64 oracle: HMC sweeps (velocity
Verlet + Metropolis, Sampling section), replica exchange (Eq. repXacc),
sample recording, checkpoint/resume and determinism.

Lock-step parity (tests/lockstep.py): before every sweep the oracle is set
to the GPU's state, both run one sweep with the same Philox streams, and the
results must agree: positions to 1e-4 A, accept decisions exactly except
where the oracle's own margin |ln u + beta dH| < 1e-3 (there float32
rounding may decide), state maps exactly unless an exchange exponent lies
within 1e-6 of its uniform.
"""
import dataclasses

import numpy as np
import pytest

import oracle
import synth
from gpu_util import dev, make_context, print_case, require_gpu, torch
from lockstep import lockstep

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _lockstep(g, lig, seed, n_sweeps, nleap, label, x0=None, waves=0):
    print_case("lockstep", label, "waves", waves)
    if x0 is not None:
        lig.x0 = x0.astype(np.float32)
    ctx, (lid,) = make_context(g, [lig], seed=seed)
    ctx.set_waves(waves)
    if waves:
        assert ctx.get_waves(lid) == max(waves, -(-lig.n_atoms // 64))
    n = lockstep(ctx, oracle.OGrid(g), [(lid, lig)], seed, n_sweeps, nleap,
                 label)
    stats = ctx.get_stats(lid)
    assert stats["hmc_try"].sum() == n_sweeps * lig.n_states
    ctx.close()
    return n[lid]


@pytest.mark.parametrize("waves", [0, 1, 2, 4])
def test_lockstep_config1(waves):
    system = synth.make_system(1)
    n = _lockstep(system.grid, system.ligands[0], system.seed, 6,
                  system.n_leapfrog, "c1", waves=waves)
    assert n >= 3


def test_lockstep_config2_full_size():
    """The benchmark's production workload at full size (48 atoms, 64
    replicas, 128^3 x 3 grids, 20-step trials) in the launch shape the
    benchmark times (automatic wavefronts, the single-ligand kernel)."""
    system = synth.make_system(2, grid_device="cuda:0")
    lig = system.ligands[0]
    n = _lockstep(system.grid, lig, system.seed, 3, system.n_leapfrog,
                  "config 2 full size")
    assert n >= 1


def test_lockstep_replicas_outside_grid_and_restrained():
    system = synth.make_system(1)
    lig = system.ligands[0]
    x0 = lig.x0.astype(np.float64).copy()
    x0[1] += np.array([6.5, 0, 0])      # beyond the grid edge, d > d0
    x0[5] += np.array([0, -4.0, 4.0])
    _lockstep(system.grid, lig, 11, 4, 10, "outside", x0=x0)


@pytest.mark.parametrize("waves", [2, 4])
def test_lockstep_ligand_wider_than_a_wavefront(waves):
    rng = np.random.default_rng(4)
    lig = synth.make_ligand(rng, 90, 4, box=9.0)
    system = synth.make_system(1)
    _lockstep(system.grid, lig, 21, 3, 8, "90 atoms", waves=waves)


def test_lockstep_five_channels():
    rng = np.random.default_rng(5)
    C = 5
    g = synth.random_grid(rng, n=(48, 48, 48), spacing=0.25,
                          origin=(-5.875,) * 3, n_channels=C,
                          transform=(4, 0, 0, 0, 4))
    g.nodes *= 0.3
    lig = synth.make_ligand(rng, 20, 6, n_channels=C)
    lig.scale[:, 3:] = rng.normal(scale=0.2, size=(20, 2))
    _lockstep(g, lig, 31, 3, 10, "C=5")


def test_exchange_decisions_bitwise():
    rng = np.random.default_rng(6)
    K = 16
    T, w = synth.ladder(K)
    lig = synth.toy_ligand(np.array([[0.0, 0, 0], [1.5, 0, 0]]), [[0, 1]],
                           10.0, T, w[:, 0])
    grid = synth.linear_field_grid(8, 1.0, (0.5, 0.0, 0.0), 0.0)
    ctx, (lid,) = make_context(grid, [lig], seed=99)
    og, ol = oracle.OGrid(grid), oracle.OLigand(lig)
    for trial in range(24):
        print_case("exchange", trial)
        comps = rng.normal(scale=3.0, size=(K, 4))
        sor = rng.permutation(K).astype(np.int32)
        counter = int(rng.integers(0, 1000))
        scheme = trial % 2
        max_sep = 1 + trial % 5
        n_sweeps = (1, 2, 3, 25)[(trial // 2) % 4]
        ctx.set_replicas(lid, lig.x0, sor, comps, counter)
        ctx.exchange(lid, scheme=scheme, max_sep=max_sep, n_sweeps=n_sweeps)
        st = ctx.get_replicas(lid)
        s = oracle.Sampler(og, ol, seed=99, lig_id=lid, x0=lig.x0)
        s.comps = np.ascontiguousarray(comps)
        s.state = sor.copy()
        s.rep_of_state = np.ascontiguousarray(np.argsort(sor).astype(np.int32))
        s.sweep_count = counter
        s.exchange(scheme=scheme, max_sep=max_sep, n_sweeps=n_sweeps)
        assert np.array_equal(st["state_of_replica"], s.state), trial
    ctx.close()


@pytest.mark.parametrize("K", [64, 256, 300])
def test_exchange_decisions_bitwise_large_ladders(K):
    """All-separation sweeps at the staged kernel's limit (256 states) and
    beyond it (one thread, global memory): labels and attempt counts equal
    the oracle's."""
    print_case("exchange large ladder", K)
    rng = np.random.default_rng(K)
    T, w = synth.ladder(K)
    lig = synth.toy_ligand(np.array([[0.0, 0, 0], [1.5, 0, 0]]), [[0, 1]],
                           10.0, T, w[:, 0])
    grid = synth.linear_field_grid(8, 1.0, (0.5, 0.0, 0.0), 0.0)
    ctx, (lid,) = make_context(grid, [lig], seed=7)
    og, ol = oracle.OGrid(grid), oracle.OLigand(lig)
    comps = rng.normal(scale=2.0, size=(K, 4))
    sor = rng.permutation(K).astype(np.int32)
    ctx.set_replicas(lid, lig.x0, sor, comps, 11)
    ctx.exchange(lid, scheme=1, max_sep=5, n_sweeps=3)
    st = ctx.get_replicas(lid)
    s = oracle.Sampler(og, ol, seed=7, lig_id=lid, x0=lig.x0)
    s.comps = np.ascontiguousarray(comps)
    s.state = sor.copy()
    s.rep_of_state = np.ascontiguousarray(np.argsort(sor).astype(np.int32))
    s.sweep_count = 11
    s.exchange(scheme=1, max_sep=5, n_sweeps=3)
    assert np.array_equal(st["state_of_replica"], s.state)
    stats = ctx.get_stats(lid)
    assert np.array_equal(stats["ex_try"], s.ex_try)
    assert np.array_equal(stats["ex_acc"], s.ex_acc)
    assert stats["ex_acc"].sum() > 0
    ctx.close()



def _exchange_ligand(K, C):
    """A ligand with K states on C channels: the two-atom toy on the linear
    ladder (C = 3) or a config-1 ligand with the soft grids on their
    schedule (C = 5)."""
    if C == 3:
        T, w = synth.ladder(K)
        lig = synth.toy_ligand(np.array([[0.0, 0, 0], [1.5, 0, 0]]),
                               [[0, 1]], 10.0, T, w[:, 0])
        return synth.linear_field_grid(8, 1.0, (0.5, 0.0, 0.0), 0.0), lig
    system = synth.make_system(1)
    g, (lig,) = synth.add_soft_grids(system.grid, system.ligands[:1])
    T, w = synth.soft_schedule(K)
    lig = dataclasses.replace(
        lig, T=T, w=w, dt=np.ones(K),
        x0=np.repeat(lig.x0[:1], K, axis=0).astype(np.float32))
    return g, lig


@pytest.mark.parametrize("K,C", [(40, 3), (163, 5)])
@pytest.mark.parametrize("mode", ["all_accepted", "all_rejected",
                                  "long_runs"])
def test_exchange_runs_edge_cases(K, C, mode):
    """All-separation sweeps in which every swap is accepted (equal energies:
    each chain carries its first replica to its top), none is (non-finite
    energies) or nearly all are (long runs of accepted swaps), on the
    energy-table path (40 states) and the staged-component path (163 states,
    five channels): labels and counts equal the oracle's."""
    print_case("exchange runs", K, C, mode)
    g, lig = _exchange_ligand(K, C)
    rng = np.random.default_rng(K + C)
    comps = rng.normal(scale=0.02, size=(K, 1 + C))
    if mode == "all_accepted":
        comps[:] = 0.0
    elif mode == "all_rejected":
        comps[:, 0] = np.inf
    sor = rng.permutation(K).astype(np.int32)
    ctx, (lid,) = make_context(g, [lig], seed=13)
    ctx.set_replicas(lid, lig.x0, sor, comps, 5)
    ctx.exchange(lid, scheme=1, max_sep=5, n_sweeps=25)
    st = ctx.get_replicas(lid)
    s = oracle.Sampler(oracle.OGrid(g), oracle.OLigand(lig), seed=13,
                       lig_id=lid, x0=lig.x0)
    s.comps = np.ascontiguousarray(comps)
    s.state = sor.copy()
    s.rep_of_state = np.ascontiguousarray(np.argsort(sor).astype(np.int32))
    s.sweep_count = 5
    s.exchange(scheme=1, max_sep=5, n_sweeps=25)
    assert np.array_equal(st["state_of_replica"], s.state)
    stats = ctx.get_stats(lid)
    assert np.array_equal(stats["ex_try"], s.ex_try)
    assert np.array_equal(stats["ex_acc"], s.ex_acc)
    n_try = 25 * (K - 1)
    assert stats["ex_try"].sum() == n_try
    if mode == "all_accepted":
        assert stats["ex_acc"].sum() == n_try
    elif mode == "all_rejected":
        assert stats["ex_acc"].sum() == 0
        assert np.array_equal(st["state_of_replica"], sor)
    else:
        assert stats["ex_acc"].sum() > 0.9 * n_try
    ctx.close()


@pytest.mark.parametrize("K,C,max_sep", [
    (2, 3, 5), (3, 5, 5), (9, 3, 9), (10, 5, 20), (63, 5, 5), (64, 3, 12),
    (65, 5, 5), (66, 3, 1), (127, 3, 2), (128, 5, 5), (129, 5, 9),
    (193, 3, 7), (255, 5, 3), (256, 5, 300)])
@pytest.mark.parametrize("scale", [0.05, 0.6, 6.0])
def test_exchange_walk_block_edges(K, C, max_sep, scale):
    """All-separation sweeps where the walk's blocks of 64 positions, its
    steps decided ahead and its wavefronts run out: chains one position
    short of, at and past a block, separations past the block's wavefronts
    and past the ladder, run lengths from one swap to several blocks.
    Labels and counts equal the oracle's."""
    print_case("exchange walk", K, C, max_sep, scale)
    g, lig = _exchange_ligand(K, C)
    rng = np.random.default_rng([K, C, int(10 * scale)])
    comps = rng.normal(scale=scale, size=(K, 1 + C))
    sor = rng.permutation(K).astype(np.int32)
    ctx, (lid,) = make_context(g, [lig], seed=29)
    ctx.set_replicas(lid, lig.x0, sor, comps, 8)
    n_sweeps = 2 if max_sep > 12 else 6
    ctx.exchange(lid, scheme=1, max_sep=max_sep, n_sweeps=n_sweeps)
    st = ctx.get_replicas(lid)
    s = oracle.Sampler(oracle.OGrid(g), oracle.OLigand(lig), seed=29,
                       lig_id=lid, x0=lig.x0)
    s.comps = np.ascontiguousarray(comps)
    s.state = sor.copy()
    s.rep_of_state = np.ascontiguousarray(np.argsort(sor).astype(np.int32))
    s.sweep_count = 8
    s.exchange(scheme=1, max_sep=max_sep, n_sweeps=n_sweeps)
    assert np.array_equal(st["state_of_replica"], s.state)
    stats = ctx.get_stats(lid)
    assert np.array_equal(stats["ex_try"], s.ex_try)
    assert np.array_equal(stats["ex_acc"], s.ex_acc)
    ctx.close()


@pytest.mark.parametrize("K,C,max_sep", [
    (10, 3, 300), (17, 5, 16), (64, 3, 9), (65, 3, 17), (73, 5, 18),
    (163, 3, 40), (192, 5, 17), (193, 3, 25), (255, 5, 254)])
@pytest.mark.parametrize("scale", [0.02, 0.6, 6.0])
def test_exchange_far_separations(K, C, max_sep, scale):
    """All-separation sweeps past the separations that are walked by a
    wavefront per class: classes of one to twenty states walked by a lane
    each, runs that end at once and runs that go past the steps decided
    ahead.  Labels and counts equal the oracle's."""
    print_case("exchange far", K, C, max_sep, scale)
    g, lig = _exchange_ligand(K, C)
    rng = np.random.default_rng([3, K, C, int(100 * scale)])
    comps = rng.normal(scale=scale, size=(K, 1 + C))
    sor = rng.permutation(K).astype(np.int32)
    ctx, (lid,) = make_context(g, [lig], seed=31)
    ctx.set_replicas(lid, lig.x0, sor, comps, 8)
    ctx.exchange(lid, scheme=1, max_sep=max_sep, n_sweeps=3)
    st = ctx.get_replicas(lid)
    s = oracle.Sampler(oracle.OGrid(g), oracle.OLigand(lig), seed=31,
                       lig_id=lid, x0=lig.x0)
    s.comps = np.ascontiguousarray(comps)
    s.state = sor.copy()
    s.rep_of_state = np.ascontiguousarray(np.argsort(sor).astype(np.int32))
    s.sweep_count = 8
    s.exchange(scheme=1, max_sep=max_sep, n_sweeps=3)
    assert np.array_equal(st["state_of_replica"], s.state)
    stats = ctx.get_stats(lid)
    assert np.array_equal(stats["ex_try"], s.ex_try)
    assert np.array_equal(stats["ex_acc"], s.ex_acc)
    ctx.close()


@pytest.mark.parametrize("Ks,C,max_sep", [
    ((4,), 5, 3), ((8,), 3, 7), ((9,), 5, 8), ((17,), 3, 5), ((32,), 5, 5),
    ((33,), 3, 5), ((8, 32), 3, 5), ((4, 33), 5, 5), ((8, 40), 3, 9)])
@pytest.mark.parametrize("scale", [0.02, 0.6])
def test_exchange_short_ladders(Ks, C, max_sep, scale):
    """All-separation sweeps of ladders around 32 states, whose classes of up
    to eight positions are walked without doublings, and of launches with
    ladders on either side of that and of the far separations' line.  Labels
    and counts equal the oracle's."""
    print_case("exchange short", Ks, C, max_sep, scale)
    made = [_exchange_ligand(K, C) for K in Ks]
    g, ligs = made[0][0], [lig for _, lig in made]
    ctx, ids = make_context(g, ligs, seed=33)
    want = []
    for lid, lig, K in zip(ids, ligs, Ks):
        rng = np.random.default_rng([4, K, C, int(100 * scale)])
        comps = rng.normal(scale=scale, size=(K, 1 + C))
        sor = rng.permutation(K).astype(np.int32)
        ctx.set_replicas(lid, lig.x0, sor, comps, 8)
        s = oracle.Sampler(oracle.OGrid(g), oracle.OLigand(lig), seed=33,
                           lig_id=lid, x0=lig.x0)
        s.comps = np.ascontiguousarray(comps)
        s.state = sor.copy()
        s.rep_of_state = np.ascontiguousarray(np.argsort(sor).astype(np.int32))
        s.sweep_count = 8
        s.exchange(scheme=1, max_sep=max_sep, n_sweeps=25)
        want.append(s)
    ctx.exchange(-1, scheme=1, max_sep=max_sep, n_sweeps=25)
    for lid, s in zip(ids, want):
        assert np.array_equal(ctx.get_replicas(lid)["state_of_replica"],
                              s.state)
        stats = ctx.get_stats(lid)
        assert np.array_equal(stats["ex_try"], s.ex_try)
        assert np.array_equal(stats["ex_acc"], s.ex_acc)
    ctx.close()


def test_exchange_far_separations_cost_no_more_than_near_ones():
    """A separation with many short classes is not dearer than one with few
    long ones (a wavefront for each of them, eight at a time, made it five
    times as dear): time a separation over all 255 of 256 states, against
    twice the time a separation over the nearest five."""
    print_case("exchange far time")
    g, lig = _exchange_ligand(256, 3)
    ctx, (lid,) = make_context(g, [lig], seed=37)

    def us(max_sep, n_sweeps):
        best = float("inf")
        for _ in range(10):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            ctx.exchange(lid, scheme=1, max_sep=max_sep, n_sweeps=n_sweeps)
            b.record()
            b.synchronize()
            best = min(best, 1e3 * a.elapsed_time(b))
        return best / (max_sep * n_sweeps)
    assert us(255, 1) < 2 * us(5, 25)
    ctx.close()


def test_checkpoint_resume_is_bitwise():
    print_case("checkpoint")
    system = synth.make_system(1)
    lig, g = system.ligands[0], system.grid
    a, (la,) = make_context(g, [lig], seed=7, capacity=8)
    a.hmc_sweep(8, 10, exchange_every=1, sample_every=2)
    ra = a.get_replicas(la)
    xa, ca = a.get_samples(la)
    b, (lb,) = make_context(g, [lig], seed=7, capacity=8)
    b.hmc_sweep(4, 10, exchange_every=1, sample_every=2)
    ck = b.get_replicas(lb)
    b.close()
    c, (lc,) = make_context(g, [lig], seed=7, capacity=8)
    c.set_replicas(lc, ck["x"], ck["state_of_replica"], ck["comps"],
                   ck["counter"])
    c.hmc_sweep(4, 10, exchange_every=1, sample_every=2)
    rc = c.get_replicas(lc)
    xc, cc = c.get_samples(lc)
    for key in ("x", "state_of_replica", "comps"):
        assert np.array_equal(ra[key], rc[key]), key
    assert rc["counter"] == 8
    # the resumed run recorded the second half of the samples
    assert np.array_equal(xa[2:], xc[:2]) and np.array_equal(ca[2:], cc[:2])
    a.close()
    c.close()


def test_same_seed_same_bits_and_recorded_samples():
    print_case("determinism")
    system = synth.make_system(1)
    lig, g = system.ligands[0], system.grid
    outs = []
    for _ in range(2):
        ctx, (lid,) = make_context(g, [lig], seed=system.seed, capacity=5)
        ctx.hmc_sweep(10, 10, exchange_every=1, sample_every=2)
        st = ctx.get_replicas(lid)
        xs, cs = ctx.get_samples(lid)
        outs.append((st, xs, cs))
        # recorded sample k of a round is the configuration of the replica
        # in state k at that time; the last round equals the final state
        ros = np.argsort(st["state_of_replica"])
        assert np.array_equal(xs[-1], st["x"][ros])
        assert np.array_equal(cs[-1], st["comps"][ros])
        ctx.close()
    (a, xa, ca), (b, xb, cb) = outs
    for key in ("x", "state_of_replica", "comps"):
        assert np.array_equal(a[key], b[key])
    assert np.array_equal(xa, xb) and np.array_equal(ca, cb)


@pytest.mark.parametrize("waves", [2, 4])
def test_records_of_a_ligand_wider_than_a_wavefront(waves):
    """Samples recorded inside multi-sweep calls (the exchange and record of
    a sweep run in the next sweep's blocks) by replicas of several
    wavefronts: every recorded configuration carries the components the
    oracle computes for it, and the last round is the final state."""
    print_case("records 90 atoms", waves)
    rng = np.random.default_rng(14)
    lig = synth.make_ligand(rng, 90, 6, box=9.0)
    system = synth.make_system(1)
    g = system.grid
    ctx, (lid,) = make_context(g, [lig], seed=23, capacity=12)
    ctx.set_waves(waves)
    ctx.hmc_sweep(16, 6, exchange_every=1, sample_every=2)
    ctx.hmc_sweep(8, 6, exchange_every=1, sample_every=2)
    xs, cs = ctx.get_samples(lid)
    st = ctx.get_replicas(lid)
    assert xs.shape[0] == 12 and np.all(np.isfinite(xs))
    ros = np.argsort(st["state_of_replica"])
    assert np.array_equal(xs[-1], st["x"][ros])
    assert np.array_equal(cs[-1], st["comps"][ros])
    og, ol = oracle.OGrid(g), oracle.OLigand(lig)
    X = xs.reshape(-1, lig.n_atoms, 3)
    t, m, _ = oracle.energy_batch(og, ol, X, np.zeros((len(X), og.nc)))
    ref = np.concatenate([t[:, :4].sum(1, keepdims=True), t[:, 4:4 + og.nc]],
                         axis=1)
    S = m.sum(axis=1)
    assert np.all(np.abs(cs.reshape(len(X), -1) - ref) <= 1e-5 * S[:, None]
                  + 1e-9)
    ctx.close()


def test_nonfinite_positions_are_rejected_and_counted():
    print_case("nonfinite")
    system = synth.make_system(1)
    lig, g = system.ligands[0], system.grid
    ctx, (lid,) = make_context(g, [lig], seed=3)
    x = lig.x0.copy()
    x[2, 4, 1] = np.nan
    ctx.set_replicas(lid, x, np.arange(lig.n_states), None, 0)
    ctx.hmc_sweep(3, 10, exchange_every=1)
    st = ctx.get_stats(lid)
    assert st["nonfinite"] == 3
    assert st["hmc_try"].sum() == 3 * lig.n_states
    rep = ctx.get_replicas(lid)
    assert np.isnan(rep["x"][2, 4, 1])
    assert np.all(np.isfinite(np.delete(rep["x"], 2, axis=0)))
    ctx.close()


def test_single_state_ligand_and_capacity_error():
    print_case("K=1")
    system = synth.make_system(1)
    rng = np.random.default_rng(12)
    lig = synth.make_ligand(rng, 12, 1)
    ctx, (lid,) = make_context(system.grid, [lig], seed=3, capacity=2)
    ctx.hmc_sweep(4, 5, exchange_every=1, sample_every=2)
    st = ctx.get_stats(lid)
    assert st["hmc_try"][0] == 4 and len(st["ex_try"]) == 0
    import paper_1507_03703_amd as pkg
    with pytest.raises(pkg.BPMFError) as ei:
        ctx.hmc_sweep(2, 5, sample_every=1)
    assert ei.value.code == -1 and "capacity" in str(ei.value)
    ctx.close()


def test_validation_errors():
    import paper_1507_03703_amd as pkg
    system = synth.make_system(1)
    lig = system.ligands[0]
    ctx = pkg.Context(seed=1)
    with pytest.raises(pkg.BPMFError) as ei:
        ctx.ligand_setup(lig)
    assert ei.value.code == -4          # no grid yet
    bad = system.grid.nodes.copy()
    bad[0, 0, 0, 0] = -1.0               # negative quartic root
    with pytest.raises(pkg.BPMFError) as ei:
        ctx.grid_upload(bad, system.grid.origin, 0.25, (4, 0, 0))
    assert ei.value.code == -1 and "quartic" in str(ei.value)
    with pytest.raises(pkg.BPMFError):
        ctx.grid_upload(system.grid.nodes, system.grid.origin, -0.25,
                        (4, 0, 0))
    g = system.grid
    ctx.grid_upload(g.nodes, g.origin, g.spacing, g.transform)
    import copy
    l2 = copy.deepcopy(lig)
    l2.bonds = l2.bonds.copy()
    l2.bonds[0, 1] = lig.n_atoms       # index out of range
    with pytest.raises(pkg.BPMFError) as ei:
        ctx.ligand_setup(l2)
    assert "out of range" in str(ei.value)
    l3 = copy.deepcopy(lig)
    l3.angles = l3.angles.copy()
    l3.angles[0, 2] = l3.angles[0, 0]  # repeated atom
    with pytest.raises(pkg.BPMFError) as ei:
        ctx.ligand_setup(l3)
    assert "repeated" in str(ei.value)
    l4 = copy.deepcopy(lig)
    l4.T = l4.T.copy()
    l4.T[3] = 0.0
    with pytest.raises(pkg.BPMFError):
        ctx.ligand_setup(l4)
    lid = ctx.ligand_setup(lig)
    with pytest.raises(pkg.BPMFError):
        ctx.hmc_sweep(1, 0)
    with pytest.raises(pkg.BPMFError):
        ctx.set_replicas(lid, lig.x0, np.zeros(lig.n_states, np.int32))
    with pytest.raises(pkg.BPMFError):
        ctx.exchange(5)
    for n in (0, 1025):
        with pytest.raises(pkg.BPMFError):
            ctx.exchange(lid, scheme=1, max_sep=2, n_sweeps=n)
    for kw in (dict(exchange_sweeps=-1), dict(exchange_sweeps=1025),
               dict(exchange_scheme=0, exchange_sweeps=2)):
        kw.setdefault("exchange_scheme", 1)
        with pytest.raises(pkg.BPMFError) as ei:
            ctx.hmc_sweep(1, 5, max_sep=2, **kw)
        assert "exchange_sweeps" in str(ei.value)
    with pytest.raises(pkg.BPMFError) as ei:
        ctx.grid_upload(g.nodes, g.origin, g.spacing, g.transform)
    assert ei.value.code == -4
    ctx.close()


def test_repeated_exchange_sweeps_inside_sweeps():
    """Sweeps with scheme 1 and 25 exchange sweeps per due exchange (the
    paper's iteration): the labelling after each sweep is the oracle's 25
    exchange sweeps applied to the labelling before it and the sweep's
    post-HMC components, bitwise; the attempt counts add up."""
    print_case("exchange sweeps in sweeps")
    system = synth.make_system(1)
    lig, g = system.ligands[0], system.grid
    og, ol = oracle.OGrid(g), oracle.OLigand(lig)
    ctx, (lid,) = make_context(g, [lig], seed=41)
    s = oracle.Sampler(og, ol, seed=41, lig_id=lid, x0=lig.x0)
    moved = 0
    for sweep in range(6):
        st0 = ctx.get_replicas(lid)
        ctx.hmc_sweep(1, 10, exchange_every=1, exchange_scheme=1, max_sep=5,
                      exchange_sweeps=25)
        st1 = ctx.get_replicas(lid)
        s.comps = np.ascontiguousarray(st1["comps"].copy())
        s.state = np.ascontiguousarray(
            st0["state_of_replica"].astype(np.int32))
        s.rep_of_state = np.ascontiguousarray(
            np.argsort(s.state).astype(np.int32))
        s.sweep_count = int(st0["counter"])
        s.exchange(scheme=1, max_sep=5, n_sweeps=25)
        assert np.array_equal(st1["state_of_replica"], s.state), sweep
        moved += int(not np.array_equal(st0["state_of_replica"],
                                        st1["state_of_replica"]))
    stats = ctx.get_stats(lid)
    assert np.array_equal(stats["ex_try"], s.ex_try)
    assert np.array_equal(stats["ex_acc"], s.ex_acc)
    assert stats["ex_try"].sum() == 6 * 25 * (lig.n_states - 1)
    assert moved > 0
    ctx.close()


@pytest.mark.parametrize("exchange_sweeps", [1, 25])
def test_exchange_sweeps_graph_replays_match_plain_launches(exchange_sweeps):
    """Scheme-1 sweeps replayed from captured graphs (chunks of 8 sweeps, and
    units closed by external moves) equal plain launches bitwise, with and
    without repeated exchange sweeps."""
    print_case("exchange sweeps graph", exchange_sweeps)
    system = synth.make_system(1)
    lig, g = system.ligands[0], system.grid
    runs = []
    for chunk in (0, 8):
        ctx, (lid,) = make_context(g, [lig], seed=19, capacity=40)
        ctx.set_graph(chunk)
        states = []
        for rep in range(3):
            ctx.hmc_sweep(16, 10, exchange_every=1, exchange_scheme=1,
                          max_sep=5, sample_every=2,
                          exchange_sweeps=exchange_sweeps)
            states.append(ctx.get_replicas(lid))
            ctx.hmc_sweep(4, 10, exchange_every=2, exchange_scheme=1,
                          max_sep=3, exchange_sweeps=exchange_sweeps,
                          external_moves=3, external_k_max=2)
            states.append(ctx.get_replicas(lid))
        xs, cs = ctx.get_samples(lid)
        runs.append((states, xs, cs, ctx.get_stats(lid)))
        ctx.close()
    (sa, xa, ca, ta), (sb, xb, cb, tb) = runs
    for a, b in zip(sa, sb):
        for key in ("x", "state_of_replica", "comps", "counter"):
            assert np.array_equal(a[key], b[key]), key
    assert np.array_equal(xa, xb) and np.array_equal(ca, cb)
    for key in ("hmc_acc", "hmc_try", "ex_acc", "ex_try"):
        assert np.array_equal(ta[key], tb[key]), key
    n_ex = 3 * (16 + 2) * exchange_sweeps * (lig.n_states - 1)
    assert ta["ex_try"].sum() == n_ex


def test_graph_replays_match_plain_launches():
    """Sweeps replayed from a captured hipGraph (chunks of 8 sweeps, with the
    fused exchange/record tail) are bitwise identical to plain launches,
    replay after replay, with eager work and synchronisation in between."""
    print_case("graph replay")
    system = synth.make_system(1)
    lig, g = system.ligands[0], system.grid
    runs = []
    for chunk in (0, 8):
        ctx, (lid,) = make_context(g, [lig], seed=17, capacity=40)
        ctx.set_graph(chunk)
        states = []
        for rep in range(5):
            ctx.hmc_sweep(16, 10, exchange_every=1, sample_every=2)
            st = ctx.get_replicas(lid)               # synchronises
            ctx.exchange(lid, scheme=1, max_sep=3)   # eager work between
            states.append(st)
        xs, cs = ctx.get_samples(lid)
        runs.append((states, xs, cs, ctx.get_stats(lid)))
        ctx.close()
    (sa, xa, ca, ta), (sb, xb, cb, tb) = runs
    for a, b in zip(sa, sb):
        for key in ("x", "state_of_replica", "comps", "counter"):
            assert np.array_equal(a[key], b[key]), key
    assert np.array_equal(xa, xb) and np.array_equal(ca, cb)
    for key in ("hmc_acc", "hmc_try", "ex_acc", "ex_try"):
        assert np.array_equal(ta[key], tb[key]), key
