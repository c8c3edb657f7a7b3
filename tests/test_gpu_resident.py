"""The resident MD sub-cycle (one launch whose workgroups hold 32 beads each
and exchange positions through memory) against the fused cycle (itself bit for
bit one launch per sub-step) and against its own redo by one workgroup (a
wait limit of zero ticks sends every replica of more than one segment there),
through the C ABI: bit for bit on every population and bead field, noise and
bending on.  Chain lengths around the segments' edges, pair lists beyond the
forces a lane keeps, remote partners beyond a segment's table (the redo), the
6 x 6 window of wall sites, beads crossing periodic boundaries, uneven
ensembles by graph replay, relaxation, and the adjoint's tape."""
import numpy as np
import pytest

from paper_0711_2665_amd.workloads import C0, initial_chain, scaled

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _state(ctx, r=0):
    ctx.torch.cuda.synchronize()
    b = {k: t.cpu().numpy().copy() for k, t in ctx.beads(r).items()}
    return ctx.pops(r).double().cpu().numpy(), b


def _same(a, b, tag):
    (pa, ba), (pb, bb) = _state(*a), _state(*b)
    diff = {k: int((ba[k] != bb[k]).sum()) for k in ("r", "v", "up", "J")}
    print(f"{tag}: pops differing {int((pa != pb).sum())}, beads {diff}", flush=True)
    assert np.array_equal(pa, pb), tag
    for k in ("r", "v", "up", "J"):
        assert np.array_equal(ba[k], bb[k]), (tag, k)


def _three(monkeypatch, make, fused=10):
    """The same context with the resident cycle, its redo, and the fused one."""
    out = [make()]
    monkeypatch.setenv("LBMD_MD_WAIT_TICKS", "0")
    out.append(make())
    monkeypatch.delenv("LBMD_MD_WAIT_TICKS")
    out.append(make())
    out[2].md_fused(fused)
    return out


@pytest.mark.parametrize("nb", [1, 2, 31, 32, 33, 34, 63, 64, 65, 97, 200])
def test_segment_edges(monkeypatch, nb):
    _torch()
    from paper_0711_2665_amd import lbmd
    cfg = scaled(C0, shape=(36, 34, 40), wall_pos=20, nb=nb, init_seed=21)
    r, v = initial_chain(cfg)

    def make():
        s = lbmd.Simulation(cfg, r, v)
        s.relax(250, 1.0)
        return s
    sims = _three(monkeypatch, make)
    for n in (1, 3):
        for s in sims:
            s.couple_step(n)
        _same((sims[0],), (sims[2],), f"{nb} beads, resident against fused")
        _same((sims[1],), (sims[2],), f"{nb} beads, redo against fused")
    for s in sims:
        s.check()


@pytest.mark.parametrize("speed", [0.7, 2.0, 9.0])
def test_drifting_chain(monkeypatch, speed):
    """A uniform drift along the wall takes beads out of the lists' range: the
    cycle goes on in blocks with new lists (from the cell table, then from all
    beads), at 9 per step (0.9 per block, more than half the skin) to the redo."""
    torch = _torch()
    from paper_0711_2665_amd import lbmd
    cfg = scaled(C0, shape=(40, 40, 40), wall_pos=20, nb=600, init_seed=9)
    r, v = initial_chain(cfg)

    def make():
        s = lbmd.Simulation(cfg, r, v)
        s.relax(300, 1.0)
        vv = np.zeros((cfg["nb"], 3))
        vv[:, 1] = speed
        s.beads()["v"].copy_(torch.as_tensor(vv, device=s.device))
        return s
    sims = _three(monkeypatch, make, fused=2)
    before = sims[0].diagnostics()["rebuilds"]
    for s in sims:
        s.couple_step(3)
    d = sims[0].diagnostics()
    print({k: d[k] for k in ("rebuilds", "cell_rebuilds", "watchdog")}, "before", before, flush=True)
    assert d["rebuilds"] > before
    _same((sims[0],), (sims[2],), f"drift {speed}, resident against fused")
    _same((sims[1],), (sims[2],), f"drift {speed}, redo against fused")


def _serpentine(n, a, layers, origin):
    """n beads along a folded path of spacing a: rows of `layers` beads in
    planes of `layers` rows."""
    out = []
    for k in range(n):
        z, rem = divmod(k, layers * layers)
        y, x = divmod(rem, layers)
        if z % 2:
            y = layers - 1 - y
        if y % 2:
            x = layers - 1 - x
        out.append((x, y, z))
    return np.asarray(out, dtype=np.float64) * a + np.asarray(origin)


@pytest.mark.parametrize("rc,sigma,spacing,layers", [
    (2.0 ** (1.0 / 6.0), 1.0, 1.05, 6),     # dense: more remote partners than usual
    (2.5, 1.0, 1.25, 6),                    # r_c > 2: 6 x 6 wall window, many pairs within r_c
    (2.5, 1.0, 1.13, 5),                    # lists at their capacity: the replica goes to the redo
])
def test_dense_chains(monkeypatch, rc, sigma, spacing, layers):
    _torch()
    from paper_0711_2665_amd import lbmd
    cfg = scaled(C0, shape=(24, 24, 30), wall_pos=15, nb=200, rc=rc, sigma=sigma, eps=0.05, r0=spacing, kappa=0.5)
    r = _serpentine(200, spacing, layers, (9.3, 9.1, 16.2))     # against the wall, across its pore

    def make():
        return lbmd.Simulation(cfg, r, None)
    sims = _three(monkeypatch, make, fused=2)
    for s in sims:
        s.couple_step(2)
    print({k: sims[0].diagnostics()[k] for k in ("nbr_max", "rebuilds", "watchdog")}, flush=True)
    assert sims[0].diagnostics()["watchdog"] == sims[2].diagnostics()["watchdog"]
    if sims[0].diagnostics()["nbr_max"] <= 48:    # beyond, lists are truncated and the run is flagged
        _same((sims[0],), (sims[2],), "resident against fused")
        _same((sims[1],), (sims[2],), "redo against fused")


@pytest.mark.parametrize("axis", [0, 1, 2])
def test_chain_across_periodic_boundaries(monkeypatch, axis):
    """Positions outside the box on every axis (several periods), wall on each axis."""
    _torch()
    from paper_0711_2665_amd import lbmd
    cfg = scaled(C0, shape=(30, 32, 34), wall_axis=axis, wall_pos=16, nb=80, init_seed=5)
    r, _ = initial_chain(cfg)
    r = r + np.array([-2.0 * 30, 32.0, 3.0 * 34])

    def make():
        s = lbmd.Simulation(cfg, r, None)
        s.relax(200, 1.0)
        return s
    sims = _three(monkeypatch, make)
    for s in sims:
        s.couple_step(3)
    _same((sims[0],), (sims[2],), f"axis {axis}, resident against fused")
    _same((sims[1],), (sims[2],), f"axis {axis}, redo against fused")


@pytest.mark.parametrize("prec", ["fp64", "fp32dev"])
def test_uneven_ensemble_by_graph(monkeypatch, prec):
    _torch()
    from paper_0711_2665_amd import lbmd
    p = lbmd.LB_FP64 if prec == "fp64" else lbmd.LB_FP32_DEV
    cfgs = [scaled(C0, shape=(32, 32, 32), nb=20, seed=3, replica=0),
            scaled(C0, shape=(40, 36, 44), wall_pos=22, nb=700, seed=4, replica=1, init_seed=4),
            scaled(C0, shape=(24, 24, 24), wall_axis=-1, wall_pos=0, pore_h=0, nb=0, replica=2),
            scaled(C0, shape=(36, 36, 36), wall_pos=18, nb=260, seed=5, replica=3, init_seed=6, kT=0.0)]
    r0s = [initial_chain(c)[0] if c["nb"] > 0 else None for c in cfgs]

    def make():
        e = lbmd.Ensemble(cfgs, r0s, precision=p)
        e.relax(300, 1.0)
        return e
    ens = _three(monkeypatch, make)
    for n in (6, 3):
        ens[0].run(n, graph=True)
        ens[0].observables()
        ens[1].run(n, graph=True)
        ens[2].run(n, graph=False)
        for k in range(len(cfgs)):
            _same((ens[0], k), (ens[2], k), f"{prec} replica {k}, resident against fused")
            _same((ens[1], k), (ens[2], k), f"{prec} replica {k}, redo against fused")


def test_adjoint_tape_from_the_redo(monkeypatch):
    """The tape of the sub-steps written by the resident cycle and by its redo
    gives the same gradient."""
    torch = _torch()
    from paper_0711_2665_amd import lbmd
    cfg = scaled(C0, nb=70, shape=(36, 36, 36), wall_pos=18, init_seed=8)
    r, v = initial_chain(cfg)
    grads = []
    for wait in (None, "0"):
        if wait is not None:
            monkeypatch.setenv("LBMD_MD_WAIT_TICKS", wait)
        s = lbmd.Simulation(cfg, r, v)
        s.relax(200, 1.0)
        s.adjoint_forward(4, 2)
        g = torch.ones(cfg["nb"], 3, dtype=torch.float64, device=s.device)
        grads.append(s.adjoint_backward(g).cpu().numpy())
    assert np.isfinite(grads[0]).all() and np.abs(grads[0]).max() > 0
    assert np.array_equal(grads[0], grads[1])


def test_context_in_the_memory_of_an_earlier_one():
    """The positions that an earlier context left in the exchange are not taken
    for the new one's: every context runs one cycle of three sub-steps, the
    last two of which stay in memory that the allocator hands out again."""
    _torch()
    from paper_0711_2665_amd import lbmd
    cfg = scaled(C0, shape=(36, 36, 36), wall_pos=18, nb=200, init_seed=30)
    s = lbmd.Simulation(cfg, initial_chain(cfg)[0], None)
    s.relax(400, 1.0)
    r = _state(s)[1]["r"]
    cfg = scaled(cfg, n_sub=3, kT=0.0)
    got = []
    for fused in (0, 3):
        got.append([])
        for k in range(6):
            s = lbmd.Simulation(cfg, r + np.array([0.37 * k, 0.0, 0.0]), None)
            if fused:
                s.md_fused(fused)
            s.couple_step(1)
            got[-1].append(_state(s)[1])
            del s
    for k, (a, b) in enumerate(zip(*got)):
        for f in ("r", "v", "up", "J"):
            assert np.array_equal(a[f], b[f]), (k, f)


def test_more_segments_than_fit_use_single_launches():
    """16640 beads in 520 segments: one launch per sub-step, whose steps equal
    those of a chain alone in its context."""
    _torch()
    from paper_0711_2665_amd import lbmd
    one = scaled(C0, shape=(32, 32, 32), nb=32)
    cfgs = [scaled(one, seed=k + 1, replica=k, init_seed=k + 1) for k in range(520)]
    chains = [initial_chain(c)[0] for c in cfgs]
    e = lbmd.Ensemble(cfgs, chains, precision=lbmd.LB_FP32_DEV)
    e.relax(200, 1.0)
    e.couple_step(2)
    for k in (0, 519):
        s = lbmd.Simulation(cfgs[k], chains[k], precision=lbmd.LB_FP32_DEV)
        s.relax(200, 1.0)
        s.couple_step(2)
        _same((e, k), (s,), f"replica {k} of 520")


@pytest.mark.parametrize("M", [4, 25, 100])
def test_mts_against_single_launches(monkeypatch, M):
    """The multiple-time-step cycle (25, 4 and 1 sub-steps between kicks): a
    resident context, its redo, and the launches of a context with more
    segments than stay resident (520 of them fill chains beside the compared
    ones).  Chains of one, three and 22 segments, one that drifts out of its
    lists' range, and a dense one."""
    _torch()
    from paper_0711_2665_amd import lbmd
    kw = dict(mts_outer=M, n_sub=100)
    folded = []                                    # rows and planes of six, neighbours 1.05 apart
    for k in range(200):
        row, x = divmod(k, 6)
        z, y = divmod(row, 6)
        folded.append((5 - x if row % 2 else x, 5 - y if z % 2 else y, z))
    folded = np.asarray(folded, dtype=np.float64) * 1.05 + np.array([9.3, 9.1, 16.2])
    test = [(scaled(C0, shape=(32, 32, 32), nb=20, seed=3, replica=0, **kw), None, 0.0),
            (scaled(C0, shape=(36, 34, 30), wall_axis=1, wall_pos=17, nb=65, seed=4, replica=1, init_seed=4, **kw), None, 0.0),
            (scaled(C0, shape=(40, 36, 44), wall_pos=22, nb=700, seed=5, replica=2, init_seed=4, **kw), None, 0.0),
            (scaled(C0, shape=(40, 40, 40), wall_pos=20, nb=300, seed=6, replica=3, init_seed=9, **kw), None, 2.0),
            (scaled(C0, shape=(24, 24, 30), wall_pos=15, nb=200, seed=7, replica=4, eps=0.05, r0=1.05, kappa=0.5, **kw),
             folded, 0.0)]
    r0 = [initial_chain(c)[0] if r is None else r for c, r, _ in test]
    fill = [scaled(C0, shape=(32, 32, 32), nb=32, seed=k, replica=k, init_seed=k, **kw) for k in range(5, 525)]

    p = lbmd.LB_FP32_DEV
    e = lbmd.Ensemble([c for c, _, _ in test] + fill, r0 + [initial_chain(c)[0] for c in fill], precision=p)
    sims = []
    for wait in (None, "0"):
        if wait is not None:
            monkeypatch.setenv("LBMD_MD_WAIT_TICKS", wait)
        sims.append([lbmd.Simulation(c, r, None, precision=p) for (c, _, _), r in zip(test, r0)])
    monkeypatch.delenv("LBMD_MD_WAIT_TICKS")
    for s in (e, *sims[0], *sims[1]):
        s.relax(200, 1.0)
    for k, (_, _, speed) in enumerate(test):
        for v in [e.beads(k)["v"]] + [group[k].beads()["v"] for group in sims]:
            v[:, 0] = speed
    for n in (1, 2):
        e.couple_step(n)
        for k in range(len(test)):
            for tag, group in zip(("resident", "redo"), sims):
                group[k].couple_step(n)
                _same((group[k],), (e, k), f"M {M}, chain {k}, {tag} against launches")
    print({k: sims[0][3].diagnostics()[k] for k in ("nbr_max", "rebuilds")}, flush=True)
    assert sims[0][3].diagnostics()["rebuilds"] > 0


@pytest.mark.parametrize("nb,speed", [(2, 0.0), (31, 0.0), (32, 0.0), (33, 0.0), (64, 0.0), (65, 0.0), (150, 0.0),
                                      (181, 0.0), (200, 0.9), (200, 9.0), (512, 0.0)])
def test_rigid_chains_against_single_launches(monkeypatch, nb, speed):
    """Rigid bonds in the resident cycle and in its redo against the launches
    that a context with a harmonic chain beside the rigid one takes: chain
    lengths at the edges of the segments, of the serial solve (32 beads) and
    of the largest chain; chains that leave their lists' range."""
    _torch()
    from paper_0711_2665_amd import lbmd
    cfg = scaled(C0, shape=(40, 40, 40), wall_pos=20, nb=nb, init_seed=7, seed=5, replica=0, constraints=1)
    other = scaled(C0, shape=(20, 20, 20), wall_pos=10, nb=3, seed=6, replica=1)
    r = initial_chain(cfg)[0]
    e = lbmd.Ensemble([cfg, other], [r, initial_chain(other)[0]])
    sims = [lbmd.Simulation(cfg, r, None)]
    monkeypatch.setenv("LBMD_MD_WAIT_TICKS", "0")
    sims.append(lbmd.Simulation(cfg, r, None))
    monkeypatch.delenv("LBMD_MD_WAIT_TICKS")
    for s in (e, *sims):
        s.relax(250, 1.0)
    for tag, s in zip(("resident", "redo"), sims):
        _same((s,), (e, 0), f"{nb} rigid beads, relaxed, {tag}")
        s.beads()["v"][:, 1] = speed
    e.beads(0)["v"][:, 1] = speed
    for n in (1, 2):
        e.couple_step(n)
        for tag, s in zip(("resident", "redo"), sims):
            s.couple_step(n)
            _same((s,), (e, 0), f"{nb} rigid beads, {tag} against launches")
    for s in (e, *sims):
        s.check()
    if speed:
        assert sims[0].diagnostics()["rebuilds"] > 0
