"""What the resident MD sub-cycle's first pass holds, and what takes over
where it does not: bit for bit the other forms of the cycle, through the C
ABI, for chains that lie along the wall."""
import numpy as np
import pytest

from paper_0711_2665_amd.workloads import C0, PAPER_LJ, initial_chain, scaled

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
        assert np.isfinite(ba[k]).all() and np.array_equal(ba[k], bb[k]), (tag, k)


def _flat(n, a, row, origin):
    """n beads in rows of `row`, forth and back, spacing a, in the plane z = origin[2]."""
    out = [(k % row if k // row % 2 == 0 else row - 1 - k % row, k // row, 0) for k in range(n)]
    return np.asarray(out, dtype=np.float64) * a + np.asarray(origin)


@pytest.mark.parametrize("rc,spacing,offset,height", [
    (2.0, 1.0, (0.07, 0.48), 0.0),     # 14 wall sites within r_c of every bead, the most there are
    (2.5, 1.25, (0.1, 0.2), 0.9),
    (2.5, 2.0, (0.5, 0.5), 0.0),       # 21 within 2.5
    (3.0, 2.0, (0.5, 0.5), 0.0),       # 32 within 3, the most there are
])
def test_chain_along_the_wall(rc, spacing, offset, height):
    _torch()
    from paper_0711_2665_amd import lbmd
    cfg = scaled(C0, shape=(64, 64, 24), wall_pos=12, nb=100, rc=rc, eps=1e-6, r0=spacing, kappa=0.5)
    r = _flat(100, spacing, 12, (2 + offset[0], 2 + offset[1], 12 + height))
    sims = [lbmd.Simulation(cfg, r, None) for _ in range(2)]
    sims[1].md_fused(2)
    for n in (1, 2):
        for s in sims:
            s.couple_step(n)
        _same((sims[0],), (sims[1],), f"r_c {rc}, resident against fused")
    for s in sims:
        s.check()


@pytest.mark.parametrize("rigid", [0, 1])
def test_redos_of_contexts_side_by_side(monkeypatch, rigid):
    """Every cycle of a chain of 16 segments goes to the redo (no wait lasts),
    in three contexts on streams of their own at once; the chains drift, so the
    redo builds new lists while other segments are on their way out."""
    torch = _torch()
    from paper_0711_2665_amd import lbmd
    cfg = scaled(C0, shape=(40, 40, 40), wall_pos=20, nb=500, init_seed=9, constraints=rigid)
    r, _ = initial_chain(cfg)

    def make():
        s = lbmd.Simulation(cfg, r, None)
        s.relax(250, 1.0)
        s.beads()["v"][:, 1] = 0.9
        s.torch.cuda.synchronize()
        return s
    want = make()
    monkeypatch.setenv("LBMD_MD_WAIT_TICKS", "0")
    sims = []
    for _ in range(3):
        with torch.cuda.stream(torch.cuda.Stream()):
            sims.append(make())
    for _ in range(3):
        for s in sims:
            s.couple_step(1)
        want.couple_step(1)
    for k, s in enumerate(sims):
        _same((s,), (want,), f"context {k}, redo against resident")
        s.check()
        assert s.diagnostics()["rebuilds"] > 0


def test_bonds_that_cannot_be_met_are_flagged(monkeypatch):
    """Beads thrown 300 bond lengths apart in half a sub-step: the projection
    does not converge, and the watchdog says so in the resident cycle, in its
    redo and in the launches (with a harmonic chain beside)."""
    torch = _torch()
    from paper_0711_2665_amd import lbmd
    cfg = scaled(C0, shape=(40, 40, 40), wall_pos=20, nb=70, init_seed=7, constraints=1, kT=0.0)
    other = scaled(C0, shape=(20, 20, 20), wall_pos=10, nb=3, replica=1)
    r = initial_chain(cfg)[0]
    sims = [lbmd.Ensemble([cfg, other], [r, initial_chain(other)[0]]), lbmd.Simulation(cfg, r, None)]
    monkeypatch.setenv("LBMD_MD_WAIT_TICKS", "0")
    sims.append(lbmd.Simulation(cfg, r, None))
    v = np.random.default_rng(1).normal(0.0, 6e4, (70, 3))
    for s in sims:
        s.relax(100, 1.0)
        assert s.diagnostics()["watchdog"] == 0
        s.beads(0)["v"].copy_(torch.as_tensor(v, device=s.device))
        s.couple_step(1)
        assert s.diagnostics()["watchdog"] & 2


def test_more_than_32_pairs_of_a_bead_in_a_redo(orc, monkeypatch):
    """45 beads within r_c of one another (44 list partners each, within the 48
    that a list holds): the resident cycle, its redo and the fused cycle (whose
    blocks hold 16 close partners, so one workgroup redoes them) equal the
    oracle bit for bit, without noise and bending."""
    _torch()
    from paper_0711_2665_amd import lbmd
    cfg = scaled(C0, shape=(24, 24, 24), wall_axis=-1, wall_pos=0, pore_h=0, nb=45, rc=3.0, sigma=0.4, eps=0.01, r0=0.5,
                 kT=0.0, kappa=0.0)
    r = []
    for k in range(45):
        row, x = divmod(k, 4)
        z, y = divmod(row, 4)
        r.append((3 - x if row % 2 else x, 3 - y if z % 2 else y, z))
    r = np.asarray(r, dtype=np.float64) * 0.5 + np.array([11.13, 10.37, 11.29])
    assert np.linalg.norm(r[:, None] - r[None], axis=2).max() < 2.9
    o = orc.Oracle(cfg, r, np.zeros_like(r))
    sims = [lbmd.Simulation(cfg, r, None) for _ in range(2)]
    sims[1].md_fused(2)
    monkeypatch.setenv("LBMD_MD_WAIT_TICKS", "0")
    sims.append(lbmd.Simulation(cfg, r, None))
    o.couple_step(3)
    ob = o.beads()
    for tag, s in zip(("resident", "fused", "redo"), sims):
        s.couple_step(3)
        b = _state(s)[1]
        print(tag, {k: int((b[k] != ob[k]).sum()) for k in ("r", "v", "up", "J")}, s.diagnostics()["nbr_max"], flush=True)
        s.check()
        for k in ("r", "v", "up", "J"):
            assert np.array_equal(b[k], ob[k]), (tag, k)


def _passes(s, n):
    """Passes of n coupled steps."""
    a = s.md_passes()
    s.couple_step(n)
    return {k: x - a[k] for k, x in s.md_passes().items()}


def test_which_pass_ran(monkeypatch):
    """The counters of the passes: an ordinary chain stays in the first one, a
    drifting one goes on in the second, a very fast one and every chain of more
    than one segment that may not wait end in the redo; the fused cycle and a
    context with too many segments run no pass."""
    _torch()
    from paper_0711_2665_amd import lbmd

    def make(nb, speed=0.0, **kw):
        cfg = scaled(C0, shape=(40, 40, 40), wall_pos=20, nb=nb, init_seed=9, **kw)
        s = lbmd.Simulation(cfg, initial_chain(cfg)[0], None)
        s.relax(1000, 1.0)
        if speed:
            s.beads()["v"][:, 1] = speed
        return s
    for nb, kw in ((20, {}), (300, {}), (300, dict(constraints=1)), (300, dict(mts_outer=5, **PAPER_LJ))):
        assert _passes(make(nb, **kw), 3) == {"cycles": 3, "second": 0, "redone": 0}, (nb, kw)
    assert _passes(make(300, 2.0), 3) == {"cycles": 3, "second": 3, "redone": 0}
    assert _passes(make(300, 9.0), 3) == {"cycles": 3, "second": 3, "redone": 0}
    assert _passes(make(300, 0.9, constraints=1), 2) == {"cycles": 2, "second": 2, "redone": 0}
    fused = make(300)
    fused.md_fused(10)
    assert _passes(fused, 2) == {"cycles": 0, "second": 0, "redone": 0}
    monkeypatch.setenv("LBMD_MD_WAIT_TICKS", "0")
    assert _passes(make(32), 2) == {"cycles": 2, "second": 0, "redone": 0}
    assert _passes(make(33), 2) == {"cycles": 2, "second": 2, "redone": 2}


@pytest.mark.parametrize("rc,spacing,height,second", [(2.0, 2.0, 0.0, 0), (2.5, 1.25, 0.9, 3), (3.0, 2.0, 0.0, 3)])
def test_chain_along_the_wall_is_not_redone(rc, spacing, height, second):
    """14 wall sites per bead stay in the first pass; more go on in the second."""
    _torch()
    from paper_0711_2665_amd import lbmd
    cfg = scaled(C0, shape=(64, 64, 24), wall_pos=12, nb=100, rc=rc, eps=1e-6, r0=spacing, kappa=0.5)
    s = lbmd.Simulation(cfg, _flat(100, spacing, 12, (2.5, 2.5, 12 + height)), None)
    assert _passes(s, 3) == {"cycles": 3, "second": second, "redone": 0}


def _cube(n, a, edge, origin):
    """n beads folded into a cube of `edge` beads a side, spacing a, every bond of length a."""
    out = []
    for k in range(n):
        row, x = divmod(k, edge)
        z, y = divmod(row, edge)
        out.append((edge - 1 - x if row % 2 else x, edge - 1 - y if z % 2 else y, z))
    return np.asarray(out, dtype=np.float64) * a + np.asarray(origin)


@pytest.mark.parametrize("nb,edge,speed,rc", [
    (600, 9, 0.0, 2.0 ** (1 / 6)),      # more than 144 remote partners of a segment
    (2080, 13, 0.0, 2.0 ** (1 / 6)),    # 65 segments: the words by way of the first one
    (2048, 13, 3.0, 2.0 ** (1 / 6)),    # 64, each reading all; new lists in the cycle
    (2500, 14, 9.0, 2.0 ** (1 / 6)),    # the same with 79, from the table and from all beads
    (300, 7, 0.7, 2.0),                 # many pairs, along the wall and through its window
])
def test_dense_chains_in_the_second_pass(nb, edge, speed, rc):
    """Chains folded densely stay out of the one-workgroup redo, bit for bit the
    fused cycle's (whose blocks they leave for its redo)."""
    _torch()
    from paper_0711_2665_amd import lbmd
    a = 1.13 if rc < 2.0 else 1.45
    cfg = scaled(C0, shape=(40, 40, 40), wall_pos=10, nb=nb, rc=rc, eps=0.05, r0=a, kappa=0.5)
    r = _cube(nb, a, edge, (11.3, 10.1, 10.93))
    sims = [lbmd.Simulation(cfg, r, None) for _ in range(2)]
    sims[1].md_fused(2)
    for s in sims:
        s.beads()["v"][:, 1] = speed
    for n in (1, 2):
        got = _passes(sims[0], n)
        sims[1].couple_step(n)
        assert got == {"cycles": n, "second": n, "redone": 0}
        _same((sims[0],), (sims[1],), f"{nb} beads at {speed}, second pass against fused")
    for s in sims:
        s.check()


def test_full_lists_are_no_overflow(orc):
    """49 beads in one another's range: 48 partners each, as many as a list holds."""
    _torch()
    from paper_0711_2665_amd import lbmd
    cfg = scaled(C0, shape=(24, 24, 24), wall_axis=-1, wall_pos=0, pore_h=0, nb=49, rc=3.0, sigma=0.4, eps=0.01, r0=0.5,
                 kT=0.0, kappa=0.0)
    r = _cube(49, 0.5, 4, (11.13, 10.37, 11.29))
    o = orc.Oracle(cfg, r, np.zeros_like(r))
    s = lbmd.Simulation(cfg, r, None)
    o.couple_step(3)
    ob = o.beads()
    assert _passes(s, 3) == {"cycles": 3, "second": 3, "redone": 0}
    assert s.diagnostics()["nbr_max"] == 48
    s.check()
    b = _state(s)[1]
    for k in ("r", "v", "up", "J"):
        assert np.array_equal(b[k], ob[k]), k


def test_more_remote_partners_than_the_second_pass_holds():
    """Consecutive beads far apart on a face-centred lattice: the 42 partners of
    each bead of a segment are others, more than 1024 in all. One workgroup
    redoes the cycle, bit for bit the fused one."""
    _torch()
    from paper_0711_2665_amd import lbmd
    cell = np.array([(0, 0, 0), (0, 1, 1), (1, 0, 1), (1, 1, 0)], dtype=np.float64)
    grid = np.stack(np.meshgrid(*[np.arange(12)] * 3, indexing="ij"), -1).reshape(-1, 1, 3)
    pts = (2.0 * grid + cell).reshape(-1, 3) * (1.25 / np.sqrt(2.0)) + 5.0     # nearest neighbours 1.25 apart
    n = len(pts)
    r = pts[np.random.default_rng(3).permutation(n)]
    cfg = scaled(C0, shape=(32, 32, 32), wall_axis=-1, wall_pos=0, pore_h=0, nb=n, k_bond=1e-6, r0=5.0, kappa=0.0)
    sims = [lbmd.Simulation(cfg, r, None) for _ in range(2)]
    sims[1].md_fused(2)
    assert _passes(sims[0], 2) == {"cycles": 2, "second": 2, "redone": 2}
    sims[1].couple_step(2)
    assert sims[0].diagnostics()["nbr_max"] == 42
    _same((sims[0],), (sims[1],), "redo against fused")
    for s in sims:
        s.check()
