"""The Verlet list's two word formats (three slots or two a word), its distance
classes and the list lengths at which a lane's words take a second batch: the
neighbour sets against the oracle's predicate, and ten steps against the
oracle's fields; a checkpoint of the older list format."""
import numpy as np
import pytest

import oracle
import workloads as wl
from gpu_common import check_increments, field_errors, gpu_run, random_state, run_oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2108_08919_amd as P
    P.lib()
    yield


# h = 1.15 dx: about 38 entries; 1.3: 44; 1.5: 67 (more than 16 words of three,
# cells of 21 particles); tile 8 of the quintic holds two slots a word; sides
# with a ragged last tile and the smallest box
CASES = [(0, 1.15, 4, 1, 37), (0, 1.3, 8, 1, 37), (0, 1.5, 4, 1, 38), (0, 1.5, 8, 2, 33), (0, 1.5, 4, 4, 14),
         (1, 1.3, 8, 1, 37), (1, 1.3, 4, 1, 22), (1, 1.5, 8, 1, 31), (1, 1.3, 8, 4, 9)]


@pytest.mark.parametrize("kernel,h,tile,lpp,L", CASES)
def test_list_against_oracle(kernel, h, tile, lpp, L):
    import paper_2108_08919_amd as P
    p = wl.Params(L=float(L), zeta=0.03, h=h, kernel=kernel)
    s0 = random_state(L, 5, amp_u=2e-3)
    print("list", kernel, h, tile, lpp, L, flush=True)
    o, _ = run_oracle(p, s0, 10)
    g, sim = gpu_run(p, s0, 10, {P.NEM_OPT_TILE: tile, P.NEM_OPT_LPP: lpp})
    rp, col, cxy, oxy = sim.neighbor_list(0, 0, offsets=True)
    nc = int(np.floor(L / (oracle.kappa(kernel) * h + p.skin)))
    orp, ocol = oracle.neighbors_offsets(p, nc, cxy, oxy)
    rows = lambda a, b: [sorted(b[a[i]:a[i + 1]]) for i in range(a.size - 1)]
    assert rows(rp, col) == rows(orp, ocol)
    e = field_errors(g, o, s0, L, 10)
    for k in ("u", "Q", "rho", "pos"):
        assert e[k] <= 1e-5, (k, e[k])
    check_increments(e)
    sim.check()
    sim.close()


def test_older_checkpoint_rebuilds_its_list():
    """A version 1 checkpoint (the list in another format) is accepted: its list
    is rebuilt by the next step, so the run continues to rounding."""
    import paper_2108_08919_amd as P
    L = 24
    p = wl.Params(L=float(L), zeta=0.03)
    s0 = random_state(L, 2, amp_u=2e-3)
    _, a = gpu_run(p, s0, 4)
    buf = a.save_raw()
    a.step(6)
    ref = a.get_state(0)
    old = buf.copy()
    old[8:16] = np.frombuffer(np.int64(1).tobytes(), dtype=np.uint8)
    old[-8 * L * L - 4 * L * L - 4 * 48 * L * L:-12 * L * L] = 0xA5   # no list of this format
    b = P.Sim([p], [L * L])
    b.load_raw(old)
    b.step(6)
    b.check()
    g = b.get_state(0)
    e = field_errors(g, ref, s0, L)
    assert e["u"] < 1e-6 and e["Q"] < 1e-6 and e["rho"] < 1e-6 and e["pos_abs_max"] < 1e-9
    a.close()
    b.close()


# variants of the learned steps' own passes: tile, lanes, kernel, momentum form,
# elastic stress, corrector; ragged last tiles and cells of 7 to 21 particles
LEARN = [(4, 1, 37, {}), (8, 2, 33, {}), (4, 4, 22, dict(kernel=1)), (8, 1, 37, dict(kernel=1)),
         (4, 1, 38, dict(form=1, h=1.5)), (4, 2, 24, dict(elastic=1)), (4, 1, 31, dict(integrator=1))]


@pytest.mark.parametrize("tile,lpp,L,kw", LEARN)
def test_learned_steps_and_ordinary_ones_take_turns(tile, lpp, L, kw):
    """Learned steps with a network of zeros are steps of mult dt, so they agree
    with ordinary ones to rounding although they walk their list in another
    order; ordinary steps, a neighbour export and a checkpoint follow either."""
    import paper_2108_08919_amd as P
    from paper_2108_08919_amd import learned
    p = wl.Params(L=float(L), zeta=0.03, **kw)
    print("learned", tile, lpp, L, kw, flush=True)
    s0 = random_state(L, 4, amp_u=2e-3)
    z = learned.zero_network()
    opts = {P.NEM_OPT_TILE: tile, P.NEM_OPT_LPP: lpp}
    ref, r = gpu_run(p.replace(dt=4 * p.dt), s0, 6, opts)
    a = P.Sim([p], [L * L])
    for k, v in opts.items():
        a.set_option(k, v)
    a.set_state(0, s0)
    assert a.step_learned(z, 6, 4, 1.0)[0] == 0
    e = field_errors(a.get_state(0), ref, s0, L)
    assert e["u"] < 1e-5 and e["Q"] < 1e-6 and e["rho"] < 1e-7 and e["pos_abs_max"] < 1e-7
    # a checkpoint between learned steps continues bit for bit, in learned and in ordinary steps
    b = P.Sim([p], [L * L])
    b.load_raw(a.save_raw())
    for s in (a, b):
        s.step_learned(z, 3, 4, 1.0)
        s.step(2)
        s.step_learned(z, 1, 4, 1.0)
    # the export rebuilds the list in its own order
    rp, col, cxy, oxy = a.neighbor_list(0, 0, offsets=True)
    nc = int(np.floor(L / (oracle.kappa(p.kernel) * p.h + p.skin)))
    orp, ocol = oracle.neighbors_offsets(p, nc, cxy, oxy)
    rows = lambda x, y: [sorted(y[x[i]:x[i + 1]]) for i in range(x.size - 1)]
    assert rows(rp, col) == rows(orp, ocol)
    for s in (a, b):
        s.step(3)
        s.check()
    ga, gb = a.get_state(0), b.get_state(0)
    assert all(np.array_equal(ga[k], gb[k]) for k in ga)
    for s in (a, b, r, z):
        s.close()


# a tile shared by several workgroups: sides around the lines of the rule (275 and
# 299 at T = 4, 537 and 559 at T = 8 of Wendland C2), tiles of four
# rounds, and persistent grids of fewer workgroups than parts
@pytest.mark.parametrize("kernel,L,tile,persist,lpp", [
    (0, 275, 4, 0, 1), (0, 299, 4, 0, 1), (0, 97, 4, 0, 2), (0, 37, 4, 7, 4), (1, 537, 8, 0, 1), (1, 559, 8, 0, 1),
    (1, 64, 8, 5, 2), (0, 45, 8, 0, 1), (0, 14, 8, 3, 4)])
def test_shared_tiles_against_oracle(kernel, L, tile, persist, lpp):
    """The bounds of test_list_against_oracle."""
    import paper_2108_08919_amd as P
    p = wl.Params(L=float(L), zeta=0.03, kernel=kernel)
    s0 = random_state(L, 7, amp_u=2e-3)
    print("shared", kernel, L, tile, persist, lpp, flush=True)
    o, _ = run_oracle(p, s0, 2)
    g, sim = gpu_run(p, s0, 2, {P.NEM_OPT_TILE: tile, P.NEM_OPT_PERSIST: persist, P.NEM_OPT_LPP: lpp})
    e = field_errors(g, o, s0, L, 2)
    for k in ("u", "Q", "rho", "pos"):
        assert e[k] <= 1e-5, (k, e[k])
    sim.check()
    sim.close()


@pytest.mark.parametrize("tile,lpp,L,kw", [(4, 1, 37, {}), (8, 2, 33, dict(kernel=1))])
def test_captured_steps_replay_after_steps_of_the_other_kind(tile, lpp, L, kw):
    """Ordinary steps captured by the caller, replayed before and after learned
    ones: a replay runs the captured launches alone, so the device itself has to
    see that the list is in the other order. Bit for bit the same calls made
    eagerly, at each replay."""
    import torch
    import paper_2108_08919_amd as P
    from paper_2108_08919_amd import learned
    p = wl.Params(L=float(L), zeta=0.03, **kw)
    s0 = random_state(L, 4, amp_u=2e-3)
    print("captured", tile, lpp, L, kw, flush=True)
    st = torch.cuda.Stream()
    sims = []
    with torch.cuda.stream(st):
        for _ in range(2):
            s = P.Sim([p], [L * L], stream=st)
            s.set_option(P.NEM_OPT_TILE, tile)
            s.set_option(P.NEM_OPT_LPP, lpp)
            s.set_state(0, s0)
            s.step(4)
            s.check()
            sims.append(s)
        z = learned.zero_network()
    a, b = sims
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        a.step(2)   # two steps: the buffers' parity after a replay is the one before it
    for k in range(3):
        with torch.cuda.stream(st):
            g.replay()
        b.step(2)
        for s in (a, b):
            s.check()
        ga, gb = a.get_state(0), b.get_state(0)
        assert all(np.array_equal(ga[f], gb[f]) for f in ga), k
        for s in (a, b):
            s.step_learned(z, 2, 4, 1.0)
    for s in (a, b, z):
        s.close()


@pytest.mark.parametrize("kernel,tile,lpp", [(0, 4, 1), (0, 8, 2), (1, 8, 1), (1, 4, 1)])
def test_list_of_full_cells(kernel, tile, lpp):
    """Cells of more than the 32 particles that one mask word of the build holds: the
    neighbour sets against the oracle's predicate, and the list itself: no entry
    twice, outer entries first, then middle, then inner."""
    import paper_2108_08919_amd as P
    L = 40
    p = wl.Params(L=float(L), kernel=kernel)
    s0 = random_state(L, 3)
    kap = oracle.kappa(kernel)
    nc = int(np.floor(L / (kap * p.h + p.skin)))
    cs = L / nc
    rng = np.random.default_rng(5)
    ex = 24 if kernel == 0 else 28
    for cx, cy in ((2, 3), (7, 1), (0, nc - 1)):
        add = dict(x=(cx + 0.02 + 0.96 * rng.random(ex)) * cs, y=(cy + 0.02 + 0.96 * rng.random(ex)) * cs, rho=np.ones(ex))
        s0 = {f: np.concatenate([s0[f], add.get(f, np.zeros(ex))]) for f in s0}
    n = s0["x"].size
    print("full cells", kernel, tile, lpp, flush=True)
    sim = P.Sim([p], [n])
    sim.set_option(P.NEM_OPT_TILE, tile)
    sim.set_option(P.NEM_OPT_LPP, lpp)
    sim.set_state(0, s0)
    rp, col, cxy, oxy = sim.neighbor_list(0, 0, offsets=True)
    sim.check()
    assert np.bincount(cxy[:, 1] * nc + cxy[:, 0]).max() > 32
    orp, ocol = oracle.neighbors_offsets(p, nc, cxy, oxy)
    rows = lambda a, b: [sorted(b[a[i]:a[i + 1]]) for i in range(a.size - 1)]
    assert rows(rp, col) == rows(orp, ocol)
    # every entry of the list, by id
    vrp, vcol = sim.neighbor_list(0, 1)
    x = np.asarray(cxy, dtype=np.float64) * cs + oxy
    delta = 0.075 * p.h
    r = np.concatenate([np.linalg.norm((d := x[vcol[vrp[i]:vrp[i + 1]]] - x[i]) - L * np.round(d / L), axis=1)
                        for i in range(n)])
    assert all(np.unique(c).size == c.size for c in (vcol[vrp[i]:vrp[i + 1]] for i in range(n)))
    assert r.max() < kap * p.h + delta + 1e-5
    brute = sum(int((np.linalg.norm((d := x - x[i]) - L * np.round(d / L), axis=1) < kap * p.h + delta).sum()) - 1
                for i in range(n))
    assert abs(vcol.size - brute) <= 4   # pairs within rounding of the radius
    # class bounds of the counts (bits 8-15, 16-23) are met by every particle of a tile's group
    buf = sim.save_raw()
    cnt = buf[-12 * n:-8 * n].view(np.uint32)
    assert (cnt & 255).sum() == vcol.size
    assert np.all((cnt >> 8 & 255) <= (cnt >> 16 & 255)) and np.all((cnt >> 16 & 255) <= (cnt & 255))
    sim.close()


def test_renewing_the_list_costs_few_walks():
    """Pass A of a step that renews the list against one that walks it, on a box that
    fills the chip: 5.1 walks; 8.1 with a sweep over the candidates for each class."""
    import paper_2108_08919_amd as P
    L = 1024
    p = wl.Params(L=float(L))
    sim = P.Sim([p], [L * L])
    sim.set_state(0, random_state(L, 3))
    sim.step(3)
    sim.check()
    ms = []
    for renew in (0, 1):
        best = np.inf
        for _ in range(12):
            if renew:
                sim.set_option(P.NEM_OPT_TILE, 4)
            sim.set_option(P.NEM_OPT_TIMING, 1)
            sim.pass_times(reset=True)
            sim.step(1)
            sim.check()
            best = min(best, sim.pass_times(reset=True)[0][1])
            sim.set_option(P.NEM_OPT_TIMING, 0)
        ms.append(best)
    print("walk", ms[0], "renewed", ms[1], flush=True)
    assert ms[1] < 6.5 * ms[0]
    sim.close()


@pytest.mark.parametrize("graph,mult", [(2, 5), (3, 3), (4, 3)])
def test_fine_steps_of_learned_calls_replay_graphs(graph, mult):
    """Fallback and sample steps with NEM_OPT_GRAPH on: whole chunks and what is left
    over, an odd chunk (the parity flips), a chunk longer than the run; with
    ordinary steps, which replay graphs of their own, between them. Bit for bit the
    same calls without graphs, at each turn."""
    import paper_2108_08919_amd as P
    L = 37
    N = L * L
    p = wl.Params(L=float(L), zeta=0.03)
    s0 = random_state(L, 4, amp_u=2e-3)
    print("graphs", graph, mult, flush=True)
    net = P.Mlp()
    net.set_weights(np.random.default_rng(2).normal(0.0, 0.1, net.nparams).astype(np.float32))
    sims = []
    for g in (graph, 0):
        s = P.Sim([p], [N])
        s.set_option(P.NEM_OPT_GRAPH, g)
        s.set_state(0, s0)
        s.step(4)
        sims.append(s)
    for turn in range(3):
        seen = []
        for s in sims:
            fallbacks, _ = s.step_learned(net, 3, mult, 1e-6)   # every macro step is replayed as fine steps
            assert fallbacks == 3
            X, T = s.samples(mult)
            s.step(7)
            s.check()
            seen.append((s.get_state(0), X.cpu().numpy(), T.cpu().numpy()))
        (ga, xa, ta), (gb, xb, tb) = seen
        assert all(np.array_equal(ga[k], gb[k]) for k in ga), turn
        assert np.array_equal(xa, xb) and np.array_equal(ta, tb), turn
    for s in sims:
        s.close()
    net.close()


def test_fine_steps_of_learned_calls_gain_from_graphs():
    """512 fine steps of a sampling call on a box where launches count, with chunks of
    32 steps replayed and with eager launches: 0.95 of the time (1.00 when these
    steps took no part in the graphs)."""
    import time
    import paper_2108_08919_amd as P
    L = 32
    sim = P.Sim([wl.Params(L=float(L))], [L * L])
    sim.set_state(0, random_state(L, 3))
    sim.step(3)
    sim.check()
    best = {0: np.inf, 32: np.inf}
    for _ in range(4):
        for g in best:
            sim.set_option(P.NEM_OPT_GRAPH, g)
            sim.samples(512)   # with the capture
            for _ in range(3):
                t0 = time.perf_counter()
                sim.samples(512)
                best[g] = min(best[g], time.perf_counter() - t0)
    print("eager", best[0], "graphs", best[32], flush=True)
    assert best[32] < 0.985 * best[0]
    sim.close()
