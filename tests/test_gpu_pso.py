"""GPU parity of the PSO generation against the oracle.

Both sides start from the same seed (the initial population is drawn by the
method itself, so it must match bit for bit), then run generation by
generation.  Positions and velocities are compared bit for bit, personal-best
fitness within the fitness tolerance, and the global-best index exactly
(a tolerance tie would be reported as such).
"""
import ctypes
import math
import os

import numpy as np
import pytest
import torch

from parity import assert_fitness, index_ok

pytestmark = pytest.mark.gpu


def pair(evox, ref, fn, N, D, seed, lb, ub, **kw):
    g = evox.Swarm(evox.make_params(evox.PSO, fn, N, D, lb, ub, seed=seed, **kw))
    r = ref.PSO(ref.make_params(fn, N, D, lb, ub, seed=seed, **kw))
    return g, r


def host(t, D):
    return t[..., :D].cpu().numpy()


def compare_state(g, r, fn, what):
    D = r.P.D
    x, v, p = host(g.x, D), host(g.v, D), host(g.pbest, D)
    assert np.array_equal(x, r.x), f"{what}: x differs in rows {np.nonzero((x != r.x).any(1))[0][:8]}"
    assert np.array_equal(v, r.v), f"{what}: v differs"
    assert np.array_equal(p, r.p), f"{what}: pbest differs"
    pf = g.pfit.cpu().numpy()
    assert_fitness(fn, r.p, pf, r.pf, f"{what}: pfit")
    gf, gi, gx = g.best(with_x=True)
    assert index_ok(fn, r.p, r.pf, gi, r.gi), f"{what}: gbest {gi} vs {r.gi}"
    assert gi == r.gi, f"{what}: gbest index {gi} vs {r.gi} (tolerance tie)"
    assert np.array_equal(gx, r.g), f"{what}: gbest row"
    assert_fitness(fn, r.p[[gi]], [gf], [r.gf], f"{what}: gf")


def test_init_is_bit_exact(evox_gpu, ref):
    g, r = pair(evox_gpu, ref, 1, 37, 13, 1, -32.768, 32.768, v_lo=-1.0, v_hi=1.0)
    torch.cuda.synchronize()
    assert np.array_equal(host(g.x, 13), r.x)
    assert np.array_equal(host(g.v, 13), r.v)
    assert np.array_equal(host(g.pbest, 13), r.p)
    assert np.all(np.isinf(g.pfit.cpu().numpy()))
    assert np.all(g.x[:, 13:].cpu().numpy() == 0)       # padding kept at zero
    f, i = g.best()
    assert np.isinf(f) and i == 0


# configs: the 100 x 10 Sphere workload, every function at ragged shapes, and
# the velocity clamp / position clamp options
CASES = [
    dict(fn=0, N=100, D=10, seed=0, lb=-32.0, ub=32.0, gens=100),
    dict(fn=1, N=64, D=37, seed=1, lb=-32.768, ub=32.768, v_lo=-1.0, v_hi=1.0, gens=30),
    dict(fn=2, N=50, D=100, seed=2, lb=-5.12, ub=5.12, vmax=2.048, gens=30),
    dict(fn=3, N=33, D=129, seed=3, lb=-600.0, ub=600.0, gens=30),
    dict(fn=4, N=20, D=1001, seed=4, lb=-2.0, ub=2.0, gens=20),
    dict(fn=5, N=17, D=5, seed=5, lb=-500.0, ub=500.0, clamp_x=1, gens=40),
    dict(fn=0, N=3, D=4100, seed=6, lb=-1.0, ub=1.0, gens=8),
    dict(fn=4, N=2, D=2050, seed=7, lb=-2.0, ub=2.0, gens=8),
]


@pytest.mark.parametrize("case", CASES, ids=[f"fn{c['fn']}-{c['N']}x{c['D']}" for c in CASES])
def test_generations_match_oracle(evox_gpu, ref, case):
    c = dict(case)
    gens = c.pop("gens")
    print(f"pso {c} gens={gens}", flush=True)
    g, r = pair(evox_gpu, ref, **c)
    for t in range(gens):
        g.step(1)
        r.step(1)
        compare_state(g, r, c["fn"], f"generation {t}")
    assert g.t == r.t == gens


def test_multi_generation_call_equals_single_steps(evox_gpu, ref):
    kw = dict(fn=2, N=40, D=64, seed=9, lb=-5.12, ub=5.12, vmax=2.048)
    a, r = pair(evox_gpu, ref, **kw)
    b = evox_gpu.Swarm(evox_gpu.make_params(evox_gpu.PSO, kw["fn"], kw["N"], kw["D"], kw["lb"],
                                             kw["ub"], seed=kw["seed"], vmax=kw["vmax"]))
    a.step(25)
    for n in (1, 4, 7, 13):
        b.step(n)
    r.step(25)
    for name in ("x", "v", "pbest", "pfit", "gbest"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name
    assert a.best() == b.best()
    compare_state(a, r, kw["fn"], "after 25")


def test_velocity_exposes_r1_and_r2(evox_gpu, ref):
    N, D, seed = 9, 23, 77
    for c1, c2 in ((1.0, 0.0), (0.0, 1.0)):
        g, r = pair(evox_gpu, ref, 0, N, D, seed, -1.0, 1.0, w=0.0, c1=c1, c2=c2)
        g.x[:, :D] = 0.0
        g.pbest[:, :D] = 1.0
        g.pfit.fill_(-np.inf)
        r.x[:] = 0.0
        r.p[:] = 1.0
        r.pf[:] = -np.inf
        g.step(1)
        r.step(1)
        v = host(g.v, D)
        assert np.array_equal(v, r.v)
        assert v.min() >= 0.0 and v.max() < 1.0 and len(np.unique(v)) > N * D // 2


def test_single_particle(evox_gpu, ref):
    g, r = pair(evox_gpu, ref, 2, 1, 30, 11, -5.12, 5.12)
    for t in range(10):
        g.step(1)
        r.step(1)
        compare_state(g, r, 2, f"generation {t}")


@pytest.mark.parametrize("D,ldx", [(1001, 1024), (10, 64), (37, 40), (1000, 1000)])
def test_padding_columns_stay_zero(evox_gpu, ref, D, ldx):
    N = 9
    g = evox_gpu.Swarm(evox_gpu.make_params(evox_gpu.PSO, 2, N, D, -5.12, 5.12, seed=4, ldx=ldx))
    r = ref.PSO(ref.make_params(2, N, D, -5.12, 5.12, seed=4))
    for _ in range(3):
        g.step(2)
        r.step(2)
        for name in ("x", "v", "pbest"):
            t = getattr(g, name).cpu().numpy()
            assert np.all(t[:, D:] == 0), name
        assert np.all(g.gbest[D:].cpu().numpy() == 0)
        compare_state(g, r, 2, f"D {D} ldx {ldx}")


COUNTER_CASES = [dict(fn=0, N=100, D=10, seed=0, lb=-32.0, ub=32.0, gens=100),
                 dict(fn=0, N=3000, D=10, seed=0, lb=-32.0, ub=32.0, gens=20),
                 dict(fn=2, N=257, D=100, seed=2, lb=-5.12, ub=5.12, vmax=2.048, gens=30),
                 dict(fn=1, N=64, D=1000, seed=1, lb=-32.768, ub=32.768, v_lo=-1.0, v_hi=1.0, gens=12)]


@pytest.mark.parametrize("case", COUNTER_CASES, ids=[f"fn{c['fn']}-{c['N']}x{c['D']}" for c in COUNTER_CASES])
def test_improved_row_counter_matches_oracle(evox_gpu, ref, case):
    """The generation kernels count the rows whose personal best improved
    (the pbest rows rewritten, part of the bytes the benchmark reports); over
    one call of `gens` generations the count equals the oracle's number of
    rows whose pfit fell, generation by generation."""
    c = dict(case)
    gens = c.pop("gens")
    g, r = pair(evox_gpu, ref, **c)
    expected = []
    for _ in range(gens):
        pf0 = r.pf.copy()
        r.step(1)
        expected.append(int((r.pf < pf0).sum()))
    g.profile(True)
    g.step(gens)
    ms, timed_gens, improved = g.profile_read()
    g.profile(False)
    compare_state(g, r, c["fn"], f"after {gens}")
    # generations performed by the timed launches: the fused ones (every
    # generation but the first evaluation and the last move), or the whole
    # call for a swarm small enough for the one-block kernel
    small = c["N"] * c["D"] <= 16384 and evox_gpu.row_layout(c["D"])[0] <= 64
    assert timed_gens == (gens if small else gens - 1)
    assert improved == sum(expected), (improved, sum(expected), expected[:5])


def test_small_and_large_swarm_paths_agree(evox_gpu, ref):
    """N D = 16384 runs in the one-block kernel, N D = 16388 in the multi-block
    generation kernels: both bit-exact against the oracle over 12 generations
    (the same row layout and reduction, so the same fitness bits)."""
    for N in (4096, 4097):
        g, r = pair(evox_gpu, ref, 2, N, 4, 21, -5.12, 5.12, vmax=2.048, v_lo=-0.5, v_hi=0.5)
        g.step(12)
        r.step(12)
        compare_state(g, r, 2, f"N = {N}")


# rows of one wave, of several waves, and of several chunk pairs per lane, with
# pitches that leave padding: the personal bests stay in x while a row improves
# and reach pbest when it stops or the call ends
LAG_CASES = [(2, 700, 65), (0, 300, 500), (1, 260, 1000), (4, 130, 2000), (3, 66, 4000), (2, 33, 8000), (0, 17, 16384),
             (5, 9, 32768)]


@pytest.mark.parametrize("fn,N,D", LAG_CASES)
def test_personal_bests_after_calls_of_several_generations(evox_gpu, ref, fn, N, D):
    lb, ub = {0: (-32.0, 32.0), 1: (-32.768, 32.768), 2: (-5.12, 5.12), 3: (-600.0, 600.0), 4: (-2.0, 2.0),
              5: (-500.0, 500.0)}[fn]
    print(f"pso lag fn={fn} N={N} D={D}", flush=True)
    g, r = pair(evox_gpu, ref, fn, N, D, 23, lb, ub, vmax=0.2 * (ub - lb))
    for n in (1, 2, 6):
        g.step(n)
        r.step(n)
        compare_state(g, r, fn, f"after a call of {n}")
        for name in ("x", "v", "pbest"):
            assert not getattr(g, name)[:, D:].any(), f"{name} padding"


# swarms that a call of at least four generations keeps on the chip: one block
# (1024 lanes) and its first size beyond, then 256 blocks with one, four and
# ten rows per lane group, each at its largest and first size beyond, for rows
# of 4, 16, 64, 128, 256 and 512 lanes
RESIDENT_CASES = [(0, 256, 13), (2, 257, 13), (4, 64, 101), (1, 65, 128), (4, 8, 1000), (4, 9, 1000), (5, 2, 4096),
                  (3, 65_536, 3), (5, 65_537, 3), (0, 131_073, 5), (2, 327_680, 2), (2, 327_681, 2),
                  (4, 16_385, 120), (1, 4_097, 512), (3, 2_049, 515), (4, 2_048, 1000), (0, 4_097, 1000),
                  (1, 10_240, 1000), (4, 1_300, 2_047), (4, 513, 2_100), (2, 1_025, 4_096)]


@pytest.mark.parametrize("fn,N,D", RESIDENT_CASES)
def test_resident_calls_match_oracle(evox_gpu, ref, fn, N, D):
    lb, ub = {0: (-32.0, 32.0), 1: (-32.768, 32.768), 2: (-5.12, 5.12), 3: (-600.0, 600.0), 4: (-2.0, 2.0),
              5: (-500.0, 500.0)}[fn]
    print(f"pso resident fn={fn} N={N} D={D}", flush=True)
    kw = dict(vmax=0.2 * (ub - lb), clamp_x=1) if N % 2 else {}
    g, r = pair(evox_gpu, ref, fn, N, D, 29, lb, ub, **kw)
    for n in (4, 1, 5):  # resident, grid-wide, resident
        g.step(n)
        r.step(n)
        compare_state(g, r, fn, f"after a call of {n}")
        for name in ("x", "v", "pbest"):
            assert not getattr(g, name)[:, D:].any(), f"{name} padding"


def test_resident_calls_on_two_streams(evox_gpu, ref):
    """Two swarms, each in 250 blocks that wait for each other, stepped on two
    streams without waiting in between, for more generations than a slot's tag
    counts."""
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    gs = [evox_gpu.Swarm(evox_gpu.make_params(evox_gpu.PSO, 2, 1999, 101, -5.12, 5.12, seed=s), stream=st)
          for s, st in enumerate(streams)]
    torch.cuda.synchronize()
    for _ in range(6):
        for g in gs:
            g.step(100)
    torch.cuda.synchronize()
    for s, g in enumerate(gs):
        one = evox_gpu.Swarm(evox_gpu.make_params(evox_gpu.PSO, 2, 1999, 101, -5.12, 5.12, seed=s))
        for _ in range(300):
            one.step(2)  # grid-wide
        for name in ("x", "v", "pbest", "pfit", "fit", "gbest"):
            assert torch.equal(getattr(g, name), getattr(one, name)), name
        assert g.best() == one.best()


def test_captured_calls_of_a_resident_size(evox_gpu, ref):
    """A call recorded into a graph, replayed between eager work, equals the
    same call made eagerly."""
    st = torch.cuda.Stream()
    mk = lambda: evox_gpu.Swarm(evox_gpu.make_params(evox_gpu.PSO, 1, 1500, 90, -32.0, 32.0, seed=5), stream=st)  # noqa: E731
    g, e = mk(), mk()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        g.step(6)
    for _ in range(3):
        with torch.cuda.stream(st):
            graph.replay()
            e.set_generation(0)
            e.step(6)
        torch.cuda.synchronize()
        for name in ("x", "v", "pbest", "pfit", "gbest"):
            assert torch.equal(getattr(g, name), getattr(e, name)), name


def test_resident_selection_with_nan_and_infinite_rows(evox_gpu, ref):
    for N, D in ((40, 12), (3000, 12)):
        g, r = pair(evox_gpu, ref, 0, N, D, 31, -1.0, 1.0)
        bad = np.full((N, D), np.nan, np.float32)
        bad[N // 2:] = np.inf
        good = N - 3
        bad[good] = 0.25
        g.x[:, :D] = torch.from_numpy(bad).cuda()
        g.v.zero_()
        r.x[:] = bad
        r.v[:] = 0.0
        g.step(5)
        r.step(5)
        assert g.best()[1] == r.gi == good
        assert np.array_equal(host(g.pbest, D), r.p)
        assert np.array_equal(host(g.x, D), r.x, equal_nan=True)


STATE = ("x", "v", "pbest", "pfit", "fit", "gbest")


# every shape of the resident kernel, with rows of part of a wave, of a wave and
# of several, and a function that looks at a neighbour across waves; the waits:
# none, about an exchange (a call is given up anywhere in it, or not at all) and
# the default
GIVE_UP_CASES = [(2, 1_000, 10), (4, 1_999, 101), (1, 700, 500), (4, 520, 1_000), (3, 65, 2_100), (4, 40, 4_096),
                 (5, 20_000, 13), (0, 4_500, 500), (4, 30_000, 70), (1, 2_100, 2_050)]


@pytest.mark.parametrize("fn,N,D", GIVE_UP_CASES)
def test_resident_calls_given_up_are_done_by_one_block(evox_gpu, fn, N, D):
    lb, ub = {0: (-32.0, 32.0), 1: (-32.768, 32.768), 2: (-5.12, 5.12), 3: (-600.0, 600.0), 4: (-2.0, 2.0),
              5: (-500.0, 500.0)}[fn]
    print(f"pso given up fn={fn} N={N} D={D}", flush=True)
    kw = dict(seed=37, v_lo=-1.0, v_hi=1.0, **(dict(vmax=0.2 * (ub - lb), clamp_x=1) if N % 2 else {}))
    g, one = (evox_gpu.Swarm(evox_gpu.make_params(evox_gpu.PSO, fn, N, D, lb, ub, **kw)) for _ in range(2))
    given_up = 0
    for wait, n in ((0.0, 4), (1e-8, 5), (1e-8, 7), (1e-6, 6), (2e-6, 9), (3e-6, 5), (0.0, 4), (-1.0, 4)):
        before = g.pso_wait(wait)
        g.step(n)
        for _ in range(n):
            one.step(1)  # grid-wide
        for name in STATE:
            assert torch.equal(getattr(g, name), getattr(one, name)), (name, wait, n)
        assert g.best() == one.best()
        after = g.pso_wait(-1.0)
        assert after - before in ((1,) if wait == 0.0 else (0, 1) if wait > 0.0 else (0,)), (wait, before, after)
        given_up += after - before
    assert given_up >= 2


def test_wait_argument(evox_gpu):
    g = evox_gpu.Swarm(evox_gpu.make_params(evox_gpu.PSO, 0, 20, 5, -1.0, 1.0))
    assert g.pso_wait(0.0) == 0 and g.pso_wait(-1.0) == 0
    for bad in (math.nan, 1e7):
        with pytest.raises(evox_gpu.EvoxError):
            g.pso_wait(bad)
    with pytest.raises(evox_gpu.EvoxError):
        evox_gpu.Swarm(evox_gpu.make_params(evox_gpu.CSO, 0, 20, 5, -1.0, 1.0)).pso_wait(0.0)


def test_resident_call_beside_a_long_kernel(evox_gpu):
    """A one-block call of many generations holds a CU while calls that need
    every CU are made on another stream: they give the same swarm as without it."""
    busy, st = torch.cuda.Stream(), torch.cuda.Stream()
    mk = lambda N, D, s: evox_gpu.Swarm(evox_gpu.make_params(evox_gpu.PSO, 1, N, D, -32.0, 32.0, seed=11), stream=s)  # noqa: E731
    long, g = mk(100, 10, busy), mk(10_000, 1_000, st)
    one = mk(10_000, 1_000, st)
    torch.cuda.synchronize()
    long.step(400_000)  # under a second in one block
    for _ in range(3):
        g.step(4)
    for _ in range(12):
        one.step(1)
    torch.cuda.synchronize()
    for name in STATE:
        assert torch.equal(getattr(g, name), getattr(one, name)), name
    assert g.best() == one.best()
    print("calls done by one block:", g.pso_wait(-1.0), flush=True)
    assert long.t == 400_000 and math.isfinite(long.best()[0])


# one block with two and three rows per lane group: from just above what it holds
# with one (1024 lanes) to its most, for rows of 4 .. 64 lanes, and first sizes
# beyond
FEW_ROW_CASES = [(2, 257, 10), (4, 512, 16), (0, 513, 16), (1, 768, 16), (5, 769, 16), (4, 129, 60), (1, 256, 64),
                 (2, 383, 57), (3, 65, 101), (5, 128, 128), (4, 192, 99), (4, 33, 250), (2, 64, 256), (0, 96, 200),
                 (4, 17, 390), (1, 32, 512), (4, 33, 490), (3, 38, 505), (4, 40, 500), (0, 600, 3)]


def small_pair(evox, ref, fn, N, D, stream=None):
    lb, ub = {0: (-32.0, 32.0), 1: (-32.768, 32.768), 2: (-5.12, 5.12), 3: (-600.0, 600.0), 4: (-2.0, 2.0),
              5: (-500.0, 500.0)}[fn]
    kw = dict(v_lo=-1.0, v_hi=1.0, **(dict(vmax=0.2 * (ub - lb), clamp_x=1) if N % 2 else {}))
    return (evox.Swarm(evox.make_params(evox.PSO, fn, N, D, lb, ub, seed=41, **kw), stream=stream),
            ref.PSO(ref.make_params(fn, N, D, lb, ub, seed=41, **kw)))


@pytest.mark.parametrize("fn,N,D", FEW_ROW_CASES)
def test_short_calls_of_small_swarms(evox_gpu, ref, fn, N, D):
    print(f"pso short fn={fn} N={N} D={D}", flush=True)
    g, r = small_pair(evox_gpu, ref, fn, N, D)
    for n in (1, 4, 30, 2):
        g.step(n)
        r.step(n)
        compare_state(g, r, fn, f"after a call of {n}")
        for name in ("x", "v", "pbest"):
            assert not getattr(g, name)[:, D:].any(), f"{name} padding"


def graph_nodes(graph):
    hip = ctypes.CDLL(os.path.join(os.path.dirname(torch.__file__), "lib", "libamdhip64.so"))
    n = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


# the nodes of a graph of one generation and of six
@pytest.mark.parametrize("N,D,one,six", [(100, 10, 1, 1), (300, 10, 1, 1), (768, 16, 1, 1), (769, 16, 3, 13),
                                         (128, 128, 1, 1), (38, 490, 1, 1), (40, 490, 3, 13)])
def test_captured_calls_of_small_swarms(evox_gpu, ref, N, D, one, six):
    print(f"pso captured N={N} D={D}", flush=True)
    for n, nodes in ((1, one), (6, six)):
        st = torch.cuda.Stream()
        g, r = small_pair(evox_gpu, ref, 2, N, D, stream=st)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(graph, stream=st):
            g.step(n)
        assert graph_nodes(graph) == nodes
        for _ in range(3):
            with torch.cuda.stream(st):
                graph.replay()
            r.t = 0
            r.step(n)
            torch.cuda.synchronize()
            for name, want in (("x", r.x), ("v", r.v), ("pbest", r.p)):
                assert np.array_equal(host(getattr(g, name), D), want), name


# one generation a call: in one block above and below 16384 elements, and grid-wide
@pytest.mark.parametrize("N,D,gens", [(300, 10, 3), (300, 64, 3), (2_000, 100, 0)])
def test_profile_counts_the_generations_of_short_calls(evox_gpu, N, D, gens):
    g = evox_gpu.Swarm(evox_gpu.make_params(evox_gpu.PSO, 2, N, D, -5.12, 5.12, seed=1))
    g.step(1)
    g.profile(True)
    for _ in range(3):
        g.step(1)
    ms, launches, improved = g.profile_read()
    g.profile(False)
    assert launches == gens and (ms > 0) == (gens > 0) and 0 < improved <= 3 * N
