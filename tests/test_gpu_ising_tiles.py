"""Tiled sweeps of a lattice in memory (two sweeps or more without strips)
against the same sweeps one at a time, which run per pass, and the oracle:
lattices of about one tile, rows and columns left over at the edge, margins
wrapped at the lattice's edge, uneven blocks, streams that do not stand at one
position, and replayed graphs."""
import numpy as np
import pytest
import torch

import hipgraph

pytestmark = pytest.mark.gpu

KINDS = ["lcg32", "lcg64", "mwc", "lcg32_sub", "lcg64_sub", "xorwow", "philox4x32_10", "philox4x32_7", "xs1024w"]


def _lattice(rx, L, kind):
    lat = rx.ising_create(L, kind, 5)
    rx.ising_set_plan(lat, 0)
    return lat


def _sweep(rx, lat, beta, n, hits, tr):
    if hits == 1:
        rx.ising_sweep(lat, beta, n, tr)
    else:
        rx.ising_sweep_hits(lat, beta, n, hits, tr)


def _same(rx, a, b):
    assert rx.ising_info(a)["strips"] == 0 and rx.ising_status(a) == 0
    assert np.array_equal(rx.ising_get_spins(a), rx.ising_get_spins(b))
    assert np.array_equal(rx.rng_get_state(rx.ising_rng(a)), rx.rng_get_state(rx.ising_rng(b)))


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("hits", [1, 3])
@pytest.mark.parametrize("size", [0, 1, 2, 3])
def test_tiles_equal_single_sweeps(rngx, kind, hits, size):
    L = ([1024, 1152, 1280, 2176] if kind == "xs1024w" else [256, 272, 480, 752])[size]
    a, b = _lattice(rngx, L, kind), _lattice(rngx, L, kind)
    for n, skip, beta in ((2, 0, 0.44), (9, 0, 0.3), (3, 1, 0.44), (17, 2, 1e9), (5, 1, 0.0)):
        print(f"case tiles {kind} L={L} hits={hits} sweeps={n} skip={skip} beta={beta}", flush=True)
        for lat in (a, b):
            rngx.rng_skip(rngx.ising_rng(lat), skip)
        ta = torch.full((n,), 7, dtype=torch.int32, device="cuda")
        tb = torch.zeros_like(ta)
        _sweep(rngx, a, beta, n, hits, ta)
        for i in range(n):
            _sweep(rngx, b, beta, 1, hits, tb[i:i + 1])
        assert torch.equal(ta, tb)
        _same(rngx, a, b)
    _sweep(rngx, a, 0.4, 4, hits, None)  # no trace
    for i in range(4):
        _sweep(rngx, b, 0.4, 1, hits, None)
    _same(rngx, a, b)


@pytest.mark.parametrize("kind", ["mwc", "xs1024w", "philox4x32_10", "xorwow"])
def test_tiles_oracle(rngx, orc, kind):
    L = 1152 if kind == "xs1024w" else 336
    lat = _lattice(rngx, L, kind)
    sp, st = orc.ising_create(L, kind, 5)
    for n, hits in ((5, 1), (2, 2)):
        print(f"case tiles oracle {kind} L={L} hits={hits} sweeps={n}", flush=True)
        tr = torch.zeros(n, dtype=torch.int32, device="cuda")
        _sweep(rngx, lat, 0.43, n, hits, tr)
        want = orc.ising_sweeps(L, kind, 0.43, st, sp, n, **({} if hits == 1 else {"hits": hits}))
        assert np.array_equal(tr.cpu().numpy(), want)
        assert np.array_equal(rngx.ising_get_spins(lat).ravel(), sp)
        assert np.array_equal(rngx.rng_get_state(rngx.ising_rng(lat)), st)


@pytest.mark.parametrize("kind", ["philox4x32_10", "xs1024w"])
def test_tiles_streams_apart(rngx, kind):
    """Streams at different positions: the tile cannot use one position for all."""
    L = 1024 if kind == "xs1024w" else 272
    a, b = _lattice(rngx, L, kind), _lattice(rngx, L, kind)
    S = L * L // 4
    state = rngx.rng_get_state(rngx.ising_rng(a)).copy()
    words = state[:state.nbytes // 8 * 8].view(np.uint64)
    if kind == "xs1024w":
        words[S // 2:S // 2 + S // 32] += np.arange(S // 32, dtype=np.uint64) % 7  # steps per instance
    else:
        words[S:2 * S] += np.arange(S, dtype=np.uint64) % 7
    for lat in (a, b):
        rngx.rng_set_state(rngx.ising_rng(lat), state)
    for hits in (1, 2):
        print(f"case tiles apart {kind} L={L} hits={hits}", flush=True)
        ta = torch.zeros(6, dtype=torch.int32, device="cuda")
        tb = torch.zeros_like(ta)
        _sweep(rngx, a, 0.4, 6, hits, ta)
        for i in range(6):
            _sweep(rngx, b, 0.4, 1, hits, tb[i:i + 1])
        assert torch.equal(ta, tb)
        _same(rngx, a, b)


@pytest.mark.parametrize("kind", ["mwc", "xs1024w"])
def test_tiles_in_a_graph(rngx, kind):
    L = 1024 if kind == "xs1024w" else 272
    a, b = _lattice(rngx, L, kind), _lattice(rngx, L, kind)
    ta = torch.zeros(5, dtype=torch.int32, device="cuda")
    tb = torch.zeros_like(ta)
    _sweep(rngx, a, 0.4, 5, 1, ta)
    _sweep(rngx, b, 0.4, 5, 1, tb)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        rngx.ising_sweep(a, 0.4, 5, ta)
    for replay in range(3):
        print(f"case tiles graph {kind} replay={replay}", flush=True)
        g.replay()
        torch.cuda.synchronize()
        for i in range(5):
            _sweep(rngx, b, 0.4, 1, 1, tb[i:i + 1])
        assert torch.equal(ta, tb)
        _same(rngx, a, b)


@pytest.mark.parametrize("kind", ["mwc", "xs1024w"])
def test_graph_of_tiles_outlives_its_plan(rngx, orc, kind):
    """A graph captured from tiled sweeps goes on giving the oracle's lattice
    after the lattice was moved to strips and after it was tuned, and writes to
    nothing but the lattice's own memory."""
    L = 1024 if kind == "xs1024w" else 512
    lat = _lattice(rngx, L, kind)
    sp, st = orc.ising_create(L, kind, 5)
    tr = torch.zeros(4, dtype=torch.int32, device="cuda")
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        rngx.ising_sweep(lat, 0.4, 4, tr)

    def check(n, got):
        want = orc.ising_sweeps(L, kind, 0.4, st, sp, n)
        assert np.array_equal(got.cpu().numpy(), want)
        assert np.array_equal(rngx.ising_get_spins(lat).ravel(), sp)
        assert np.array_equal(rngx.rng_get_state(rngx.ising_rng(lat)), st)

    plans = [p for p in rngx.ising_plans(lat) if p]
    for step in ("memory", "strips", "tuned"):
        print(f"case tiles graph after {step} {kind}", flush=True)
        if step == "strips":
            rngx.ising_set_plan(lat, plans[0])
        elif step == "tuned":
            rngx.ising_autotune(lat, 0.4, 2, reps=1)
        torch.cuda.empty_cache()
        other = [torch.full((L * L * b // 4,), 7, dtype=torch.int32, device="cuda") for b in (1, 1, 2, 2)]
        t2 = torch.zeros(3, dtype=torch.int32, device="cuda")
        rngx.ising_sweep(lat, 0.4, 3, t2)
        check(3, t2)
        for _ in range(2):
            g.replay()
            torch.cuda.synchronize()
            check(4, tr)
        assert all(bool((t == 7).all()) for t in other)


@pytest.mark.parametrize("kind", ["lcg32", "xorwow", "philox4x32_7"])
@pytest.mark.parametrize("n", [3, 5])
def test_every_tile_block_sweeps(rngx, orc, kind, n):
    """An odd number of sweeps with many hits, which would take one sweep a
    block: no block without a sweep is launched, and the lattice is the
    oracle's."""
    L, hits = 272, 100
    lat = _lattice(rngx, L, kind)
    sp, st = orc.ising_create(L, kind, 5)
    print(f"case tile blocks {kind} n={n}", flush=True)
    # one launch clears the energies
    tr = torch.zeros(n, dtype=torch.int32, device="cuda")
    launches = hipgraph.kernel_launches(lambda s: rngx.ising_sweep_hits(lat, 0.42, n, hits, tr, stream=s))
    assert len(launches) <= 1 + n, launches
    rngx.ising_sweep_hits(lat, 0.42, n, hits, tr)
    assert np.array_equal(tr.cpu().numpy(), orc.ising_sweeps(L, kind, 0.42, st, sp, n, hits=hits))
    assert np.array_equal(rngx.ising_get_spins(lat).ravel(), sp)
    assert np.array_equal(rngx.rng_get_state(rngx.ising_rng(lat)), st)
