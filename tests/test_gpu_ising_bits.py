"""Strips whose spins are held as bits, at the shapes where their layout can
go wrong: rows that leave threads idle, strips whose rows do not fill the last
slot, one row per thread, several rows side by side, and thresholds that
accept every draw.  Bit-exact against the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

KINDS = ["lcg32", "lcg64", "mwc", "xorwow", "philox4x32_10", "xs1024w", "philox4x32_7", "lcg32_sub", "lcg64_sub",
         "mwc_diff"]


def _parity(rx, orc, L, kind, beta, calls, hits=1, plan=None, skip=0, trace=True):
    lat = rx.ising_create(L, kind, 3)
    if plan is not None:
        rx.ising_set_plan(lat, plan)
    sp, st = orc.ising_create(L, kind, 3)
    if skip:  # the streams no longer start a call at a block's first word
        rx.rng_skip(rx.ising_rng(lat), skip)
        orc.jump(kind, L * L // 4, st, skip)
    for n in calls:
        print(f"case bits {kind} L={L} plan={plan} hits={hits} beta={beta} sweeps={n}", flush=True)
        tr = torch.zeros(n, dtype=torch.int32, device="cuda") if trace else None
        if hits == 1:
            rx.ising_sweep(lat, beta, n, tr)
            want = orc.ising_sweeps(L, kind, beta, st, sp, n)
        else:
            rx.ising_sweep_hits(lat, beta, n, hits, tr)
            want = orc.ising_sweeps(L, kind, beta, st, sp, n, hits=hits)
        assert rx.ising_status(lat) == 0
        if trace:
            assert np.array_equal(tr.cpu().numpy(), want)
        assert np.array_equal(rx.ising_get_spins(lat).ravel(), sp)
        assert np.array_equal(rx.rng_get_state(rx.ising_rng(lat)), st)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("L", [112, 240, 272, 400, 592, 976])
def test_ragged_rows(rngx, orc, kind, L):
    """Columns that do not fill whole waves, single- and multi-strip."""
    _parity(rngx, orc, L, kind, 0.44, (3, 2))


@pytest.mark.parametrize("kind", ["lcg32", "philox4x32_10", "xs1024w", "xorwow"])
@pytest.mark.parametrize("L", [192, 480, 720])
def test_every_plan(rngx, orc, kind, L):
    """Strips of every height that fits, the rows of some not a multiple of
    the rows side by side."""
    for plan in rngx.ising_plans(rngx.ising_create(L, kind, 3)):
        _parity(rngx, orc, L, kind, 0.42, (2, 1), plan=plan)


@pytest.mark.parametrize("kind", ["lcg64", "philox4x32_7", "xs1024w", "mwc_diff"])
@pytest.mark.parametrize("L", [48, 512])
@pytest.mark.parametrize("beta", [0.0, 0.02, 1e9])
def test_extreme_thresholds(rngx, orc, kind, L, beta):
    _parity(rngx, orc, L, kind, beta, (3,))
    _parity(rngx, orc, L, kind, beta, (2,), hits=3)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("hits", [2, 3, 7])
def test_multi_hit(rngx, orc, kind, hits):
    for L in (80, 400):
        _parity(rngx, orc, L, kind, 0.4, (2, 1), hits=hits)


@pytest.mark.parametrize("kind", ["philox4x32_10", "philox4x32_7"])
@pytest.mark.parametrize("skip", [1, 2, 3])
@pytest.mark.parametrize("hits", [1, 3])
def test_philox_inside_a_block(rngx, orc, kind, skip, hits):
    for L in (64, 416):
        _parity(rngx, orc, L, kind, 0.4, (2, 1), hits=hits, skip=skip)


@pytest.mark.parametrize("kind", ["philox4x32_10", "xs1024w"])
@pytest.mark.parametrize("hits", [1, 4])
def test_streams_at_different_positions(rngx, orc, kind, hits):
    """The general form, where a strip's streams share no position."""
    for L in (96, 512):
        lat = rngx.ising_create(L, kind, 3)
        sp, st = orc.ising_create(L, kind, 3)
        S = L * L // 4
        n = S // 32 if kind == "xs1024w" else S
        at = 4 * S if kind == "xs1024w" else 8 * S
        st = np.array(st, dtype=np.uint8)
        pos = np.random.default_rng(1).integers(0, 1000, n).astype(np.uint64)
        st[at:at + 8 * n] = pos.view(np.uint8)
        rngx.rng_set_state(rngx.ising_rng(lat), st)
        print(f"case bits positions {kind} L={L} hits={hits}", flush=True)
        tr = torch.zeros(3, dtype=torch.int32, device="cuda")
        rngx.ising_sweep_hits(lat, 0.4, 3, hits, tr)
        want = orc.ising_sweeps(L, kind, 0.4, st, sp, 3, hits=hits)
        assert np.array_equal(tr.cpu().numpy(), want)
        assert np.array_equal(rngx.ising_get_spins(lat).ravel(), sp)
        assert np.array_equal(rngx.rng_get_state(rngx.ising_rng(lat)), st)


@pytest.mark.parametrize("kind", ["lcg32", "xs1024w"])
def test_without_trace(rngx, orc, kind):
    for L in (64, 512):
        _parity(rngx, orc, L, kind, 0.4, (3, 1), trace=False)


@pytest.mark.parametrize("kind", KINDS)
def test_batch_sizes(rngx, orc, kind):
    """A batch whose replicas all hold bits: one workgroup (some with idle
    waves) to gangs with a shorter last strip, under several launch shapes, run
    after run like the oracle's lattices."""
    Ls = [16, 48, 64, 112, 256, 272, 416, 784]
    betas = [0.3, 0.41, 0.44, 0.5, 0.38, 0.45, 0.42, 0.6]
    sweeps = [5, 2, 3, 2, 2, 3, 2, 2]
    lats = [rngx.ising_create(L, kind, 70 + i) for i, L in enumerate(Ls)]
    refs = [orc.ising_create(L, kind, 70 + i) for i, L in enumerate(Ls)]
    traces = [torch.full((n,), 7, dtype=torch.int32, device="cuda") for n in sweeps]
    batch = rngx.ising_batch_create(lats, betas, sweeps, traces)
    for shape in (0, 0, 2, 4):
        print(f"case bits batch {kind} shape={shape}", flush=True)
        rngx.ising_batch_set_shape(batch, shape)
        rngx.ising_batch_run(batch)
        assert rngx.ising_batch_status(batch) == 0
        for i, (sp, st) in enumerate(refs):
            want = orc.ising_sweeps(Ls[i], kind, betas[i], st, sp, sweeps[i])
            assert np.array_equal(traces[i].cpu().numpy(), want), (shape, Ls[i])
            assert np.array_equal(rngx.ising_get_spins(lats[i]).ravel(), sp), (shape, Ls[i])
            assert np.array_equal(rngx.rng_get_state(rngx.ising_rng(lats[i])), st), (shape, Ls[i])


@pytest.mark.parametrize("kind", KINDS)
def test_batch_replicas_without_sweeps(rngx, orc, kind):
    """Replicas of zero sweeps among others, lone workgroups and gangs, their
    streams at one position and apart: such a replica's spins and streams stay
    as they are."""
    Ls = [48, 64, 256, 784, 784, 112, 64]
    sweeps = [0, 3, 0, 0, 2, 2, 0]
    lats = [rngx.ising_create(L, kind, 90 + i) for i, L in enumerate(Ls)]
    refs = [orc.ising_create(L, kind, 90 + i) for i, L in enumerate(Ls)]
    if kind.startswith("philox") or kind == "xs1024w":  # the last replica's streams at positions of their own
        S = Ls[-1] ** 2 // 4
        st = np.array(refs[-1][1], dtype=np.uint8)
        at, n = (4 * S, S // 32) if kind == "xs1024w" else (8 * S, S)
        st[at:at + 8 * n] = np.random.default_rng(2).integers(0, 1000, n).astype(np.uint64).view(np.uint8)
        rngx.rng_set_state(rngx.ising_rng(lats[-1]), st)
        refs[-1] = (refs[-1][0], st)
    traces = [torch.full((max(n, 1),), 7, dtype=torch.int32, device="cuda") for n in sweeps]
    batch = rngx.ising_batch_create(lats, [0.42] * len(Ls), sweeps, traces)
    for shape in (0, 4):
        print(f"case bits batch without sweeps {kind} shape={shape}", flush=True)
        rngx.ising_batch_set_shape(batch, shape)
        rngx.ising_batch_run(batch)
        assert rngx.ising_batch_status(batch) == 0
        for i, (sp, st) in enumerate(refs):
            if sweeps[i]:
                want = orc.ising_sweeps(Ls[i], kind, 0.42, st, sp, sweeps[i])
                assert np.array_equal(traces[i].cpu().numpy(), want), (shape, i)
            else:
                assert int(traces[i][0]) == 7, (shape, i)
            assert np.array_equal(rngx.ising_get_spins(lats[i]).ravel(), sp), (shape, i, Ls[i])
            assert np.array_equal(rngx.rng_get_state(rngx.ising_rng(lats[i])), st), (shape, i, Ls[i])


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("L", [48, 112, 128, 160, 640, 720, 1040])
def test_multi_hit_shapes(rngx, orc, kind, L):
    """Multi-hit sweeps lie on more threads than single-hit ones: sides where
    the two shapes differ, called in turn on one lattice, whose strips exchange
    rows under both."""
    lat = rngx.ising_create(L, kind, 3)
    sp, st = orc.ising_create(L, kind, 3)
    for n, hits in ((2, 5), (1, 1), (1, 2), (2, 1), (1, 9)):
        print(f"case bits shapes {kind} L={L} hits={hits} sweeps={n}", flush=True)
        tr = torch.zeros(n, dtype=torch.int32, device="cuda")
        rngx.ising_sweep_hits(lat, 0.43, n, hits, tr)
        want = orc.ising_sweeps(L, kind, 0.43, st, sp, n, hits=hits)
        assert rngx.ising_status(lat) == 0
        assert np.array_equal(tr.cpu().numpy(), want)
        assert np.array_equal(rngx.ising_get_spins(lat).ravel(), sp)
        assert np.array_equal(rngx.rng_get_state(rngx.ising_rng(lat)), st)
