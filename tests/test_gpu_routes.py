"""GPU tests of the kernel variants that the library chooses by size: each
variant against the general path on the same inputs, bit for bit."""
import os

import numpy as np
import pytest

import sbqa_instances as inst

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sb():
    import paper_2604_01050_amd as sb
    return sb


def _log(msg):
    print(msg, flush=True)


def _sparse(N, d, seed):
    """Random graph of degree at most d (at least one spin has degree d)."""
    rng = np.random.default_rng(seed)
    E = np.concatenate([np.sort(np.stack([p, np.roll(p, 1)], 1), 1) for p in (rng.permutation(N) for _ in range(d // 2))])
    E = np.unique(E, axis=0)
    return inst.edges_to_csr(N, E, rng.standard_normal(len(E))), rng.standard_normal(N) * 0.1


# rows of 1 to 4 per thread and their edges, 2, 4 and 8 columns per workgroup
# (C up to 128, up to 512, above), rings of one workgroup and of several
@pytest.mark.parametrize("N,d,R,runs,fmode", [
    (1, 2, 8, 1, 0), (512, 4, 8, 3, 0), (513, 6, 16, 8, 1), (1025, 12, 24, 5, 0), (2048, 16, 8, 16, 0),
    (2049, 4, 16, 8, 0), (3073, 6, 32, 4, 0), (4096, 4, 16, 8, 1),
    (300, 16, 16, 32, 0), (1024, 8, 16, 20, 0), (2048, 16, 8, 32, 0), (3000, 6, 32, 8, 1), (4095, 6, 16, 16, 0),
    (700, 6, 16, 40, 0), (2000, 12, 8, 130, 0)])
def test_resident_columns_per_workgroup(sb, N, d, R, runs, fmode):
    """The resident sparse loop at every split of the columns equals the
    one-launch-per-step kernel over launches of 1, 2 and 20 steps with readouts
    between them."""
    csr, h = _sparse(N, d, 7) if N > 1 else ((np.zeros(2, np.int32), np.zeros(0, np.int32), np.zeros(0)), np.ones(1))
    out = []
    for kern in (sb.LOOP_STREAM, sb.LOOP_RESIDENT):
        _log("columns per workgroup N=%d d=%d R=%d runs=%d kernel %d" % (N, d, R, runs, kern))
        ctx = sb.sbqa_create(csr=csr, h=h, R=R, runs=runs, steps=40, fmode=fmode, loop_kernel=kern, seed=9)
        got = []
        for n in (1, 2, 20):
            sb.sbqa_step(ctx, n)
            got += [*sb.sbqa_best(ctx), *sb.sbqa_get_state(ctx)]
        sb.sbqa_set_state(ctx, got[-2], got[-1])
        sb.sbqa_step(ctx, 17)
        out.append(got + [*sb.sbqa_get_state(ctx), *sb.sbqa_best(ctx)])
    for a, b in zip(*out):
        assert np.array_equal(a, b)


# dense +-1 instances that AUTO steps in the many-step loop: every launch shape
# (row blocks per wave, workgroups per group, one or two column blocks, whole
# and part rings of 16 and 32, several runs in a group), edges of its tiles
@pytest.mark.parametrize("N,R,runs,prec,fmode,ee", [
    (129, 16, 8, "AUTO", 0, 0), (256, 4, 3, "FP8", 1, 7), (257, 16, 2, "FP32", 0, 0), (400, 1, 40, "AUTO", 0, 0),
    (511, 10, 8, "AUTO", 1, 9), (512, 32, 4, "FP8", 0, 0), (513, 8, 9, "INT8", 0, 0), (601, 16, 8, "AUTO", 0, 11),
    (640, 20, 3, "FP32", 1, 0), (1000, 32, 4, "AUTO", 0, 0), (1024, 5, 7, "AUTO", 0, 0), (1025, 16, 8, "FP8", 0, 0),
    (1300, 24, 2, "AUTO", 1, 0), (2047, 16, 8, "AUTO", 0, 0), (2048, 16, 16, "FP8", 0, 0),
    (300, 16, 200, "AUTO", 0, 0), (480, 16, 300, "AUTO", 0, 0), (1000, 16, 150, "FP8", 0, 0)])
def test_dense_many_step_loop(sb, N, R, runs, prec, fmode, ee):
    """The many-step loop equals one launch per step bit for bit: states,
    fields, energies, best spins and steps, over launches of 1, 2 and 22 steps
    and after a state overwrite."""
    J, h = inst.sk_pm1(N, 11), np.round(inst.gaussian_fields(N, 1.0, 12))
    out, size = [], []
    for kern in (sb.LOOP_STREAM, sb.LOOP_AUTO):
        _log("many-step loop N=%d R=%d runs=%d %s kernel %d" % (N, R, runs, prec, kern))
        ctx = sb.sbqa_create(J=J, h=h, R=R, runs=runs, steps=50, fmode=fmode, loop_kernel=kern, seed=3, energy_every=ee,
                             precision=getattr(sb, "PREC_" + prec))
        size.append(sb.sbqa_info(ctx)["device_bytes"])
        got = []
        for n in (1, 2, 22):
            sb.sbqa_step(ctx, n)
            got += [*sb.sbqa_best(ctx), *sb.sbqa_get_state(ctx)]
        got.append(sb.sbqa_fields(ctx))
        sb.sbqa_set_state(ctx, 0.5 * got[-3], got[-2])
        sb.sbqa_step(ctx, 25)
        out.append(got + [*sb.sbqa_get_state(ctx), *sb.sbqa_best(ctx), sb.sbqa_best_step(ctx)])
    assert size[1] > size[0], "AUTO did not take the many-step loop"
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("kind,N,R,runs,K", [("dense", 601, 16, 8, 1), ("dense", 601, 16, 8, 9), ("dense", 200, 8, 2, 4),
                                             ("sparse", 1000, 16, 8, 1), ("sparse", 3000, 32, 4, 7)])
def test_captured_steps_replay(sb, kind, N, R, runs, K):
    """Steps captured into a graph and replayed from new states equal the same
    steps taken directly (the words that workgroups exchange carry a tag that
    no earlier replay used)."""
    import torch
    kw = dict(J=inst.sk_pm1(N, 21)) if kind == "dense" else dict(csr=_sparse(N, 4, 21)[0])
    kw.update(R=R, runs=runs, steps=K, seed=4)
    ctx = sb.sbqa_create(**kw)
    stream = torch.cuda.Stream()
    sb.sbqa_set_stream(ctx, stream)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        sb.sbqa_step(ctx, K)
    for q in range(4):
        _log("replay %d %s N=%d K=%d" % (q, kind, N, K))
        X, Y = inst.uniform_state(N, R * runs, 0.3, 30 + q)
        ref = sb.sbqa_create(**kw)
        sb.sbqa_set_state(ref, X, Y)
        sb.sbqa_step(ref, K)
        sb.sbqa_set_state(ctx, X, Y)
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(sb.sbqa_get_state(ref), sb.sbqa_get_state(ctx)):
            assert np.array_equal(a, b)


# the dense step's tile follows the grid: with few columns 16 or 32 spins per
# workgroup, with many the 64-spin (or split-K) tiles
@pytest.mark.parametrize("coup,prec,fmode,packing", [
    ("gauss", "FP32", 0, 0), ("gauss", "BF16X3", 2, 0), ("sidon", "INT8", 0, 0), ("sk", "FP8", 0, 0), ("sk", "FP8", 1, 1),
    ("sk", "FP4", 0, 0), ("sk", "FP4", 1, 1)])
def test_dense_step_tiles_by_grid(sb, coup, prec, fmode, packing):
    """A column's trajectory does not depend on how many columns are stepped
    beside it, nor on the tile: few columns (fine tiles, padded columns and
    rows) against the same columns among 768 (64-, 128- and 256-column tiles)."""
    N = 700 if coup == "gauss" else 1100
    J = {"gauss": inst.dense_gaussian, "sidon": inst.sidon28_dense, "sk": inst.sk_pm1}[coup](N, 41)
    h = inst.gaussian_fields(N, 0.3, 42) if coup == "gauss" else np.round(inst.gaussian_fields(N, 2.0, 42))
    R, runs = 8, 96 if coup != "gauss" else 192
    X, Y = inst.uniform_state(N, R * runs, 0.4, 43)
    kw = dict(J=J, h=h, R=R, steps=12, fmode=fmode, precision=getattr(sb, "PREC_" + prec), j_packing=packing,
              jp_kind=sb.JP_LINEAR, jp_start=0.5, jp_end=0.0, loop_kernel=sb.LOOP_STREAM)
    ref = None
    for few, tile in ((runs, 64), (runs, 128), (runs, 256), (2, 64), (7, 64), (20, 64), (20, 128), (20, 256), (40, 64)):
        C = R * few
        _log("tiles by grid %s %s C=%d tile %d" % (coup, prec, C, tile))
        ctx = sb.sbqa_create(runs=few, dense_tile=tile, **kw)
        sb.sbqa_set_state(ctx, X[:, :C], Y[:, :C])
        sb.sbqa_step(ctx, 11)
        got = (*sb.sbqa_get_state(ctx), sb.sbqa_fields(ctx))
        E, s = sb.sbqa_best(ctx)
        if ref is None:
            ref = (got, E, s)
        for a, b in zip(ref[0], got):
            assert np.array_equal(a[:, :C], b)
        assert np.array_equal(ref[1][:few], E) and np.array_equal(ref[2][:few], s)


@pytest.mark.parametrize("N,count", [(1, 1), (127, 3), (128, 128), (129, 129), (257, 5), (640, 300), (1000, 1), (2100, 130)])
def test_energies_from_the_lower_triangle(sb, N, count):
    """float64 energies of given spins with real and integer couplings: blocks
    of 128 spins alone, in pairs and with a middle one, part rows; integer
    couplings exact, real ones within 1e-13 of the sum of magnitudes."""
    s = inst.spins_pm1(count, N, 51)
    for J, h in ((inst.dense_gaussian(N, 52), inst.gaussian_fields(N, 0.5, 53)),
                 (inst.sidon28_dense(N, 54) * 1001.0, np.round(inst.gaussian_fields(N, 9.0, 55)))):
        _log("energies N=%d count=%d" % (N, count))
        ctx = sb.sbqa_create(J=J, h=h, R=1, runs=1, steps=1, precision=sb.PREC_FP32)
        E = sb.sbqa_energy(ctx, s)
        sl, Jl, hl = s.astype(np.longdouble), J.astype(np.longdouble), h.astype(np.longdouble)
        ref = np.array([-(r @ (Jl @ r)) / 2 - hl @ r for r in sl[:8]])
        scale = np.abs(Jl).sum() / 2 + np.abs(hl).sum()
        if np.array_equal(J, np.round(J)):
            assert np.array_equal(E[:8], ref.astype(np.float64))
        else:
            assert np.all(np.abs(E[:8] - ref) <= 1e-13 * scale)
        if count > 8:   # the rest against plain float64
            f = s.astype(np.float64)
            assert np.all(np.abs(E - (-0.5 * (f * (f @ J)).sum(1) - f @ h)) <= 1e-13 * float(scale))


# mixes whose grouped dense step takes tiles of 16, 32 and 64 spins
@pytest.mark.parametrize("mix", [[(200, 2), (300, 7)], [(300, 9), (1100, 8), (700, 3)], [(1100, 48), (2300, 48), (300, 3)]])
@pytest.mark.parametrize("coup,prec,packing", [("gauss", "FP32", 0), ("gauss", "BF16X3", 0), ("sidon", "INT8", 0),
                                               ("sk", "FP8", 0), ("sk", "FP8", 1), ("sk", "FP4", 0), ("sk", "FP4", 1)])
def test_served_mix_tiles(sb, coup, prec, packing, mix):
    """Instances of one precision served together (m-block counts and a sparse
    instance side by side in a launch, whole and part step blocks) equal their
    standalone runs."""
    import time
    gen = {"gauss": inst.dense_gaussian, "sidon": inst.sidon28_dense, "sk": inst.sk_pm1}[coup]
    items = [dict(J=gen(N, 61 + q), R=16, runs=runs, steps=70 + 3 * q, seed=65 + q, dense_tile=64 << (q % 3),
                  precision=getattr(sb, "PREC_" + prec), j_packing=packing) for q, (N, runs) in enumerate(mix)]
    items.append(dict(csr=_sparse(777, 5, 60)[0], R=16, runs=mix[0][1], steps=90, seed=60))
    srv = sb.sbqa_server_create(4 << 30, 4)
    _log("served mix %s %s %s" % (coup, prec, mix))
    tickets = [sb.sbqa_submit(srv, **kw) for kw in items]
    for t, kw in zip(tickets, items):
        ctx = sb.sbqa_create(loop_kernel=sb.LOOP_STREAM, **kw)
        sb.sbqa_step(ctx, kw["steps"])
        E, s = sb.sbqa_best(ctx)
        got, t0 = None, time.time()
        while got is None and time.time() - t0 < 60:
            got = sb.sbqa_poll(srv, t)
            time.sleep(0.002)
        assert got is not None and np.array_equal(got[0], E) and np.array_equal(got[1], s)
    sb.sbqa_server_destroy(srv)


# the split-K step at its four workgroup shapes (64 x 64 up to 128 x 128), K
# ranges of uneven and no chunks, padded spins and columns, a lone column tile
@pytest.mark.parametrize("N,C,other", [(2049, 350, 64), (3000, 700, 128), (1100, 1300, 64), (4500, 320, 64), (6100, 500, 256)])
@pytest.mark.parametrize("coup,prec,packing,fmode", [("sidon", "INT8", 0, 0), ("sk", "FP8", 0, 1), ("sk", "FP8", 1, 0),
                                                     ("sk", "FP4", 0, 0), ("sk", "FP4", 1, 1)])
def test_split_k_shapes(sb, N, C, other, coup, prec, packing, fmode):
    """Fields of many columns (split-K) equal those of 32 of them alone (the fine
    tile) and, on sampled spins, the integer product; the steps that follow are
    equal too."""
    R, few = 2, 32
    J = {"sidon": inst.sidon28_dense, "sk": inst.sk_pm1}[coup](N, 71)
    X, Y = inst.uniform_state(N, C, 0.4, 72)
    rows = np.random.default_rng(73).integers(0, N, 40)
    got = []
    for c in (C, few):
        _log("split-K %s %s N=%d C=%d" % (coup, prec, N, c))
        ctx = sb.sbqa_create(J=J, R=R, runs=c // R, steps=8, fmode=fmode, precision=getattr(sb, "PREC_" + prec),
                             j_packing=packing, dense_tile=other, loop_kernel=sb.LOOP_STREAM, jp_kind=sb.JP_LINEAR,
                             jp_start=0.5, jp_end=0.0)
        sb.sbqa_set_state(ctx, X[:, :c], Y[:, :c])
        phi = sb.sbqa_fields(ctx)
        if fmode == 1:   # f = sign(x)
            assert np.array_equal(phi[rows], (J[rows] @ np.sign(X[:, :c]).astype(np.float64)).astype(np.float32))
        sb.sbqa_step(ctx, 5)
        got.append([phi, *sb.sbqa_get_state(ctx), sb.sbqa_fields(ctx)])
    for a, b in zip(*got):
        assert np.array_equal(a[:, :few], b)


@pytest.mark.parametrize("N,d,R,runs", [(8192, 3, 4, 5), (8193, 3, 4, 5), (9001, 9, 16, 20), (40000, 12, 8, 9)])
def test_sparse_readout_batches(sb, N, d, R, runs):
    """Readout of a streamed sparse state around the split of the best update, with
    rows of fewer and more than 8 neighbours and a part last group of rows: the
    best replica's spins and its energy, integer couplings exact."""
    _log("sparse readout N=%d d=%d" % (N, d))
    (rp, col, val), h = _sparse(N, d, 91)
    val, h = np.sign(val) * np.ceil(np.abs(val) * 3), np.round(h * 40)
    ctx = sb.sbqa_create(csr=(rp, col, val), h=h, R=R, runs=runs, steps=4, seed=92, loop_kernel=sb.LOOP_STREAM)
    sb.sbqa_step(ctx, 3)
    E, s = sb.sbqa_best(ctx)
    X, _ = sb.sbqa_get_state(ctx)
    S = np.where(X >= 0, 1.0, -1.0)
    rows = np.repeat(np.arange(N), np.diff(rp))
    phi = np.zeros((N, R * runs))
    np.add.at(phi, rows, val[:, None] * S[col])
    Eall = (-0.5 * (S * phi).sum(0) - h @ S).reshape(runs, R)
    k = Eall.argmin(1)
    assert np.array_equal(E, Eall.min(1))
    assert np.array_equal(s, np.stack([S[:, r * R + k[r]] for r in range(runs)]).astype(np.int8))
