"""GPU tests of the library's choices between kernels for a call: every choice
gives the same bits."""
import os
import subprocess
import sys

import numpy as np
import pytest

import sbqa_instances as inst

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def sb():
    import paper_2604_01050_amd as sb
    return sb


def _log(msg):
    print(msg, flush=True)


_FORMS = """
import os, sys
sys.path.insert(0, %r)
import numpy as np, torch
import paper_2604_01050_amd as sb
import sbqa_instances as inst
p = torch.cuda.get_device_properties(0)
dev = "%%s %%d" %% (p.gcnArchName, p.multi_processor_count)
N, R, few = 1500, 2, 32
cases = [("sidon", "INT8", 0, 4, 0), ("sk", "FP8", 0, 5, 1), ("sk", "FP8", 1, 1, 0), ("sk", "FP4", 0, 7, 0),
         ("sk", "FP4", 1, 6, 1), ("gauss", "FP32", 0, 0, 2), ("gauss", "BF16X3", 0, 2, 2)]
keys = {}   # (case, columns): form and operand grouping named in the tile file
with open(os.environ["SBQA_TUNE_CACHE"], "w") as f:
    for coup, prec, packing, path, fmode in cases:
        q = 0
        for form in (range(1, 8) if coup != "gauss" else range(1, 4)):
            for mbw in (1, 2, 4):
                q += 1
                keys[prec, packing, 128 * q] = (form, mbw)
                f.write("sbqa-tile-v1 %%s %%d %%d 1536 %%d\\n" %% (dev, path + 16 * form, 128 * q, mbw))
J = {c: {"sidon": inst.sidon28_dense, "sk": inst.sk_pm1, "gauss": inst.dense_gaussian}[c](N, 71) for c in ("sidon", "sk", "gauss")}
X, Y = inst.uniform_state(N, 128 * 21, 0.4, 72)
X[:, 0] = 0.0
h = np.round(inst.gaussian_fields(N, 2.0, 73))
for coup, prec, packing, path, fmode in cases:
    ref = None
    for C in [few] + sorted(c for p_, k, c in keys if (p_, k) == (prec, packing)):
        form, mbw = keys.get((prec, packing, C), (0, 0))
        print(coup, prec, packing, "C=%%d form %%d mbw %%d" %% (C, form, mbw), flush=True)
        ctx = sb.sbqa_create(J=J[coup], h=h, R=R, runs=C // R, steps=8, fmode=fmode, precision=getattr(sb, "PREC_" + prec),
                             j_packing=packing, dense_tile=64 if C == few else 0, loop_kernel=sb.LOOP_STREAM,
                             jp_kind=sb.JP_LINEAR, jp_start=0.5, jp_end=0.0)
        assert C == few or sb.sbqa_info(ctx)["tile_cols"] == 64 * mbw
        sb.sbqa_set_state(ctx, X[:, :C], Y[:, :C])
        phi = sb.sbqa_fields(ctx)
        if coup != "gauss":   # the threshold is 0 at the first step: f = sign(x)
            assert np.array_equal(phi, (J[coup] @ np.sign(X[:, :C]).astype(np.float64)).astype(np.float32))
        sb.sbqa_step(ctx, 5)
        E, s = sb.sbqa_best(ctx)
        got = [phi, *sb.sbqa_get_state(ctx), sb.sbqa_fields(ctx), E[None], s.T]
        if ref is None:
            ref = got
        for a, b in zip(ref, got):
            assert np.array_equal(a, b[:, :a.shape[1]])
print("forms agree")
"""


def test_every_form_of_the_dense_step(tmp_path):
    """The dense step in each of its forms (16- and 32-spin tiles, the 64-spin
    tile, split-K at its four workgroup shapes) and operand groupings, named
    through the tile file: fields exact for integer couplings, then fields, states
    and readouts equal to those of 32 columns alone."""
    _log("forms of the dense step")
    r = subprocess.run([sys.executable, "-u", "-c", _FORMS % ROOT], capture_output=True, text=True, timeout=110,
                       env=dict(os.environ, SBQA_TUNE_CACHE=str(tmp_path / "tiles.txt")))
    assert r.returncode == 0 and "forms agree" in r.stdout, r.stdout[-500:] + r.stderr[-2000:]


# one slab and several (rows of 8 to 4100 columns; above 8 MB for x and y), all three
# orders of the state in memory, relabelled rows
@pytest.mark.parametrize("kind,N,R,runs", [("dense", 60, 1, 1), ("dense", 300, 10, 6), ("dense", 700, 4, 1025),
                                           ("resident", 777, 8, 1), ("resident", 600, 16, 130), ("stream", 3001, 3, 5),
                                           ("relabelled", 9000, 4, 2), ("relabelled", 9001, 7, 33),
                                           ("stream", 40000, 4, 16)])
def test_state_transfer(sb, kind, N, R, runs):
    """A state handed in comes back bit for bit, whole or one half of it, the
    start of a context is the same draw in every order, and a refused state
    changes nothing."""
    _log("state transfer %s N=%d C=%d" % (kind, N, R * runs))
    if kind == "dense":
        kw = dict(J=inst.sk_pm1(N, 5))
    else:
        E = inst.regular_graph(N, 3 if N % 2 == 0 else 4, 6)
        kw = dict(csr=inst.edges_to_csr(N, E, inst.gaussian_edges(len(E), 7)), seed=8,
                  reorder=sb.REORDER_ON if kind == "relabelled" else sb.REORDER_OFF,
                  loop_kernel=sb.LOOP_RESIDENT if kind == "resident" else sb.LOOP_STREAM)
    ctx = sb.sbqa_create(R=R, runs=runs, steps=4, **kw)
    assert sb.sbqa_info(ctx)["reordered"] == (kind == "relabelled")
    x0, y0 = sb.sbqa_get_state(ctx)
    if kind in ("relabelled", "resident"):
        ref = sb.sbqa_create(R=R, runs=runs, steps=4, **dict(kw, reorder=sb.REORDER_OFF, loop_kernel=sb.LOOP_STREAM))
        assert all(np.array_equal(a, b) for a, b in zip((x0, y0), sb.sbqa_get_state(ref)))
    x, y = inst.uniform_state(N, R * runs, 0.7, 9)
    sb.sbqa_set_state(ctx, x, y)
    bad = y.copy()
    bad[-1, -1] = np.inf
    with pytest.raises(sb.SbqaError):
        sb.sbqa_set_state(ctx, x0, bad)
    gx, gy = sb.sbqa_get_state(ctx)
    assert np.array_equal(gx, x) and np.array_equal(gy, y)
    only = np.full_like(y, 7.0)
    assert sb.lib.sbqa_get_state(ctx.ptr, None, only.ctypes.data) == sb.OK and np.array_equal(only, y)
    only[:] = 7.0
    assert sb.lib.sbqa_get_state(ctx.ptr, only.ctypes.data, None) == sb.OK and np.array_equal(only, x)
    assert sb.lib.sbqa_get_state(ctx.ptr, None, None) == sb.OK


# the loops of every shape that takes few steps another way
@pytest.mark.parametrize("kind,N,R,runs", [("sk", 200, 16, 8), ("sk", 601, 16, 8), ("sk", 700, 16, 40), ("sk", 1000, 16, 30),
                                           ("sk", 1500, 32, 8), ("sparse", 200, 8, 4), ("sparse", 1000, 16, 8),
                                           ("sparse", 200, 64, 16), ("sparse", 2500, 16, 2)])
def test_calls_of_few_and_many_steps(sb, kind, N, R, runs):
    """Steps taken in calls of 1 to 40, with readouts, fields and a state
    overwrite between them, equal one launch per step."""
    if kind == "sk":
        kw = dict(J=inst.sk_pm1(N, 31), h=np.round(inst.gaussian_fields(N, 1.0, 32)))
    else:
        E = inst.regular_graph(N, 4, 33)
        kw = dict(csr=inst.edges_to_csr(N, E, inst.gaussian_edges(len(E), 34)), h=inst.gaussian_fields(N, 0.1, 35))
    out = []
    for kern in (sb.LOOP_STREAM, sb.LOOP_AUTO):
        _log("calls of few and many steps %s N=%d C=%d kernel %d" % (kind, N, R * runs, kern))
        ctx = sb.sbqa_create(R=R, runs=runs, steps=150, loop_kernel=kern, seed=36, **kw)
        got = []
        for q, K in enumerate((1, 1, 3, 40, 1, 2, 1, 5, 20, 4, 1, 1, 30, 1)):
            sb.sbqa_step(ctx, K)
            if q % 3 == 0:
                got += [*sb.sbqa_best(ctx)]
            if q % 3 == 1:
                got += [sb.sbqa_fields(ctx), *sb.sbqa_get_state(ctx)]
            if q in (4, 8):
                sb.sbqa_set_state(ctx, *inst.uniform_state(N, R * runs, 0.5, 37 + q))
        out.append(got + [*sb.sbqa_get_state(ctx), *sb.sbqa_best(ctx)])
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("kind,N", [("dense", 601), ("sparse", 1000)])
def test_recorded_steps_between_direct_ones(sb, kind, N):
    """Steps recorded into a graph replay on the context's state after direct
    steps, of one and of several, taken before and after the recording."""
    import torch
    E = inst.regular_graph(N + N % 2, 4, 41)
    kw = dict(J=inst.sk_pm1(N, 41)) if kind == "dense" else dict(csr=inst.edges_to_csr(N, E, inst.gaussian_edges(len(E), 42)))
    kw.update(R=16, runs=8, steps=40, seed=4, jp_kind=sb.JP_LINEAR, jp_start=0.5, jp_end=0.0)
    ctx = sb.sbqa_create(**kw)
    sb.sbqa_step(ctx, 1)
    stream = torch.cuda.Stream()
    sb.sbqa_set_stream(ctx, stream)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        sb.sbqa_step(ctx, 7)        # steps 1..7
    X, Y = inst.uniform_state(N, 128, 0.3, 43)
    for q in range(3):
        _log("replay %d after direct steps %s" % (q, kind))
        sb.sbqa_step(ctx, 1 + q)    # (the state they leave is overwritten)
        sb.sbqa_set_state(ctx, X, Y)
        graph.replay()
        torch.cuda.synchronize()
        ref = sb.sbqa_create(loop_kernel=sb.LOOP_STREAM, **kw)
        sb.sbqa_step(ref, 1)
        sb.sbqa_set_state(ref, X, Y)
        sb.sbqa_step(ref, 7)
        for a, b in zip(sb.sbqa_get_state(ref), sb.sbqa_get_state(ctx)):
            assert np.array_equal(a, b)


def test_exchanging_launches_on_several_streams(sb):
    """Contexts whose loops' workgroups wait for each other, on streams of their
    own and from two threads: more of them than fit on the device together give
    what each gives alone."""
    import threading

    import torch

    def sparse(N, d, seed):
        E = inst.regular_graph(N, d, seed)
        return dict(csr=inst.edges_to_csr(N, E, inst.gaussian_edges(len(E), seed + 1)), h=inst.gaussian_fields(N, 0.1, seed + 2))

    kinds = [dict(sparse(4096, 6, 51), R=2048, runs=1),               # 8 columns: a ring of 256 workgroups
             dict(J=inst.sk_pm1(2048, 52), R=16, runs=8),             # many-step dense loop
             dict(sparse(1000, 3, 53), R=16, runs=8),                 # narrow loop
             dict(sparse(4096, 6, 54), R=32, runs=64),                # 8 columns: 256 workgroups
             dict(J=inst.sk_pm1(601, 55), R=16, runs=16)]

    def advance(ctx, get):
        for K in (20, 1, 150, 7, 60):
            sb.sbqa_step(ctx, K)
        return get(ctx)

    make = lambda kw: sb.sbqa_create(steps=240, seed=5, **kw)
    alone = []
    for kw in kinds:
        _log("alone R=%d runs=%d" % (kw["R"], kw["runs"]))
        alone.append(advance(make(kw), lambda c: (*sb.sbqa_get_state(c), *sb.sbqa_best(c))))
    streams = [torch.cuda.Stream() for _ in kinds]
    for rep in range(3):
        _log("together, pass %d" % rep)
        ctxs = [make(kw) for kw in kinds]
        for c, st in zip(ctxs, streams):
            sb.sbqa_set_stream(c, st)
        ts = [threading.Thread(target=lambda part: [advance(c, lambda _: None) for c in part], args=(ctxs[q::2],)) for q in range(2)]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        for c, ref in zip(ctxs, alone):
            for a, b in zip(ref, (*sb.sbqa_get_state(c), *sb.sbqa_best(c))):
                assert np.array_equal(a, b)
        for c in ctxs:
            sb.sbqa_destroy(c)


@pytest.mark.parametrize("kind", ["dense", "sparse"])
def test_steps_above_the_longest_launch(sb, kind):
    """A call of more steps than one launch of an exchanging loop takes."""
    N = 300
    E = inst.regular_graph(N, 3, 61)
    kw = dict(J=inst.sk_pm1(N, 62)) if kind == "dense" else dict(csr=inst.edges_to_csr(N, E, inst.gaussian_edges(len(E), 63)))
    _log("9000 steps in one call, %s" % kind)
    out = []
    for kern in (sb.LOOP_STREAM, sb.LOOP_AUTO):
        ctx = sb.sbqa_create(R=8, runs=2, steps=9000, loop_kernel=kern, seed=3, **kw)
        sb.sbqa_step(ctx, 9000)
        out.append((*sb.sbqa_get_state(ctx), *sb.sbqa_best(ctx)))
    for a, b in zip(*out):
        assert np.array_equal(a, b)


def test_wait_timeout_of_the_dense_loop_is_reported(sb):
    """A wait of the many-step dense loop that timed out: the next calls that
    synchronise report it, the kernels end normally, and the context of another
    instance is not touched. One workgroup per group waits for nobody."""
    _log("injected wait timeout, dense loop")
    kw = dict(J=inst.sk_pm1(601, 64), R=16, runs=8, steps=40)
    ctx, other = sb.sbqa_create(**kw), sb.sbqa_create(**kw)
    sb.sbqa_step(ctx, 9)
    sb.sbqa_best(ctx)
    sb.sbqa_inject_wait_timeout(ctx)
    sb.sbqa_step(ctx, 9)
    for call in (sb.sbqa_best, sb.sbqa_sync, sb.sbqa_get_state):
        with pytest.raises(sb.SbqaError) as ei:
            call(ctx)
        assert ei.value.status == sb.EDEVICE and "wait timed out" in ei.value.message
    sb.sbqa_step(other, 18)
    sb.sbqa_best(other)
    with pytest.raises(sb.SbqaError) as ei:
        sb.sbqa_inject_wait_timeout(sb.sbqa_create(J=inst.sk_pm1(200, 65), R=16, runs=8, steps=40))
    assert ei.value.status == sb.EINVAL


def test_cached_memory_goes_back(sb):
    """What destroyed contexts leave cached is bounded and goes back when asked."""
    import gc

    import torch
    _log("cached memory")
    make = lambda: sb.sbqa_create(J=inst.sk_pm1(1500, 71), R=16, runs=16, steps=10, precision=sb.PREC_FP32)
    sb.sbqa_destroy(make())
    gc.collect()
    sb.sbqa_release_cached()
    free0 = torch.cuda.mem_get_info()[0]
    kept = [make() for _ in range(3)]
    for c in kept:
        sb.sbqa_destroy(c)
    free1 = torch.cuda.mem_get_info()[0]
    sb.sbqa_release_cached()
    free2 = torch.cuda.mem_get_info()[0]
    assert 0 < free0 - free1 <= 288 << 20 and free2 >= free0 - (4 << 20), (free0, free1, free2)
    c = make()
    sb.sbqa_step(c, 3)
    sb.sbqa_best(c)


@pytest.mark.parametrize("kind,kern", [("dense", "AUTO"), ("dense", "STREAM"), ("small", "AUTO"), ("sparse", "AUTO"),
                                       ("sparse", "STREAM")])
def test_destroy_while_a_recorded_block_replays(sb, kind, kern):
    """A context destroyed while its recorded steps replay on another stream: its
    memory reaches later contexts only once they have ended."""
    import torch
    _log("destroy under replays, %s %s" % (kind, kern))
    N = 60 if kind == "small" else 1000
    E = inst.regular_graph(N, 3, 81)
    kw = dict(csr=inst.edges_to_csr(N, E, inst.gaussian_edges(len(E), 82))) if kind == "sparse" else dict(J=inst.sk_pm1(N, 83))
    kw.update(R=16, runs=8, steps=400, seed=6, loop_kernel=getattr(sb, "LOOP_" + kern))

    def solve():
        c = sb.sbqa_create(**kw)
        sb.sbqa_step(c, 30)
        return (*sb.sbqa_get_state(c), *sb.sbqa_best(c))

    ref = solve()
    for rep in range(2):
        ctx = sb.sbqa_create(**kw)
        A, B = torch.cuda.Stream(), torch.cuda.Stream()
        sb.sbqa_set_stream(ctx, A)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=A):
            sb.sbqa_step(ctx, 200)
        sb.sbqa_sync(ctx)
        with torch.cuda.stream(B):
            for _ in range(20):
                graph.replay()
        sb.sbqa_destroy(ctx)
        for a, b in zip(ref, solve()):
            assert np.array_equal(a, b)
        torch.cuda.synchronize()
