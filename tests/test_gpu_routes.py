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
