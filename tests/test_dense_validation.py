"""Validation of dense couplings (CPU): +-1 matrices take a pass over their
bits, everything else the general scan; both have to accept and refuse the same
matrices with the same messages."""
import numpy as np
import pytest

import paper_2604_01050_amd as sb
import sbqa_instances as inst


def _outcome(J, **kw):
    """None when validation passes (creation then stops at the missing GPU)."""
    try:
        sb.sbqa_create(J=J, R=2, runs=1, steps=2, **kw)
    except sb.SbqaError as e:
        return None if e.status == sb.EDEVICE else e.message
    return None


def _expected(J):
    """The general scan's verdict: blocks of 64 rows in order; in a block the
    diagonal and finiteness row by row, then symmetry by 64-column blocks."""
    N = len(J)
    for b in range(0, N, 64):
        for i in range(b, min(N, b + 64)):
            if J[i, i] != 0.0:
                return "J has a non-zero diagonal at %d" % i
            bad = np.nonzero(~np.isfinite(J[i]))[0]
            if len(bad):
                return "J[%d][%d] is not finite" % (i, bad[0])
        for c in range(b, N, 64):
            for i in range(b, min(N, b + 64)):
                for j in range(max(c, i + 1), min(N, c + 64)):
                    if J[i, j] != J[j, i] and not (np.isnan(J[i, j]) and np.isnan(J[j, i])):
                        return "J is not symmetric at (%d,%d)" % (i, j)
    return None


@pytest.mark.parametrize("N", [2, 63, 64, 65, 127, 130, 700])
def test_pm1_pass_refuses_what_the_general_scan_refuses(N):
    J0 = inst.sk_pm1(N, 3)
    assert _outcome(J0) is None and _outcome(J0, precision=sb.PREC_FP8) is None
    J = J0.copy()
    J[range(N), range(N)] = -0.0                      # a negative zero on the diagonal is a zero
    assert _outcome(J, precision=sb.PREC_FP4) is None
    rng = np.random.default_rng(N)
    for q in range(12):
        J = J0.copy()
        i, j = sorted(rng.choice(N, 2, replace=False)) if N > 2 else (0, 1)
        if q % 4 == 0:
            J[i, j] = -J[i, j]                        # not symmetric (either half)
        elif q % 4 == 1:
            J[j, i] = -J[j, i]
        elif q % 4 == 2:
            J[i, i] = rng.choice([1.0, -1.0, 0.5, np.nan])
        else:
            J[i, j] = rng.choice([np.nan, np.inf, 2.0, 0.0])
        assert _outcome(J) == _expected(J), (q, i, j)


def test_nearly_pm1_matrices_take_the_general_scan():
    J = inst.sk_pm1(130, 4)
    J[5, 70] = J[70, 5] = 0.0                          # ternary: e4m3 accepts it
    assert _outcome(J, precision=sb.PREC_FP8) is None
    J[5, 70] = J[70, 5] = 2.0
    assert "J in {-1,0,+1}" in _outcome(J, precision=sb.PREC_FP8)
    assert _outcome(J, precision=sb.PREC_INT8) is None
    J[5, 70] = J[70, 5] = 1.5
    assert "integer J" in _outcome(J, precision=sb.PREC_INT8)
    J[5, 70] = J[70, 5] = 2147483648.0                 # an integer outside the 32-bit range
    assert "integer J" in _outcome(J, precision=sb.PREC_INT8)
    assert _outcome(J, precision=sb.PREC_FP32) is None
