"""Rules of the host side that need no GPU, through the library's internal
entry points."""
import ctypes as ct

import pytest

import paper_2604_01050_amd as sb

FINE16, FINE32, TILE, SK11, SK21, SK12, SK22 = range(1, 8)
F32, FP8, BF16X3, I8, FP8PK, FP4, FP4PK = 0, 1, 2, 4, 5, 6, 7


def _form(path, Np, mbw, Cg):
    return sb.lib._ZN4sbqa18default_dense_formENS_4PathEiii(path, Np, mbw, Cg)


@pytest.mark.parametrize("path", [FP8, I8, FP8PK, FP4, FP4PK])
def test_split_k_only_in_full_rounds(path):
    """A split-K workgroup has a CU to itself: with two or fewer 64 x 64 tiles
    per CU it takes them, above that only where its rounds are nearly full (and J
    bit-packed) or the 64-spin tile is one of 256 columns; every other grid keeps
    the tiles of which a CU runs several."""
    for Np in (512, 1536, 4096, 5120, 16384):
        for C64 in range(1, 49):
            for mbw in (1, 2, 4):
                if C64 % mbw:
                    continue
                n, form = Np // 64 * C64, _form(path, Np, mbw, 64 * C64)
                if n <= 512:
                    assert form != TILE
                    assert form not in (SK11, SK22) or n <= 256
                elif path in (FP8PK, FP4PK) and C64 % 2 == 0 and n / 1024 >= 0.85 * -(-n // 1024):
                    assert form == SK22
                else:
                    assert form == (SK22 if mbw == 4 and n <= 1024 else TILE)
                assert form not in (SK12, SK22) or C64 % 2 == 0   # whole column pairs


@pytest.mark.parametrize("path", [F32, BF16X3])
def test_real_paths_never_split_k(path):
    for Np in (128, 1536, 8192):
        for C64 in range(1, 20):
            assert _form(path, Np, 1, 64 * C64) <= TILE


class _EnergyPlan(ct.Structure):
    _fields_ = [("T", ct.c_int), ("Z", ct.c_int), ("units", ct.c_int), ("cp", ct.c_int)]


def test_energy_plan_splits_small_instances():
    """The K tiles (16 spins) that one work unit of the float64 energies walks
    one after the other are few in small instances, and the partial
    sums stay within the scratch that the allocation-free entry point allows."""
    plan = sb.lib._ZN4sbqa11energy_planEii
    plan.restype = _EnergyPlan
    for N in list(range(1, 300, 7)) + [511, 512, 700, 1000, 1500, 2000, 4100, 16384]:
        for count in (1, 128, 129, 1000, 5000):
            e = plan(N, count)
            T, cp = -(-N // 128), -(-count // 128) * 128
            assert (e.T, e.cp, e.units) == (T, cp, (T + 1) // 2 * e.Z) and 1 <= e.Z <= 16
            chain = -(-8 * (T + 1) // e.Z)       # of the pair of spin blocks of a unit
            if N <= 1024 and count <= 1000:
                assert chain <= 5, (N, count, chain)
            Np = -(-N // 128) * 128
            assert e.units <= Np                 # doubles per row: the smallest allowance is Np
