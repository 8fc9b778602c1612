"""The parity tests once more on tables that are no exact product plus a small error: the multiplier of the configurations has a
byte form (9 bits and more: a column form), which kernels of its own serve, so that the kernels for arbitrary tables (derived
tables of 16-bit entries and of two digits, gathers from memory) would otherwise run in few of these tests."""
import numpy as np
import pytest

from test_gpu_parity import *       # noqa: F401,F403 (the tests, their fixture and their marker)
from paper_2203_04071_amd import workloads as wl

del test_stored_small_cases         # noqa: F821 (stored for the tables of the configurations)


@pytest.fixture(autouse=True)
def general_tables(monkeypatch):
    make = wl.make_lut

    def general(bits, err=None, seed=None, symmetric=True):
        return make(bits, err=200 if bits <= 8 else 40000, seed=seed, symmetric=symmetric)

    monkeypatch.setattr(wl, "make_lut", general)


def test_the_tables_here_have_neither_form():
    for bits in range(4, 13):
        h = 1 << (bits - 1)
        v = np.arange(-h, h, dtype=np.int64)
        t = wl.make_lut(bits).astype(np.int64)
        if bits > 8:
            assert np.ptp(t - v[:, None] * v[None, :]) > 65535
            continue
        assert abs(t).max() <= 32767
        for da in range(4):
            for dw in range(4):
                assert np.ptp(t - (v & -(1 << da))[:, None] * (v & -(1 << dw))[None, :]) > 255
