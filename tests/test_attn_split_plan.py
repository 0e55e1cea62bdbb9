"""The attention's key split (attn_split_plan, host code) for 256 compute units: which
units are split and into how many pieces.  The function is not part of the C ABI; the
library's own C++ symbol is called."""
import ctypes
import os

import numpy as np
import pytest

import paper_2609_34144_amd as cast

CUS = 256


class Plan(ctypes.Structure):
    _fields_ = [("n_full", ctypes.c_int), ("n_split", ctypes.c_int), ("split", ctypes.c_int),
                ("bytes", ctypes.c_size_t)]


@pytest.fixture(scope="module")
def plan():
    if not os.path.exists(cast.LIB_PATH):
        pytest.skip("libcast.so not built (run __graft_entry__.build())")
    fn = getattr(cast.load(), "_ZN4cast15attn_split_planEiiiixi")
    fn.restype = Plan
    fn.argtypes = [ctypes.c_int] * 4 + [ctypes.c_longlong, ctypes.c_int]
    return lambda units, dh, tiles: fn(1, 1, units, dh, 64 * tiles, CUS)


@pytest.mark.parametrize("dh", [32, 64])
@pytest.mark.parametrize("rounds", [0, 1, 2])
@pytest.mark.parametrize("past", [1, 4, 20, 44, 86, 128])
@pytest.mark.parametrize("tiles", [32, 33, 64, 98, 501])
def test_units_past_one_per_compute_unit_are_split(plan, dh, rounds, past, tiles):
    """One whole unit per compute unit and the few past them in pieces: whole, those few
    held the launch at the rate of two workgroups per unit."""
    units = rounds * 2 * CUS + CUS + past
    p = plan(units, dh, tiles)
    assert (p.n_full, p.n_split) == (units - past, past)
    assert p.split == min(8, CUS // past, tiles // 16) >= 2


@pytest.mark.parametrize("dh,units,tiles,split", [
    # (dh = 128: 27.2 us whole, 31.3 in four; 41.3 in three, 47.2 in four; 20.0 and 21.7)
    (128, 64, 14, 1), (128, 64, 48, 3), (128, 24, 8, 1), (128, 128, 24, 1),
    # (16.5 whole, 19.3 in five; 19.2 and 21.4)
    (64, 40, 10, 1), (32, 128, 16, 1)])
def test_split_that_costs_more_than_it_saves(plan, dh, units, tiles, split):
    assert max(plan(units, dh, tiles).split, 1) == split


def test_pieces_fit_the_grid(plan):
    rng = np.random.default_rng(0)
    for _ in range(20000):
        units, tiles = int(np.exp(rng.uniform(0, 8))), int(np.exp(rng.uniform(0, 7)))
        dh = int(rng.choice([32, 64, 128]))
        slots = CUS if dh == 128 else 2 * CUS
        p = plan(units, dh, tiles)
        assert p.n_full + p.n_split == units and p.n_full >= 0
        if p.n_split == 0:
            continue
        assert 2 <= p.split <= 16 and 2 * p.split <= tiles and p.n_split * p.split <= slots
        assert p.n_full % CUS == 0
        assert p.bytes >= p.n_split * p.split * 256 * (dh + 1) * 4


def test_workspace_never_falls_as_the_history_grows(plan):
    """A workspace sized for the longest history serves every shorter one."""
    rng = np.random.default_rng(1)
    shapes = [(128, 64), (32, 64), (64, 16)] + [
        (int(rng.choice([32, 64, 128])), int(np.exp(rng.uniform(0, 7.5)))) for _ in range(400)]
    for dh, units in shapes:
        size = 0
        for tiles in list(range(1, 200)) + [256, 300, 500, 511, 512, 1000, 5000]:
            p = plan(units, dh, tiles)
            assert p.bytes >= size, (dh, units, tiles)
            assert p.bytes >= p.n_split * p.split * 256 * (dh + 1) * 4
            size = p.bytes
