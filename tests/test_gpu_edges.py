"""Edges of the kernels' tiles, splits and dispatch rules, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2507_13681_amd import binding, inputs
from tests.test_gpu_decode import _case, _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,cap,T,d,ragged", [
    (1, 2, 2, 31, 1, 128, False),      # a partial tile and a one-row tail tile
    (1, 16, 1, 32, 32, 64, False),     # whole tiles only; a full block of 16 heads
    (1, 17, 1, 33, 0, 128, True),      # a second block of heads with one head
    (2, 12, 2, 545, 33, 64, True),     # 20 tiles: two or three a wave and several splits; the tail's tiles move with the count
    (1, 32, 8, 575, 1, 128, True),     # 19 tiles: beyond one workgroup's share, splits of unequal length
    (1, 24, 1, 9000, 40, 128, True),   # many splits, two blocks of heads
])
def test_decode_tiles_and_splits(oracle, B, Hq, Hkv, cap, T, d, ragged):
    print(f"decode edge B={B} Hq={Hq} Hkv={Hkv} cap={cap} T={T} d={d}", flush=True)
    _check(oracle, _case(B, Hq, Hkv, cap, T, d, seed=3 * cap + T, ragged=ragged))
