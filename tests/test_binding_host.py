"""The binding's packed configuration structure equals the one filled field by
field, for every level count, and keeps accepting what that accepted."""
import ctypes
import itertools

import numpy as np
import pytest

from paper_1909_10616_amd import gemmtune as gt


def by_fields(cfg):
    c = gt.gt_config()
    c.d_m, c.d_k, c.d_n = (len(x) for x in cfg[:3])
    for arr, vals in ((c.m, cfg[0]), (c.k, cfg[1]), (c.n, cfg[2])):
        for i, v in enumerate(vals):
            arr[i] = int(v)
    c.mfma = int(cfg[3]) if len(cfg) > 3 else 0
    return c


@pytest.mark.parametrize("d", itertools.product((1, 4), (2, 3), (1, 4)))
@pytest.mark.parametrize("convert", [int, float, np.int64])
def test_packed_configuration_equals_the_fields(d, convert):
    levels = [[convert(2 ** (i + j)) for i in range(n)] for j, n in enumerate(d)]
    for cfg in ((*levels, 16), (*map(tuple, levels), 0), tuple(levels), (*levels, convert(32)),
                ([1 << 40], [3], [-5], 0)):
        assert bytes(gt.to_c(cfg)) == bytes(by_fields(cfg))
    assert ctypes.sizeof(gt.gt_config) == gt._CONFIG.size


def test_too_many_levels_still_raise():
    with pytest.raises(IndexError):
        gt.to_c(((1,) * 5, (1,), (1,), 0))
