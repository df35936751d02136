"""Shared exponents in one launch (marked gpu): rows per block, partial blocks, contractions of
partial rounds and long ones split over blocks, in both layouts, against numpy's maxima."""
import numpy as np
import pytest

from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oz():
    need_gpu()
    from paper_2609_27831_amd import oz2h
    return oz2h


@pytest.mark.parametrize("rows,count", [(1, 1), (1, 5000), (3, 64), (15, 65), (17, 1025), (33, 8192), (1023, 100),
                                        (1024, 257), (1500, 4100), (40, 8193), (9000, 33), (4097, 8200)])
@pytest.mark.parametrize("contig", [True, False])
def test_row_maxima(oz, rows, count, contig):
    import torch
    rng = np.random.default_rng(rows + count)
    ld = (count if contig else rows) + 3
    shape = (rows, ld) if contig else (count, ld)
    exp = rng.integers(-2000, 2000, shape).astype(np.int32)
    sign = rng.integers(-1, 2, shape).astype(np.int8)
    exp[rng.random(shape) < 0.01] = 5000          # next to the row's end as well: the padding must not count
    s, e = (sign[:, :count], exp[:, :count]) if contig else (sign[:, :rows].T, exp[:, :rows].T)
    s[rows // 2] = 0                               # an all-zero row has exponent 0
    if count > 1:
        s[0], s[0, count - 1], e[0, count - 1] = 0, -1, -7
    ref = np.where((s != 0).any(1), np.where(s != 0, e, -2 ** 31).max(1), 0)
    print(f"exponents {rows} x {count} contiguous={contig}", flush=True)
    rs, cs = (ld, 1) if contig else (1, ld)
    got = oz.exponents(torch.from_numpy(sign).cuda(), torch.from_numpy(exp).cuda(), rows, count, rs, cs)
    assert np.array_equal(got.cpu().numpy(), ref)
