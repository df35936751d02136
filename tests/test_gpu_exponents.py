"""Shared exponents in one launch (marked gpu): rows per block, partial blocks, contractions of
partial rounds and long ones split over blocks, in both layouts, against numpy's maxima."""
import numpy as np
import pytest

import synth
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


# the lines of the rules for strided sides: 128 rows, a contraction of 2048, 3500 alone
@pytest.mark.parametrize("rows,count", [(16, 2049), (128, 2049), (128, 8000), (129, 3500), (129, 3501), (300, 6000), (2000, 3600)])
def test_strided_rows(oz, rows, count):
    test_row_maxima(oz, rows, count, False)


@pytest.mark.parametrize("K", [6144, 6145])
def test_sides_of_one_product(oz, K):
    """A strided side that shares the launch, or is split while the other is not, against sides on their own."""
    import torch
    M, N, p = 200, 210, 53
    A, B = (oz.to_device(synth.mp_random(K + i, *s, p, -90, 90)) for i, s in enumerate([(M, K), (K, N)]))
    plan = oz.Plan.create(p, K)
    print(f"exponents of a product, K = {K}", flush=True)
    C = oz.gemm(plan, A, B)
    D = oz.gemm_from_residues(plan, ra=oz.Residues(plan, A, oz.SIDE_A), rb=oz.Residues(plan, B, oz.SIDE_B))
    assert all(torch.equal(a, b) for a, b in ((C.sign, D.sign), (C.exp, D.exp), (C.limbs, D.limbs)))
