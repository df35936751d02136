"""Products and scans of more rows than one launch of small blocks holds (marked gpu)."""
import pytest

from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oz():
    need_gpu()
    from paper_2609_27831_amd import oz2h
    return oz2h


def _random(oz, gen, rows, cols, p):
    X = oz.empty_mp(rows, cols, p)
    X.sign.random_(0, 2, generator=gen).mul_(2).sub_(1)
    X.exp.random_(-3, 4, generator=gen)
    X.limbs.random_(1 << (p - 1), 1 << p, generator=gen)
    return X


def test_product_of_more_than_65535_tiles_of_rows(oz):
    """128-row tiles would be 65539 to a launch (and no multiple of 8): the product equals its two halves'."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(5)
    p, M, N, K = 8, 65538 * 128 + 5, 70, 4
    plan = oz.Plan.custom(p, 8, K, [251, 253, 255])
    A, B = _random(oz, gen, M, K, p), _random(oz, gen, K, N, p)
    print(f"{M} x {N} x {K}", flush=True)
    C = oz.gemm(plan, A, B)
    half = M // 2
    for lo, hi in ((0, half), (half, M)):
        D = oz.gemm(plan, oz.DeviceMP(A.sign[lo:hi], A.exp[lo:hi], A.limbs[lo:hi], p), B)
        for a, b in ((C.sign, D.sign), (C.exp, D.exp), (C.limbs, D.limbs)):
            assert torch.equal(a[lo:hi], b)
