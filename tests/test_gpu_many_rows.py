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


@pytest.mark.parametrize("rows,strided", [(40_000_003, False), (140_000_003, True)])
def test_exponents_of_many_rows(oz, rows, strided):
    """Contiguous rows beyond a launch's threads at 64 to a row, and strided ones at 32."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(6)
    shape = (2, rows) if strided else (rows, 2)
    sign = torch.randint(-1, 2, shape, dtype=torch.int8, device="cuda", generator=gen)
    exp = torch.randint(-9, 10, shape, dtype=torch.int32, device="cuda", generator=gen)
    print(f"exponents of {rows} rows", flush=True)
    out = oz.exponents(sign, exp, rows, 2, *((1, rows) if strided else (2, 1)))
    masked = torch.where(sign != 0, exp, torch.full_like(exp, -100)).amax(0 if strided else 1)
    assert torch.equal(out, torch.where(masked == -100, torch.zeros_like(masked), masked))
    assert not oz.exponents(sign, exp, rows, 0, 1, rows, out=out).any()   # an empty contraction
