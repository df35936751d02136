"""The matrix-core CRT beyond 32 digits (marked gpu): every step count, the digit counts where the
vector kernels it is compared with change, against plain plans bit for bit; flags set later and
backward products."""
import pytest

import synth
from tests.gpu_util import dev_mp, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oz():
    need_gpu()
    from paper_2609_27831_amd import oz2h
    return oz2h


def _same(a, b):
    import torch
    return torch.equal(a.sign, b.sign) and torch.equal(a.exp, b.exp) and torch.equal(a.limbs, b.limbs)


# 460 is the first beyond 32 digits at K = 60; 1560 has more than 255 moduli (the row CRT again)
@pytest.mark.parametrize("p", [450, 460, 470, 520, 600, 700, 705, 830, 1024, 1200, 1400, 1480, 1560])
def test_products_against_the_vector_kernels(oz, p):
    M, N, K = 37, 41, 60
    A, B = dev_mp(synth.mp_random(p, M, K, p, -20, 20)), dev_mp(synth.mp_random(p + 1, K, N, p, -20, 20))
    ref = oz.Plan.create(p, K)
    print(f"p={p} digits={ref.nd32} L={ref.L}", flush=True)
    plan = oz.Plan.create(p, K, oz.default_opts(flags=oz.FLAG_CRT_MMA))
    R = oz.gemm(ref, A, B)
    assert _same(oz.gemm(plan, A, B), R)
    x, y = oz.gemm_integers(plan, A, B), oz.gemm_integers(ref, A, B)
    assert all((a == b).all() for a, b in zip(x, y))
    ref.set_flags(oz.FLAG_CRT_MMA)
    assert _same(oz.gemm(ref, A, B), R)
    plan.set_flags(0)
    assert _same(oz.gemm(plan, A, B), R)


def test_extreme_integers(oz):
    """The least CRT margin with operands of all-ones significands: |c^| up to K (2^t - 1)^2."""
    from tests.test_gpu_crt_paths import _extreme_operands
    for p, K in ((1024, 64), (700, 256)):
        A, B = (dev_mp(X) for X in _extreme_operands(70, 50, K, p))
        R = oz.gemm(oz.Plan.create(p, K, oz.default_opts(crt_margin=1)), A, B)
        print(f"extreme p={p}", flush=True)
        assert _same(oz.gemm(oz.Plan.create(p, K, oz.default_opts(crt_margin=1, flags=oz.FLAG_CRT_MMA)), A, B), R)
