"""One workspace for products of several shapes (marked gpu): a workspace of the size that a
product asks for serves every one of no more rows and columns on the same plan, whatever the
plan's flags, with the same results bit for bit."""
import itertools

import pytest

import synth
from tests.gpu_util import dev_mp, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oz():
    need_gpu()
    from paper_2609_27831_amd import oz2h
    return oz2h


def _same(X, Y):
    import torch
    return torch.equal(X.sign, Y.sign) and torch.equal(X.exp, Y.exp) and torch.equal(X.limbs, Y.limbs)


def _ws(n):
    import torch
    return torch.full((n,), 0x5A, dtype=torch.uint8, device="cuda")


def _operands(seed, M, N, K, p):
    return dev_mp(synth.mp_random(seed, M, K, p, -5, 5)), dev_mp(synth.mp_random(seed + 1, K, N, p, -5, 5))


DIMS = [1, 8, 64, 65, 128, 129, 256, 257, 300, 384, 640, 641, 768, 896, 1280, 1281, 2048, 2049]


def _least_of_larger(size):
    """For each (M, N) the smallest size asked for by a product of at least M x N."""
    return {mn: min(n for (a, b), n in size.items() if a >= mn[0] and b >= mn[1]) for mn in size}


@pytest.mark.parametrize("p,K", [(53, 64), (113, 1100), (256, 512)])
def test_every_larger_workspace_is_taken(oz, p, K):
    """Every product of the grid in the smallest workspace that one of at least its size asks for."""
    import torch
    plan = oz.Plan.create(p, K)
    top = max(DIMS)
    A = dev_mp(synth.mp_random(68, top, K, p, -5, 5))
    B = dev_mp(synth.mp_random(69, top, K, p, -5, 5))   # stored transposed: its first rows are N columns
    size = {mn: plan.workspace_size(*mn) for mn in itertools.product(DIMS, DIMS)}
    ws = _ws(max(size.values()))
    least = _least_of_larger(size)
    print(f"grid of products, p = {p}, K = {K}", flush=True)
    for (M, N), n in least.items():
        X = oz.DeviceMP(A.sign[:M], A.exp[:M], A.limbs[:M], p)
        Y = oz.DeviceMP(B.sign[:N], B.exp[:N], B.limbs[:N], p)
        C = oz.gemm(plan, X, Y, opB=oz.OP_T, ws=ws)
        if n < size[M, N]:
            assert _same(oz.gemm(plan, X, Y, opB=oz.OP_T, ws=ws[:n]), C), (M, N)
    plan.set_flags(oz.FLAG_RESIDUES_MMA | oz.FLAG_CRT_MMA)
    assert all(plan.workspace_size(*mn) == n for mn, n in size.items())
    torch.cuda.synchronize()


@pytest.mark.parametrize("p,K", [(113, 1100), (512, 64)])
def test_mixed_size_never_falls(oz, p, K):
    plan = oz.Plan.create(p, K, oz.default_opts(flags=oz.FLAG_BACKEND_MIXED))
    size = {mn: plan.workspace_size(*mn) for mn in itertools.product(DIMS, DIMS)}
    assert _least_of_larger(size) == size


@pytest.mark.parametrize("p,K,large,small", [
    (256, 4096, (384, 128), (300, 64)), (113, 4096, (256, 64), (129, 1)),
    (256, 1024, (1281, 384), (1280, 384)), (256, 1024, (640, 896), (640, 768)),
    (64, 1100, (300, 65), (300, 64)), (512, 128, (390, 256), (390, 128)),
])
def test_smaller_product_in_a_larger_ones_workspace(oz, p, K, large, small):
    M, N = small
    plan = oz.Plan.create(p, K)
    ws = _ws(plan.workspace_size(*large))
    A, B = _operands(70, M, N, K, p)
    print(f"{M} x {N} x {K}, p = {p} in the workspace of {large}", flush=True)
    C = oz.gemm(plan, A, B)
    assert _same(oz.gemm(plan, A, B, ws=ws), C)
    ra = oz.Residues(plan, A, oz.SIDE_A)
    assert _same(oz.gemm_from_residues(plan, B=B, ra=ra, ws=ws), C)
    rb = oz.Residues(plan, B, oz.SIDE_B)
    assert _same(oz.gemm_from_residues(plan, A=A, rb=rb, ws=ws), C)


def test_flags_set_after_the_size_was_asked_for(oz):
    M, N, K, p = 300, 64, 1024, 256
    plan = oz.Plan.create(p, K, oz.default_opts(flags=oz.FLAG_RESIDUES_MMA))
    ws = _ws(plan.workspace_size(M, N))
    A, B = _operands(72, M, N, K, p)
    print("flags after the size call", flush=True)
    C = oz.gemm(plan, A, B, ws=ws)
    for flags in (0, oz.FLAG_CRT_MMA, oz.FLAG_RESIDUES_MMA):
        assert _same(oz.gemm(plan.set_flags(flags), A, B, ws=ws), C)


@pytest.mark.parametrize("scheme", [3, 4])
def test_complex(oz, scheme):
    p, K, large, (M, N) = 128, 1100, (640, 896), (640, 768)
    plan = oz.Plan.create(p, 2 * K)
    ws = _ws(oz.lib().oz2h_zgemm_workspace_size(plan.handle, scheme, *large))
    (Ar, Br), (Ai, Bi) = _operands(74, M, N, K, p), _operands(76, M, N, K, p)
    print(f"complex, scheme {scheme}", flush=True)
    own = oz.zgemm(plan, Ar, Ai, Br, Bi, scheme)
    for X, Y in zip(oz.zgemm(plan, Ar, Ai, Br, Bi, scheme, ws=ws), own):
        assert _same(X, Y)


def test_forward_state_in_a_larger_ones_workspace(oz):
    """A grad plan's own product keeps the layout that the backward reads."""
    M, N, K, p = 640, 768, 1024, 113
    plan = oz.Plan.create_grad(p, M, N, K)
    A, B = _operands(78, M, N, K, p)
    W = dev_mp(synth.mp_random(80, M, N, p, -5, 5))
    print("forward state", flush=True)
    want = oz.gemm_backward(plan, _saved(oz, plan, A, B, plan.workspace_size(M, N)), W)
    got = oz.gemm_backward(plan, _saved(oz, plan, A, B, plan.workspace_size(M, 896)), W)
    assert all(_same(X, Y) for X, Y in zip(got, want))


def _saved(oz, plan, A, B, n):
    ws = _ws(n)
    oz.gemm(plan, A, B, ws=ws)
    return ws


@pytest.mark.parametrize("p,K", [(53, 2000), (113, 1100), (640, 1100), (1024, 64)])
def test_noalloc_limit_is_the_stated_one(oz, p, K):
    """The largest M of a column block of 128 that the header's formula lets through, and one more tile."""
    N, plan = 128, oz.Plan.create(p, K)
    cap = oz.lib().oz2h_gemm_noalloc_max_bytes()
    k = -(-K // 128) * 128

    def bytes_of(m):
        dig = oz.lib().oz2h_crt_workspace_size(plan.handle, m, 256)
        return 2 * plan.L * m * N + max(plan.G * (m + N) * k, dig) + 4 * (m + N)

    m = 128
    while bytes_of(m + 128) + 1280 <= cap:
        m += 128
    assert bytes_of(m) + 1280 <= cap < bytes_of(m + 128), "a case next to the limit is wanted"
    A, B = _operands(82, m, N, K, p)
    print(f"noalloc limit: {m} x {N} x {K}, p = {p}", flush=True)
    assert _same(oz.gemm_noalloc(plan, A, B, out=oz.empty_mp(m, N, p)), oz.gemm(plan, A, B))
    A = dev_mp(synth.mp_random(84, m + 128, K, p, -5, 5))
    with pytest.raises(oz.Oz2hError):
        oz.gemm_noalloc(plan, A, B, out=oz.empty_mp(m + 128, N, p))


@pytest.mark.parametrize("K", [1100, 1300, 2049])
def test_planes_are_padded_for_the_tiles_they_meet(oz, K):
    """Planes of products with 128 x 128 tiles are padded to 128 along the contraction, not to 256."""
    import torch
    M, N, p = 120, 100, 113
    k = -(-K // 128) * 128
    A, B = _operands(86, M, N, K, p)
    print(f"k padding, K = {K}", flush=True)
    C = oz.gemm(oz.Plan.create(p, K), A, B)
    out = oz.empty_mp(M, N, p)
    bp = oz.BatchedPlan([(A, B, out, oz.OP_N, oz.OP_N)])
    info = oz.Plan.create(p, K)
    assert bp.workspace_size() <= info.G * 512 * k + 2 * info.L * 256 * 256 + 4096
    bp.run(bp.workspace())
    torch.cuda.synchronize()
    assert _same(out, C)
    # dA = W B^T contracts over N, dB = A^T W over M, both K here
    grad = oz.Plan.create_grad(p, K, K, 120)
    assert grad.backward_workspace_size() <= grad.G * (k + 128) * k + 2 * grad.L * k * 128 + 8 * k + 4096
