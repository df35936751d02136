"""The 256 x 256 residue GEMM (marked gpu): its stage output against int64 products, the int32
limit, and whole products (plain, from handles, complex, backward, without a workspace) against
the same calls on plans fixed to 128 x 128 tiles, bit for bit."""
import math

import numpy as np
import pytest

import synth
from tests.gpu_util import dev_mp, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oz():
    need_gpu()
    from paper_2609_27831_amd import oz2h
    return oz2h


def _planes(rng, plan, rows, kpad):
    X = np.zeros((plan.G, rows, kpad), np.int8)
    for li, m in enumerate(plan.moduli.tolist()):
        g0 = li if li < plan.L1 else plan.L1 + 3 * (li - plan.L1)
        r = rng.integers(-(m // 2), (m - 1) // 2 + 1, (rows, kpad))
        if m <= 255:
            X[g0] = r
        else:
            r0 = ((r + 64) & 127) - 64
            r1 = (r - r0) // 128
            X[g0], X[g0 + 1], X[g0 + 2] = r0, r1, r0 + r1
    return X


# one modulus tile (fewer items than blocks x 2), no even split over the XCDs, an even one,
# the shortest k-loop, products of several k-tile pairs
@pytest.mark.parametrize("p,mpad,npad,kpad", [(2048, 256, 256, 256), (256, 256, 1280, 512),
                                              (256, 768, 512, 768), (53, 1024, 1024, 256)])
def test_stage_mod_m(oz, p, mpad, npad, kpad):
    import torch
    plan = oz.Plan.create(p, 320)
    assert plan.L * (mpad // 256) * (npad // 256) >= 320   # the 256 x 256 kernel's range
    rng = np.random.default_rng(p + kpad)
    A, B = _planes(rng, plan, mpad, kpad), _planes(rng, plan, npad, kpad)
    print(f"residue gemm p={p} {mpad}x{npad}x{kpad}", flush=True)
    v = oz.residue_gemm(plan, torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda())
    v = v.cpu().numpy().astype(np.int64)
    P = math.prod(plan.moduli.tolist())
    for li, m in enumerate(plan.moduli.tolist()):
        g0 = li if li < plan.L1 else plan.L1 + 3 * (li - plan.L1)
        a, b = A[g0].astype(np.float64), B[g0].astype(np.float64)
        if m > 255:
            a = a + 128.0 * A[g0 + 1]
            b = b + 128.0 * B[g0 + 1]
        prod = (a @ b.T).astype(np.int64)   # exact: below 2^53
        minv = pow((P // m) % m, -1, m)
        assert np.abs(v[li]).max() <= m // 2, f"modulus {m}: not centred"
        assert np.array_equal(np.mod(v[li], m), np.mod(np.mod(prod, m) * minv, m)), f"modulus {m}"


def test_int32_limit(oz):
    """kpad = 133120 (the largest a K of 133000 pads to): sums of +-K 127^2 beside a folded
    residue still fit int32; v follows analytically."""
    import torch
    kpad = 133120
    plan = oz.Plan.custom(53, 8, 133000, [251, 16189, 16187])
    ms = plan.moduli.tolist()
    P = math.prod(ms)
    mpad, npad = 1024, 6912
    assert plan.L * (mpad // 256) * (npad // 256) >= 320
    sa = [127, -127, 127, 127, -127, -127, 127]
    sb = [-127, -127, 127, 127, 127, -127, -127]
    a = torch.empty((plan.G, mpad, kpad), dtype=torch.int8, device="cuda")
    b = torch.empty((plan.G, npad, kpad), dtype=torch.int8, device="cuda")
    for g in range(plan.G):
        a[g].fill_(sa[g])
        b[g].fill_(sb[g])
    print("residue gemm at kpad 133120", flush=True)
    u = oz.residue_gemm(plan, a, b)
    for li, m in enumerate(ms):
        minv = pow((P // m) % m, -1, m)
        if m <= 255:
            c = kpad * sa[li] * sb[li]
        else:
            g0 = 1 + 3 * (li - 1)
            P0, P2, Ps = (kpad * sa[g0 + i] * sb[g0 + i] for i in range(3))
            c = -127 * P0 + 16256 * P2 + 128 * Ps
        want = (c * minv + m // 2) % m - m // 2
        assert int(u[li].min()) == int(u[li].max()) == want, f"modulus {m}"


def _same(X, Y):
    import torch
    return all(torch.equal(a, b) for a, b in ((X.sign, Y.sign), (X.exp, Y.exp), (X.limbs, Y.limbs)))


# ragged sizes, a K whose padding goes to 256, transposed operands, both residue kernels
@pytest.mark.parametrize("M,N,K,p,opA,opB", [(1000, 760, 1100, 128, 0, 0), (512, 1023, 257, 512, 1, 0),
                                             (300, 256, 200, 1100, 0, 1), (897, 1025, 2500, 53, 1, 1)])
def test_products_match_small_tiles(oz, M, N, K, p, opA, opB):
    A = dev_mp(synth.mp_random(31, *((K, M) if opA else (M, K)), p, -9, 9))
    B = dev_mp(synth.mp_random(32, *((N, K) if opB else (K, N)), p, -9, 9))
    print(f"{M}x{N}x{K} p={p}", flush=True)
    ref = oz.gemm(oz.Plan.create(p, K, oz.default_opts(tile=oz.TILE_128x128)), A, B, opA, opB)
    plan = oz.Plan.create(p, K)
    assert _same(oz.gemm(plan, A, B, opA, opB), ref)
    ra = oz.Residues(plan, A, oz.SIDE_A, opA)
    assert _same(oz.gemm_from_residues(plan, B=B, ra=ra, opB=opB), ref)


@pytest.mark.parametrize("M,N,K,p", [(768, 1024, 600, 113), (1024, 500, 1200, 256)])
def test_complex_matches_small_tiles(oz, M, N, K, p):
    X = [dev_mp(synth.mp_random(40 + i, *s, p, -5, 5)) for i, s in enumerate([(M, K)] * 2 + [(K, N)] * 2)]
    small = oz.Plan.create(p, 2 * K, oz.default_opts(tile=oz.TILE_128x128))
    ref = oz.zgemm(small, *X, scheme=oz.ZGEMM_4M)
    for scheme in (oz.ZGEMM_3M, oz.ZGEMM_4M):
        print(f"complex {M}x{N}x{K} p={p} scheme={scheme}", flush=True)
        got = oz.zgemm(oz.Plan.create(p, 2 * K), *X, scheme=scheme)
        assert _same(got[0], ref[0]) and _same(got[1], ref[1]), scheme


def test_backward_matches_small_tiles(oz):
    M, N, K, p = 900, 1030, 1300, 128
    A, B, W = (dev_mp(synth.mp_random(50 + i, *s, p, -5, 5)) for i, s in enumerate([(M, K), (K, N), (M, N)]))
    out = []
    for tile in (oz.TILE_128x128, oz.TILE_AUTO):
        plan = oz.Plan.create_grad(p, M, N, K, oz.default_opts(tile=tile))
        ws = oz.workspace(plan, M, N)
        print(f"backward tile={tile}", flush=True)
        out.append((oz.gemm(plan, A, B, ws=ws), *oz.gemm_backward(plan, ws, W)))
    assert all(_same(x, y) for x, y in zip(*out))


def test_noalloc_near_its_limit(oz):
    """A product that fits the static scratch only with the least padding stays accepted."""
    M, N, K, p = 256, 128, 1100, 640
    plan = oz.Plan.create(p, K)
    cap = oz.lib().oz2h_gemm_noalloc_max_bytes()
    least = plan.G * (M + N) * 1152 + 2 * plan.L * M * N + 2048
    assert least < cap < plan.workspace_size(M, N)
    A, B = dev_mp(synth.mp_random(60, M, K, p, -5, 5)), dev_mp(synth.mp_random(61, K, N, p, -5, 5))
    print("noalloc near the limit", flush=True)
    assert _same(oz.gemm_noalloc(plan, A, B, out=oz.empty_mp(M, N, p)), oz.gemm(plan, A, B))


# padding by a third more for a product that nearly fills 128 x 128 tiles and one that does not, and by less
@pytest.mark.parametrize("M,N", [(384, 500), (256, 300), (500, 1100), (512, 600)])
def test_padding_rule(oz, M, N):
    K, p = 1100, 512
    A, B = dev_mp(synth.mp_random(90, M, K, p, -5, 5)), dev_mp(synth.mp_random(91, K, N, p, -5, 5))
    print(f"padding {M} x {N}", flush=True)
    C = oz.gemm(oz.Plan.create(p, K), A, B)
    assert _same(C, oz.gemm(oz.Plan.create(p, K, oz.default_opts(tile=oz.TILE_256x128)), A, B))
