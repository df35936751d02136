"""The four- and eight-wave residue GEMM tiles (marked gpu): both depths of the k-loop with even
and odd counts of 128-byte k-tiles, one and three products per modulus, thin tiles, against int64
products and against the same calls on another fixed tile, bit for bit."""
import math

import numpy as np
import pytest

import synth
from tests.gpu_util import dev_mp, need_gpu
from tests.test_gpu_gemm256 import _planes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oz():
    need_gpu()
    from paper_2609_27831_amd import oz2h
    return oz2h


# few blocks and kpad >= 512: four stages; otherwise two
@pytest.mark.parametrize("p,mpad,npad,kpad,tile", [(53, 128, 128, 128, 1), (53, 128, 128, 512, 1), (256, 128, 128, 640, 1),
                                                   (256, 256, 256, 640, 1), (53, 256, 128, 640, 2), (256, 512, 384, 384, 2),
                                                   (53, 128, 256, 768, 3), (600, 128, 128, 128, 1), (600, 128, 128, 896, 1)])
def test_stage_mod_m(oz, p, mpad, npad, kpad, tile):
    import torch
    plan = oz.Plan.create(p, kpad, oz.default_opts(tile=tile))
    rng = np.random.default_rng(p + kpad)
    A, B = _planes(rng, plan, mpad, kpad), _planes(rng, plan, npad, kpad)
    print(f"residue gemm p={p} {mpad}x{npad}x{kpad} tile {tile}", flush=True)
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


@pytest.mark.parametrize("M,N,K,tile", [(128, 128, 128, 1)] + [(*s, t) for t in (1, 2, 3) for s in (
    (256, 256, 640), (2304, 2048, 384), (256, 768, 1024))])
def test_i8gemm(oz, M, N, K, tile):
    import torch
    g = torch.Generator(device="cuda").manual_seed(M + K)
    A, B = (torch.randint(-127, 128, (r, K), dtype=torch.int8, device="cuda", generator=g) for r in (M, N))
    print(f"i8gemm {M}x{N}x{K} tile {tile}", flush=True)
    C = oz.i8gemm(A, B, tile)
    ref = A.cpu().double().numpy() @ B.cpu().double().numpy().T   # exact: below 2^53
    assert np.array_equal(C.cpu().numpy(), ref.astype(np.int32))


# up to 64 rows or columns take 64-wide tiles; one more does not
@pytest.mark.parametrize("M,N,K", [(300, 1, 130), (256, 64, 700), (257, 65, 130), (1, 300, 700), (64, 256, 130), (33, 900, 1100)])
@pytest.mark.parametrize("p,flags", [(113, 0), (600, 0), (1024, 0), (300, 3)])
def test_thin_products_against_square_tiles(oz, M, N, K, p, flags):
    import torch
    A, B = dev_mp(synth.mp_random(M, M, K, p, -9, 9)), dev_mp(synth.mp_random(N, K, N, p, -9, 9))
    print(f"thin {M}x{N}x{K} p={p} flags={flags}", flush=True)
    C = oz.gemm(oz.Plan.create(p, K, oz.default_opts(flags=flags)), A, B)
    D = oz.gemm(oz.Plan.create(p, K, oz.default_opts(flags=flags, tile=oz.TILE_128x128)), A, B)
    assert all(torch.equal(a, b) for a, b in ((C.sign, D.sign), (C.exp, D.exp), (C.limbs, D.limbs)))


@pytest.mark.parametrize("scheme", [3, 4])
def test_complex_depths(oz, scheme):
    import torch
    M, N, K, p = 100, 90, 600, 53
    X = [dev_mp(synth.mp_random(20 + i, *s, p, -5, 5)) for i, s in enumerate([(M, K), (M, K), (K, N), (K, N)])]
    print(f"complex scheme {scheme}", flush=True)
    R = [oz.zgemm(oz.Plan.create(p, 2 * K, oz.default_opts(tile=t)), *X, scheme=scheme) for t in (0, 2, 3)]
    for other in R[1:]:
        for a, b in zip(R[0], other):
            assert torch.equal(a.sign, b.sign) and torch.equal(a.exp, b.exp) and torch.equal(a.limbs, b.limbs)


def test_batch_of_every_gemm_class(oz):
    """Products with 256 x 256 tiles (their own launches), ordinary and thin ones in one batch,
    and the same batch with every product in the grouped launch, against plain calls."""
    import torch
    probs = []
    for i, (M, N, K, p) in enumerate([(1024, 1000, 1100, 256), (130, 140, 150, 53), (20, 700, 90, 113), (1500, 1530, 250, 113),
                                      (300, 300, 1025, 400), (770, 1020, 500, 512)]):
        A, B = dev_mp(synth.mp_random(60 + i, M, K, p, -6, 6)), dev_mp(synth.mp_random(80 + i, K, N, p, -6, 6))
        probs.append((A, B, oz.empty_mp(M, N, p), 0, 0))
    bp = oz.BatchedPlan(probs)
    ws = bp.workspace()
    refs = [oz.gemm(oz.Plan.create(A.p, A.shape[1]), A, B) for A, B, _, _, _ in probs]
    for tile in (oz.TILE_AUTO, oz.TILE_256x128, oz.TILE_AUTO):
        bp.set_config(tile, 0)
        print(f"batch over the GEMM classes, tile {tile}", flush=True)
        for _ in range(2):
            for _, _, C, _, _ in probs:
                C.limbs.zero_()
            bp.run(ws)
            torch.cuda.synchronize()
            for (_, _, C, _, _), R in zip(probs, refs):
                assert torch.equal(R.sign, C.sign) and torch.equal(R.exp, C.exp) and torch.equal(R.limbs, C.limbs)


@pytest.mark.parametrize("M,N,K,p", [(300, 9, 700, 113), (9, 300, 700, 113), (300, 64, 130, 1024), (70, 260, 1100, 256)])
def test_thin_products_from_handles_and_without_a_workspace(oz, M, N, K, p):
    A, B = dev_mp(synth.mp_random(M, M, K, p, -9, 9)), dev_mp(synth.mp_random(N, K, N, p, -9, 9))
    plan = oz.Plan.create(p, K)
    print(f"handles {M}x{N}x{K} p={p}", flush=True)
    R = oz.gemm(oz.Plan.create(p, K, oz.default_opts(tile=oz.TILE_256x128)), A, B)
    ra, rb = oz.Residues(plan, A, oz.SIDE_A), oz.Residues(plan, B, oz.SIDE_B)
    out = oz.empty_mp(M, N, p)
    for C in (oz.gemm_from_residues(plan, B=B, ra=ra), oz.gemm_from_residues(plan, A=A, rb=rb),
              oz.gemm_from_residues(plan, ra=ra, rb=rb), oz.gemm_noalloc(plan, A, B, out=out)):
        assert (C.sign == R.sign).all() and (C.exp == R.exp).all() and (C.limbs == R.limbs).all()


# on both sides of the rule for 64-wide tiles: blocks of 256 rows (80, or 300 where they pad by more than a sixth)
@pytest.mark.parametrize("large,p", [(256, 256), (256, 384), (300, 384), (385, 384), (600, 384), (384, 1024), (385, 113)])
def test_thin_rule(oz, large, p):
    import torch
    K, n = 520, 17
    A, B = dev_mp(synth.mp_random(large, large, K, p, -9, 9)), dev_mp(synth.mp_random(p, K, n, p, -9, 9))
    print(f"thin rule {large} x {n} x {K}, p = {p}", flush=True)
    auto, square = oz.Plan.create(p, K), oz.Plan.create(p, K, oz.default_opts(tile=oz.TILE_128x128))
    for X, Y, ops in ((A, B, (0, 0)), (B, A, (1, 1))):
        C, D = oz.gemm(auto, X, Y, *ops), oz.gemm(square, X, Y, *ops)
        assert all(torch.equal(a, b) for a, b in ((C.sign, D.sign), (C.exp, D.exp), (C.limbs, D.limbs)))


# one to four k-tiles (three stages), and both sides of the rule for long products of few blocks
@pytest.mark.parametrize("M,N,K", [(256, 256, 128), (256, 256, 256), (256, 512, 384), (256, 256, 512), (256, 256, 1920),
                                   (256, 256, 2048), (512, 768, 2176), (4352, 4096, 2048)])
@pytest.mark.parametrize("tile", [1, 2, 3])
def test_i8gemm_rule(oz, M, N, K, tile):
    test_i8gemm(oz, M, N, K, tile)


# tiles that do not divide among the XCDs: four stages from 2048 on, or from 1024 with more than 768 blocks
@pytest.mark.parametrize("M,N,K,p", [(600, 580, 1000, 113), (600, 580, 1030, 113), (300, 290, 1030, 113), (300, 290, 2000, 113),
                                     (300, 290, 2170, 53), (610, 824, 2048, 53)])
def test_depth_rule(oz, M, N, K, p):
    import torch
    A, B = dev_mp(synth.mp_random(M, M, K, p, -9, 9)), dev_mp(synth.mp_random(N, K, N, p, -9, 9))
    print(f"depth {M} x {N} x {K}, p = {p}", flush=True)
    C, D = (oz.gemm(oz.Plan.create(p, K, oz.default_opts(tile=t)), A, B) for t in (oz.TILE_AUTO, oz.TILE_256x128))
    assert all(torch.equal(a, b) for a, b in ((C.sign, D.sign), (C.exp, D.exp), (C.limbs, D.limbs)))
