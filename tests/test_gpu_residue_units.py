"""Residue kernels by units (marked gpu): pairs of one-limb moduli and single two-limb moduli, at
the word counts where a kernel or its arithmetic changes, for one-limb moduli left over, and in a
batch, against the oracle's integers and plain calls."""
import numpy as np
import pytest

import synth
from tests.gpu_util import dev_mp, need_gpu
from tests.test_gpu_stages import check_residue_planes, rng_idx

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oz():
    need_gpu()
    from paper_2609_27831_amd import oz2h
    return oz2h


# K = 150: t = p + 24.  12 / 13 words: registers / LDS; 16 / 17: a pair's sum beyond 2^51; 23 / 24:
# entry kernel / rows; 32 n - 1 bits: one signed digit more than words
@pytest.mark.parametrize("p", [32 * w - 25 for w in (12, 13, 16, 17, 23, 24, 33)] + [711, 712, 1000])
@pytest.mark.parametrize("side", ["A", "B"])
def test_planes_at_word_counts(oz, c_oracle, p, side):
    R, C = (70, 150) if side == "A" else (150, 70)
    plan = oz.Plan.create(p, 150)
    assert plan.nw32 == (p + 24 + 32) // 32
    X = synth.mp_random(5 + p, R, C, p, -40, 40)
    X.sign[rng_idx(R, C, 0.05, p)] = 0
    check_residue_planes(oz, c_oracle, plan, X, side, 150, f"p={p} side={side} words={plan.nw32}")


# (one-limb moduli taken, two-limb moduli taken, p): lone moduli, the even one alone and in a
# pair, partial and full groups of either kind, one kind only
@pytest.mark.parametrize("n1,n2,p", [(1, 30, 113), (7, 4, 53), (8, 5, 53), (9, 27, 113), (54, 0, 64), (3, 100, 600),
                                     (0, 40, 200), (5, 130, 800)])
def test_planes_of_custom_sets(oz, c_oracle, n1, n2, p):
    all_ = oz.Plan.create(1500, 150).moduli.tolist()
    one = [128] + [m for m in all_ if m <= 255 and m != 128]
    mods = one[:n1] + [m for m in all_ if m > 255][:n2]
    room = (sum(np.log2(m) for m in mods) - 1 - 8) / 2
    t = min(p + 24, int(room) - 1)
    plan = oz.Plan.custom(p, t, 150, mods)
    X = synth.mp_random(77 + n1, 70, 150, p, -20, 20)
    X.sign[rng_idx(70, 150, 0.05, n1 + n2)] = 0
    check_residue_planes(oz, c_oracle, plan, X, "A", 150, f"{n1} + {n2} moduli p={p} t={t}")


# the unit groups shared by two blocks (500 rows) and by none (2000) against four (few rows)
@pytest.mark.parametrize("rows", [500, 2000])
@pytest.mark.parametrize("p", [8, 53, 113, 256, 400, 620])
def test_shared_groups(oz, rows, p):
    import torch
    K = 300
    A, B = synth.mp_random(rows + p, rows, K, p, -20, 20), synth.mp_random(p, K, 40, p, -20, 20)
    plan, dB = oz.Plan.create(p, K), dev_mp(B)
    print(f"{rows} rows p={p}", flush=True)
    C = oz.gemm(plan, dev_mp(A), dB)
    for r0 in (0, rows - 9):
        part = synth.mp_zeros(9, K, p)
        part.sign[:], part.exp[:], part.limbs[:] = (getattr(A, n)[r0:r0 + 9] for n in ("sign", "exp", "limbs"))
        R = oz.gemm(plan, dev_mp(part), dB)
        for n in ("sign", "exp", "limbs"):
            assert torch.equal(getattr(C, n)[r0:r0 + 9], getattr(R, n)), n


def test_batch_of_every_residue_class(oz):
    import torch
    probs = []
    for i, p in enumerate([30, 53, 300, 360, 420, 700, 760, 1100, 2048]):
        M, N, K = 40 + 30 * i, 150 - 9 * i, 130 + 17 * i
        A, B = dev_mp(synth.mp_random(60 + i, M, K, p, -6, 6)), dev_mp(synth.mp_random(80 + i, K, N, p, -6, 6))
        probs.append((A, B, oz.empty_mp(M, N, p), 0, 0))
    bp = oz.BatchedPlan(probs)
    ws = bp.workspace()
    print("batch over the residue classes", flush=True)
    for _ in range(2):
        bp.run(ws)
        torch.cuda.synchronize()
        for A, B, C, _, _ in probs:
            P = oz.gemm(oz.Plan.create(A.p, A.shape[1]), A, B)
            assert all(torch.equal(a, b) for a, b in ((P.sign, C.sign), (P.exp, C.exp), (P.limbs, C.limbs))), A.p
