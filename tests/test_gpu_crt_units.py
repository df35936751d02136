"""CRT by units (marked gpu): digit counts where the kernel changes, moduli left without a partner,
one and two columns per thread with odd widths, integers next to P / 2 on a set found for that,
and batches, against the oracle, exact integers and plain calls."""
import math

import numpy as np
import pytest

import synth
from tests.gpu_util import dev_mp, mp_to_ints, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oz():
    need_gpu()
    from paper_2609_27831_amd import oz2h
    return oz2h


def _check(oz, c_oracle, plan, A, B, tag):
    print(tag, flush=True)
    ref = c_oracle.gemm(A, B)
    C = oz.gemm(plan, dev_mp(A), dev_mp(B))
    assert np.array_equal(C.sign.cpu().numpy(), ref["c_sign"]), tag
    assert np.array_equal(C.exp.cpu().numpy(), ref["c_exp"]), tag
    assert np.array_equal(C.limbs.cpu().numpy().view(np.uint64), ref["c_limbs"]), tag


# plans from 4 to 54 digits: every kernel of the unit CRT, and the row CRT from 49 on
@pytest.mark.parametrize("p", [2, 24, 53] + [16 * w + 5 for w in range(3, 52, 2)])
def test_products_at_digit_counts(oz, c_oracle, p):
    A, B = synth.mp_random(p, 33, 40, p, -30, 30), synth.mp_random(p + 1, 40, 29, p, -30, 30)
    _check(oz, c_oracle, oz.Plan.create(p, 40), A, B, f"p={p}")


# one-limb and two-limb moduli taken: an odd one over, one kind only, a single unit
@pytest.mark.parametrize("n1,n2,p", [(1, 30, 113), (7, 4, 30), (8, 5, 40), (9, 27, 113), (53, 0, 64), (0, 40, 200),
                                     (3, 1, 4), (2, 100, 600)])
def test_products_of_custom_sets(oz, n1, n2, p):
    all_ = oz.Plan.create(1500, 150).moduli.tolist()
    one = [m for m in all_ if m <= 255]
    mods = one[:n1] + [m for m in all_ if m > 255][:n2]
    t = min(p + 24, int((sum(np.log2(m) for m in mods) - 1 - 6) / 2) - 1)
    plan, full = oz.Plan.custom(p, t, 50, mods), oz.Plan.create(1500, 50)
    A, B = synth.mp_random(n1, 40, 50, p, 0, 0), synth.mp_random(n2, 50, 31, p, 0, 0)
    print(f"{n1} + {n2} moduli, p={p}, t={t}", flush=True)
    cs, cm, e, f = oz.gemm_integers(plan, dev_mp(A), dev_mp(B))
    a = np.array(mp_to_ints(A.sign, A.limbs), dtype=object).reshape(40, 50)
    b = np.array(mp_to_ints(B.sign, B.limbs), dtype=object).reshape(50, 31)
    trunc = lambda x, s: int(math.copysign(1, x)) * (abs(x) << s if s >= 0 else abs(x) >> -s)
    assert full.L > plan.L
    # exponents are equal within rows and columns, so every significand scales by 2^(t - p)
    a, b = (np.vectorize(lambda x: trunc(x, t - p), otypes=[object])(x) for x in (a, b))
    got = oz.limbs_to_ints(cm.cpu().numpy().view(np.uint64), cs.cpu().numpy())
    assert list(got) == list(np.dot(a, b).ravel())


def _tight_set(moduli, t_min, gap):
    """Moduli whose product exceeds a power of two 2^(2t + 1) by a factor below 1 + gap: subset
    products of two halves of a list, matched on the fraction of their logarithm."""
    base, pool = moduli[:8], moduli[8:44]
    lg = np.log2(np.array(pool, float))

    def sums(x):
        s = np.zeros(1)
        for v in x:
            s = np.concatenate([s, s + v])
        return s
    lo, hi = sums(lg[:18]) + np.log2(np.array(base, float)).sum(), sums(lg[18:])
    flo, order = lo % 1.0, np.argsort(hi % 1.0)
    fhi = (hi % 1.0)[order]
    pos = np.searchsorted(fhi, (1.0 - flo) % 1.0)   # the least fraction that carries the sum over
    for i in np.argsort(np.where(pos < len(fhi), (flo + fhi[np.minimum(pos, len(fhi) - 1)]) % 1.0, 1.0))[:64]:
        j = int(order[pos[i]])
        ms = base + [m for k, m in enumerate(pool[:18]) if i >> k & 1] + [m for k, m in enumerate(pool[18:]) if j >> k & 1]
        P = math.prod(ms)
        n = P.bit_length() - 1
        if n % 2 == 1 and (P - (1 << n)) / (1 << n) < gap and n // 2 >= t_min:
            return ms, n // 2
    raise AssertionError("no set")


@pytest.mark.parametrize("K", [1, 4])
def test_integers_next_to_half_P(oz, K):
    """|c^| = (K / K') (2^t - 1)^2, K' = K as a power of two, on P within 2^-33 of 2 K 2^(2t):
    quotients within 2^-30 of a half-integer, which take the paper's sequence."""
    all_ = oz.Plan.create(800, 64).moduli.tolist()
    one, two = [m for m in all_ if m <= 255], [m for m in all_ if m > 255]
    ms, t = _tight_set(one[:6] + two[:2] + [m for q in zip(one[6:24], two[2:20]) for m in q], 60, 2.0 ** -33)
    t -= (K.bit_length() - 1) // 2
    P = math.prod(ms)
    plan = oz.Plan.custom(t, t, K, ms)
    M, N = 37, 23
    A, B = synth.mp_zeros(M, K, t), synth.mp_zeros(K, N, t)
    rng = np.random.default_rng(3)
    for X in (A, B):
        X.sign[:] = np.where(rng.random(X.sign.shape) < 0.5, 1, -1)
        full = (1 << t) - 1
        for l in range(X.limbs.shape[-1]):
            X.limbs[..., l] = np.uint64((full >> (64 * l)) & ((1 << 64) - 1))
    A.sign[:9], B.sign[:, :9] = 1, 1
    print(f"next to P/2: L={plan.L} t={t} K={K}", flush=True)
    cs, cm, _, _ = oz.gemm_integers(plan, dev_mp(A), dev_mp(B))
    got = oz.limbs_to_ints(cm.cpu().numpy().view(np.uint64), cs.cpu().numpy())
    ref = (A.sign.astype(object) @ B.sign.astype(object) * ((1 << t) - 1) ** 2).ravel()
    assert list(got) == list(ref)
    assert (P // 2 - max(ref)) / P < 2.0 ** -31


# more than 2^18 entries: two columns per thread up to 26 digits; odd widths leave a column over;
# 33 to 48 digits: the unit kernel from 2^17 entries on, against the row kernels for few
@pytest.mark.parametrize("p,M,N", [(30, 513, 513), (150, 300, 875), (330, 515, 513), (460, 363, 363), (520, 512, 257),
                                   (590, 363, 364), (660, 400, 331)])
def test_two_columns_per_thread(oz, p, M, N):
    import torch
    K = 20
    A, B = synth.mp_random(p, M, K, p, -20, 20), synth.mp_random(p + 1, K, N, p, -20, 20)
    plan, dB = oz.Plan.create(p, K), dev_mp(B)
    print(f"{M}x{N} p={p}", flush=True)
    C = oz.gemm(plan, dev_mp(A), dB)
    for r0 in (0, M - 9):
        rows = synth.mp_zeros(9, K, p)
        rows.sign[:], rows.exp[:], rows.limbs[:] = (getattr(A, n)[r0:r0 + 9] for n in ("sign", "exp", "limbs"))
        R = oz.gemm(plan, dev_mp(rows), dB)
        for n in ("sign", "exp", "limbs"):
            assert torch.equal(getattr(C, n)[r0:r0 + 9], getattr(R, n)), (p, n, r0)


def test_batch_of_every_digit_class(oz):
    import torch
    probs = []
    for i, p in enumerate([2, 30, 80, 113, 150, 200, 256, 300, 350, 400, 450, 500, 620, 700, 900, 1000, 1100]):
        M, N, K = 30 + 17 * i, 140 - 7 * i, 20 + i
        A, B = dev_mp(synth.mp_random(60 + i, M, K, p, -6, 6)), dev_mp(synth.mp_random(80 + i, K, N, p, -6, 6))
        probs.append((A, B, oz.empty_mp(M, N, p), 0, 0))
    bp = oz.BatchedPlan(probs)
    ws = bp.workspace()
    print("batch over the digit classes", flush=True)
    for _ in range(2):
        bp.run(ws)
        torch.cuda.synchronize()
        for A, B, C, _, _ in probs:
            P = oz.gemm(oz.Plan.create(A.p, A.shape[1]), A, B)
            assert all(torch.equal(a, b) for a, b in ((P.sign, C.sign), (P.exp, C.exp), (P.limbs, C.limbs))), A.p


# the row kernels beyond 48 digits: pairs in one chunk of 16 units and in two, an odd modulus over,
# none, the bound on pairs (many moduli), through the stage call and products
@pytest.mark.parametrize("n1,n2,p", [(0, 110, 700), (5, 105, 700), (32, 100, 700), (33, 99, 700), (53, 96, 700), (53, 400, 2700)])
def test_row_kernels_of_custom_sets(oz, c_oracle, n1, n2, p):
    all_ = oz.Plan.create(2800, 20).moduli.tolist()
    one, two = [m for m in all_ if m <= 255], [m for m in all_ if m > 255]
    mods = one[:n1] + two[:n2]
    t = min(p + 24, int((sum(np.log2(m) for m in mods) - 1 - 6) / 2) - 1)
    plan = oz.Plan.custom(p, t, 20, mods)
    A, B = synth.mp_random(n1, 21, 20, p, 0, 0), synth.mp_random(n2, 20, 19, p, 0, 0)
    print(f"{n1} + {n2} moduli, p={p}, t={t}, digits={plan.nd32}", flush=True)
    assert plan.nd32 > 48
    cs, cm, _, _ = oz.gemm_integers(plan, dev_mp(A), dev_mp(B))
    a = np.array(mp_to_ints(A.sign, A.limbs), dtype=object).reshape(21, 20)
    b = np.array(mp_to_ints(B.sign, B.limbs), dtype=object).reshape(20, 19)
    sh = lambda x: (1 if x > 0 else -1) * (abs(x) << t - p if t >= p else abs(x) >> p - t)
    a, b = (np.vectorize(sh, otypes=[object])(x) for x in (a, b))
    assert list(oz.limbs_to_ints(cm.cpu().numpy().view(np.uint64), cs.cpu().numpy())) == list(np.dot(a, b).ravel())


# limbs stored together or by each entry: the rule's limbs and entries
@pytest.mark.parametrize("M,N,p", [(512, 512, 1856), (512, 512, 1857), (512, 511, 1856), (513, 513, 1030)])
def test_row_finish_stores(oz, M, N, p):
    """Rows of a product of many entries against the same rows on their own."""
    K = 3
    A, B = dev_mp(synth.mp_random(p, M, K, p, -3, 3)), dev_mp(synth.mp_random(p + 1, K, N, p, -3, 3))
    print(f"row finish {M} x {N}, p = {p}", flush=True)
    plan = oz.Plan.create(p, K)
    C = oz.gemm(plan, A, B)
    for r in (0, 77, M - 1):
        X = oz.DeviceMP(A.sign[r:r + 1], A.exp[r:r + 1], A.limbs[r:r + 1], p)
        D = oz.gemm(plan, X, B)
        assert (C.sign[r] == D.sign[0]).all() and (C.exp[r] == D.exp[0]).all() and (C.limbs[r] == D.limbs[0]).all()
