"""Row-broadcast CRT on planes whose M * ldu is a multiple of 16 but not of 64 (stage call)."""
import os
import random
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_27831_amd", "csrc")

SOURCE = r"""
#include "oz2h_plan.hpp"
#include <cstdio>
int main() {   // every row of every tile of 64 reads 16 of the nent entries a plane holds
    for (int64_t nent = 16; nent <= 16 * 70; nent += 16)
        for (int64_t tile = 0; tile * 64 < nent; ++tile)
            for (int q = 0; q < 4; ++q) {
                const int64_t e = oz2h::crt_row_first(nent, tile, q);
                const bool own = 64 * tile + 16 * q < nent;
                if (e < 0 || e % 16 || e + 16 > nent || (own && e != 64 * tile + 16 * q))
                    return printf("%ld entries, tile %ld, row %d: reads from %ld\n", (long)nent, (long)tile, q, (long)e), 1;
            }
    return 0;
}
"""


def test_rows_read_inside_the_planes(tmp_path):
    (tmp_path / "t.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(tmp_path / "t.cpp"), "-o", str(tmp_path / "t")], check=True)
    r = subprocess.run([str(tmp_path / "t")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,ldu", [(1, 16, 16), (3, 11, 16), (5, 16, 16), (1, 33, 48), (7, 80, 80)])
def test_short_planes(M, N, ldu):
    import torch

    from paper_2609_27831_amd import oz2h as oz
    plan = oz.Plan.create(512, 64)
    assert plan.nd32 > 32
    ms = plan.moduli.tolist()
    P = 1
    for m in ms:
        P *= m
    rng = random.Random(100 * M + ldu)
    want = [rng.randrange(-(P // 3), P // 3) for _ in range(M * N)]
    u = np.zeros((len(ms), M, ldu), np.int16)
    for li, m in enumerate(ms):
        u[li, :, :N] = np.array([v % m for v in want], np.int64).reshape(M, N)
    print(f"row CRT: {M} x {N}, ldu {ldu}", flush=True)
    cs, cm = oz.crt(plan, torch.from_numpy(u).cuda(), M, N, ws="auto")
    assert oz.limbs_to_ints(cm.cpu().numpy(), cs.cpu().numpy()) == want
