"""The schedule of the 256 x 256 residue GEMM, replayed on the CPU.

The kernel includes oz2h_gemm8_schedule.inc; the program below includes the same text with
operations that record loads, stores, waits, LDS reads and barriers, once per wave group, and
then checks, interval by interval between barriers:
  - a part of LDS is read only after every wave group has waited for its own loads of it in an
    earlier interval (waits count operations in order, the newest n may be outstanding), and
    holds the k-tile the product needs;
  - a part is loaded again only in a later interval than its last read by either group;
  - reads are waited for before the next barrier, and both groups meet the same barriers.
"""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_27831_amd", "csrc")

SOURCE = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <type_traits>
#include <vector>
#define OZ2H_INL

struct v4i {};
struct Part { int s, p; };
template <int S, int P> Part gemm8_part() { return Part{S, P}; }

struct Load { int s, p; long t; int interval, landed; long last; };   // last: number of its last operation
struct Read { int s, p; long t; int interval; };
struct Log {
    std::vector<Load> loads;
    std::vector<Read> reads;
    int interval = 0;
    long ops = 0;
    bool pending = false;   // reads not yet waited for
    bool bad = false;
};

Log run_group(int wr, int nk, const std::vector<int> &items, bool counted) {
    Log g;
    long total = 0;
    for (int n : items) total += (long)n * nk;
    struct { long a, b; int ko; } cur{0, 0, 0};
    long pa = 0;
    int pko = 0;
    long nread[4] = {0, 0, 0, 0};
    size_t item = 0;
    int prod = 0, nprod = items[0];
    v4i fb0[2][2], fb1[2][2], fb2[2][2];
    int acc[2][2];

    auto advance = [&]() {
        pa = cur.a;
        pko = cur.ko;
        cur.a = cur.b = std::min(cur.a + 1, total - 1);
    };
    auto issue = [&](auto s_, auto p_, long t, int) {
        g.ops += 2;
        g.loads.push_back(Load{decltype(s_)::value, decltype(p_)::value, t, g.interval, -1, g.ops});
    };
    auto read = [&](Part q) {
        const long t = std::min(nread[q.p]++, total - 1);
        g.reads.push_back(Read{q.s, q.p, t, g.interval});
        g.pending = true;
    };
    auto read_a = [&](Part q) { read(q); };
    auto read_b = [&](Part q, v4i (&)[2][2]) { read(q); };
    auto mult = [&](int &, v4i (&)[2][2]) {};
    auto finish = [&](auto) {
        if (prod + 1 == nprod && counted) g.ops += 8;
    };
    auto fence = [&]() {};
    auto barrier = [&]() {
        g.bad = g.bad || g.pending;
        ++g.interval;
    };
    auto wait = [&](int n) {
        for (Load &l : g.loads)
            if (l.landed < 0 && g.ops - l.last >= n) l.landed = g.interval;
    };
    auto half_end = [&](int stores) {
        g.pending = false;
        wait(8 + stores * (counted ? 8 : 0));
        barrier();
    };
    auto wait_vm = [&](auto n_) { wait(decltype(n_)::value); };
    auto next_item = [&]() {
        if (++item >= items.size()) return false;
        nprod = items[item];
        return true;
    };
#include "oz2h_gemm8_schedule.inc"
    (void)pko;
    return g;
}

int main(int argc, char **argv) {
    const int nk = atoi(argv[1]);
    const bool counted = atoi(argv[2]) != 0;
    std::vector<int> items;
    for (int i = 3; i < argc; ++i) items.push_back(atoi(argv[i]));
    const Log g[2] = {run_group(0, nk, items, counted), run_group(1, nk, items, counted)};
    if (g[0].interval != g[1].interval || g[0].bad || g[1].bad) return printf("barriers or LDS waits differ\n"), 1;
    int faults = 0;
    for (int r = 0; r < 2; ++r)
        for (const Read &x : g[r].reads)
            for (int w = 0; w < 2; ++w) {
                bool there = false, torn = false;
                for (const Load &l : g[w].loads) {
                    if (l.s != x.s || l.p != x.p) continue;
                    if (l.t == x.t && l.landed >= 0 && l.landed < x.interval) there = true;
                    // another k-tile's load that has gone out by then, and was not before this one
                    if (l.t > x.t && l.interval <= x.interval) torn = true;
                }
                if (!there || torn) {
                    if (!faults++)
                        printf("group %d reads part %d of k-tile %ld in interval %d: group %d's load %s\n", r, x.p,
                               x.t, x.interval, w, torn ? "of a later k-tile may overwrite it" : "has not been waited for");
                }
            }
    printf("%d unguarded reads\n", faults);
    return faults != 0;
}
"""


@pytest.fixture(scope="module")
def replay(tmp_path_factory):
    d = tmp_path_factory.mktemp("gemm8")
    (d / "replay.cpp").write_text(SOURCE)
    exe = str(d / "replay")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "replay.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("nk", [2, 4, 8])
@pytest.mark.parametrize("counted", [1, 0], ids=["stores-counted", "stores-waited-for"])
@pytest.mark.parametrize("items", [[1], [3], [1] * 5, [3] * 4, [3, 3, 1, 1, 1]], ids=str)
def test_every_read_is_guarded(replay, nk, counted, items):
    r = subprocess.run([replay, str(nk), str(counted), *map(str, items)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
