"""The DMA ring's waits on the CPU: a wave's pieces complete in order and as
late as its waits allow, a piece without lanes is never counted, and every
stage that is read has landed.

The schedules are those of the whole-branch kernels: stages 0 .. 2 requested
and awaited at the start; at stage st the wait for stage st, or one ahead for
st + 1, which lets the pieces of the later ones stay in flight; then the
request of stage st + 3.  The lane masks are csrc/ring.h's, compiled here; with
empty masks past the last stage the model reads a stage that is in flight.
"""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_02963_amd", "csrc")

MODEL = r"""
#include <cstdio>
#include <cstring>
#include <deque>
#include "ring.h"

// the number of reads of a stage that had not landed; stages before switch_at
// wait one ahead
int run(bool empty, int nst, int pps, int switch_at)
{
    std::deque<int> flight;  // one entry per counted piece, its stage
    auto request = [&](int st) {
        const uint64_t lanes = empty && st >= nst ? 0 : pdec::ring_lanes(st, nst);
        if (lanes) flight.insert(flight.end(), pps, st);
    };
    for (int st = 0; nst > 0 && st < 3; ++st) request(st);
    flight.clear();  // the start waits for everything
    int bad = 0;
    for (int st = 0; st < nst; ++st) {
        const int awaited = st < switch_at ? st + 1 : st;
        while ((int)flight.size() > pps * (st + 2 - awaited)) flight.pop_front();
        bad += !flight.empty() && flight.front() <= awaited && flight.front() < nst;
        request(st + 3);
    }
    return bad;
}

int main(int, char** v)
{
    int bad = 0;
    for (int nst = 0; nst <= 12; ++nst)
        for (int pps : {2, 4, 5, 8, 9})
            for (int at = 0; at <= nst; ++at) bad += run(!strcmp(v[1], "empty"), nst, pps, at);
    printf("%d\n", bad);
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_every_stage_that_is_read_has_landed(tmp_path):
    (tmp_path / "m.cpp").write_text(MODEL)
    exe = str(tmp_path / "m")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, str(tmp_path / "m.cpp"), "-o", exe], check=True)
    said = {k: int(subprocess.run([exe, k], check=True, capture_output=True, text=True).stdout) for k in ("ring", "empty")}
    assert said["ring"] == 0
    assert said["empty"] > 0  # the model sees a wait that counts on pieces without lanes
