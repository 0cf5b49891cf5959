"""The X stage's LDS ring on the host, for every number of inputs, form and work split: the plan fits its
LDS, takes no more of it than the block needs, gives every wave k-steps to do, and no stage is read before all its transfers have landed or
overwritten before it has been read.

The replay runs the kernel's loop (csrc/xring.h holds its plan and its counts) with each wave's
transfers in a queue that a wait shortens from the front to the count it names: the weakest order the
hardware may take.
"""

import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1801_04834_amd", "csrc")

REPLAY = r"""
#include <cstdio>
#include <set>
#include <utility>
#include <vector>
#include "xring.h"
using namespace cobalt;

static int bad = 0;
#define CHECK(ok, ...) do { if (!(ok)) { if (++bad <= 20) { std::printf(__VA_ARGS__); std::printf("\n"); } } } while (0)

struct Queue { std::vector<int> stage; size_t landed = 0; };   // stages of a wave's transfers, in issue order

static void replay(const char* form, int M, int waves, int n_c, const XRing& q, int steps, int parts, int lds_b, int behind) {
    CHECK(q.nch >= 1 && q.depth >= 2, "%s M=%d waves=%d: ring of %d stages of %d chunks", form, M, waves, q.depth, q.nch);
    CHECK((long)q.depth * q.nch * q.chunk_b + behind <= lds_b, "%s M=%d waves=%d: ring past its LDS", form, M, waves);
    CHECK(q.nch * steps % parts == 0, "%s M=%d waves=%d: %d k-steps per stage for %d waves", form, M, waves, q.nch * steps, parts);
    CHECK(q.chunk_b == (M + 3) / 4 * 4 * kRowB && q.ipw * waves >= q.nch * q.n_inst, "%s M=%d waves=%d: transfers", form, M, waves);
    if (q.nch < 1 || q.depth < 1) return;
    const int n_stage = q.n_stage;
    CHECK(n_stage == (q.n_chunk + q.nch - 1) / q.nch && q.n_full == q.n_chunk / q.nch, "%s M=%d n_c=%d: stages", form, M, n_c);
    CHECK((long)ring_slots(q) * q.chunk_b + behind <= q.lds_b && q.lds_b <= lds_b, "%s M=%d n_c=%d: LDS", form, M, n_c);
    for (int s = 0; s < n_stage; ++s)                           // the last byte of every stage's chunks
        CHECK((s % q.depth * q.nch + (s + 1 < n_stage ? q.nch : q.n_chunk - s * q.nch)) * q.chunk_b + behind <= q.lds_b,
              "%s M=%d n_c=%d: stage %d past the LDS", form, M, n_c, s);
    std::vector<Queue> wave(waves);
    std::vector<int> slot(q.depth, -1), need(n_stage, 0);       // stage held by a slot; its transfers
    auto issue = [&](int s) {
        slot[s % q.depth] = s;
        const int nch = s * q.nch + q.nch <= q.n_chunk ? q.nch : q.n_chunk - s * q.nch;
        std::set<std::pair<int, int>> moved;
        for (int w = 0; w < waves; ++w) {
            int ck = 0, i = w;
            for (int k = 0; k < q.ipw; ++k, i += waves) {
                while (i >= q.n_inst) { i -= q.n_inst; ++ck; }
                if (ck >= nch) {
                    if (nch < q.nch) break;
                    ck = nch - 1;
                    i = q.n_inst - 1;
                }
                moved.insert({ck, i});
                wave[w].stage.push_back(s);
            }
        }
        CHECK((int)moved.size() == nch * q.n_inst, "%s M=%d waves=%d: stage %d moves %d transfers", form, M, waves, s, (int)moved.size());
    };
    for (int s = 0; s < ring_ahead(q); ++s) issue(s);
    for (int s = 0; s < n_stage; ++s) {
        const size_t fly = (size_t)ring_may_fly(q, s);
        for (auto& v : wave)
            if (v.stage.size() - v.landed > fly) v.landed = v.stage.size() - fly;
        // barrier: stage s - 1 has been read by every wave, its slot is free
        if (s + q.depth - 1 < n_stage) {
            CHECK(slot[(s + q.depth - 1) % q.depth] < s, "%s M=%d waves=%d n_c=%d: a slot is overwritten early", form, M, waves, n_c);
            issue(s + q.depth - 1);
        }
        CHECK(slot[s % q.depth] == s, "%s M=%d waves=%d n_c=%d: stage %d is not in its slot", form, M, waves, n_c, s);
        for (auto& v : wave)
            for (size_t k = v.landed; k < v.stage.size(); ++k)
                CHECK(v.stage[k] != s, "%s M=%d waves=%d n_c=%d: stage %d is read while in flight", form, M, waves, n_c, s);
    }
}

int main() {
    const int lens[] = {1, 32, 33, 64, 65, 257, 300, 512, 1501, 3072};
    for (int n_c : lens) {
        for (int M = 2; M <= 160; M += 2)
            for (int nwv : {1, 4, 8})
                for (int i8 = 0; i8 < 2; ++i8) {
                    const int nb = (M + 15) / 16;
                    if (nwv == 1 && ks_waves(i8 != 0, nb, n_c, 4096, 256) != 1) continue;
                    const XRing q = ks_ring(i8 != 0, nb, nwv, M, n_c);
                    // where a chunk lacks some of the last row block's rows, a row of zeros sits behind the ring
                    const int behind = (M + 3) / 4 * 4 < 16 * nb ? kRowB : 0, parts = nwv / ks_groups(i8 != 0, nb, nwv);
                    CHECK(ks_zero_b(nb, M) == behind && q.parts == parts, "M=%d: split", M);
                    CHECK(ring_ok(q, ks_steps(i8 != 0)), "M=%d waves=%d: the launch refuses its plan", M, nwv);
                    // a block of one chunk leaves room for several workgroups per CU
                    if (nwv == 4 && nb <= 4 && n_c <= 32) CHECK(q.lds_b <= 163840 / 4, "M=%d n_c=%d: %d B of LDS", M, n_c, q.lds_b);
                    replay(i8 ? "int8" : "fp16", M, nwv, n_c, q, ks_steps(i8 != 0), parts, ks_lds(i8 != 0, nb, nwv), behind);
                }
        for (int M = 2; M <= 256; M += 2)
            for (long n_chan : {1L, 64L, 128L, 256L, 257L, 320L, 4096L}) {
                const XF32 f = f32_split(M, n_c, n_chan, 256);
                CHECK(f.tpw >= 1 && f.tpw <= kF32MaxTpw && f.groups * f.n_tg * f.tpw >= f.n_tiles, "fp32 M=%d: split", M);
                if (f.n_tg < 1) continue;
                CHECK(ring_ok(f32_ring(f, M, n_c), kF32Steps), "fp32 M=%d: the launch refuses its plan", M);
                if (M <= 64 && n_c <= 32) CHECK(f32_ring(f, M, n_c).lds_b <= 163840 / 4, "fp32 M=%d n_c=%d: LDS", M, n_c);
                // the last row block's fragments run past the last chunk
                replay("fp32", M, kF32Waves, n_c, f32_ring(f, M, n_c), kF32Steps, kF32Waves / f.n_tg, kF32LdsB,
                       (16 * f.nb - (M + 3) / 4 * 4) * kRowB);
            }
    }
    std::printf("%d faults\n", bad);
    return bad != 0;
}
"""


def test_no_stage_is_read_early_and_every_wave_has_work(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "replay.cpp", tmp_path / "replay"
    src.write_text(REPLAY)
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
