"""The rules of the automatic launch word (csrc/launch_rules.h), on the CPU: the
calls that earlier rules made slower, each with its neighbours on the other side
of the line."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "launch_rules.h"
using namespace qsq;
// argv: question, then key=value pairs
int main(int argc, char **argv)
{
    StepCall c{};
    int loads = kLoadsDirect, order = 1;
    double edge = 1e3;
    for (int i = 2; i < argc; ++i) {
        char *v = strchr(argv[i], '=');
        *v++ = 0;
        const char *k = argv[i];
        const double x = atof(v);
        if (!strcmp(k, "step64")) c.step64 = x != 0;
        if (!strcmp(k, "euler")) c.euler = x != 0;
        if (!strcmp(k, "batch")) c.batch = x != 0;
        if (!strcmp(k, "record")) c.record = (int)x;
        if (!strcmp(k, "field")) c.field = (uint64_t)x;
        if (!strcmp(k, "spread")) c.spread = x != 0;
        if (!strcmp(k, "volume")) c.volume = x != 0;
        if (!strcmp(k, "slice")) c.slice = x != 0;
        if (!strcmp(k, "lattice")) c.lattice = x != 0;
        if (!strcmp(k, "halves")) c.halves = (int64_t)x;
        if (!strcmp(k, "cap")) c.cap = x;
        if (!strcmp(k, "loads")) loads = (int)x;
        if (!strcmp(k, "order")) order = (int)x;
        if (!strcmp(k, "edge")) edge = x;
    }
    if (!strcmp(argv[1], "waves")) printf("%d\n", auto_waves(c, (StepLoads)loads));
    if (!strcmp(argv[1], "quads")) printf("%lld\n", (long long)quad_list(c, edge, order));
    if (!strcmp(argv[1], "finish")) printf("%lld\n", (long long)finish_seeds(c, order));
}
"""

DIRECT, CELLS, LDS, REGS, BRICKS, DIRS = range(6)


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "p.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_1609_00724_amd", "csrc"),
                    "-o", d / "p", d / "p.cpp"], check=True)

    def run(question, n=(128, 128, 64), seeds=250000, **kw):
        kw = dict(dict(record=16, spread=1, cap=1.0, halves=2 * seeds), **kw)
        kw["field"] = n[0] * n[1] * n[2] * kw["record"]
        out = subprocess.run([d / "p", question, *(f"{k}={v}" for k, v in kw.items())], check=True, capture_output=True)
        return int(out.stdout)
    return run


def test_fp64_stepping_keeps_one_wave_where_two_overflow_the_caches(ask):
    # 224 x 224 x 112 FP32 records, FP64 stepping: 6.6 ms with one, 11.0 with two
    assert ask("waves", (224, 224, 112), step64=1) == 1
    assert ask("waves", (224, 224, 112), 10**6, step64=1) == 1
    assert ask("waves", (64, 64, 32), 140000, step64=1) == 1     # two lines a lane: uneven ends
    assert ask("waves", (64, 64, 32), 500000, step64=1) == 0     # the caches hold it
    assert ask("waves", (224, 224, 112), 500000, step64=1, spread=0) == 0   # seeds on a face
    assert ask("waves", (224, 224, 112), step64=1, euler=1) == 0
    assert ask("waves", (224, 224, 112), step64=1, batch=1) == 0


def test_register_cache_keeps_two_waves_where_lines_share_no_cells(ask):
    # one million spread seeds, 4-cell cap: 5.74 ms with two, 6.98 with three
    assert ask("waves", (224, 224, 112), 10**6, cap=4.0, loads=REGS) == 2
    assert ask("waves", (128, 128, 64), 10**6, cap=4.0, loads=REGS) == 2
    assert ask("waves", (128, 128, 64), 10**6, cap=1.0, loads=REGS) == 0
    assert ask("waves", (224, 224, 112), 10**6, cap=1.0, loads=REGS) == 2
    assert ask("waves", (256, 256, 128), 1 << 20, cap=8.0, spread=0, loads=REGS) == 0
    assert ask("waves", (64, 64, 32), 10**6, cap=4.0, loads=REGS) == 0                   # in one L2
    assert ask("waves", (224, 224, 112), 10**6, cap=4.0, loads=BRICKS) == 2
    assert ask("waves", (224, 224, 112), 10**6, cap=4.0, loads=BRICKS, record=8) == 0
    assert ask("waves", (224, 224, 112), 10**6, cap=4.0, loads=DIRS) == 0


def test_four_lanes_take_only_the_euler_lists_they_shorten(ask):
    # 128 000 half-lines over 64 x 64 x 32 FP32 records, FP64 stepping: one lane 0.68 ms, four 0.76
    assert ask("quads", (64, 64, 32), euler=1, step64=1) == 1 << 16
    # 256 000 over 128 x 128 x 64: FP32 1.47 against 1.55, BF16 1.46 against 1.65
    assert ask("quads", euler=1) == ask("quads", euler=1, record=8) == 1 << 17
    assert ask("quads", (224, 224, 112), euler=1) == 1 << 19
    assert ask("quads", (224, 224, 112), euler=1, step64=1) == 1 << 17
    assert ask("quads", (64, 64, 32), euler=1, record=32) == 1 << 19
    assert ask("quads", (64, 64, 32), euler=1, record=32, step64=1) == 1 << 17
    assert ask("quads", euler=1, batch=1, step64=1) == 1 << 17
    # what the rule says of adaptive steps
    assert ask("quads") == 1 << 19 and ask("quads", step64=1) == ask("quads", batch=1) == 1 << 17
    assert ask("quads", edge=31.9) == ask("quads", edge=float("nan")) == 1 << 16
    assert ask("quads", order=3, edge=4) == 1 << 30


def test_one_kernel_ends_only_the_calls_it_is_faster_for(ask):
    # landing and Q of Euler lines: 200 000 seeds 85 us in one kernel, 74 apart; a batch of 617 000 195 and 138
    assert ask("finish", euler=1) == ask("finish", euler=1, batch=1) == 1 << 17
    assert ask("finish", euler=1, order=2) == ask("finish") == 1 << 18
    assert ask("finish", batch=1) == 1 << 20


def test_volumes_keep_fewer_waves_where_their_fields_overflow_the_caches(ask):
    # 128^3 cells and a level: FP64 stepping, 384 x 384 x 256 FP32 records: 60.6 ms with one wave, 100.3 with two
    def waves(n, seeds=2**21, **kw):
        return ask("waves", n, seeds, spread=0, volume=1, **kw)
    for rec in (16, 32):
        assert waves((384, 384, 256), step64=1, record=rec) == 1
        assert waves((224, 224, 112), step64=1, record=rec) == 1
        assert waves((128, 128, 64), step64=1, record=rec) == 0
    assert waves((384, 384, 256), step64=1, record=8) == 1
    assert waves((224, 224, 112), step64=1, record=8) == 0
    # register caches: 56.7 ms with two waves, 66.2 with three; a 1-cell cap 86.4 and 90.3
    assert waves((384, 384, 256), cap=4.0, loads=REGS) == 2
    assert waves((384, 384, 256), cap=1.0, loads=REGS) == 2
    assert waves((224, 224, 112), cap=4.0, loads=REGS) == 2
    assert waves((224, 224, 112), cap=1.0, loads=REGS) == 0
    assert waves((128, 128, 64), cap=4.0, loads=REGS) == 0
    # bricks: 34.5 against 38.2 ms, a 1-cell cap 78.9 against 74.1
    assert waves((384, 384, 256), cap=4.0, loads=BRICKS) == 2
    assert waves((384, 384, 256), cap=1.0, loads=BRICKS) == 0
    assert waves((224, 224, 112), cap=4.0, loads=BRICKS) == 0
    # the longer queue of each lane evens out the ends of short lists
    assert waves((128, 128, 64), 2**18, step64=1) == 1
    assert waves((128, 128, 64), 2**18, cap=8.0, loads=REGS) == 2
    assert waves((224, 224, 112), 2**18, cap=8.0, loads=BRICKS) == 2
    # a slice's samples are no volume's
    assert ask("waves", (384, 384, 256), 2**20, spread=0, step64=1) == 0
    assert ask("waves", (384, 384, 256), 2**20, spread=0, cap=4.0, loads=REGS) == 0


def test_large_lattices_end_in_separate_kernels(ask):
    # 512^2 cells of FP32 or BF16 records: 0.204 and 0.199 ms against 0.226 and 0.236
    for rec in (8, 16, 32):
        assert 4**8 <= ask("finish", lattice=1, record=rec) < 4**9
    for rec in (8, 16):
        assert 8**5 <= ask("finish", lattice=1, volume=1, record=rec) < 8**6
    assert ask("finish", lattice=1, volume=1, record=32) >= 8**6    # FP64 records: k_finish ahead
    assert ask("finish", lattice=1, record=16, order=3) == 2**18
    assert ask("finish", record=16) == 2**18                # a trace, a map's rounds


def test_fp64_stepping_of_slices_over_bf16_records(ask):
    # 256^2 pixels, 65 536 half-lines: four lanes a line 1.3 times one lane's speed
    assert ask("quads", step64=1, slice=1, record=8) == 2**17
    # 512^2 pixels: 3.00 ms with two waves, 3.18 with one
    assert ask("waves", (256, 256, 128), 2**18, step64=1, slice=1, spread=0, record=8) == 0
    assert ask("waves", (256, 256, 128), 2**18, step64=1, slice=1, spread=0, record=16) == 0
    assert ask("waves", (256, 256, 128), 2**18, step64=1, slice=1, spread=0, record=32) == 1


def test_short_fp64_batches_over_bf16_records_keep_one_wave(ask):
    # 186 000 lines: 2.45 ms with one wave, 2.98 with two; 354 000 3.95 and 3.59
    assert ask("waves", seeds=186000, step64=1, batch=1, record=8) == 1
    assert ask("waves", seeds=354000, step64=1, batch=1, record=8) == 0
    assert ask("waves", seeds=186000, step64=1, batch=1, record=16) == 0
    assert ask("waves", seeds=186000, batch=1, record=8) == 0
