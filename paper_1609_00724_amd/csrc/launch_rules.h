// Rules of the automatic launch word: which stepping kernel a call takes and how
// many waves of it stay resident.  Plain functions of sizes and types, so that
// they can be checked without a GPU.
#pragma once
#include <cstdint>

namespace qsq {

// what the rules look at
struct StepCall {
    bool step64, euler, batch;
    int record;             // bytes of a node record: 8, 16 or 32
    uint64_t field;         // bytes of the field's node records
    bool spread;            // lines spread through the box: most seeds send one both ways
    bool volume;            // lines from the cells of a volume map, in curve order
    bool slice;             // lines of a slice map, in curve order
    bool lattice;           // the base lattice of a map: all its cells, in curve order
    int64_t halves;         // half-lines at most
    double cap;             // longest step, in cells
};

enum StepLoads { kLoadsDirect, kLoadsCells, kLoadsLds, kLoadsRegs, kLoadsBricks, kLoadsDirs };

// Waves per SIMD of the one-lane stepping kernel (0: as many as its registers
// let in), where the launch word names no lanes.  More waves hide more latency,
// but each brings 64 more lines' cells into the caches.  Seeds on a face of the
// box (a list of about one half-line per seed, counted on the device) and the
// samples of a map start side by side and share cells; lines spread through the
// box do not.
//   FP64 stepping (230 .. 250 registers: two waves fit): 500 000 half-lines of
// 224 x 224 x 112 FP32 records at a 1-cell cap step in 11.0 ms with two waves, half
// of them L2 misses, in 6.6 with one; over 64 x 64 x 32 cells one million take 3.01
// ms with two and 3.16 with one, and from 500 000 seeds on the bottom face of
// 224 x 224 x 112 3.10 and 3.34.  Up to 2^19 half-lines the longer queue of each
// lane evens out the ends as well (280 000 over 64 x 64 x 32 cells 1.67 against
// 1.27 ms), save for the side by side lines of a slice over FP32 or BF16 records (512^2
// pixels and a level, 256 x 256 x 128 cells at a 2-cell cap, BF16 3.00 with two, 3.18
// with one).
//   FP32 stepping, register caches (three fit): the third wave's cells push the
// others' out of the L1 and the L2: one million seeds, 4-cell cap, 224 x 224 x 112
// FP32 records 6.98 ms with three waves, 5.74 with two; 128 x 128 x 64 2.54 against
// 2.29.  Three stay for a field that one L2 of 4 MB holds (64 x 64 x 32 1.28 ms, two
// 1.39), and for one that the L2s hold together, stepped cell by cell (128 x 128 x
// 64, 1-cell cap, 5.02 against 5.48).  One million seeds on the bottom face of
// 224 x 224 x 112, 4-cell cap: 1.17 with three, 1.21 with two.  BF16 bricks are half the
// size and gain from three throughout (1.18 against 1.26 ms).
//   A volume's lines fill the box too, but neighbours of the list are neighbours
// in space, so the line lies at larger fields, and lists of up to 2^19
// half-lines gain from the longer queue of each lane.  FP64
// stepping, 128^3 cells and a level, 4-cell cap: 384 x 384 x 256 FP32 records 100.3 ms
// with two waves, 60.6 with one, 224 x 224 x 112 23.2 and 20.5, 128 x 128 x 64 10.8
// and 11.9; BF16 records 224 x 224 x 112 17.2 and 17.8, 384 x 384 x 256 79.2 and 47.4.
// Register caches, three waves and two: 384 x 384 x 256 66.2 and 56.7 (1-cell cap
// 90.3 and 86.4), 224 x 224 x 112 18.1 and 16.3 (1-cell cap 31.9 and 34.5), 128 x 128
// x 64 8.55 and 8.92; bricks 38.2 and 34.5 (1-cell cap 74.1 and 78.9), 14.0 and 14.3,
// 8.5 and 8.9.  64^3 cells and a level, 8-cell cap: FP64 stepping 128 x 128 x 64 2.89
// and 2.84, nodes 2.67 and 2.54, bricks 224 x 224 x 112 4.13 and 4.00.
//   A batch keeps what fits, but for its short lists of FP64 stepping over BF16 records:
// 186 000 lines of two fields of 64 to 128 nodes 2.98 ms with two waves, 2.45 with
// one (354 000 of six 3.59 and 3.95).
constexpr int64_t kShortList = (int64_t)1 << 19;
inline int auto_waves(const StepCall &c, StepLoads loads)
{
    if (c.euler) return 0;
    if (c.batch) return c.step64 && c.record == 8 && c.halves <= kShortList ? 1 : 0;
    if (c.volume) {
        const uint64_t MB = (uint64_t)1 << 20;
        const bool few = c.halves <= kShortList;
        if (c.step64) return few || c.field > 64 * MB ? 1 : 0;
        if (loads == kLoadsRegs) return few || c.field > (c.cap <= 2.0 ? 256 : 32) * MB ? 2 : 0;
        if (loads == kLoadsBricks && c.record == 16) return few || (c.cap > 2.0 && c.field > 256 * MB) ? 2 : 0;
        return 0;
    }
    if (c.step64) return (c.halves <= kShortList && !(c.slice && c.record < 32)) || (c.spread && c.field > (uint64_t)8 << 20) ? 1 : 0;
    const uint64_t MB = (uint64_t)1 << 20;
    const bool caches = loads == kLoadsRegs || (loads == kLoadsBricks && c.record == 16);
    if (caches) return c.spread && c.field > 4 * MB && !(c.cap <= 2.0 && c.field <= 32 * MB) ? 2 : 0;
    return 0;
}

// Largest call, in seeds, whose ends k_finish takes; a larger one is landed by
// one lane per half-line over a compacted list and assembled in a kernel of its
// own.  k_finish replaces eight launches, and its chain is a third as long: 2000
// seeds at 8 cells a step 260 -> 203 us, 200 000 592 -> 530 us; over the 1.3 M seeds of
// a 1024^2 map, where FP64 issue is the bound and four lanes cost more of it, it
// takes 0.84 ms against 0.53.  A batch reloads a grid per seed in every kernel: 570
// 000 seeds 0.67 against 0.73 ms, 1.2 M 0.83 against 0.90.  A trilinear Euler step is
// landed without a root find, and the separate kernels overtake sooner: landing and
// Q of 60 000 random seeds 31 against 39 us, 131 072 58 and 52, 200 000 85 and 74; in a
// batch 109 000 43 and 47, 217 000 75 and 69.  The base lattice of a map comes side
// by side: 512^2 cells of FP32 and BF16 records 0.226 and 0.236 ms against 0.204 and
// 0.199 (64^3 of a volume 0.716 and 0.689 against 0.679 and 0.618), 256^2 0.09 and 0.09
// against 0.16 and 0.15; a slice of FP64 records that lines leave both ways 0.376 against
// 0.319.  64^3 cells of FP64 records k_finish takes faster (1.06 against 1.07, of 224 x
// 224 x 112 nodes 1.22 against 1.33).
inline int64_t finish_seeds(const StepCall &c, int order)
{
    if (c.lattice && order == 1 && (c.record < 32 || !c.volume)) return (int64_t)1 << 17;
    if (c.euler && order == 1) return (int64_t)1 << 17;
    return (int64_t)1 << (c.batch ? 20 : 18);
}

// a list of more half-lines than this, of n seeds, is spread
inline int64_t spread_halves(int64_t n) { return n + n / 2; }

// Longest work list (half-lines) that is stepped with four lanes a line; edge: the
// box's longest edge in longest steps.  A list that fits the grid lasts as long
// as its longest line, and four lanes a line shorten that chain: 60 000
// half-lines of 192 x 192 x 96 cells at a 1-cell cap take 0.91 ms against 1.67 (4
// cells: 0.55 against 0.91), 240 000 1.98 against 2.55.  A longer list is bound by
// VALU issue, where four lanes a line cost 1.7 times the instructions and the
// refills weigh more the shorter the lines: 520 000 half-lines 3.36 against 3.54
// ms; 64^2 x 32 cells at 8 cells a step 128 000 0.42 against 0.40, 512 000 1.02
// against 0.87.  So lines of 32 steps or more across the box's longest edge go
// four lanes each up to 2^19, shorter ones up to 2^16.  (FP32 stepping over BF16
// records, 64^2 x 32 cells at 1 cell, 500 000: 1.60 against 1.76; over FP64 records,
// which one lane loads directly, 2.00 against 2.86.)  FP64 stepping keeps half as
// many waves resident and a batch reloads its grid with every line: up to 2^17
// (FP64, 128^2 x 64 cells at 1 cell: 128 000 half-lines 1.53 against 1.74 ms, 256 000
// 2.45 against 2.34).
//   An Euler step has one evaluation, and one lane's does little beside it.  While
// the caches hold a field of FP32 or BF16 records, lists of up to 2^17 gain (128^2
// x 64 cells, FP32 records: 64 000 half-lines 0.77 against 1.25 ms, 128 000 1.21
// against 1.30, 256 000 1.55 against 1.47), of FP64 stepping up to 2^16 (64 000 0.89
// against 1.16, 128 000 1.37 against 1.32); over 90 MB of them the adaptive
// steps' lists do (256 000 2.76 ms both ways, 500 000 4.16 against 4.74, FP64 stepping
// 128 000 2.33 against 3.03), and so over FP64 records of any size (64^2 x 32 cells, 500
// 000: 1.44 against 2.14; FP64 stepping 128 000 0.76 against 0.79) and in a batch (12
// fields, 89 000 seeds, FP64 stepping 1.13 against 1.46).
//   Quadratic and cubic stencils have 27 and 64 records: loading a row of them
// across the quad beats one lane's loads at any length (cubic, 4 cells a step:
// 4000 half-lines 1.5 against 2.5 ms, 10^6 13.8 against 15.3; FP64 stepping 1.7 to
// 2.7 times).
inline int64_t quad_list(const StepCall &c, double edge, int order)
{
    if (order > 1) return (int64_t)1 << 30;
    if (!(edge >= 32.0)) return (int64_t)1 << 16;
    if (c.euler && !c.batch && c.record < 32 && c.field <= (uint64_t)64 << 20) return (int64_t)1 << (c.step64 ? 16 : 17);
    return (int64_t)1 << (c.step64 || c.batch ? 17 : 19);
}

}  // namespace qsq
