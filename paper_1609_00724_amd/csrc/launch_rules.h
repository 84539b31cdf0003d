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
// 1.27 ms).
//   FP32 stepping, register caches (three fit): the third wave's cells push the
// others' out of the L1 and the L2: one million seeds, 4-cell cap, 224 x 224 x 112
// FP32 records 6.98 ms with three waves, 5.74 with two; 128 x 128 x 64 2.54 against
// 2.29.  Three stay for a field that one L2 of 4 MB holds (64 x 64 x 32 1.28 ms, two
// 1.39), and for one that the L2s hold together, stepped cell by cell (128 x 128 x
// 64, 1-cell cap, 5.02 against 5.48).  One million seeds on the bottom face of
// 224 x 224 x 112, 4-cell cap: 1.17 with three, 1.21 with two.  BF16 bricks are half the
// size and gain from three throughout (1.18 against 1.26 ms).
inline int auto_waves(const StepCall &c, StepLoads loads)
{
    if (c.euler || c.batch) return 0;
    if (c.step64) return c.halves <= (int64_t)1 << 19 || (c.spread && c.field > (uint64_t)8 << 20) ? 1 : 0;
    const uint64_t MB = (uint64_t)1 << 20;
    const bool caches = loads == kLoadsRegs || (loads == kLoadsBricks && c.record == 16);
    if (caches) return c.spread && c.field > 4 * MB && !(c.cap <= 2.0 && c.field <= 32 * MB) ? 2 : 0;
    return 0;
}

// a list of more half-lines than this, of n seeds, is spread
inline int64_t spread_halves(int64_t n) { return n + n / 2; }

}  // namespace qsq
