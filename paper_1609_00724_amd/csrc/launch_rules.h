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
    bool spread;            // seeds anywhere (traces), not along a curve over a slice or volume (maps)
    int64_t halves;         // half-lines at most
    double cap;             // longest step, in cells
};

enum StepLoads { kLoadsDirect, kLoadsCells, kLoadsLds, kLoadsRegs, kLoadsDirs };

// Waves per SIMD of the one-lane stepping kernel (0: as many as its registers
// let in), where the launch word names no lanes.  More waves hide more latency,
// but each brings 64 more lines' cells into the caches.
//   FP64 stepping (230 .. 250 registers: two waves fit), direct loads: 500 000
// half-lines of 224 x 224 x 112 FP32 records at a 1-cell cap step in 11.0 ms with
// two waves, half of them L2 misses, in 6.6 with one; over 64 x 64 x 32 cells one
// million take 3.01 ms with two and 3.16 with one.  Up to 2^19 half-lines the
// longer queue of each lane evens out the ends as well (280 000 over 64 x 64 x 32
// cells 1.67 against 1.27 ms).
inline int auto_waves(const StepCall &c, StepLoads loads)
{
    if (c.euler || c.batch) return 0;
    if (c.step64) return c.halves <= (int64_t)1 << 19 || (c.spread && c.field > (uint64_t)8 << 20) ? 1 : 0;
    return 0;
}

}  // namespace qsq
