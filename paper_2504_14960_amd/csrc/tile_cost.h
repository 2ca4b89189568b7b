// What a launch of the large-tile persistent kernels takes for each height of its tiles: the kernels choose the height by it
// (from the rows every expert really has), the host chooses between them and the weight-streaming kernels.
#pragma once

#include "common.h"

namespace moe {

// A tile takes `end` and for every k-tile (128 bytes of the operands' rows) what the products take (`alone` on the chip,
// `shared` more with all compute units at work) and what the weights take to come from memory (`stream`, with all compute
// units at work and each M-tile the only one of its expert).  us.
struct HeightCost {
    float alone, shared, stream, end;
};
struct TileCosts {
    HeightCost h256, h192, h128;
};
// Fitted to 950 products each (12 layers, 24 to 4096 rows per expert, routers without bias, with a normal and a Zipf-1.2
// one) on the 32x32 matrix instructions; the present kernels take less.  Over 1364 products each of theirs (31 layers of 2 to 128
// experts, 40 to 2200 rows per expert, even and skewed experts) the estimate is 6, 12 and 12 % too long (256, 192 and 128 rows, bf16)
// and 10, 13 and 14 % (FP8), spread by 7 to 13 %.  The height they choose is behind the best of the three by 0.2 and 0.3 % on
// average, 14 and 10 % at most; with the choice itself, 1.5 us of a launch, 2.8 and 3.6 %.
// Constants refitted to those products, to 2 % on average, choose no better height and move the line to the other kernels the
// wrong way as often as the right one: of 682 products each gate/up takes 0.998 and down 0.997 of the time (FP8 1.004 and 0.998), 74
// faster and 52 slower by more than 3 % (FP8 84 and 81), the worst by a fifth (FP8 by 42 %: 8 x 160 rows, 2048 x 4096, down 23 / 33 us).
constexpr TileCosts kCostBf16 = {{1.02f, 0.49f, 0.52f, 2.5f}, {0.94f, 0.30f, 0.94f, 2.2f}, {0.70f, 0.20f, 1.19f, 2.0f}};
constexpr TileCosts kCostFp8 = {{0.95f, 0.45f, 0.80f, 5.8f}, {0.73f, 0.42f, 1.08f, 4.5f}, {0.71f, 0.12f, 1.20f, 3.4f}};

// mt M-tiles of `experts` experts (with rows), ntn N-tiles each, on `slots` workgroups: whole rounds and a last one whose
// tiles have the memory and the power of the chip to fewer
__host__ __device__ inline float tiles_us(const HeightCost& c, float mt, float experts, int ntn, int slots, int kt) {
    const float tiles = mt * (float)ntn, whole = floorf(tiles / (float)slots), left = tiles / (float)slots - whole;
    auto round = [&](float fill) {
        const float mul = c.alone + c.shared * fill, mem = c.stream * fill * experts / mt;
        return (float)kt * sqrtf(mul * mul + mem * mem) + c.end;
    };
    return whole * round(1.f) + (left > 0.f ? round(left) : 0.f);
}

}  // namespace moe
