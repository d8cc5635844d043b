// The bins of the selection's histogram: 2048 over scores in [-4, 12).  Plain C++: the CPU tests compile this file by itself.
#pragma once

namespace tri {

constexpr int kBinsPerUnit = 128, kBinOfZero = 512;   // a score's place among the bins is fmaf(score, 128, 512)

// The least score whose place is bin `bin` (1 to 2047) or above, in double, where it is exact (scores are floats: the least float from
// there on).  Places are rounded, and a bin's number, an even mantissa, takes the ties: what lies half a float's spacing below the
// number, in the binade that ends at it or holds it, still rounds to it.
constexpr double bin_edge(int bin)
{
    const int binade = bin > 1 ? 32 - __builtin_clz((unsigned)bin - 1u) : 0;   // 2^(binade - 1) < bin <= 2^binade
    const double half = (double)(1 << binade) / (double)(1 << 25);
    return ((double)(bin - kBinOfZero) - half) / (double)kBinsPerUnit;
}

}  // namespace tri
