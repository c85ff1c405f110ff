// How a linear system of the dense cell is solved: chunk products, or forward substitution, in how many stretches.  Host only.
#pragma once

namespace pararnn {

constexpr int kWaveIters = 4;         // iterations that a wavefront runs at once
constexpr int kWarm = 64;             // steps that a stretch starts early
constexpr int kWarmLeast = 32;        // steps of a stretch at least: shorter ones would be half warm-up and more
constexpr int kStretches = 256;       // of all sequences at most: one for each compute unit
// Substitution addresses the rows of a sequence, 256 bytes each, by 32-bit offsets: those up to 128 behind the last one, which its
// waves ask for ahead of time, must not come round to the front, and as many in front of the first one must lie behind its end, for
// such rows to read zero.
constexpr int kMostSteps = (1 << 24) - 256;

// n: stretches of a sequence (1: none, the whole sequence at once; 0: chunk products); len: steps of each but the last
struct DensePlan { int n, len; };

// Substitution or chunk products, and in how many stretches?  Nanoseconds, measured on config 4's shape and on 1 to 16
// sequences of 500 to 2000 steps: a forward substitution step takes 225, an adjoint one 160, whatever the number of sequences
// while each has a compute unit; an iteration with chunk products takes 3.94 per row but at least 67 us (the chain of one
// chunk), 17 per step for the carry and 25-30 us for the sweeps, and four iterations are what a solve needs.
//
// Stretches: one for each compute unit.  Two workgroups on a unit, 512 stretches, take 590 ns a step instead of 225 (64
// sequences of 1024 steps: 108 us with 256, 136 with 512).  Whether a recurrence forgets within kWarm steps is known only
// afterwards, so they are a bet: won, the chain is that of one stretch; lost, all of it and the warm-up.  It is taken where it
// loses at most half of what it gains.  us, without stretches / won / lost (W orthogonal, u a tenth):
//
//            forward              backward
//   1 x 200   53 /  34 /  62       43 / 25 /  48     not taken
//   1 x 300   73 /  35 /  83       61 / 26 /  64
//   6 x 523  122 /  35 / 133      100 / 27 / 102
//   16 x 600 143 /  37 / 157      116 / 30 / 120
//   64 x 272  75 /  43 /  93       66 / 36 /  72     not taken
//   64 x 400 106 /  50 / 122       87 / 41 /  94
//   64 x 1024 244 / 85 / 262      194 / 69 / 197
//   16 x 1000 231 / 43 / 240      144 / 34 / 182     backward not taken: chunk products
// (those not taken measured without the rule)
inline DensePlan dense_stretches(int B, int L, double step, double products)
{
    const int most = kStretches / B;
    if (most < 2) return {1, L};
    const int len = (L + most - 1) / most > kWarmLeast ? (L + most - 1) / most : kWarmLeast;
    if (len >= L) return {1, L};
    const double chain = step * L, without = chain < products ? chain : products;
    const double warm = step * (kWarm + kWaveIters) + 3e3;                 // and the look at the borders
    if (chain + warm - without > 0.5 * (without - step * len - warm)) return {1, L};
    return {(L + len - 1) / len, len};
}

inline DensePlan wavefront_plan(int B, int L, bool backward)
{
    if (L > kMostSteps) return {0, 0};
    const double rows = (double)B * L, step = backward ? 160.0 : 225.0;
    const double products = ((rows * 3.94 > 67e3 ? rows * 3.94 : 67e3) + 17.0 * L + 27e3) * (backward ? 1.0 : 4.0);
    const DensePlan p = dense_stretches(B, L, step, products);
    const double chain = step * L * (double)((B + 511) / 512);              // two workgroups share a compute unit
    return p.n == 1 && chain >= products ? DensePlan{0, 0} : p;
}

}  // namespace pararnn
