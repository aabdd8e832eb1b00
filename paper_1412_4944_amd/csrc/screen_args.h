// Arguments of the screened block choice (code_screen.h) and its entry points.
#pragma once

#include "sbo_internal.h"
#include "device_utils.h"

namespace sbo {

// Bounds of home and guessed blocks (code_screen.h): t, in units of |y|^2 / P; of the sum of min(c^2, t) over kHomeRows of the P
// coefficients of a random direction, in units of |y|^2, mean and spread.
constexpr float kHomeT = 0.8f;
constexpr int home_rows(int P) { return P > 64 ? 64 : 32; }
constexpr float home_sum(int P) { return 0.447f * home_rows(P) / P; }
constexpr float home_spread(int P) { return P > 64 ? 0.010f : 0.026f; }
// A signal is weak if its best block keeps less than 1 + s0 t - home_rest: there such bounds leave one block in 160 in (mean + 2.5
// spreads, and what the arithmetic may lose).  A block that represents a signal keeps 1 + s0 t - (the sum over all atoms): s0 t of it are
// the kept ones.
constexpr float home_rest(int P) { return home_sum(P) - 2.5f * home_spread(P) - 0.006f; }

// What the resolution reads, besides Dh: Dx = the dictionary in the exact arithmetic's operand order.
struct ScrArgs {
    const float* Y;
    int m;
    const u32x4* Dh;           // two fp16 parts per entry (device_utils.h)
    const void* Dx;            // ARITH 3: Dh, 1: three bf16 parts, 0: fp32 order
    const float2* dnorm;       // per 16 atoms: largest norm, largest norm of the fp16 remainder
    int K, s0;
    int32_t* blk;
    int32_t* chunk_count;      // or nullptr
    int chunk;
    // iterations of sbo_iterate (home blocks, code_screen.h): three counts of weak signals, in turn, and the iteration
    int* weak = nullptr;
    int turn = 0;
    int* short_cut = nullptr;  // home and guessed blocks: whether a workgroup got by with them
    // ... from the second one on: the last grouping, and the blocks whose last update was by Newton-Schulz (negative)
    const int32_t *perm = nullptr, *offsets = nullptr, *sweeps = nullptr;
    bool load_only = false;    // nothing is launched, but the kernel is there afterwards
    // ... in the first one, and in sbo_code: per block |Q Q^T - I|_F^2 in two parts
    const float2* dev = nullptr;
    const unsigned* sample = nullptr;        // ... and the signals of the sample that it represents, [K][kSample / 32]
    // workgroups of 64 signals, split: rows of workgroups that share out the blocks, and what they exchange (choice_split)
    int rows = 1;
    unsigned *split_E = nullptr, *split_x = nullptr;
    int split_room = 0;
    int* split_done = nullptr;
    // energy_direct_kernel only
    const float* D = nullptr;
    float* E = nullptr;        // [K][m]
};

// One translation unit per p (code_screen_<p>.hip): the kernels are many.
hipError_t launch_screen_16(const ScrArgs& a, int arith, LdsRaised* raised, hipStream_t st);
hipError_t launch_screen_32(const ScrArgs& a, int arith, LdsRaised* raised, hipStream_t st);
hipError_t launch_screen_64(const ScrArgs& a, int arith, LdsRaised* raised, hipStream_t st);
hipError_t launch_screen_256(const ScrArgs& a, int arith, LdsRaised* raised, hipStream_t st);
// With home blocks (perm, offsets, sweeps given), and whether there is a kernel for it.
hipError_t launch_home_64(const ScrArgs& a, int arith, LdsRaised* raised, hipStream_t st);
hipError_t launch_home_256(const ScrArgs& a, int arith, LdsRaised* raised, hipStream_t st);
bool home_takes_64(const ScrArgs& a);
bool home_takes_256(const ScrArgs& a);
// Guessing them (dev given).
hipError_t launch_guess_64(const ScrArgs& a, int arith, LdsRaised* raised, hipStream_t st);
bool guess_takes_64(const ScrArgs& a);
// The full-precision energies of every (signal, block), from D itself.
hipError_t launch_direct_16(const ScrArgs& a, int arith, hipStream_t st);
hipError_t launch_direct_32(const ScrArgs& a, int arith, hipStream_t st);
hipError_t launch_direct_64(const ScrArgs& a, int arith, hipStream_t st);

}  // namespace sbo
