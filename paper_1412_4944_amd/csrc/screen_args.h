// Arguments of the screened block choice (code_screen.h) and its entry points.
#pragma once

#include "sbo_internal.h"
#include "device_utils.h"

namespace sbo {

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
