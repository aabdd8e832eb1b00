// Block choice that guesses the home blocks (code_screen.h), for p = 64.
#include "code_screen.h"

namespace sbo {

hipError_t launch_guess_64(const ScrArgs& a, int arith, LdsRaised* raised, hipStream_t st) {
    return launch_home_p<64, kGuess>(a, arith, raised, st);
}

// Where the steps saved are worth the steps added: the listing, and the resolution of what the bounds leave in, which grow
// with s0.  The rule is on K against s0: 262144 signals, s0 = 8, K = 16 104 -> 108 us, 32 136 -> 126, 64 208 -> 178; s0 = 5, K = 16 100 ->
// 99, 64 207 -> 170; s0 = 9, K = 32 142 -> 143, 64 210 -> 209.  A round that does not even give a compute unit its workgroup is a
// chain of latencies, and the added steps are most of them: 53000 signals, s0 = 8, K = 32 50 -> 54 us, 64 74 -> 75; s0 = 5, 64 75 -> 66.
bool guess_takes_64(const ScrArgs& a) {
    const int least = (a.m <= kNumCU * 256 ? 10 : 4) * a.s0;
    return home_takes<64>(a) && a.s0 <= kGuessMaxS0 && a.K >= (least > kGuessMinK ? least : kGuessMinK) && a.K <= kGuessMaxK;
}

}  // namespace sbo
