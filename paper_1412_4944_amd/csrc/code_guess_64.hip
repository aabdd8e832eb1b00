// Block choice that guesses the home blocks (code_screen.h), for p = 64.
#include "code_screen.h"

namespace sbo {

hipError_t launch_guess_64(const ScrArgs& a, int arith, LdsRaised* raised, hipStream_t st) {
    return launch_home_p<64, kGuess>(a, arith, raised, st);
}

// Where the steps saved are worth the steps added: the listing, and the resolution of what the bounds leave in, which grow
// with s0.  The rule is on K against s0; choice, full / guesses (us): 262144 signals, s0 = 8, K = 16 104 / 108, 32 106 / 94, 64 187 / 152; s0 = 3,
// K = 16 63 / 63, 20 73 / 67, 24 83 / 74; s0 = 9, K = 32 142 / 143, 64 210 / 209.  Up to 65536 signals full screening has one workgroup of 256 on
// every compute unit, one signal more and some have two, which takes a quarter longer; guesses leave room for the second.  Choice, and the call
// in brackets: K = 32, s0 = 8 53000 37 / 40 (56 / 61), 65000 39 / 42 (60 / 68), 65537 49 / 42 (73 / 69), 80000 53 / 52 (76 / 78), 100003 54 / 49 (85 / 85), 130000
// 58 / 52 (95 / 95); s0 = 5 65000 39 / 35 (60 / 60), 65537 48 / 36 (72 / 62); K = 64, s0 = 8 65000 64 / 64 (87 / 89), 65537 85 / 65 (110 / 95); K = 24,
// s0 = 5 65000 32 / 34 (53 / 60), 65537 39 / 31 (62 / 58).  Below, only K >= 10 s0 gains: 53000 signals, K = 64, s0 = 5 58 / 48, K = 40, s0 = 4 40 / 35,
// K = 20, s0 = 2 27 / 24, K = 80, s0 = 8 68 / 67.
bool guess_takes_64(const ScrArgs& a) {
    const int least = (a.m <= kNumCU * 256 ? 10 : 4) * a.s0;
    return home_takes<64>(a) && a.s0 <= kGuessMaxS0 && a.K >= (least > kGuessMinK ? least : kGuessMinK) && a.K <= kGuessMaxK;
}

}  // namespace sbo
