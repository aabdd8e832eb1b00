// Block choice with home blocks (code_screen.h), for p = 64.
#include "code_screen.h"

namespace sbo {

hipError_t launch_home_64(const ScrArgs& a, int arith, LdsRaised* raised, hipStream_t st) {
    return launch_home_p<64, kHome>(a, arith, raised, st);
}

bool home_takes_64(const ScrArgs& a) { return home_takes<64>(a); }

}  // namespace sbo
