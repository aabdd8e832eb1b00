// Block choice with home blocks (code_screen.h), for p = 256.
#include "code_screen.h"

namespace sbo {

hipError_t launch_home_256(const ScrArgs& a, int arith, LdsRaised* raised, hipStream_t st) {
    return launch_home_p<256, kHome>(a, arith, raised, st);
}

bool home_takes_256(const ScrArgs& a) { return home_takes<256>(a); }

}  // namespace sbo
