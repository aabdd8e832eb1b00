// Block choice, screened (code_screen.h), for p = 64.
#include "code_screen.h"

namespace sbo {

hipError_t launch_screen_64(const ScrArgs& a, int arith, LdsRaised* raised, hipStream_t st) {
    return launch_p<64>(a, arith, raised, st);
}

hipError_t launch_direct_64(const ScrArgs& a, int arith, hipStream_t st) { return launch_direct_p<64>(a, arith, st); }

}  // namespace sbo
