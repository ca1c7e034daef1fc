// md_step.hip -- instantiations of the one-launch coupled step.  Compiled once per variant (the
// build passes MD_STORAGE and MD_POLY), so that the variants compile side by side.
#include "md_bead.hpp"

#ifndef MD_STORAGE
#error "md_step.hip is compiled with -DMD_STORAGE=0..3 -DMD_POLY=0|1"
#endif

namespace lbmd {
template hipError_t prepare_step_one_g<MD_STORAGE, MD_POLY != 0>();
template hipError_t launch_step_one_g<MD_STORAGE, MD_POLY != 0>(const Context&, int, bool, hipStream_t);
}  // namespace lbmd
