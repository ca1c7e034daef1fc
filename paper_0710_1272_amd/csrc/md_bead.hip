// md_bead.hip -- instantiations of the bead kernel.  Compiled once per variant (the build passes
// MD_REAL, MD_PERIODIC and MD_POLY), so that the variants compile side by side.
#include "md_bead.hpp"

#ifndef MD_REAL
#error "md_bead.hip is compiled with -DMD_REAL=float|double -DMD_PERIODIC=0|1 -DMD_POLY=0|1"
#endif

namespace lbmd {
template hipError_t launch_md_g<MD_REAL, MD_PERIODIC != 0, MD_POLY != 0>(const Context&, const void*, int, const StepCount&,
                                                                         hipStream_t);
}  // namespace lbmd
