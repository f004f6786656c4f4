// seq16.hip -- the few-wavefront sequential product (seq.hpp) for binary16 components.
#include "seq.hpp"

namespace mcf {

hipError_t launch_seq16(const MmLaunch &L, hipStream_t s) { return seq_typed<_Float16>(L, s); }

}  // namespace mcf
