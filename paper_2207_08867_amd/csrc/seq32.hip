// seq32.hip -- the few-wavefront sequential product (seq.hpp) for binary32 components.
#include "seq.hpp"

namespace mcf {

hipError_t launch_seq32(const MmLaunch &L, hipStream_t s) { return seq_typed<float>(L, s); }

}  // namespace mcf
