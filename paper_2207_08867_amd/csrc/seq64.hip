// seq64.hip -- the few-wavefront sequential product (seq.hpp) for binary64 components.
#include "seq.hpp"

namespace mcf {

hipError_t launch_seq64(const MmLaunch &L, hipStream_t s) { return seq_typed<double>(L, s); }

}  // namespace mcf
