// The instances of pass 2's tile kernel that are compiled with the scheduler that puts instruction
// parallelism first.
#include "colsum_pass.h"

namespace sgdkv {

hipError_t launch_colsum_ilp(const CompressArgs& a, hipStream_t st) { return ColsumTiles<true>::launch(a, st); }

}  // namespace sgdkv
