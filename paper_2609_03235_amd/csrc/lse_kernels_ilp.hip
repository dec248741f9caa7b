// The instances of pass 1 that are compiled with the scheduler that puts instruction parallelism first.
#include "lse_pass.h"

namespace sgdkv {

hipError_t launch_lse_ilp(const CompressArgs& a, hipStream_t st) { return LsePass<true>::launch(a, st); }

}  // namespace sgdkv
