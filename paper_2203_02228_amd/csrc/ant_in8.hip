// ant_in8.hip -- the initial search with 3-opt: its workgroup (8 waves) and its
// sweeps.
#include "ant_kernels.hpp"
#include "faco_init.hpp"

AntKernelFn faco_init_search_kernel(int k) {
  return k <= 16 ? faco::init_search_kernel<16> : faco::init_search_kernel<32>;
}

InitSweepFn faco_init_sweep3_kernel(int k) {
  return k <= 16 ? faco::init_sweep3_kernel<16> : faco::init_sweep3_kernel<32>;
}
