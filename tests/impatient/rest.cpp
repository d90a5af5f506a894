/* What the host code of the library links to besides the compress kernels, for the copy of these whose workgroups do not wait
 * (test_gpu_chain.py): not called there. */
#include "zipccl_internal.h"

namespace zipccl {
int launch_estimate(int, const MomentArgs&, void*) { return 1; }
int launch_estimate_robust(int, const HistArgs&, void*) { return 1; }
int launch_decompress(int, const DecompressArgs&, void*) { return 1; }
int launch_decompress_reduce(int, int, const ReduceArgs&, void*) { return 1; }
} // namespace zipccl
