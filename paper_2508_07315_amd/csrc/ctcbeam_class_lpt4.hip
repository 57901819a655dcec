// Instantiation unit: class decode kernels for up to 2048 tokens (4 label(s) per lane).
#include "ctcbeam_class.inl"

namespace ctcbeam {
hipError_t launch_class_lpt4(const KernelParams& p, hipStream_t s) { return classes::launch_class_lpt<4>(p, s); }
}  // namespace ctcbeam
