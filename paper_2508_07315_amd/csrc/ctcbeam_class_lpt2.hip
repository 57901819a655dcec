// Instantiation unit: class decode kernels for up to 1024 tokens (2 label(s) per lane).
#include "ctcbeam_class.inl"

namespace ctcbeam {
hipError_t launch_class_lpt2(const KernelParams& p, hipStream_t s) { return classes::launch_class_lpt<2>(p, s); }
}  // namespace ctcbeam
