// Instantiation unit: class decode kernels for up to 512 tokens (1 label(s) per lane).
#include "ctcbeam_class.inl"

namespace ctcbeam {
hipError_t launch_class_lpt1(const KernelParams& p, hipStream_t s) { return classes::launch_class_lpt<1>(p, s); }
}  // namespace ctcbeam
