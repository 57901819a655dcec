// Instantiation unit: class decode kernels for up to 4096 tokens (8 label(s) per lane).
#include "ctcbeam_class.inl"

namespace ctcbeam {
hipError_t launch_class_lpt8(const KernelParams& p, hipStream_t s) { return classes::launch_class_lpt<8>(p, s); }
}  // namespace ctcbeam
