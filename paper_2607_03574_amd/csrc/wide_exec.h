// Library functions of the wide kernel, shared by the kernel and the host
// emulator that checks the scheduler.  Adjoint rules follow Appendix C, table
// tab:adjoints; w is the adjoint so far, or +0.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>

namespace ndvm {
namespace wide {

#define NDVM_WIDE_HD __host__ __device__ __forceinline__

NDVM_WIDE_HD double clamp_eps(double x) { return x < 1e-8 ? 1e-8 : x; }
NDVM_WIDE_HD double f_logc(double x) { return log(clamp_eps(x)); }
NDVM_WIDE_HD double f_sqrtc(double x) { return sqrt(clamp_eps(x)); }
NDVM_WIDE_HD double f_accsin(double x, double y, double w) {
    const double c = cos(y);
    return x != 0.0 ? w + x * c : w;
}
NDVM_WIDE_HD double f_acccos(double x, double y, double w) {
    const double s = -sin(y);
    return x != 0.0 ? w + x * s : w;
}
NDVM_WIDE_HD double f_acclog(double x, double y, double w) { return ((x != 0.0) & (y > 1e-8)) ? w + x / y : w; }
NDVM_WIDE_HD double f_accabs(double x, double y, double w) {
    const double d = y > 0.0 ? x : (y < 0.0 ? -x : 0.0);
    return x != 0.0 ? w + d : w;
}
NDVM_WIDE_HD double f_accpow(double x, double y, double z, double w) {
    const double c = log(y);
    return x != 0.0 ? w + z * c : w;
}
NDVM_WIDE_HD double f_accsqrt(double x, double y, double z, double w) {
    const double d = 2.0 * z;
    return ((x != 0.0) & (y > 1e-8)) ? w + x / d : w;
}

}  // namespace wide
}  // namespace ndvm
