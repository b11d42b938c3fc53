// The plane rotation of the Jacobi eigensolver (init.hip).
#pragma once

namespace falqon {

// What the refinement below starts from.  The hardware's estimates are within 2^-24 (2^20 values over 1900 exponents).
struct JacobiEstimates {
    static __host__ __device__ double rsqrt_of(double x)
    {
#ifdef __HIP_DEVICE_COMPILE__
        return __builtin_amdgcn_rsq(x);
#else
        return 1.0 / sqrt(x);
#endif
    }
    static __host__ __device__ double reciprocal_of(double x)
    {
#ifdef __HIP_DEVICE_COMPILE__
        return __builtin_amdgcn_rcp(x);
#else
        return 1.0 / x;
#endif
    }
};

// Root, reciprocal and reciprocal root of positive normal numbers to a few 1e-16: an estimate and two Newton steps, a
// fifth of the instructions of the correctly rounded operations.
template <class E = JacobiEstimates>
__host__ __device__ inline double jacobi_rsqrt(double x)
{
    double y = E::rsqrt_of(x);
    y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}
template <class E = JacobiEstimates>
__host__ __device__ inline double jacobi_sqrt(double x)
{
    const double y = jacobi_rsqrt<E>(x), r = x * y;
    return fma(0.5 * y, fma(-r, r, x), r);
}
template <class E = JacobiEstimates>
__host__ __device__ inline double jacobi_reciprocal(double x)
{
    double y = E::reciprocal_of(x);
    y = fma(fma(-x, y, 1.0), y, y);
    return fma(fma(-x, y, 1.0), y, y);
}

// Cosine and sine of the rotation that annihilates hab between the diagonal entries haa and hbb; false (and the
// identity) for an entry below the rounding level of the two, which is left alone.
template <class E = JacobiEstimates>
__host__ __device__ inline bool jacobi_rotation(double haa, double hbb, double hab, double& c, double& s)
{
    c = 1.0;
    s = 0.0;
    // Entries between directions that are null up to rounding can be so small that their squares underflow: all three
    // are scaled by a power of two.
    const bool small = fmax(fmax(fabs(haa), fabs(hbb)), fabs(hab)) < 0x1p-400;
    const double scale = small ? 0x1p+500 : 1.0;
    if (!(fabs(hab) > 1e-300 && (hab * scale) * (hab * scale) > 1e-32 * fabs((haa * scale) * (hbb * scale)))) return false;
    // tangent of the smaller angle: 2 hab / (d +- sqrt(d^2 + 4 hab^2)), d = hbb - haa
    const double d = (hbb - haa) * scale, x = 2.0 * hab * scale;
    const double root = jacobi_sqrt<E>(d * d + x * x);
    const double tn = x * jacobi_reciprocal<E>(d >= 0.0 ? d + root : d - root);
    c = jacobi_rsqrt<E>(1.0 + tn * tn);
    s = tn * c;
    return true;
}

}  // namespace falqon
