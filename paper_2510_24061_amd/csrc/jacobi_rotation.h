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

// Reciprocal root of a positive normal number to a few 1e-16: an estimate and one step of third order (its error is the cube
// of the estimate's), a fifth of the instructions of the correctly rounded operation.
template <class E = JacobiEstimates>
__host__ __device__ inline double jacobi_rsqrt(double x)
{
    const double y = E::rsqrt_of(x), e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// Cosine, sine and tangent of the rotation that annihilates hab between the diagonal entries haa and hbb; false (and the
// identity) for an entry below the rounding level of the two, which is left alone.
// The tangent comes straight from the estimates: a relative error d of it leaves d hab of the entry, here 2^-23, and the
// next sweep takes that; the rotation is as orthogonal as with an exact tangent, and the chain of dependent instructions, which is
// what an eigensolver's round waits for, half as long.
template <class E = JacobiEstimates>
__host__ __device__ inline bool jacobi_rotation(double haa, double hbb, double hab, double& c, double& s, double& tn)
{
    // Entries between directions that are null up to rounding can be so small that their squares underflow: all three
    // are scaled by a power of two.
    const bool small = fmax(fmax(fabs(haa), fabs(hbb)), fabs(hab)) < 0x1p-400;
    const double scale = small ? 0x1p+500 : 1.0;
    const bool turns = fabs(hab) > 1e-300 && (hab * scale) * (hab * scale) > 1e-32 * fabs((haa * scale) * (hbb * scale));
    // tangent of the smaller angle: 2 hab / (d +- sqrt(d^2 + 4 hab^2)), d = hbb - haa
    const double d = (hbb - haa) * scale, x = 2.0 * hab * scale, square = d * d + x * x;
    const double root = square * E::rsqrt_of(square);
    const double t = x * E::reciprocal_of(d >= 0.0 ? d + root : d - root);
    tn = turns ? t : 0.0;
    c = turns ? jacobi_rsqrt<E>(1.0 + t * t) : 1.0;
    s = tn * c;
    return turns;
}

}  // namespace falqon
