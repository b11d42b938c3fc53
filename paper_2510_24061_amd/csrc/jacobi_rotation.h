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

// Squared length of a column as it follows from the rotations since it was last formed from the column itself, and the lengths
// that went into it: its rounding errors are some 1e-16 of these.
struct JacobiLength {
    double now, carried;
};

// What the rotation makes of the lengths of its two columns; false if they have to be formed anew.  No term of a sum exceeds
// its column's old length (tn^2 hbb <= haa for the shorter one, as hab^2 <= haa hbb), so a rotation adds some roundings of
// that; errors of before come with the weights of the lengths, but do not cancel where these do.  Where less than a
// thousandth of them is left, a length is no longer good.  (Compared with the column's own largest length, errors go from
// column to column and grow by a thousand on each.)
__host__ __device__ inline bool jacobi_follow(double c, double tn, double hab, JacobiLength& a, JacobiLength& b)
{
    const double haa = a.now, hbb = b.now, carried = a.carried, c2 = c * c, t2 = tn * tn;
    a.now = c2 * fma(tn, fma(tn, hbb, -2.0 * hab), haa);
    b.now = c2 * fma(tn, fma(tn, haa, 2.0 * hab), hbb);
    a.carried = fmax(a.now, c2 * fma(t2, b.carried, carried));
    b.carried = fmax(b.now, c2 * fma(t2, carried, b.carried));
    return a.now >= 1e-3 * a.carried && b.now >= 1e-3 * b.carried;
}

}  // namespace falqon
