// The plane rotation of the Jacobi eigensolver (init.hip).
#pragma once

namespace falqon {

// Cosine and sine of the rotation that annihilates hab between the diagonal entries haa and hbb; false (and the
// identity) for an entry below the rounding level of the two, which is left alone.
__host__ __device__ inline bool jacobi_rotation(double haa, double hbb, double hab, double& c, double& s)
{
    c = 1.0;
    s = 0.0;
    if (!(fabs(hab) > 1e-300 && fabs(hab) > 1e-16 * sqrt(fabs(haa * hbb)))) return false;
    // tangent of the smaller angle: 2 hab / (d +- sqrt(d^2 + 4 hab^2)), d = hbb - haa.  Entries between directions
    // that are null up to rounding can be so small that the squares underflow: scaled by a power of two.
    double d = hbb - haa, x = 2.0 * hab;
    const double scale = fmax(fabs(d), fabs(x)) < 0x1p-460 ? 0x1p+500 : 1.0;
    d *= scale;
    x *= scale;
    const double root = sqrt(d * d + x * x);
    const double tn = x / (d >= 0.0 ? d + root : d - root);
    c = rsqrt(1.0 + tn * tn);
    s = tn * c;
    return true;
}

}  // namespace falqon
