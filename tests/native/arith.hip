// arith.hip -- counts where recip, quotient and root of the step's arithmetic (lbm_device.hpp) differ
// from the compiler's correctly rounded division and square root: every FP32 operand of their range,
// random FP64 ones.  Built with the library's own flags.
#include <hip/hip_runtime.h>
#include <math.h>

#include "lbm_device.hpp"

namespace {

constexpr int kGroups = 1024, kItems = 256;

__device__ unsigned long long mix(unsigned long long z) {
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ bool differ(double a, double b) { return !(a == b) && !(a != a && b != b); }

// Every non-negative float: out[0] recip on [1, 2^65), out[1] root from 1/4 on, out[2] reciprocal on
// [2^-126, 2^126].
__global__ void every_float(unsigned long long* out) {
    unsigned long long bad[3] = {0, 0, 0};
    const unsigned stride = gridDim.x * blockDim.x;
    for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < 0x7f800000u; i += stride) {
        const float x = __uint_as_float(i);
        if (x >= 1.0f && x < 0x1p65f) bad[0] += differ(lbm::recip(x), 1.0f / x);
        if (x >= 0.25f) bad[1] += differ(lbm::root(x), sqrtf(x));
        if (x >= 0x1p-126f && x <= 0x1p126f) bad[2] += differ(lbm::reciprocal(x), 1.0f / x);
    }
    for (int k = 0; k < 3; ++k)
        if (bad[k]) atomicAdd(out + k, bad[k]);
}

template <typename R>
__device__ R draw(unsigned long long h, int emin, int emax) {   // magnitude in [2^emin, 2^emax)
    const double m = 1.0 + double(h >> 12) * 0x1p-52;
    return R(ldexp(m, emin + int(mix(h) % unsigned(emax - emin))));
}

// Random operands: out[0] quotient FP32 (numerator of at least 2^-100, a normal result), out[1] quotient
// FP64 (2^-960, likewise), out[2] root FP64 from 2^-970 on, out[3] reciprocal FP64, out[4] root FP64 below
// 2^-970, subnormals included, off by more than 2^-44 of it: there its last correction vanishes, and
// one Newton step has squared the hardware's error (2^-23).
__global__ void random_operands(unsigned long long* out, int rounds) {
    unsigned long long bad[5] = {0, 0, 0, 0, 0};
    const unsigned long long id = blockIdx.x * (unsigned long long)blockDim.x + threadIdx.x;
    for (int k = 0; k < rounds; ++k) {
        const unsigned long long h = mix(id * rounds + k), g = mix(h ^ 0x5555);
        const float sign = h & 1 ? -1.0f : 1.0f;
        const float a = sign * draw<float>(h, -100, 60), b = draw<float>(g, 0, 24);
        bad[0] += differ(lbm::quotient(a, b, lbm::recip(b)), a / b);
        const double c = sign * draw<double>(h, -960, 400), d = draw<double>(g, 0, 60);
        bad[1] += differ(lbm::quotient(c, d, lbm::recip(d)), c / d);
        const double x = draw<double>(h, -970, 1020), y = draw<double>(g, -1000, 1000);
        bad[2] += differ(lbm::root(x), sqrt(x));
        bad[3] += differ(lbm::reciprocal(y), 1.0 / y);
        const double z = draw<double>(g, -1074, -970), w = sqrt(z);
        bad[4] += !(fabs(lbm::root(z) - w) <= 0x1p-44 * w);
    }
    for (int k = 0; k < 5; ++k)
        if (bad[k]) atomicAdd(out + k, bad[k]);
}

// one: 1, unknown to the compiler, which would otherwise work the results out by itself
template <typename R>
__device__ int specials(R one) {
    const R inf = INFINITY * one, nan = NAN * one;
    int bad = 0;
    const R a[6] = {R(0) * one, R(-0.0) * one, inf, -inf, nan, R(3) * one};
    const R b[4] = {one, R(2.5) * one, inf, nan};
    for (R x : a)
        for (R y : b) bad += differ(lbm::quotient(x, y, lbm::recip(y)), x / y);
    const R s[4] = {R(0) * one, inf, nan, R(0.3) * one};
    for (R x : s) {
        bad += differ(lbm::root(x), sizeof(R) == 4 ? R(sqrtf(float(x))) : R(sqrt(double(x))));
        bad += differ(lbm::reciprocal(x), R(1) / x);
    }
    const R n[3] = {-one, -inf, R(-1e-30) * one};   // negative: NaN, not what root makes of them
    for (R x : n) bad += lbm::rsq_1ulp(x) == lbm::rsq_1ulp(x);
    return bad;
}

__global__ void special_operands(unsigned long long* out, float one) {
    out[0] = specials<float>(one);
    out[1] = specials<double>(one);
}

}  // namespace

// counts[0..2] of every_float, [3..7] of random_operands, [8..9] of special_operands; 0, or the
// failing call's hipError_t.
extern "C" int arith_check(unsigned long long* counts, int rounds) {
    unsigned long long* dev = nullptr;
    hipError_t e = hipMalloc(&dev, 10 * sizeof *dev);
    if (e != hipSuccess) return e;
    e = hipMemset(dev, 0, 10 * sizeof *dev);
    if (e == hipSuccess) {
        every_float<<<kGroups, kItems>>>(dev);
        random_operands<<<kGroups, kItems>>>(dev + 3, rounds);
        special_operands<<<1, 1>>>(dev + 8, 1.0f);
        e = hipMemcpy(counts, dev, 10 * sizeof *dev, hipMemcpyDeviceToHost);
    }
    (void)hipFree(dev);
    return e;
}
