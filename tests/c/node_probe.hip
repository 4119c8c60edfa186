// The node arithmetic's square root, reciprocal and corrected-rate quotient
// (csrc/node.hpp) on the GPU, for tests/test_gpu_node_math.py.
// Usage: node_probe <in> <out>
// in: int64 count n, then n doubles each of x (square root, in [1, 4)), d (reciprocal), u
// (largest |u_a|, below 1) and t (2 tau - 1); out: n doubles each of sqrt(x), 1 / d, and
// numerator, denominator and quotient of the corrected rate at u and t.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <vector>

#include "node.hpp"

using namespace lbm;

static __global__ void probe(const double *in, double *out, long long n) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const double x = in[i], d = in[n + i], u = in[2 * n + i], t = in[3 * n + i];
    out[i] = sqrt_1to4(x);
    out[n + i] = recip_density(d);
    const double S = sqrt_1to4(fma(3.0 * u, u, 1.0));
    double num, den;
    corrected_omega_terms(u, S, t, num, den);
    out[2 * n + i] = num;
    out[3 * n + i] = den;
    out[4 * n + i] = corrected_omega_node(u, S, t);
}

static bool ok(hipError_t e, const char *what) {
    if (e != hipSuccess)
        fprintf(stderr, "%s: %s\n", what, hipGetErrorString(e));
    return e == hipSuccess;
}

int main(int argc, char **argv) {
    if (argc != 3)
        return 2;
    FILE *f = fopen(argv[1], "rb");
    long long n = 0;
    if (!f || fread(&n, 8, 1, f) != 1 || n < 1 || n > (1 << 26))
        return 3;
    std::vector<double> in(4 * n), out(5 * n);
    if (fread(in.data(), 8, in.size(), f) != in.size())
        return 3;
    fclose(f);
    double *din = nullptr, *dout = nullptr;
    if (!ok(hipMalloc(&din, in.size() * 8), "alloc") || !ok(hipMalloc(&dout, out.size() * 8), "alloc") ||
        !ok(hipMemcpy(din, in.data(), in.size() * 8, hipMemcpyHostToDevice), "copy in"))
        return 4;
    hipLaunchKernelGGL(probe, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, 0, din, dout, n);
    if (!ok(hipGetLastError(), "launch") ||
        !ok(hipMemcpy(out.data(), dout, out.size() * 8, hipMemcpyDeviceToHost), "copy out"))
        return 4;
    f = fopen(argv[2], "wb");
    if (!f || fwrite(out.data(), 8, out.size(), f) != out.size())
        return 5;
    fclose(f);
    return ok(hipFree(din), "free") && ok(hipFree(dout), "free") ? 0 : 4;
}
