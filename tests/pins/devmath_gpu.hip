// The kernels' binary32 math functions evaluated on the GPU over every input of
// a range and compared with a reference (the oracle's function, passed in by
// the test) on host threads.  The cube root's device code starts from the
// device's own logarithm and exponential instructions, so only a device run
// checks it.  Test infrastructure: built by build() into
// tests/pins/libdevmath_gpu.so and loaded by tests/test_gpu_devmath.py.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <thread>
#include <vector>

#include "../../paper_2510_03964_amd/csrc/fwrs_device.hpp"

namespace {

constexpr uint64_t kChunk = uint64_t(1) << 25;   // inputs per device pass (128 MiB of results)

__global__ void cube_root_kernel(uint32_t lo, uint32_t stride, uint64_t n, float* out)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = fwrs::cube_root(__builtin_bit_cast(float, (uint32_t)(lo + i * stride)));
}

__global__ void log2_unit_kernel(uint32_t m0, uint64_t n, float* out)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = fwrs::log2_unit((uint32_t)(m0 + i - 1u) << 8);
}

// Counts the inputs (bit patterns in[i]) whose device result differs from ref.
template <typename In, typename Ref>
void compare(const std::vector<float>& got, uint64_t n, In in, Ref ref, int threads, int64_t& bad, uint32_t& first)
{
    std::vector<int64_t> count(threads, 0);
    std::vector<uint32_t> low(threads, 0xFFFFFFFFu);
    std::vector<std::thread> pool;
    for (int w = 0; w < threads; ++w)
        pool.emplace_back([&, w] {
            for (uint64_t i = (uint64_t)w; i < n; i += (uint64_t)threads) {
                const uint32_t x = in(i);
                const float b = ref(x);
                uint32_t ua, ub;
                std::memcpy(&ua, &got[i], 4);
                std::memcpy(&ub, &b, 4);
                if (ua != ub) {
                    ++count[w];
                    if (x < low[w]) low[w] = x;
                }
            }
        });
    for (auto& t : pool) t.join();
    for (int w = 0; w < threads; ++w) {
        bad += count[w];
        if (low[w] < first) first = low[w];
    }
}

// ---- the short reciprocal, root, quotient and variate test ----------------
// Each kernel counts its inputs whose short form differs from the correctly
// rounded value, taken in binary64 and rounded once (innocuous: 53 >= 2 * 24 + 2).
__global__ void short_unary_kernel(int root, uint32_t lo, uint32_t hi, unsigned long long* bad)
{
    unsigned long long n = 0;
    for (uint64_t b = lo + blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; b < hi; b += (uint64_t)gridDim.x * blockDim.x) {
        const float x = __builtin_bit_cast(float, (uint32_t)b);
        const float got = root ? fwrs::sqrt_rn(x) : fwrs::rcp_rn(x);
        const float want = root ? (float)sqrt((double)x) : (float)(1.0 / (double)x);
        n += __builtin_bit_cast(uint32_t, got) != __builtin_bit_cast(uint32_t, want);
    }
    if (n) atomicAdd(bad, n);
}

__device__ unsigned long long div_differs(uint32_t a, uint32_t b)
{
    const float n = (float)a * 0x1p-23f, d = (float)b * 0x1p-23f;      // 24-bit significands
    return fwrs::div_rn(n, d) != (float)((double)n / (double)d);
}

// The quotients nearest to a rounding boundary.  With a, b in [2^23, 2^24) the
// quotient a / b lies c / (b 2^K) from the boundary N / 2^K, N odd in
// [2^24, 2^25), K = 24 if a >= b, else 25, where a 2^K = b N + c.  Its distance
// is at least |c| 2^-25 units in the last place, and the correction's error is
// below 6 of these, so every pair with an odd or even c up to 15 is tried, for
// every b: N = -c / b modulo 2^K.
__global__ void short_div_kernel(unsigned long long* bad, unsigned long long* tried)
{
    const uint32_t b = (1u << 23) + blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= 1u << 24) return;
    const uint32_t j = __builtin_ctz(b), odd = b >> j;
    uint32_t inv = odd;                                                // odd * inv = 1 modulo 2^32
    for (int i = 0; i < 5; ++i) inv *= 2u - odd * inv;
    unsigned long long n = 0, seen = 0;
    for (int K = 24; K <= 25; ++K)
        for (int c = -15; c <= 15; ++c) {
            if (c == 0 || (c & ((1 << j) - 1)) != 0 || j > 3u) continue;
            const uint32_t mod = K - j;
            const uint32_t N0 = ((uint32_t)(-(c >> j)) * inv) & ((1u << mod) - 1u);
            for (uint64_t N = N0; N < 1u << 25; N += 1u << mod) {
                if (N < 1u << 24 || !(N & 1u)) continue;
                const uint64_t a = ((uint64_t)b * N + (uint64_t)(int64_t)c) >> K;
                if (a < 1u << 23 || a >= 1u << 24 || (a >= b) != (K == 24)) continue;
                n += div_differs((uint32_t)a, b);
                ++seen;
            }
        }
    if (n) atomicAdd(bad, n);
    if (seen) atomicAdd(tried, seen);
}

// Every numerator for the divisors whose significand is all ones or next to it,
// and random pairs.
__global__ void short_div_more_kernel(unsigned long long* bad)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;          // 2^23 threads
    unsigned long long n = 0;
    for (uint32_t k = 1; k <= 8; ++k) n += div_differs((1u << 23) + i, (1u << 24) - k);
    uint64_t z = i;
    for (int r = 0; r < 256; ++r) {
        z = (z + 0x9E3779B97F4A7C15ull) * 0xBF58476D1CE4E5B9ull;
        z ^= z >> 31;
        n += div_differs((1u << 23) | (uint32_t)(z & 0x7FFFFF), (1u << 23) | (uint32_t)((z >> 32) & 0x7FFFFF));
    }
    if (n) atomicAdd(bad, n);
}

// The short variate test against the general one for every variate, W1b taken
// at the product itself, one binary32 below and one above.
__global__ void short_takes_kernel(const float* s, int ns, unsigned long long* bad)
{
    const uint32_t word = (blockIdx.x * blockDim.x + threadIdx.x) << 8;
    unsigned long long n = 0;
    for (int i = 0; i < ns; ++i) {
        const float at = fwrs::unit_variate(word) * s[i];
        for (int o = -1; o <= 1; ++o) {
            const float W = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, at) + (uint32_t)o);
            n += fwrs::takes<true>(word, s[i], W) != fwrs::takes<false>(word, s[i], W);
        }
    }
    if (n) atomicAdd(bad, n);
}

}  // namespace

extern "C" {

// Mismatches of the short forms (-1 on a HIP error): which = 0 the reciprocal,
// 1 the root, over the bit patterns [lo, hi); 2 the quotient (lo, hi unused;
// *tried = the near-boundary pairs tried); 3 the variate test for the hi sums
// at `sums`.
int64_t gpu_short_math_mismatches(int which, uint32_t lo, uint32_t hi, const float* sums, uint64_t* tried)
{
    unsigned long long* d = nullptr;
    float* s = nullptr;
    if (hipMalloc(&d, 16) != hipSuccess) return -1;
    unsigned long long h[2] = {0, 0};
    bool ok = hipMemcpy(d, h, 16, hipMemcpyHostToDevice) == hipSuccess;
    if (ok && which < 2) {
        hipLaunchKernelGGL(short_unary_kernel, dim3(4096), dim3(256), 0, 0, which, lo, hi, d);
    } else if (ok && which == 2) {
        hipLaunchKernelGGL(short_div_kernel, dim3(1u << 15), dim3(256), 0, 0, d, d + 1);
        hipLaunchKernelGGL(short_div_more_kernel, dim3(1u << 15), dim3(256), 0, 0, d);
    } else if (ok) {
        ok = hipMalloc(&s, 4 * (size_t)hi) == hipSuccess && hipMemcpy(s, sums, 4 * (size_t)hi, hipMemcpyHostToDevice) == hipSuccess;
        if (ok) hipLaunchKernelGGL(short_takes_kernel, dim3(1u << 16), dim3(256), 0, 0, s, (int)hi, d);
    }
    ok = ok && hipMemcpy(h, d, 16, hipMemcpyDeviceToHost) == hipSuccess;
    (void)hipFree(d);
    if (s) (void)hipFree(s);
    if (tried) *tried = h[1];
    return ok ? (int64_t)h[0] : -1;
}

// fwrs::cube_root on the GPU for every binary32 whose bit pattern is in [lo, hi)
// with the given stride, against reference(t) on the host.  Returns the number
// of differing inputs (-1 on a HIP error); *first = the smallest such bit
// pattern (0xFFFFFFFF if none).
int64_t gpu_cube_root_mismatches(uint32_t lo, uint32_t hi, uint32_t stride, float (*reference)(float), int threads,
                                 uint32_t* first)
{
    if (threads < 1) threads = 1;
    if (stride < 1) stride = 1;
    const uint64_t total = hi > lo ? ((uint64_t)hi - lo + stride - 1) / stride : 0;
    float* d = nullptr;
    if (hipMalloc(&d, kChunk * 4) != hipSuccess) return -1;
    std::vector<float> got(kChunk);
    int64_t bad = 0;
    uint32_t low = 0xFFFFFFFFu;
    for (uint64_t at = 0; at < total; at += kChunk) {
        const uint64_t n = total - at < kChunk ? total - at : kChunk;
        const uint32_t base = (uint32_t)(lo + at * stride);
        hipLaunchKernelGGL(cube_root_kernel, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, 0, base, stride, n, d);
        if (hipMemcpy(got.data(), d, n * 4, hipMemcpyDeviceToHost) != hipSuccess) {
            (void)hipFree(d);
            return -1;
        }
        compare(got, n, [&](uint64_t i) { return (uint32_t)(base + i * stride); },
                [&](uint32_t x) { float t; std::memcpy(&t, &x, 4); return reference(t); }, threads, bad, low);
    }
    (void)hipFree(d);
    if (first) *first = low;
    return bad;
}

// fwrs::log2_unit on the GPU for every variate (m = 1 .. 2^24, bits = (m - 1) << 8)
// against reference(bits) on the host; as above.
int64_t gpu_log2_unit_mismatches(float (*reference)(uint32_t), int threads, uint32_t* first)
{
    if (threads < 1) threads = 1;
    const uint64_t total = uint64_t(1) << 24;
    float* d = nullptr;
    if (hipMalloc(&d, kChunk * 4) != hipSuccess) return -1;
    std::vector<float> got(kChunk);
    int64_t bad = 0;
    uint32_t low = 0xFFFFFFFFu;
    for (uint64_t at = 0; at < total; at += kChunk) {
        const uint64_t n = total - at < kChunk ? total - at : kChunk;
        const uint32_t m0 = (uint32_t)(1 + at);
        hipLaunchKernelGGL(log2_unit_kernel, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, 0, m0, n, d);
        if (hipMemcpy(got.data(), d, n * 4, hipMemcpyDeviceToHost) != hipSuccess) {
            (void)hipFree(d);
            return -1;
        }
        compare(got, n, [&](uint64_t i) { return (uint32_t)(m0 + i - 1u) << 8; },
                [&](uint32_t x) { return reference(x); }, threads, bad, low);
    }
    (void)hipFree(d);
    if (first) *first = low;
    return bad;
}

}  // extern "C"
