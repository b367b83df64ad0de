// Check of quotient (paper_1906_04576_amd/csrc/recip.hpp) against the IEEE
// division.  Scaling by powers of two changes neither, so that the mantissas
// decide: every mantissa of the divisor meets 64 mantissas of the dividend,
// among them 0, all ones, the divisor's own and its neighbours, at exponents
// spread over the ranges that the callers state (divisors in [2^-40, 2^60),
// dividends in [2^-63, 2^64)).  Prints one line "quotient_check values <n>
// mismatches <m>" and exits 0 when m == 0.  Built by __graft_entry__.build();
// run by the GPU test suite.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>

#include "../../paper_1906_04576_amd/csrc/recip.hpp"

constexpr unsigned kDividends = 64;

__device__ unsigned mix(unsigned x) {
    x = (x ^ (x >> 16)) * 0x7feb352du;
    x = (x ^ (x >> 15)) * 0x846ca68bu;
    return x ^ (x >> 16);
}

// one thread per divisor mantissa (2^23 of them: the grid covers them exactly)
__global__ void k_check(unsigned long long* mismatches, unsigned* first) {
    const unsigned md = blockIdx.x * 256u + threadIdx.x;
    unsigned long long c = 0;
    for (unsigned j = 0; j < kDividends; ++j) {
        const unsigned h = mix(md * kDividends + j);
        unsigned mn = mix(h) & 0x7FFFFFu;
        if (j == 0) mn = 0u;
        if (j == 1) mn = 0x7FFFFFu;
        if (j == 2) mn = md;
        if (j == 3) mn = (md + 1u) & 0x7FFFFFu;
        if (j == 4) mn = (md - 1u) & 0x7FFFFFu;
        const unsigned ed = 127u - 40u + (h & 0xFFFFu) % 100u, en = 127u - 63u + (h >> 16) % 127u;
        const float d = __builtin_bit_cast(float, ed << 23 | md);
        const float n = __builtin_bit_cast(float, (h & 0x80000000u) | en << 23 | mn);
        const float q = mr::quotient(n, d, mr::recip_fast(d));
        if (__builtin_bit_cast(unsigned, q) != __builtin_bit_cast(unsigned, n / d)) {
            ++c;
            atomicMin(first, md);
        }
    }
    if (c) atomicAdd(mismatches, c);
}

int main() {
    unsigned long long* mism = nullptr;
    unsigned* first = nullptr;
    if (hipMalloc(&mism, sizeof(unsigned long long)) != hipSuccess || hipMalloc(&first, sizeof(unsigned)) != hipSuccess) {
        printf("quotient_check: allocation failed\n");
        return 2;
    }
    const unsigned long long zero = 0;
    const unsigned none = 0xFFFFFFFFu;
    if (hipMemcpy(mism, &zero, sizeof(zero), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(first, &none, sizeof(none), hipMemcpyHostToDevice) != hipSuccess) {
        printf("quotient_check: copy failed\n");
        return 2;
    }
    hipLaunchKernelGGL(k_check, dim3((1u << 23) / 256u), dim3(256), 0, 0, mism, first);
    unsigned long long m = 0;
    unsigned f = 0;
    if (hipDeviceSynchronize() != hipSuccess || hipMemcpy(&m, mism, sizeof(m), hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemcpy(&f, first, sizeof(f), hipMemcpyDeviceToHost) != hipSuccess) {
        printf("quotient_check: kernel failed\n");
        return 2;
    }
    printf("quotient_check values %llu mismatches %llu first 0x%08x\n", (1ull << 23) * kDividends, m, m ? f : 0u);
    (void)hipFree(mism);
    (void)hipFree(first);
    return m == 0 ? 0 : 1;
}
