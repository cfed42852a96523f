// What the chip's power leaves of the clock under matrix instructions alone: a loop of bf16 products from registers, eight
// wavefronts a workgroup (two a SIMD), operands of zeros or random, on one workgroup or one per CU.  Each workgroup reports core cycles (s_memtime)
// and 10 ns ticks.  Build: hipcc --offload-arch=gfx950 -O3 -Xclang -target-feature -Xclang -packed-fp32-ops matrix_loop_clock.hip -o matrix_loop_clock
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <vector>

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kRounds = 4000, kOps = 8;   // products per wavefront: kRounds * kOps (32x32x16; 16x16x32: twice as many)
constexpr int kWaves = 8, kWords = 2 * kOps * 64 * kWaves;   // operands, 16 bytes each

template <bool WIDE> __global__ __launch_bounds__(64 * kWaves) void loop(const uint4 *in, float *out, unsigned long long *clk)
{
    const int t = threadIdx.x;
    bf16x8 a[kOps], b[kOps];
    for (int i = 0; i < kOps; ++i) {
        a[i] = __builtin_bit_cast(bf16x8, in[(2 * i) * 64 * kWaves + t]);
        b[i] = __builtin_bit_cast(bf16x8, in[(2 * i + 1) * 64 * kWaves + t]);
    }
    f32x16 c[2] = {};
    f32x4 d[8] = {};
    __syncthreads();
    const unsigned long long t0 = __builtin_amdgcn_s_memrealtime(), c0 = __builtin_amdgcn_s_memtime();
    for (int r = 0; r < kRounds; ++r) {
#pragma unroll
        for (int i = 0; i < kOps; ++i) {
            if constexpr (WIDE) {
                c[i & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[i], c[i & 1], 0, 0, 0);
            } else {
                d[i & 3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[i], d[i & 3], 0, 0, 0);
                d[4 + (i & 3)] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[i], a[i], d[4 + (i & 3)], 0, 0, 0);
            }
        }
    }
    __syncthreads();
    const unsigned long long c1 = __builtin_amdgcn_s_memtime(), t1 = __builtin_amdgcn_s_memrealtime();
    float s = 0.f;
    for (int i = 0; i < 16; ++i) s += c[0][i] + c[1][i];
    for (int i = 0; i < 8; ++i) s += d[i][0] + d[i][1] + d[i][2] + d[i][3];
    out[blockIdx.x * 64 * kWaves + t] = s;
    if (t == 0) {
        clk[2 * blockIdx.x] = c1 - c0;
        clk[2 * blockIdx.x + 1] = t1 - t0;
    }
}

#define CHECK(x) do { const hipError_t e_ = (x); if (e_ != hipSuccess) { fprintf(stderr, "%s: %s\n", #x, hipGetErrorString(e_)); return 1; } } while (0)

int main()
{
    int cus = 0;
    CHECK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, 0));
    uint4 *in = nullptr;
    float *out = nullptr;
    unsigned long long *clk = nullptr;
    CHECK(hipMalloc(&in, kWords * sizeof(uint4)));
    CHECK(hipMalloc(&out, (size_t)cus * 64 * kWaves * sizeof(float)));
    CHECK(hipMalloc(&clk, (size_t)cus * 2 * sizeof(unsigned long long)));
    for (int random = 0; random < 2; ++random) {
        std::vector<uint16_t> h((size_t)kWords * 8, 0);
        uint32_t x = 12345u;
        if (random)
            for (auto &v : h) {
                x = x * 1664525u + 1013904223u;
                v = (uint16_t)((x >> 16 & 0x807fu) | 0x3f00u | (x >> 2 & 0x80u));   // +- 0.5 .. 2, all bits of the fraction
            }
        CHECK(hipMemcpy(in, h.data(), (size_t)kWords * sizeof(uint4), hipMemcpyHostToDevice));
        for (int wide = 1; wide >= 0; --wide)
            for (int wgs : {1, cus}) {
                std::vector<unsigned long long> c((size_t)wgs * 2);
                std::vector<double> mhz, us;
                for (int rep = 0; rep < 12; ++rep) {   // (long enough for the chip to settle; the last is reported)
                    if (wide) loop<true><<<wgs, 64 * kWaves>>>(in, out, clk); else loop<false><<<wgs, 64 * kWaves>>>(in, out, clk);
                    CHECK(hipGetLastError());
                }
                CHECK(hipDeviceSynchronize());
                CHECK(hipMemcpy(c.data(), clk, c.size() * sizeof(c[0]), hipMemcpyDeviceToHost));
                for (int w = 0; w < wgs; ++w) {
                    mhz.push_back((double)c[2 * w] / (double)c[2 * w + 1] * 100.0);
                    us.push_back((double)c[2 * w + 1] / 100.0);
                }
                std::sort(mhz.begin(), mhz.end());
                std::sort(us.begin(), us.end());
                const double flops = 2.0 * 32 * 32 * 16 * kRounds * kOps * kWaves * wgs;
                printf("%-7s %-9s %3d workgroups: %6.0f MHz (median; %.0f .. %.0f), %7.1f us, %8.1f TFLOP/s\n", random ? "random" : "zeros", wide ? "32x32x16" : "16x16x32",
                       wgs, mhz[mhz.size() / 2], mhz.front(), mhz.back(), us[us.size() / 2], flops / us[us.size() / 2] * 1e-6);
                fflush(stdout);
            }
    }
    return 0;
}
