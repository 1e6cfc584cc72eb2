// Map readout (Y_l = phi(Z_l), not stored between strides) and zero fill.
#include "device_common.h"

namespace ssc {

template <bool BF16>
__global__ __launch_bounds__(256) void read_kernel(const float* __restrict__ Z, void* __restrict__ dst, long long n4,
                                                   int relu) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n4;
         i += (long long)gridDim.x * blockDim.x) {
        f4v z = reinterpret_cast<const f4v*>(Z)[i];
        if (relu) {
            z.x = fmaxf(z.x, 0.f); z.y = fmaxf(z.y, 0.f); z.z = fmaxf(z.z, 0.f); z.w = fmaxf(z.w, 0.f);
        }
        if constexpr (BF16) {
            uint2 p;
            p.x = f32_to_bf16_bits(z.x) | (f32_to_bf16_bits(z.y) << 16);
            p.y = f32_to_bf16_bits(z.z) | (f32_to_bf16_bits(z.w) << 16);
            reinterpret_cast<uint2*>(dst)[i] = p;
        } else {
            reinterpret_cast<f4v*>(dst)[i] = z;
        }
    }
}

// phi of a map whose channels differ in their activation: relu_bits, bit b for
// the channels 16b .. 16b + 15 (the neck map: every upsampler's own).  One
// launch over whole rows: 27 us for 384 channels of a 248x216 map (165 MB, the
// copy rate), where a launch per upsampler took 12 to 14 us for each 128
// of them: 1.05 x c3 with its neck (267 -> 255 us).
template <bool BF16>
__global__ __launch_bounds__(256) void read_mixed_kernel(const float* __restrict__ Z, void* __restrict__ dst,
                                                         long long n4, int ctot4, uint64_t relu_bits) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n4;
         i += (long long)gridDim.x * blockDim.x) {
        const int c4 = (int)(i % ctot4);
        f4v z = reinterpret_cast<const f4v*>(Z)[i];
        if ((relu_bits >> (c4 >> 2)) & 1ull) {
            z.x = fmaxf(z.x, 0.f); z.y = fmaxf(z.y, 0.f); z.z = fmaxf(z.z, 0.f); z.w = fmaxf(z.w, 0.f);
        }
        if constexpr (BF16) {
            uint2 p;
            p.x = f32_to_bf16_bits(z.x) | (f32_to_bf16_bits(z.y) << 16);
            p.y = f32_to_bf16_bits(z.z) | (f32_to_bf16_bits(z.w) << 16);
            reinterpret_cast<uint2*>(dst)[i] = p;
        } else {
            reinterpret_cast<f4v*>(dst)[i] = z;
        }
    }
}

// phi(Z) at the active sites of a sparse layer, zero elsewhere.
template <bool BF16>
__global__ __launch_bounds__(256) void read_masked_kernel(const float* __restrict__ Z, void* __restrict__ dst,
                                                          long long cells, int cout4, const uint64_t* __restrict__ memb,
                                                          int relu) {
    const long long n4 = cells * cout4;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n4;
         i += (long long)gridDim.x * blockDim.x) {
        f4v z = reinterpret_cast<const f4v*>(Z)[i];
        if (relu) {
            z.x = fmaxf(z.x, 0.f); z.y = fmaxf(z.y, 0.f); z.z = fmaxf(z.z, 0.f); z.w = fmaxf(z.w, 0.f);
        }
        if (!memb_now(memb[i / cout4])) z = f4v{0.f, 0.f, 0.f, 0.f};
        if constexpr (BF16) {
            uint2 p;
            p.x = f32_to_bf16_bits(z.x) | (f32_to_bf16_bits(z.y) << 16);
            p.y = f32_to_bf16_bits(z.z) | (f32_to_bf16_bits(z.w) << 16);
            reinterpret_cast<uint2*>(dst)[i] = p;
        } else {
            reinterpret_cast<f4v*>(dst)[i] = z;
        }
    }
}

// Zero fill of several buffers in one launch: a workgroup takes chunks of 64 KB,
// numbered through all buffers, and finds a chunk's buffer in the table of
// first chunks (uniform).  A reset clears a dozen or more maps, small and
// large: one launch each took 2.8 us at the median for 19 of them on the
// 432x496 backbone (116 MB, 23 us at the copy rate).
__global__ __launch_bounds__(256) void fill_zero_kernel(FillArgs a) {
    for (int c = (int)blockIdx.x; c < a.first[a.n]; c += (int)gridDim.x) {
        int lo = 0, hi = a.n;                            // the last buffer whose first chunk is <= c
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (a.first[mid] <= c) lo = mid;
            else hi = mid;
        }
        const long long n16 = a.n16[lo], at = (long long)(c - a.first[lo]) * FILL_CHUNK;
        uint4* p = static_cast<uint4*>(a.p[lo]) + at;
        const int m = (int)min((long long)FILL_CHUNK, n16 - at);
        for (int i = (int)threadIdx.x; i < m; i += 256) p[i] = make_uint4(0u, 0u, 0u, 0u);
    }
}

static unsigned grid_for(long long n) {
    long long b = (n + 255) / 256;
    if (b < 1) b = 1;
    if (b > 8192) b = 8192;
    return (unsigned)b;
}

// n = element count, a multiple of 4 (channel counts are multiples of 8).
hipError_t launch_read(const float* Z, void* dst, long long n, int relu, bool bf16, hipStream_t s) {
    const long long n4 = n / 4;
    if (bf16) hipLaunchKernelGGL(read_kernel<true>, dim3(grid_for(n4)), dim3(256), 0, s, Z, dst, n4, relu);
    else hipLaunchKernelGGL(read_kernel<false>, dim3(grid_for(n4)), dim3(256), 0, s, Z, dst, n4, relu);
    return hipGetLastError();
}

hipError_t launch_read_masked(const float* Z, void* dst, long long cells, int cout, const uint64_t* memb, int relu,
                              bool bf16, hipStream_t s) {
    const long long n4 = cells * (cout / 4);
    if (bf16)
        hipLaunchKernelGGL(read_masked_kernel<true>, dim3(grid_for(n4)), dim3(256), 0, s, Z, dst, cells, cout / 4, memb,
                           relu);
    else
        hipLaunchKernelGGL(read_masked_kernel<false>, dim3(grid_for(n4)), dim3(256), 0, s, Z, dst, cells, cout / 4,
                           memb, relu);
    return hipGetLastError();
}

// ctot a multiple of 16, at most 1024.
hipError_t launch_read_mixed(const float* Z, void* dst, long long cells, int ctot, uint64_t relu_bits, bool bf16,
                             hipStream_t s) {
    const long long n4 = cells * (ctot / 4);
    if (bf16)
        hipLaunchKernelGGL(read_mixed_kernel<true>, dim3(grid_for(n4)), dim3(256), 0, s, Z, dst, n4, ctot / 4, relu_bits);
    else
        hipLaunchKernelGGL(read_mixed_kernel<false>, dim3(grid_for(n4)), dim3(256), 0, s, Z, dst, n4, ctot / 4, relu_bits);
    return hipGetLastError();
}

bool FillList::add(void* p, size_t bytes) {
    if (!p || bytes < 16) return true;
    if (args.n == FILL_MAX) return false;
    const long long n16 = (long long)(bytes / 16);
    args.p[args.n] = p;
    args.n16[args.n] = n16;
    args.first[args.n + 1] = args.first[args.n] + (int)((n16 + FILL_CHUNK - 1) / FILL_CHUNK);
    ++args.n;
    return true;
}

hipError_t launch_fill_zero(const FillList& f, hipStream_t s) {
    const int chunks = f.args.first[f.args.n];
    if (chunks == 0) return hipSuccess;
    hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)(chunks < 4096 ? chunks : 4096)), dim3(256), 0, s, f.args);
    return hipGetLastError();
}

}  // namespace ssc
