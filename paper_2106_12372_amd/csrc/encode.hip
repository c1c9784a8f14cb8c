// Input encoding kernel (Sec. 3.6 "Input Encoding", Table "parameters", and
// Sec. 5 "High-performance primitives for encoding").
//
// A workgroup of five waves takes 64 path vertices: it stages their raw records
// in LDS with 16-byte loads, wave p encodes part p of every vertex's row (a lane
// each, so no wave diverges) into LDS, and the workgroup writes the rows back
// with 16-byte stores, so both HBM streams stay fully coalesced.
//
// Large batches are bound by HBM: 56 (or 64) bytes in and 128 (FP16/BF16) or 256
// (FP32) bytes out per vertex; small ones by the latency of one vertex's
// arithmetic, which five waves share.  us, a thread per vertex before and now:
// 1,000 vertices FP16 3.2 / 2.4, BF16 unit-vector records 3.8 / 2.7; 70,001 4.8 / 4.1
// and 5.6 / 4.7; 500,003 16.5 / 15.2 (6.1 TB/s) and 18.6 / 16.8; FP32 with Gaussian
// one-blobs 500,003 36 / 25.5.
#include "encode_impl.h"

namespace nrc {
namespace {

constexpr int kEncRows = 64, kEncBlock = 5 * 64;   // vertices and threads per workgroup
constexpr int64_t kEncMax = 1 << 29;               // vertices per launch (a grid has fewer than 2^32 threads)

template <typename T> __device__ inline T to_t(float x);
template <> __device__ inline float to_t<float>(float x) { return x; }
template <> __device__ inline _Float16 to_t<_Float16>(float x) { return (_Float16)x; }
template <> __device__ inline __bf16 to_t<__bf16>(float x) { return (__bf16)x; }

template <typename T, int PRESET, int LAYOUT>
__global__ __launch_bounds__(kEncBlock) void k_encode(const float* __restrict__ raw, int64_t n,
                                                      T* __restrict__ enc) {
    constexpr int RW = LAYOUT == NRC_RAW14 ? 14 : 16;
    constexpr int ROW = 64 + 16 / (int)sizeof(T);                            // padded LDS row, elements
    constexpr int EPC = 16 / (int)sizeof(T), CPR = 64 / EPC;                 // 16-byte chunks: elements, per row
    __shared__ __attribute__((aligned(16))) float sraw[kEncRows * RW];
    __shared__ __attribute__((aligned(16))) T sout[kEncRows * ROW];
    const int64_t base = (int64_t)blockIdx.x * kEncRows;
    const int nrows = (int)min((int64_t)kEncRows, n - base);
    const float* src = raw + base * RW;
    const int nf = nrows * RW;
    const int nf4 = nf >> 2;
    for (int i = threadIdx.x; i < nf4; i += kEncBlock)
        reinterpret_cast<float4*>(sraw)[i] = reinterpret_cast<const float4*>(src)[i];
    for (int i = (nf4 << 2) + threadIdx.x; i < nf; i += kEncBlock) sraw[i] = src[i];
    __syncthreads();
    const int r = threadIdx.x & 63, part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (r < nrows) {
        const float* x = sraw + r * RW;
        T* o = sout + r * ROW;
        float f[64];
        auto put = [&](auto first, auto past) {
            typedef T t4 __attribute__((ext_vector_type(4)));
            #pragma unroll
            for (int k = decltype(first)::value; k < decltype(past)::value; ++k)
                if (__is_same(T, _Float16)) asm("" : "+v"(f[k]));   // a product is rounded to FP32 first
            #pragma unroll
            for (int k = decltype(first)::value; k < decltype(past)::value; k += 4)
                *reinterpret_cast<t4*>(o + k) = t4{to_t<T>(f[k]), to_t<T>(f[k + 1]), to_t<T>(f[k + 2]), to_t<T>(f[k + 3])};
        };
        if (part == 0) {
            encode_part<PRESET, LAYOUT, 0>(x, f);
            put(IntC<0>{}, IntC<12>{});
        } else if (part == 1) {
            encode_part<PRESET, LAYOUT, 1>(x, f);
            put(IntC<12>{}, IntC<24>{});
        } else if (part == 2) {
            encode_part<PRESET, LAYOUT, 2>(x, f);
            put(IntC<24>{}, IntC<36>{});
        } else if (part == 3) {
            encode_part<PRESET, LAYOUT, 3>(x, f);
            put(IntC<36>{}, IntC<44>{});
        } else {
            encode_part<PRESET, LAYOUT, 4>(x, f);
            put(IntC<44>{}, IntC<64>{});
        }
    }
    __syncthreads();
    T* dst = enc + base * 64;
    for (int i = threadIdx.x; i < nrows * CPR; i += kEncBlock) {
        const int rr = i / CPR, cc = i - rr * CPR;
        const uint4 v = *reinterpret_cast<const uint4*>(sout + rr * ROW + cc * EPC);
        *reinterpret_cast<uint4*>(dst + (int64_t)rr * 64 + cc * EPC) = v;
    }
}

template <typename T>
hipError_t dispatch_encode(int preset, int layout, const float* raw, int64_t n, T* enc,
                           hipStream_t s) {
#define NRC_ENC_LAUNCH(PR, LA)                                                                                    \
    for (int64_t at = 0; at < n; at += kEncMax) {                                                                 \
        const int64_t k = n - at < kEncMax ? n - at : kEncMax;                                                    \
        hipLaunchKernelGGL((k_encode<T, PR, LA>), dim3((unsigned)((k + kEncRows - 1) / kEncRows)), dim3(kEncBlock), \
                           0, s, raw + at * (LA == NRC_RAW14 ? 14 : 16), k, enc + at * 64);                       \
    }
#define NRC_ENC_LAYOUT(PR)             \
    if (layout == NRC_RAW14) {         \
        NRC_ENC_LAUNCH(PR, NRC_RAW14)  \
    } else {                           \
        NRC_ENC_LAUNCH(PR, NRC_RAW16)  \
    }
    if (preset == NRC_PRESET_PAPER_GAUSS) {
        NRC_ENC_LAYOUT(NRC_PRESET_PAPER_GAUSS)
    } else if (preset == NRC_PRESET_PAPER_TRI) {
        NRC_ENC_LAYOUT(NRC_PRESET_PAPER_TRI)
    } else if (preset == NRC_PRESET_PAPER) {
        NRC_ENC_LAYOUT(NRC_PRESET_PAPER)
    } else {
        NRC_ENC_LAYOUT(NRC_PRESET_CONFIG)
    }
#undef NRC_ENC_LAYOUT
#undef NRC_ENC_LAUNCH
    return n > 0 ? hipGetLastError() : hipSuccess;
}

}  // namespace

hipError_t launch_encode(int precision, int preset, int layout, const float* raw, int64_t n,
                         void* enc, hipStream_t s) {
    switch (precision) {
        case NRC_FP32:
        case NRC_FP32_VALU: return dispatch_encode<float>(preset, layout, raw, n, (float*)enc, s);
        case NRC_FP16: return dispatch_encode<_Float16>(preset, layout, raw, n, (_Float16*)enc, s);
        default: return dispatch_encode<__bf16>(preset, layout, raw, n, (__bf16*)enc, s);
    }
}

}  // namespace nrc
