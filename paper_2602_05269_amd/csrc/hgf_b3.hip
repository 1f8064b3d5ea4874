// Base-3 packing of the ternary weights, five per byte (1.6 bits per weight).
//
// The HGF paper calls its backbone "1.58-bit" (Sec. 4.1, Def. "Effective Bit-Width": log2 3 bits
// per ternary weight).  The 2-bit layout of the main path spends 0.42 bits per weight on a code
// that never occurs; five ternary digits fit one byte (3^5 = 243 <= 256), which is 20 % fewer
// bytes to stream at decode, where the weights are nearly all the traffic.  The price is the
// decode: a byte no longer splits into fields with a shift and a mask.
//
// Layout.  Row n of the [d_out, d_in] matrix is ceil(d_in / 5) bytes, padded to a multiple of 16
// so that every row starts 16-byte aligned and a lane's load is 16 bytes = 80 weights of one row.
// Byte g of a row holds columns 5g .. 5g+4 as  b = sum_i (T[n, 5g+i] + 1) * 3^i ; columns past d_in count as T = 0, so
// padding bytes are 121.
//
// The kernel that reads it for a handful of tokens is the direct kernel (hgf_decode.hip).
#include "hgf_internal.h"

namespace hgf {

namespace {

constexpr int kB3Group = 5;

__host__ __device__ inline int b3_groups(int K) { return (K + kB3Group - 1) / kB3Group; }
__host__ __device__ inline int b3_row_bytes(int K) { return (b3_groups(K) + 15) / 16 * 16; }

// One thread per output byte.
__global__ __launch_bounds__(256) void pack_b3_kernel(const float *__restrict__ W, int N, int K, int Rb,
                                                      const float *__restrict__ s_w, unsigned char *__restrict__ out)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)N * Rb) return;
    const int n = (int)(i / Rb), g = (int)(i % Rb);
    const float inv = 1.0f / *s_w;
    unsigned b = 0, p3 = 1;
#pragma unroll
    for (int d = 0; d < kB3Group; ++d) {
        const int k = g * kB3Group + d;
        int t = 0;
        if (k < K) {
            float q = rintf(W[(size_t)n * K + k] * inv);
            q = fminf(fmaxf(q, -1.0f), 1.0f);
            t = (int)q;
        }
        b += (unsigned)(t + 1) * p3;
        p3 *= 3;
    }
    out[i] = (unsigned char)b;
}

__global__ __launch_bounds__(256) void unpack_b3_kernel(const unsigned char *__restrict__ packed, int N, int K, int Rb,
                                                        int8_t *__restrict__ T)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)N * K) return;
    const int n = (int)(i / K), k = (int)(i % K);
    unsigned b = packed[(size_t)n * Rb + k / kB3Group];
    for (int d = 0; d < k % kB3Group; ++d) b /= 3;
    T[i] = (int8_t)((int)(b % 3) - 1);
}

}  // namespace

size_t b3_packed_bytes(int d_out, int d_in) { return (size_t)d_out * b3_row_bytes(d_in); }

hipError_t launch_pack_b3(const float *W, int N, int K, const float *s_w, unsigned char *packed, hipStream_t st)
{
    const int Rb = b3_row_bytes(K);
    const size_t n = (size_t)N * Rb;
    hipLaunchKernelGGL(pack_b3_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, W, N, K, Rb, s_w, packed);
    return hipGetLastError();
}

hipError_t launch_unpack_b3(const unsigned char *packed, int N, int K, int8_t *T, hipStream_t st)
{
    const size_t n = (size_t)N * K;
    hipLaunchKernelGGL(unpack_b3_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, packed, N, K,
                       b3_row_bytes(K), T);
    return hipGetLastError();
}

}  // namespace hgf
