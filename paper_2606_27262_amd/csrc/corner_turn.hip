// Corner turn of a filterbank block: time-major samples [n_t][nch] (the SIGPROC order,
// one byte per sample) to the channel-major rows [nch][pitch] the dedispersion reads.
// Pure data movement, bound by HBM: each byte is read once and written once.
//
// A workgroup moves a tile of 128 samples x 128 channels through the LDS: 16-byte global
// loads along channels (eight threads read a sample's 128 bytes), then each thread takes
// 16 consecutive samples of four channels as dwords, transposes them 4 x 4 bytes at a time
// and writes four 16-byte pieces (byte by byte from the LDS, a 4096 x 26305 block that lay in the
// last-level cache took 38.3 us, now 34.2; from HBM it takes 51.6 us either way); eight neighbouring threads cover a row's 128 samples, so reads and writes both move
// 128-byte pieces.  (Measured on a 4096 x 26305 block against 64 x 256, 128 x 256,
// 64 x 512 and 256 x 128 tiles: the fastest, 73 % of a plain device copy's rate.)  The
// LDS row stride of 132 bytes spreads a wave's gathers over the banks (2-way at most).
#include <hip/hip_runtime.h>

#include "corner_turn.h"

namespace spl {

namespace {
constexpr int kTT = 128;      // samples per tile
constexpr int kTC = 128;      // channels per tile
constexpr int kStride = 132;  // LDS bytes per sample row of the tile
constexpr int kVecRow = kTC / 16;    // 16-byte vectors per sample row
constexpr int kParts = kTT / 16;     // 16-sample parts per channel row
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
}  // namespace

__global__ __launch_bounds__(256) void k_corner_turn(const uint8_t *__restrict__ in, int64_t in_stride, int64_t n_t,
                                                     int nch, uint8_t *__restrict__ out, int64_t pitch) {
    __shared__ __align__(16) uint8_t tile[kTT * kStride];
    const int tid = threadIdx.x;
    const int64_t t0 = (int64_t)blockIdx.x * kTT;
    const int c0 = blockIdx.y * kTC;
#pragma unroll
    for (int q = 0; q < kTT * kVecRow / 256; ++q) {
        const int idx = q * 256 + tid;
        const int r = idx / kVecRow, c16 = (idx % kVecRow) * 16;
        const int64_t t = t0 + r;
        u32x4 v = {0u, 0u, 0u, 0u};
        if (t < n_t && c0 + c16 < nch) v = *(const u32x4 *)(in + t * in_stride + c0 + c16);
        uint32_t *d = (uint32_t *)(tile + r * kStride + c16);
        d[0] = v.x;
        d[1] = v.y;
        d[2] = v.z;
        d[3] = v.w;
    }
    __syncthreads();
    // the thread's 16 samples of 4 channels, transposed 4 x 4 bytes at a time
    static_assert(kTC / 4 * kParts == 256, "one (part, 4 channels) a thread");
    const int part = tid % kParts, c = 4 * (tid / kParts);
    uint32_t w[4][4];   // [channel][4 samples]
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint8_t *s = tile + (part * 16 + 4 * k) * kStride + c;
        const uint32_t s0 = *(const uint32_t *)s, s1 = *(const uint32_t *)(s + kStride),
                       s2 = *(const uint32_t *)(s + 2 * kStride), s3 = *(const uint32_t *)(s + 3 * kStride);
        const uint32_t a0 = __builtin_amdgcn_perm(s1, s0, 0x05010400u), a1 = __builtin_amdgcn_perm(s1, s0, 0x07030602u);
        const uint32_t b0 = __builtin_amdgcn_perm(s3, s2, 0x05010400u), b1 = __builtin_amdgcn_perm(s3, s2, 0x07030602u);
        w[0][k] = __builtin_amdgcn_perm(b0, a0, 0x05040100u);
        w[1][k] = __builtin_amdgcn_perm(b0, a0, 0x07060302u);
        w[2][k] = __builtin_amdgcn_perm(b1, a1, 0x05040100u);
        w[3][k] = __builtin_amdgcn_perm(b1, a1, 0x07060302u);
    }
    const int64_t t = t0 + part * 16;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (c0 + c + i >= nch) continue;
        uint8_t *dst = out + (int64_t)(c0 + c + i) * pitch + t;
        if (t + 16 <= n_t) {
            const u32x4 v = {w[i][0], w[i][1], w[i][2], w[i][3]};
            *(u32x4 *)dst = v;
        } else {
#pragma unroll
            for (int j = 0; j < 16; ++j)
                if (t + j < n_t) dst[j] = (uint8_t)(w[i][j >> 2] >> (8 * (j & 3)));
        }
    }
}

hipError_t launch_corner_turn(const uint8_t *in, int64_t in_stride, int64_t n_t, int nch, uint8_t *out, int64_t pitch,
                              hipStream_t s) {
    if (n_t <= 0 || nch <= 0) return hipSuccess;
    const int64_t gx = (n_t + kTT - 1) / kTT;
    const int gy = (nch + kTC - 1) / kTC;
    if (gx > 0x7fffffff || gy > 65535) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_corner_turn, dim3((unsigned)gx, (unsigned)gy), dim3(256), 0, s, in, in_stride, n_t, nch, out,
                       pitch);
    return hipGetLastError();
}

}  // namespace spl
