// Dedispersion with shared partial sums (the tables and the reason: shared_sums.h).
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "shared_sums.h"
#include "spl_device.h"
#include "spl_internal.h"

namespace spl {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) const i32x4 gi32x4;
typedef __attribute__((address_space(1))) const int32_t gi32;

// Workgroup = NP wavefronts that stage and 8 that sum; work item = (beam, tile of 8*DW
// trials x 128*M samples).
//
// Staging.  A row of partial sums holds packed elements i = (y[i], y[i + 64 M]) in 16-bit
// fields, so a trial's shift of any number of samples is a shift of whole dwords and a
// wavefront reads 64 consecutive ones (no copies for odd shifts, no bank conflicts).  One
// wavefront forms 64 elements of every pattern row of a run with the matrix cores:
// rows = patterns, columns = samples, K = channels x 8 consecutive samples, A the one-hot
// choice of a sample per (pattern, channel), B the raw bytes.  Lane (n = l % 16, q =
// l / 16) holds the dwords of samples 4n .. 4n+7 of four channels; it loads the first and
// takes the second from lane n + 1 (a wave's 8-byte loads at 4-byte steps take 16 clocks,
// 32 when not dword-aligned, where a dword load takes 5).  The sums at samples 4n + j, j < 4, use the same B and A's choice j
// bytes later.  Bytes enter as signed (x - 128), the sums fall short by 128 a channel, and
// the packed element is y[i] + 65536 y[i + 64 M] as one integer; what is missing is added
// before the fields are taken apart.  Every step is exact in 32-bit integers.
//
// Summing.  Summing wavefront w owns trials DW w .. DW w + DW-1, lane l the packed samples
// l + 64 m, m < M: one LDS dword read per (trial, run, m), two runs added at a time with
// v_add3_u32 into packed accumulators.  Where the chunk table says so the fields' high
// bytes move to a second packed accumulator, before 255 + 256 channels of 255 can exceed
// 16 bits; the two halves hold sums of up to 65536 channels in half the registers of
// int32 pairs.
//
// Chunk k+1 is staged into one LDS buffer while chunk k is summed from the other, behind
// one barrier per chunk.  The staging wavefronts run through their items with the loads
// ahead: descriptors of item i+4, tables of i+3 and raw samples of i+1 and i+2 are in flight
// while item i is formed, and their waits do not hold up the summing (with all wavefronts
// doing both, the 4096-channel band ran at 127 adds per clock and CU).  Descriptors are
// vector loads, their fields read lane by lane: scalar loads return out of order with LDS
// reads, and every LDS wait would then wait for them.
template <int NP, int DW, int M, int GP>
__global__ __launch_bounds__(64 * (NP + 8)) void k_dedisp_shared(const DevBeam *__restrict__ beams,
                                                        const DedispItem *__restrict__ items, int item_lo,
                                                        int item_hi, int *queue) {
    extern __shared__ __align__(16) uint8_t lds[];
    __shared__ int s_item;
    constexpr int TD = 8 * DW, H = 64 * M;
    const int lane = lane_id(), wave = wave_id();
    // the lane number, computed where it is used: what depends on it would otherwise be
    // held in registers across the loops
    auto here = [&]() {
        uint32_t l = (uint32_t)lane;
        asm volatile("" : "+v"(l));
        return l;
    };
    auto field = [](int v, int i) { return __builtin_amdgcn_readlane(v, i); };

    int it = item_lo + blockIdx.x;
    for (;;) {
        __syncthreads();   // the previous item's last chunk is no longer read
        if (queue) {
            if (threadIdx.x == 0) s_item = item_lo + atomicAdd(queue, 1);
            __syncthreads();
            it = __builtin_amdgcn_readfirstlane(s_item);
        }
        if (it >= item_hi) break;
        const DedispItem item = items[it];
        const DevBeam &B = beams[item.beam];
        const int t0 = item.t0, d0 = item.d0;
        const uint8_t *tab = B.shared;
        const cint32 *tl = as_const((const int32_t *)tab) + 4 * (d0 / TD);
        const int buf_bytes = B.sh_buffer;

        if (wave < NP) {
            // ------------------------------------------------------------ staging
            const int nrounds = tl[1];
            const int64_t pitch = B.pitch;
            const uint8_t *x = B.x;
            const int nch = B.nch;
            const uint32_t lane_off = 2u * (lane >> 4) * (uint32_t)pitch + 4u * (lane & 15);
            const gi32 *list = (const gi32 *)(tab + B.sh_items) + ((size_t)tl[0] * NP + wave) * 8;
            const gi32 *taps = (const gi32 *)(tab + B.sh_taps);
            const gi32x4 *starts = (const gi32x4 *)(tab + B.sh_starts);
            auto load_item = [&](int r) {   // past the end: the last round's, never staged
                return (list + (size_t)min(r, nrounds - 1) * (8 * NP))[here() & 7];
            };
            auto load_start = [&](int d) { return (starts + (size_t)field(d, 0) * 4)[here() >> 4]; };
            auto load_tap = [&](int d) { return (taps + (size_t)field(d, 0) * 64)[here()]; };
            // raw[g][h][u]: the dword at 64 (group + g) + 4 n of channel u, h = 1: H samples
            // later, g <= the item's groups.  A buffer over the block from row c0 on bounds
            // the tiles at the rows' ends: what they read past a row is not needed, past the
            // block (or before it, offsets then wrap) it reads as zero.  16 rows lie within
            // 2^32 bytes (the host checks).  Groups that the item does not have load from an
            // empty buffer: with the same number of loads on every path a wait can be for
            // some of them, not all.
            auto load_raw = [&](int d, const i32x4 &start, uint32_t (&raw)[GP + 1][2][4]) {
                const int png = field(d, 1), c0 = field(d, 4);
                const int i0 = 64 * ((png >> 16) & 255) + t0, ng = png >> 24;
                const int64_t left = min((int64_t)(nch - c0) * pitch, (int64_t)0xFFFFFF00);
                // kept out of the compiler's sight: it would hold four lane offsets in
                // registers across the loop
                uint32_t step = (uint32_t)pitch;
                asm volatile("" : "+s"(step));
                uint32_t o[4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    o[u] = lane_off + (uint32_t)start[u] + (uint32_t)(8 * (u >> 1) + (u & 1)) * step + (uint32_t)i0;
#pragma unroll
                for (int g = 0; g <= GP; ++g) {
                    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                        (void *)(x + (int64_t)c0 * pitch), 0, g <= ng ? (int)(uint32_t)left : 0, 0x00027000);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        raw[g][0][u] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(o[u] + 64 * g), 0, 0);
                        raw[g][1][u] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(o[u] + H + 64 * g), 0, 0);
                    }
                }
            };
            // every pattern row's elements of the item's groups, into buffer buf
            auto stage = [&](int d, int tap, uint32_t (&raw)[GP + 1][2][4], int buf) {
                const int png = field(d, 1), rowb = field(d, 3), ng = png >> 24, np = png & 255;
                // A: channel u's choice as two dwords of bytes 0 or 1, j bytes later for j
                i32x4 a[4][2];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    uint32_t lo = __umul24(((uint32_t)tap >> (8 * u)) & 15u, 0x204081u) & 0x01010101u;
                    uint32_t hi = ((uint32_t)tap >> (8 * u + 4)) & 1u;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        a[j][u >> 1][2 * (u & 1)] = (int)lo;
                        a[j][u >> 1][2 * (u & 1) + 1] = (int)hi;
                        hi = __builtin_amdgcn_alignbyte(hi, lo, 3);
                        lo <<= 8;
                    }
                }
                const i32x4 zero = {0, 0, 0, 0};
                const int l = (int)here(), p0 = 4 * (l >> 4);
                uint8_t *dst = lds + buf * buf_bytes + field(d, 2) + p0 * rowb + 16 * (l & 15);
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int u = 0; u < 4; ++u) raw[0][h][u] ^= 0x80808080u;
#pragma unroll
                for (int g = 0; g < GP; ++g) {
                    if (g >= ng) break;
                    // B: a channel's dword and the next, which lane n + 1 holds (for n = 15
                    // lane 0 of the next group)
                    i32x4 b[2][2];
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            raw[g + 1][h][u] ^= 0x80808080u;
                            const int mine = (int)raw[g][h][u];
                            const int wrap = __builtin_amdgcn_update_dpp(0, (int)raw[g + 1][h][u], 0x12F, 15, 15, true);
                            b[h][u >> 1][2 * (u & 1)] = mine;
                            b[h][u >> 1][2 * (u & 1) + 1] = __builtin_amdgcn_update_dpp(wrap, mine, 0x101, 15, 15, false);
                        }
                    uint32_t out[4][4];   // [pattern 4q + p][element 4n + j]
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        i32x4 s0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[j][0], b[0][0], zero, 0, 0, 0);
                        i32x4 s1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[j][0], b[1][0], zero, 0, 0, 0);
                        s0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[j][1], b[0][1], s0, 0, 0, 0);
                        s1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[j][1], b[1][1], s1, 0, 0, 0);
#pragma unroll
                        for (int p = 0; p < 4; ++p) {
                            out[p][j] = (uint32_t)s0[p] + ((uint32_t)s1[p] << 16);
                            // packed here, not in the branches below: 16 registers wait, not 32
                            asm volatile("" : "+v"(out[p][j]));
                        }
                        if (j & 1) __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                    for (int p = 0; p < 4; ++p)
                        if (p0 + p < np)
                            *(uint4 *)(dst + p * rowb + 256 * g) = make_uint4(out[p][0], out[p][1], out[p][2], out[p][3]);
                }
            };

            // two sets of raw registers: while one is formed, the loads of the next item (the
            // other set) and of the one after it are on their way
            uint32_t raw0[GP + 1][2][4], raw1[GP + 1][2][4];
            int it0 = load_item(0), it1 = load_item(1), it2 = load_item(2), it3 = load_item(3);
            i32x4 start0, start1;   // of the items after the next, by turns
            int tap0, tap1;
            {
                const i32x4 s0 = load_start(it0), s1 = load_start(it1);
                load_raw(it0, s0, raw0);
                tap0 = load_tap(it0);
                __builtin_amdgcn_sched_barrier(0);
                start0 = load_start(it2);
                __builtin_amdgcn_sched_barrier(0);
                load_raw(it1, s1, raw1);
                tap1 = load_tap(it1);
                __builtin_amdgcn_sched_barrier(0);
            }
            int buf = 0;
            // loads return in order: the starts are loaded before the raw samples of the
            // round, so that waiting for them is not waiting for those
            auto round = [&](int r, uint32_t (&raw)[GP + 1][2][4], int &tap, const i32x4 &start, i32x4 &next) {
                const int ahead = load_item(r + 4);
                __builtin_amdgcn_sched_barrier(0);
                stage(it0, tap, raw, buf);
                const bool last = field(it0, 5) != 0;
                __builtin_amdgcn_sched_barrier(0);
                next = load_start(it3);
                __builtin_amdgcn_sched_barrier(0);
                load_raw(it2, start, raw);
                tap = load_tap(it2);
                __builtin_amdgcn_sched_barrier(0);
                it0 = it1;
                it1 = it2;
                it2 = it3;
                it3 = ahead;
                if (last) {
                    buf ^= 1;
                    __syncthreads();   // the chunk is staged, the one before no longer read
                }
            };
            for (int r = 0;;) {
                round(r, raw0, tap0, start0, start1);
                if (++r >= nrounds) break;
                round(r, raw1, tap1, start1, start0);
                if (++r >= nrounds) break;
            }
        } else {
            // ------------------------------------------------------------ summing
            const int nchunks = tl[3], w = wave - NP;
            const gi32 *blocks = (const gi32 *)(tab + B.sh_blocks) + ((size_t)tl[2] * 8 + w) * kSharedBlock;
            auto load_block = [&](int k) {
                return (blocks + (size_t)min(k, nchunks - 1) * (8 * kSharedBlock))[here() & (kSharedBlock - 1)];
            };
            // packed sums (t, t + H): 256 high + low, both in 16-bit fields
            uint32_t pk[DW][M], high[DW][M];
#pragma unroll
            for (int i = 0; i < DW; ++i)
#pragma unroll
                for (int m = 0; m < M; ++m) pk[i][m] = high[i][m] = 0u;
            constexpr int R = DW * M > 16 ? (M < 16 ? 16 / M : 1) : DW;   // trials read together
            int blk = load_block(0), blk1 = load_block(1);
            for (int k = 0; k < nchunks; ++k) {
                const int ahead = load_block(k + 2);
                __syncthreads();   // chunk k is staged, chunk k - 1 no longer read
                const int hdr = field(blk, 0), nsub = hdr & 255;
                const uint8_t *src = lds + (k & 1) * buf_bytes + 4 * here();
                auto load_rows = [&](int row, uint32_t (&v)[R][M]) {
#pragma unroll
                    for (int i = 0; i < R; ++i) {
                        const uint32_t *p = (const uint32_t *)(src + field(blk, 1 + row + i));
#pragma unroll
                        for (int m = 0; m < M; ++m) v[i][m] = p[64 * m];
                    }
                };
                int s = 0;
                for (; s + 2 <= nsub; s += 2) {
#pragma unroll
                    for (int i0 = 0; i0 < DW; i0 += R) {
                        uint32_t v0[R][M], v1[R][M];
                        load_rows(s * DW + i0, v0);
                        load_rows((s + 1) * DW + i0, v1);
#pragma unroll
                        for (int i = 0; i < R; ++i)
#pragma unroll
                            for (int m = 0; m < M; ++m) pk[i0 + i][m] += v0[i][m] + v1[i][m];
                    }
                }
                if (s < nsub) {
#pragma unroll
                    for (int i0 = 0; i0 < DW; i0 += R) {
                        uint32_t v0[R][M];
                        load_rows(s * DW + i0, v0);
#pragma unroll
                        for (int i = 0; i < R; ++i)
#pragma unroll
                            for (int m = 0; m < M; ++m) pk[i0 + i][m] += v0[i][m];
                    }
                }
                if (hdr >> 8) {   // channels since the high bytes last moved on
                    const uint32_t short_by = (uint32_t)(hdr >> 8) * (128u * 65537u);
#pragma unroll
                    for (int i = 0; i < DW; ++i)
#pragma unroll
                        for (int m = 0; m < M; ++m) {
                            const uint32_t v = pk[i][m] + short_by;
                            high[i][m] += (v >> 8) & 0x00FF00FFu;
                            pk[i][m] = v & 0x00FF00FFu;
                        }
                }
                blk = blk1;
                blk1 = ahead;
            }
            const int ndm = B.ndm, n_dd = B.n_dd;
#pragma unroll
            for (int i = 0; i < DW; ++i) {
                const int d = d0 + w * DW + i;
                if (d >= ndm) continue;
                int32_t *Xr = B.X + (size_t)d * B.xpitch;
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int m = 0; m < M; ++m) {
                        const int t = t0 + h * H + 64 * m + lane;
                        const uint32_t hi = h ? high[i][m] >> 16 : high[i][m] & 0xFFFFu;
                        const uint32_t lo = h ? pk[i][m] >> 16 : pk[i][m] & 0xFFFFu;
                        if (t < n_dd) Xr[t] = (int32_t)(256u * hi + lo);
                    }
            }
        }
        if (!queue) break;
    }
}

// (staging wavefronts, trials per summing wavefront, packed dwords per lane and trial, groups per item)
#define SPL_SHARED_SHAPES(X) X(4, 8, 8, 3)

bool shared_shape_supported(const SharedShape &s) {
#define SPL_X(a, b, c, d) \
    if (s.np == a && s.dw == b && s.m == c && s.gp == d) return true;
    SPL_SHARED_SHAPES(SPL_X)
#undef SPL_X
    return false;
}

template <int NP, int DW, int M, int GP>
static hipError_t prepare_t(size_t lds_bytes, int *blocks_per_cu) {
    hipError_t e = hipFuncSetAttribute((const void *)k_dedisp_shared<NP, DW, M, GP>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (e != hipSuccess) return e;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_dedisp_shared<NP, DW, M, GP>, 64 * (NP + 8),
                                                        lds_bytes);
}

hipError_t prepare_dedisp_shared(const SharedShape &s, size_t lds_bytes, int *blocks_per_cu) {
#define SPL_X(a, b, c, d) \
    if (s.np == a && s.dw == b && s.m == c && s.gp == d) return prepare_t<a, b, c, d>(lds_bytes, blocks_per_cu);
    SPL_SHARED_SHAPES(SPL_X)
#undef SPL_X
    return hipErrorInvalidValue;
}

hipError_t launch_dedisp_shared(const SharedShape &s, const DevBeam *beams, const DedispItem *items, int item_lo,
                                int item_hi, int *queue, int grid, size_t lds_bytes, hipStream_t stream) {
#define SPL_X(a, b, c, d)                                                                                           \
    if (s.np == a && s.dw == b && s.m == c && s.gp == d) {                                                          \
        hipLaunchKernelGGL((k_dedisp_shared<a, b, c, d>), dim3(grid), dim3(64 * (a + 8)), lds_bytes, stream, beams, items, \
                           item_lo, item_hi, queue);                                                                \
        return hipGetLastError();                                                                                   \
    }
    SPL_SHARED_SHAPES(SPL_X)
#undef SPL_X
    return hipErrorInvalidValue;
}

}  // namespace spl
