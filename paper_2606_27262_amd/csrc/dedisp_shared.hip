// Dedispersion with shared partial sums (the tables and the reason: shared_sums.h).
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "shared_sums.h"
#include "spl_device.h"
#include "spl_internal.h"

namespace spl {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const i32x4 gi32x4;
typedef __attribute__((address_space(1))) const int32_t gi32;
typedef __attribute__((address_space(3))) uint8_t lu8;
typedef __attribute__((address_space(3))) i32x4 li32x4;

template <int I>
struct Int {
    static constexpr int value = I;
};
template <int N, int I = 0, typename F>
static __device__ __forceinline__ void each(F &&f) {
    if constexpr (I < N) {
        f(Int<I>{});
        each<N, I + 1>(f);
    }
}

// lane 15 of every 16 takes lane K of its 16 (the others, lanes that the caller does not use)
template <int K>
static __device__ __forceinline__ int to_last(uint32_t v) {
    return __builtin_amdgcn_update_dpp(0, (int)v, 0x120 + 15 - K, 15, 15, true);
}

// Workgroup = NP wavefronts that stage and 8 that sum; work item = (beam, tile of 8*DW
// trials x 128*M samples).
//
// Staging.  A row of partial sums holds packed elements i = (y[i], y[i + 64 M]) in 16-bit
// fields, so a trial's shift of any number of samples is a shift of whole dwords and a
// wavefront reads 64 consecutive ones (no copies for odd shifts, no bank conflicts).  One
// wavefront forms 64 elements of every pattern row of a run with the matrix cores: columns =
// dwords of four samples, K = channels x 8 consecutive samples, B the raw bytes, rows =
// 4 patterns x the 4 elements of a dword, A the one-hot choice of a sample per (pattern,
// channel), moved on by the element.  So lane (n = l % 16, q = l / 16) ends with elements
// 4n .. 4n+3 of pattern 4k + q, in the order of its 16-byte LDS write.  It holds the dwords
// of samples 4n .. 4n+7 of four channels; it loads the first and takes the second from lane
// n + 1 (a wave's 8-byte loads at 4-byte steps take 16 clocks, 32 when not dword-aligned,
// where a dword load takes 5).  Bytes enter as signed (x - 128), the sums fall short by 128 a
// channel, and the packed element is y[i] + 65536 y[i + 64 M] as one integer; what is missing
// is added before the fields are taken apart.  Every step is exact in 32-bit integers.
//
// A SIMD has one staging wavefront, which issues some 75 instructions per 64 elements, so its
// chain of waits sets the pace: the next group's operands are made between the matrix
// products, the packing of a quarter of the sums waits for the next quarter's products, and
// items are long (5 groups of 64 elements on average; two runs share a chunk, so that their
// groups divide well), as an item costs as much as a group to begin.  With 3 groups an item
// and each step waiting for the one before it, 8 beams of the 4096-channel band took 10.4 ms
// in this kernel; now 7.4 ms (242 adds per clock and CU; the row-staging kernel: 37 ms).
// What bounds it now is still the staging (650 clocks a group, 300 if it issued every 4th): of
// 24 beams' 22.9 ms the LDS is active in 50 % (reads of 8 summing wavefronts mostly, 11.6 ms by
// themselves), vector instructions are issued in 54 %, the matrix cores are busy in 25 %, and
// 45 GB move to and from memory, 2.0 TB/s (counted).
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
// ahead: descriptors of item i+3, tables of i+1 and i+2 and the raw samples of the RS groups
// ahead are in flight while a group is formed, and their waits do not hold up the summing
// (with all wavefronts doing both, the 4096-channel band ran at 127 adds per clock and CU).
// Descriptors are vector loads, their fields read lane by lane: scalar loads return out of
// order with LDS reads, and every LDS wait would then wait for them.
template <int NP, int DW, int M, int GP, int RS>
__global__ __launch_bounds__(64 * (NP + 8)) void k_dedisp_shared(const DevBeam *__restrict__ beams,
                                                        const DedispItem *__restrict__ items, int item_lo,
                                                        int item_hi, int *queue) {
    extern __shared__ __align__(16) uint8_t lds[];
    __shared__ int s_item;
    constexpr int TD = 8 * DW, H = 64 * M;
    const int wave = wave_id();
    // the lane number, computed where it is used: what depends on it would otherwise be
    // held in registers across the loops
    auto here = [&]() {
        uint32_t none = 0;
        asm volatile("" : "+s"(none));
        return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, none)) & 63u;
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
        const uint8_t *tab = B.tables;
        const cint32 *tl = as_const((const int32_t *)tab) + 4 * (d0 / TD);
        const int buf_bytes = B.sh_buffer;

        if (wave < NP) {
            // ------------------------------------------------------------ staging
            const int nrounds = tl[1];
            const uint32_t pitch = (uint32_t)B.pitch;   // 16 rows lie within 2^32 bytes (the host checks)
            const uint8_t *x = B.x;
            const int nch = B.nch;
            const gi32 *list = (const gi32 *)(tab + B.sh_items) + ((size_t)tl[0] * NP + wave) * 8;
            const gi32x4 *taps = (const gi32x4 *)(tab + B.sh_taps);
            const gi32x4 *starts = (const gi32x4 *)(tab + B.sh_starts);
            auto load_item = [&](int r, uint32_t l) {   // past the end: the last round's, never staged
                return (list + (uint32_t)min(r, nrounds - 1) * (8u * NP))[l & 7];
            };
            auto load_start = [&](int d, uint32_t l) { return (starts + (uint32_t)field(d, 0) * 4u)[l >> 4]; };
            auto load_tap = [&](int d, uint32_t l) { return (taps + (uint32_t)field(d, 0) * 16u)[l >> 2]; };
            // raw[g][h][u]: the dword at 64 (group + g) + 4 n of channel u, h = 1: H samples
            // later, g up to the item's groups.  A buffer over the block from row c0 on bounds
            // the tiles at the rows' ends: what they read past a row is not needed, past the
            // block it reads as zero.  Before the block's first sample (starts of -4 or -8, at
            // t = 0) nothing is needed, but an offset that wraps must not be brought back by an
            // instruction's own offset: offsets are held for the second group, and the first's
            // are cut off at zero.  Groups that the item does not have load from an
            // empty buffer: with the same number of loads on every path a wait can be for
            // some of them, not all.
            struct Rows { const uint8_t *base; uint32_t bytes; int groups; };
            const uint64_t block_bytes = (uint64_t)nch * pitch;
            auto rows_of = [&](int d) {
                const uint64_t at = (uint64_t)(uint32_t)field(d, 4) * pitch, left = block_bytes - at;
                Rows w{x + at, left >> 32 ? 0xFFFFFFFFu : (uint32_t)left, field(d, 1) >> 24};
                // held, not computed again for every group
                asm volatile("" : "+s"(w.base), "+s"(w.bytes), "+s"(w.groups));
                return w;
            };
            auto load_raw = [&](const Rows &w, int g, const uint32_t (&o)[4], uint32_t (&raw)[2][4]) {
                const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                    (void *)w.base, 0, g <= w.groups ? (int)w.bytes : 0, 0x00027000);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int at = (int)(g > 0 ? o[u] + 64 * (g - 1) : o[u] - min(o[u], 64u));
                    raw[0][u] = __builtin_amdgcn_raw_buffer_load_b32(rs, at, 0, 0);
                    raw[1][u] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(o[u] + H - 64 + 64 * g), 0, 0);
                }
            };
            auto raw_offsets = [&](int d, const i32x4 &start, uint32_t l, uint32_t (&o)[4]) {
                const uint32_t i1 = (uint32_t)(64 * ((field(d, 1) >> 16) & 255) + t0 + 64);
                // kept out of the compiler's sight: it would hold four lane offsets in
                // registers across the loop
                uint32_t step = pitch;
                asm volatile("" : "+s"(step));
                const uint32_t lane_off = 2u * (l >> 4) * step + 4u * (l & 15);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    o[u] = lane_off + (uint32_t)start[u] + (uint32_t)(8 * (u >> 1) + (u & 1)) * step + i1;
            };

            // the dwords after an item's GP groups, those of (h, u) in lane n = 4 h + u
            auto load_edge = [&](const Rows &w, uint32_t l, const uint32_t (&o)[4]) {
                const __amdgpu_buffer_rsrc_t rs =
                    __builtin_amdgcn_make_buffer_rsrc((void *)w.base, 0, GP <= w.groups ? (int)w.bytes : 0, 0x00027000);
                uint32_t at = o[0];   // of channel l & 3
#pragma unroll
                for (int u = 1; u < 4; ++u) {
                    const uint32_t ou = o[u];
                    at = (l & 3) == (uint32_t)u ? ou : at;
                }
                return __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(at - 4u * (l & 15) + (l & 4 ? H : 0) + 64u * (GP - 1)), 0, 0);
            };

            // RS groups' raw samples in registers: group g's are replaced as soon as it is formed
            // by those of group g + RS, of this item or of the next.  Loads return in order: the
            // tables of the next items are loaded ahead of the raw samples.
            uint32_t raw[RS][2][4], edge, o[4];
            const uint32_t l0 = here();
            int it0 = load_item(0, l0), it1 = load_item(1, l0), it2 = load_item(2, l0);
            i32x4 start = load_start(it1, l0), tap = load_tap(it0, l0);
            raw_offsets(it0, load_start(it0, l0), l0, o);
            Rows here_rows = rows_of(it0), next_rows;
            __builtin_amdgcn_sched_barrier(0);   // the order of the loop's loads, for the counts of its waits
            edge = load_edge(here_rows, l0, o);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < RS; ++g) {
                load_raw(here_rows, g, o, raw[g]);
                __builtin_amdgcn_sched_barrier(0);
            }
            int buf = 0;
            for (int r = 0; r < nrounds; ++r) {
                const int png = field(it0, 1), rowb = field(it0, 3), ng = png >> 24, np = png & 255;
                // A, rows 4 p + j of pattern 4 k + p: channel u's choice, a one-hot byte of 8
                i32x4 a[4][2];
                const uint32_t l = here();
                const uint32_t later = (l & 3) * 0x208208u;   // 8 j in every field
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const uint64_t one = ((uint32_t)tap[0] >> (24 + u)) & 1u;   // 0: no such channel in the run
                        const uint64_t hot = one << ((((uint32_t)tap[k] + later) >> (6 * u)) & 63u);
                        a[k][u >> 1][2 * (u & 1)] = (int)(uint32_t)hot;
                        a[k][u >> 1][2 * (u & 1) + 1] = (int)(uint32_t)(hot >> 32);
                    }
                lu8 *dst[4];   // of the rows of pattern 4 k + l / 16; past the last: the last's
                {
                    uint8_t *base = lds + buf * buf_bytes + field(it0, 2) + 16u * (l & 15);
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        dst[k] = (lu8 *)base + (uint32_t)min(4 * k + (int)(l >> 4), np - 1) * (uint32_t)rowb;
                        asm volatile("" : "+v"(dst[k]));
                    }
                }
                const uint32_t edge_now = edge;
                uint32_t flip = 0x80808080u;   // in a register, as an operand beside a lane shift
                asm volatile("" : "+v"(flip));
                __builtin_amdgcn_sched_barrier(0);
                const int ahead = load_item(r + 3, l);
                tap = load_tap(it1, l);
                const i32x4 start_now = start;
                start = load_start(it2, l);
                __builtin_amdgcn_sched_barrier(0);
                const i32x4 zero = {0, 0, 0, 0};
                // B of group g, operand i = (channel u, half h): the channel's dword and the next,
                // which lane n + 1 holds (for n = 15 lane 0 of the next group).  The shift of a
                // register takes two instructions' distance from its writing.
                auto dwords = [&](auto gc, auto ic, i32x4 (&b)[2][2]) {
                    constexpr int g = decltype(gc)::value, h = decltype(ic)::value % 2, u = decltype(ic)::value / 2;
                    int wrap;
                    if constexpr (g + 1 < GP)
                        wrap = to_last<0>(raw[(g + 1) % RS][h][u]);
                    else
                        wrap = to_last<4 * h + u>(edge_now);
                    b[h][u >> 1][2 * (u & 1)] = (int)(raw[g % RS][h][u] ^ flip);
                    b[h][u >> 1][2 * (u & 1) + 1] = wrap ^ (int)flip;
                };
                auto shift = [&](auto ic, i32x4 (&b)[2][2]) {
                    constexpr int h = decltype(ic)::value % 2, u = decltype(ic)::value / 2;
                    b[h][u >> 1][2 * (u & 1) + 1] = __builtin_amdgcn_update_dpp(
                        b[h][u >> 1][2 * (u & 1) + 1], b[h][u >> 1][2 * (u & 1)], 0x101, 15, 15, false);
                };
                i32x4 b[2][2][2];
                each<8>([&](auto i) { dwords(Int<0>{}, i, b[0]); });
                each<8>([&](auto i) { shift(i, b[0]); });
                // sums of rows 4 k + p (k by turns), packed and written while the next are formed
                i32x4 s0[2], s1[2];
                auto pack = [&](int k, int half, i32x4 &out) {
                    out[half] = (int)((uint32_t)s0[k & 1][half] + ((uint32_t)s1[k & 1][half] << 16));
                    out[half + 1] = (int)((uint32_t)s0[k & 1][half + 1] + ((uint32_t)s1[k & 1][half + 1] << 16));
                };
                // given some value here: else the registers would be taken as kept from the loop's
                // last turn, through the summing branch too
                asm volatile("" : "=v"(b[1][0][0]), "=v"(b[1][0][1]), "=v"(b[1][1][0]), "=v"(b[1][1][1]), "=v"(s0[1]), "=v"(s1[1]));
                __builtin_amdgcn_sched_barrier(0);
                each<GP>([&](auto gc) {
                    constexpr int g = decltype(gc)::value;
                    if (g < ng) {
                        const i32x4 (&bg)[2][2] = b[g & 1];
                        i32x4 (&bn)[2][2] = b[(g + 1) & 1];
                        // between the products of quarter k: the next group's operands 2 k and
                        // 2 k + 1, the packing of quarter k - 1 (of the last one, a group later)
                        each<4>([&](auto kc) {
                            constexpr int k = decltype(kc)::value;
                            i32x4 out;
                            s0[k & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[k][0], bg[0][0], zero, 0, 0, 0);
                            if constexpr (g + 1 < GP) {
                                dwords(Int<g + 1>{}, Int<2 * k>{}, bn);
                                if constexpr (k > 0) shift(Int<2 * k - 1>{}, bn);
                            }
                            __builtin_amdgcn_sched_barrier(0);
                            s1[k & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[k][0], bg[1][0], zero, 0, 0, 0);
                            if constexpr (g + 1 < GP) {
                                dwords(Int<g + 1>{}, Int<2 * k + 1>{}, bn);
                                shift(Int<2 * k>{}, bn);
                            }
                            __builtin_amdgcn_sched_barrier(0);
                            s0[k & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[k][1], bg[0][1], s0[k & 1], 0, 0, 0);
                            if constexpr (g > 0 || k > 0) pack(k + 3, 0, out);
                            if constexpr (g + 1 < GP && k == 3) shift(Int<7>{}, bn);
                            __builtin_amdgcn_sched_barrier(0);
                            s1[k & 1] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[k][1], bg[1][1], s1[k & 1], 0, 0, 0);
                            if constexpr (g > 0 || k > 0) {
                                pack(k + 3, 2, out);
                                *(li32x4 *)(dst[(k + 3) & 3] + 256 * (k > 0 ? g : g - 1)) = out;
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        });
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if (g == GP - RS) {
                        const uint32_t ln = here();
                        raw_offsets(it1, start_now, ln, o);
                        next_rows = rows_of(it1);
                        edge = load_edge(next_rows, ln, o);
                    }
                    load_raw(g < GP - RS ? here_rows : next_rows, g < GP - RS ? g + RS : g + RS - GP, o, raw[g % RS]);
                    __builtin_amdgcn_sched_barrier(0);
                });
                if (ng > 0) {
                    i32x4 out;
                    pack(3, 0, out);
                    pack(3, 2, out);
                    *(li32x4 *)(dst[3] + 256 * (ng - 1)) = out;
                }
                const bool last = field(it0, 5) != 0;
                it0 = it1;
                it1 = it2;
                it2 = ahead;
                here_rows = next_rows;
                if (last) {
                    buf ^= 1;
                    __syncthreads();   // the chunk is staged, the one before no longer read
                }
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
                        const int t = t0 + h * H + 64 * m + (int)here();
                        const uint32_t hi = h ? high[i][m] >> 16 : high[i][m] & 0xFFFFu;
                        const uint32_t lo = h ? pk[i][m] >> 16 : pk[i][m] & 0xFFFFu;
                        if (t < n_dd) Xr[t] = (int32_t)(256u * hi + lo);
                    }
            }
        }
        if (!queue) break;
    }
}

// (staging wavefronts, trials per summing wavefront, packed dwords per lane and trial, groups per item, of raw samples held)
#define SPL_SHARED_SHAPES(X) X(4, 8, 8, 6, 6)

template <int NP, int DW, int M, int GP, int RS>
static hipError_t prepare_t(size_t lds_bytes, int *blocks_per_cu) {
    hipError_t err = hipFuncSetAttribute((const void *)k_dedisp_shared<NP, DW, M, GP, RS>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (err != hipSuccess) return err;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_dedisp_shared<NP, DW, M, GP, RS>, 64 * (NP + 8),
                                                        lds_bytes);
}

hipError_t prepare_dedisp_shared(const SharedShape &s, size_t lds_bytes, int *blocks_per_cu) {
#define SPL_X(a, b, c, d, e) \
    if (s.np == a && s.dw == b && s.m == c && s.gp == d) return prepare_t<a, b, c, d, e>(lds_bytes, blocks_per_cu);
    SPL_SHARED_SHAPES(SPL_X)
#undef SPL_X
    return hipErrorInvalidValue;
}

hipError_t launch_dedisp_shared(const SharedShape &s, const DevBeam *beams, const DedispItem *items, int item_lo,
                                int item_hi, int *queue, int grid, size_t lds_bytes, hipStream_t stream) {
#define SPL_X(a, b, c, d, e)                                                                                           \
    if (s.np == a && s.dw == b && s.m == c && s.gp == d) {                                                          \
        hipLaunchKernelGGL((k_dedisp_shared<a, b, c, d, e>), dim3(grid), dim3(64 * (a + 8)), lds_bytes, stream, beams, items, \
                           item_lo, item_hi, queue);                                                                \
        return hipGetLastError();                                                                                   \
    }
    SPL_SHARED_SHAPES(SPL_X)
#undef SPL_X
    return hipErrorInvalidValue;
}

}  // namespace spl
