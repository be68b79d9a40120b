// HIP kernels (gfx950) of the single-pulse search hot path.
//
//  k_dedisp      brute-force incoherent dedispersion (dedispersion section, Eq. (1)
//                delays) into the int32 DM transform, rows staged in the LDS;
//  k_dedisp_direct  the same without staging, for small or coarse plans
//  k_thresholds  exact moments, mean / sigma per (DM row, segment) and the smallest
//                boxcar sum reaching the S/N threshold per width (single pulse search)
//  k_boxcar      boxcar filters via wrapping 32-bit prefix sums, threshold test, best
//                width; writes the hits in (row, t) order, each tile's offset found by
//                decoupled look-back over the tiles before it
//  k_rows        row starts and block index of a hit list
//  k_nms         peak filter over the sorted hit list (3x3, then 11x11 windows)
//  k_survivors   its survivors in order: the next list, or candidate records
//
// All integer work is exact; binary64 is evaluated with contraction disabled so
// every rounding is the one written in the expression.
#include <hip/hip_runtime.h>
#include <limits.h>

#include "kernels.h"
#include "spl_device.h"
#include "spl_internal.h"

#pragma clang fp contract(off)

namespace spl {

__device__ __forceinline__ int beam_of_chunk(const DevBeam *beams, int lo, int hi, int g) {
    int b = lo;
    while (b + 1 < hi && beams[b + 1].chunk_base <= g) ++b;
    return b;
}
__device__ __forceinline__ int beam_of_row(const DevBeam *beams, int lo, int hi, int r) {
    int a = lo, z = hi - 1;   // largest b with row_base <= r
    while (a < z) {
        int m = (a + z + 1) >> 1;
        if (beams[m].row_base <= r) a = m; else z = m - 1;
    }
    return a;
}

// ------------------------------------------------------------------- fill
// Zeroes up to three ranges of words in one launch (the start of a run).
__global__ void k_clear(uint64_t *a, int64_t na, uint64_t *b, int64_t nb, uint64_t *c, int64_t nc) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < na + nb + nc; i += stride) {
        if (i < na) a[i] = 0;
        else if (i < na + nb) b[i - na] = 0;
        else c[i - na - nb] = 0;
    }
}

// ------------------------------------------------------------- dedispersion
// Workgroup = NW wavefronts; item = (beam, DM tile of NW*DW trials, time tile of 256*J
// samples).  Wavefront w owns DM trials d0 + w*DW ... + DW-1; lane l owns samples
// t0 + 256 j + 4 l + {0,1,2,3}, j < J.
//
// Channels are staged chan_chunk at a time.  Row r of the LDS holds channel c from
// ws_c = t0 + (tile_base_c & ~15) (16-aligned start of the tile's smallest delay) in
// four copies, copy k shifted by k bytes (copy k, byte i = sample ws_c + k + i), so that
// the 4 samples a lane needs for any delay s are one aligned dword of copy s & 3, at
// byte ((s - ws_c + t0) & ~3) + (s & 3)*quarter of the row.  That offset is precomputed
// per (channel, trial) in the plan table; the chunk's slice of the table is staged in
// LDS with the samples.  Per (trial, channel) a lane does one address add, per 256
// samples one dword read (lanes read consecutive dwords: conflict-free, paired into
// ds_read2st64_b32), and a v_perm that spreads bytes (t+1, t+3) into 16-bit fields; these
// and the dwords as they are (carries between the bytes included) are summed for two
// channels at a time with v_add3_u32.  Bytes (t, t+2) are what is left of the sum of the
// dwords less 256 times the fields, exact for up to 256 channels; then both are widened
// into int32 accumulators.  That is 4 instructions for 8 sums; spreading both pairs of
// bytes took 6.  Registers are held to 128, so that a CU has 16 wavefronts of 4 SIMDs: the
// 8-wavefront tiles of 256 x 2 samples took 131 and 145, and one workgroup a CU then
// neither staged nor summed while it waited at its barriers (two beams of the 2048-channel
// 300-500 MHz band: 12.1 ms in this kernel, 11.4 with fewer sums' instructions, 7.2 with
// two workgroups a CU).  Of the shapes that would take more, (4,2,8) then spills 3 registers,
// (4,2,8) with two vectors a row 14 and (8,1,8) 1, and all are faster for it: 4 x 512 trials x
// 1024 channels x 16384 samples take (4,2,8) 0.99 ms (1.45 unbounded), with long rows 1.55
// (2.07), (8,1,8) 1.18 (1.73), (8,1,4) 1.47 (1.55), (4,2,4) 1.26 (1.35).  The LDS loads of the next
// channel are in flight while the current one is summed, and the global loads of the
// next chunk while the current chunk is summed.
// SV: 16-byte input vectors staged per lane and row (rows of up to 1024*SV bytes).
// NBUF: LDS buffers.  With one, every chunk is staged between two barriers while no
// wavefront sums.  With two (chunks of at most NW channels, one staged row per
// wavefront), chunk k+1 is staged into the other buffer while chunk k is summed, behind
// one barrier per chunk; half of the wavefronts stage before summing and half after,
// so that the LDS writes and byte shifts of some wavefronts fall in the LDS waits of
// the others (wavefronts w with w/4 odd stage first: with wavefronts dealt to the four
// SIMDs in turn, each SIMD holds two of each kind).
// Each wavefront stages up to dedisp_stage_rows(NBUF) rows per chunk.
template <int DW, int J, int NW, int SV, int NBUF>
__global__ __launch_bounds__(64 * NW, 4) void k_dedisp(const DevBeam *__restrict__ beams,
                                                    const DedispItem *__restrict__ items,
                                                    int item_lo, int item_hi, int *queue) {
    extern __shared__ __align__(16) uint8_t lds[];
    __shared__ int s_item;
    const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
    constexpr int TD = NW * DW;
    static_assert(NBUF == 1 || NBUF == 2, "one or two LDS buffers");
    constexpr int kStageRows = dedisp_stage_rows(NBUF);
    constexpr int kStageVecs = SV;
    constexpr int kTabRows = kStageRows * NW + 4;   // chan_chunk rows + 4 rows of prefetch padding
    constexpr int kTabRegs = (kTabRows * TD + 64 * NW - 1) / (64 * NW);
    constexpr uint32_t kSelOdd = 0x0C030C01u;    // bytes 1, 3 -> 16-bit fields

    int it = item_lo + blockIdx.x;
    for (;;) {
        if (queue) {
            __syncthreads();
            if (tid == 0) s_item = item_lo + atomicAdd(queue, 1);
            __syncthreads();
            it = __builtin_amdgcn_readfirstlane(s_item);
        }
        if (it >= item_hi) break;

        const DedispItem item = items[it];
        const DevBeam &B = beams[item.beam];
        const int nch = B.nch, ndm_pad = B.ndm_pad, R = item.row_bytes, quarter = B.lds_quarter;
        const int t0 = item.t0, d0 = item.d0;
        const int32_t *__restrict__ tab = (const int32_t *)B.tables;
        const int32_t *__restrict__ base = B.tile_base + (size_t)(d0 / B.tile_dm) * nch;
        const int64_t pitch = B.pitch;
        const uint8_t *__restrict__ x = B.x;
        const int cchunk = B.chan_chunk;
        const int nvec = R >> 4;   // 16-byte vectors per row and copy
        // buffer b: four copies of chan_chunk + 1 rows, then its slice of the offset table
        const int buf_bytes = 4 * quarter + kTabRows * TD * 4;

        int32_t acc[DW][4 * J];
        uint32_t aw[DW][J], ao[DW][J];   // sums of the dwords, of their bytes 1 and 3
#pragma unroll
        for (int i = 0; i < DW; ++i) {
#pragma unroll
            for (int k = 0; k < 4 * J; ++k) acc[i][k] = 0;
#pragma unroll
            for (int j = 0; j < J; ++j) aw[i][j] = ao[i][j] = 0u;
        }

        // staging registers: rows wave + NW*m, vectors lane + 64*q, and the chunk's slice
        // of the offset table (cc x TD entries, thread tid takes entries tid + 64*NW*e)
        uint4 pv[kStageRows][kStageVecs];
        uint32_t pv4[kStageRows][kStageVecs];
        int32_t pt[kTabRegs];
        auto load_chunk = [&](int c0) {
            const int cc = min(cchunk, nch - c0);
#pragma unroll
            for (int e = 0; e < kTabRegs; ++e) {
                const int idx = tid + 64 * NW * e;
                const int r = idx / TD, k = idx % TD;
                pt[e] = r < cc ? tab[(size_t)(c0 + r) * ndm_pad + d0 + k] : 0;
            }
#pragma unroll
            for (int m = 0; m < kStageRows; ++m) {
                const int r = wave + NW * m;
                const int c = c0 + r;
                const int64_t ws = r < cc ? (int64_t)((t0 + as_const(base)[c]) & ~15) : 0;
                const gu8 *src = (const gu8 *)(x + (size_t)c * pitch);
#pragma unroll
                for (int q = 0; q < kStageVecs; ++q) {
                    const int k = lane + 64 * q;
                    const int64_t off = ws + 16 * (int64_t)k;
                    pv[m][q] = make_uint4(0, 0, 0, 0);
                    pv4[m][q] = 0;
                    if (r < cc && k < nvec) {
                        if (off + 16 <= pitch) {
                            const u32x4 w = *(const gu32x4 *)(src + off);
                            pv[m][q] = make_uint4(w.x, w.y, w.z, w.w);
                        }
                        if (off + 20 <= pitch) pv4[m][q] = *(const gu32 *)(src + off + 16);
                    }
                }
            }
        };
        auto store_chunk = [&](int c0, int b) {
            const int cc = min(cchunk, nch - c0);
            uint8_t *bl = lds + b * buf_bytes;
            int32_t *lds_tab = (int32_t *)(bl + 4 * quarter);
#pragma unroll
            for (int e = 0; e < kTabRegs; ++e) {
                const int idx = tid + 64 * NW * e;
                const int r = idx / TD;
                // rows past cc (read by the branch-free prefetch) point at row cc; the
                // last register's entries beyond kTabRows rows lie outside the table.
                // Entries are byte offsets from the start of the LDS.
                if (r < kTabRows) lds_tab[idx] = (r < cc ? pt[e] + r * R : cc * R) + b * buf_bytes;
            }
            if (cc & 1) {   // an odd chunk ends with a zero row (the pair's second row)
                for (int v = tid; v < 4 * nvec; v += 64 * NW)
                    *(uint4 *)(bl + (v / nvec) * quarter + cc * R + 16 * (v % nvec)) = make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for (int m = 0; m < kStageRows; ++m) {
                const int r = wave + NW * m;
                uint8_t *row = bl + r * R;
#pragma unroll
                for (int q = 0; q < kStageVecs; ++q) {
                    const int k = lane + 64 * q;
                    if (!(r < cc && k < nvec)) continue;
                    const uint4 v = pv[m][q];
                    const uint32_t v4 = pv4[m][q];
                    uint4 c1, c2, c3;
                    c1.x = __builtin_amdgcn_alignbyte(v.y, v.x, 1);
                    c1.y = __builtin_amdgcn_alignbyte(v.z, v.y, 1);
                    c1.z = __builtin_amdgcn_alignbyte(v.w, v.z, 1);
                    c1.w = __builtin_amdgcn_alignbyte(v4, v.w, 1);
                    c2.x = __builtin_amdgcn_alignbyte(v.y, v.x, 2);
                    c2.y = __builtin_amdgcn_alignbyte(v.z, v.y, 2);
                    c2.z = __builtin_amdgcn_alignbyte(v.w, v.z, 2);
                    c2.w = __builtin_amdgcn_alignbyte(v4, v.w, 2);
                    c3.x = __builtin_amdgcn_alignbyte(v.y, v.x, 3);
                    c3.y = __builtin_amdgcn_alignbyte(v.z, v.y, 3);
                    c3.z = __builtin_amdgcn_alignbyte(v.w, v.z, 3);
                    c3.w = __builtin_amdgcn_alignbyte(v4, v.w, 3);
                    *(uint4 *)(row + 16 * k) = v;
                    *(uint4 *)(row + quarter + 16 * k) = c1;
                    *(uint4 *)(row + 2 * quarter + 16 * k) = c2;
                    *(uint4 *)(row + 3 * quarter + 16 * k) = c3;
                }
            }
        };

        const uint8_t *lane_lds = lds + 4 * lane;
        const int32_t *wtab0 = (const int32_t *)(lds + 4 * quarter) + wave * DW;
        const int32_t *wtab = wtab0;   // the table of the buffer being summed
        // the wave's DW offsets of one staged row (16-byte LDS reads)
        auto read_tab = [&](int r, int32_t (&t)[DW]) {
            if constexpr (DW % 4 == 0) {
#pragma unroll
                for (int i = 0; i < DW; i += 4) {
                    const int4 v = *(const int4 *)(wtab + r * TD + i);
                    t[i] = v.x;
                    t[i + 1] = v.y;
                    t[i + 2] = v.z;
                    t[i + 3] = v.w;
                }
            } else {
#pragma unroll
                for (int i = 0; i < DW; ++i) t[i] = wtab[r * TD + i];
            }
        };
        auto load_row = [&](const int32_t (&t)[DW], uint32_t (&v)[DW][J]) {
#pragma unroll
            for (int i = 0; i < DW; ++i) {
                const uint32_t *p = (const uint32_t *)(lane_lds + t[i]);
#pragma unroll
                for (int j = 0; j < J; ++j) v[i][j] = p[64 * j];
            }
        };
        auto add_rows = [&](const uint32_t (&u)[DW][J], const uint32_t (&v)[DW][J]) {
#pragma unroll
            for (int i = 0; i < DW; ++i)
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    aw[i][j] += u[i][j] + v[i][j];
                    ao[i][j] += __builtin_amdgcn_perm(u[i][j], u[i][j], kSelOdd) +
                                __builtin_amdgcn_perm(v[i][j], v[i][j], kSelOdd);
                }
        };

        // the chunk's channel pairs (an odd chunk ends with the zero row).  Software
        // pipeline: while pair k is summed, the samples of pair k+1 and the offsets of
        // pair k+2 are in flight (ping-pong buffers, branch-free steady state).
        // da, db: the samples of a chunk's last channel pair.  sum_chunk reads them but
        // leaves their adds to the caller: with two buffers they are added after the
        // chunk's barrier, while the next chunk's first offsets are in flight (the reads
        // completed before the barrier, so the buffer may be restaged meanwhile); every
        // 256 channels, and at the end, they are added before the 16-bit fields widen.
        uint32_t da[DW][J], db[DW][J];
        auto sum_chunk = [&](const int cc, const bool have_def) {
            const int np = (cc + 1) >> 1;
            int32_t ta[DW], tb[DW];
            uint32_t la[DW][J], lb[DW][J], na[DW][J], nb[DW][J];
            read_tab(0, ta);
            read_tab(1, tb);
            if (have_def) add_rows(da, db);
            load_row(ta, la);
            load_row(tb, lb);
            read_tab(2, ta);
            read_tab(3, tb);
            int k = 0;
            for (; k + 3 <= np; k += 2) {
                load_row(ta, na);               // pair k+1
                load_row(tb, nb);
                read_tab(2 * k + 4, ta);        // offsets of pair k+2
                read_tab(2 * k + 5, tb);
                add_rows(la, lb);               // pair k
                load_row(ta, la);               // pair k+2
                load_row(tb, lb);
                read_tab(2 * k + 6, ta);        // offsets of pair k+3 (padding rows past the end)
                read_tab(2 * k + 7, tb);
                add_rows(na, nb);               // pair k+1
            }
            if (np - k == 2) {
                load_row(ta, na);
                load_row(tb, nb);
                add_rows(la, lb);
                if constexpr (NBUF == 1) {
                    add_rows(na, nb);
                    return;
                }
#pragma unroll
                for (int i = 0; i < DW; ++i)
#pragma unroll
                    for (int j = 0; j < J; ++j) { da[i][j] = na[i][j]; db[i][j] = nb[i][j]; }
            } else {
                if constexpr (NBUF == 1) {
                    add_rows(la, lb);
                    return;
                }
#pragma unroll
                for (int i = 0; i < DW; ++i)
#pragma unroll
                    for (int j = 0; j < J; ++j) { da[i][j] = la[i][j]; db[i][j] = lb[i][j]; }
            }
        };
        // widen the 16-bit fields every 256 channels (chan_chunk is a power of two <= 256)
        auto widen = [&](const int c_end) {
            if ((c_end & 255) == 0 || c_end >= nch) {
#pragma unroll
                for (int i = 0; i < DW; ++i)
#pragma unroll
                    for (int j = 0; j < J; ++j) {
                        const uint32_t even = aw[i][j] - (ao[i][j] << 8);
                        acc[i][4 * j + 0] += (int32_t)(even & 0xFFFFu);
                        acc[i][4 * j + 2] += (int32_t)(even >> 16);
                        acc[i][4 * j + 1] += (int32_t)(ao[i][j] & 0xFFFFu);
                        acc[i][4 * j + 3] += (int32_t)(ao[i][j] >> 16);
                        aw[i][j] = ao[i][j] = 0u;
                    }
            }
        };

        load_chunk(0);
        if constexpr (NBUF == 1) {
            for (int c0 = 0; c0 < nch; c0 += cchunk) {
                const int cc = min(cchunk, nch - c0);
                __syncthreads();          // the previous chunk is no longer read
                store_chunk(c0, 0);
                if (c0 + cchunk < nch) load_chunk(c0 + cchunk);
                __syncthreads();          // the chunk is staged
                sum_chunk(cc, false);      // (one buffer: no deferral, no VGPRs to spare)
                widen(c0 + cc);
            }
        } else {
            __syncthreads();              // the previous item's last chunk is no longer read
            store_chunk(0, 0);
            if (cchunk < nch) load_chunk(cchunk);
            __syncthreads();              // the first chunk is staged
            const bool stage_first = ((wave >> 2) & 1) != 0;
            int buf = 0;
            bool have_def = false;
            for (int c0 = 0; c0 < nch; c0 += cchunk, buf ^= 1) {
                const int cc = min(cchunk, nch - c0);
                const bool more = c0 + cchunk < nch;
                // the other buffer was last read for chunk c0 - cchunk, before the
                // barrier that ended that chunk
                auto stage_next = [&]() {
                    store_chunk(c0 + cchunk, buf ^ 1);
                    if (c0 + 2 * cchunk < nch) load_chunk(c0 + 2 * cchunk);
                };
                wtab = (const int32_t *)((const uint8_t *)wtab0 + buf * buf_bytes);
                if (more && stage_first) stage_next();
                sum_chunk(cc, have_def);
                if (more && !stage_first) stage_next();
                __syncthreads();          // the next chunk is staged, this one no longer read
                const int c_end = c0 + cc;
                have_def = !((c_end & 255) == 0 || c_end >= nch);
                if (!have_def) add_rows(da, db);
                widen(c_end);
            }
        }

        // write the DM transform
        const int ndm = B.ndm, n_dd = B.n_dd;
        const int dw0 = d0 + wave * DW;
#pragma unroll
        for (int i = 0; i < DW; ++i) {
            const int d = dw0 + i;
            if (d >= ndm) continue;
            int32_t *Xr = B.X + (size_t)d * B.xpitch;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int t = t0 + 256 * j + 4 * lane;
                if (t + 3 < n_dd) {
                    *(int4 *)(Xr + t) = make_int4(acc[i][4 * j], acc[i][4 * j + 1],
                                                  acc[i][4 * j + 2], acc[i][4 * j + 3]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (t + e < n_dd) Xr[t + e] = acc[i][4 * j + e];
                }
            }
        }
        if (!queue) break;
    }
}

// 16 trials x 256 samples without staging: every trial's samples are read where they are.
// Workgroup = 16 wavefronts; wavefront w sums trials d0 + 4 (w & 3) ... + 3 over the channels
// of its quarter w >> 2.  Lane l holds trial l >> 4 and the 16 samples from t0 + 16 (l & 15):
// of a channel one 16-byte load from the dword below them, shifted into place with the next
// lane's first dword (the last lane's is a load of its own, one address per trial).  The
// quarters' sums meet in the LDS.  Bound by the loads: one 16-byte load from an address that
// is no multiple of 4 takes as long as four dwords (60.8 us in place of 35.8 below).  Nothing
// depends on the delays' spread, and the quarters give a plan of few tiles four times the
// loads in flight.  1 beam of 256 channels x 128 trials x 8192 samples over 0-500: 71 us
// staged in tiles of the same size, 36 us now; 64 trials x 1024 channels x 4096 samples 160
// and 53; 4 x 34 billion sums 2.24 ms (long rows) and 1.58 ms, 35 adds a clock and CU.
constexpr int kDirectGroup = 4;   // channels in flight while as many are summed (8 spill at 128 registers)
typedef uint32_t u32x4_word __attribute__((ext_vector_type(4), aligned(4)));
typedef int32_t i32x4_word __attribute__((ext_vector_type(4), aligned(4)));
typedef __attribute__((address_space(1))) const u32x4_word gu32x4_word;
typedef __attribute__((address_space(1))) const i32x4_word gi32x4_word;
typedef __attribute__((address_space(1))) const int32_t gi32;

__global__ __launch_bounds__(1024, 4) void k_dedisp_direct(const DevBeam *__restrict__ beams,
                                                           const DedispItem *__restrict__ items, int item_lo,
                                                           int item_hi, int *queue, int beam) {
    __shared__ int32_t s_sum[4][4][3][4][64];   // trials of a wavefront, samples 4 j.., the other quarters'
    __shared__ int s_item;
    constexpr uint32_t kSelOdd = 0x0C030C01u;   // bytes 1, 3 -> 16-bit fields
    constexpr int G = kDirectGroup;
    const int tid = threadIdx.x, lane = lane_id();
    const int quad = __builtin_amdgcn_readfirstlane(wave_id() & 3), quarter = __builtin_amdgcn_readfirstlane(wave_id() >> 2);

    int it = item_lo + blockIdx.x;
    for (;;) {
        if (queue) {
            __syncthreads();
            if (tid == 0) s_item = item_lo + atomicAdd(queue, 1);
            __syncthreads();
            it = __builtin_amdgcn_readfirstlane(s_item);
        }
        if (it >= item_hi) break;
        DedispItem item;
        if (items) {
            item = items[it];
        } else {   // the tiles of one beam, counted
            const int across = (beams[beam].ndm + 15) / 16;
            item.beam = beam;
            item.d0 = 16 * (it % across);
            item.t0 = 256 * (it / across);
        }
        const DevBeam &B = beams[item.beam];
        const int nch = B.nch, ndm = B.ndm, n_dd = B.n_dd;
        const int64_t pitch = B.pitch;
        const uint8_t *__restrict__ x = B.x;
        const int d = item.d0 + 4 * quad + (lane >> 4), t = item.t0 + 16 * (lane & 15);
        const gi32 *delays = (const gi32 *)B.delays + (size_t)min(d, ndm - 1) * nch;
        // this quarter's channels; those whose loads could pass the end of the block (its last
        // channel, in the last time tile) are read byte by byte
        const int per = (nch + 4 * G - 1) / (4 * G) * G;
        const int c_lo = min(nch, quarter * per), c_hi = min(nch, c_lo + per);
        const int64_t past = (int64_t)item.t0 + 260 + (B.n_in - n_dd) - pitch;
        const int c_safe = (int)max((int64_t)0, past > 0 ? nch - (past + pitch - 1) / pitch : (int64_t)nch);
        const int c_wide = min(c_hi, max(c_lo, c_safe));

        int32_t acc[16];
        uint32_t aw[4], ao[4];   // sums of the dwords, of their bytes 1 and 3
#pragma unroll
        for (int k = 0; k < 16; ++k) acc[k] = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) aw[j] = ao[j] = 0u;
        auto load_delays = [&](int g, int32_t (&dl)[G]) {
#pragma unroll
            for (int k = 0; k < G; k += 4) {
                const i32x4_word v = *(gi32x4_word *)(delays + c_lo + g * G + k);
                dl[k] = v.x;
                dl[k + 1] = v.y;
                dl[k + 2] = v.z;
                dl[k + 3] = v.w;
            }
        };
        auto load_row = [&](const uint8_t *row, int32_t delay, u32x4 &v, uint32_t &end) {
            const uint32_t o = (uint32_t)(item.t0 + (delay & ~3));
            v = *(gu32x4_word *)((const gu8 *)row + o + 16 * (lane & 15));
            end = *(gu32 *)((const gu8 *)row + o + 256);
        };
        auto load_samples = [&](int g, const int32_t (&dl)[G], u32x4 (&v)[G], uint32_t (&end)[G], uint32_t (&sh)[G]) {
            const uint8_t *row = x + (size_t)(c_lo + g * G) * pitch;
#pragma unroll
            for (int k = 0; k < G; ++k) {
                load_row(row, dl[k], v[k], end[k]);
                sh[k] = (uint32_t)dl[k];
                row += pitch;
            }
        };
        // the 16 samples of a lane from its dwords and the next one, the next lane's first
        auto samples = [&](const u32x4 &v, uint32_t end, uint32_t sh) {
            const uint32_t next = __builtin_amdgcn_update_dpp(end, v[0], 0x101, 0xF, 0xF, false);   // row_shl:1
            u32x4 r;
            r[0] = __builtin_amdgcn_alignbyte(v[1], v[0], sh);
            r[1] = __builtin_amdgcn_alignbyte(v[2], v[1], sh);
            r[2] = __builtin_amdgcn_alignbyte(v[3], v[2], sh);
            r[3] = __builtin_amdgcn_alignbyte(next, v[3], sh);
            return r;
        };
        auto add = [&](const u32x4 (&v)[G], const uint32_t (&end)[G], const uint32_t (&sh)[G]) {
#pragma unroll
            for (int k = 0; k < G; k += 2) {
                const u32x4 p = samples(v[k], end[k], sh[k]), q = samples(v[k + 1], end[k + 1], sh[k + 1]);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    aw[j] += p[j] + q[j];
                    ao[j] += __builtin_amdgcn_perm(p[j], p[j], kSelOdd) + __builtin_amdgcn_perm(q[j], q[j], kSelOdd);
                }
            }
        };
        auto widen = [&]() {   // at most every 256 channels
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t even = aw[j] - (ao[j] << 8);
                acc[4 * j + 0] += (int32_t)(even & 0xFFFFu);
                acc[4 * j + 2] += (int32_t)(even >> 16);
                acc[4 * j + 1] += (int32_t)(ao[j] & 0xFFFFu);
                acc[4 * j + 3] += (int32_t)(ao[j] >> 16);
                aw[j] = ao[j] = 0u;
            }
        };
        const int n = (c_wide - c_lo) / G;
        if (n > 0) {
            int32_t da[G], db[G];
            u32x4 va[G], vb[G];
            uint32_t ea[G], eb[G], sa[G], sb[G];
            load_delays(0, da);
            load_delays(min(1, n - 1), db);
            load_samples(0, da, va, ea, sa);
            int g = 0;
            for (; g + 2 < n; g += 2) {   // a group's delays are asked for before the samples of the one ahead of it
                load_delays(g + 2, da);
                load_samples(g + 1, db, vb, eb, sb);
                add(va, ea, sa);
                load_delays(min(g + 3, n - 1), db);
                load_samples(g + 2, da, va, ea, sa);
                add(vb, eb, sb);
                if ((g + 2) % (256 / G) == 0) widen();
            }
            if (g + 1 < n) {
                load_samples(g + 1, db, vb, eb, sb);
                add(va, ea, sa);
                add(vb, eb, sb);
            } else {
                add(va, ea, sa);
            }
            widen();
        }
        int c = c_lo + n * G;
        if (c < c_wide) {   // fewer than G channels: the others' places hold zeros
            u32x4 v[G];
            int32_t dl[G];
            uint32_t end[G], sh[G];
#pragma unroll
            for (int k = 0; k < G; ++k) dl[k] = delays[min(c + k, c_wide - 1)];
#pragma unroll
            for (int k = 0; k < G; ++k) load_row(x + (size_t)min(c + k, c_wide - 1) * pitch, dl[k], v[k], end[k]);
#pragma unroll
            for (int k = 0; k < G; ++k) {
                sh[k] = (uint32_t)dl[k];
                if (c + k >= c_wide) v[k] = (u32x4)0, end[k] = 0;
            }
            add(v, end, sh);
            widen();
            c = c_wide;
        }
        for (; c < c_hi; ++c) {
            const gu8 *row = (const gu8 *)(x + (size_t)c * pitch) + delays[c];
#pragma unroll
            for (int k = 0; k < 16; ++k)
                if (t + k < n_dd) acc[k] += row[t + k];
        }

        // the quarters' sums: quarter j ends with samples 4 j ... of every lane
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j != quarter)
#pragma unroll
                for (int e = 0; e < 4; ++e) s_sum[quad][j][(quarter - j - 1) & 3][e][lane] = acc[4 * j + e];
        int32_t r[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            r[e] = quarter < 2 ? (quarter == 0 ? acc[e] : acc[4 + e]) : (quarter == 2 ? acc[8 + e] : acc[12 + e]);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] += s_sum[quad][quarter][q][e][lane];
        const int to = t + 4 * quarter;
        if (d < ndm) {
            int32_t *Xr = B.X + (size_t)d * B.xpitch;
            if (to + 3 < n_dd) {
                *(int4 *)(Xr + to) = make_int4(r[0], r[1], r[2], r[3]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (to + e < n_dd) Xr[to + e] = r[e];
            }
        }
        if (!queue) {
            it += gridDim.x;
            __syncthreads();   // the quarters' sums are read
        }
    }
}

// ------------------------------------------------------- moments + thresholds
// One workgroup per DM row: exact moments n, S1 = sum X, S2 = sum X^2 of every
// segment of the owned samples, then mu, sigma and, for every width w, the smallest
// integer boxcar sum T with snr(T, w) >= theta.  snr is non-decreasing in the sum,
// so "sum >= T" is exactly "snr >= theta".
__global__ __launch_bounds__(kThreads) void k_thresholds(const DevBeam *__restrict__ beams, int beam_lo,
                                                         int beam_hi, int row_lo) {
    __shared__ int64_t sh[kThreads / 64];
    const int r = row_lo + blockIdx.x;
    const DevBeam &B = beams[beam_of_row(beams, beam_lo, beam_hi, r)];
    const int d = r - B.row_base;
    const int32_t *Xr = B.X + (size_t)d * B.xpitch;
    for (int sg = 0; sg < B.nseg; ++sg) {
        const int lo = sg * B.L, hi = min((sg + 1) * B.L, B.n_out);
        // exact integer moments: 16-byte loads over the aligned middle of the segment
        // (rows start 256-byte aligned), single values at its ends
        int64_t s1 = 0, s2 = 0;
        const int a0 = min(hi, (lo + 3) & ~3), a1 = max(a0, hi & ~3);
        for (int t = lo + (int)threadIdx.x; t < a0; t += kThreads) {
            const int64_t v = Xr[t];
            s1 += v;
            s2 += v * v;
        }
        for (int t = a1 + (int)threadIdx.x; t < hi; t += kThreads) {
            const int64_t v = Xr[t];
            s1 += v;
            s2 += v * v;
        }
        const int4 *V = (const int4 *)(Xr + a0);
        const int nv = (a1 - a0) >> 2;
#pragma unroll 4
        for (int i = (int)threadIdx.x; i < nv; i += kThreads) {
            const int4 q = V[i];
            const int64_t x = q.x, y = q.y, z = q.z, w = q.w;
            s1 += (x + y) + (z + w);
            s2 += (x * x + y * y) + (z * z + w * w);
        }
        int64_t t1, t2;
        (void)block_exclusive_scan<int64_t>(s1, &t1, sh);
        (void)block_exclusive_scan<int64_t>(s2, &t2, sh);
        const size_t idx = (size_t)d * B.nseg + sg;
        if (threadIdx.x == 0) {
            B.S1[idx] = t1;
            B.S2[idx] = t2;
            double mu, sigma;
            mu_sigma(hi - lo, t1, t2, mu, sigma);
            B.mu[idx] = mu;
            B.sigma[idx] = sigma;
        }
        if ((int)threadIdx.x < B.nw) {
            double mu, sigma;
            mu_sigma(hi - lo, t1, t2, mu, sigma);
            const int j = threadIdx.x;
            const int w = B.widths[j];
            int32_t T = INT_MAX;
            if (sigma > 0.0) {
                const int64_t bmax = (int64_t)w * B.nch * 255;
                const double est = ceil((double)w * mu + B.theta * sigma * sqrt((double)w));
                int64_t b = est < 0.0 ? 0 : (est > (double)(bmax + 1) ? bmax + 1 : (int64_t)est);
                while (b > 0 && snr_of(b - 1, w, mu, sigma) >= B.theta) --b;
                while (b <= bmax && snr_of(b, w, mu, sigma) < B.theta) ++b;
                T = b > bmax ? INT_MAX : (int32_t)b;
            }
            B.T[idx * B.nw + j] = T;
        }
    }
}

// ------------------------------------------------------------------- boxcars
// Workgroup = one row chunk of kBoxTile owned samples.  The LDS holds the exclusive
// prefix sums S[i] = X[t0] + ... + X[t0+i-1] as wrapping uint32; a window sum S[t+w] - S[t] is
// exact because every true sum is below 2^31.
// Thread k evaluates the 4 consecutive samples 4k + 1024q + {0..3} of each quarter q, so
// its LDS reads are 16-byte vectors at consecutive addresses across lanes.  Hits of a
// sample form a bitmask over the widths; only samples with hits evaluate the binary64
// S/N to pick the best width.  One launch counts and writes the hits in (row, t) order:
// workgroups take chunks in order from a ticket counter, publish their hit count, find
// their offset by looking back over the counts and prefixes their predecessors
// published (decoupled look-back), and write their hits from registers.
// Bound by the chain of one chunk (ticket, loads, scan, widths, look-back; ~25 us with 5
// workgroups on a CU): per sample and width three instructions, one barrier for all stripes
// of the scan and polls that leave the status lines alone took 15 % off 2048 x 16384 samples
// (173 -> 152 us) and 22 % off 128 x 8192 (25.8 -> 20.2).  Chunks of 8192 or 16384 samples in
// as many more threads are slower (171, 184 us), as are look-backs over 256 or 512 chunks at
// once (173, 179 us).
__device__ __forceinline__ uint32_t lds_u32(const uint32_t *S, int i) { return S[i]; }

// Look-back status words: flag in the top two bits, value below.
constexpr uint64_t kStatAggregate = 1ull << 62;   // the chunk's own hit count
constexpr uint64_t kStatInclusive = 2ull << 62;   // hits of every chunk up to and including it
constexpr uint64_t kStatValue = (1ull << 62) - 1;
constexpr int kLookbackPolls = 1 << 16;           // gives up (and reports it) after this many polls: each
                                                  // sleeps 16 x 64 clocks, 28 ms together without
                                                  // their loads, against ~25 us per chunk

// The hit count tot of chunk idx, published as soon as it is known (chunk 0's count is
// its inclusive prefix).
__device__ __forceinline__ void box_publish_count(uint64_t *status, int idx, int64_t tot) {
    __hip_atomic_store(&status[idx], (idx == 0 ? kStatInclusive : kStatAggregate) | (uint64_t)tot,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Run by one wavefront of the workgroup holding chunk idx (count tot, already published):
// sums the published values of the predecessors, nearest first, 64 at a time, up to the
// nearest one that has published its inclusive prefix; publishes its own inclusive
// prefix and returns the exclusive one.  A predecessor took its ticket earlier, so it
// runs and publishes without waiting on this workgroup; the poll limit only guards
// against a broken invariant (*stall is set and the offset is wrong).
__device__ int64_t box_lookback(uint64_t *status, int idx, int64_t tot, int32_t *stall) {
    const int lane = lane_id();
    int64_t excl = 0;
    int j = idx - 1;   // the nearest predecessor not summed yet
    int polls = 0;
    while (j >= 0) {
        const int k = j - lane;
        // before chunk 0 reads as an inclusive prefix of 0
        const uint64_t v = k >= 0 ? __hip_atomic_load(&status[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                  : kStatInclusive;
        const uint64_t flag = v >> 62;
        const uint64_t waiting = __ballot(flag == 0);
        const uint64_t inclusive = __ballot(flag == 2);
        const int first = inclusive ? __builtin_ctzll(inclusive) : 64;
        const uint64_t need = first >= 63 ? ~0ull : (2ull << first) - 1;   // lanes 0 .. first
        if (waiting & need) {
            if (++polls > kLookbackPolls) {
                if (lane == 0) atomicOr(stall, 1);
                break;
            }
            __builtin_amdgcn_s_sleep(16);   // (polls of 64 clocks take the status lines from the publishers)
            continue;
        }
        excl += wave_sum<int64_t>(lane <= first ? (int64_t)(v & kStatValue) : 0);
        if (first < 64) break;
        j -= 64;
    }
    if (lane == 0 && idx > 0)
        __hip_atomic_store(&status[idx], kStatInclusive | (uint64_t)(excl + tot), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    return excl;
}

// status, *ticket: n_chunks words and the ticket counter, zero; offsets gets each
// chunk's first hit index, n_total the range's hit count and stall the look-back's
// give-up flag.
__global__ __launch_bounds__(kThreads, 5) void k_boxcar(const DevBeam *__restrict__ beams, int beam_lo,
                                                     int beam_hi, int chunk_lo, int n_chunks, int64_t *offsets,
                                                     Hit *hits, int32_t *hit_t, int64_t cap, uint64_t *status,
                                                     uint64_t *ticket, int64_t *n_total, int32_t *stall) {
    extern __shared__ __align__(16) uint32_t S[];
    __shared__ __align__(16) uint32_t sh32[5][kThreads / 64];   // kPre stripes' wavefront totals
    __shared__ int64_t sh64[kThreads / 64];
    __shared__ int64_t s_base;
    __shared__ int s_idx;
    constexpr int kQ = kBoxTile / 1024;   // quarters of 1024 samples
    const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
    if (tid == 0) s_idx = (int)atomicAdd((unsigned long long *)ticket, 1ull);
    __syncthreads();
    const int idx = s_idx;   // tickets follow the order in which workgroups start
    const int g = chunk_lo + idx;
    const DevBeam &B = beams[beam_of_chunk(beams, beam_lo, beam_hi, g)];
    const int local = g - B.chunk_base;
    const int d = local / B.nchunk_t;
    const int t0 = (local - d * B.nchunk_t) * kBoxTile;
    const int M = kBoxTile + B.w_max - 1;              // prefix entries needed
    const int nvalid = min(M, B.n_dd - t0);
    const int32_t *Xr = B.X + (size_t)d * B.xpitch + t0;

    // prefix sums in stripes of 1024 (4 consecutive per thread), S[i] the sum before i: the
    // loads and the wavefronts' scans of up to kPre stripes run together, one barrier for all
    // of them, and each thread's four entries are one 16-byte store.
    constexpr int kPre = 5;
    constexpr int kStripe = 4 * kThreads;
    uint32_t carry = 0;
    int s0 = 0;
    for (; s0 < M; s0 += kPre * kStripe) {
        uint32_t v[kPre][4], x[kPre];
#pragma unroll
        for (int k = 0; k < kPre; ++k) {
            // one unconditional 16-byte load per thread and stripe (no branch, so the
            // loads of all stripes are in flight together).  Rows are padded to a
            // multiple of 64 entries and t0 is a multiple of 4, so a read starting at
            // i0 < nvalid stays inside the row; past nvalid the row's first vector is
            // read and the values are replaced by zeros.
            const int i0 = s0 + k * kStripe + 4 * tid;
            const u32x4 q4 = *(gu32x4 *)(Xr + (i0 < nvalid ? i0 : 0));
            v[k][0] = i0 < nvalid ? q4.x : 0u;
            v[k][1] = i0 + 1 < nvalid ? q4.y : 0u;
            v[k][2] = i0 + 2 < nvalid ? q4.z : 0u;
            v[k][3] = i0 + 3 < nvalid ? q4.w : 0u;
        }
        if (s0 > 0) __syncthreads();   // the totals before are read
#pragma unroll
        for (int k = 0; k < kPre; ++k) {
            v[k][1] += v[k][0];
            v[k][2] += v[k][1];
            v[k][3] += v[k][2];
            x[k] = wave_inclusive_scan(v[k][3]);
            if (lane == 63) sh32[k][wave] = x[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPre; ++k) {
            uint32_t pre = carry + x[k] - v[k][3];
#pragma unroll
            for (int w = 0; w < kThreads / 64; ++w) {
                if (w < wave) pre += sh32[k][w];
                carry += sh32[k][w];
            }
            const int i0 = s0 + k * kStripe + 4 * tid;
            if (i0 <= M) *(uint4 *)&S[i0] = make_uint4(pre, pre + v[k][0], pre + v[k][1], pre + v[k][2]);
        }
    }
    if (tid == 0 && s0 <= M) S[s0] = carry;   // the entry after the last stripe
    __syncthreads();   // every prefix entry is written

    const int nw = B.nw, L = B.L, nseg = B.nseg;
    const int tend = min(t0 + kBoxTile, B.n_out);   // owned samples of this chunk: [t0, tend)
    uint32_t mask[kQ][4];
#pragma unroll
    for (int q = 0; q < kQ; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) mask[q][e] = 0u;

    if (tend > t0) {
        uint32_t lo[kQ][4];
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            const uint4 l4 = *(const uint4 *)&S[1024 * q + 4 * tid];
            lo[q][0] = l4.x; lo[q][1] = l4.y; lo[q][2] = l4.z; lo[q][3] = l4.w;
        }
        // segments spanned by the chunk (usually one); thresholds of a segment are uniform
        for (int sg = t0 / L; sg <= (tend - 1) / L; ++sg) {
            const int s_lo = max(sg * L, t0) - t0, s_hi = min((sg + 1) * L, tend) - t0;
            const cint32 *Tp = as_const(B.T + ((size_t)d * nseg + sg) * nw);
            // Sums and thresholds lie in [0, 2^31), so the sign of their difference says which is
            // larger; it is shifted in from the right, width by width.
            uint32_t below[kQ][4];
#pragma unroll
            for (int q = 0; q < kQ; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) below[q][e] = 0u;
            for (int j = 0; j < nw; ++j) {
                const int w = B.widths[j];
                const uint32_t T = (uint32_t)Tp[j];
                uint32_t hi[kQ][4];
                if ((w & 3) == 0) {
#pragma unroll
                    for (int q = 0; q < kQ; ++q) {
                        const uint4 h = *(const uint4 *)&S[1024 * q + 4 * tid + w];
                        hi[q][0] = h.x; hi[q][1] = h.y; hi[q][2] = h.z; hi[q][3] = h.w;
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < kQ; ++q)
#pragma unroll
                        for (int e = 0; e < 4; ++e) hi[q][e] = lds_u32(S, 1024 * q + 4 * tid + w + e);
                }
#pragma unroll
                for (int q = 0; q < kQ; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        below[q][e] = __builtin_amdgcn_alignbit(below[q][e], hi[q][e] - lo[q][e] - T, 31);
            }
#pragma unroll
            for (int q = 0; q < kQ; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int lt = 1024 * q + 4 * tid + e;
                    if (lt >= s_lo && lt < s_hi) mask[q][e] = __builtin_bitreverse32(~below[q][e]) >> (32 - nw);
                }
        }
    }
    // hits are emitted in t order: quarter by quarter, thread by thread within a quarter.
    // The four per-quarter counts (<= 1024 each) are scanned together in 16-bit fields.
    uint64_t packed = 0;
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
        uint64_t cq = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) cq += mask[q][e] ? 1 : 0;
        packed |= cq << (16 * q);
    }
    uint64_t ptot;
    const uint64_t pex = block_exclusive_scan<uint64_t>(packed, &ptot, (uint64_t *)sh64);
    const int row = B.row_base + d;
    int64_t tot = 0;
#pragma unroll
    for (int q = 0; q < kQ; ++q) tot += (int64_t)((ptot >> (16 * q)) & 0xFFFFu);
    if (tid == 0) box_publish_count(status, idx, tot);

    // best width of every hit (widths in ascending order; an equal S/N keeps the smaller
    // width) while the earlier chunks finish: its mask keeps only that width's bit
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t m = mask[q][e];
            if (!m || (m & (m - 1)) == 0) continue;   // no hit, or a single width
            const int li = 1024 * q + 4 * tid + e, t = t0 + li;
            const size_t ms = (size_t)d * nseg + t / L;
            const double mu = B.mu[ms], sigma = B.sigma[ms];
            const uint32_t lo = S[li];
            double best = 0.0;
            int bj = -1;
            while (m) {
                const int j = __builtin_ctz(m);
                m &= m - 1;
                const int w = B.widths[j];
                const double sn = snr_of((int32_t)(S[li + w] - lo), w, mu, sigma);
                if (bj < 0 || sn > best) {
                    best = sn;
                    bj = j;
                }
            }
            mask[q][e] = 1u << bj;
        }
    }

    if (wave == 0) {
        const int64_t excl = box_lookback(status, idx, tot, stall);
        if (lane == 0) {
            s_base = excl;
            offsets[idx] = excl;
            if (idx == n_chunks - 1) *n_total = excl + tot;
        }
    }
    __syncthreads();
    int64_t qbase = s_base;
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
        int64_t pos = qbase + (int64_t)((pex >> (16 * q)) & 0xFFFFu);
        qbase += (int64_t)((ptot >> (16 * q)) & 0xFFFFu);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t m = mask[q][e];   // the best width's bit only
            if (!m) continue;
            if (pos < cap) {
                const int li = 1024 * q + 4 * tid + e, t = t0 + li;
                const size_t ms = (size_t)d * nseg + t / L;
                const int w = B.widths[__builtin_ctz(m)];
                const int32_t Bw = (int32_t)(S[li + w] - S[li]);
                Hit h;
                h.row = row;
                h.t = t;
                h.w = w;
                h.B = Bw;
                h.snr = snr_of(Bw, w, B.mu[ms], B.sigma[ms]);   // the same binary64 value as above
                hits[pos] = h;
                hit_t[pos] = t;
            }
            ++pos;
        }
    }
}

// ------------------------------------------------------- rows of a hit list
// One wavefront per row: the row's first hit (clamped to the stored hits) and its block
// index, blk[r][b] = index (within row r) of the first hit with t >= 64 b, or the row's hit
// count, from the packed times (which the list's writer left beside the records: the peak
// filter's searches and window scans read 4 bytes per hit in place of a 24-byte one).  Rows of
// up to 64 hits, held one a lane, count the hits before each block; in longer ones every hit
// writes the blocks between its predecessor's and its own.  Starts come from the boxcar's
// chunk offsets (first list) or from the places of the first filter's survivors.  Also
// clears the look-back words of the compaction that follows, as many as the list needs.
// What bounds small searches here is launches of 4-5 us and chains of loads in few
// workgroups: with row starts, fill, mark, suffix pass, three-kernel scans and compactions as
// launches of their own a search had 25 where it has 12 now.  1 beam of 256 channels x 128
// trials x 8192 samples: filters and lists 101 us -> 59 (with the chunks of k_survivors below).
__device__ __forceinline__ int64_t list_size(const int64_t *n, int64_t cap) { return min(*n, cap); }

template <bool FIRST>
__global__ __launch_bounds__(kThreads) void k_rows(const DevBeam *__restrict__ beams, int beam_lo, int beam_hi,
                                                   int row_lo, int n_rows, int chunk_lo,
                                                   const int64_t *__restrict__ chunk_off,
                                                   const int64_t *__restrict__ start_before,
                                                   const int64_t *__restrict__ pos, const int64_t *n_before,
                                                   const int64_t *n_list, int64_t cap, int64_t *row_start,
                                                   const int32_t *__restrict__ hit_t, int32_t *__restrict__ blk,
                                                   int nblk, uint64_t *status, int64_t ticket) {
    const int lane = lane_id();
    const int64_t n = list_size(n_list, cap), g = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    for (int64_t i = g; i * kScanPerBlock < n; i += (int64_t)gridDim.x * kThreads) status[i] = 0;
    if (g == 0) status[ticket] = 0;
    const int r = blockIdx.x * (kThreads / 64) + wave_id();
    if (r >= n_rows) return;   // uniform per wavefront
    int64_t at = n;
    if (lane < 2 && r + lane < n_rows) {   // of this row and the next
        const int rr = r + lane;
        if constexpr (FIRST) {
            const DevBeam &B = beams[beam_of_row(beams, beam_lo, beam_hi, row_lo + rr)];
            at = min(chunk_off[B.chunk_base + (row_lo + rr - B.row_base) * B.nchunk_t - chunk_lo], n);
        } else {
            const int64_t i = start_before[rr];
            if (i < list_size(n_before, cap)) at = min(pos[i], n);
        }
    }
    const int64_t s = __shfl(at, 0), e = __shfl(at, 1);
    if (lane == 0) row_start[r] = s;
    if (r == n_rows - 1 && lane == 1) row_start[n_rows] = e;
    const int nh = (int)(e - s);
    int32_t *row = blk + (int64_t)r * nblk;
    if (nh <= 64) {
        const int32_t t = lane < nh ? hit_t[s + lane] : 0;
        for (int c = 0; c < nblk; c += 64) {
            const int b = c + lane;
            int before = 0;
            for (int i = 0; i < nh; ++i) before += __builtin_amdgcn_readlane(t, i) < b << kNmsBlockShift ? 1 : 0;
            if (b < nblk) row[b] = before;
        }
        return;
    }
    int done = -1;   // the block of the last hit so far
    for (int i0 = 0; i0 < nh; i0 += 64) {
        const int i = i0 + lane;
        const int b = i < nh ? min(hit_t[s + i] >> kNmsBlockShift, nblk - 1) : INT_MAX;
        int prev = __shfl_up(b, 1);
        if (lane == 0) prev = done;
        if (i < nh)
            for (int x = prev + 1; x <= b; ++x) row[x] = i;
        done = __shfl(b, min(63, nh - 1 - i0));
    }
    for (int x = done + 1 + lane; x < nblk; x += 64) row[x] = nh;
}

// ------------------------------------------------------- survivors of a peak filter
// The survivors (alive[p] != 0) in order, each chunk of hits placed by a
// look-back over the chunks before it (tickets follow the order in which workgroups take
// them).  Bound by the tickets (one address, 10-15 ns each) and, in a short list, by a chunk's
// dependent loads: chunks of 512 hits, 2 turns a wavefront, while every chunk has its
// workgroup (the others take no ticket), of 4096 in longer lists.  The two launches of 1 beam
// of 128 trials 14 and 14 -> 6 and 4 us against a ticket for each of 1024 workgroups; 18
// million hits 486 -> 169 us against chunks of 512.  CANDS: as candidate records after `*base`
// earlier ones; else as the list that the later, wider filters see, with its packed times, and
// pos[p] the survivors before p.
struct Survivors {
    const Hit *hits;
    const int64_t *n_hits;
    int64_t cap;
    const uint8_t *alive;
    uint64_t *status;
    int64_t ticket;     // place of the ticket counter in status
    int64_t *n_out;
    int32_t *stall;
};

__device__ __forceinline__ void write_candidate(const DevBeam *__restrict__ beams, int beam_lo, int beam_hi, const Hit &h,
                                                spl_candidate *cand) {
    const DevBeam &B = beams[beam_of_row(beams, beam_lo, beam_hi, h.row)];
    spl_candidate c;
    c.beam = B.beam;
    c.dm_index = h.row - B.row_base;
    c.t_sample = h.t;
    c.width = h.w;
    c.boxcar_sum = h.B;
    c.snr = (float)h.snr;
    c.dm = (float)B.dms[c.dm_index];
    c.flags = 0u;
    *cand = c;
}

template <bool CANDS, int TURNS>
__device__ __forceinline__ void place_survivors(const Survivors &v, int64_t n, Hit *__restrict__ out,
                                                int32_t *__restrict__ hit_t, int64_t *__restrict__ pos,
                                                const DevBeam *__restrict__ beams, int beam_lo, int beam_hi,
                                                const int64_t *base, spl_candidate *cands, int64_t cand_cap) {
    __shared__ int64_t s_idx, s_base;
    __shared__ int s_tot[kThreads / 64];
    constexpr int kTurns = TURNS, kChunk = TURNS * kThreads;   // turns of 64 hits a wavefront
    const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
    const int64_t n_chunks = (n + kChunk - 1) / kChunk;
    if (blockIdx.x >= n_chunks) return;
    do {
        __syncthreads();   // the chunk before is placed
        if (tid == 0) s_idx = (int64_t)atomicAdd((unsigned long long *)&v.status[v.ticket], 1ull);
        __syncthreads();
        const int64_t idx = s_idx, p0 = idx * kChunk + wave * (kTurns * 64) + lane;
        if (idx * kChunk >= n) break;   // uniform
        uint64_t alive[kTurns];
        int mine = 0;
#pragma unroll
        for (int k = 0; k < kTurns; ++k) {
            const int64_t p = p0 + 64 * k;
            alive[k] = __ballot(p < n && v.alive[p] != 0);
            mine += __builtin_popcountll(alive[k]);
        }
        if (lane == 0) s_tot[wave] = mine;
        __syncthreads();
        int tot = 0, before = 0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) {
            if (w < wave) before += s_tot[w];
            tot += s_tot[w];
        }
        if (tid == 0) box_publish_count(v.status, (int)idx, tot);
        if (wave == 0) {
            const int64_t excl = box_lookback(v.status, (int)idx, tot, v.stall);
            if (lane == 0) {
                s_base = excl;
                if ((idx + 1) * kChunk >= n) *v.n_out = excl + tot;
            }
        }
        __syncthreads();
        int64_t first = s_base + before;
        if constexpr (CANDS) first += *base;
#pragma unroll
        for (int k = 0; k < kTurns; ++k) {
            const int64_t p = p0 + 64 * k, o = first + __builtin_popcountll(alive[k] & ((1ull << lane) - 1));
            const bool mine_alive = alive[k] >> lane & 1;
            if constexpr (CANDS) {
                if (mine_alive && o < cand_cap) write_candidate(beams, beam_lo, beam_hi, v.hits[p], cands + o);
            } else {
                if (p < n) pos[p] = o;
                if (mine_alive) {
                    const Hit h = v.hits[p];
                    out[o] = h;
                    hit_t[o] = h.t;
                }
            }
            first += __builtin_popcountll(alive[k]);
        }
    } while (n_chunks > gridDim.x);   // (else a chunk each: no further ticket)
}

template <bool CANDS>
__global__ __launch_bounds__(kThreads) void k_survivors(Survivors v, Hit *__restrict__ out, int32_t *__restrict__ hit_t,
                                                        int64_t *__restrict__ pos, const DevBeam *__restrict__ beams,
                                                        int beam_lo, int beam_hi, const int64_t *base,
                                                        spl_candidate *cands, int64_t cand_cap) {
    const int64_t n = list_size(v.n_hits, v.cap);
    if (n == 0 && blockIdx.x == 0 && threadIdx.x == 0) *v.n_out = 0;
    if (n <= (int64_t)kScanPerBlock * gridDim.x)
        place_survivors<CANDS, kScanPerBlock / kThreads>(v, n, out, hit_t, pos, beams, beam_lo, beam_hi, base, cands, cand_cap);
    else
        place_survivors<CANDS, 16>(v, n, out, hit_t, pos, beams, beam_lo, beam_hi, base, cands, cand_cap);
}

// ---------------------------------------------------------------- peak filter
// q beats p when (snr_q, -d_q, -t_q) > (snr_p, -d_p, -t_p).  p survives when no other
// alive hit of its beam within |dd| <= rd, |dt| <= rt beats it.  Rows of a beam are
// contiguous in the hit list and sorted by t; a neighbour row's window starts at the
// first hit with t >= t_p - rt, found by bisection between the row's first hits of that
// 64-sample block and of the next (the block index, built for the list by k_rows): at most 6 dependent loads instead of one per halving of the row.  A row
// holds at most one hit per sample, so in p's own row the window starts no more than rt
// entries before p and needs no search.  Searches and scans read the packed times; a
// hit's S/N is loaded only when it lies in the window.
__global__ __launch_bounds__(kThreads) void k_nms(const DevBeam *__restrict__ beams, int beam_lo, int beam_hi,
                                                  int row_lo, const Hit *__restrict__ hits,
                                                  const int64_t *n_hits, int64_t cap,
                                                  const int64_t *__restrict__ row_start,
                                                  const int32_t *__restrict__ blk, int nblk, int stencil,
                                                  const uint8_t *alive_in, uint8_t *alive_out,
                                                  int64_t *n_alive, const int32_t *__restrict__ hit_t) {
    __shared__ int64_t sh[kThreads / 64];
    // first rows of the beams, for the bisection from a hit's row to its beam in the LDS
    // (when the batch has more beams than fit, the bisection reads the descriptors)
    constexpr int kBeamCache = 256;
    __shared__ int32_t s_rb[kBeamCache];
    const int nbm = beam_hi - beam_lo;
    const bool cached = nbm <= kBeamCache;
    if (cached)
        for (int b = threadIdx.x; b < nbm; b += kThreads) s_rb[b] = beams[beam_lo + b].row_base;
    __syncthreads();
    const int64_t n = min(*n_hits, cap);
    int64_t kept = 0;
    for (int64_t p = blockIdx.x * (int64_t)kThreads + threadIdx.x; p < n; p += (int64_t)gridDim.x * kThreads) {
        if (alive_in && !alive_in[p]) {
            alive_out[p] = 0;
            continue;
        }
        const Hit h = hits[p];
        int bi;
        if (cached) {   // largest b with row_base <= row
            int a = 0, z = nbm - 1;
            while (a < z) {
                const int m = (a + z + 1) >> 1;
                if (s_rb[m] <= h.row) a = m; else z = m - 1;
            }
            bi = beam_lo + a;
        } else {
            bi = beam_of_row(beams, beam_lo, beam_hi, h.row);
        }
        const DevBeam &B = beams[bi];
        if (stencil >= B.nst) {   // this beam's plan has fewer filters: pass through
            alive_out[p] = 1;
            ++kept;
            continue;
        }
        const int rd = B.rd[stencil], rt = B.rt[stencil];
        const int d = h.row - B.row_base;
        bool keep = true;
        // rows in the order 0, -1, +1, -2, +2, ...: the own row needs no search and the
        // nearest rows most often hold a hit that beats p (the outcome does not depend
        // on the order, only how early the loop stops)
        for (int i = 0; i <= 2 * rd && keep; ++i) {
            const int dd = (i & 1) ? -((i + 1) >> 1) : (i >> 1);
            const int d2 = d + dd;
            if (d2 < 0 || d2 >= B.ndm) continue;
            const int r2 = B.row_base + d2 - row_lo;
            const int tmin = h.t - rt;
            const int64_t end = row_start[r2 + 1];
            // where the window [tmin, t_p + rt] starts in row r2
            int64_t lo = row_start[r2], hi = end;
            if (dd == 0) {
                lo = max(lo, p - rt);   // own row: no earlier entry can have t >= tmin
            } else {
                // the first index with t >= tmin lies between the first hits of tmin's
                // 64-sample block and of the next block (block index): bisect in between
                if (tmin > 0) {
                    const int b = tmin >> kNmsBlockShift;
                    const int32_t *br = blk + (int64_t)r2 * nblk;
                    hi = lo + br[b + 1];   // b + 1 < nblk: the index has a block past every t
                    lo += br[b];
                }
                while (lo < hi) {
                    const int64_t m = (lo + hi) >> 1;
                    if (hit_t[m] < tmin) lo = m + 1; else hi = m;
                }
            }
            for (int64_t q = lo; q < end; ++q) {
                const int gt = hit_t[q];
                if (gt > h.t + rt) break;
                if (gt < tmin || q == p || (alive_in && !alive_in[q])) continue;
                const double gs = hits[q].snr;
                const bool beats = gs != h.snr ? gs > h.snr : (d2 != d ? d2 < d : gt < h.t);
                if (beats) {
                    keep = false;
                    break;
                }
            }
        }
        alive_out[p] = keep ? 1 : 0;
        kept += keep ? 1 : 0;
    }
    int64_t tot;
    (void)block_exclusive_scan<int64_t>(kept, &tot, sh);
    if (threadIdx.x == 0 && tot) atomicAdd((unsigned long long *)n_alive, (unsigned long long)tot);
}

// Candidate records of all hits (plans without a peak filter), after `*base` earlier records.
__global__ __launch_bounds__(kThreads) void k_all_hits(const DevBeam *__restrict__ beams, int beam_lo, int beam_hi,
                                                       const Hit *__restrict__ hits, const int64_t *n_hits,
                                                       int64_t cap, const int64_t *base, spl_candidate *cands,
                                                       int64_t cand_cap) {
    const int64_t n = list_size(n_hits, cap), b0 = *base;
    for (int64_t p = blockIdx.x * (int64_t)kThreads + threadIdx.x; p < n; p += (int64_t)gridDim.x * kThreads)
        if (b0 + p < cand_cap) write_candidate(beams, beam_lo, beam_hi, hits[p], cands + b0 + p);
}

// End of the launch sequence of a beam range: fold the range's counts into the run
// statistics; the next range's candidates go after this one's, and its boxcar chunks are
// counted from 0 again.  The last range's end closes the statistics.
__global__ void k_pass_end(DevRun *run, uint64_t *box_ticket, spl_run_stats *stats, int64_t hit_cap, int nst, bool last,
                           int64_t cand_cap) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    *box_ticket = 0;
    stats->n_hits += run->n_hits;
    if (run->n_hits > hit_cap && stats->hit_overflow == 0) stats->hit_overflow = 1;
    if (run->box_stall) stats->hit_overflow = 2;
    for (int k = 0; k < nst; ++k) {
        stats->n_after_stencil[k] += run->n_alive[k];
        run->n_alive[k] = 0;
    }
    run->n_cand_total += nst ? run->n_cand_beam : min(run->n_hits, hit_cap);
    if (!last) return;
    stats->n_candidates = run->n_cand_total;
    stats->cand_overflow = run->n_cand_total > cand_cap ? 1 : 0;
}

// Position-weighted checksum of a DM transform (verifies that retiled kernels give
// identical output): sum over (d, t) of X[d][t] * (1 + d * 65599 + t * 131), wrapping.
__global__ void k_checksum(const int32_t *X, int ndm, int xpitch, int n_dd, unsigned long long *out) {
    __shared__ unsigned long long sh[kThreads / 64];
    unsigned long long s = 0;
    const int64_t n = (int64_t)ndm * n_dd;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int d = (int)(i / n_dd), t = (int)(i - (int64_t)d * n_dd);
        s += (unsigned long long)(uint32_t)X[(size_t)d * xpitch + t] *
             (1ull + (unsigned long long)d * 65599ull + (unsigned long long)t * 131ull);
    }
    unsigned long long tot;
    (void)block_exclusive_scan<unsigned long long>(s, &tot, sh);
    if (threadIdx.x == 0) atomicAdd(out, tot);
}

// Normaliser test hook: mu and sigma from exact moments, as the search computes them.
__global__ void k_mu_sigma(const int64_t *n, const int64_t *s1, const int64_t *s2, int64_t count,
                           double *mu, double *sigma) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < count) mu_sigma(n[i], s1[i], s2[i], mu[i], sigma[i]);
}

// ---------------------------------------------------------------- launchers
#define SPL_HIP_LAUNCH_CHECK() \
    do { hipError_t e__ = hipGetLastError(); if (e__ != hipSuccess) return e__; } while (0)

template <int DW, int J, int NW, int SV, int NBUF>
static hipError_t prepare_dedisp_t(size_t lds_bytes, int *blocks_per_cu) {
    if constexpr (dedisp_direct(DW, J, NW)) {
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_dedisp_direct, 1024, 0);
    } else {
        if (lds_bytes > 64 * 1024) {
            hipError_t e = hipFuncSetAttribute((const void *)k_dedisp<DW, J, NW, SV, NBUF>,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
            if (e != hipSuccess) return e;
        }
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_dedisp<DW, J, NW, SV, NBUF>, 64 * NW,
                                                            lds_bytes);
    }
}

template <int DW, int J, int NW, int SV, int NBUF>
static hipError_t launch_dedisp_t(const DevBeam *beams, const DedispItem *items, int item_lo, int item_hi,
                                  int *queue, int grid, size_t lds_bytes, hipStream_t s) {
    if constexpr (dedisp_direct(DW, J, NW))
        hipLaunchKernelGGL(k_dedisp_direct, dim3(grid), dim3(1024), 0, s, beams, items, item_lo, item_hi, queue, 0);
    else
        hipLaunchKernelGGL((k_dedisp<DW, J, NW, SV, NBUF>), dim3(grid), dim3(64 * NW), lds_bytes, s, beams, items,
                           item_lo, item_hi, queue);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_dedisp_beam(const DevBeam *beams, int beam, int ndm, int n_dd, hipStream_t s) {
    const int64_t n = (int64_t)((ndm + 15) / 16) * ((n_dd + 255) / 256);
    if (n < 1 || n > INT_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_dedisp_direct, dim3((unsigned)std::min<int64_t>(n, 1 << 20)), dim3(1024), 0, s, beams,
                       (const DedispItem *)nullptr, 0, (int)n, (int *)nullptr, beam);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

// The compiled dedispersion shapes: (DM trials per wavefront, 256-sample groups per
// lane, wavefronts per workgroup, 16-byte vectors staged per lane and row, LDS buffers).
// Double buffering is compiled for the 16-wavefront shapes, which hold one workgroup
// per CU, so that no other workgroup sums while one stages.
#define SPL_DEDISP_SHAPES(X)                                                                                 \
    X(2, 2, 8, 1, 1) X(4, 1, 4, 1, 1) X(4, 2, 4, 1, 1) X(4, 1, 8, 1, 1) X(4, 2, 8, 1, 1) X(8, 1, 4, 1, 1)   \
    X(8, 1, 8, 1, 1) X(2, 2, 8, 2, 1) X(4, 1, 8, 2, 1) X(4, 2, 8, 2, 1) X(4, 1, 16, 1, 1)                  \
    X(4, 2, 16, 1, 1) X(2, 2, 16, 1, 1) X(2, 2, 16, 2, 1) X(4, 1, 16, 1, 2) X(4, 2, 16, 1, 2)              \
    X(2, 2, 16, 1, 2) X(2, 2, 16, 2, 2)

bool dedisp_shape_supported(int dw, int j, int nw, int sv, int nbuf) {
#define SPL_X(a, b, c, d, e) if (dw == a && j == b && nw == c && sv == d && nbuf == e) return true;
    SPL_DEDISP_SHAPES(SPL_X)
#undef SPL_X
    return false;
}

hipError_t prepare_dedisp(int dw, int j, int nw, int sv, int nbuf, size_t lds_bytes, int *blocks_per_cu) {
#define SPL_X(a, b, c, d, e)                                          \
    if (dw == a && j == b && nw == c && sv == d && nbuf == e)         \
        return prepare_dedisp_t<a, b, c, d, e>(lds_bytes, blocks_per_cu);
    SPL_DEDISP_SHAPES(SPL_X)
#undef SPL_X
    return hipErrorInvalidValue;
}

hipError_t launch_dedisp(int dw, int j, int nw, int sv, int nbuf, const DevBeam *beams, const DedispItem *items,
                         int item_lo, int item_hi, int *queue, int grid, size_t lds_bytes, hipStream_t s) {
#define SPL_X(a, b, c, d, e)                                                                                 \
    if (dw == a && j == b && nw == c && sv == d && nbuf == e)                                                \
        return launch_dedisp_t<a, b, c, d, e>(beams, items, item_lo, item_hi, queue, grid, lds_bytes, s);
    SPL_DEDISP_SHAPES(SPL_X)
#undef SPL_X
    return hipErrorInvalidValue;
}

hipError_t launch_thresholds(const DevBeam *beams, int beam_lo, int beam_hi, int row_lo, int row_hi, hipStream_t s) {
    const int n = row_hi - row_lo;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_thresholds, dim3(n), dim3(kThreads), 0, s, beams, beam_lo, beam_hi, row_lo);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_clear(uint64_t *a, int64_t na, uint64_t *b, int64_t nb, uint64_t *c, int64_t nc, hipStream_t s) {
    const int64_t n = na + nb + nc;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_clear, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 1024)), dim3(256), 0, s, a, na, b, nb, c,
                       nc);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_boxcar_one_pass(const DevBeam *beams, int beam_lo, int beam_hi, int chunk_lo, int chunk_hi,
                                  int w_max, uint64_t *status, uint64_t *ticket, int64_t *offsets, Hit *hits,
                                  int32_t *hit_t, int64_t cap, int64_t *n_total, int32_t *stall, hipStream_t s) {
    const int n = chunk_hi - chunk_lo;
    if (!status || !ticket || !offsets || !hits || !hit_t || !n_total || !stall) return hipErrorInvalidValue;
    if (n <= 0) return launch_clear((uint64_t *)n_total, 1, nullptr, 0, nullptr, 0, s);
    const size_t lds = (size_t)(kBoxTile + w_max + 8) * sizeof(uint32_t);
    hipLaunchKernelGGL(k_boxcar, dim3(n), dim3(kThreads), lds, s, beams, beam_lo, beam_hi, chunk_lo, n, offsets,
                       hits, hit_t, cap, status, ticket, n_total, stall);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

int scan_blocks(int64_t n_max) { return (int)((n_max + kScanPerBlock - 1) / kScanPerBlock); }

static int grid_for(int64_t cap) {
    int64_t g = (cap + kThreads - 1) / kThreads;
    if (g > 8192) g = 8192;
    if (g < 1) g = 1;
    return (int)g;
}

hipError_t launch_rows_first(const DevBeam *beams, int beam_lo, int beam_hi, int row_lo, int n_rows, int chunk_lo,
                             const int64_t *chunk_off, const int64_t *n_hits, int64_t cap, int64_t *row_start,
                             const int32_t *hit_t, int32_t *blk, int nblk, uint64_t *status, hipStream_t s) {
    if (n_rows <= 0) return hipErrorInvalidValue;
    const int waves = kThreads / 64;
    hipLaunchKernelGGL(k_rows<true>, dim3((unsigned)((n_rows + waves - 1) / waves)), dim3(kThreads), 0, s, beams, beam_lo,
                       beam_hi, row_lo, n_rows, chunk_lo, chunk_off, (const int64_t *)nullptr, (const int64_t *)nullptr,
                       (const int64_t *)nullptr, n_hits, cap, row_start, hit_t, blk, nblk, status,
                       (int64_t)scan_blocks(cap));
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_rows_survivors(int n_rows, const int64_t *start_before, const int64_t *pos, const int64_t *n_before,
                                 const int64_t *n_list, int64_t cap, int64_t *row_start, const int32_t *hit_t,
                                 int32_t *blk, int nblk, uint64_t *status, hipStream_t s) {
    if (n_rows <= 0) return hipErrorInvalidValue;
    const int waves = kThreads / 64;
    hipLaunchKernelGGL(k_rows<false>, dim3((unsigned)((n_rows + waves - 1) / waves)), dim3(kThreads), 0, s,
                       (const DevBeam *)nullptr, 0, 0, 0, n_rows, 0, (const int64_t *)nullptr, start_before, pos, n_before,
                       n_list, cap, row_start, hit_t, blk, nblk, status, (int64_t)scan_blocks(cap));
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

static dim3 survivor_grid(int64_t cap) { return dim3((unsigned)std::max(1, std::min(scan_blocks(cap), 1024))); }

hipError_t launch_compact(const Hit *hits, const int64_t *n_hits, int64_t cap, const uint8_t *alive, uint64_t *status,
                          Hit *out, int32_t *hit_t, int64_t *pos, int64_t *n_out, int32_t *stall, hipStream_t s) {
    const Survivors v{hits, n_hits, cap, alive, status, (int64_t)scan_blocks(cap), n_out, stall};
    hipLaunchKernelGGL(k_survivors<false>, survivor_grid(cap), dim3(kThreads), 0, s, v, out, hit_t, pos,
                       (const DevBeam *)nullptr, 0, 0, (const int64_t *)nullptr, (spl_candidate *)nullptr, (int64_t)0);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_candidates(const DevBeam *beams, int beam_lo, int beam_hi, const Hit *hits, const int64_t *n_hits,
                             int64_t cap, const uint8_t *alive, uint64_t *status, const int64_t *base, int64_t *n_out,
                             int32_t *stall, spl_candidate *cands, int64_t cand_cap, hipStream_t s) {
    if (!alive) {
        hipLaunchKernelGGL(k_all_hits, dim3(grid_for(cap)), dim3(kThreads), 0, s, beams, beam_lo, beam_hi, hits, n_hits,
                           cap, base, cands, cand_cap);
    } else {
        const Survivors v{hits, n_hits, cap, alive, status, (int64_t)scan_blocks(cap), n_out, stall};
        hipLaunchKernelGGL(k_survivors<true>, survivor_grid(cap), dim3(kThreads), 0, s, v, (Hit *)nullptr,
                           (int32_t *)nullptr, (int64_t *)nullptr, beams, beam_lo, beam_hi, base, cands, cand_cap);
    }
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_nms(const DevBeam *beams, int beam_lo, int beam_hi, int row_lo, const Hit *hits,
                      const int64_t *n_hits, int64_t cap, const int64_t *row_start, const int32_t *blk, int nblk,
                      int stencil, const uint8_t *alive_in, uint8_t *alive_out, int64_t *n_alive,
                      const int32_t *hit_t, hipStream_t s) {
    hipLaunchKernelGGL(k_nms, dim3(grid_for(cap)), dim3(kThreads), 0, s, beams, beam_lo, beam_hi, row_lo, hits,
                       n_hits, cap, row_start, blk, nblk, stencil, alive_in, alive_out, n_alive, hit_t);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_pass_end(DevRun *run, uint64_t *box_ticket, spl_run_stats *stats, int64_t hit_cap, int nst, bool last,
                           int64_t cand_cap, hipStream_t s) {
    hipLaunchKernelGGL(k_pass_end, dim3(1), dim3(64), 0, s, run, box_ticket, stats, hit_cap, nst, last, cand_cap);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_checksum(const int32_t *X, int ndm, int xpitch, int n_dd, unsigned long long *out,
                           hipStream_t s) {
    hipLaunchKernelGGL(k_checksum, dim3(1024), dim3(kThreads), 0, s, X, ndm, xpitch, n_dd, out);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_mu_sigma(const int64_t *n, const int64_t *s1, const int64_t *s2, int64_t count, double *mu,
                           double *sigma, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mu_sigma, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, n, s1, s2, count, mu,
                       sigma);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

}  // namespace spl
