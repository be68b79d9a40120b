// Candidate ranker on gfx950: feature snippets of each candidate and a small CNN
// (4 x [3x3 conv -> ReLU -> 2x2 max pool], 2 -> 32 -> 32 -> 32 -> 32 channels, then
// 2048 -> 64 -> 1 fully connected), standing in for the paper's FETCH classifier
// (classification section).  Every convolution and the first fully connected layer,
// forward and backward, is a GEMM on BF16 MFMA (v_mfma_f32_16x16x32_bf16) with FP32
// accumulation; activations are stored as BF16 (round to nearest even), weights are kept
// in FP32 (Adam) and packed to BF16 for the GEMMs.
//
// Activation layout: NHWC.  Convolutions are implicit GEMMs over K = (ky*3 + kx)*Cin + ci
// (padded with zeros to a multiple of 32), reading the activation directly.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ranker.h"
#include "spl_device.h"
#include "spl_internal.h"

#pragma clang fp contract(off)

namespace spl {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

__device__ inline uint16_t f2bf(float f) {   // round to nearest even (finite inputs)
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ inline float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// ----------------------------------------------------------------- snippets
// A channel's samples through a buffer that ends with the block (bytes past it, and
// offsets before the row, which wrap, read as zero or as other samples of the block: the
// entries they belong to are not valid).  An absent channel's buffer is empty.  A negative
// offset must not be brought back by an instruction's own offset, which is added without
// wrapping: apart() keeps the sum in a register.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t channel_rows(const DevBeam &B, int c, bool present) {
    const uint64_t at = (uint64_t)c * (uint64_t)B.pitch, left = (uint64_t)B.nch * (uint64_t)B.pitch - at;
    const uint32_t bytes = left >> 32 ? 0xFFFFFFFCu : (uint32_t)left;
    return __builtin_amdgcn_make_buffer_rsrc((void *)(B.x + at), 0, present ? (int)bytes : 0, 0x00027000);
}

__device__ __forceinline__ int apart(int offset) {
    asm volatile("" : "+v"(offset));
    return offset;
}

// whether a record names a (beam, trial, owned sample) of this batch
__device__ inline bool in_batch(const spl_candidate &cd, const DevBeam *beams, int nbeams) {
    return cd.beam >= 0 && cd.beam < nbeams && cd.dm_index >= 0 && cd.dm_index < beams[cd.beam].ndm &&
           cd.t_sample >= 0 && cd.t_sample < beams[cd.beam].n_out;
}

// Plane 0: rows d*-32..d*+31 of the DM transform over t*-128..t*+127, each row
// standardised by the search's own (mu, sigma) of the segment of t*.  Plane 1: 64
// sub-bands of nch/64 adjacent channels summed along the delays of trial d*, each
// standardised over its valid samples with the same exact-moment recipe.  Values
// float((v - mu)/sigma) in binary64 -> BF16; entries outside the DM range or outside
// [0, n_dd) are 0.  With `fine` plane 0 is another kernel's.
//
// One wavefront per row of the two planes: 64 per candidate, so a few candidates fill the
// chip, and nothing waits for other wavefronts.  Plane 1: lane l adds samples 4l .. 4l+3
// of a channel from two aligned dwords (a wavefront's dword load takes 5 clocks, an
// unaligned one 16) as 16-bit pairs, moved to 32 bits every 256 channels; 16 loads are
// under way at a time.  256 candidates of the 4096-channel band read 400 MB in lines of
// 128 bytes: 72 us, where one workgroup per candidate with three barriers per sub-band
// took 640 us.
__global__ __launch_bounds__(256) void k_snippets(const DevBeam *__restrict__ beams, int nbeams,
                                                  const spl_candidate *__restrict__ cands, int64_t n, bool fine,
                                                  uint16_t *__restrict__ out) {
    constexpr uint32_t kSelEven = 0x0C020C00u;   // bytes 0, 2 -> 16-bit fields
    constexpr uint32_t kSelOdd = 0x0C030C01u;    // bytes 1, 3 -> 16-bit fields
    const int lane = lane_id(), wave = wave_id();
    for (int64_t item = blockIdx.x; item < n * 16; item += gridDim.x) {
        const spl_candidate cd = cands[item >> 4];
        const int k = 4 * (int)(item & 15) + wave;   // row of the planes
        uint16_t *o0 = out + (size_t)(item >> 4) * 2 * 64 * 256 + k * 256;
        uint16_t *o1 = o0 + 64 * 256;
        if (!in_batch(cd, beams, nbeams) || (fine && cd.width < 1)) {   // zero planes
            for (int j = 0; j < 4; ++j) o0[lane + 64 * j] = o1[lane + 64 * j] = 0;
            continue;
        }
        const DevBeam &B = beams[cd.beam];
        const int ds = cd.dm_index, ts = cd.t_sample;
        if (!fine) {
            const int d = ds - 32 + k;
            const bool row = d >= 0 && d < B.ndm;
            const size_t idx = row ? (size_t)d * B.nseg + ts / B.L : 0;
            const double mu = B.mu[idx], sg = B.sigma[idx];
            const int32_t *Xr = B.X + (row ? (size_t)d * B.xpitch : 0);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int t = ts - 128 + lane + 64 * j;
                float v = 0.f;
                if (row && sg > 0.0 && t >= 0 && t < B.n_dd) v = (float)(((double)Xr[t] - mu) / sg);
                o0[lane + 64 * j] = f2bf(v);
            }
        }
        const int per = B.nch / 64;
        const cint32 *drow = as_const(B.delays) + (size_t)ds * B.nch + (size_t)k * per;
        const int ta = ts - 128 + 4 * lane;   // the lane's first sample
        int32_t sv[4] = {0, 0, 0, 0};
        for (int c0 = 0; c0 < per; c0 += 256) {
            uint32_t ae = 0u, ao = 0u;
            const int c1 = min(per, c0 + 256);
            for (int c = c0; c < c1; c += 8) {
                uint32_t w[8][2], shift[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int ci = min(c + i, c1 - 1), off = ts - 128 + drow[ci];
                    const __amdgpu_buffer_rsrc_t rs = channel_rows(B, k * per + ci, c + i < c1);
                    w[i][0] = __builtin_amdgcn_raw_buffer_load_b32(rs, (off & ~3) + 4 * lane, 0, 0);
                    w[i][1] = __builtin_amdgcn_raw_buffer_load_b32(rs, apart((off & ~3) + 4 * lane + 4), 0, 0);
                    shift[i] = (uint32_t)(off & 3);
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const uint32_t word = __builtin_amdgcn_alignbyte(w[i][1], w[i][0], shift[i]);
                    ae += __builtin_amdgcn_perm(word, word, kSelEven);
                    ao += __builtin_amdgcn_perm(word, word, kSelOdd);
                }
            }
            sv[0] += (int32_t)(ae & 0xFFFFu);
            sv[2] += (int32_t)(ae >> 16);
            sv[1] += (int32_t)(ao & 0xFFFFu);
            sv[3] += (int32_t)(ao >> 16);
        }
        // exact moments of the sub-band over the valid columns
        int64_t s1 = 0, s2 = 0;
        int nv = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (ta + j >= 0 && ta + j < B.n_dd) {
                s1 += sv[j];
                s2 += (int64_t)sv[j] * sv[j];
                nv += 1;
            }
        }
        s1 = wave_sum(s1);
        s2 = wave_sum(s2);
        nv = (int)wave_sum((int64_t)nv);
        double mu = 0.0, sg = 0.0;
        if (nv > 0) mu_sigma(nv, s1, s2, mu, sg);
        uint16_t v16[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float v = 0.f;
            if (ta + j >= 0 && ta + j < B.n_dd && sg > 0.0) v = (float)(((double)sv[j] - mu) / sg);
            v16[j] = f2bf(v);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) o1[4 * lane + j] = v16[j];
    }
}

// ------------------------------------------------------- fine-DM DM-time plane
// Plane 0 replaced by the DM transform at 64 DMs DM* + (r - 32) * dDM/32 around the
// candidate's trial DM, dDM the half-range at which a Gaussian pulse of the candidate's
// width keeps `keep` of its S/N (Eq. snrlossapprox with zeta of Eq. zetadef; the paper's
// Eq. deltadm with its unit conversion corrected): dDM = (sqrt(pi)/2 / keep) * W_ms *
// nu_GHz^3 / (6.91e-3 * B_MHz), nu the band centre, B = nch * |foff|.  Delays follow
// Eq. (1) exactly as the plan computes them (binary64, same order, round half away).
// Entry (r, t) sums the block over all channels at t*-128+t plus the row's delays; it is
// valid when every channel's sample lies in [0, n_in) (the extremes are the channels of
// the highest and lowest frequency).  The plane is standardised by the exact moments
// of its valid entries (one mu, sigma for all rows, so the S/N falling off away from
// DM* stays visible), float((v - mu)/sigma) in binary64 -> BF16, invalid entries 0.
__device__ inline int64_t fine_delay(double dd, double k, double tsamp) {
    const double v = (dd * k) / tsamp;
    if (!(fabs(v) < 1.0e9)) return v > 0 ? (int64_t)1 << 40 : -((int64_t)1 << 40);
    return llround(v);
}

// The same within +-2^30 (beyond, no entry is valid).
__device__ inline int32_t fine_delay32(double dd, double k, double tsamp) {
    const int64_t v = fine_delay(dd, k, tsamp);
    return (int32_t)(v > (1 << 30) ? (1 << 30) : (v < -(1 << 30) ? -(1 << 30) : v));
}

// DM of row 32 and step between the rows of a candidate's fine plane.
__device__ inline void fine_range(const DevBeam &B, const spl_candidate &cd, double keep, double &dm_star, double &step) {
    const double w_ms = ((double)cd.width * B.tsamp) * 1000.0;
    const double nu = ((B.fref + B.flo) * 0.5) / 1000.0;
    const double bw = (double)B.nch * fabs(B.foff);
    const double half = (((0.88622692545275801365 / keep) * w_ms) * ((nu * nu) * nu)) / (6.91e-3 * bw);
    step = half / 32.0;
    dm_star = B.dms[cd.dm_index];
}

// The 64 x 256 sums of a candidate, kept as int32 where its two BF16 planes of the same
// size will be.  A workgroup owns one slice of the channels, each of its 4 wavefronts 16
// rows.  The window of a channel that the 64 rows read (256 samples and the spread of
// their delays) is staged in the LDS once, as many channels together as fit 12 KB (1 to
// 16), the next ones' loads under way meanwhile; lane l adds samples 4l .. 4l+3 of a row
// from two adjacent dwords.  Read from the block instead, the rows of wide pulses take
// 25 KB of cache lines a channel, and that is what they wait for.  Windows beyond 12 KB
// are read from the block all the same.
// Delays are held in registers, lane = channel, their division by tsamp done only where
// a product leaves a doubt.
// Sums: `all` adds the four bytes as one word, the carries between them included, `odd`
// bytes 1 and 3 as 16-bit fields; bytes 0 and 2 are all - 256 odd, before the fields are
// full (256 channels), when their high bytes move on.
//
// The slices' sums meet in integer atomics.  256 candidates of the 4096-channel band, 205
// of them 256 samples wide: 1.4 ms (of 1 sample: 1.05 ms), bound by the five vector and
// one LDS instruction of every (row, channel) and by 3 wavefronts a SIMD not hiding all of
// the reads' latency.  6.0 ms before, with a workgroup of 1024 threads per candidate that
// read windows beyond 2 KB sample by sample: as long as the widest one took.
constexpr int kFineRows = 16;          // rows of a wavefront
constexpr int kFineWindow = 12288;     // bytes of the windows of a chunk of channels

template <bool kAligned>
__device__ __forceinline__ void put_sum(uint16_t *p, uint32_t v, bool add) {
    if (kAligned && add) {
        atomicAdd((int32_t *)p, (int32_t)v);
    } else if (kAligned) {
        *(uint32_t *)p = v;
    } else {
        p[0] = (uint16_t)v;
        p[1] = (uint16_t)(v >> 16);
    }
}

template <bool kAligned>
__global__ __launch_bounds__(256, 3) void k_fine_sums(const DevBeam *__restrict__ beams, int nbeams,
                                                      const spl_candidate *__restrict__ cands, int64_t n, double keep,
                                                      int slices, uint16_t *__restrict__ out) {
    constexpr double kD = 4148.8064239;   // Eq. (1), MHz^2 pc^-1 cm^3 s
    constexpr uint32_t kFields = 0x00FF00FFu;
    constexpr int R = kFineRows, P = kFineWindow / 16 / 256;   // 16-byte pieces of a thread
    __shared__ __align__(16) uint8_t windows[2][kFineWindow];
    const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
    for (int64_t item = blockIdx.x; item < n * slices; item += gridDim.x) {
        const int64_t ci = item / slices;
        const int slice = (int)(item - ci * slices);
        const spl_candidate cd = cands[ci];
        if (!in_batch(cd, beams, nbeams) || cd.width < 1) continue;   // uniform across the workgroup
        const DevBeam &B = beams[cd.beam];
        double dm_star, step;
        fine_range(B, cd, keep, dm_star, step);
        const double fch1 = B.fch1, foff = B.foff, tsamp = B.tsamp, rate = 1.0 / tsamp, k_ref = 1.0 / (B.fref * B.fref);
        const int t_first = cd.t_sample - 128;   // sample of column 0
        const int64_t pitch = B.pitch;
        const int nch = B.nch, nblk = nch / 64;
        const int blk0 = (int)((int64_t)nblk * slice / slices), blk1 = (int)((int64_t)nblk * (slice + 1) / slices);
        // bytes of a channel's window: the lowest channel's rows spread most
        const double widest = ((kD * (63.0 * step)) * ((1.0 / (B.flo * B.flo)) - k_ref)) * rate;
        const bool staged = widest < (double)(kFineWindow - 320) && pitch < ((int64_t)1 << 25);
        // (rounding, 16-byte starts, 64 dwords and the next)
        const int win = staged ? ((int)widest + 2 + 16 + 264 + 15) & ~15 : kFineWindow;
        int per_chunk = 16;
        while (per_chunk * win > kFineWindow) per_chunk >>= 1;
        // piece i lies in channel i / (win / 16) of the chunk, by a product (i < 768 pieces)
        const uint32_t pieces = (uint32_t)win / 16, inv = ((1u << 22) + pieces - 1) / pieces;

        auto k_of = [&](int blk) {
            const double f = fch1 + (double)(64 * blk + lane) * foff;
            return (1.0 / (f * f)) - k_ref;
        };
        // windows' first samples, lane = channel: row 0 has the least delays (they are monotone)
        auto window_start = [&](int blk) {
            const int32_t v = fine_delay32(kD * (dm_star + -32.0 * step), k_of(blk), tsamp);
            return (int32_t)((uint32_t)v + (uint32_t)t_first) & ~15;
        };
        u32x4 piece[P];
        auto load = [&](int blk, int c0, int32_t start) {
            const uint64_t at = (uint64_t)(64 * blk) * (uint64_t)pitch, left = (uint64_t)nch * (uint64_t)pitch - at;
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(B.x + at), 0, left >> 32 ? (int)0xFFFFFFFCu : (int)(uint32_t)left, 0x00027000);
#pragma unroll
            for (int j = 0; j < P; ++j) {
                const uint32_t i = (uint32_t)(tid + 256 * j), cc = (i * inv) >> 22;
                const int c = c0 + (int)min(cc, (uint32_t)per_chunk - 1);   // past the chunk: not used
                const uint32_t o = (uint32_t)c * (uint32_t)pitch + (uint32_t)__shfl(start, c) + 16u * (i - cc * pieces);
                piece[j] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)o, 0, 0));
            }
        };
        auto store = [&](int buf) {
#pragma unroll
            for (int j = 0; j < P; ++j) {
                const uint32_t i = (uint32_t)(tid + 256 * j);
                if (i < pieces * (uint32_t)per_chunk) *(u32x4 *)(windows[buf] + 16u * i) = piece[j];
            }
        };

        uint32_t all[R], odd[R], high[R][2];
#pragma unroll
        for (int r = 0; r < R; ++r) all[r] = odd[r] = high[r][0] = high[r][1] = 0u;
        int32_t start = 0, start_next = 0;
        int buf = 0;
        if (staged && blk0 < blk1) {
            start = window_start(blk0);
            load(blk0, 0, start);
            store(0);
        }
        for (int blk = blk0; blk < blk1; ++blk) {
            if (((blk - blk0) & 3) == 0) {   // a byte is left and 256 channels follow: < 2^16
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const uint32_t even = all[r] - (odd[r] << 8);
                    high[r][0] += (even >> 8) & kFields;
                    high[r][1] += (odd[r] >> 8) & kFields;
                    odd[r] &= kFields;
                    all[r] = (even & kFields) + (odd[r] << 8);
                }
            }
            const double kc = k_of(blk);
            int32_t del[R];
            double row0 = (double)(R * wave - 32);   // or the compiler holds 16 products across the loop
            asm volatile("" : "+v"(row0));
            // the product with the rounded 1 / tsamp is off by less than 1e-15 of it
            bool doubt = false;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const double q = ((kD * (dm_star + (row0 + r) * step)) * kc) * rate, whole = rint(q);
                doubt |= !((fabs(q) < 0.9e9) & (fabs(fabs(q - whole) - 0.5) > 1.0e-15 * fabs(q)));
                del[r] = (int32_t)whole;
            }
            if (__any(doubt)) {
#pragma unroll 1
                for (int r = 0; r < R; ++r) {
                    const int32_t v = fine_delay32(kD * (dm_star + (row0 + r) * step), kc, tsamp);
#pragma unroll
                    for (int i = 0; i < R; ++i) del[i] = i == r ? v : del[i];
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) del[r] = (int32_t)((uint32_t)del[r] + (uint32_t)t_first);   // the row's first sample
            if (staged) {
                if (blk + 1 < blk1) start_next = window_start(blk + 1);
#pragma unroll
                for (int r = 0; r < R; ++r) del[r] = max(0, min(del[r] - start, win - 264));
                for (int c0 = 0; c0 < 64; c0 += per_chunk) {
                    __syncthreads();   // the chunk is staged, the one before no longer read
                    const bool last = c0 + per_chunk >= 64, more = !last || blk + 1 < blk1;
                    if (more) load(last ? blk + 1 : blk, last ? 0 : c0 + per_chunk, last ? start_next : start);
                    const uint8_t *base = windows[buf] + 4 * lane;
#pragma unroll 1
                    for (int c = c0; c < c0 + per_chunk; ++c, base += win) {
#pragma unroll
                        for (int r0 = 0; r0 < R; r0 += 8) {   // 8 rows' reads under way together
                            uint32_t w[8][2];
                            int at[8];
#pragma unroll
                            for (int r = 0; r < 8; ++r) {
                                at[r] = __builtin_amdgcn_readlane(del[r0 + r], c);
                                const uint32_t *p = (const uint32_t *)(base + (at[r] & ~3));
                                w[r][0] = p[0];
                                w[r][1] = p[1];
                            }
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int r = 0; r < 8; ++r) {
                                const uint32_t word = __builtin_amdgcn_alignbyte(w[r][1], w[r][0], (uint32_t)at[r]);
                                all[r0 + r] += word;
                                odd[r0 + r] += __builtin_amdgcn_perm(word, word, 0x0C030C01u);
                            }
                        }
                    }
                    buf ^= 1;
                    if (more) store(buf);
                }
                start = start_next;
            } else {
#pragma unroll 1
                for (int c = 0; c < 64; ++c) {
                    const __amdgpu_buffer_rsrc_t rs = channel_rows(B, 64 * blk + c, true);
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const int at = __builtin_amdgcn_readlane(del[r], c), o = (at & ~3) + 4 * lane;
                        const uint32_t w0 = __builtin_amdgcn_raw_buffer_load_b32(rs, o, 0, 0);
                        const uint32_t w1 = __builtin_amdgcn_raw_buffer_load_b32(rs, apart(o + 4), 0, 0);
                        const uint32_t word = __builtin_amdgcn_alignbyte(w1, w0, (uint32_t)at);
                        all[r] += word;
                        odd[r] += __builtin_amdgcn_perm(word, word, 0x0C030C01u);
                    }
                }
            }
        }
        __syncthreads();   // the windows are no longer read
        uint16_t *o = out + (((size_t)ci * 64 + R * wave) * 256 + 4 * lane) * 2;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t even = all[r] - (odd[r] << 8);
            put_sum<kAligned>(o + 512 * r, 256u * (high[r][0] & 0xFFFFu) + (even & 0xFFFFu), slices > 1);
            put_sum<kAligned>(o + 512 * r + 2, 256u * (high[r][1] & 0xFFFFu) + (odd[r] & 0xFFFFu), slices > 1);
            put_sum<kAligned>(o + 512 * r + 4, 256u * (high[r][0] >> 16) + (even >> 16), slices > 1);
            put_sum<kAligned>(o + 512 * r + 6, 256u * (high[r][1] >> 16) + (odd[r] >> 16), slices > 1);
        }
    }
}

// The sums of a candidate standardised into its plane 0 (of 1024 threads, thread (g = tid / 64,
// q = tid % 64) takes columns 4q .. 4q+3 of rows g, g + 16, g + 32, g + 48).
template <bool kAligned>
__global__ __launch_bounds__(1024) void k_fine_plane(const DevBeam *__restrict__ beams, int nbeams,
                                                     const spl_candidate *__restrict__ cands, int64_t n, double keep,
                                                     uint16_t *out) {
    constexpr double kD = 4148.8064239;
    __shared__ int64_t sh[3][16];
    const int lane = lane_id(), wave = wave_id();
    const int g = wave, q = lane;
    for (int64_t ci = blockIdx.x; ci < n; ci += gridDim.x) {
        const spl_candidate cd = cands[ci];
        if (!in_batch(cd, beams, nbeams) || cd.width < 1) continue;   // uniform across the workgroup
        uint16_t *o0 = out + (size_t)ci * 2 * 64 * 256;
        const DevBeam &B = beams[cd.beam];
        double dm_star, step;
        fine_range(B, cd, keep, dm_star, step);
        const double k_lo = (1.0 / (B.flo * B.flo)) - (1.0 / (B.fref * B.fref));
        const int64_t ta = (int64_t)cd.t_sample - 128 + 4 * q;   // the thread's first sample
        int32_t acc[4][4];
        // bit 4i + j: sample j (0..3) of row g + 16i is valid (ta + j + smin >= 0 and
        // ta + j + smax < n_in, the extremes of the row's delays)
        uint32_t vmask = 0u;
        int64_t s1 = 0, s2 = 0, nv = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = g + 16 * i;
            const int64_t s_lo = fine_delay(kD * (dm_star + (double)(r - 32) * step), k_lo, B.tsamp);
            const int64_t smin = s_lo < 0 ? s_lo : 0, smax = s_lo > 0 ? s_lo : 0;
            const uint16_t *p = o0 + 2 * (256 * r + 4 * q);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[i][j] = kAligned ? *(const int32_t *)(p + 2 * j)
                                     : (int32_t)((uint32_t)p[2 * j] | (uint32_t)p[2 * j + 1] << 16);
                if (ta + j + smin >= 0 && ta + j + smax < (int64_t)B.n_in) {
                    vmask |= 1u << (4 * i + j);
                    s1 += acc[i][j];
                    s2 += (int64_t)acc[i][j] * acc[i][j];
                    nv += 1;
                }
            }
        }
        // exact moments of the plane's valid entries
        s1 = wave_sum(s1);
        s2 = wave_sum(s2);
        nv = wave_sum(nv);
        if (lane == 0) {
            sh[0][wave] = s1;
            sh[1][wave] = s2;
            sh[2][wave] = nv;
        }
        __syncthreads();   // and every sum is read before the plane takes its place
        int64_t S1 = 0, S2 = 0, NV = 0;
        for (int k = 0; k < 16; ++k) {
            S1 += sh[0][k];
            S2 += sh[1][k];
            NV += sh[2][k];
        }
        double mu = 0.0, sg = 0.0;
        if (NV > 0) mu_sigma(NV, S1, S2, mu, sg);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float v = 0.f;
                if ((vmask >> (4 * i + j) & 1u) && sg > 0.0) v = (float)(((double)acc[i][j] - mu) / sg);
                o0[(g + 16 * i) * 256 + 4 * q + j] = f2bf(v);
            }
        }
        __syncthreads();   // sh is reused by the next candidate
    }
}

// --------------------------------------------------------------------- GEMM
// C[M][N] (FP32, row stride ldc) = (mode 1: C +) A[M][K] * B[N][K]^T with A and B BF16,
// K contiguous, row strides lda/ldb multiples of 8, K a multiple of 32.  Workgroup =
// 4 wavefronts; wavefront w computes rows 64*bx + 16w .. +15 and columns 32*by .. +31
// (two 16x16 tiles); split z of gridDim.z covers K range [z*klen, (z+1)*klen) and adds
// atomically (mode 1).  MFMA operand lanes: lane l supplies A[l%16][8(l/16) .. +7] and
// B^T[l%16][8(l/16) .. +7] and receives D[4(l/16) + i][l%16].
__global__ __launch_bounds__(256) void k_gemm(const uint16_t *__restrict__ A, int64_t lda,
                                              const uint16_t *__restrict__ Bm, int64_t ldb, float *C, int64_t ldc,
                                              int M, int N, int K, int klen, int mode) {
    const int lane = lane_id(), wave = wave_id();
    const int m_base = blockIdx.x * 64 + wave * 16;
    const int n_base = blockIdx.y * 32;
    const int k_lo = blockIdx.z * klen, k_hi = min(K, k_lo + klen);
    const int arow = m_base + (lane & 15), kq = 8 * (lane >> 4);
    const int b0 = n_base + (lane & 15), b1 = b0 + 16;
    f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
    const u16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int k0 = k_lo; k0 < k_hi; k0 += 32) {
        const u16x8 a = arow < M ? *(const u16x8 *)(A + (size_t)arow * lda + k0 + kq) : zero;
        const u16x8 x0 = b0 < N ? *(const u16x8 *)(Bm + (size_t)b0 * ldb + k0 + kq) : zero;
        const u16x8 x1 = b1 < N ? *(const u16x8 *)(Bm + (size_t)b1 * ldb + k0 + kq) : zero;
        acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, x0),
                                                       acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, x1),
                                                       acc1, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int m = m_base + 4 * (lane >> 4) + i;
        if (m >= M) continue;
        const int n0 = n_base + (lane & 15), n1 = n0 + 16;
        if (n0 < N) {
            if (mode) atomicAdd(&C[(size_t)m * ldc + n0], acc0[i]);
            else C[(size_t)m * ldc + n0] = acc0[i];
        }
        if (n1 < N) {
            if (mode) atomicAdd(&C[(size_t)m * ldc + n1], acc1[i]);
            else C[(size_t)m * ldc + n1] = acc1[i];
        }
    }
}

// ------------------------------------------------------- implicit-GEMM convolution
// Z[p][co] = sum over taps t = ky*3 + kx and input channels ci of X[src(p, t)][ci] *
// Wt[co][t*32 + ci], without an im2col buffer: with 32 input channels each K-step of 32 is
// one tap, and the MFMA A operand of lane l is the 16 bytes of channels 8(l/16) .. +7 of
// one source pixel.
//
// A wavefront computes 4 tiles of 16 pixels x all 32 columns.  In the forward layers a tile is
// a 2 x 8 pixel patch, so the result holds four whole 2 x 2 windows: lane l keeps rows
// 4(l/16) .. +3, i.e. two horizontal pairs of one image row, and lane l ^ 32 the pairs below
// them.  One exchange of half a wavefront gives lanes 0-31 both rows of columns 0-15 and
// lanes 32-63 both rows of columns 16-31; bias, ReLU and the max pool (with the window
// position of the first maximum, 255 when no element is positive) then run in registers,
// and only the pooled BF16 activation and the decision bytes are written, 64 bytes a pixel.
__device__ __forceinline__ void pool_tile(const f32x4 acc0, const f32x4 acc1, float bias,
                                          uint16_t *__restrict__ pooled, uint8_t *__restrict__ arg, size_t o) {
    float above[4], below[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc0[i]), __float_as_uint(acc1[i]), false, false);
        above[i] = __uint_as_float(halves[0]);
        below[i] = __uint_as_float(halves[1]);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const float z[4] = {above[2 * k] + bias, above[2 * k + 1] + bias, below[2 * k] + bias, below[2 * k + 1] + bias};
        float best = 0.f;
        int ba = 255;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (z[j] > best) {
                best = z[j];
                ba = j;
            }
        }
        arg[o + 32 * k] = (uint8_t)ba;
        pooled[o + 32 * k] = f2bf(best);
    }
}

__device__ __forceinline__ f32x4 mfma_bf16(u16x8 a, u16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The first layer: input NCHW with 2 channels (the snippet planes), images n >= nvalid read
// as zero.  Workgroup = 4 wavefronts = a strip of 2 rows x 128 columns; its input window, 4
// rows x 130 columns with the zero padding, is staged in the LDS with both channels of a
// sample in one dword.  K = 32: k = 2 t + ci, so a lane's 8 values are the dwords of four
// taps, read with no unpacking; taps past the ninth read zeros.  256 snippets:
// 42 us, of which the activations and decisions written take 17; 92 with 8 two-byte LDS reads
// a lane and tile and half of the lanes pooling.
__global__ __launch_bounds__(256) void k_conv_first(const uint16_t *__restrict__ X, int nvalid, int H, int W,
                                                    const uint16_t *__restrict__ Wt, const float *__restrict__ bias,
                                                    uint16_t *__restrict__ pooled, uint8_t *__restrict__ arg) {
    constexpr int kWc = 130, kZeros = 4 * kWc;   // columns of a staged row; then 32 zeros
    __shared__ uint32_t win[kZeros + 32];
    const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
    const int strips = W / 128;
    const int64_t strip = blockIdx.x;
    const int sc = (int)(strip % strips), ph = (int)(strip / strips % (H / 2));
    const int64_t n = strip / strips / (H / 2);
    {
        const int row = tid >> 6, d = tid & 63, hs = 2 * ph - 1 + row;
        const bool in = n < nvalid && hs >= 0 && hs < H;
        const bool aligned = ((uintptr_t)X & 3) == 0;
        const uint16_t *src = X + ((size_t)(in ? n : 0) * 2 * H + (in ? hs : 0)) * W + 128 * sc + 2 * d;
        const size_t plane = (size_t)H * W;   // even
        uint32_t v0 = 0u, v1 = 0u;
        if (in) {
            v0 = aligned ? *(const uint32_t *)src : (uint32_t)src[0] | (uint32_t)src[1] << 16;
            v1 = aligned ? *(const uint32_t *)(src + plane) : (uint32_t)src[plane] | (uint32_t)src[plane + 1] << 16;
        }
        if (tid < 8) {   // the columns left and right of the strip
            const int e_row = tid >> 1, e_ws = 128 * sc - 1 + 129 * (tid & 1), e_hs = 2 * ph - 1 + e_row;
            uint32_t e = 0u;
            if (n < nvalid && e_hs >= 0 && e_hs < H && e_ws >= 0 && e_ws < W) {
                const uint16_t *p = X + ((size_t)n * 2 * H + e_hs) * W + e_ws;
                e = (uint32_t)p[0] | (uint32_t)p[plane] << 16;
            }
            win[e_row * kWc + 129 * (tid & 1)] = e;
        } else if (tid < 40) {
            win[kZeros + tid - 8] = 0u;
        }
        win[row * kWc + 2 * d + 1] = (v0 & 0xFFFFu) | v1 << 16;
        win[row * kWc + 2 * d + 2] = v0 >> 16 | (v1 & 0xFFFF0000u);
    }
    __syncthreads();
    const int r = lane & 15, q = lane >> 4, co = r + 16 * (lane >> 5);
    const u16x8 b0 = *(const u16x8 *)(Wt + (size_t)r * 32 + 8 * q), b1 = *(const u16x8 *)(Wt + (size_t)(r + 16) * 32 + 8 * q);
    int at[4];   // of taps 4 q .. 4 q + 3, tile 0
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int t = 4 * q + j, ky = (t * 11) >> 5;   // t / 3
        at[j] = t < 9 ? ((r >> 3) + ky) * kWc + 32 * wave + (r & 7) + t - 3 * ky : kZeros;
    }
    const float b = bias[co];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
        typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
        const u32x4v a = {win[at[0] + 8 * mt], win[at[1] + 8 * mt], win[at[2] + 8 * mt], win[at[3] + 8 * mt]};
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        const f32x4 acc0 = mfma_bf16(__builtin_bit_cast(u16x8, a), b0, zero);
        const f32x4 acc1 = mfma_bf16(__builtin_bit_cast(u16x8, a), b1, zero);
        const size_t pw = 64 * sc + 16 * wave + 4 * mt + 2 * (q & 1);
        pool_tile(acc0, acc1, b, pooled, arg, (((size_t)n * (H / 2) + ph) * (W / 2) + pw) * 32 + co);
    }
}

// The layers of 32 input channels, NHWC.  Forward (pooled): src = (h + ky - 1, w + kx - 1).
// BACK: input gradient, src = (h - ky + 1, w - kx + 1): the input is dZ, Wt the weights repacked as [ci][t*32 + co], the result FP32 [P][32].
//
// Workgroup = 4 wavefronts = 256 pixels, 256/W whole rows (W = 32, 64 or 128).  Read straight
// from memory, a tile's nine taps and their weights took 54 KB of 16-byte loads per 64
// pixels, 860 clocks of a CU (the products take 290); now the rows and the two around them are staged in
// the LDS and the weights stay in registers (72) over the tiles of a workgroup.  A pixel's four
// 16-byte pieces lie at places (piece ^ pixel / 4 mod 4), and rows W + 8 pixels apart, so the
// 16 pixels of a tile meet no bank twice; a step of one row or 8 columns then changes an
// address by a constant and bit 5.  256 snippets, the three
// layers forward: 45 us, 108 before; back: 61, 100 before.
template <bool BACK, int W>
__global__ __launch_bounds__(256, 3) void k_conv32(const uint16_t *__restrict__ X, int64_t ntiles, int H,
                                                   const uint16_t *__restrict__ Wt, float *__restrict__ C,
                                                   const float *__restrict__ bias, uint16_t *__restrict__ pooled,
                                                   uint8_t *__restrict__ arg) {
    constexpr int R = 256 / W, LD = W + 8;         // rows of a tile; pixels of a staged row
    constexpr int V = (R + 2) * W * 4 / 256;       // 16-byte pieces a thread stages
    __shared__ __align__(16) uint8_t win[(R + 2) * LD * 64];
    const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
    const int r = lane & 15, q = lane >> 4;
    const u16x8 none = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int i = tid; i < (R + 2) * 8; i += 256) {   // the columns left and right of the image
        const int row = i >> 3, side = (i >> 2) & 1;
        *(u16x8 *)(win + (row * LD + side * (W + 1)) * 64 + (i & 3) * 16) = none;
    }
    u16x8 b0[9], b1[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        b0[t] = *(const u16x8 *)(Wt + (size_t)r * 288 + 32 * t + 8 * q);
        b1[t] = *(const u16x8 *)(Wt + (size_t)(r + 16) * 288 + 32 * t + 8 * q);
    }
    const int rp = wave / (W / 32), cb = wave % (W / 32);   // the wavefront's two rows and 32 columns
    // of kx: the pixel of tap (0, kx), tile 0
    uint32_t at[3];
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) {
        const int p = BACK ? 2 * rp * LD + 32 * cb + r + kx : (2 * rp + (r >> 3)) * LD + 32 * cb + (r & 7) + kx;
        at[kx] = (uint32_t)(p * 64 + ((q ^ (p >> 2 & 3)) << 4));
    }
    const int co = r + 16 * (lane >> 5);
    const float b = BACK ? 0.f : bias[co];
    const int per_img = H / R;
    for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int64_t n = tile / per_img;
        const int hb = (int)(tile - n * per_img) * R;
        u16x8 v[V];
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const int i = tid + 256 * j, row = i / (W * 4), hs = hb + row - 1;
            v[j] = none;
            if (hs >= 0 && hs < H) v[j] = *(const u16x8 *)(X + ((size_t)n * H + hs) * (W * 32) + 8 * (i % (W * 4)));
        }
        __syncthreads();   // the tile before is no longer read
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const int i = tid + 256 * j, p = i / (W * 4) * LD + (i / 4) % W + 1;
            *(u16x8 *)(win + p * 64 + (((i & 3) ^ (p >> 2 & 3)) << 4)) = v[j];
        }
        __syncthreads();
        f32x4 acc0[4], acc1[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) acc0[mt] = acc1[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const int ky = BACK ? 2 - t / 3 : t / 3, kx = BACK ? 2 - t % 3 : t % 3;   // place in the window
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const int down = BACK ? ky + (mt >> 1) : ky, flip = BACK ? down & 1 : (ky + mt) & 1;
                const int step = down * LD * 64 + (BACK ? (mt & 1) * 1024 : mt * 512);
                const u16x8 a = *(const u16x8 *)(win + (at[kx] ^ (flip ? 32u : 0u)) + step);
                acc0[mt] = mfma_bf16(a, b0[t], acc0[mt]);
                acc1[mt] = mfma_bf16(a, b1[t], acc1[mt]);
            }
        }
        if constexpr (BACK) {
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                float *o = C + (((size_t)n * H + hb + 2 * rp + (mt >> 1)) * W + 32 * cb + 16 * (mt & 1) + 4 * q) * 32 + r;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    o[32 * i] = acc0[mt][i];
                    o[32 * i + 16] = acc1[mt][i];
                }
            }
        } else {
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) {
                const size_t pw = 16 * cb + 4 * mt + 2 * (q & 1);
                pool_tile(acc0[mt], acc1[mt], b, pooled, arg,
                          (((size_t)n * (H / 2) + hb / 2 + rp) * (W / 2) + pw) * 32 + co);
            }
        }
    }
}

// ------------------------------------------------------- weight gradient (LDS)
// part[blockIdx.x][k][co] (FP32 [gridDim.x][288][32]) = sum over the pixels p of the
// workgroup's slabs of A[p][k] * dZ[p][co], A the (implicit) im2col of the layer input:
// k = t*32 + ci (32 input channels, NHWC).  A slab is 32 consecutive pixels (the MFMA
// K-step); its dZ and the 9 shifted input tiles are staged transposed in LDS
// ([channel][pixel]) so that MFMA operands are 16-byte LDS reads.  Tiles of the 288 x 32
// result (9 taps x 2 x 2 of 16 x 16) are spread over the 4 waves.
__global__ __launch_bounds__(256) void k_wgrad(const uint16_t *__restrict__ X, int N, int H, int W,
                                               const uint16_t *__restrict__ dZ, float *__restrict__ part) {
    constexpr int kTiles = 36;                           // 16x16 tiles of the K x 32 result
    constexpr int kPerWave = kTiles / 4;
    constexpr int kRows = 9 * 32;                        // staged A^T rows
    constexpr int kLd = 40;                              // LDS row stride (elements), 80 bytes
    __shared__ __align__(16) uint16_t sA[kRows * kLd];
    __shared__ __align__(16) uint16_t sZ[32 * kLd];
    const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
    const uint32_t HW = (uint32_t)(H * W);
    const uint32_t nslab = (uint32_t)N * HW / 32u;       // N H W is a multiple of 32 (< 2^31)
    f32x4 acc[kPerWave];
#pragma unroll
    for (int i = 0; i < kPerWave; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int kq = 8 * (lane >> 4);
    // thread -> (pixel tid/8, channels 4*(tid%8) .. +3) of a slab; the next slab's dZ and
    // nine input tiles are loaded into registers while the current one is multiplied
    const int px = tid >> 3, c4 = (tid & 7) * 4;
    uint64_t vz = 0, va[9];
    auto load = [&](uint32_t sl) {
        const uint32_t p = sl * 32u + (uint32_t)px;
        vz = *(const uint64_t *)(dZ + (size_t)p * 32 + c4);
        const uint32_t n = p / HW, hw = p - n * HW, h = hw / (uint32_t)W, w = hw - h * (uint32_t)W;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const int hs = (int)h + t / 3 - 1, ws = (int)w + t % 3 - 1;
            va[t] = 0;
            if (hs >= 0 && hs < H && ws >= 0 && ws < W)
                va[t] = *(const uint64_t *)(X + (((size_t)n * H + hs) * W + ws) * 32 + c4);
        }
    };
    uint32_t sl = blockIdx.x;
    if (sl < nslab) load(sl);
    for (; sl < nslab; sl += gridDim.x) {
#pragma unroll
        for (int i = 0; i < 4; ++i) sZ[(c4 + i) * kLd + px] = (uint16_t)(vz >> (16 * i));
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) sA[(t * 32 + c4 + i) * kLd + px] = (uint16_t)(va[t] >> (16 * i));
        __syncthreads();
        if (sl + gridDim.x < nslab) load(sl + gridDim.x);
#pragma unroll
        for (int i = 0; i < kPerWave; ++i) {
            const int tile = wave + 4 * i;
            const int it = tile >> 1, jt = tile & 1;   // A^T row tile (16 rows of k), dZ^T row tile (co)
            const u16x8 a = *(const u16x8 *)(sA + (it * 16 + (lane & 15)) * kLd + kq);
            const u16x8 b = *(const u16x8 *)(sZ + (jt * 16 + (lane & 15)) * kLd + kq);
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                             __builtin_bit_cast(bf16x8, b), acc[i], 0, 0, 0);
        }
        __syncthreads();
    }
    float *out = part + (size_t)blockIdx.x * kRows * 32;
#pragma unroll
    for (int i = 0; i < kPerWave; ++i) {
        const int tile = wave + 4 * i;
        const int it = tile >> 1, jt = tile & 1;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int k = it * 16 + 4 * (lane >> 4) + r;
            out[(size_t)k * 32 + jt * 16 + (lane & 15)] = acc[i][r];
        }
    }
}

// Weight gradient of the first layer (2 input channels, K = 18 used of 32):
// part[blockIdx.x][k][co] = sum over the pixels p of the workgroup's slabs of
// A[p][k] * dZ[p][co], k = t*2 + ci, dZ[p][co] = BF16 of dOut[pooled][co] at the window's arg
// position, 0 elsewhere; the bias gradient (the sum of dOut over windows with a chosen
// element) is added to dbias.  dZ, four times the size of dOut, is made in the LDS only: no
// other kernel needs it (written out and read back, as the other layers' is, this layer took
// 155 us for 256 snippets, and 62 now).  Each wavefront works alone on slabs of two rows x 32 columns, the two
// rows of 16 windows (W a multiple of 32): the input is NCHW, so the 32 values of row k are
// 32 neighbouring samples of one plane (shifted by the tap), read straight into the LDS
// row.  No workgroup barrier in the loop: a wavefront's LDS writes and reads execute in
// order.  The four wavefronts' sums are added in a fixed order at the end.
__global__ __launch_bounds__(256) void k_wgrad_first(const uint16_t *__restrict__ X, int N, int nvalid, int H,
                                                     int W, const float *__restrict__ dOut,
                                                     const uint8_t *__restrict__ arg, float *__restrict__ part,
                                                     float *__restrict__ dbias) {
    constexpr int kLd = 40;
    __shared__ __align__(16) uint16_t lds[2 * 4 * 32 * kLd];   // per wave: A rows, then dZ^T rows
    __shared__ float sb[4][32];
    const int lane = lane_id(), wave = wave_id();
    uint16_t *A = lds + wave * 2 * 32 * kLd, *Zt = A + 32 * kLd;
    for (int i = lane; i < 32 * kLd; i += 64) A[i] = 0;   // rows 18..31 stay zero
    __builtin_amdgcn_wave_barrier();
    f32x4 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint32_t H2 = (uint32_t)H / 2u, W2 = (uint32_t)W / 2u, across = (uint32_t)W / 32u;
    const uint32_t nslab = (uint32_t)N * H2 * across;
    const uint32_t nwaves = gridDim.x * 4u;
    const int kq = 8 * (lane >> 4);
    // lane -> dOut: window lane/4, channels 8*(lane%4) .. +7; A: pixel lane%32, channel
    // lane/32, four rows and three columns.  The next slab is loaded into registers while
    // the current one is multiplied.
    const int win = lane >> 2, grp = lane & 3;
    const int apx = lane & 31, aci = lane >> 5;
    float bias_part[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) bias_part[c] = 0.f;
    float4 g0, g1;
    uint2 at;
    uint16_t av[4][3];
    auto load = [&](uint32_t sl) {
        const uint32_t n = sl / (H2 * across), rem = sl - n * (H2 * across), h2 = rem / across, w0 = 32u * (rem - h2 * across);
        const size_t q = ((size_t)n * H2 + h2) * W2 + w0 / 2u + win;
        g0 = *(const float4 *)(dOut + q * 32 + 8 * grp);
        g1 = *(const float4 *)(dOut + q * 32 + 8 * grp + 4);
        at = *(const uint2 *)(arg + q * 32 + 8 * grp);
        const bool img_ok = (int)n < nvalid;
        const uint16_t *plane = X + ((size_t)n * 2 + aci) * H * W;
#pragma unroll
        for (int y = 0; y < 4; ++y)
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                const int hs = 2 * (int)h2 + y - 1, ws = (int)w0 + apx + x - 1;
                av[y][x] = (img_ok && hs >= 0 && hs < H && ws >= 0 && ws < W) ? plane[(size_t)hs * W + ws] : (uint16_t)0;
            }
    };
    uint32_t sl = blockIdx.x * 4u + (uint32_t)wave;
    if (sl < nslab) load(sl);
    for (; sl < nslab; sl += nwaves) {
        const float g[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
        uint32_t a[8], b[8];
        uint16_t x[4][3];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            a[c] = ((c < 4 ? at.x : at.y) >> (8 * (c & 3))) & 0xFFu;
            b[c] = f2bf(g[c]);
            if (a[c] != 255u) bias_part[c] += g[c];
        }
#pragma unroll
        for (int y = 0; y < 4; ++y)
#pragma unroll
            for (int t = 0; t < 3; ++t) x[y][t] = av[y][t];
        if (sl + nwaves < nslab) load(sl + nwaves);
#pragma unroll
        for (int y = 0; y < 2; ++y) {   // the slab's two rows
#pragma unroll
            for (int c = 0; c < 8; ++c)
                *(uint32_t *)&Zt[(8 * grp + c) * kLd + 2 * win] =
                    (a[c] == 2u * y ? b[c] : 0u) | (a[c] == 2u * y + 1u ? b[c] << 16 : 0u);
#pragma unroll
            for (int t = 0; t < 9; ++t) A[(2 * t + aci) * kLd + apx] = x[y + t / 3][t % 3];
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                const u16x8 av8 = *(const u16x8 *)(A + (it * 16 + (lane & 15)) * kLd + kq);
#pragma unroll
                for (int jt = 0; jt < 2; ++jt)
                    acc[it][jt] = mfma_bf16(av8, *(const u16x8 *)(Zt + (jt * 16 + (lane & 15)) * kLd + kq), acc[it][jt]);
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        float v = bias_part[c];
#pragma unroll
        for (int o = 4; o < 64; o <<= 1) v += __shfl_xor(v, o);
        if (lane < 4) sb[wave][8 * grp + c] = v;
    }
    // the four wavefronts' sums, added in a fixed order (the staging area is reused)
    __syncthreads();
    if (threadIdx.x < 32)
        atomicAdd(&dbias[threadIdx.x], sb[0][threadIdx.x] + sb[1][threadIdx.x] + sb[2][threadIdx.x] + sb[3][threadIdx.x]);
    float *red = (float *)lds;   // [4 waves][4 tiles][4][64]: 16 KiB of the 20 KiB
#pragma unroll
    for (int it = 0; it < 2; ++it)
#pragma unroll
        for (int jt = 0; jt < 2; ++jt)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[((wave * 4 + 2 * it + jt) * 4 + r) * 64 + lane] = acc[it][jt][r];
    __syncthreads();
    if (wave == 0) {
        float *out = part + (size_t)blockIdx.x * 32 * 32;
#pragma unroll
        for (int tl = 0; tl < 4; ++tl)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float v = ((red[((0 * 4 + tl) * 4 + r) * 64 + lane] + red[((1 * 4 + tl) * 4 + r) * 64 + lane]) +
                                 red[((2 * 4 + tl) * 4 + r) * 64 + lane]) + red[((3 * 4 + tl) * 4 + r) * 64 + lane];
                const int it = tl >> 1, jt = tl & 1;
                const int k = it * 16 + 4 * (lane >> 4) + r;
                out[(size_t)k * 32 + jt * 16 + (lane & 15)] = v;
            }
    }
}

// out[g][i] = sum over the parts j of group g (j in [g*group, min((g+1)*group, nparts)),
// g = blockIdx.y) of part[j][i], i < n, in a fixed order (deterministic).  Workgroup =
// 16 wavefronts over 64 consecutive i: wavefront w adds the group's parts w, w+16, ...
// (eight loads in flight), then the 16 partial sums of each i are added in order through
// the LDS.
__global__ __launch_bounds__(1024) void k_sum_parts(const float *__restrict__ part, int nparts, int group, int64_t n,
                                                    float *__restrict__ out) {
    __shared__ float red[16][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * 64 + lane;
    const int j0 = blockIdx.y * group, j1 = min(nparts, j0 + group);
    float s = 0.f;
    if (i < n) {
        int j = j0 + g;
        for (; j + 16 * 7 < j1; j += 16 * 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = part[(size_t)(j + 16 * u) * n + i];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; j < j1; j += 16) s += part[(size_t)j * n + i];
    }
    red[g][lane] = s;
    __syncthreads();
    if (g == 0 && i < n) {
        float t = 0.f;
#pragma unroll
        for (int k = 0; k < 16; ++k) t += red[k][lane];
        out[(size_t)blockIdx.y * n + i] = t;
    }
}

// Transpose of a BF16 matrix: out[c][r] = in[r][c] (rows x cols, row strides ldi/ldo).
__global__ void k_transpose16(const uint16_t *__restrict__ in, int64_t rows, int64_t cols, int64_t ldi,
                              uint16_t *__restrict__ out, int64_t ldo) {
    __shared__ uint16_t tile[32][33];
    const int64_t r0 = (int64_t)blockIdx.x * 32, c0 = (int64_t)blockIdx.y * 32;   // rows on x (the long side)
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 256 threads: 32 x 8
    for (int j = ty; j < 32; j += 8) {
        const int64_t r = r0 + j, c = c0 + tx;
        tile[j][tx] = (r < rows && c < cols) ? in[r * ldi + c] : (uint16_t)0;
    }
    __syncthreads();
    for (int j = ty; j < 32; j += 8) {
        const int64_t c = c0 + j, r = r0 + tx;
        if (c < cols && r < rows) out[c * ldo + r] = tile[tx][j];
    }
}

// Gradient through pool + ReLU: dZ[p][co] = dOut[pooled][co] at the window's arg position,
// 0 elsewhere (BF16 [P][32]); the bias gradient (the sum of dOut over windows with a
// chosen element) is accumulated.  Thread = one pooled pixel and 8 channels: two 16-byte
// loads of dOut, one 8-byte load of the decisions, four 16-byte stores (one per window
// position).  Bias partial sums are reduced over the wavefront's lanes of the same
// channel group, then over the workgroup in the LDS, then added to dbias.
__global__ __launch_bounds__(256) void k_unpool(const float *__restrict__ dOut, const uint8_t *__restrict__ arg,
                                                int N, int H, int W, uint16_t *__restrict__ dZ,
                                                float *__restrict__ dbias) {
    __shared__ float sb[4][32];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int H2 = H >> 1, W2 = W >> 1;
    const uint32_t per_img = (uint32_t)(H2 * W2);
    const uint32_t nq = (uint32_t)N * per_img;          // pooled pixels (< 2^31)
    const int grp = lane & 3;                           // channels 8 grp .. 8 grp + 7
    float part[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) part[c] = 0.f;
    const uint32_t stride = gridDim.x * 64u;
    for (uint32_t q = blockIdx.x * 64u + (uint32_t)(threadIdx.x >> 2); q < nq; q += stride) {
        const float4 g0 = *(const float4 *)(dOut + (size_t)q * 32 + 8 * grp);
        const float4 g1 = *(const float4 *)(dOut + (size_t)q * 32 + 8 * grp + 4);
        const uint2 av = *(const uint2 *)(arg + (size_t)q * 32 + 8 * grp);
        const float g[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
        uint32_t a[8];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            a[c] = (av.x >> (8 * c)) & 0xFFu;
            a[c + 4] = (av.y >> (8 * c)) & 0xFFu;
        }
        uint16_t b[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            b[c] = f2bf(g[c]);
            if (a[c] != 255u) part[c] += g[c];
        }
        const uint32_t n = q / per_img, hw = q - n * per_img, h2 = hw / (uint32_t)W2, w2 = hw - h2 * (uint32_t)W2;
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
            uint32_t w[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t lo = a[2 * c] == j ? b[2 * c] : 0u;
                const uint32_t hi = a[2 * c + 1] == j ? b[2 * c + 1] : 0u;
                w[c] = lo | (hi << 16);
            }
            const size_t p = ((size_t)n * H + 2 * h2 + (j >> 1)) * W + 2 * w2 + (j & 1);
            *(uint4 *)(dZ + p * 32 + 8 * grp) = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        float v = part[c];
        v += __shfl_xor(v, 4);
        v += __shfl_xor(v, 8);
        v += __shfl_xor(v, 16);
        v += __shfl_xor(v, 32);
        part[c] = v;
    }
    if (lane < 4) {
#pragma unroll
        for (int c = 0; c < 8; ++c) sb[wave][8 * lane + c] = part[c];
    }
    __syncthreads();
    if (threadIdx.x < 32) {
        const float t = sb[0][threadIdx.x] + sb[1][threadIdx.x] + sb[2][threadIdx.x] + sb[3][threadIdx.x];
        atomicAdd(&dbias[threadIdx.x], t);
    }
}

// --------------------------------------------------- fully connected head (VALU)
// H [Nb][64] FP32 (GEMM output), b1, f2w, f2b -> logits; with labels: mean BCE loss,
// gradients of f2w, f2b, b1 and dH (BF16 [Nb][64] and transposed [64][ldT]).  One
// workgroup of 1024 threads; rows n >= N (batch padding) produce zero gradients.  Sums
// over the candidates run in a fixed order: per hidden unit j, 16 threads add every 16th
// candidate and their partial sums are added in order.
__global__ __launch_bounds__(1024) void k_head(const float *__restrict__ Hm, const float *__restrict__ b1,
                                               const float *__restrict__ f2w, const float *__restrict__ f2b, int N,
                                               int Nb, float *__restrict__ logits, const float *__restrict__ labels,
                                               float *__restrict__ loss, float *__restrict__ g_f2w,
                                               float *__restrict__ g_f2b, float *__restrict__ g_b1,
                                               uint16_t *__restrict__ dH, uint16_t *__restrict__ dHT, int64_t ldT) {
    __shared__ float zl[1024];
    __shared__ float dl[1024];
    __shared__ float pw[16][64], pb[16][64];
    const int tid = threadIdx.x;
    for (int n = tid; n < Nb; n += 1024) {
        float z = 0.f;
        if (n < N) {
            z = f2b[0];
            for (int j = 0; j < 64; ++j) {
                const float h = fmaxf(Hm[(size_t)n * 64 + j] + b1[j], 0.f);
                z += f2w[j] * h;
            }
            logits[n] = z;
        }
        zl[n] = z;
    }
    if (!labels) return;
    __syncthreads();
    for (int n = tid; n < Nb; n += 1024) {
        float g = 0.f, l = 0.f;
        if (n < N) {
            const float z = zl[n], y = labels[n];
            l = fmaxf(z, 0.f) - z * y + log1pf(expf(-fabsf(z)));
            g = (1.f / (1.f + expf(-z)) - y) / (float)N;
        }
        dl[n] = g;
        zl[n] = l;
    }
    __syncthreads();
    {
        const int j = tid & 63, q = tid >> 6;
        float gw = 0.f, gb = 0.f;
        for (int n = q; n < N; n += 16) {
            const float pre = Hm[(size_t)n * 64 + j] + b1[j];
            gw += dl[n] * fmaxf(pre, 0.f);
            gb += pre > 0.f ? dl[n] * f2w[j] : 0.f;
        }
        pw[q][j] = gw;
        pb[q][j] = gb;
    }
    if (tid == 1023) {   // the loss and the output bias gradient: one thread, candidates in order
        float sl = 0.f, sg = 0.f;
        for (int n = 0; n < N; ++n) {
            sl += zl[n];
            sg += dl[n];
        }
        loss[0] = sl / (float)N;
        g_f2b[0] = sg;
    }
    __syncthreads();
    if (tid < 64) {
        float gw = 0.f, gb = 0.f;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            gw += pw[q][tid];
            gb += pb[q][tid];
        }
        g_f2w[tid] = gw;
        g_b1[tid] = gb;
    }
    for (int i = tid; i < Nb * 64; i += 1024) {
        const int n = i >> 6, j = i & 63;
        float g = 0.f;
        if (n < N) {
            const float pre = Hm[(size_t)n * 64 + j] + b1[j];
            g = pre > 0.f ? dl[n] * f2w[j] : 0.f;
        }
        const uint16_t v = f2bf(g);
        dH[i] = v;
        dHT[(size_t)j * ldT + n] = v;
    }
}

// Packed BF16 weights: out[i] = bf16(master[idx[i]]), 0 where idx[i] < 0.
__global__ void k_pack_idx(const float *__restrict__ master, const int32_t *__restrict__ idx, int64_t n,
                           uint16_t *__restrict__ out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t k = idx[i];
        out[i] = k >= 0 ? f2bf(master[k]) : (uint16_t)0;
    }
}

// Gradients of packed weights back to the master layout: master[idx[i]] = in[i] (idx >= 0;
// every master index appears at most once).
__global__ void k_scatter_idx(const float *__restrict__ in, const int32_t *__restrict__ idx, int64_t n,
                              float *__restrict__ master) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t k = idx[i];
        if (k >= 0) master[k] = in[i];
    }
}

__global__ void k_zero_u16(uint16_t *p, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

// Adam on the FP32 master parameters (bias-corrected, step t >= 1).
__global__ void k_adam(float *__restrict__ w, float *__restrict__ m, float *__restrict__ v,
                       const float *__restrict__ g, int64_t n, float lr, float b1, float b2, float eps, float c1,
                       float c2) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        w[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    }
}

__global__ void k_zero_f32(float *p, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.f;
}

// ---------------------------------------------------------------- launchers
#define SPL_HIP_LAUNCH_CHECK() \
    do { hipError_t e__ = hipGetLastError(); if (e__ != hipSuccess) return e__; } while (0)

static unsigned grid_1d(int64_t n) {
    int64_t g = (n + 255) / 256;
    if (g > 65536) g = 65536;
    return (unsigned)(g < 1 ? 1 : g);
}

static hipError_t launch_planes(const DevBeam *beams, int nbeams, const spl_candidate *cands, int64_t n, bool fine,
                                uint16_t *out, hipStream_t s) {
    const unsigned g = (unsigned)(n < 65536 ? 16 * n : 1048576);
    hipLaunchKernelGGL(k_snippets, dim3(g), dim3(256), 0, s, beams, nbeams, cands, n, fine, out);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_snippets(const DevBeam *beams, int nbeams, const spl_candidate *cands, int64_t n, uint16_t *out,
                           hipStream_t s) {
    return n <= 0 ? hipSuccess : launch_planes(beams, nbeams, cands, n, false, out, s);
}

hipError_t launch_fine_dm(const DevBeam *beams, int nbeams, int min_nch, const spl_candidate *cands, int64_t n,
                          double keep, uint16_t *out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const bool aligned = ((uintptr_t)out & 3) == 0;   // atomics, and whole words
    // Slices of the channels: 1536 workgroups are two turns of the 3 that a CU holds (256
    // candidates in 6 slices 1.39 ms, in 4 slices 1.51, in 8 1.40), but more than 24 atomics
    // on one word cost more than they share (32 candidates: 8 slices 393 us, 16 320, 24 283,
    // 48 407; 8 candidates: 24 slices 176 us, 64 205).
    int64_t slices = aligned ? std::min<int64_t>(1536 / n, 24) : 1;
    slices = std::max<int64_t>(1, std::min<int64_t>(slices, min_nch / 64));
    if (slices > 1) {
        if (hipError_t e = launch_zero_f32((float *)out, n * 64 * 256, s); e != hipSuccess) return e;
    }
    const unsigned g = (unsigned)std::min<int64_t>(n * slices, 1048576), gp = (unsigned)std::min<int64_t>(n, 65536);
    if (aligned) {
        hipLaunchKernelGGL(k_fine_sums<true>, dim3(g), dim3(256), 0, s, beams, nbeams, cands, n, keep, (int)slices, out);
        SPL_HIP_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_fine_plane<true>, dim3(gp), dim3(1024), 0, s, beams, nbeams, cands, n, keep, out);
    } else {
        hipLaunchKernelGGL(k_fine_sums<false>, dim3(g), dim3(256), 0, s, beams, nbeams, cands, n, keep, (int)slices, out);
        SPL_HIP_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_fine_plane<false>, dim3(gp), dim3(1024), 0, s, beams, nbeams, cands, n, keep, out);
    }
    SPL_HIP_LAUNCH_CHECK();
    return launch_planes(beams, nbeams, cands, n, true, out, s);   // plane 1, and the zero planes
}

hipError_t launch_gemm(const uint16_t *A, int64_t lda, const uint16_t *B, int64_t ldb, float *C, int64_t ldc, int M,
                       int N, int K, int splits, bool accumulate, hipStream_t s) {
    if (M <= 0 || N <= 0 || K <= 0 || (K & 31) || (lda & 7) || (ldb & 7)) return hipErrorInvalidValue;
    if (splits < 1) splits = 1;
    int klen = (K / 32 + splits - 1) / splits * 32;
    splits = (K + klen - 1) / klen;
    dim3 grid((M + 63) / 64, (N + 31) / 32, splits);
    hipLaunchKernelGGL(k_gemm, grid, dim3(256), 0, s, A, lda, B, ldb, C, ldc, M, N, K, klen,
                       (accumulate || splits > 1) ? 1 : 0);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

template <bool BACK>
static hipError_t launch_conv32(const uint16_t *X, int N, int H, int W, const uint16_t *Wt, float *C, const float *bias,
                                uint16_t *pooled, uint8_t *arg, hipStream_t s) {
    if (N < 1 || (W != 32 && W != 64 && W != 128) || H < 256 / W || H % (256 / W)) return hipErrorInvalidValue;
    const int64_t ntiles = (int64_t)N * H * W / 256;
    const dim3 grid((unsigned)std::min<int64_t>(ntiles, 3 * 256));   // 3 workgroups a CU
    if (W == 128)
        hipLaunchKernelGGL((k_conv32<BACK, 128>), grid, dim3(256), 0, s, X, ntiles, H, Wt, C, bias, pooled, arg);
    else if (W == 64)
        hipLaunchKernelGGL((k_conv32<BACK, 64>), grid, dim3(256), 0, s, X, ntiles, H, Wt, C, bias, pooled, arg);
    else
        hipLaunchKernelGGL((k_conv32<BACK, 32>), grid, dim3(256), 0, s, X, ntiles, H, Wt, C, bias, pooled, arg);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_conv_back(const uint16_t *dZ, int N, int H, int W, const uint16_t *Wt, float *dX, hipStream_t s) {
    return launch_conv32<true>(dZ, N, H, W, Wt, dX, nullptr, nullptr, nullptr, s);
}

hipError_t launch_conv_pool(const uint16_t *X, int N, int H, int W, const uint16_t *Wt, const float *bias,
                            uint16_t *pooled, uint8_t *arg, hipStream_t s) {
    return launch_conv32<false>(X, N, H, W, Wt, nullptr, bias, pooled, arg, s);
}

hipError_t launch_conv_first(const uint16_t *X, int N, int nvalid, int H, int W, const uint16_t *Wt, const float *bias,
                             uint16_t *pooled, uint8_t *arg, hipStream_t s) {
    const int64_t strips = (int64_t)N * (H / 2) * (W / 128);
    if (N < 1 || (H & 1) || (W % 128) || strips > INT32_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_conv_first, dim3((unsigned)strips), dim3(256), 0, s, X, nvalid, H, W, Wt, bias, pooled, arg);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_wgrad_first(const uint16_t *X, int N, int nvalid, int H, int W, const float *dOut, const uint8_t *arg,
                              float *part, int nparts, float *dbias, hipStream_t s) {
    const int64_t P = (int64_t)N * H * W;
    if (P <= 0 || nparts < 1 || (H & 1) || (W & 31) || P >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_wgrad_first, dim3(nparts), dim3(256), 0, s, X, N, nvalid, H, W, dOut, arg, part, dbias);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_wgrad(const uint16_t *X, int N, int H, int W, const uint16_t *dZ, float *part, int nparts,
                        hipStream_t s) {
    const int64_t P = (int64_t)N * H * W;
    if (P <= 0 || (P & 31) || nparts < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_wgrad, dim3(nparts), dim3(256), 0, s, X, N, H, W, dZ, part);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_sum_parts(const float *part, int nparts, int64_t n, float *out, float *tmp, hipStream_t s) {
    const unsigned gx = (unsigned)((n + 63) / 64);
    if (nparts <= 256) {
        hipLaunchKernelGGL(k_sum_parts, dim3(gx), dim3(1024), 0, s, part, nparts, nparts, n, out);
        SPL_HIP_LAUNCH_CHECK();
        return hipSuccess;
    }
    // two passes: groups of 128 parts into tmp [groups][n], then the groups
    const int groups = (nparts + 127) / 128;
    if (groups > kSumPartsMaxGroups) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_sum_parts, dim3(gx, (unsigned)groups), dim3(1024), 0, s, part, nparts, 128, n, tmp);
    SPL_HIP_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_sum_parts, dim3(gx), dim3(1024), 0, s, (const float *)tmp, groups, groups, n, out);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_transpose16(const uint16_t *in, int64_t rows, int64_t cols, int64_t ldi, uint16_t *out, int64_t ldo,
                              hipStream_t s) {
    if ((cols + 31) / 32 > 65535) return hipErrorInvalidValue;
    dim3 grid((unsigned)((rows + 31) / 32), (unsigned)((cols + 31) / 32));
    hipLaunchKernelGGL(k_transpose16, grid, dim3(256), 0, s, in, rows, cols, ldi, out, ldo);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_unpool(const float *dOut, const uint8_t *arg, int N, int H, int W, uint16_t *dZ, float *dbias,
                         hipStream_t s) {
    const int64_t nq = (int64_t)N * (H / 2) * (W / 2);
    if (nq <= 0 || nq >= ((int64_t)1 << 31) || (H & 1) || (W & 1)) return hipErrorInvalidValue;
    const unsigned grid = (unsigned)std::min<int64_t>((nq + 63) / 64, 2048);
    hipLaunchKernelGGL(k_unpool, dim3(grid), dim3(256), 0, s, dOut, arg, N, H, W, dZ, dbias);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_head(const float *Hm, const float *b1, const float *f2w, const float *f2b, int N, int Nb,
                       float *logits, const float *labels, float *loss, float *g_f2w, float *g_f2b, float *g_b1,
                       uint16_t *dH, uint16_t *dHT, int64_t ldT, hipStream_t s) {
    if (Nb > 1024) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_head, dim3(1), dim3(1024), 0, s, Hm, b1, f2w, f2b, N, Nb, logits, labels, loss, g_f2w, g_f2b,
                       g_b1, dH, dHT, ldT);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_pack_idx(const float *master, const int32_t *idx, int64_t n, uint16_t *out, hipStream_t s) {
    hipLaunchKernelGGL(k_pack_idx, dim3(grid_1d(n)), dim3(256), 0, s, master, idx, n, out);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_scatter_idx(const float *in, const int32_t *idx, int64_t n, float *master, hipStream_t s) {
    hipLaunchKernelGGL(k_scatter_idx, dim3(grid_1d(n)), dim3(256), 0, s, in, idx, n, master);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_zero_u16(uint16_t *p, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero_u16, dim3(grid_1d(n)), dim3(256), 0, s, p, n);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_adam(float *w, float *m, float *v, const float *g, int64_t n, float lr, float b1, float b2, float eps,
                       int64_t t, hipStream_t s) {
    const float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
    hipLaunchKernelGGL(k_adam, dim3(grid_1d(n)), dim3(256), 0, s, w, m, v, g, n, lr, b1, b2, eps, c1, c2);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

hipError_t launch_zero_f32(float *p, int64_t n, hipStream_t s) {
    hipLaunchKernelGGL(k_zero_f32, dim3(grid_1d(n)), dim3(256), 0, s, p, n);
    SPL_HIP_LAUNCH_CHECK();
    return hipSuccess;
}

}  // namespace spl
