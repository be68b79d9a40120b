// Launchers of the HIP kernels (kernels.hip); every call enqueues on stream `s` and
// returns the launch status.
#pragma once

#include "shared_sums.h"
#include "spl_internal.h"
#include "spotlight.h"

namespace spl {

// Staged rows per wavefront and chunk: chan_chunk <= dedisp_stage_rows(buffers) * waves
// (one LDS buffer: two rows; two buffers: one row each, so two buffers of a 16-wavefront
// tile hold what one buffer of 32 channels holds).
constexpr int dedisp_stage_rows(int buffers) { return buffers == 2 ? 1 : 2; }
// A staged row holds up to 1024 * sv bytes (sv = 16-byte vectors per lane, 1 or 2);
// nbuf = LDS buffers (1 or 2).
bool dedisp_shape_supported(int dw, int j, int nw, int sv, int nbuf);
hipError_t prepare_dedisp(int dw, int j, int nw, int sv, int nbuf, size_t lds_bytes, int *blocks_per_cu);
hipError_t launch_dedisp(int dw, int j, int nw, int sv, int nbuf, const DevBeam *beams, const DedispItem *items,
                         int item_lo, int item_hi, int *queue, int grid, size_t lds_bytes, hipStream_t s);
// The shape whose kernel reads the samples where they are: it stages no rows, and chan_chunk
// and lds_bytes mean nothing to it.
constexpr bool dedisp_direct(int dw, int j, int nw) { return dw == 4 && j == 1 && nw == 4; }
// The same kernel over one beam whatever its tiling, with no work items and no tables but the
// delays; rows may lie any distance apart.
hipError_t launch_dedisp_beam(const DevBeam *beams, int beam, int ndm, int n_dd, hipStream_t s);
// The shared-row kernel, which addresses 16 rows by 32-bit offsets: rows lie less than kSharedPitch
// bytes apart; lds_bytes holds both row buffers.
constexpr int64_t kSharedPitch = (int64_t)1 << 28;
hipError_t prepare_dedisp_shared(const SharedShape &s, size_t lds_bytes, int *blocks_per_cu);
hipError_t launch_dedisp_shared(const SharedShape &s, const DevBeam *beams, const DedispItem *items, int item_lo,
                                int item_hi, int *queue, int grid, size_t lds_bytes, hipStream_t stream);
hipError_t launch_thresholds(const DevBeam *beams, int beam_lo, int beam_hi, int row_lo, int row_hi,
                             hipStream_t s);
// Zeroes up to three ranges of 8-byte words.
hipError_t launch_clear(uint64_t *a, int64_t na, uint64_t *b, int64_t nb, uint64_t *c, int64_t nc, hipStream_t s);
// Boxcar hits of chunks [chunk_lo, chunk_hi) in one launch (decoupled look-back): status
// holds chunk_hi - chunk_lo words and ticket one, zero at the start, offsets gets each chunk's first
// hit index, hit_t the hits' times, *n_total the range's hit count; *stall is set if a
// look-back gave up.
hipError_t launch_boxcar_one_pass(const DevBeam *beams, int beam_lo, int beam_hi, int chunk_lo, int chunk_hi,
                                  int w_max, uint64_t *status, uint64_t *ticket, int64_t *offsets, Hit *hits,
                                  int32_t *hit_t, int64_t cap, int64_t *n_total, int32_t *stall, hipStream_t s);
// Chunks of kScanPerBlock hits in a list (the shortest in use): the look-back words of launch_compact and launch_candidates are
// one more (the ticket counter), and are cleared by the launch_rows call of the list before.
int scan_blocks(int64_t n_max);
// Row starts of the boxcar's hits, or of launch_compact's survivors (start_before, pos and
// n_before those of the list they were taken from), and the block index of the rows:
// blk[r][b] = index within row r of its first hit with t >= 64 b (the row's count when none);
// 64 nblk > the largest t.
hipError_t launch_rows_first(const DevBeam *beams, int beam_lo, int beam_hi, int row_lo, int n_rows, int chunk_lo,
                             const int64_t *chunk_off, const int64_t *n_hits, int64_t cap, int64_t *row_start,
                             const int32_t *hit_t, int32_t *blk, int nblk, uint64_t *status, hipStream_t s);
hipError_t launch_rows_survivors(int n_rows, const int64_t *start_before, const int64_t *pos, const int64_t *n_before,
                                 const int64_t *n_list, int64_t cap, int64_t *row_start, const int32_t *hit_t,
                                 int32_t *blk, int nblk, uint64_t *status, hipStream_t s);
// The survivors of a peak filter (alive flags) compacted in order into out, with their times
// in hit_t and the survivors before each hit in pos; *n_out their count.
hipError_t launch_compact(const Hit *hits, const int64_t *n_hits, int64_t cap, const uint8_t *alive, uint64_t *status,
                          Hit *out, int32_t *hit_t, int64_t *pos, int64_t *n_out, int32_t *stall, hipStream_t s);
hipError_t launch_nms(const DevBeam *beams, int beam_lo, int beam_hi, int row_lo, const Hit *hits,
                      const int64_t *n_hits, int64_t cap, const int64_t *row_start, const int32_t *blk, int nblk,
                      int stencil, const uint8_t *alive_in, uint8_t *alive_out, int64_t *n_alive,
                      const int32_t *hit_t, hipStream_t s);
// Candidate records of the survivors in order (alive null: of every hit, and *n_out is left
// as it is), after *base earlier ones; *n_out their count.
hipError_t launch_candidates(const DevBeam *beams, int beam_lo, int beam_hi, const Hit *hits, const int64_t *n_hits,
                             int64_t cap, const uint8_t *alive, uint64_t *status, const int64_t *base, int64_t *n_out,
                             int32_t *stall, spl_candidate *cands, int64_t cand_cap, hipStream_t s);
// End of a beam range; last: also of the run's statistics.
hipError_t launch_pass_end(DevRun *run, uint64_t *box_ticket, spl_run_stats *stats, int64_t hit_cap, int nst, bool last,
                           int64_t cand_cap, hipStream_t s);
hipError_t launch_checksum(const int32_t *X, int ndm, int xpitch, int n_dd, unsigned long long *out,
                           hipStream_t s);
hipError_t launch_mu_sigma(const int64_t *n, const int64_t *s1, const int64_t *s2, int64_t count, double *mu,
                           double *sigma, hipStream_t s);

}  // namespace spl
