// Shared partial sums of the dedispersion: tables that tell k_dedisp_shared which sums
// over a few adjacent channels the trials of a tile have in common.
//
// The delays of a run of adjacent channels, taken relative to the run's first channel,
// repeat from trial to trial: over the 64 trials of a tile some ten channels of the
// 4096-channel band show fifteen different patterns.  A row of sums per pattern is formed
// once per tile, and every trial then adds one row, shifted by the first channel's delay,
// in place of the run's channels one by one.  The sums are the same integers.
//
// Per tile of td trials the channels are cut into runs (greedily, first channel first) of
// at most 16 channels with at most 16 patterns.  A channel's samples are read from an
// aligned dword on, and every pattern takes them at most 4 samples later, so that the
// bytes of four consecutive elements lie in two dwords; a run's rows may start up to 3
// samples early where that keeps more of its channels within those 4.  The runs of a tile are gathered
// into chunks, staged together.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <vector>

namespace spl {

// A shape of the kernel: 8 summing wavefronts of dw trials, tiles of 128 m samples held as
// packed pairs (t, t + 64 m); np staging wavefronts, each forming up to gp groups of 64
// elements per item.
struct SharedShape {
    int np = 0, dw = 0, m = 0, gp = 0;
    int td() const { return 8 * dw; }
    int half() const { return 64 * m; }
    bool operator==(const SharedShape &o) const { return np == o.np && dw == o.dw && m == o.m && gp == o.gp; }
};

constexpr int kSharedChans = 16;      // channels of a run
constexpr int kSharedPatterns = 16;   // patterns of a run (rows of the matrix product)
constexpr int kSharedLate = 4;        // samples a pattern may lie behind its channel's aligned start
constexpr int kSharedBuffer = 79 * 1024;   // LDS bytes of one of the two row buffers
constexpr int kSharedRun = kSharedBuffer / 2;   // LDS bytes of a run: two share a chunk
constexpr int kSharedBlock = 64;      // int32 of a summing wavefront's block of a chunk

// Staging item: one wavefront forms up to gp groups of 64 packed elements of every pattern
// row of a run.  The items of a chunk are dealt to the wavefronts in rounds.
struct SharedItem {
    int32_t sub;        // run (index into the per-run tables)
    int32_t png;        // patterns | channels << 8 | first group << 16 | groups << 24 (0: none)
    int32_t lds;        // byte offset in the buffer of the run's row 0, element 64 * first group
    int32_t row_bytes;  // LDS bytes of a row
    int32_t c0;         // channels c0 .. c0 + 15 are read
    int32_t last;       // 1: the chunk's last round
    int32_t pad[2];     // 8 words: lane l & 7 of a staging wavefront loads word l
};
// A summing wavefront's block of a chunk (kSharedBlock int32, read lane by lane): runs |
// channels << 8 (where the 16-bit fields' high bytes move on after the chunk: the channels
// summed since they last did; else 0), then the LDS byte offsets of its dw trials' rows,
// run by run.
struct SharedTile {
    int32_t round, nrounds, chunk, nchunks;
};

// The tables of one plan and shape; offsets in bytes from the blob's start.
struct SharedTables {
    SharedShape shape;
    int ntiles = 0, nsubs = 0, nrounds = 0, nchunks = 0;
    int buffer = 0;          // LDS bytes of one buffer, the largest chunk's
    double clocks = 0;       // modelled clocks of a CU for one time tile of every DM tile
    std::vector<uint8_t> blob;
    // items [round][np wavefronts]; blocks [chunk][8 wavefronts][kSharedBlock]; taps
    // [run][4 q][4 p][4 k] uint32: of pattern 4 k + p (past the last: of the last) and the
    // channels 2q, 2q + 1, 8 + 2q, 9 + 2q: in six bits from 6 u on 8 times the samples after
    // the channel's start, bit 24 + u where the run has the channel; starts [run][4 q][4]
    // those channels' first samples from t0 (multiples of 4)
    size_t off_items = 0, off_blocks = 0, off_taps = 0, off_starts = 0;
};

// Builds the tables for delays [ndm][nch] (rows past ndm repeat the last trial).  False
// when nch is not in [16, 65536], a run of one channel does not fit the shape, the tables exceed
// max_bytes, their clocks are seen to exceed max_clocks by far, or memory runs out.
bool build_shared(const int32_t *delays, int ndm, int nch, SharedShape shape, size_t max_bytes, double max_clocks,
                  SharedTables *out);

// Delays [ntiles * td][nch] that the tables encode (for checking them on the host).
void decode_shared(const SharedTables &t, int nch, std::vector<int32_t> *out);

}  // namespace spl
