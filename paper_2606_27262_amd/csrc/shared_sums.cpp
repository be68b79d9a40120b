// Host half of the shared partial sums: cuts each DM tile's channels into runs, finds the
// runs' delay patterns and lays the kernel's tables out (see shared_sums.h).
#include "shared_sums.h"

#include <algorithm>
#include <atomic>
#include <cstring>
#include <new>
#include <system_error>
#include <thread>

namespace spl {

namespace {

constexpr int kSumming = 8;   // summing wavefronts
constexpr int kMaxTrials = 64;
constexpr int kTaps = 64;   // words of a run

// One run of channels of one tile.
struct Run {
    int c0, n, patterns, groups;         // groups: row elements / 64
    uint8_t pattern[kMaxTrials];         // of every trial
    int32_t shift[kMaxTrials];           // delay of channel c0 less its smallest
    uint8_t e[kSharedPatterns][kSharedChans];   // samples of (pattern, channel) after start, 0..4
    int32_t start[kSharedChans];         // first sample of the channel's rows from t0, a multiple of 4
};

// The longest run starting at channel c0, from the delays rows[trial][channel] of a tile.
bool make_run(const int32_t *const *rows, int td, int nch, int c0, const SharedShape &sh, Run *r) {
    const int half = sh.half();
    int32_t lo = rows[0][c0], hi = lo;
    int32_t first[kMaxTrials];
    for (int d = 0; d < td; ++d) {
        first[d] = rows[d][c0];
        lo = std::min(lo, first[d]);
        hi = std::max(hi, first[d]);
    }
    r->c0 = c0;
    r->n = 1;
    r->patterns = 1;
    const int64_t groups = ((int64_t)half + (hi - lo) + 3 + 63) / 64;   // rows may start 3 samples early
    if (groups > 255 || groups * 256 > kSharedRun) return false;
    r->groups = (int)groups;
    const int most = (int)std::min<int64_t>(kSharedPatterns, kSharedRun / (groups * 256));
    std::memset(r->pattern, 0, sizeof r->pattern);
    r->e[0][0] = 0;
    r->start[0] = lo;
    uint32_t early = 15;   // bit s: rows starting s samples early keep every channel within kSharedLate
    while (r->n < kSharedChans && c0 + r->n < nch) {
        const int c = c0 + r->n;
        int32_t dl[kMaxTrials], least = INT32_MAX, largest = INT32_MIN;
        for (int d = 0; d < td; ++d) {
            dl[d] = rows[d][c] - first[d];
            least = std::min(least, dl[d]);
            largest = std::max(largest, dl[d]);
        }
        uint32_t ok = 0;
        for (int s = 0; s < 4; ++s)
            if (((lo + least - s) & 3) + (largest - least) <= kSharedLate) ok |= 1u << s;
        ok &= early;
        if (!ok) break;
        // (pattern so far, extra delay) -> pattern
        int8_t id[kSharedPatterns * (kSharedLate + 1)];
        uint8_t from[kSharedPatterns], extra[kSharedPatterns], next[kMaxTrials];
        std::memset(id, -1, sizeof id);
        int np = 0;
        bool fits = true;
        for (int d = 0; d < td; ++d) {
            const int key = r->pattern[d] * (kSharedLate + 1) + (dl[d] - least);
            if (id[key] < 0) {
                if (np == most) {
                    fits = false;
                    break;
                }
                from[np] = r->pattern[d];
                extra[np] = (uint8_t)(dl[d] - least);
                id[key] = (int8_t)np++;
            }
            next[d] = (uint8_t)id[key];
        }
        if (!fits) break;
        uint8_t old[kSharedPatterns][kSharedChans];
        std::memcpy(old, r->e, sizeof old);
        for (int p = 0; p < np; ++p) {
            std::memcpy(r->e[p], old[from[p]], r->n);
            r->e[p][r->n] = extra[p];
        }
        std::memcpy(r->pattern, next, td);
        r->start[r->n] = lo + least;
        r->patterns = np;
        early = ok;
        ++r->n;
    }
    int s = 0;
    while (!(early >> s & 1)) ++s;
    for (int d = 0; d < td; ++d) r->shift[d] = first[d] - lo + s;
    for (int c = 0; c < r->n; ++c) {
        const int32_t at = r->start[c] - s, aligned = at & ~3;
        r->start[c] = aligned;
        for (int p = 0; p < r->patterns; ++p) r->e[p][c] = (uint8_t)(r->e[p][c] + (at - aligned));
    }
    return true;
}

// The tables of one tile, counted from its own first run.
struct Tile {
    std::vector<SharedItem> items;
    std::vector<int32_t> blocks, starts;
    std::vector<uint32_t> taps;
    std::vector<int> channels;   // of every chunk
    int buffer = 0;
    double clocks = 0;
    bool ok = false;
};

// (delay rows lie `stride` entries apart)
void build_tile(const int32_t *delays, int stride, int ndm, int nch, const SharedShape &sh, int k, Tile *o) {
    const int td = sh.td();
    const int max_runs = (kSharedBlock - 1) / sh.dw;   // rows of a chunk's runs fit the block
    std::vector<Run> in_chunk;
    const int32_t *rows[kMaxTrials];
    // the channels ahead of a run, copied together
    std::vector<int32_t> block((size_t)kMaxTrials * 64);
    int used_bytes = 0;
    auto close_chunk = [&]() {
        if (in_chunk.empty()) return;
        const size_t base = o->blocks.size();
        o->blocks.resize(base + (size_t)kSumming * kSharedBlock, 0);
        auto block = [&](int wave) { return o->blocks.data() + base + (size_t)wave * kSharedBlock; };
        for (int w = 0; w < kSumming; ++w) block(w)[0] = (int32_t)in_chunk.size();
        std::vector<SharedItem> first_item;   // of every run
        int lds = 0, chans = 0, groups = 0;
        for (size_t ri = 0; ri < in_chunk.size(); ++ri) {
            const Run &r = in_chunk[ri];
            const int sub = (int)(o->taps.size() / kTaps);
            const int rb = r.groups * 256;
            // all 16 channels read exist: a run at the band's end moves up
            const int col0 = std::min(r.c0, nch - kSharedChans), skip = r.c0 - col0;
            int32_t start[kSharedChans];
            for (int c = 0; c < kSharedChans; ++c)
                start[c] = r.start[std::max(0, std::min(c - skip, r.n - 1))];
            SharedItem it{};
            it.sub = sub;
            it.row_bytes = rb;
            it.c0 = col0;
            it.lds = lds;
            first_item.push_back(it);
            groups += r.groups;
            for (int i = 0; i < kTaps; ++i) {
                const int q = i / 16, p = std::min(4 * (i % 4) + i / 4 % 4, r.patterns - 1);
                uint32_t v = 0;
                for (int u = 0; u < 4; ++u) {
                    const int c = 8 * (u >> 1) + 2 * q + (u & 1) - skip;
                    if (c >= 0 && c < r.n) v |= 1u << (24 + u) | 8u * r.e[p][c] << (6 * u);
                }
                o->taps.push_back(v);
            }
            for (int q = 0; q < 4; ++q)
                for (int u = 0; u < 4; ++u) o->starts.push_back(start[8 * (u >> 1) + 2 * q + (u & 1)]);
            for (int d = 0; d < td; ++d)
                block(d / sh.dw)[1 + ri * sh.dw + d % sh.dw] = lds + r.pattern[d] * rb + r.shift[d] * 4;
            lds += r.patterns * rb;
            chans += r.n;
        }
        // the chunk's groups dealt to the staging wavefronts in items of one run each; an
        // item costs its groups and about one more, `most` is the least that a wavefront
        // can be asked for
        std::vector<std::vector<SharedItem>> part;
        int rounds = 1;
        for (int most = 1 + groups / sh.np;; ++most) {
            part.assign(sh.np, {});
            rounds = 1;
            size_t run = 0;
            int g = 0;
            for (int w = 0; w < sh.np; ++w) {
                for (int left = most; left > 1 && run < in_chunk.size();) {
                    const Run &r = in_chunk[run];
                    const int ng = std::min(std::min(left - 1, r.groups - g), sh.gp);
                    SharedItem it = first_item[run];
                    it.png = (int32_t)((uint32_t)r.patterns | (uint32_t)r.n << 8 | (uint32_t)g << 16 |
                                       (uint32_t)ng << 24);
                    it.lds += g * 256;
                    part[w].push_back(it);
                    left -= ng + 1;
                    g += ng;
                    if (g == r.groups) {
                        ++run;
                        g = 0;
                    }
                }
                rounds = std::max(rounds, (int)part[w].size());
            }
            if (run == in_chunk.size()) break;
        }
        for (int i = 0; i < rounds; ++i)
            for (int w = 0; w < sh.np; ++w) {
                // an empty item names an existing run: its tables are loaded all the same
                SharedItem it = i < (int)part[w].size() ? part[w][i] : part[w].empty() ? first_item[0] : part[w].back();
                if (i >= (int)part[w].size()) it.png &= 0xFFFFFF;
                it.last = i + 1 == rounds;
                o->items.push_back(it);
            }
        o->buffer = std::max(o->buffer, lds);
        o->channels.push_back(chans);
        // modelled clocks of a CU: a staging wavefront takes about 650 per group, 690 per
        // item and 470 for the chunk's hand-over (the 4096-channel band: 4850 per chunk of
        // 21.8 groups in 1.16 rounds)
        o->clocks += (double)groups / sh.np * 650.0 + rounds * 690.0 + 470.0;
        in_chunk.clear();
        used_bytes = 0;
    };
    int c = 0, block_c0 = 0, block_n = 0;
    while (c < nch) {
        if (c + kSharedChans > block_c0 + block_n && block_c0 + block_n < nch) {
            block_c0 = c;
            block_n = std::min(64, nch - c);
            for (int d = 0; d < td; ++d) {
                const int ds = std::min(k * td + d, ndm - 1);
                std::memcpy(block.data() + (size_t)d * 64, delays + (size_t)ds * stride + c,
                            (size_t)block_n * sizeof(int32_t));
                rows[d] = block.data() + (size_t)d * 64;
            }
        }
        Run r;
        if (!make_run(rows, td, block_n, c - block_c0, sh, &r)) return;
        r.c0 = c;
        const int bytes = r.patterns * r.groups * 256;
        if (used_bytes + bytes > kSharedBuffer || (int)in_chunk.size() == max_runs) close_chunk();
        used_bytes += bytes;
        in_chunk.push_back(r);
        c += r.n;
    }
    close_chunk();
    // the 16-bit fields hold a low byte and 256 channels of 255: the high bytes move on
    // before the chunk that would exceed that
    const int nchunks = (int)o->channels.size();
    for (int j = 0, pending = 0; j < nchunks; ++j) {
        pending += o->channels[j];
        if (j + 1 < nchunks && pending + o->channels[j + 1] <= 256) continue;
        for (int w = 0; w < kSumming; ++w) o->blocks[((size_t)j * kSumming + w) * kSharedBlock] |= pending << 8;
        pending = 0;
    }
    o->ok = true;
}

// Threads that are joined whatever ends the scope.
struct Helpers {
    std::vector<std::thread> threads;
    ~Helpers() {
        for (std::thread &t : threads) t.join();
    }
};

bool build(const int32_t *delays, int ndm, int nch, SharedShape sh, size_t max_bytes, double max_clocks,
           SharedTables *out) {
    const int td = sh.td(), ntiles = (ndm + td - 1) / td;
    if (td < 1 || td > kMaxTrials || nch < kSharedChans || nch > 65536 || ndm < 1) return false;
    std::vector<Tile> tiles(ntiles);
    // 128 channels in the middle speak for the others: a plan far from worth it is not built
    const int some = std::min(nch, 128);
    Tile probe;
    build_tile(delays + (nch - some) / 2, nch, ndm, some, sh, ntiles / 2, &probe);
    if (!probe.ok || probe.clocks * nch / some * ntiles > 1.5 * max_clocks) return false;
    std::atomic<int> next{0};
    auto work = [&]() {
        for (int k; (k = next.fetch_add(1)) < ntiles;) {
            try {
                build_tile(delays, nch, ndm, nch, sh, k, &tiles[k]);
            } catch (const std::bad_alloc &) {   // not ok: no tables
            }
        }
    };
    // a tile of the 4096-channel band takes 2.5 ms: helpers from a few tiles of such size on
    const int64_t size = (int64_t)ntiles * td * nch;
    const int n_help = size < (1 << 18) ? 0 : std::min({7, ntiles - 1, (int)std::thread::hardware_concurrency() - 1});
    {
        Helpers helpers;
        try {
            for (int i = 0; i < n_help; ++i) helpers.threads.emplace_back(work);
        } catch (const std::system_error &) {   // fewer helpers
        } catch (const std::bad_alloc &) {
        }
        work();
    }

    size_t n_items = 0, n_blocks = 0, n_taps = 0, n_starts = 0;
    SharedTables &t = *out;
    t.buffer = 0;
    t.clocks = 0;
    for (const Tile &o : tiles) {
        if (!o.ok) return false;
        n_items += o.items.size();
        n_blocks += o.blocks.size();
        n_taps += o.taps.size();
        n_starts += o.starts.size();
        t.buffer = std::max(t.buffer, o.buffer);
        t.clocks += o.clocks;
    }
    t.shape = sh;
    t.ntiles = ntiles;
    t.nsubs = (int)(n_taps / kTaps);
    t.nrounds = (int)(n_items / sh.np);
    t.nchunks = (int)(n_blocks / ((size_t)kSumming * kSharedBlock));
    auto up = [](size_t v) { return (v + 127) & ~(size_t)127; };
    t.off_items = up(ntiles * sizeof(SharedTile));
    t.off_blocks = up(t.off_items + n_items * sizeof(SharedItem));
    t.off_taps = up(t.off_blocks + n_blocks * sizeof(int32_t));
    t.off_starts = up(t.off_taps + n_taps * sizeof(uint32_t));
    const size_t bytes = up(t.off_starts + n_starts * sizeof(int32_t));
    if (bytes > max_bytes || bytes > INT32_MAX) return false;
    t.blob.assign(bytes, 0);
    SharedTile *tile = (SharedTile *)t.blob.data();
    SharedItem *items = (SharedItem *)(t.blob.data() + t.off_items);
    int32_t *blocks = (int32_t *)(t.blob.data() + t.off_blocks);
    uint32_t *taps = (uint32_t *)(t.blob.data() + t.off_taps);
    int32_t *starts = (int32_t *)(t.blob.data() + t.off_starts);
    int round = 0, chunk = 0, sub = 0;
    for (const Tile &o : tiles) {
        tile->round = round;
        tile->nrounds = (int32_t)(o.items.size() / sh.np);
        tile->chunk = chunk;
        tile->nchunks = (int32_t)o.channels.size();
        round += tile->nrounds;
        chunk += tile->nchunks;
        ++tile;
        for (SharedItem it : o.items) {
            it.sub += sub;
            *items++ = it;
        }
        sub += (int)(o.taps.size() / kTaps);
        blocks = std::copy(o.blocks.begin(), o.blocks.end(), blocks);
        taps = std::copy(o.taps.begin(), o.taps.end(), taps);
        starts = std::copy(o.starts.begin(), o.starts.end(), starts);
    }
    return true;
}

}  // namespace

bool build_shared(const int32_t *delays, int ndm, int nch, SharedShape sh, size_t max_bytes, double max_clocks,
                  SharedTables *out) {
    try {
        return build(delays, ndm, nch, sh, max_bytes, max_clocks, out);
    } catch (const std::bad_alloc &) {   // (no exception leaves the C ABI: the plan goes without tables)
        return false;
    }
}

void decode_shared(const SharedTables &t, int nch, std::vector<int32_t> *out) {
    const int td = t.shape.td(), dw = t.shape.dw;
    out->assign((size_t)t.ntiles * td * nch, -1);
    const uint8_t *b = t.blob.data();
    const SharedTile *tiles = (const SharedTile *)b;
    const SharedItem *items = (const SharedItem *)(b + t.off_items);
    const int32_t *blocks = (const int32_t *)(b + t.off_blocks);
    const uint32_t *taps = (const uint32_t *)(b + t.off_taps);
    const int32_t *starts = (const int32_t *)(b + t.off_starts);
    for (int k = 0; k < t.ntiles; ++k) {
        int pending = 0;   // channels in the 16-bit fields
        int round = tiles[k].round;
        for (int j = tiles[k].chunk; j < tiles[k].chunk + tiles[k].nchunks; ++j) {
            auto block = [&](int w) { return blocks + ((size_t)j * kSumming + w) * kSharedBlock; };
            std::vector<SharedItem> mine;   // the chunk's items
            for (bool last = false; !last && round < tiles[k].round + tiles[k].nrounds; ++round)
                for (int w = 0; w < t.shape.np; ++w) {
                    const SharedItem &it = items[(size_t)round * t.shape.np + w];
                    last = it.last != 0;
                    if ((uint32_t)it.png >> 24) mine.push_back(it);
                }
            std::sort(mine.begin(), mine.end(), [](const SharedItem &a, const SharedItem &b) { return a.lds < b.lds; });
            const int runs = block(0)[0] & 255;
            int ri = 0;
            for (const SharedItem &it : mine) {
                if ((it.png >> 16) & 255) continue;   // a run's first item names it
                const int np = it.png & 255, n = (it.png >> 8) & 255;
                int groups = 0;   // staged groups of the run, each at its place
                for (const SharedItem &o : mine) {
                    const int g0 = (o.png >> 16) & 255, ng = (int)((uint32_t)o.png >> 24);
                    if (o.sub != it.sub || o.lds != it.lds + 256 * g0 || o.row_bytes != it.row_bytes ||
                        o.c0 != it.c0 || g0 != groups || ng < 1 || ng > t.shape.gp)
                        continue;
                    groups += ng;
                }
                bool good = groups * 256 == it.row_bytes && it.lds + np * it.row_bytes <= t.buffer && ri < runs &&
                            it.c0 >= 0 && it.c0 + kSharedChans <= nch;
                pending += n;
                good = good && pending <= 256;
                for (int d = 0; d < td; ++d) {
                    const int off = block(d / dw)[1 + ri * dw + d % dw] - it.lds;
                    const int p = off / it.row_bytes, shift = (off % it.row_bytes) / 4;
                    int taken = 0;
                    for (int c = 0; c < kSharedChans && off >= 0 && p < np; ++c) {
                        const int q = (c % 8) / 2, u = 2 * (c / 8) + c % 2;
                        auto tap = [&](int pattern) {
                            const uint32_t v = taps[(size_t)it.sub * kTaps + 16 * q + 4 * (pattern % 4) + pattern / 4];
                            const int at = (int)((v >> (6 * u)) & 63u);
                            return !(v >> (24 + u) & 1u) ? -1 : at % 8 == 0 ? at / 8 : 99;
                        };
                        const int e = tap(p);
                        bool same = true;   // the patterns past the last repeat it
                        for (int past = np; past < kSharedPatterns && p + 1 == np; ++past) same = same && tap(past) == e;
                        if (e < 0 && same) continue;
                        ++taken;
                        const int s = starts[(size_t)it.sub * 16 + 4 * q + u];
                        int32_t &o = (*out)[((size_t)k * td + d) * nch + it.c0 + c];
                        const bool fine = good && o == -1 && same && e <= kSharedLate && !(off & 3) &&
                                          !(s & 3) && shift * 4 + t.shape.half() * 4 <= it.row_bytes;
                        o = fine ? s + shift + e : -2;
                    }
                    if (taken != n) (*out)[((size_t)k * td + d) * nch + it.c0] = -2;
                }
                ++ri;
            }
            for (int w = 0; w < kSumming; ++w)
                if (block(w)[0] != block(0)[0] || ri != runs) (*out)[(size_t)k * td * nch] = -2;
            if (block(0)[0] >> 8) {
                if (block(0)[0] >> 8 != pending) (*out)[(size_t)k * td * nch] = -2;
                pending = 0;
            }
        }
        if (pending || round != tiles[k].round + tiles[k].nrounds) (*out)[(size_t)k * td * nch] = -2;
    }
}

}  // namespace spl
