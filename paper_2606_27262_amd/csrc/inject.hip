// Quantised-domain injection (the appendix on injecting a signal into an M-bit quantised
// stream): every sample of a signal window moves from its state n to a state k >= n
// with the probability that Gaussian noise known to lie in state n, shifted by the
// signal, lands in state k.
//
// One wave per (window, channel) row, its lanes on 64 consecutive samples at a time, so
// the byte loads and stores and the FP32/u32 window loads are coalesced; zero signal
// (the padding of narrow bursts) costs one load.  The work is
// binary64 arithmetic (an erfc per sample), not memory: a burst's window holds
// ~10^5-10^6 values per beam.
//
// The transition row is never formed.  The cumulative row sum up to state k is the mass
// of [e_{n-1}, min(e_n, e_k - S)) over the mass of state n, monotone in k: SAMPLE mode
// takes the first k where it exceeds u; ARGMAX compares the masses of the
// candidate states, successive differences of that cumulative mass.  Only states whose
// shifted interval can meet state n are visited: from n + floor(S/w) - 1 to
// n + floor(S/w) + 2 (w the state width), one state of slack on each side for rounding;
// state 0, unbounded below, can reach any state up to the last of those.
#include <hip/hip_runtime.h>

#include <cmath>

#include "inject.h"

namespace spl {

namespace {

struct Edges {
    double mu, sigma, width, offset;
    int half, top;

    // Upper edge of state k (k in [-1, top)): -inf below state 0.
    __device__ double edge(int k) const {
        if (k < 0) return -INFINITY;
        return mu + ((double)(k + 1 - half) + offset) * width;
    }
};

// Gaussian mass inside one state [lo, hi), measured from lo: g(x) = mass of
// [lo, min(x, hi)).  All values come from one tail of the distribution (the upper one
// for a state above the mean), so the narrow differences near the band's ends keep
// their relative precision; one erfc per evaluation.  The mass below lo and the state's
// own (two erfc) are the same for every sample of a state and come from a table.
struct StateMass {
    double mu, inv_sigma, lo, hi, f_lo, den;
    bool upper;

    __device__ double tail(double x) const {
        const double z = (x - mu) * inv_sigma * 0.70710678118654752440;   // 1/sqrt(2)
        return 0.5 * erfc(upper ? z : -z);   // one call: the states of a wavefront lie on both sides
    }
    __device__ void edges(const Edges &E, int n) {
        mu = E.mu;
        inv_sigma = 1.0 / E.sigma;
        lo = E.edge(n - 1);
        hi = E.edge(n);
        upper = lo >= E.mu;
    }
    __device__ void masses() {
        f_lo = tail(lo);
        const double f_hi = tail(hi);
        den = upper ? f_lo - f_hi : f_hi - f_lo;
    }
    __device__ double inside(double x) const { return upper ? f_lo - tail(x) : tail(x) - f_lo; }   // lo < x < hi
    __device__ double g(double x) const {
        if (!(x > lo)) return 0.0;
        if (x >= hi) return den;
        return inside(x);
    }
};

// n < top; S > 0.  The edges e_k - S lie one state width apart, so (state 0 aside, which has
// no lower edge) one of them, two at most by rounding, lies inside state n: the states before
// it receive nothing, those after it the rest, and one erfc a sample decides.
template <bool ARGMAX>
__device__ int new_state(const Edges &E, const StateMass &M, int n, double S, uint32_t word) {
    if (!(M.den > 0.0)) return n;
    const double f = fmin(floor(S / E.width), (double)(E.top + 2));
    const int shift = (int)f;
    int k_lo = n == 0 ? 0 : min(E.top, max(n, n + shift - 1));
    int k_hi = min(E.top, n + shift + 2);
    int k_in = k_lo;   // the first state whose shifted upper edge lies above lo
    if (n > 0)
        while (k_in < k_hi && k_in < E.top && !(E.edge(k_in) - S > M.lo)) ++k_in;
    if constexpr (ARGMAX) {
        // mass landing in state k: g(e_k - S) - g(e_{k-1} - S); the top state takes the rest
        const double x_in = E.edge(k_in) - S;
        const double g_in = n > 0 && k_in < E.top && x_in > M.lo && x_in < M.hi ? M.inside(x_in) : 0.0;
        auto mass_below = [&](int k) {
            const double x = E.edge(k) - S;
            return n > 0 && k == k_in && x > M.lo && x < M.hi ? g_in : M.g(x);
        };
        double prev = k_lo == 0 ? 0.0 : mass_below(k_lo - 1);
        int best = k_lo;
        double best_mass = -1.0;
        for (int k = k_lo; k <= k_hi; ++k) {
            const double cur = k >= E.top ? M.den : mass_below(k);
            if (cur - prev > best_mass) {
                best_mass = cur - prev;
                best = k;
            }
            prev = cur;
        }
        return best;
    }
    // first k whose cumulative row sum g(e_k - S) / den exceeds u
    const double target = ((double)word + 0.5) * (1.0 / 4294967296.0) * M.den;
    if (n > 0) {
        for (int k = k_in; k < k_hi; ++k) {
            const double x = E.edge(k) - S;
            if (k >= E.top || x >= M.hi || M.inside(x) > target) return k;   // (den exceeds every target)
        }
        return k_hi;
    }
    while (k_lo < k_hi) {
        const int k = (k_lo + k_hi) >> 1;
        if (k >= E.top || M.g(E.edge(k) - S) > target)
            k_hi = k;
        else
            k_lo = k + 1;
    }
    return k_lo;
}

constexpr int kRowsPerBlock = 4;     // one wave per (window, channel) row
constexpr int kMaxBlocks = 1024;     // 4 a CU; each makes the table of states once
constexpr int kMaxStates = 256;

// Bound by the erfc of a sample: 10 bursts of 100 samples in 4096 channels take 48 us (2048
// blocks the same), 93 with five erfc a sample, two of them for the tables of its state.
template <bool ARGMAX>
__global__ __launch_bounds__(64 * kRowsPerBlock) void k_inject(uint8_t *__restrict__ block, int64_t pitch,
                                                                int64_t n_t, int nch,
                                                                const int32_t *__restrict__ t_start,
                                                                const float *__restrict__ signal,
                                                                const uint32_t *__restrict__ words, int64_t n_rows,
                                                                int n_sig, Edges E) {
    __shared__ double s_f_lo[kMaxStates], s_den[kMaxStates];
    for (int n = threadIdx.x; n < E.top; n += 64 * kRowsPerBlock) {
        StateMass M;
        M.edges(E, n);
        M.masses();
        s_f_lo[n] = M.f_lo;
        s_den[n] = M.den;
    }
    __syncthreads();
    for (int64_t row = (int64_t)blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6); row < n_rows;
         row += (int64_t)gridDim.x * kRowsPerBlock) {
        const int c = (int)(row % nch);
        const int64_t t0 = t_start[row];
        uint8_t *line = block + (int64_t)c * pitch;
        const int64_t base = row * n_sig;
        for (int j = threadIdx.x & 63; j < n_sig; j += 64) {
            const double S = (double)signal[base + j];
            if (!(S > 0.0)) continue;
            const int64_t t = t0 + j;
            if (t < 0 || t >= n_t) continue;
            const int n = line[t];
            if (n >= E.top) continue;   // the top state keeps its samples; bytes above it are not states
            const uint32_t word = words ? words[base + j] : 0u;
            StateMass M;
            M.edges(E, n);
            M.f_lo = s_f_lo[n];
            M.den = s_den[n];
            line[t] = (uint8_t)new_state<ARGMAX>(E, M, n, S, word);
        }
    }
}

}  // namespace

hipError_t launch_inject(uint8_t *block, int64_t pitch, int64_t n_t, int nch, const int32_t *t_start,
                         const float *signal, const uint32_t *words, int n_win, int n_sig, int bits, double mu,
                         double sigma, double level, double offset, int mode, hipStream_t s) {
    if (n_win <= 0 || n_sig <= 0 || nch <= 0 || n_t <= 0) return hipSuccess;
    Edges E;
    E.mu = mu;
    E.sigma = sigma;
    E.width = level * sigma;
    E.offset = offset;
    E.half = 1 << (bits - 1);
    E.top = (1 << bits) - 1;
    const int64_t n_rows = (int64_t)n_win * nch;
    const int64_t gx = (n_rows + kRowsPerBlock - 1) / kRowsPerBlock;
    if (gx > 0x7fffffff || E.top > kMaxStates) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(gx < kMaxBlocks ? gx : kMaxBlocks)), threads(64 * kRowsPerBlock);
    if (mode == SPL_INJECT_ARGMAX_MODE)
        hipLaunchKernelGGL(k_inject<true>, grid, threads, 0, s, block, pitch, n_t, nch, t_start, signal, words, n_rows,
                           n_sig, E);
    else
        hipLaunchKernelGGL(k_inject<false>, grid, threads, 0, s, block, pitch, n_t, nch, t_start, signal, words, n_rows,
                           n_sig, E);
    return hipGetLastError();
}

}  // namespace spl
