// ebic_breed.hip -- the stand-in evolutionary driver's breeding on the
// device: the next generation from the current one (CSR in device memory)
// and its matched counts, by the rules of ebic_breed.h, so that a run can
// alternate evaluation and breeding on one stream while the population
// stays in device memory. The host driver (ebic_ea_step) applies the same
// rules to the same streams: both breed the same generation.
//
// Children of up to 64 columns are bred by one wave each (k_breed_waves:
// lane j holds column j, so a membership test is one compare and one
// ballot), into slots of k_max columns; the same launch ranks the
// individuals (a wave counts the ones that rank before its own) and copies
// the elites. A second kernel (k_breed_pack) turns the lengths into offsets
// and packs the slots into the CSR. Two things remain for the other calls:
//   - k_breed_small, one workgroup that needs no scratch, for populations of
//     up to 1,024 (whose arrays fit LDS) where the stream's scratch is not
//     to be used: under a capture, on the per-thread stream, or when its
//     allocation fails; and for those with k_max above 64;
//   - five kernels for larger populations with k_max above 64: fitness; the
//     elites' order; one thread per child breeding into its slot; one block
//     turning the lengths into offsets; one thread per child copying its
//     slot into the packed CSR.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>

#include "../../include/ebic.h"
#include "ebic_breed.h"
#include "ebic_runtime_internal.h"

namespace ebic {
namespace {

constexpr int kThreads = 256;
constexpr int kRankTile = 2048;  // fitnesses staged per LDS tile (16 KB)

__global__ void k_breed_fitness(int32_t n, const int32_t *__restrict__ offsets, const int32_t *__restrict__ matched,
                                double *__restrict__ f)
{
    const int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n) f[i] = breed::fitness(matched[i], offsets[i + 1] - offsets[i]);
}

// order[r] = the individual of rank r, for r < ne (rank: higher fitness
// first, then the lower index); best, if not null, gets rank 0's index.
// Each thread counts the individuals that rank before its own over the
// whole population, read tile by tile from LDS (every lane reads the same
// element: a broadcast), without a data-dependent exit.
__global__ void __launch_bounds__(kThreads) k_breed_order(int32_t n, const double *__restrict__ f, int32_t ne,
                                                          int32_t *__restrict__ order, int32_t *__restrict__ best)
{
    constexpr int kTile = 2048;
    __shared__ double ft[kTile];
    const int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    const double fi = i < n ? f[i] : 0.0;
    int32_t r = 0;
    for (int32_t j0 = 0; j0 < n; j0 += kTile) {
        const int32_t m = min(kTile, n - j0);
        __syncthreads();
        for (int32_t j = threadIdx.x; j < m; j += blockDim.x) ft[j] = f[j0 + j];
        __syncthreads();
        for (int32_t j = 0; j < m; ++j) r += breed::ranks_before(ft[j], j0 + j, fi, i) ? 1 : 0;
    }
    if (i >= n) return;
    if (r < ne) order[r] = i;
    if (r == 0 && best) *best = i;
}

// Child c (of more than 64 columns at most) into slots[c k_max ...], its
// length into lens[c].
__global__ void __launch_bounds__(kThreads) k_breed_children(ebic_ea_params p, int64_t generation, int32_t n,
                                 const int32_t *__restrict__ offsets, const int32_t *__restrict__ cols,
                                 const double *__restrict__ f, const int32_t *__restrict__ order,
                                 int32_t *__restrict__ slots, int32_t *__restrict__ lens)
{
    const int32_t c = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (c >= n) return;
    const breed::Strided child{slots + (int64_t)c * p.k_max, 1};
    int32_t len;
    if (c < p.elite) {  // the elites, best first, carried over unchanged
        const int32_t e = order[c];
        len = breed::parent_len(p, offsets, e);
        for (int32_t j = 0; j < len; ++j) child[j] = cols[offsets[e] + j];
    } else {
        breed::Rng rng = breed::stream(p.seed, generation, n, c);
        breed::Strided buf = child;
        len = breed::breed_child(p, rng, n, offsets, cols, f, buf);
    }
    lens[c] = len;
}

// offsets[0] = 0, offsets[i + 1] = lens[0] + ... + lens[i]: one block; each
// thread sums a contiguous segment, the segment sums are scanned in LDS.
__global__ void __launch_bounds__(1024) k_breed_offsets(int32_t n, const int32_t *__restrict__ lens,
                                                        int32_t *__restrict__ offsets)
{
    __shared__ int32_t part[1024];
    const int32_t t = (int32_t)threadIdx.x, T = (int32_t)blockDim.x;
    const int32_t per = (n + T - 1) / T;
    const int32_t lo = min(n, t * per), hi = min(n, lo + per);
    int32_t s = 0;
    for (int32_t i = lo; i < hi; ++i) s += lens[i];
    part[t] = s;
    __syncthreads();
    for (int32_t d = 1; d < T; d <<= 1) {
        const int32_t v = t >= d ? part[t - d] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    int32_t run = part[t] - s;  // the sum of the segments before this one
    if (t == 0) offsets[0] = 0;
    for (int32_t i = lo; i < hi; ++i) {
        run += lens[i];
        offsets[i + 1] = run;
    }
}

__global__ void k_breed_compact(int32_t n, int32_t k_max, const int32_t *__restrict__ slots,
                                const int32_t *__restrict__ offsets, int32_t *__restrict__ cols)
{
    const int32_t c = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (c >= n) return;
    const int32_t o = offsets[c], len = offsets[c + 1] - o;
    const int32_t *src = slots + (int64_t)c * k_max;
    for (int32_t j = 0; j < len; ++j) cols[o + j] = src[j];
}

// ---------------------------------------------------------------------------
// One wave per child (k_max <= 64): lane j holds column j of the child. The
// functions follow ebic_breed.h step by step and draw in the same order, so
// the children are the same; every lane draws the same numbers.
// ---------------------------------------------------------------------------
struct WaveChild {
    int32_t col;   // lane j: column j (any value for j >= len)
    int32_t len;   // wave-uniform
    int32_t lane;
    __device__ bool contains(int32_t c) const { return __ballot(lane < len && col == c) != 0; }
    __device__ void append(int32_t c)
    {
        if (lane == len) col = c;
        ++len;
    }
};

__device__ __forceinline__ int32_t wave_unused(const ebic_ea_params &p, breed::Rng &rng, const WaveChild &w)
{
    int32_t c;
    do c = (int32_t)rng.below((uint32_t)p.n_cols);
    while (w.contains(c));
    return c;
}

__device__ __forceinline__ void wave_random(const ebic_ea_params &p, breed::Rng &rng, WaveChild &w)
{
    const int32_t k = p.k_min + (int32_t)rng.below((uint32_t)(p.k_max - p.k_min + 1));
    w.len = 0;
    while (w.len < k) w.append(wave_unused(p, rng, w));
}

// lane j: columns j of parents a (ca, ka) and b (cb, kb)
__device__ __forceinline__ void wave_crossover(const ebic_ea_params &p, breed::Rng &rng, int32_t ca, int32_t ka,
                                               int32_t cb, int32_t kb, WaveChild &w)
{
    const int32_t cut = ka > 1 ? 1 + (int32_t)rng.below((uint32_t)ka - 1) : 1;
    const int32_t from = (int32_t)rng.below((uint32_t)kb);
    w.col = ca;
    w.len = min(cut, ka);
    for (int32_t j = from; j < kb && w.len < p.k_max; ++j) {
        const int32_t c = __builtin_amdgcn_readlane(cb, j);
        if (!w.contains(c)) w.append(c);
    }
    while (w.len < p.k_min) w.append(wave_unused(p, rng, w));
}

__device__ __forceinline__ void wave_mutate(const ebic_ea_params &p, breed::Rng &rng, WaveChild &w)
{
    const int32_t k = w.len;
    const uint32_t op = rng.below(4);
    if (op == 0 && k < p.k_max && k < p.n_cols) {  // insert
        const int32_t c = wave_unused(p, rng, w);
        const int32_t at = (int32_t)rng.below((uint32_t)k + 1);
        const int32_t before = __shfl(w.col, max(w.lane - 1, 0));
        w.col = w.lane > at ? before : w.lane == at ? c : w.col;
        w.len = k + 1;
    } else if (op == 1 && k > p.k_min) {  // delete
        const int32_t at = (int32_t)rng.below((uint32_t)k);
        const int32_t after = __shfl(w.col, min(w.lane + 1, kWave - 1));
        if (w.lane >= at) w.col = after;
        w.len = k - 1;
    } else if (op == 2 && k >= 2) {  // swap
        const int32_t a = (int32_t)rng.below((uint32_t)k), b = (int32_t)rng.below((uint32_t)k);
        const int32_t va = __shfl(w.col, a), vb = __shfl(w.col, b);
        w.col = w.lane == a ? vb : w.lane == b ? va : w.col;
    } else if (k < p.n_cols) {  // substitute
        const int32_t c = wave_unused(p, rng, w);
        if (w.lane == (int32_t)rng.below((uint32_t)k)) w.col = c;
    }
}

// Ranks and elites (the first `rank_blocks` blocks) and the bred children
// (the others), four waves per block. Nothing is passed between the two, so
// they run side by side.
//
// A rank block stages the population's fitnesses tile by tile in LDS; each
// of its waves counts, for I individuals, the ones that rank before (64 per
// step, counted by ballot). An individual of rank r < elite is child r.
// I = 1 up to 8,192 individuals: a block per four individuals, so that even
// 800 of them fill 200 CUs; eight past that, where the staging of every
// fitness by every block would cost more than the counting.
//
// A child's wave reads both tournaments' individuals in one round, its
// parents' columns in a second, and stores its slot. Bound by that chain of
// loads and by the draws (a 64-bit multiply chain). At 1,600 individuals of
// 2-30 columns ranks, elites and children took 4.6 + 97 + 63 us as three
// launches (a thread per individual) and now take 7.3 us; at 800 the
// one-workgroup kernel took 76-107 us against 5.3 us.
template <int I>
__global__ void __launch_bounds__(kThreads) k_breed_waves(ebic_ea_params p, int64_t generation, int32_t n,
                                                          const int32_t *__restrict__ offsets,
                                                          const int32_t *__restrict__ cols,
                                                          const int32_t *__restrict__ matched, int32_t rank_blocks,
                                                          int32_t *__restrict__ slots, int32_t *__restrict__ lens,
                                                          int32_t *__restrict__ best)
{
    __shared__ double ft[kRankTile];
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int32_t wave = __builtin_amdgcn_readfirstlane((int32_t)threadIdx.x / kWave);
    constexpr int32_t waves = kThreads / kWave;
    auto fit = [&](int32_t j) { return breed::fitness(matched[j], offsets[j + 1] - offsets[j]); };
    if ((int32_t)blockIdx.x < rank_blocks) {
        const int32_t i0 = ((int32_t)blockIdx.x * waves + wave) * I;
        double fi[I];
        int32_t r[I];
#pragma unroll
        for (int s = 0; s < I; ++s) {
            fi[s] = fit(min(i0 + s, n - 1));
            r[s] = 0;
        }
        for (int32_t j0 = 0; j0 < n; j0 += kRankTile) {
            const int32_t m = min(kRankTile, n - j0);
            if (j0) __syncthreads();
            // (padded to whole waves with entries that rank before nothing)
            for (int32_t j = (int32_t)threadIdx.x; j < (m + kWave - 1) / kWave * kWave; j += kThreads)
                ft[j] = j < m ? fit(j0 + j) : -HUGE_VAL;
            __syncthreads();
            for (int32_t j = lane; j - lane < m; j += kWave) {
                const double fj = ft[j];
                const int32_t at = j < m ? j0 + j : INT32_MAX;
#pragma unroll
                for (int s = 0; s < I; ++s)
                    r[s] += (int32_t)__popcll(__ballot(breed::ranks_before(fj, at, fi[s], i0 + s)));
            }
        }
#pragma unroll
        for (int s = 0; s < I; ++s) {
            const int32_t i = i0 + s;
            if (i >= n) continue;
            if (r[s] == 0 && best && lane == 0) *best = i;
            if (r[s] < p.elite) {  // the elites, best first, carried over unchanged
                const int32_t len = breed::parent_len(p, offsets, i);
                if (lane < len) slots[(int64_t)r[s] * p.k_max + lane] = cols[offsets[i] + lane];
                if (lane == 0) lens[r[s]] = len;
            }
        }
        return;
    }
    const int32_t c = p.elite + ((int32_t)blockIdx.x - rank_blocks) * waves + wave;
    if (c >= n) return;
    breed::Rng rng = breed::stream(p.seed, generation, n, c);
    // The draws up to the crossover's own do not depend on the individuals:
    // both tournaments' are made first, so that their loads go out together.
    const int32_t a0 = (int32_t)rng.below((uint32_t)n), a1 = (int32_t)rng.below((uint32_t)n);
    const bool cross = rng.uniform() < p.p_crossover;
    int32_t b0 = a0, b1 = a1;
    if (cross) {
        b0 = (int32_t)rng.below((uint32_t)n);
        b1 = (int32_t)rng.below((uint32_t)n);
    }
    // lane 0..3: the four drawn individuals' spans and fitnesses
    const int32_t who = lane == 0 ? a0 : lane == 1 ? a1 : lane == 2 ? b0 : b1;
    const int32_t start = offsets[who], k = offsets[who + 1] - start;
    const double f = breed::fitness(matched[who], k);
    auto wins = [&](int x, int32_t ix, int32_t iy) {  // the first of lanes x, x + 1 (individuals ix, iy)?
        const double fx = __shfl(f, x), fy = __shfl(f, x + 1);
        return fx > fy || (fx == fy && ix <= iy);
    };
    const int la = __builtin_amdgcn_readfirstlane(wins(0, a0, a1) ? 0 : 1);
    const int lb = __builtin_amdgcn_readfirstlane(wins(2, b0, b1) ? 2 : 3);
    const int32_t ka = min(__builtin_amdgcn_readlane(k, la), p.k_max);
    const int32_t sa = __builtin_amdgcn_readlane(start, la);
    const int32_t kb = min(__builtin_amdgcn_readlane(k, lb), p.k_max);
    const int32_t sb = __builtin_amdgcn_readlane(start, lb);
    const int32_t ca = lane < ka ? cols[sa + lane] : 0;
    const int32_t cb = cross && lane < kb ? cols[sb + lane] : 0;
    WaveChild w{ca, ka, lane};
    if (ka <= 0 || (cross && kb <= 0)) wave_random(p, rng, w);
    else if (cross) wave_crossover(p, rng, ca, ka, cb, kb, w);
    if (rng.uniform() < p.p_mutation) wave_mutate(p, rng, w);
    if (lane < w.len) slots[(int64_t)c * p.k_max + lane] = w.col;
    if (lane == 0) lens[c] = w.len;
}

// Lengths to offsets and slots to the packed CSR: block b takes `per` (at
// most 64) children; its threads sum the lengths before them, each wave
// scans the block's own, and the waves copy the children in turn. Every
// block sums the lengths from the start (6 KB at 1,600 individuals): one
// launch of 3.2 us instead of a scan and a copy (4.8 + 6.1 us) at 1,600.
__global__ void __launch_bounds__(kThreads) k_breed_pack(int32_t n, int32_t k_max, int32_t per,
                                                         const int32_t *__restrict__ slots,
                                                         const int32_t *__restrict__ lens,
                                                         int32_t *__restrict__ offsets, int32_t *__restrict__ cols)
{
    constexpr int32_t waves = kThreads / kWave;
    __shared__ int32_t part[waves];
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int32_t wave = __builtin_amdgcn_readfirstlane((int32_t)threadIdx.x / kWave);
    const int32_t c0 = (int32_t)blockIdx.x * per, m = min(per, n - c0);
    const int32_t own = lane < m ? lens[c0 + lane] : 0;
    // (a slot is read whole, before its length is known: the loads go out
    // with those of the lengths)
    constexpr int kAhead = 4;
    int32_t ahead[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
        const int32_t t = wave + u * waves;
        ahead[u] = t < m && lane < k_max ? slots[(int64_t)(c0 + t) * k_max + lane] : 0;
    }
    int32_t before = 0;
#pragma unroll 4
    for (int32_t j = (int32_t)threadIdx.x; j < c0; j += kThreads) before += lens[j];
    for (int d = kWave / 2; d; d >>= 1) before += __shfl_xor(before, d);
    if (lane == 0) part[wave] = before;
    int32_t end = own;
    for (int d = 1; d < kWave; d <<= 1) {
        const int32_t v = __shfl_up(end, d);
        if (lane >= d) end += v;
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < waves; ++v) end += part[v];
    if (wave == 0 && lane < m) offsets[c0 + lane + 1] = end;
    if (blockIdx.x == 0 && threadIdx.x == 0) offsets[0] = 0;
    auto put = [&](int32_t t, int32_t col) {
        const int32_t len = __builtin_amdgcn_readlane(own, t), at = __builtin_amdgcn_readlane(end, t) - len;
        if (lane < len) cols[at + lane] = col;
    };
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
        if (wave + u * waves < m) put(wave + u * waves, ahead[u]);
#pragma unroll 4
    for (int32_t t = wave + kAhead * waves; t < m; t += waves)
        put(t, lane < k_max ? slots[(int64_t)(c0 + t) * k_max + lane] : 0);
}

// The whole breeding of a population of at most 1,024 in one workgroup of
// one thread per individual, everything in LDS: fitness; the rank order by
// a bitonic sort of (fitness, index) pairs (padded to a power of two with
// entries that rank last); one child per thread, built in an interleaved
// LDS array; the lengths' scan; the packed copy out. Five launches and
// their gaps become one.
__global__ void __launch_bounds__(1024) k_breed_small(ebic_ea_params p, int64_t generation, int32_t n,
                                                      const int32_t *__restrict__ offsets,
                                                      const int32_t *__restrict__ cols,
                                                      const int32_t *__restrict__ matched, int32_t n2,
                                                      int32_t *__restrict__ next_offsets,
                                                      int32_t *__restrict__ next_cols, int32_t *__restrict__ best)
{
    extern __shared__ __align__(16) unsigned char sm[];
    __shared__ int32_t part[1024];
    double *f = reinterpret_cast<double *>(sm);  // n, by individual
    double *key = f + n2;                        // n2, sorted into rank order
    int32_t *id = reinterpret_cast<int32_t *>(key + n2);
    int32_t *children = id + n2;
    const int32_t t = (int32_t)threadIdx.x, T = (int32_t)blockDim.x;
    const bool live = t < n;
    if (live) f[t] = breed::fitness(matched[t], offsets[t + 1] - offsets[t]);
    __syncthreads();
    for (int32_t i = t; i < n2; i += T) {
        key[i] = i < n ? f[i] : -HUGE_VAL;
        id[i] = i < n ? i : INT32_MAX;  // (padding ranks after every individual)
    }
    __syncthreads();
    for (int32_t k = 2; k <= n2; k <<= 1) {
        for (int32_t j = k >> 1; j > 0; j >>= 1) {
            for (int32_t i = t; i < n2; i += T) {
                const int32_t o = i ^ j;
                if (o > i) {
                    // blocks with (i & k) == 0 end in rank order, the others reversed
                    const bool first = (i & k) == 0;
                    const bool o_first = breed::ranks_before(key[o], id[o], key[i], id[i]);
                    if (o_first == first) {
                        const double kt = key[i];
                        key[i] = key[o];
                        key[o] = kt;
                        const int32_t it = id[i];
                        id[i] = id[o];
                        id[o] = it;
                    }
                }
            }
            __syncthreads();
        }
    }
    if (t == 0 && best) *best = id[0];
    int32_t len = 0;
    const breed::Strided child{children + t, T};
    if (live) {
        if (t < p.elite) {  // the elites, best first, carried over unchanged
            const int32_t e = id[t];
            len = breed::parent_len(p, offsets, e);
            for (int32_t j = 0; j < len; ++j) child[j] = cols[offsets[e] + j];
        } else {
            breed::Rng rng = breed::stream(p.seed, generation, n, t);
            breed::Strided buf = child;
            len = breed::breed_child(p, rng, n, offsets, cols, f, buf);
        }
    }
    part[t] = len;
    __syncthreads();
    for (int32_t d = 1; d < T; d <<= 1) {
        const int32_t v = t >= d ? part[t - d] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    const int32_t end = part[t], start = end - len;
    if (t == 0) next_offsets[0] = 0;
    if (live) {
        next_offsets[t + 1] = end;
        for (int32_t j = 0; j < len; ++j) next_cols[start + j] = child[j];
    }
}

}  // namespace
}  // namespace ebic

using namespace ebic;

extern "C" ebic_status ebic_ea_breed(ebic_ctx *ctx, const ebic_ea_params *params, int64_t generation,
                                     int32_t n_ind, const int32_t *d_offsets, const int32_t *d_cols,
                                     const int32_t *d_matched, int32_t *d_next_offsets, int32_t *d_next_cols,
                                     int32_t *d_best, void *hip_stream)
{
    return guarded([&] {
        if (!ctx || !params) fail(EBIC_EINVAL, "ctx and params are required");
        const ebic_ea_params p = *params;
        if (const char *why = breed::params_error(p)) fail(EBIC_EINVAL, why);
        if (n_ind != p.pop_size) fail(EBIC_EINVAL, "n_ind must equal params->pop_size");
        if (generation < 1) fail(EBIC_EINVAL, "generation must be >= 1 (0 is the random first generation)");
        if (!d_offsets || !d_cols || !d_matched || !d_next_offsets || !d_next_cols)
            fail(EBIC_EINVAL, "d_offsets, d_cols, d_matched, d_next_offsets and d_next_cols are required");
        const hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
        const int32_t n = n_ind;
        const int32_t ne = std::max(p.elite, 1);
        DeviceGuard g(ctx->device);
        const size_t l_bytes = ((size_t)n * sizeof(int32_t) + 255) / 256 * 256;
        const size_t s_bytes = (size_t)n * p.k_max * sizeof(int32_t);
        // Up to 1,024 individuals whose fitness, elite order and children
        // fit LDS can be bred by one workgroup without scratch.
        const int32_t T = (n + kWave - 1) / kWave * kWave;
        int32_t n2 = 1;
        while (n2 < n) n2 <<= 1;
        const size_t small_lds = (size_t)n2 * (2 * sizeof(double) + sizeof(int32_t)) +
                                 (size_t)T * p.k_max * sizeof(int32_t);
        const bool small = n <= 1024 && small_lds + 1024 * sizeof(int32_t) <= ctx->lds_per_block;
        // Scratch and launches go out together: the stream's scratch is
        // shared with the evaluations on it.
        const std::unique_lock<std::mutex> lk = launch_lock(ctx, s);
        if (p.k_max <= kWave) {
            unsigned char *base = nullptr;
            if (small) {
                // A population of this size needs no memory of the library's:
                // a captured call takes none, so that its graph holds nothing
                // that a later call on the stream may replace or write beside
                // a replay, nor does one on the per-thread stream (one handle,
                // many streams), and without memory one workgroup breeds as
                // well.
                hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
                const bool own = s != hipStreamPerThread && hipStreamIsCapturing(s, &st) == hipSuccess &&
                                 st == hipStreamCaptureStatusNone;
                clear_last_error();
                try {
                    if (own) base = static_cast<unsigned char *>(stream_scratch(ctx, s, l_bytes + s_bytes, true));
                } catch (const Error &) {
                    // (whatever kept the memory from being had)
                }
            } else {
                base = static_cast<unsigned char *>(stream_scratch(ctx, s, l_bytes + s_bytes));
            }
            if (base) {
                int32_t *lens = reinterpret_cast<int32_t *>(base);
                int32_t *slots = reinterpret_cast<int32_t *>(base + l_bytes);
                fault_point_launch(ctx, "breeding launch");
                constexpr int32_t waves = kThreads / kWave;
                const bool one = n <= 8192;
                const int32_t rank_blocks = one ? (n + waves - 1) / waves : (n + waves * 8 - 1) / (waves * 8);
                const int32_t blocks = rank_blocks + (n - p.elite + waves - 1) / waves;
                clear_last_error();
                if (one)
                    hipLaunchKernelGGL(k_breed_waves<1>, dim3(blocks), dim3(kThreads), 0, s, p, generation, n, d_offsets,
                                       d_cols, d_matched, rank_blocks, slots, lens, d_best);
                else
                    hipLaunchKernelGGL(k_breed_waves<8>, dim3(blocks), dim3(kThreads), 0, s, p, generation, n, d_offsets,
                                       d_cols, d_matched, rank_blocks, slots, lens, d_best);
                // 16 children per block up to 4,096 (a hundred blocks at
                // 1,600); 64 past that, where summing the lengths from the
                // start is most of a block's work.
                const int32_t per = n <= 4096 ? 16 : kWave;
                hip_check(hipGetLastError(), "breeding kernel");
                hipLaunchKernelGGL(k_breed_pack, dim3((n + per - 1) / per), dim3(kThreads), 0, s, n, p.k_max, per, slots,
                                   lens, d_next_offsets, d_next_cols);
                hip_check(hipGetLastError(), "breeding kernels");
                return;
            }
        }
        if (small) {
            fault_point_launch(ctx, "breeding launch");
            hip_check(hipFuncSetAttribute(reinterpret_cast<const void *>(&k_breed_small),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)small_lds),
                      "hipFuncSetAttribute");
            clear_last_error();
            hipLaunchKernelGGL(k_breed_small, dim3(1), dim3(T), small_lds, s, p, generation, n, d_offsets, d_cols,
                               d_matched, n2, d_next_offsets, d_next_cols, d_best);
            hip_check(hipGetLastError(), "breeding kernel");
            return;
        }
        // Scratch on the stream: fitness | elite order | lengths | child slots.
        const size_t f_bytes = (size_t)n * sizeof(double);
        const size_t o_bytes = ((size_t)ne * sizeof(int32_t) + 255) / 256 * 256;
        auto *base = static_cast<unsigned char *>(stream_scratch(ctx, s, f_bytes + o_bytes + l_bytes + s_bytes));
        double *f = reinterpret_cast<double *>(base);
        int32_t *order = reinterpret_cast<int32_t *>(base + f_bytes);
        int32_t *lens = reinterpret_cast<int32_t *>(base + f_bytes + o_bytes);
        int32_t *slots = reinterpret_cast<int32_t *>(base + f_bytes + o_bytes + l_bytes);
        fault_point_launch(ctx, "breeding launch");
        const unsigned blocks = (unsigned)((n + kThreads - 1) / kThreads);
        clear_last_error();
        hipLaunchKernelGGL(k_breed_fitness, dim3(blocks), dim3(kThreads), 0, s, n, d_offsets, d_matched, f);
        clear_last_error();
        hipLaunchKernelGGL(k_breed_order, dim3(blocks), dim3(kThreads), 0, s, n, f, ne, order, d_best);
        clear_last_error();
        hipLaunchKernelGGL(k_breed_children, dim3(blocks), dim3(kThreads), 0, s, p, generation, n, d_offsets, d_cols,
                           f, order, slots, lens);
        clear_last_error();
        hipLaunchKernelGGL(k_breed_offsets, dim3(1), dim3(1024), 0, s, n, lens, d_next_offsets);
        clear_last_error();
        hipLaunchKernelGGL(k_breed_compact, dim3(blocks), dim3(kThreads), 0, s, n, p.k_max, slots,
                           d_next_offsets, d_next_cols);
        hip_check(hipGetLastError(), "breeding kernels");
    });
}
