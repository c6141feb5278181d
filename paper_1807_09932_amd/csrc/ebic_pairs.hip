// ebic_pairs.hip -- the predicate over pairwise order bitmaps.
//
// The trend relation of an individual (c_0, ..., c_{k-1}) on a row holds
// when every consecutive pair does: x[r, c_j] >= x[r, c_{j-1}] for the
// positive chain, x[r, c_{j-1}] >= x[r, c_j] for the reversed one (Methods,
// "Handling missing values": the rows are counted by this relation). Both
// chains are conjunctions over the individual's consecutive column pairs,
// and there are only cols^2 ordered pairs. So the library can compare every
// ordered pair of columns once per row, on first use, and keep the answers
// as bitmaps:
//
//   G[a * cols + b] bit r  =  x[r, b] >= x[r, a]      (IEEE single: a NaN
//                                                       on either side is 0)
//
// The diagonal pair (a, a) is then "x[r, a] is present". An individual's
// positive chain on 32 rows is one AND per pair of one 32-bit word per
// lane, its reversed chain the same over the reversed pairs, and a row
// matched by both directions (constant along the individual) counts once,
// as positive. The results are those of the comparisons themselves, bit for
// bit: the bitmaps hold the compares' outcomes, ties and signed zeros
// included.
//
// Layout: panel by panel (1,024 rows, two to a chunk of 2,048), and within
// a panel pair by pair, pair (a, b) of panel h at word
// ((h * cols + a) * cols + b) * 32; bit i of word w is row 1024 h + 32 w + i.
// A pair's words on a panel are one 128-byte cache line. Rows past the
// matrix are 0. A panel's pairs span cols^2 x 128 bytes, so a wave addresses
// them with 32-bit offsets from the panel's base. Include mode reads a
// second set built from the fill-substituted values (the same set when no
// cell is missing).
//
// Behind the bitmaps, 512 bytes per chunk list its ties: word 0 counts the
// entries, word 1 is non-zero if a NaN occurs in the chunk, and words
// 64 .. 95 hold the byte offsets of the pairs (a, b), a < b, with two equal
// values on some row (a count past 32 means more). Where a chunk has no NaN
// and a pair is not listed, every row has x_a, x_b present and distinct, so
// the reversed pair's word is the complement of the pair's on the matrix's
// rows: one orientation (the ascending one) serves both chains of both
// orientations, and a panel's working set is half its pairs.
//
// Evaluation: a wave takes eight individuals at a time (a step), eight lanes
// each, on one panel: a lane holds 128 rows, one 16-byte load per pair, so a
// load instruction reads eight cache lines whole. A prep kernel writes each
// individual's header (ebic_prep.h); a step's eight headers (256 bytes) go
// through LDS, where every lane reads its group's. The wave loads the seven
// window pairs, ANDs them for one chain and takes the complement of their OR
// for the other; where the chunk is dirty (NaN, or more ties than the list
// holds) or a window pair is tied, both orientations are loaded. Individuals
// with rows left and columns past the window wait in LDS, with their rows,
// until eight of them (or the last of the item) are finished together, four
// pairs at a time: a step goes on without them, and where one individual in
// four has such rows (any population that follows a trend) the dependent
// loads of their columns and words are paid once for eight. Counts are
// summed over a group's lanes by DPP moves into a lane per individual, and
// added to the outputs once per item.
//
// What bounds it, and why this shape. The kernel began with one individual
// per wave on a chunk: a 4-byte load per lane, both orientations stored and
// read. Three things held it (rocprofv3 counters, 436,444 x 64 and the batch
// of 64 populations on 100,000 x 256, matrices and populations in turn):
//   - the texture units return four lanes a clock whatever a lane asks for:
//     256 bytes took as long as the kilobyte of a 16-byte load;
//   - the scalar unit's 54 instructions per individual and chunk are now
//     shared by eight individuals;
//   - L2 misses. A panel of 256 columns in one orientation is 4.2 MB, about
//     an XCD's L2; a chunk in both was 16.8 MB, read 3.6 times over.
// 436,444 x 64, 800 individuals 38.6 -> 31.6 us an evaluation, x 310 51 ->
// 50 us (there 263 MB of distinct lines come from HBM at about 5.5 TB/s),
// the batch 822 -> 379 us. Four individuals of 16 lanes (8-byte loads): 38,
// 57 and 585 us.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "ebic_internal.h"
#include "ebic_prep.h"

namespace ebic {
namespace {

constexpr int kChunkRows = 2048;  // rows of one tie list, and of a build wave: 64 lanes x 32 rows
constexpr int kChunkWords = 64;
constexpr int kTieWords = 128;    // per chunk: count, NaN flag, ..., up to 32 listed offsets
constexpr int kTieList = 64;      // (the list's first word)
constexpr int kTieMax = 32;       // pairs it holds
// No listed pair's offset (of 1,024 columns the last diagonal pair has it,
// and lists hold pairs a < b only).
constexpr uint32_t kNoPair = kHeadOffset;
constexpr int kPanelRows = 1024;  // rows of one step: 8 lanes x 128 rows
constexpr int kPanelWords = 32;
constexpr int kGroup = 8;         // lanes per individual (16 bytes of a pair's line each)
constexpr int kStep = kWave / kGroup;  // individuals per wave and step
constexpr int kQueue = 2 * kStep - 1;  // individuals that wait for their columns past the window
// LDS of a wave: a step's headers, and the queue's rows and (k, start, index).
constexpr size_t kWaveLdsFew = kStep * (2 * 128 + 16);
constexpr size_t kWaveLds = kStep * 32 + kQueue * (2 * 128 + 16);

__global__ void __launch_bounds__(256) k_prep_pairs(ReqDesc d, IndHead *__restrict__ heads)
{
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int32_t i = (int32_t)(blockIdx.x * (blockDim.x / 16) + threadIdx.x / 16);
    const PairPrep p = prep_pairs_quad(d, i, i < d.n, lane);
    if (i < d.n) prep_pairs_store(d, i, p, heads, lane);
}

// ---------------------------------------------------------------------------
// The build. A block takes 16 columns a (two to each of its eight waves, in
// registers: lane l holds rows 32 l .. 32 l + 31 of the chunk) against a run
// of `run` columns b >= a, staged four at a time through LDS: read from the
// matrix in whole lines, each once per block, and from LDS as every lane's
// 128 bytes (rows padded to 144 bytes: no bank conflicts). The grid is
// (8 x tiles, chunks / 8): block (x, y) takes chunk 8 y + x mod 8 and tile
// x / 8, so a chunk's blocks run on one XCD and its columns stay in its L2.
//
// A pair's word is built bit by bit. Without missing cells (FULL false) only
// the ascending orientation's words are written, from the signs of the
// differences: a subtraction, a shift that takes the sign in, and half a
// three-way minimum that finds the pairs with a tie, whose reverse is then
// computed and written too and which go to the chunk's list: two and a half
// vector instructions per row and pair. Once an infinity has been staged,
// compares take their place: a compare into a scalar pair, an add with carry
// that shifts the word left and takes the bit, and a second compare (equal,
// kept as one mask per word). With missing cells (FULL), or on the chunks
// whose list has overflowed (a second launch; `dirty` = the list's limit,
// chunks below it exit at once), both orientations are built by compares
// with four. The first version compared both ways with about eight (a
// compare, its wait states, a select, half an or), read each column with
// lanes 128 bytes apart (64 lines per load) and wrote both orientations of
// every pair.
//
// Bound by the vector unit (some 100 instructions per pair and 2,048 rows)
// and, with four waves per SIMD, by the waits for LDS and the barriers. The
// first version, compares and differences: 54,675 x 178 507, 195 and 178 us,
// 436,444 x 64 330, 257 and 232 us, 436,444 x 310 5.0, 3.05 and 2.77 ms,
// 100,000 x 256 1.16, 0.82 and 0.71 ms; 20,000 x 200 with 5% missing cells
// 476 and 147 us, and 818 and 156 us of the substituted values, whose every
// pair ties: a block stops listing once the list has overflowed.
// ---------------------------------------------------------------------------
constexpr int kBuildWaves = 8;
constexpr int kBuildA = 2;                          // columns a per wave
constexpr int kBuildCols = kBuildWaves * kBuildA;   // columns a per block
constexpr int kBuildB = 4;                          // columns b staged together
constexpr int kLaneFloats = 36;                     // a lane's 32 rows in LDS, padded
constexpr int kBuildTile = kBuildWaves * kWave * kLaneFloats;  // (the waves' columns a; then four columns b twice)

// Bits of x[i] >= y[i] for four rows, the highest first, into `word`, and
// the lanes with x[i] == y[i] into `tie` (no NaN).
__device__ __forceinline__ void ge4_ties(uint32_t &word, uint64_t &tie, const float *x, const float *y)
{
    uint64_t g0, g1, g2, g3, t0, t1, t2, t3;
    asm volatile("v_cmp_ge_f32_e64 %[g3], %[x3], %[y3]\n\t"
                 "v_cmp_ge_f32_e64 %[g2], %[x2], %[y2]\n\t"
                 "v_cmp_ge_f32_e64 %[g1], %[x1], %[y1]\n\t"
                 "v_cmp_ge_f32_e64 %[g0], %[x0], %[y0]\n\t"
                 "v_cmp_eq_f32_e64 %[t3], %[x3], %[y3]\n\t"
                 "v_addc_co_u32_e64 %[w], %[g3], %[w], %[w], %[g3]\n\t"
                 "v_cmp_eq_f32_e64 %[t2], %[x2], %[y2]\n\t"
                 "v_addc_co_u32_e64 %[w], %[g2], %[w], %[w], %[g2]\n\t"
                 "v_cmp_eq_f32_e64 %[t1], %[x1], %[y1]\n\t"
                 "v_addc_co_u32_e64 %[w], %[g1], %[w], %[w], %[g1]\n\t"
                 "v_cmp_eq_f32_e64 %[t0], %[x0], %[y0]\n\t"
                 "v_addc_co_u32_e64 %[w], %[g0], %[w], %[w], %[g0]\n\t"
                 "s_or_b64 %[t3], %[t3], %[t2]\n\t"
                 "s_or_b64 %[t1], %[t1], %[t0]\n\t"
                 "s_or_b64 %[tie], %[tie], %[t3]\n\t"
                 "s_or_b64 %[tie], %[tie], %[t1]"
                 : [w] "+v"(word), [tie] "+s"(tie), [g0] "=&s"(g0), [g1] "=&s"(g1), [g2] "=&s"(g2), [g3] "=&s"(g3),
                   [t0] "=&s"(t0), [t1] "=&s"(t1), [t2] "=&s"(t2), [t3] "=&s"(t3)
                 : [x0] "v"(x[0]), [x1] "v"(x[1]), [x2] "v"(x[2]), [x3] "v"(x[3]), [y0] "v"(y[0]), [y1] "v"(y[1]),
                   [y2] "v"(y[2]), [y3] "v"(y[3])
                 : "scc");
}

// The same from the differences, for 32 rows without infinities and negative
// zeros: a difference's sign bit is the comparison (it is exact in its sign,
// subnormal ones included), and it is +0, the smallest bit pattern, exactly
// where the two are equal.
__device__ __forceinline__ uint32_t ge32_ties(uint64_t &tie, const float *x, const float *y)
{
    uint32_t less = 0, least = ~0u;
#pragma unroll
    for (int r = 30; r >= 0; r -= 2) {
        const uint32_t d1 = __float_as_uint(x[r + 1] - y[r + 1]), d0 = __float_as_uint(x[r] - y[r]);
        less = __builtin_amdgcn_alignbit(less, d1, 31);
        less = __builtin_amdgcn_alignbit(less, d0, 31);
        asm volatile("v_min3_u32 %0, %0, %1, %2" : "+v"(least) : "v"(d1), "v"(d0));
    }
    tie = __ballot(least == 0);
    return ~less;
}

// The comparisons' bits alone.
__device__ __forceinline__ void ge4(uint32_t &word, const float *x, const float *y)
{
    uint64_t g0, g1, g2, g3;
    asm volatile("v_cmp_ge_f32_e64 %[g3], %[x3], %[y3]\n\t"
                 "v_cmp_ge_f32_e64 %[g2], %[x2], %[y2]\n\t"
                 "v_cmp_ge_f32_e64 %[g1], %[x1], %[y1]\n\t"
                 "v_cmp_ge_f32_e64 %[g0], %[x0], %[y0]\n\t"
                 "v_addc_co_u32_e64 %[w], %[g3], %[w], %[w], %[g3]\n\t"
                 "v_addc_co_u32_e64 %[w], %[g2], %[w], %[w], %[g2]\n\t"
                 "v_addc_co_u32_e64 %[w], %[g1], %[w], %[w], %[g1]\n\t"
                 "v_addc_co_u32_e64 %[w], %[g0], %[w], %[w], %[g0]"
                 : [w] "+v"(word), [g0] "=&s"(g0), [g1] "=&s"(g1), [g2] "=&s"(g2), [g3] "=&s"(g3)
                 : [x0] "v"(x[0]), [x1] "v"(x[1]), [x2] "v"(x[2]), [x3] "v"(x[3]), [y0] "v"(y[0]), [y1] "v"(y[1]),
                   [y2] "v"(y[2]), [y3] "v"(y[3]));
}

template <bool FULL>
__global__ void __launch_bounds__(kBuildWaves *kWave) __attribute__((amdgpu_waves_per_eu(4)))
k_pair_bits(const float *__restrict__ X, int64_t rows, int64_t ld, int32_t cols, int32_t subst, float fill, int32_t run,
            int32_t dirty, uint32_t *__restrict__ G, uint32_t *__restrict__ T)
{
    __shared__ __align__(16) float tile[kBuildTile];
    __shared__ int32_t infinite;  // an infinity has been staged
    const int64_t chunk = 8 * (int64_t)blockIdx.y + (blockIdx.x & 7);
    const int32_t runs = (cols + run - 1) / run;
    const int32_t a0 = (int32_t)(blockIdx.x >> 3) / runs * kBuildCols, b0 = (int32_t)(blockIdx.x >> 3) % runs * run;
    const int32_t b1 = min(b0 + run, cols);
    if (chunk * kChunkRows >= rows || b1 <= a0) return;
    uint32_t *tl = T + chunk * kTieWords;
    if (dirty && (int32_t)__builtin_amdgcn_readfirstlane(tl[0]) <= dirty) return;
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int64_t c0 = chunk * kChunkRows, r0 = c0 + 32 * lane;
    const int64_t panel = 2 * chunk + (lane >> 5);
    const int64_t nvalid = rows - r0;
    const uint32_t vmask = nvalid >= 32 ? ~0u : nvalid <= 0 ? 0u : ((1u << nvalid) - 1u);

    // Rows r .. r + 3 of column c; rows past the matrix take `pad` (unequal
    // for a and b, so that they never tie).
    auto fetch = [&](int32_t c, int64_t r) {
        return r < ld && c < cols ? *reinterpret_cast<const float4 *>(X + (int64_t)c * ld + r) : make_float4(0.f, 0.f, 0.f, 0.f);
    };
    auto fixed = [&](float4 f, int64_t r, float pad) {
        if (subst) {
            f.x = f.x != f.x ? fill : f.x;
            f.y = f.y != f.y ? fill : f.y;
            f.z = f.z != f.z ? fill : f.z;
            f.w = f.w != f.w ? fill : f.w;
        }
        if (!FULL) {
            // (no negative zeros)
            f.x += 0.f;
            f.y += 0.f;
            f.z += 0.f;
            f.w += 0.f;
            const float inf = __builtin_inff();
            const bool some = (fabsf(f.x) == inf || fabsf(f.y) == inf) || (fabsf(f.z) == inf || fabsf(f.w) == inf);
            if (some) infinite = 1;
        }
        if (r + 3 >= rows) {
            if (r >= rows) f.x = pad;
            if (r + 1 >= rows) f.y = pad;
            if (r + 2 >= rows) f.z = pad;
            f.w = pad;
        }
        return f;
    };
    // (four rows f of a column go to lane f / 8's part)
    auto place = [](int f) { return (f >> 3) * kLaneFloats + (f & 7) * 4; };
    auto take = [&](const float *column, float (&v)[32]) {
        const float4 *p = reinterpret_cast<const float4 *>(column + lane * kLaneFloats);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float4 f = p[i];
            v[4 * i] = f.x;
            v[4 * i + 1] = f.y;
            v[4 * i + 2] = f.z;
            v[4 * i + 3] = f.w;
        }
    };
    static_assert(kChunkRows == 4 * kBuildWaves * kWave, "a thread stages four rows of each column b");
    if (!FULL) {
        if (threadIdx.x == 0) infinite = 0;
        __syncthreads();
    }
    // The wave's columns a, through a part of the LDS of its own.
    float xa[kBuildA][32];
    {
        float *own = tile + wave * kWave * kLaneFloats;
#pragma unroll
        for (int i = 0; i < kBuildA; ++i) {
#pragma unroll
            for (int q = 0; q < kBuildWaves; ++q) {
                const int f = q * kWave + lane;
                *reinterpret_cast<float4 *>(own + place(f)) =
                    fixed(fetch(a0 + kBuildA * wave + i, c0 + 4 * f), c0 + 4 * f, 1.f);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            take(own, xa[i]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    }
    bool listing = dirty == 0;
    const int64_t rb = c0 + 4 * (int64_t)threadIdx.x;
    float4 pre[kBuildB];
    const int32_t aw = a0 + kBuildA * wave;
    const int32_t bs = max(b0, a0) / kBuildB * kBuildB;  // (a0 and b0 are multiples of the step)
#pragma unroll
    for (int q = 0; q < kBuildB; ++q) pre[q] = fetch(bs + q, rb);
    __syncthreads();
    // (two buffers in turn: one barrier per step)
    float *buf = tile;
    for (int32_t bt = bs; bt < b1; bt += kBuildB) {
#pragma unroll
        for (int q = 0; q < kBuildB; ++q)
            *reinterpret_cast<float4 *>(buf + q * kWave * kLaneFloats + place((int)threadIdx.x)) = fixed(pre[q], rb, 0.f);
        __syncthreads();
        if (bt + kBuildB < b1)
#pragma unroll
            for (int q = 0; q < kBuildB; ++q) pre[q] = fetch(bt + kBuildB + q, rb);
#pragma unroll 1
        for (int q = 0; q < kBuildB; ++q) {  // (the same columns for every wave)
            const int32_t b = bt + q;
            if (b >= b1 || b < aw) continue;
            float xb[32];
            take(buf + q * kWave * kLaneFloats, xb);
            const bool differ = !FULL && __builtin_amdgcn_readfirstlane(infinite) == 0;
#pragma unroll
            for (int i = 0; i < kBuildA; ++i) {
                const int32_t a = aw + i;
                if (a > b || a >= cols) continue;
                __builtin_amdgcn_sched_barrier(0);  // (pair by pair: registers)
                uint32_t ge = 0;
                uint64_t tie = 0;
                const int64_t up = ((panel * cols + a) * cols + b) * kPanelWords + (lane & 31);
                const int64_t down = ((panel * cols + b) * cols + a) * kPanelWords + (lane & 31);
                if (!FULL) {
                    if (differ) {
                        ge = ge32_ties(tie, xb, xa[i]);
                    } else {
#pragma unroll
                        for (int r = 28; r >= 0; r -= 4) ge4_ties(ge, tie, xb + r, xa[i] + r);
                    }
                    G[up] = ge & vmask;
                    if (a == b || tie == 0) continue;
                } else {
#pragma unroll
                    for (int r = 28; r >= 0; r -= 4) ge4(ge, xb + r, xa[i] + r);
                    G[up] = ge & vmask;
                }
                __builtin_amdgcn_sched_barrier(0);
                uint32_t le = 0;
#pragma unroll
                for (int r = 28; r >= 0; r -= 4) ge4(le, xa[i] + r, xb + r);
                if (a != b) G[down] = le & vmask;
                const uint32_t odd = (a == b ? ~ge : (ge & le)) & vmask;  // rows with NaN; tied rows
                if (listing && __ballot(odd != 0) != 0) {
                    if (a == b) {
                        if (lane == 0) atomicOr(tl + 1, 1u);
                        listing = false;
                    } else {
                        uint32_t slot = 0;
                        if (lane == 0) {
                            slot = atomicAdd(tl, 1u);
                            if (slot < (uint32_t)kTieMax) tl[kTieList + slot] = pair_offset((uint32_t)cols, (uint32_t)a, (uint32_t)b);
                        }
                        // (a list that has overflowed takes no more)
                        listing = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot) < (uint32_t)kTieMax;
                    }
                }
            }
        }
        buf = buf == tile ? tile + kBuildB * kWave * kLaneFloats : tile;
    }
}

// Moves within the groups of eight lanes (half a DPP row), one individual
// each: lane u of the group to all of it; the sum over the group in every
// lane; the group's bits of a wave mask.
template <int U>
__device__ __forceinline__ uint32_t group_bcast(uint32_t v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, (int)v, 0x150 + U, 0xf, 0x3, false);      // row_newbcast:U, lanes 0..7
    return (uint32_t)__builtin_amdgcn_update_dpp(lo, (int)v, 0x158 + U, 0xf, 0xc, false);   // row_newbcast:8 + U, lanes 8..15
}
__device__ __forceinline__ uint32_t group_total(uint32_t v)
{
    int s = (int)v;
    s += __builtin_amdgcn_update_dpp(0, s, 0xb1, 0xf, 0xf, true);   // quad_perm:[1,0,3,2]
    s += __builtin_amdgcn_update_dpp(0, s, 0x4e, 0xf, 0xf, true);   // quad_perm:[2,3,0,1]
    s += __builtin_amdgcn_update_dpp(0, s, 0x141, 0xf, 0xf, true);  // row_half_mirror
    return (uint32_t)s;
}
__device__ __forceinline__ uint32_t group_bits(uint64_t m, int lane)
{
    const uint32_t w = lane & 32 ? (uint32_t)(m >> 32) : (uint32_t)m;
    return __builtin_amdgcn_ubfe(w, (uint32_t)lane & 24u, 8u);
}

// 128 rows of a lane.
struct Bits {
    uint32_t w[4];
};
// The two chains of one individual on them.
struct Rows {
    Bits p, n;
    __device__ __forceinline__ bool any() const
    {
        return ((p.w[0] | p.w[1] | p.w[2]) | (p.w[3] | n.w[0] | n.w[1]) | (n.w[2] | n.w[3])) != 0;
    }
};

// A wave's walk over (individual, panel) units, eight individuals at a time
// (lane group g: the step's individual g).
template <bool NEG, bool COUNT>
struct PairWave {
    const ReqDesc &d;
    const int lane, j, g;
    const uint32_t lane16;  // this lane's byte in a pair's line
    const uint32_t cols;
    const int64_t panel_words;
    uint64_t steps = 0;

    __device__ PairWave(const ReqDesc &dd, int l)
        : d(dd), lane(l), j(l & (kGroup - 1)), g(l / kGroup), lane16((uint32_t)(l & (kGroup - 1)) * 16u),
          cols((uint32_t)dd.cols), panel_words((int64_t)dd.cols * dd.cols * kPanelWords)
    {
    }

    __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(int64_t panel) const
    {
        const uint32_t *p = reinterpret_cast<const uint32_t *>(d.B) + panel * panel_words;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(p), (short)0, (int)(panel_words * 4), 0x00020000);
    }
    __device__ __forceinline__ const uint32_t *ties(int64_t panel) const
    {
        return reinterpret_cast<const uint32_t *>(d.T) + (panel >> 1) * kTieWords;
    }
    __device__ __forceinline__ static Bits load(__amdgpu_buffer_rsrc_t rs, uint32_t off)
    {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0);
        return Bits{{v[0], v[1], v[2], v[3]}};
    }
    template <int N, class F>
    __device__ __forceinline__ static void each(F &&f)
    {
        if constexpr (N > 0) {
            each<N - 1>(f);
            f(std::integral_constant<int, N - 1>{});
        }
    }

    __device__ __forceinline__ uint32_t line(uint32_t word) const
    {
        return (word & kHeadOffset) | (lane16 & ~kHeadOffset);  // (one v_bfi)
    }

    // The groups with one of their pairs among the chunk's n_tied listed
    // ones (lane e of `tie`: entry e, so that all lanes have to be active).
    // asc: the header's word j in lane j < 7 (kNoPair in lanes without a
    // pair); hit: the lane's own pair is one.
    __device__ __forceinline__ bool listed(uint32_t asc, uint32_t tie, uint32_t n_tied, bool &hit) const
    {
        asc &= kHeadOffset;
        hit = false;
#pragma unroll 1
        for (uint32_t e = 0; e < n_tied; ++e) hit |= asc == (uint32_t)__builtin_amdgcn_readlane((int)tie, (int)e);
        return group_bits(__ballot(hit), lane) != 0;
    }

    // N pairs from their lines in one orientation, ANDed into both chains: a
    // pair's line is its own for the chain that it ascends or descends with
    // (own = ~0: the >= chain). w: lane u of the group holds pair u's word
    // (offset, and its direction in bit 31); lanes with sk set are left out.
    // The lines of lanes with comp set are complemented.
    template <int N, bool SKIP>
    __device__ __forceinline__ void lines(Rows &o, int64_t panel, uint32_t w, uint32_t rest, uint32_t sk, uint32_t comp) const
    {
        // (rare in most calls: its broadcasts stay here, not in registers of
        // the loop around it)
        asm volatile("" : "+v"(w));
        __builtin_amdgcn_sched_barrier(0);
        const auto rs = rsrc(panel);
        Bits f[N];
        each<N>([&](auto u) { f[u] = load(rs, line(group_bcast<u>(w))); });
        each<N>([&](auto u) {
            const uint32_t m = (uint32_t)((int32_t)group_bcast<u>(w) >> 31) ^ rest;
            const uint32_t s = SKIP ? group_bcast<u>(sk) : 0u, c = group_bcast<u>(comp);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t x = f[u].w[q] ^ c;
                o.p.w[q] &= x | m | s;
                if (NEG) o.n.w[q] &= x | ~m | s;
                // (pair by pair: words held back to be folded together
                // would take registers that the hot path pays for)
                asm volatile("" : "+v"(o.p.w[q]), "+v"(o.n.w[q]));
            }
        });
    }
    // N pairs in both orientations: asc as above, desc the offset of the
    // other orientation's line, which the build has written for the pairs
    // with a tie (`both` set) and for every pair of a dirty chunk; the
    // others' is the complement of the ascending one.
    template <int N, bool SKIP>
    __device__ __forceinline__ void both_ways(Rows &o, int64_t panel, uint32_t asc, uint32_t desc, uint32_t sk, bool both) const
    {
        lines<N, SKIP>(o, panel, asc, 0u, sk, 0u);
        lines<N, SKIP>(o, panel, both ? (desc & kHeadOffset) | (asc & ~kHeadOffset) : asc, ~0u, sk, both ? 0u : ~0u);
    }

    // Masks of the group's individual (its index in the request).
    __device__ __forceinline__ void put_masks(const Rows &o, int64_t panel, int64_t ind, bool there) const
    {
        if (!(d.mmask || d.nmask)) return;
        int32_t jj = j;
        asm volatile("" : "+v"(jj));  // (no address kept in registers for calls without masks)
        const int64_t words = (d.rows + 63) / 64, word = panel * (kPanelRows / 64) + 2 * jj;
        auto put = [&](uint64_t *m, const Bits &v) {
            if (word < words) m[ind * words + word] = (uint64_t)v.w[0] | ((uint64_t)v.w[1] << 32);
            if (word + 1 < words) m[ind * words + word + 1] = (uint64_t)v.w[2] | ((uint64_t)v.w[3] << 32);
        };
        Bits m, e;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            m.w[q] = o.p.w[q] | o.n.w[q];
            e.w[q] = o.n.w[q] & ~o.p.w[q];
        }
        if (there && d.mmask) put(d.mmask, m);
        if (there && d.nmask) put(d.nmask, e);
    }
    // The group's counts on the panel, in each of its lanes: matched, and
    // negative in the high half (at most 1,024 rows).
    __device__ __forceinline__ uint32_t counts(const Rows &o) const
    {
        uint32_t c = 0, e = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            c += (uint32_t)__builtin_popcount(o.p.w[q] | o.n.w[q]);
            if (NEG) e += (uint32_t)__builtin_popcount(o.n.w[q] & ~o.p.w[q]);
        }
        return group_total(c | (e << 16));
    }
    __device__ __forceinline__ void add(int64_t ind, uint32_t c) const
    {
        if (c & 0xffffu) atomicAdd(d.matched + ind, (int32_t)(c & 0xffffu));
        if (NEG && c >> 16 && d.negative) atomicAdd(d.negative + ind, (int32_t)(c >> 16));
    }

    // LDS of a wave: the step's headers, and the individuals with rows left
    // past the window: the two chains' rows and (k, CSR start, index). Eight
    // of them are finished together, whichever steps they come from.
    template <int N>
    struct Queue {
        Bits p[N][kGroup], n[N][kGroup];
        int4 who[N];
    };
    struct Shared {
        uint32_t head[kStep][8];
        Queue<kQueue> queue;
    };
    // What a wave knows of its panel.
    struct Panel {
        int64_t at;
        bool dirty, last;    // both orientations are needed; the matrix's last panel
        uint32_t n_tied, tie;  // the chunk's listed pairs: their number, entry e in lane e
    };
    __device__ __forceinline__ Panel panel_of(int64_t at, uint32_t n_ties, uint32_t nan) const
    {
        Panel p;
        p.at = at;
        p.dirty = n_ties > (uint32_t)kTieMax || nan != 0;
        p.last = (at + 1) * kPanelRows > d.rows;
        p.n_tied = p.dirty ? 0u : n_ties;
        return p;
    }
    __device__ __forceinline__ Panel panel_of(int64_t at) const
    {
        const uint32_t *tl = ties(at);
        Panel p = panel_of(at, __builtin_amdgcn_readfirstlane(tl[0]), __builtin_amdgcn_readfirstlane(tl[1]));
        p.tie = p.n_tied ? tl[kTieList + (lane & (kTieMax - 1))] : 0u;
        return p;
    }
    // The same from a word loaded before: in lanes 0 .. 31 the list, in lane
    // 32 the count, in 33 the NaN flag.
    __device__ __forceinline__ uint32_t panel_word(int64_t at) const
    {
        return ties(at)[lane < kTieMax ? kTieList + lane : lane & 1];
    }
    __device__ __forceinline__ Panel panel_from(int64_t at, uint32_t word) const
    {
        Panel p = panel_of(at, __builtin_amdgcn_readlane(word, kTieMax), __builtin_amdgcn_readlane(word, kTieMax + 1));
        p.tie = word;
        return p;
    }
    // The group's header, from LDS each time that it is needed (not kept in
    // registers in between).
    __device__ __forceinline__ void read_head(const uint32_t (*head)[8], uint32_t (&w)[8]) const
    {
        int32_t at = g;
        asm volatile("" : "+v"(at));
        const uint4 *p = reinterpret_cast<const uint4 *>(head[at]);
        const uint4 x = p[0], y = p[1];
        w[0] = x.x, w[1] = x.y, w[2] = x.z, w[3] = x.w;
        w[4] = y.x, w[5] = y.y, w[6] = y.z, w[7] = y.w;
    }
    // out(individual, counts) in one lane of each.
    template <class Queue, class Out>
    __device__ __forceinline__ void finish_queued(Queue *q, int32_t from, int32_t count, const Panel &pn, Out &&out)
    {
        const int64_t panel = pn.at;
        const bool dirty = pn.dirty;
        const uint32_t n_tied = pn.n_tied, tie = pn.tie;
        const bool mine = g < count;
        const int32_t at = from + (mine ? g : 0);
        const int4 who = q->who[at];
        Rows o;
        o.p = q->p[at][j];
        o.n = q->n[at][j];
        const int32_t k = who.x;
        const int32_t *cc = d.colidx + who.y;
        bool left = mine;
#pragma unroll 1
        for (int32_t u = 8; __ballot(left && u < k) != 0; u += 4) {
            // lane j: column u - 1 + j and the next (a group that is done
            // reads its individual's last column)
            const bool now = left && u < k;
            const uint32_t a = (uint32_t)cc[min(u - 1 + j, k - 1)], b = row_next(a);
            const uint32_t f = pair_offset(cols, a, b), r = pair_offset(cols, b, a);
            const uint32_t asc = min(f, r) | (f > r ? 0x80000000u : 0u), sk = a == b ? ~0u : 0u;
            bool exact = dirty, both = dirty;
            // (with every lane active: the list is spread over them; before
            // the loads, whose registers the lookup would have to share)
            if (n_tied) exact = listed(now && j < 4 ? asc : kNoPair, tie, n_tied, both);
            if (now) {
                if (!exact) {
                    const auto rs = rsrc(panel);
                    Bits w[4];
                    each<4>([&](auto e) { w[e] = load(rs, line(group_bcast<e>(asc))); });
                    each<4>([&](auto e) {
                        const uint32_t m = (uint32_t)((int32_t)group_bcast<e>(asc) >> 31), s = group_bcast<e>(sk);
#pragma unroll
                        for (int x = 0; x < 4; ++x) {
                            o.p.w[x] &= (w[e].w[x] ^ m) | s;
                            if (NEG) o.n.w[x] &= ~(w[e].w[x] ^ m) | s;
                            asm volatile("" : "+v"(o.p.w[x]), "+v"(o.n.w[x]));
                        }
                    });
                }
                if (exact) both_ways<4, true>(o, panel, asc, max(f, r), sk, both);
                if (COUNT && j == 0) steps += (uint64_t)min(4, k - u);
                left = group_bits(__ballot(o.any()), lane) != 0;
            }
        }
        put_masks(o, panel, who.z, mine);
        const uint32_t c = counts(o);
        if (mine && j == 0) out(who.z, c);
    }

    // One step on a panel: the individuals of the headers at `head` (group g:
    // individual ind of the request, if `there`). Returns the group's counts
    // and queues the individuals with columns and rows left (their counts
    // are 0 here). window(w8, w) gives the seven words of the headers'
    // ascending lines, desc() the lane's word of the second headers.
    template <class Queue, class Window, class Desc>
    __device__ __forceinline__ uint32_t step(const uint32_t (*head)[8], Queue *q, int32_t &queued, const Panel &pn,
                                             int32_t ind, bool there, Window &&window, Desc &&desc)
    {
        const int64_t panel = pn.at;
        const uint32_t flags = head[g][0];
        Rows o;
        bool exact = pn.dirty, both = pn.dirty;
        if (!pn.dirty) {
            uint32_t w8[8];
            read_head(head, w8);
            Bits w[7];
            window(w8, w);
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                uint32_t a = ~0u, b = 0;
#pragma unroll
                for (int u = 0; u < 7; ++u) {
                    const uint32_t m = (uint32_t)((int32_t)w8[u] >> 31);
                    a &= w[u].w[x] ^ m;
                    if (NEG) b |= w[u].w[x] ^ m;
                }
                o.p.w[x] = a;
                o.n.w[x] = NEG ? ~b : 0u;
                asm volatile("" : "+v"(o.p.w[x]), "+v"(o.n.w[x]));
            }
            if (pn.n_tied) exact = listed(j < 7 ? head[g][j] : kNoPair, pn.tie, pn.n_tied, both);
        }
        if (exact) {
#pragma unroll
            for (int x = 0; x < 4; ++x) o.p.w[x] = ~0u, o.n.w[x] = NEG ? ~0u : 0u;
            both_ways<7, false>(o, panel, head[g][j], desc(), 0, both);
        }
        const bool live = there && (flags & kHeadValid) != 0;
        if (pn.last || __ballot(live) != ~0ull) {  // the matrix's rows, the valid individuals
            int32_t rows = (int32_t)min(d.rows - panel * kPanelRows, (int64_t)kPanelRows);
            asm volatile("" : "+s"(rows));
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const int32_t c = rows - (128 * j + 32 * x);
                const uint32_t v = !live ? 0u : c >= 32 ? ~0u : c <= 0 ? 0u : ((1u << c) - 1u);
                o.p.w[x] &= v;
                o.n.w[x] &= v;
            }
        }
        if (COUNT && j == 0 && live) steps += 7;
        const uint64_t any = __ballot(o.any());
        const bool wait = (flags & kHeadLonger) != 0 && group_bits(any, lane) != 0;
        const uint64_t waiting = __ballot(wait), leads = waiting & 0x0101010101010101ull;
        if (waiting) {
            if (wait) {
                // (the leading lanes of the groups before this one)
                const int32_t to = queued - (j > 0 ? 1 : 0) +
                                   (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(leads >> 32),
                                                                      __builtin_amdgcn_mbcnt_lo((uint32_t)leads, 0));
                q->p[to][j] = o.p;
                q->n[to][j] = o.n;
                if (j == 0) {
                    uint32_t w8[8], k = 0;  // (six bits in each of words 1 .. 6)
                    read_head(head, w8);
#pragma unroll
                    for (int u = 1; u < 7; ++u) k |= (w8[u] & 63u) << (6 * (u - 1));
                    q->who[to] = make_int4((int32_t)k, (int32_t)w8[7], ind, 0);
                }
            }
            queued += (int32_t)__popcll(leads);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
        put_masks(o, panel, ind, there && !wait);
        if ((any & ~waiting) == 0) return 0u;
        const uint32_t c = counts(o);
        return wait ? 0u : c;
    }

    // Individuals [first, first + n) of the request (at most 64), eight per
    // step, on one panel.
    __device__ __forceinline__ void item(const IndHead *__restrict__ heads, int32_t first, int32_t n, int64_t panel, Shared *q)
    {
        const Panel pn = panel_of(panel);
        // headers of 8 words; the descending orientations' offsets past them
        const uint32_t *hw = reinterpret_cast<const uint32_t *>(heads + d.head_base) + 8 * (int64_t)first;
        const uint32_t *hd = hw + 8 * (int64_t)d.n;
        auto at = [&](int32_t i) { return (uint32_t)(8 * min(i + g, n - 1) + j); };
        uint32_t h = __builtin_nontemporal_load(hw + at(0));
        uint32_t acc = 0;
        int32_t queued = 0;
#pragma unroll 1
        for (int32_t i = 0; i < n || queued > 0; i += kStep) {
            if (i < n) {
                // lane j of the group has word j of its header; all of them
                // to all of its lanes
                q->head[g][j] = h;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                const uint32_t c = step(
                    q->head, &q->queue, queued, pn, first + i + g, i + g < n,
                    [&](const uint32_t (&w8)[8], Bits (&w)[7]) {
                        const auto rs = rsrc(panel);
#pragma unroll
                        for (int u = 0; u < 7; ++u) w[u] = load(rs, line(w8[u]));
                        h = __builtin_nontemporal_load(hw + at(i + kStep));
                    },
                    [&] { return __builtin_nontemporal_load(hd + at(i)); });
                if (pn.dirty) h = __builtin_nontemporal_load(hw + at(i + kStep));
                if (j == i / kStep) acc = c;
            }
            // eight that wait, or the last ones
            if (queued >= kStep || (i + kStep >= n && queued > 0)) {
                const int32_t now = min(queued, kStep);
                queued -= now;
                finish_queued(&q->queue, queued, now, pn, [&](int32_t ind, uint32_t c) { add(ind, c); });
            }
        }
        if (kStep * j + g < n) add(first + kStep * j + g, acc);
    }
};

// The plain launch: a grid of (8 x groups, panels / 8 over y and z) blocks.
// Block (x, y, z) works on panel 8 (z Y + y) + x mod 8 and group x / 8 (P
// individuals, `per` to a wave): blocks are dispatched x first, and with
// gridDim.x a multiple of 8 the linear block index is x mod 8 modulo 8, so
// on MI355X's round-robin placement of blocks over the eight XCDs the blocks
// of a panel all run on one XCD and share its L2, and the blocks of eight
// consecutive panels (all their groups) are dispatched together.
// (72 vector registers: seven waves per SIMD without spills)
template <bool NEG, bool COUNT>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(7)))
k_eval_pairs(ReqDesc d, const IndHead *__restrict__ heads, int32_t P, int32_t per, unsigned long long *step_counter)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const int64_t panel = 8 * ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) + (blockIdx.x & 7);
    if (panel * kPanelRows >= d.rows) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int32_t i0 = (int32_t)(blockIdx.x >> 3) * P;
    const int32_t first = i0 + wave * per, n = min(min(d.n, i0 + P) - first, per);
    if (n <= 0) return;
    using Wave = PairWave<NEG, COUNT>;
    Wave w(d, lane);
    w.item(heads, first, n, panel, reinterpret_cast<typename Wave::Shared *>(lds) + wave);
    if (COUNT && w.steps) atomicAdd(step_counter, (unsigned long long)w.steps);
}

// The launch for matrices of few panels: the whole evaluation in one kernel.
// A block takes eight individuals on the panels slice, slice + S, ... of one
// of S slices: its first two waves make the headers (as the prep kernel
// does, into LDS), each wave works on every W-th of those panels, and the
// counts are summed in LDS, so that neither headers nor zeroed outputs come
// from a kernel before. With one slice a block writes its counts; with more,
// each adds them to an accumulator per individual (negative and matched 26
// bits each, the slices added above them) and the one that adds last writes
// them. A call zeroes the accumulators that the call before it used.
// Bound by the launch and by a wave's chain of loads. AHEAD: the next panel's
// window is loaded while one is worked on (at four waves per SIMD); without
// it six waves fit, for slices of a panel per wave. Individuals that wait
// are finished on each panel. The whole call, one after the other, with two
// kernels and with one: 54,675 x 178 with masks, 200 individuals 14.4 and 11.9
// us; 20,000 x 200 with missing values, 800 individuals 11.8 and 8.8 (11.2 in
// one slice of 16 waves).
template <bool NEG, bool COUNT, bool AHEAD>
__global__ void __launch_bounds__(1024) k_eval_few(ReqDesc d, int32_t n_panels, int32_t S, FewSums sums,
                                                   unsigned long long *step_counter)
{
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ __align__(16) uint32_t head[kStep][8], desc[kStep][8];
    __shared__ int32_t matched[kStep], negative[kStep];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int W = blockDim.x / kWave;
    const int32_t slice = (int32_t)blockIdx.x % S, i0 = (int32_t)blockIdx.x / S * kStep;
    for (int32_t i = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x); i < sums.n_used; i += (int32_t)(gridDim.x * blockDim.x))
        sums.used[i] = 0;
    for (int32_t t = wave; t < 2; t += W) {
        const int32_t own = 4 * t + (lane >> 4), j = lane & 15;
        const PairPrep p = prep_pairs_quad(d, i0 + own, i0 + own < d.n, lane);
        if (j < 8) {
            head[own][j] = p.word;
            desc[own][j] = p.desc;
        }
        if (j == 0) matched[own] = negative[own] = 0;
    }
    __syncthreads();
    using Wave = PairWave<NEG, COUNT>;
    Wave w(d, lane);
    using Queue = typename Wave::template Queue<kStep>;
    Queue *q = reinterpret_cast<Queue *>(lds) + wave;
    const bool there = i0 + w.g < d.n;
    uint32_t m = 0, e = 0;
    Bits next[7];
    uint32_t word = 0;
    auto fetch = [&](int32_t r) {
        uint32_t w8[8];
        w.read_head(head, w8);
        word = w.panel_word(r);
        const auto rs = w.rsrc(r);
#pragma unroll
        for (int u = 0; u < 7; ++u) next[u] = w.load(rs, w.line(w8[u]));
    };
    const int32_t first = slice + wave * S, stride = W * S;
    if (AHEAD && first < n_panels) fetch(first);
#pragma unroll 1
    for (int32_t r = first; r < n_panels; r += stride) {
        if (!AHEAD) fetch(r);
        Bits now[7];
#pragma unroll
        for (int u = 0; u < 7; ++u) now[u] = next[u];
        const auto pn = w.panel_from(r, word);
        if (AHEAD && r + stride < n_panels) fetch(r + stride);
        int32_t queued = 0;
        const uint32_t c = w.step(
            head, q, queued, pn, i0 + w.g, there,
            [&](const uint32_t (&)[8], Bits (&x)[7]) {
#pragma unroll
                for (int u = 0; u < 7; ++u) x[u] = now[u];
            },
            [&] { return desc[w.g][w.j]; });
        m += c & 0xffffu;
        e += c >> 16;
        if (queued > 0)
            w.finish_queued(q, 0, queued, pn, [&](int32_t ind, uint32_t x) {
                atomicAdd(&matched[ind - i0], (int32_t)(x & 0xffffu));
                if (NEG) atomicAdd(&negative[ind - i0], (int32_t)(x >> 16));
            });
    }
    if (w.j == 0) {
        if (m) atomicAdd(&matched[w.g], (int32_t)m);
        if (NEG && e) atomicAdd(&negative[w.g], (int32_t)e);
    }
    __syncthreads();
    const int32_t i = (int32_t)threadIdx.x;
    if (i < kStep && i0 + i < d.n) {
        uint64_t total = (uint64_t)(uint32_t)matched[i] | (uint64_t)(uint32_t)negative[i] << 26 | 1ull << 52;
        if (S > 1) total += atomicAdd(reinterpret_cast<unsigned long long *>(sums.acc + i0 + i), (unsigned long long)total);
        if (S == 1 || (int32_t)(total >> 52) == S) {
            const bool ok = (head[i][0] & kHeadValid) != 0;
            d.matched[i0 + i] = ok ? (int32_t)(total & 0x3ffffffu) : kInvalid;
            if (d.negative) d.negative[i0 + i] = ok ? (int32_t)(total >> 26 & 0x3ffffffu) : kInvalid;
        }
    }
    if (COUNT && w.steps) atomicAdd(step_counter, (unsigned long long)w.steps);
}

// The batched launch: a fixed grid (a multiple of 8 blocks) over eight item
// lists, one per XCD slice. Block b starts on item b / 8 of list b mod 8;
// short lists are walked with a stride of grid / 8 from there, with no
// counter to contend for, long ones (`dynamic`) by taking the list's next
// item from a counter, fetched while the block works on the item before. A
// stride lets the blocks of a slice drift apart over the items, so that two
// panels and more are in the L2 at a time; from the counter they stay
// within one (the batch above: 19.7 to 9.5 million L2 misses, 462 -> 383
// us). The counters have cache lines of their own: eight in one line took
// 24 ns an item. A list walks its slice's panels in order,
// segment by segment (the requests that read one set of bitmaps), every
// group of every request of the segment on a panel before the next panel:
// item k of slice x in segment g is panel 8 (l / groups) + x and group
// l mod groups (l = k minus the segment's first item in the list), the
// group found among the segment's requests by their first groups.
// (five waves per SIMD, without spills: 402 us for the batch above against
// 412 with six and a few)
template <bool COUNT>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(5)))
k_eval_pairs_batch(const PairQueues *__restrict__ pq, const ReqDesc *__restrict__ descs,
                   const PairSeg *__restrict__ segs, const int32_t *__restrict__ seg_req,
                   const int32_t *__restrict__ seg_gstart, const IndHead *__restrict__ heads,
                   uint32_t *__restrict__ next, unsigned long long *step_counter)
{
    extern __shared__ __align__(16) unsigned char lds[];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int W = blockDim.x / kWave;
    const int32_t n_seg = pq->n_seg;
    const int32_t P = min(pq->P, 64 * W);  // (the planner keeps it there)
    const int32_t per = (P + W - 1) / W;
    const int slice = (int)(blockIdx.x % 8);
    const int32_t stride = (int32_t)(gridDim.x / 8);
    const int32_t total = pq->total[slice];
    uint64_t steps = 0;
    int32_t g = 0;  // (items come in order: the segment only moves forward)
    __shared__ int32_t ticket[2];
    int slot = 0;
    for (int32_t k = (int32_t)(blockIdx.x / 8); k < total;) {
        int32_t mine = 0;
        if (pq->dynamic && threadIdx.x == 0) mine = (int32_t)atomicAdd(next + slice * kPairNextStride, 1u);
        while (g + 1 < n_seg && segs[g + 1].base[slice] <= k) ++g;
        const int32_t local = k - segs[g].base[slice];
        const int32_t groups = segs[g].groups;
        const int64_t panel = 8 * (int64_t)(local / groups) + slice;
        const int32_t pos = local % groups;
        int32_t lo = segs[g].e0, hi = segs[g].e0 + segs[g].n_req - 1;  // the last entry starting at or before pos
        while (lo < hi) {
            const int32_t mid = (lo + hi + 1) >> 1;
            if (seg_gstart[mid] <= pos) lo = mid;
            else hi = mid - 1;
        }
        const ReqDesc &d = descs[seg_req[lo]];
        const int32_t first = (pos - seg_gstart[lo]) * P + wave * per;
        const int32_t n = min(min(d.n, (pos - seg_gstart[lo]) * P + P) - first, per);
        if (n <= 0) {
        } else if (d.flags & kFlagNeg) {
            using Wave = PairWave<true, COUNT>;
            Wave w(d, lane);
            w.item(heads, first, n, panel, reinterpret_cast<typename Wave::Shared *>(lds) + wave);
            steps += w.steps;
        } else {
            using Wave = PairWave<false, COUNT>;
            Wave w(d, lane);
            w.item(heads, first, n, panel, reinterpret_cast<typename Wave::Shared *>(lds) + wave);
            steps += w.steps;
        }
        if (pq->dynamic) {
            if (threadIdx.x == 0) ticket[slot] = mine;
            __syncthreads();
            k = stride + __builtin_amdgcn_readfirstlane(ticket[slot]);
            slot ^= 1;
        } else {
            k += stride;
        }
    }
    if (COUNT && steps) atomicAdd(step_counter, (unsigned long long)steps);
}

}  // namespace

int64_t pair_words(int64_t rows) { return (rows + kChunkRows - 1) / kChunkRows * kChunkWords; }

int64_t pair_panels(int64_t rows) { return (rows + kPanelRows - 1) / kPanelRows; }

int64_t pair_tie_bytes(int64_t rows)
{
    return (rows + kChunkRows - 1) / kChunkRows * kTieWords * (int64_t)sizeof(uint32_t);
}

hipError_t launch_pair_bits(const float *X, int64_t rows, int64_t ld, int32_t cols, bool full, bool subst, float fill,
                            uint32_t *G, int64_t w32, uint32_t *T, hipStream_t s)
{
    if (cols < 1 || cols > kMaxPairCols || w32 != pair_words(rows) || ld % 64 != 0) return hipErrorInvalidValue;
    const int64_t chunks = w32 / kChunkWords;
    const int64_t per_slice = (chunks + 7) / 8;
    if (per_slice > 65535) return hipErrorInvalidValue;
    // Columns b per block: 32; 64 where the tiles still make eight blocks per
    // CU (less time goes to staging the columns a: 436,444 x 310 3.12 -> 2.99
    // ms), 16 where they make less than two (1,000 x 50 45 -> 27 us). At
    // 54,675 x 178 16, 32 and 64 take 199, 190 and 209 us.
    auto tiles = [&](int32_t r) { return (int64_t)((cols + kBuildCols - 1) / kBuildCols) * ((cols + r - 1) / r); };
    const int32_t run = tiles(64) * chunks >= 2048 ? 64 : tiles(32) * chunks < 512 ? 16 : 32;
    const dim3 grid((unsigned)(8 * tiles(run)), (unsigned)per_slice), block(kBuildWaves * kWave);
    const int sub = subst ? 1 : 0;
    clear_last_error();
    if (full) {
        hipLaunchKernelGGL(k_pair_bits<true>, grid, block, 0, s, X, rows, ld, cols, sub, fill, run, 0, G, T);
    } else {
        hipLaunchKernelGGL(k_pair_bits<false>, grid, block, 0, s, X, rows, ld, cols, sub, fill, run, 0, G, T);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        // the chunks whose list has overflowed: both orientations
        hipLaunchKernelGGL(k_pair_bits<true>, grid, block, 0, s, X, rows, ld, cols, sub, fill, run, kTieMax, G, T);
    }
    return hipGetLastError();
}

hipError_t launch_prep_pairs(const ReqDesc &d, IndHead *heads, hipStream_t s)
{
    const int threads = 256;
    const int per_block = threads / 16;  // 16 lanes per individual
    clear_last_error();
    hipLaunchKernelGGL(k_prep_pairs, dim3((d.n + per_block - 1) / per_block), dim3(threads), 0, s, d, heads);
    return hipGetLastError();
}

static const void *pairs_batch_kernel(bool count)
{
    return count ? (const void *)&k_eval_pairs_batch<true> : (const void *)&k_eval_pairs_batch<false>;
}

int pairs_batch_occupancy(int32_t W)
{
    int blocks = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, pairs_batch_kernel(false), W * kWave, W * kWaveLds) !=
        hipSuccess)
        return 0;
    return blocks;
}

hipError_t launch_pairs_batch(const PairQueues *pq, const ReqDesc *descs, const PairSeg *segs,
                              const int32_t *seg_req, const int32_t *seg_gstart, const IndHead *heads,
                              uint32_t *next, int32_t W, int32_t grid, unsigned long long *step_counter, hipStream_t s)
{
    if (W < 1 || W > 16 || grid < 8 || grid % 8 != 0) return hipErrorInvalidValue;
    const bool count = step_counter != nullptr;
    clear_last_error();
    if (count)
        hipLaunchKernelGGL(k_eval_pairs_batch<true>, dim3(grid), dim3(W * kWave), W * kWaveLds, s, pq, descs, segs, seg_req,
                           seg_gstart, heads, next, step_counter);
    else
        hipLaunchKernelGGL(k_eval_pairs_batch<false>, dim3(grid), dim3(W * kWave), W * kWaveLds, s, pq, descs, segs, seg_req,
                           seg_gstart, heads, next, step_counter);
    return hipGetLastError();
}

hipError_t launch_pairs_few(const ReqDesc &d, int32_t W, int32_t S, const FewSums &sums,
                            unsigned long long *step_counter, hipStream_t s)
{
    const int64_t panels = pair_panels(d.rows), groups = ((int64_t)d.n + kStep - 1) / kStep;
    if (W < 1 || W > 16 || panels > kFewPanels || S < 1 || S > panels || (S > 1 && (!sums.acc || d.n > kFewInd)) ||
        groups * S * W * kWave > 0xffffffffll)
        return hipErrorInvalidValue;
    const bool neg = (d.flags & kFlagNeg) != 0;
    clear_last_error();
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)(groups * S)), dim3(W * kWave), W * kWaveLdsFew, s, d, (int32_t)panels, S,
                           sums, step_counter);
        return hipGetLastError();
    };
    if ((int64_t)W * S >= panels) {
        if (step_counter) return neg ? go(k_eval_few<true, true, false>) : go(k_eval_few<false, true, false>);
        return neg ? go(k_eval_few<true, false, false>) : go(k_eval_few<false, false, false>);
    }
    if (step_counter) return neg ? go(k_eval_few<true, true, true>) : go(k_eval_few<false, true, true>);
    return neg ? go(k_eval_few<true, false, true>) : go(k_eval_few<false, false, true>);
}

hipError_t launch_pairs(const ReqDesc &d, const IndHead *heads, int32_t P, int32_t W,
                        unsigned long long *step_counter, hipStream_t s)
{
    if (W < 1 || W > 16 || P < 1 || P > 64 * W) return hipErrorInvalidValue;
    // (a grid's x has less than 2^32 threads: larger groups past that, up to
    // 64 individuals per wave)
    auto threads = [&] { return 8 * (((int64_t)d.n + P - 1) / P) * W * kWave; };
    while (threads() > 0xffffffffll && P < 64 * W) P = P * 2 < 64 * W ? P * 2 : 64 * W;
    if (threads() > 0xffffffffll) return hipErrorInvalidValue;
    const int64_t groups = ((int64_t)d.n + P - 1) / P, per_slice = (pair_panels(d.rows) + 7) / 8;
    const int32_t per = (P + W - 1) / W;
    const bool neg = (d.flags & kFlagNeg) != 0;
    // a slice's panels over y and z (65,535 of each are the grid's limit)
    const unsigned y = (unsigned)(per_slice < 32768 ? per_slice : 32768), z = (unsigned)((per_slice + y - 1) / y);
    const dim3 grid((unsigned)(8 * groups), y, z);
    clear_last_error();
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(W * kWave), W * kWaveLds, s, d, heads, P, per, step_counter);
    };
    if (step_counter) {
        if (neg) go(k_eval_pairs<true, true>);
        else go(k_eval_pairs<false, true>);
    } else {
        if (neg) go(k_eval_pairs<true, false>);
        else go(k_eval_pairs<false, false>);
    }
    return hipGetLastError();
}

}  // namespace ebic
