// ebic_direct.hip -- the predicate read straight from the column-major
// matrix: the default past 512 columns, and on request.
//
// A wave takes one individual on 256 rows: lane l holds rows 4 l .. 4 l + 3
// of a column as one 16-byte load, so a column step is one load instruction
// and, per row of the lane, one compare for each trend. The first six
// columns of two individuals are loaded together; the window's other two
// only by lanes with a row left on a chain (after six columns of a random
// individual that is one lane in twelve, so most cache lines stay unread;
// 20,000 x 900, 800 individuals: 32.5, 31.9, 31.0 and 31.9 us an evaluation
// with four, five, six and seven columns first), and the columns past the
// window four at a time in the same way while any row is left. A row's two
// chains are carried as two predicates; the counts are population counts of
// ballots, kept in a lane per individual and added to the outputs once at
// the end.
//
// Every individual reads its first columns on every row, from the L2 as far
// as it holds them: 0.39 GB at 20,000 x 900 with 800 individuals, about 14
// TB/s; the compares and the scalar ANDs of the predicates take about as
// long as the loads. Blocks are placed as those of the pair bitmaps: the
// blocks of a 256-row chunk run on one XCD and are dispatched together, so
// that the chunk's columns (0.9 MB at 900) are read once into that XCD's L2
// and shared by the individuals. The kernel it replaced (one row per lane,
// one column of one 64-row tile at a time) took 131 us there, this one 27;
// at 20,000 x 620 the FP32 tile in LDS, which still fits one block per CU,
// takes 56 us an evaluation and this kernel 31.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "ebic_internal.h"

namespace ebic {
namespace {

constexpr int kDirectRows = 256;  // rows of one wave step: 64 lanes x 4 rows
constexpr int kFirst = 6;          // columns every lane loads; the window's others where a row is left
constexpr int kRest = kWin - kFirst;

// One individual's state on the wave's rows.
struct Chain {
    bool p[4], n[4];
    float v[4];  // the last column's values
};

template <bool NEG>
__device__ __forceinline__ void chain_step(Chain &c, const float4 &f)
{
    const float x[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        c.p[r] = c.p[r] & (x[r] >= c.v[r]);
        if (NEG) c.n[r] = c.n[r] & (x[r] <= c.v[r]);
        c.v[r] = x[r];
    }
}

template <bool NEG>
__device__ __forceinline__ bool chain_live(const Chain &c)
{
    const bool p = (c.p[0] | c.p[1]) | (c.p[2] | c.p[3]);
    if (!NEG) return p;
    return p | ((c.n[0] | c.n[1]) | (c.n[2] | c.n[3]));
}

template <bool NEG, bool COUNT>
__global__ void __launch_bounds__(1024) k_eval_direct(ReqDesc d, const IndHead *__restrict__ heads, int32_t P,
                                                      unsigned long long *step_counter)
{
    // block (x, y, z): chunk 8 (z gridDim.y + y) + x mod 8, group x / 8
    const int64_t row0 = (8 * ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) + (blockIdx.x & 7)) * kDirectRows;
    if (row0 >= d.rows) return;
    const int32_t i0 = (int32_t)(blockIdx.x >> 3) * P;
    const int32_t np = min(P, d.n - i0);
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int32_t wave = __builtin_amdgcn_readfirstlane((int32_t)threadIdx.x / kWave);
    const int32_t W = (int32_t)blockDim.x / kWave;
    const IndHead *hb = heads + d.head_base + i0;
    const int64_t row = row0 + 4 * lane;
    // (lanes past the padded rows read the last ones; their rows are not valid)
    const float *X = d.X + min(row, d.ld - 4);
    const bool subst = (d.flags & kFlagSubst) != 0;
    const int64_t words32 = 2 * ((d.rows + 63) / 64);
    uint64_t steps = 0;
    auto ld = [&](int32_t c) {
        float4 f = *reinterpret_cast<const float4 *>(X + (int64_t)c * d.ld);
        if (subst) {
            f.x = f.x != f.x ? d.fill : f.x;
            f.y = f.y != f.y ? d.fill : f.y;
            f.z = f.z != f.z ? d.fill : f.z;
            f.w = f.w != f.w ? d.fill : f.w;
        }
        return f;
    };
    struct Head {
        int32_t k, c[kWin];
    };
    auto head = [&](int32_t ii) {
        const int4 *h = reinterpret_cast<const int4 *>(hb + ii);
        const int4 x0 = h[0], x2 = h[2], x3 = h[3];
        Head r;
        r.k = __builtin_amdgcn_readfirstlane(x0.x);
        r.c[0] = __builtin_amdgcn_readfirstlane(x2.x);
        r.c[1] = __builtin_amdgcn_readfirstlane(x2.y);
        r.c[2] = __builtin_amdgcn_readfirstlane(x2.z);
        r.c[3] = __builtin_amdgcn_readfirstlane(x2.w);
        r.c[4] = __builtin_amdgcn_readfirstlane(x3.x);
        r.c[5] = __builtin_amdgcn_readfirstlane(x3.y);
        r.c[6] = __builtin_amdgcn_readfirstlane(x3.z);
        r.c[7] = __builtin_amdgcn_readfirstlane(x3.w);
        return r;
    };
    // the first four columns (a header's columns repeat its last one: a
    // repeat changes nothing, and one column is compared with itself)
    auto begin = [&](Chain &c, const Head &h, const float4 *f) {
        const float x[4] = {f[0].x, f[0].y, f[0].z, f[0].w};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            c.p[r] = h.k > 0 && row + r < d.rows;
            c.n[r] = NEG && c.p[r];
            c.v[r] = x[r];
        }
#pragma unroll
        for (int u = 1; u < kFirst; ++u) chain_step<NEG>(c, f[u]);
        if (COUNT && lane == 0) steps += 4 * (uint64_t)max(min(h.k, kFirst) - 1, min(h.k, 1));
    };
    uint32_t acc_m = 0, acc_g = 0;
    // the columns past the window, then masks and counts
    auto finish = [&](Chain &c, const Head &h, int32_t ii, int32_t t) {
        if (h.k > kWin && __ballot(chain_live<NEG>(c)) != 0) {
            const int32_t *cc = d.colidx + __builtin_amdgcn_readfirstlane(hb[ii].begin);
            for (int32_t u = kWin; u < h.k; u += 4) {
                const bool live = chain_live<NEG>(c);
                if (__ballot(live) == 0) break;
                int32_t cn[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) cn[e] = __builtin_amdgcn_readfirstlane(cc[min(u + e, h.k - 1)]);
                if (live) {
                    float4 f[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) f[e] = ld(cn[e]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) chain_step<NEG>(c, f[e]);
                }
                if (COUNT && lane == 0) steps += 4 * (uint64_t)min(4, h.k - u);
            }
        }
        int32_t m = 0, g = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            m += (int32_t)__popcll(__ballot(c.p[r] | c.n[r]));
            if (NEG) g += (int32_t)__popcll(__ballot(c.n[r] & !c.p[r]));
        }
        if (lane == t) {
            acc_m = (uint32_t)m;
            acc_g = (uint32_t)g;
        }
        if (d.mmask || d.nmask) {
            // Eight lanes' rows make a 32-bit mask word (little-endian
            // halves of the uint64 words).
            uint32_t mw = 0, gw = 0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                mw |= (c.p[r] | c.n[r] ? 1u : 0u) << r;
                gw |= (c.n[r] & !c.p[r] ? 1u : 0u) << r;
            }
            mw <<= 4 * (lane & 7);
            gw <<= 4 * (lane & 7);
#pragma unroll
            for (int x = 1; x < 8; x <<= 1) {
                mw |= __shfl_xor(mw, x);
                gw |= __shfl_xor(gw, x);
            }
            const int64_t word = row >> 5;
            if ((lane & 7) == 0 && word < words32) {
                const int64_t at = (int64_t)(i0 + ii) * words32 + word;
                if (d.mmask) reinterpret_cast<uint32_t *>(d.mmask)[at] = mw;
                if (d.nmask) reinterpret_cast<uint32_t *>(d.nmask)[at] = gw;
            }
        }
    };
    // the wave's individuals wave + t W, up to 64 of them between two adds
    for (int32_t base = wave; base < np; base += kWave * W) {
        const int32_t end = min(np, base + kWave * W);
        acc_m = acc_g = 0;
        int32_t t = 0;
        for (int32_t ii = base; ii < end; ii += 2 * W, t += 2) {
            const bool two = ii + W < end;
            const Head ha = head(ii), hc = head(two ? ii + W : ii);
            float4 fa[kFirst], fb[kFirst];
#pragma unroll
            for (int u = 0; u < kFirst; ++u) fa[u] = ld(ha.c[u]);
#pragma unroll
            for (int u = 0; u < kFirst; ++u) fb[u] = ld(hc.c[u]);
            Chain A, B;
            begin(A, ha, fa);
            const bool la = ha.k > kFirst && chain_live<NEG>(A);
            if (la) {
#pragma unroll
                for (int u = 0; u < kRest; ++u) fa[u] = ld(ha.c[kFirst + u]);
            }
            begin(B, hc, fb);
            const bool lb = two && hc.k > kFirst && chain_live<NEG>(B);
            if (lb) {
#pragma unroll
                for (int u = 0; u < kRest; ++u) fb[u] = ld(hc.c[kFirst + u]);
            }
            if (la) {
#pragma unroll
                for (int u = 0; u < kRest; ++u) chain_step<NEG>(A, fa[u]);
            }
            if (COUNT && lane == 0) steps += 4 * (uint64_t)max(0, min(ha.k, kWin) - kFirst);
            finish(A, ha, ii, t);
            if (!two) continue;
            if (lb) {
#pragma unroll
                for (int u = 0; u < kRest; ++u) chain_step<NEG>(B, fb[u]);
            }
            if (COUNT && lane == 0) steps += 4 * (uint64_t)max(0, min(hc.k, kWin) - kFirst);
            finish(B, hc, ii + W, t + 1);
        }
        const int32_t ii = base + lane * W;
        if (ii < end) {
            if (acc_m) atomicAdd(d.matched + i0 + ii, (int32_t)acc_m);
            if (NEG && acc_g && d.negative) atomicAdd(d.negative + i0 + ii, (int32_t)acc_g);
        }
    }
    if (COUNT && lane == 0 && steps) atomicAdd(step_counter, (unsigned long long)steps);
}

}  // namespace

int64_t direct_chunks(int64_t rows) { return (rows + kDirectRows - 1) / kDirectRows; }

hipError_t launch_direct(const ReqDesc &d, const IndHead *heads, int32_t P, int32_t W,
                         unsigned long long *step_counter, hipStream_t s)
{
    const int64_t groups = (d.n + P - 1) / P, per_slice = (direct_chunks(d.rows) + 7) / 8;
    if (W < 1 || W > 16 || P < 1 || d.ld % 4 != 0 || 8 * groups * W * kWave > 0xffffffffll) return hipErrorInvalidValue;
    const bool neg = (d.flags & kFlagNeg) != 0;
    clear_last_error();
    // a slice's chunks over y and z (up to 2^31 rows: 32 z of 32,768)
    const unsigned y = (unsigned)std::min<int64_t>(32768, per_slice), z = (unsigned)((per_slice + y - 1) / y);
    const dim3 grid((unsigned)(8 * groups), y, z);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(W * kWave), 0, s, d, heads, P, step_counter); };
    if (step_counter) {
        if (neg) go(k_eval_direct<true, true>);
        else go(k_eval_direct<false, true>);
    } else {
        if (neg) go(k_eval_direct<true, false>);
        else go(k_eval_direct<false, false>);
    }
    return hipGetLastError();
}

}  // namespace ebic
