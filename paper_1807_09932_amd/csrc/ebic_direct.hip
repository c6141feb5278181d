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
// with four, five, six and seven columns first, before the two savings
// below), and the columns past the window four at a time in the same way
// while any row is left. A row's two chains are carried as masks over the
// lanes; their population counts are kept in a lane per individual and
// added to the outputs once at the end.
//
// Every individual reads its first columns on every row, from the L2 as far
// as it holds them: 0.36 GB at 20,000 x 900 with 800 individuals, 15 TB/s
// over the kernel's 24 us. Bound by instruction issue, per individual and 256
// rows 93 vector and 131 scalar ones (115 and 161 with 64-bit addresses and
// an AND for every compare: 30.3 us an evaluation; 109 and 122 with buffer loads, a
// column's address a 32-bit scalar offset: 27.7; 26.3 with the first
// compares narrowing the execution mask as well). Blocks are placed as
// those of the pair bitmaps: the blocks of a 256-row chunk run on one XCD
// and are dispatched together, so that the chunk's columns (0.9 MB at 900)
// are read once into that XCD's L2 and shared by the individuals. The
// kernel it replaced (one row per lane, one column of one 64-row tile at a
// time) took 134 us an evaluation; at 20,000 x 620 the FP32 tile in LDS,
// which still fits one block per CU, takes 54.8 us and this kernel 25.2.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "ebic_internal.h"

namespace ebic {
namespace {

constexpr int kDirectRows = 256;  // rows of one wave step: 64 lanes x 4 rows
constexpr int kFirst = 6;          // columns every lane loads; the window's others where a row is left
constexpr int kRest = kWin - kFirst;

// One individual's state on the wave's rows: row r of every lane as a mask
// over the lanes, for each direction.
struct Chain {
    uint64_t p[4], n[4];
    float v[4];  // the last column's values
};

template <bool NEG>
__device__ __forceinline__ void chain_step(Chain &c, const float4 &f)
{
    const float x[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        c.p[r] &= __ballot(x[r] >= c.v[r]);
        if (NEG) c.n[r] &= __ballot(x[r] <= c.v[r]);
        c.v[r] = x[r];
    }
}

template <bool NEG>
__device__ __forceinline__ uint64_t chain_live(const Chain &c)
{
    const uint64_t p = (c.p[0] | c.p[1]) | (c.p[2] | c.p[3]);
    if (!NEG) return p;
    return p | ((c.n[0] | c.n[1]) | (c.n[2] | c.n[3]));
}

// The first six columns of one row: every compare narrows the execution
// mask, so that a direction takes five instructions and no masks between
// them (the kernel is bound by scalar as much as by vector instructions).
// All lanes are active around it.
template <bool NEG>
__device__ __forceinline__ void first_columns(uint64_t &p, uint64_t &n, float x0, float x1, float x2, float x3, float x4,
                                              float x5)
{
    uint64_t all;
    if (NEG)
        asm volatile("s_mov_b64 %[all], exec\n\t"
                     "s_mov_b64 exec, %[p]\n\t"
                     "v_cmpx_ge_f32_e32 vcc, %[x1], %[x0]\n\t"
                     "v_cmpx_ge_f32_e32 vcc, %[x2], %[x1]\n\t"
                     "v_cmpx_ge_f32_e32 vcc, %[x3], %[x2]\n\t"
                     "v_cmpx_ge_f32_e32 vcc, %[x4], %[x3]\n\t"
                     "v_cmpx_ge_f32_e32 vcc, %[x5], %[x4]\n\t"
                     "s_mov_b64 %[p], exec\n\t"
                     "s_mov_b64 exec, %[n]\n\t"
                     "v_cmpx_le_f32_e32 vcc, %[x1], %[x0]\n\t"
                     "v_cmpx_le_f32_e32 vcc, %[x2], %[x1]\n\t"
                     "v_cmpx_le_f32_e32 vcc, %[x3], %[x2]\n\t"
                     "v_cmpx_le_f32_e32 vcc, %[x4], %[x3]\n\t"
                     "v_cmpx_le_f32_e32 vcc, %[x5], %[x4]\n\t"
                     "s_mov_b64 %[n], exec\n\t"
                     "s_mov_b64 exec, %[all]\n\t"
                     "s_nop 1"  // (four wait states from a VALU write of EXEC to a lane access; no DPP move follows)
                     : [p] "+s"(p), [n] "+s"(n), [all] "=&s"(all)
                     : [x0] "v"(x0), [x1] "v"(x1), [x2] "v"(x2), [x3] "v"(x3), [x4] "v"(x4), [x5] "v"(x5)
                     : "vcc");
    else
        asm volatile("s_mov_b64 %[all], exec\n\t"
                     "s_mov_b64 exec, %[p]\n\t"
                     "v_cmpx_ge_f32_e32 vcc, %[x1], %[x0]\n\t"
                     "v_cmpx_ge_f32_e32 vcc, %[x2], %[x1]\n\t"
                     "v_cmpx_ge_f32_e32 vcc, %[x3], %[x2]\n\t"
                     "v_cmpx_ge_f32_e32 vcc, %[x4], %[x3]\n\t"
                     "v_cmpx_ge_f32_e32 vcc, %[x5], %[x4]\n\t"
                     "s_mov_b64 %[p], exec\n\t"
                     "s_mov_b64 exec, %[all]\n\t"
                     "s_nop 1"  // (four wait states from a VALU write of EXEC to a lane access)
                     : [p] "+s"(p), [all] "=&s"(all)
                     : [x0] "v"(x0), [x1] "v"(x1), [x2] "v"(x2), [x3] "v"(x3), [x4] "v"(x4), [x5] "v"(x5)
                     : "vcc");
}

// NEAR: every column starts within 4 GB of the first, so that a column's
// address is a 32-bit scalar offset.
template <bool NEG, bool COUNT, bool NEAR>
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
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(d.X) + row0, (short)0, NEAR ? (int)((uint32_t)((int64_t)d.cols * d.ld - row0) * 4u) : 0, 0x00020000);
    const uint32_t at = NEAR ? (uint32_t)(min(row, d.ld - 4) - row0) * 4u : 0u, stride = (uint32_t)d.ld * 4u;
    auto ld = [&](int32_t c) {
        float4 f;
        if (NEAR) {
            const auto w = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)at, (int)((uint32_t)c * stride), 0);
            __builtin_memcpy(&f, &w, 16);
        } else {
            f = *reinterpret_cast<const float4 *>(X + (int64_t)c * d.ld);
        }
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
    uint64_t valid[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) valid[r] = __ballot(row + r < d.rows);
    // the first columns (a header's columns repeat its last one: a repeat
    // changes nothing, and one column is compared with itself)
    auto begin = [&](Chain &c, const Head &h, const float4 *f) {
        static_assert(kFirst == 6, "the columns of first_columns");
        auto x = [&](int u, int r) { return reinterpret_cast<const float *>(&f[u])[r]; };
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            c.p[r] = h.k > 0 ? valid[r] : 0;
            c.n[r] = NEG ? c.p[r] : 0;
            first_columns<NEG>(c.p[r], c.n[r], x(0, r), x(1, r), x(2, r), x(3, r), x(4, r), x(5, r));
            c.v[r] = x(5, r);
        }
        if (COUNT && lane == 0) steps += 4 * (uint64_t)max(min(h.k, kFirst) - 1, min(h.k, 1));
    };
    auto mine = [&](uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); };
    uint32_t acc_m = 0, acc_g = 0;
    // the columns past the window, then masks and counts
    auto finish = [&](Chain &c, const Head &h, int32_t ii, int32_t t) {
        if (h.k > kWin && chain_live<NEG>(c) != 0) {
            const int32_t *cc = d.colidx + __builtin_amdgcn_readfirstlane(hb[ii].begin);
            for (int32_t u = kWin; u < h.k; u += 4) {
                const uint64_t live = chain_live<NEG>(c);
                if (live == 0) break;
                int32_t cn[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) cn[e] = __builtin_amdgcn_readfirstlane(cc[min(u + e, h.k - 1)]);
                float4 f[4] = {};
                if (mine(live)) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) f[e] = ld(cn[e]);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) chain_step<NEG>(c, f[e]);
                if (COUNT && lane == 0) steps += 4 * (uint64_t)min(4, h.k - u);
            }
        }
        int32_t m = 0, g = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            m += (int32_t)__popcll(c.p[r] | c.n[r]);
            if (NEG) g += (int32_t)__popcll(c.n[r] & ~c.p[r]);
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
                mw |= (mine(c.p[r] | c.n[r]) ? 1u : 0u) << r;
                gw |= (mine(c.n[r] & ~c.p[r]) ? 1u : 0u) << r;
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
            // (lanes without a row left are not loaded for: their rows stay out)
            const uint64_t la = ha.k > kFirst ? chain_live<NEG>(A) : 0;
            if (mine(la)) {
#pragma unroll
                for (int u = 0; u < kRest; ++u) fa[u] = ld(ha.c[kFirst + u]);
            }
            begin(B, hc, fb);
            const uint64_t lb = two && hc.k > kFirst ? chain_live<NEG>(B) : 0;
            if (mine(lb)) {
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
    if (W < 1 || W > 16 || P < 1 || d.ld % 4 != 0) return hipErrorInvalidValue;
    // (a grid's x has less than 2^32 threads: larger groups past that, from
    // 33.5 million individuals on in the default shape)
    auto threads = [&] { return 8 * (((int64_t)d.n + P - 1) / P) * W * kWave; };
    while (threads() > 0xffffffffll) P *= 2;
    const int64_t groups = ((int64_t)d.n + P - 1) / P, per_slice = (direct_chunks(d.rows) + 7) / 8;
    const bool neg = (d.flags & kFlagNeg) != 0;
    clear_last_error();
    // a slice's chunks over y and z (up to 2^31 rows: 32 z of 32,768)
    const unsigned y = (unsigned)std::min<int64_t>(32768, per_slice), z = (unsigned)((per_slice + y - 1) / y);
    const dim3 grid((unsigned)(8 * groups), y, z);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(W * kWave), 0, s, d, heads, P, step_counter); };
    const bool near = (int64_t)d.cols * d.ld * 4 <= 0xffffffffll;
    auto pick = [&](auto count) {
        constexpr bool C = decltype(count)::value;
        if (near) return neg ? go(k_eval_direct<true, C, true>) : go(k_eval_direct<false, C, true>);
        return neg ? go(k_eval_direct<true, C, false>) : go(k_eval_direct<false, C, false>);
    };
    if (step_counter) pick(std::true_type());
    else pick(std::false_type());
    return hipGetLastError();
}

}  // namespace ebic
