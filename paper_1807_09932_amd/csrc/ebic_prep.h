// ebic_prep.h -- the per-individual scan shared by the prep kernels.
//
// One wave per individual: the lanes read its columns together (one round
// of independent loads for up to 64 columns), check every column against
// the matrix width, find the leading run of repeats of the first column,
// and gather the header's window of eight columns.
//
// A leading run of repeats of the first column is dropped from the header
// (begin moves to the run's last entry, k shrinks by the same amount):
// comparing a cell with itself always holds (x >= x and x <= x for any
// present value; a missing one is excluded by the kept copy of the column
// in exclude mode and takes the fill value in include mode), so
// c, c, ..., c, rest follows exactly the rows of c, rest, on both chains.
// The evaluation then never sees a first pair that compares a cell with
// itself, which is what lets a chunk without two equal values in any row
// skip the tie handling of the first pair (the SWAR sequences' tie-free
// variants classify every row as rising or falling there), and what gives
// every individual of two or more columns a first pair of two different
// columns.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "ebic_internal.h"

namespace ebic {

constexpr int32_t kInvalid = -1;  // the counts of an individual with an invalid column

struct PrepScan {
    bool ok;      // a non-empty span of valid columns (wave-uniform)
    int32_t k;    // columns from the header's start (0 when not ok)
    int32_t bb;   // the header's CSR start (the last leading repeat)
    int32_t win;  // lanes 8..15: window column lane - 8 from bb (clamped to the last column)
};

__device__ __forceinline__ PrepScan prep_scan(const ReqDesc &d, int32_t i, int lane)
{
    const int32_t b = d.offsets[i], e = d.offsets[i + 1];
    const bool span = b >= 0 && e > b;
    bool bad = false;
    int32_t first = 0;  // lane l: column l of the individual (first 64)
    int32_t run = 0;    // entries b .. b + run hold the first column
    if (span) {
        const int32_t c0 = d.colidx[b];
        run = e - b - 1;  // unless a different column follows
        bool found = false;
        for (int32_t jb = b; jb < e; jb += kWave) {  // (wave-uniform trip count)
            const int32_t j = jb + lane;
            const bool in = j < e;
            const int32_t c = in ? d.colidx[j] : c0;
            if (jb == b) first = c;
            bad |= in && (c < 0 || c >= d.cols);
            const uint64_t differ = __ballot(in && c != c0);
            if (!found && differ != 0) {
                found = true;
                run = (jb - b) + (int32_t)__builtin_ctzll(differ) - 1;
            }
        }
    }
    PrepScan sc;
    sc.ok = span && __ballot(bad) == 0;
    sc.bb = b + run;
    sc.k = sc.ok ? e - sc.bb : 0;
    const int32_t src = run + min(lane - 8, e - sc.bb - 1);
    int32_t win = __shfl(first, (src >= 0 && src < kWave) ? src : 0);
    if (span && lane >= 8 && lane < 16 && src >= kWave) win = d.colidx[b + src];
    sc.win = win;
    return sc;
}

// ---------------------------------------------------------------------------
// The pairs headers of the pair-bitmap kernels: two arrays of 32 bytes per
// individual in a request's header storage (64 bytes per individual).
// The first, read by every evaluation step:
//   words 0 .. 6   window pair u, (c_u, c_{u+1}): the byte offset in a panel
//                  of its ascending orientation (bits 7 .. 26), and bit 31
//                  set where c_u > c_{u+1}. A pair of equal columns is
//                  implied by the pairs next to it and takes pair 0's place
//                  (which is of two different columns, or the diagonal pair
//                  of an individual of one column).
//                  Word 0 also has bit 0 set for a valid individual and bit
//                  1 for one of more than eight columns; words 1 .. 6 hold
//                  k, the columns from the start on, six bits in each (the
//                  lowest first).
//   word 7         the CSR start (the last leading repeat of the first column)
// The second, behind the first array, for panels with ties or missing cells:
//   words 0 .. 6   the offsets of the descending orientations
// ---------------------------------------------------------------------------
constexpr uint32_t kHeadOffset = 0x07ffff80u;
constexpr uint32_t kHeadValid = 1u, kHeadLonger = 2u;

// DPP moves within a row of 16 lanes: lane 0 to all of it; lane j + 1 to
// lane j.
__device__ __forceinline__ uint32_t row_first(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150, 0xf, 0xf, true);  // row_newbcast:0
}
__device__ __forceinline__ uint32_t row_next(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x101, 0xf, 0xf, false);  // row_shl:1
}

// Pair (a, b)'s bytes in a panel: a cache line.
__device__ __forceinline__ uint32_t pair_offset(uint32_t cols, uint32_t a, uint32_t b)
{
    return (a * cols + b) << 7;
}

struct PairPrep {
    uint32_t word, desc;  // lane j < 8 of the row: word j of the two headers
    bool ok;              // a non-empty span of valid columns
};

// Four individuals per wave, one per row of 16 lanes: individual i of
// request d (rows with !active do nothing). The row's lanes read its columns
// 16 at a time, check them against the matrix width and find the leading run
// of repeats; the window's pairs are formed in lanes 0 .. 6.
__device__ __forceinline__ PairPrep prep_pairs_quad(const ReqDesc &d, int32_t i, bool active, int lane)
{
    const int j = lane & 15, base = lane & 48;
    auto bits = [&](bool v) { return (uint32_t)(__ballot(v) >> base) & 0xffffu; };
    int32_t b = 0, e = 0;
    if (active) {
        b = d.offsets[i];
        e = d.offsets[i + 1];
    }
    const bool span = b >= 0 && e > b;
    const int32_t len = span ? e - b : 1;
    int32_t c = 0;
    if (span) c = d.colidx[b + min(j, len - 1)];
    const int32_t c0 = (int32_t)row_first((uint32_t)c);
    bool bad = c < 0 || c >= d.cols;
    uint32_t differ = bits(span && c != c0);
    int32_t run = differ ? (int32_t)__builtin_ctz(differ) - 1 : len - 1;
    for (int32_t r = 16; __ballot(span && r < len) != 0; r += 16) {
        const int32_t x = span && r + j < len ? d.colidx[b + r + j] : c0;
        bad |= x < 0 || x >= d.cols;
        const uint32_t df = bits(span && x != c0);
        if (!differ && df) run = r + (int32_t)__builtin_ctz(df) - 1;
        differ |= df;
    }
    PairPrep p;
    p.ok = span && bits(bad) == 0;
    const int32_t k = p.ok ? len - run : 0, bb = b + run;
    // (past a leading run the window's columns are read again)
    if (p.ok && run > 0) c = d.colidx[bb + min(j, k - 1)];
    const uint32_t cols = (uint32_t)d.cols, a = (uint32_t)c, n = row_next(a);
    uint32_t f = pair_offset(cols, a, n), r = pair_offset(cols, n, a);
    const uint32_t f0 = row_first(f), r0 = row_first(r);
    if (a == n) {
        f = f0;
        r = r0;
    }
    const uint32_t extra = j == 0 ? kHeadValid | (k > 8 ? kHeadLonger : 0u) : ((uint32_t)k >> (6 * (j - 1) & 31)) & 63u;
    p.word = j < 7 ? min(f, r) | (f > r ? 0x80000000u : 0u) | extra : (uint32_t)bb;
    p.desc = max(f, r);
    if (!p.ok) p.word = p.desc = 0;
    return p;
}

// The header and the outputs' initialisation.
__device__ __forceinline__ void prep_pairs_store(const ReqDesc &d, int32_t i, const PairPrep &p,
                                                 IndHead *__restrict__ heads, int lane)
{
    const int j = lane & 15;
    if (j < 8) {
        uint32_t *h = reinterpret_cast<uint32_t *>(heads + d.head_base) + 8 * (int64_t)i + j;
        h[0] = p.word;
        h[8 * (int64_t)d.n] = p.desc;
    }
    if (j == 0) {
        d.matched[i] = p.ok ? 0 : kInvalid;
        if (d.negative) d.negative[i] = p.ok ? 0 : kInvalid;
    }
}

}  // namespace ebic
