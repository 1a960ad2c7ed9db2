// Which launches a state scan takes, from its sizes alone (host code; no GPU types, so that the
// rules can be compiled and checked without one).
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace mesa {

constexpr int kComputeUnits = 256;

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Segments of the wide scan for bh sequences of n_chunks chunks: doubled while the
// (sequence, part, segment) workgroups still fit the compute units once (the kernel's
// LDS allows one workgroup per unit) and each segment keeps at least kMinSegChunks
// chunks, so the extra totals launch stays small next to the walk it shortens.
constexpr int kMinSegChunks = 8;
inline int wide_segments(int64_t bh, int n_chunks)
{
    int S = 1;
    while (2 * bh * (2 * S) <= kComputeUnits && n_chunks / (2 * S) >= kMinSegChunks) S *= 2;
    return S;
}

// Bytes of `slots` segment totals a sequence (elems floats each) and one decay per segment.
inline size_t segment_bytes(int64_t bh, int slots, int segments, int64_t elems)
{
    return size_t(bh * slots * elems + bh * segments) * sizeof(float);
}

// Chunks per segment of a states-only scan, whose segments all run side by side in one launch
// (no second walk: their totals are the result but for the combination); n_chunks = one
// segment.  Segments shorten the walk while their workgroups find room on the chip (LDS holds
// one a compute unit at d_k = 128, two or three at 64, which together take four fifths of
// their times one after the other); from there on they only add totals, which the
// combination reads back from memory and whose bytes are what limits many sequences.  In ns,
// fitted to every plan of 187 shapes (1 to 300 sequences, 4 to 1000 chunks, the four pairs of
// widths; the plan taken is within 14% of the fastest and 5% of one segment), us at d 128: 200
// sequences of 32 chunks 104 in one segment, 277 in 16; 130 of 64 196 in one, 150 in 3, 369 in
// 32; 48 of 10 20.7 in one, 22.6 in 2; 4 of 14 25.6 in one, 12.5 in 7.  A segment has at least
// two chunks, and its total and decay fit the scratch.
constexpr int kMaxFinalSegments = 128;
inline int64_t final_cost_ns(int64_t bh, int n_chunks, int d_k, int d_v, int len)
{
    const int64_t S = ceil_div(n_chunks, len), elems = int64_t(d_k) * (d_k + d_v), step = 600 + elems * 132 / 4096;
    const int share = d_k == 128 ? 1 : d_v == 128 ? 2 : 3;  // workgroups a compute unit holds
    const int64_t each = ceil_div(2 * bh * S, kComputeUnits);
    const int64_t walk = len * step * (4 * each + ceil_div(each, share)) / 5;
    return S == 1 ? walk : walk + 3600 + 340 * S + bh * S * elems * 4 / 3100;
}
inline int final_segment_len(int64_t bh, int n_chunks, int d_k, int d_v, size_t scratch_bytes)
{
    int best = n_chunks;
    int64_t cost = final_cost_ns(bh, n_chunks, d_k, d_v, best);
    for (int want = 2; want <= kMaxFinalSegments && n_chunks / want >= 2; ++want) {
        const int len = int(ceil_div(n_chunks, want)), S = int(ceil_div(n_chunks, len));
        if (segment_bytes(bh, S, S, int64_t(d_k) * (d_k + d_v)) > scratch_bytes) break;  // S does not fall from here on
        const int64_t c = final_cost_ns(bh, n_chunks, d_k, d_v, len);
        if (c < cost) {
            cost = c;
            best = len;
        }
    }
    return best;
}

// The chunk states of few, short sequences from the chunks' own totals, side by side in one
// launch, and one scan over them, instead of the walk (in `segments` of len chunks each).  The
// walk is a chain of chunk steps that leaves most of the chip idle (its segments too: they keep
// at least kMinSegChunks chunks and run twice); the totals are rounds of one step each, but move
// the states twice more, and the scan is a chain of its own.  Both cost more once the states
// outgrow the last-level cache (~150 MB written).  In ns, for the walks of split products and of
// the single one, whose steps are shorter; fitted to both forms at 999 shapes of each (1 to 128
// sequences, 2 to 1000 chunks, to 537 MB of states) and to 303 of the backward's, where the form
// taken is within 12% of the faster one.  us of the state
// pass, walk / scan, d 128 unless given:
//   split: 4 of 32 38.2 / 33.6, 24 of 20 45.3 / 42.6, 2 of 8 19.4 / 12.3;
//     not 64 of 13 31.9 / 64.3, 8 of 128 53.7 / 104, 16 of 256 (537 MB) 187 / 456
//   single: 2 of 32 d 64 18.5 / 12.7, 1 of 109 d 128 x 64 44.0 / 32.5, 2 of 64 33.2 / 26.8;
//     not 16 of 13 21.6 / 29.2, 12 of 13 21.2 / 26.1, 128 of 32 (537 MB) 83 / 327
constexpr int kScanChunks = 1024;  // longest sequence scanned (its decays are kept in LDS)
constexpr int64_t kCacheBytes = 150000000;
inline int64_t bytes_beyond_cache(int64_t bytes) { return bytes > kCacheBytes ? bytes - kCacheBytes : 0; }
inline bool wide_takes_scan(bool single, int64_t bh, int n_chunks, int64_t elems, int segments, int len)
{
    if (n_chunks < 2 || n_chunks > kScanChunks) return false;
    const int64_t e = elems / 4096, S = segments, nc = n_chunks;
    const int64_t units = ceil_div(2 * bh * S, kComputeUnits), rounds = ceil_div(2 * bh * (nc - 1), kComputeUnits);
    const int64_t bytes = bh * nc * elems * 4, over = bytes_beyond_cache(bytes);
    if (single) {
        const int64_t step = 489 + 104 * e;
        return 4700 + 138 * nc + rounds * step * 82 / 100 + bytes / 2390 + over / 7350 <
               units * (S > 1 ? 2 * len * step + 2860 + 66 * S * e : nc * step) + over / 11850;
    }
    const int64_t step = 615 + 189 * e;
    return 3500 + nc * (441 + 3 * e) + rounds * step * 9 / 10 + bytes / 2675 + over / 3340 <
           units * (S > 1 ? 2 * len * step + 1500 + 89 * S * e : nc * step) + over / 7900;
}

// The same choice for fp32 states (chunk 64): `each` workgroups walk side by side on a compute
// unit, a step of 0.79 us and half a microsecond for every further one.  Fitted to both forms at
// 999 shapes (to 537 MB) and to 303 of the backward's, where the form taken is within 15% of the
// faster one, the scan never more than 8% the slower; us of the state pass, walk / scan, d 64
// unless given: 8 of 13 14.4 / 10.8, 8 of 13 d 64 x 128 14.5 / 12.1, 2 of 256 221 / 54, 24 of 32
// d 64 x 128 (two a unit) 48.7 / 41.4, 8 of 1000 (262 MB) 865 / 478; not 2 of 8 9.7 / 10.8, 32 of
// 32 31.8 / 36.6, 16 of 64 d 128 (134 MB) 96 / 133, 24 of 256 (201 MB) 229 / 259.
inline bool f32_takes_scan(int64_t bh, int n_chunks, int d_k, int d_v)
{
    if (n_chunks < 2 || n_chunks > kScanChunks) return false;
    const int64_t nc = n_chunks, blocks = bh * ((d_k + d_v) / 16) * (d_k / 64), each = ceil_div(blocks, kComputeUnits);
    const int64_t bytes = bh * nc * d_k * (d_k + d_v) * 4, over = bytes_beyond_cache(bytes);
    return 5270 + 110 * nc + blocks * (nc - 1) * 184 / 100 + bytes / 3742 + over / 1462 <
           nc * (788 + 508 * (each - 1)) + over / 5384;
}

}  // namespace mesa
