// edt_bracket.h -- exact strided pass over long lines by bracketing each
// element's nearest row (paper, Section 2.3.2: one exact 1-D minimisation
// per line), for the first strided pass: the field is the distance d(r) of
// each row's element to the nearest site of its row, f(r) = d(r)^2.
//
//     euclidean   g(q) = min over r of  f(r) + (q - r)^2
//     chessboard  g(q) = min over r of  max(d(r), |q - r|)
//
// In both, once a row r' > r is at least as good as r for some q it stays so
// for every later q (total monotonicity), so with row ra a minimiser for row
// a and rb one for row b > a, every row between a and b has its first
// minimiser in [ra, rb] (euclidean: rows outside are strictly worse there).
// A search outward from each element costs one step per unit of its distance
// (8 x 1024^2 discs: 85 rows a side on average, 280 VALU instructions per
// element); the brackets of the segments of a line add up to the line once, a
// mean of S + 1 rows per S elements whatever the distances.
//
// A workgroup owns 16 adjacent lines, staged whole in LDS as 16-bit d
// (kBkNone: no site in the row), [row][line], rows 9 words apart: a wave
// takes 16 lines x 4 segments of S = 8 rows, and segments 8 rows apart then
// start on different banks.  Phases:
//   1. near search (distance passes): patches of 16 rows by the windowed search
//      in packed 16-bit arithmetic, which is the cheaper one up to about 48
//      rows; patches with farther elements are left over, and the workgroup
//      ends here when none is; when few are, they are searched on (to 249 rows);
//   2. top anchors, one row in 64, searched outward by 8 lanes per line pair;
//   3. anchors halfway, three levels down to one row in 8: the bracket between
//      the two known neighbours, of which only the blocks of 8 rows are walked
//      whose smallest d could improve on the best value so far;
//   4. segments: the lane holds its 8 rows' best values in registers and walks
//      the bracket between its anchors; a row's 8 candidates are one addition
//      each (f + t^2 + 2 t s, t = q0 - r, s^2 added at the end).  The 8 rows
//      at either end of the bracket are walked in full; between them (brackets
//      that jump from one object's rows to another's) a block of 8 rows is
//      walked only when its smallest d could improve some row of the lane.
//
// Bound by VALU issue (147 instructions per element, 60 % of the issue time) and
// the spread of work over the workgroups (two per compute unit for 8 x 1024^2,
// all at once): column pass of 8 x 1024^2 discs, windowed and ordered against
// bracketed, 83 -> 52 us, chessboard 71 -> 46 us, one background pixel 31 -> 15 us;
// index pass of 16 x 375 x 500 516 -> 39 us (43 % of the issue time).  Segments of
// 12 or 16 rows (larger walks, spills) and a top anchor per 4 or 16 segments
// measured the same or slower.
// Walking a row outside a lane's bracket is harmless (it is a candidate like
// any other), so lanes of a wave need no masks.
// Workgroups of which at most kBkDirect rows hold a site take the minimum
// over those rows directly.
//
// MODE kBkIndex (2-D, final): the field is the index carrier; the staged
// value is 2 |c - x| + (c < x) for site column c, and the winner's row and
// value give the coordinates back.  Minimisers are the canonical ones
// (smallest row): an anchor's row is the last of its segment, so that any of
// its minimisers bounds the first minimisers of the rows up to it and after
// it.  KEY: value and row in one 32-bit key (an addition and a minimum per
// candidate); otherwise compare and select.
#pragma once

#include "edt_fh.h"

namespace tmedt {

constexpr int kBkLines = 16;                 // lines per workgroup
constexpr int kBkPitch = 18;                 // row pitch in 16-bit values (16 + 2: bank skew)
constexpr int kBkSeg = 8;                    // rows per segment
constexpr int kBkG = 8;                      // guard rows of "no site" per side
constexpr uint32_t kBkNone = 16384;          // d of a row without sites
constexpr uint32_t kBkMaxD = 16000;          // largest row extent
constexpr uint32_t kBkMaxN = 2048;           // longest line
constexpr int kBkDirect = 32;                // at most this many site rows: direct minimum

constexpr int kTop = 8;                      // segments per top anchor
constexpr int kBkRoots = 512;
constexpr int kBkNear = 16;                  // rows of a near-search patch
constexpr int kBkReach = 49;                 // distances the near search settles
constexpr int kBkFewReach = 249;             // the same where few patches are farther

enum BkMode : int { kBkField = 0, kBkDist = 1, kBkIndex = 2 };

struct BracketArgs {
    int32_t *buf;          // field: packed rows (PK), or int32 d (kInfI: none); kBkIndex: the carrier
    float *dist;           // kBkDist / kBkIndex outputs (each may be null)
    int32_t *sq;
    uint32_t lines;        // lines of this pass
    uint32_t n;            // line length
    uint32_t inner;        // element stride of the line
    Div32 div_inner;
    uint32_t vox;          // elements per sample (kBkIndex)
    uint64_t cstride;      // kBkIndex: carrier elements per sample
    int32_t coords;        // kBkIndex: write the coordinate slices at buf
    uint32_t kbits;        // KEY: bits of the row in a key
    uint32_t fcap;         // KEY: value of rows without sites
};

__host__ __device__ constexpr uint32_t bk_segs(uint32_t n, int s) { return (n + uint32_t(s) - 1) / uint32_t(s); }
// tile with guard rows, anchors' rows, block minima
__host__ __device__ constexpr size_t bk_lds(uint32_t n, int s) {
    return (size_t(n + 2 * kBkG) * kBkPitch + size_t(bk_segs(n, s)) * kBkLines + size_t((n + 7) / 8) * kBkLines + 1) / 2 * 4;
}

// METRIC kL2 or kLinf.  PK: rows packed to 16 bits in strips of 16 columns
// (k_scan_word<..., 16>).  S: rows per segment.
template <int METRIC, int MODE, bool PK, bool KEY, int S>
__global__ void __launch_bounds__(1024, 8) k_line_bracket(BracketArgs a) {
    static_assert(!KEY || MODE == kBkIndex, "keys carry the row of an index pass");
    static_assert(MODE != kBkIndex || (METRIC == kL2 && !PK), "index passes: euclidean, int32 carrier");
    constexpr int SH = MODE == kBkIndex ? 1 : 0;     // staged value = d << SH | sign
    extern __shared__ __attribute__((aligned(16))) uint16_t bk_tile[];
    __shared__ uint32_t claim, claim_near, claim_few, site_rows, far_count, far_left;
    __shared__ uint32_t has_site[kBkLines];
    __shared__ uint64_t line_base[kBkLines];               // row 0 of each line
    __shared__ uint8_t far[kBkMaxN / kBkNear];             // patches the near search left over
    __shared__ float root[kBkRoots];                       // square roots of 0 .. kBkRoots - 1
    __shared__ uint16_t site_row[kBkDirect];
    const int t = threadIdx.x;
    const int lane = t & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(t / kWave);
    const int nthreads = int(blockDim.x), nwaves = nthreads / kWave;
    const int n = int(a.n);
    const int ns = int(bk_segs(a.n, S)), nb = (n + 7) / 8;
    uint16_t *const row0 = bk_tile + kBkG * kBkPitch;
    uint16_t *const arg = bk_tile + (n + 2 * kBkG) * kBkPitch;     // [segment][line]: a minimiser of its last row
    uint16_t *const bmin = arg + ns * kBkLines;                    // [block of 8 rows][line]: smallest staged value

    // Two consecutive groups of 16 lines share each 128-byte line of a row:
    // they go to the workgroups b and b + 8, which the dispatcher sends to one
    // XCD (one L2).
    uint32_t g = blockIdx.x;
    if (g < (gridDim.x & ~15u)) {
        const uint32_t x = g & 7u, i = g >> 3;
        g = (i >> 1) * 16u + x * 2u + (i & 1u);
    }
    const int j = t & (kBkLines - 1);
    const uint32_t L0 = g * uint32_t(kBkLines), L = L0 + uint32_t(j);
    const bool live = L < a.lines;
    const uint32_t o = a.div_inner.div(live ? L : L0);
    const uint32_t i = (live ? L : L0) - o * a.inner;
    const uint64_t base = uint64_t(o) * a.n * a.inner + i;         // row 0 of this lane's line
    const int32_t *const src = MODE == kBkIndex ? a.buf + uint64_t(o) * a.cstride + i : a.buf + base;

    // ---- staging ---------------------------------------------------------------
    if (t == 0) {
        claim = 0;
        claim_near = 0;
        claim_few = 0;
        far_left = 0;
        site_rows = 0;
        far_count = 0;
    }
    if (t < kBkLines) {
        has_site[t] = 0;
        line_base[t] = base;
    }
    if (MODE == kBkDist && METRIC == kL2)
        for (int k = t; k < kBkRoots; k += nthreads) root[k] = sqrt_rn_int(uint32_t(k));
    constexpr uint16_t kNoneV = uint16_t(kBkNone << SH);
    for (int k = t; k < kBkG * kBkPitch; k += nthreads) {
        bk_tile[k] = kNoneV;
        row0[n * kBkPitch + k] = kNoneV;
    }
    __syncthreads();
    if constexpr (PK) {
        // thread t: half t & 1 (8 lines) of rows t / 2, t / 2 + nthreads / 2, ...
        const int h = t & 1;
        const uint64_t strip = base - uint32_t(j);
        uint32_t seen[4] = {0, 0, 0, 0};                  // per pair of lines: 16-bit flags
        for (int r = t >> 1; r < n; r += nthreads / 2) {
            const int4 p = *reinterpret_cast<const int4 *>(a.buf + strip + uint64_t(r >> 1) * a.inner + 8 * (r & 1) + 4 * h);
            const uint32_t pw[4] = {uint32_t(p.x), uint32_t(p.y), uint32_t(p.z), uint32_t(p.w)};
            uint32_t *dst = reinterpret_cast<uint32_t *>(row0 + r * kBkPitch) + 4 * h;
            bool any = false;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const u16x2 v = __builtin_elementwise_min(as_pair(pw[k]), splat(int(kBkNone)));
                const u16x2 s = __builtin_elementwise_sub_sat(splat(int(kBkNone)), v);   // nonzero: site
                dst[k] = as_word(v);
                seen[k] |= as_word(s);
                any = any || as_word(s) != 0u;
            }
            // (both halves of a row hold a site or none does: it lies in one image row)
            const bool row_any = any || __shfl_xor(int(any), 1) != 0;
            if (row_any && h == 0) {
                const uint32_t k = atomicAdd(&site_rows, 1u);
                if (k < uint32_t(kBkDirect)) site_row[k] = uint16_t(r);
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (seen[k] & 0xffffu) has_site[8 * h + 2 * k] = 1;
            if (seen[k] >> 16) has_site[8 * h + 2 * k + 1] = 1;
        }
    } else {
        constexpr int SB = 8;                             // rows in flight per lane
        const int step = nthreads / kBkLines;
        bool seen = false;
        for (int r0 = t / kBkLines; r0 < n; r0 += step * SB) {
            int32_t v[SB];
#pragma unroll
            for (int s = 0; s < SB; ++s) v[s] = src[uint64_t(min(r0 + s * step, n - 1)) * a.inner];
#pragma unroll
            for (int s = 0; s < SB; ++s) {
                const int r = r0 + s * step;
                uint32_t e;
                if (MODE == kBkIndex) {
                    const int d = v[s] - (r * int(a.inner) + int(i));      // site column - own column
                    e = v[s] >= 0 ? (uint32_t(abs(d)) << 1) | (d < 0 ? 1u : 0u) : uint32_t(kNoneV);
                } else {
                    e = min(uint32_t(v[s]), kBkNone);
                }
                if (!live) e = kNoneV;
                const bool site = r < n && e < uint32_t(kNoneV);
                if (r < n) row0[r * kBkPitch + j] = uint16_t(e);
                seen |= site;
                const uint64_t b = __ballot(site) >> (lane & ~(kBkLines - 1));
                if (j == 0 && (b & 0xffffu)) {
                    const uint32_t k = atomicAdd(&site_rows, 1u);
                    if (k < uint32_t(kBkDirect)) site_row[k] = uint16_t(r);
                }
            }
        }
        if (seen) has_site[j] = 1;
    }
    __syncthreads();
    const bool has = live && has_site[j] != 0u;
    const uint32_t nsites = site_rows;

    auto value = [&](uint32_t v) -> uint32_t {           // f of a staged value (d for the chessboard)
        const uint32_t d = v >> SH;
        if (METRIC == kLinf) return d;
        if (KEY) return min(d * d, a.fcap);
        return __umul24(d, d);
    };
    // element (row q, this lane's line, batch-flat e): value c at row r (ignored without sites)
    auto emit = [&](int q, uint64_t e, uint32_t c, int r) {
        if constexpr (METRIC == kLinf) {
            a.buf[e] = has ? int32_t(c) : (MODE == kBkField ? kInfI : -1);
        } else if constexpr (MODE == kBkField) {
            a.buf[e] = has ? int32_t(c) : kInfI;
        } else {
            // without background: the virtual element (-1, 0)
            const uint32_t d2 = has ? c : uint32_t(q + 1) * uint32_t(q + 1) + i * i;
            if (MODE == kBkIndex && a.coords) {
                const uint32_t v = row0[r * kBkPitch + j];
                const int dx = (v & 1u) ? -int(v >> 1) : int(v >> 1);
                int32_t *s0 = a.buf + e + uint64_t(o) * (a.cstride - a.vox);
                s0[0] = has ? r : -1;
                s0[a.vox] = has ? int(i) + dx : 0;
            }
            if (a.dist) a.dist[e] = d2 < (1u << 24) ? sqrt_rn_int(d2) : float(sqrt(double(d2)));
            if (a.sq) a.sq[e] = int32_t(d2);
        }
    };

    if (nsites <= uint32_t(kBkDirect)) {
        // few site rows: the minimum over them, for every element
        for (int q = t / kBkLines; q < n; q += nthreads / kBkLines) {
            uint32_t best = 0xffffffffu;
            int br = 0;
            for (uint32_t k = 0; k < nsites; ++k) {
                const int r = site_row[k];
                const uint32_t dq = uint32_t(abs(q - r));
                const uint32_t v = row0[r * kBkPitch + j], f = (v >> SH) * (v >> SH);
                const uint32_t c = METRIC == kLinf ? max(v, dq) : f + dq * dq;
                if (MODE == kBkIndex) br = c < best || (c == best && r < br) ? r : br;
                best = min(best, c);
            }
            if (live) emit(q, base + uint64_t(q) * a.inner, best, br);
        }
        return;
    }

    // The next number of a counter in LDS, for the whole wave.  The barrier (no
    // instruction) keeps the compiler from threading an earlier test of the lane
    // into this one, which would leave the other lanes looping on their own.
    auto next = [&](uint32_t *counter) {
        __builtin_amdgcn_wave_barrier();
        uint32_t k = 0;
        if (lane == 0) k = atomicAdd(counter, 1u);
        return int(__builtin_amdgcn_readfirstlane(k));
    };

    // ---- near search ---------------------------------------------------------------
    // Elements within kBkReach of a site, patch by patch (16 rows x 16 lines):
    // the windowed search in packed 16-bit arithmetic, two lines per word and two
    // adjacent rows per lane, rows q - d and q + d at once.  A patch of which
    // some element is farther is left over; it is given up early when its values
    // after 8 steps say so.
    if constexpr (MODE != kBkIndex) {
        constexpr int kRowWords = kBkPitch / 2;
        const int jw = lane & 7, rho = lane >> 3;
        const uint32_t *const col = reinterpret_cast<const uint32_t *>(row0) + jw;
        const u16x2 on = {uint16_t(L0 + 2 * jw < a.lines ? 0xffff : 0), uint16_t(L0 + 2 * jw + 1 < a.lines ? 0xffff : 0)};
        const int nnear = (n + kBkNear - 1) / kBkNear, nq = (nnear + 3) / 4;
        // Patch p with steps up to kBkReach (FEW: kBkFewReach): true and its
        // elements written, or false if one is farther.  Euclidean values past
        // the reach only have to stay past its square: 250^2 + kBkReach^2 fits
        // 16 bits (one multiply-add per step), FEW saturates.
        static_assert(250 * 250 + (kBkReach + 4) * (kBkReach + 4) < 65536 && 255 * 255 >= kBkFewReach * kBkFewReach &&
                          (kBkFewReach + 4) * (kBkFewReach + 4) < 65536,
                      "near search: 16-bit values");
        auto past = [](u16x2 m, int r) {                   // some value past distance r
            return as_word(__builtin_elementwise_sub_sat(m, splat(METRIC == kLinf ? r : r * r))) != 0;
        };
        auto settle = [&](int p, auto few) -> bool {
            constexpr bool FEW = decltype(few)::value;
            constexpr int reach = FEW ? kBkFewReach : kBkReach;
            auto val = [](u16x2 e, int d) -> u16x2 {
                if (METRIC == kLinf) return __builtin_elementwise_max(e, splat(d));
                const u16x2 c = __builtin_elementwise_min(e, splat(FEW ? 255 : 250));
                return FEW ? __builtin_elementwise_add_sat(c * c, splat(d * d)) : c * c + splat(d * d);
            };
            const int q = kBkNear * p + 2 * rho, qc = min(q, n);      // (row n: guard)
            u16x2 bA = val(as_pair(col[qc * kRowWords]), 0) & on;
            u16x2 bB = val(as_pair(col[(qc + 1) * kRowWords]), 0) & on;
            if (q >= n) bA = splat(0);
            if (q + 1 >= n) bB = splat(0);
#pragma unroll 1
            for (int d = 1; d < reach; d += 4) {
                const u16x2 m = __builtin_elementwise_max(bA, bB);
                if (!__any(past(m, d))) break;
                if (!FEW && d % 8 == 1 && d > 1 && __any(past(m, reach - 1))) return false;
                const uint32_t *pl = col + max(qc - d - 3, -kBkG) * kRowWords;
                const uint32_t *ph = col + min(qc + d, n + kBkG - 5) * kRowWords;
                u16x2 U[5], W[5];
#pragma unroll
                for (int k = 0; k < 5; ++k) {
                    U[k] = as_pair(pl[k * kRowWords]);         // rows q-d-3 .. q-d+1
                    W[k] = as_pair(ph[k * kRowWords]);         // rows q+d .. q+d+4
                }
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    bA = __builtin_elementwise_min(bA, val(__builtin_elementwise_min(U[3 - s], W[s]), d + s));
                    bB = __builtin_elementwise_min(bB, val(__builtin_elementwise_min(U[4 - s], W[s + 1]), d + s));
                }
            }
            if (__any(past(__builtin_elementwise_max(bA, bB), reach))) return false;
            const uint32_t h[4] = {bA.x, bA.y, bB.x, bB.y};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int qq = q + (k >> 1), l = 2 * jw + (k & 1);
                if (qq >= n || L0 + uint32_t(l) >= a.lines) continue;
                const uint64_t e = line_base[l] + uint64_t(qq) * a.inner;
                if (METRIC == kLinf || MODE == kBkField) {
                    a.buf[e] = int32_t(h[k]);
                } else {
                    if (a.dist) a.dist[e] = h[k] < uint32_t(kBkRoots) ? root[h[k]] : sqrt_rn_int(h[k]);
                    if (a.sq) a.sq[e] = int32_t(h[k]);
                }
            }
            return true;
        };
        for (int k = next(&claim_near); k < 4 * nq; k = next(&claim_near)) {
            // four runs of rows in turn, so that the first patches sample the lines
            const int p = (k & 3) * nq + (k >> 2);
            if (p >= nnear) continue;
            const int nfar = int(__builtin_amdgcn_readfirstlane(
                __hip_atomic_load(&far_count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)));
            // most patches so far were left over: this one is not tried
            const bool left = (nfar >= 4 && 2 * nfar > k) || !settle(p, std::false_type{});
            far[p] = left ? 1 : 0;
            if (left && lane == 0) atomicAdd(&far_count, 1u);
        }
        __syncthreads();
        const int nfar = int(far_count);
        if (nfar == 0) return;
        // A few patches left over (corners and gaps of a sparse background) are
        // searched on: the brackets' phases are a chain whose length hardly
        // depends on how many patches need them (1 % background: 8 x 1024^2 40
        // -> 34 us per call, 9 x 900 x 800 48 -> 39 us, chessboard 37 -> 31 and 45
        // -> 35 us; a limit of 1/2 instead of 1/4 loses 8 us on 8 x 1024^2 discs).
        if (4 * nfar <= nnear) {
            for (int p = next(&claim_few); p < nnear; p = next(&claim_few)) {
                if (!__builtin_amdgcn_readfirstlane(int(far[p]))) continue;
                const bool left = !settle(p, std::true_type{});
                far[p] = left ? 1 : 0;
                if (left && lane == 0) far_left = 1;
            }
            __syncthreads();
            if (far_left == 0) return;
        }
    }

    // ---- block minima and anchors ------------------------------------------------
    for (int k = t; k < nb * kBkLines; k += nthreads) {
        const uint16_t *p = row0 + (k / kBkLines) * 8 * kBkPitch + j;
        uint32_t m = p[0];
#pragma unroll
        for (int s = 1; s < 8; ++s) m = min(m, uint32_t(p[s * kBkPitch]));
        bmin[k] = uint16_t(m);
    }
    auto cand = [](uint32_t d, int k) -> uint32_t {            // d of a row, k rows away
        return METRIC == kLinf ? max(d, uint32_t(abs(k))) : __umul24(d, d) + uint32_t(__mul24(k, k));
    };
    // Top anchors, one per kTop segments: a wave takes 8 pairs of lines of one
    // anchor, lane (pair, part); part p searches the blocks of 8 steps p, p + 8,
    // ... outward, and the parts share their best values after each round.
    // Candidates are at most 2^28 + n^2, so value << 3 | step fits 32 bits.
    {
        constexpr int kPairs = kBkLines / 2, kRowWords = kBkPitch / 2;
        const int jp = lane & (kPairs - 1), part = lane / kPairs;
        const uint32_t *const col = reinterpret_cast<const uint32_t *>(row0) + jp;
        const bool h0 = has_site[2 * jp] != 0u, h1 = has_site[2 * jp + 1] != 0u;
        auto dpair = [](uint32_t w) { return SH ? as_pair(w) >> u16x2{1, 1} : as_pair(w); };
        for (int p = wv; kTop * p + kTop - 1 < ns; p += nwaves) {
            const int seg = kTop * p + kTop - 1;
            const int q = min(S * seg + S - 1, n - 1);
            const u16x2 own = dpair(col[q * kRowWords]);
            // best over this lane's blocks, and over all parts
            uint32_t b0 = h0 ? cand(own.x, 0) << 3 : 0u, b1 = h1 ? cand(own.y, 0) << 3 : 0u;
            int d0 = 0, d1 = 0;
            uint32_t s0 = b0, s1 = b1;
            for (int dr = 1; dr <= n; dr += 64) {
                if (__all(max(s0, s1) <= (cand(0, dr) << 3))) break;
                const int d = dr + 8 * part;
                const uint32_t *pl = col + max(q - d - 7, -kBkG) * kRowWords;
                const uint32_t *ph = col + min(q + d, n + kBkG - 8) * kRowWords;
                uint32_t u[8], w[8], m0 = 0xffffffffu, m1 = 0xffffffffu;
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    u[s] = pl[(7 - s) * kRowWords];
                    w[s] = ph[s * kRowWords];
                }
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    const u16x2 e = dpair(as_word(__builtin_elementwise_min(as_pair(u[s]), as_pair(w[s]))));
                    m0 = min(m0, (cand(e.x, d + s) << 3) | uint32_t(s));
                    m1 = min(m1, (cand(e.y, d + s) << 3) | uint32_t(s));
                }
                d0 = m0 < b0 ? d : d0;
                d1 = m1 < b1 ? d : d1;
                b0 = min(b0, m0);
                b1 = min(b1, m1);
                s0 = b0;
                s1 = b1;
#pragma unroll
                for (int x = kPairs; x < kWave; x <<= 1) {
                    s0 = min(s0, uint32_t(__shfl_xor(int(s0), x)));
                    s1 = min(s1, uint32_t(__shfl_xor(int(s1), x)));
                }
            }
            // the side of the best step (0: the row itself); a part with the
            // smallest value writes (any minimiser will do)
            const int e0 = d0 > 0 ? d0 + int(b0 & 7u) : 0, e1 = d1 > 0 ? d1 + int(b1 & 7u) : 0;
            const uint32_t v0 = dpair(col[max(q - e0, -1) * kRowWords]).x, v1 = dpair(col[max(q - e1, -1) * kRowWords]).y;
            const int r0 = cand(v0, e0) == (b0 >> 3) ? q - e0 : q + e0;
            const int r1 = cand(v1, e1) == (b1 >> 3) ? q - e1 : q + e1;
            if (b0 == s0) arg[seg * kBkLines + 2 * jp] = h0 ? uint16_t(r0) : uint16_t(0);
            if (b1 == s1) arg[seg * kBkLines + 2 * jp + 1] = h1 ? uint16_t(r1) : uint16_t(0);
        }
    }
    const int sub = lane / kBkLines;
    // Anchors halfway between those known, until every segment has one: the
    // rows of the bracket within the best value's reach, in runs of 4 blocks of
    // 8 rows of which those are walked whose smallest d could improve on it.
    // h parts (lanes of a line 16 apart) share an anchor's runs, so that every
    // level keeps the same number of waves busy.
    // key: value << 3 | row & 7, beside the row's block
#pragma unroll 1
    for (int h = kTop / 2; h >= 1; h >>= 1) {
        __syncthreads();                                   // (also: block minima)
        const int cnt = (ns + h) / (2 * h);                // segments h - 1 + 2 h k below ns
        const int hp = min(h, 4), per = 4 / hp, part = sub & (hp - 1);       // anchors per wave, part of this lane
        for (int p = wv; per * p < cnt; p += nwaves) {
            const int k = min(per * p + sub / hp, cnt - 1);
            const int seg = h - 1 + 2 * h * k;
            const int q = min(S * seg + S - 1, n - 1);
            int lo = seg - h >= 0 ? arg[(seg - h) * kBkLines + j] : 0;
            int hi = seg + h < ns ? arg[(seg + h) * kBkLines + j] : n - 1;
            if (METRIC == kLinf) {
                const int x = min(lo, hi);
                hi = max(lo, hi);
                lo = x;
            }
            auto key = [&](int r) { return (cand(row0[r * kBkPitch + j] >> SH, q - r) << 3) | uint32_t(r & 7); };
            const int mid = min(max(q, lo), hi);
            const uint32_t k0 = key(lo), k1 = key(hi), k2 = key(mid);
            uint32_t best = k0;
            int blk = lo >> 3;
            auto take = [&](uint32_t kk, int b) {
                blk = kk < best ? b : blk;
                best = min(best, kk);
            };
            take(k1, hi >> 3);
            take(k2, mid >> 3);
            // rows farther than the best value's root cannot improve on it
            const int reach = METRIC == kLinf ? int(min(best >> 3, 4096u))
                                              : int(__builtin_amdgcn_sqrtf(float(best >> 3))) + 1;
            int b = (max(lo, q - reach) >> 3) + 4 * part;
            int be = min(hi, q + reach) >> 3;
            if (!has) be = -1;
            for (; __any(b <= be); b += 4 * hp) {
                uint32_t low[4];
                bool any = false;
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int bc = min(b + x, nb - 1);
                    const int gap = max(max(8 * bc - q, q - (8 * bc + 7)), 0);
                    low[x] = cand(bmin[bc * kBkLines + j] >> SH, gap) << 3;
                    low[x] = b + x <= be ? low[x] : 0xffffffffu;
                    any = any || low[x] < (best & ~7u);
                }
                if (!__any(any)) continue;
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    if (!__any(low[x] < (best & ~7u))) continue;
                    const int bc = min(b + x, nb - 1);
                    uint32_t v[8], m = 0xffffffffu;
#pragma unroll
                    for (int s = 0; s < 8; ++s) v[s] = row0[(8 * bc + s) * kBkPitch + j];
#pragma unroll
                    for (int s = 0; s < 8; ++s)
                        m = min(m, (cand(v[s] >> SH, q - 8 * bc - s) << 3) | uint32_t(s));
                    take(m, bc);
                }
            }
            for (int x = 1; x < hp; x <<= 1) {
                const uint32_t kk = uint32_t(__shfl_xor(int(best), kBkLines * x));
                take(kk, __shfl_xor(blk, kBkLines * x));
            }
            if (part == 0 && per * p + sub / hp < cnt)
                arg[seg * kBkLines + j] = has ? uint16_t(8 * blk + int(best & 7u)) : uint16_t(0);
        }
    }
    __syncthreads();

    // ---- segments ------------------------------------------------------------------
    const int npatch = (ns + 3) / 4;                       // a wave's 16 lines x 4 segments
    for (int p = next(&claim); p < npatch; p = next(&claim)) {
        const int seg = min(4 * p + sub, ns - 1);
        const bool mine = 4 * p + sub < ns;
        if (MODE != kBkIndex) {
            const int f0 = 4 * S * p / kBkNear, f1 = min((4 * S * p + 4 * S - 1) / kBkNear, (n - 1) / kBkNear);
            bool any = false;
            for (int k = f0; k <= f1; ++k) any = any || far[k] != 0;
            if (!any) continue;
        }
        const int q0 = S * seg;
        int ra = seg > 0 ? arg[(seg - 1) * kBkLines + j] : 0;
        int rb = arg[seg * kBkLines + j];
        if (METRIC == kLinf) {
            const int lo = min(ra, rb);
            rb = max(ra, rb);
            ra = lo;
        }
        if (!has) ra = rb = 0;
        // best values less s^2 (euclidean; plus S^2 and shifted above the row in a key)
        uint32_t best[S];
        int arg_of[MODE == kBkIndex && !KEY ? S : 1];
#pragma unroll
        for (int s = 0; s < S; ++s) best[s] = KEY ? 0xffffffffu : 0x7fffffffu;
        if (MODE == kBkIndex && !KEY) {
#pragma unroll
            for (int s = 0; s < (KEY ? 1 : S); ++s) arg_of[MODE == kBkIndex && !KEY ? s : 0] = 0;
        }
        // rows r .. r + 7, in pairs; rows past `last` are left out once no lane
        // of the wave wants them (all of them may be walked)
        auto walk = [&](int r, int last) {
            uint32_t v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = row0[(r + k) * kBkPitch + j];
#pragma unroll
            for (int k2 = 0; k2 < 8; k2 += 2) {
                if (k2 > 0 && __all(r + k2 > last)) break;
#pragma unroll
                for (int k = k2; k < k2 + 2; ++k) {
                    const uint32_t f = value(v[k]);
                    const int tq = q0 - r - k;
                    if constexpr (METRIC == kLinf) {
#pragma unroll
                        for (int s = 0; s < S; ++s) best[s] = min(best[s], max(f, uint32_t(abs(tq + s))));
                    } else if constexpr (KEY) {
                        uint32_t c = ((f + uint32_t(__mul24(tq, tq)) + uint32_t(S * S)) << a.kbits) + uint32_t(r + k);
                        const uint32_t du = uint32_t(2 * tq) << a.kbits;
#pragma unroll
                        for (int s = 0; s < S; ++s) {
                            best[s] = min(best[s], c);
                            c += du;
                        }
                    } else {
                        int c = int(f) + __mul24(tq, tq);
#pragma unroll
                        for (int s = 0; s < S; ++s) {
                            if (MODE == kBkIndex)
                                arg_of[s] = c < int(best[s]) || (c == int(best[s]) && r + k < arg_of[s]) ? r + k : arg_of[s];
                            best[s] = uint32_t(min(int(best[s]), c));
                            c += 2 * tq;
                        }
                    }
                }
            }
        };
        auto result = [&](int s) -> uint32_t {
            if (METRIC == kLinf) return best[s];
            if (KEY) return (best[s] >> a.kbits) + uint32_t(s * s) - uint32_t(S * S);
            return best[s] + uint32_t(s * s);
        };
        // the first 8 rows of the bracket (guard rows beyond the line hold no site)
        walk(ra, rb);
        if (__any(ra + 8 <= rb)) {
            // the last 8 rows, then the blocks between the two ends
            const int re = min(max(rb - 7, ra + 8), n);
            walk(re, rb);
            int b = (ra + 8) >> 3;
            const int be = re > ra + 8 ? (re - 1) >> 3 : -1;      // last block holding a middle row
            if (__any(b <= be)) {
                auto worst = [&]() {
                    uint32_t m = 0;
#pragma unroll
                    for (int s = 0; s < S; ++s) m = max(m, result(s));
                    return m;
                };
                uint32_t bound = worst();
                for (; __any(b <= be); ++b) {
                    const int bc = min(b, nb - 1);
                    const uint32_t d = bmin[bc * kBkLines + j] >> SH;
                    const int gap = max(max(8 * bc - (q0 + S - 1), q0 - (8 * bc + 7)), 0);
                    const uint32_t low = METRIC == kLinf ? max(d, uint32_t(gap)) : __umul24(d, d) + uint32_t(__mul24(gap, gap));
                    // index: a block that only ties may hold the smaller row
                    const bool need = b <= be && has && (MODE == kBkIndex ? low <= bound : low < bound);
                    if (!__any(need)) continue;
                    walk(8 * bc, n);
                    bound = worst();
                }
            }
        }
        if (!(live && mine)) continue;
        uint64_t e = base + uint64_t(q0) * a.inner;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            if (q0 + s < n) {
                int r = 0;
                if (MODE == kBkIndex && has) r = KEY ? int(best[s] & ((1u << a.kbits) - 1u)) : arg_of[KEY ? 0 : s];
                emit(q0 + s, e, result(s), r);
            }
            e += a.inner;
        }
    }
}

}  // namespace tmedt
