// Brute-force distance transform (the paper's exactness check, Section
// 2.3.2): for every element, the nearest background element under the
// euclidean, taxicab or chessboard metric with optional per-axis sampling,
// by visiting every background element of the sample.
//
// A workgroup owns kBfOut consecutive elements of one sample.  It walks the
// sample's mask in chunks of PB bytes per thread: the chunk's background
// elements are compacted, in row-major order, into an LDS list of their
// coordinates (scaled by the sampling when sampled), and every thread runs
// the list against its elements, keeping the first strictly smaller value,
// so ties go to the smallest flat index.  The coordinate loop is unrolled
// for ranks 2 and 3 (other ranks loop over the rank).  Unit sampling is
// exact integer arithmetic; sampled values are float.
//
// Two things bounded it on sparse masks (8 x 256^2, 1 % background: 163 us): 64
// chunks of 1024 bytes per workgroup, each with ten background elements and three
// barriers, and 32-bit multiplies (a quarter of the rate of 24-bit ones).
// Chunks are now 4096 bytes for ranks 2 and 3 (3072 for many workgroups of the
// other forms), and unit euclidean transforms
// whose squared extents sum to at most 2^21 (KEY) take
//     d^2 - |x|^2 = |y|^2 - 2 x . y
// with the list's number below it in one 32-bit key: one 24-bit multiply-add per
// axis and half a minimum per pair of elements.  63 us (8 x 256^2; chunks of 2048
// bytes 87 us, two elements per thread 83 us).
#pragma once

#include "edt_common.h"

namespace tmedt {

constexpr int kBfThreads = 256;
constexpr int kBfPer = 4;                        // elements per thread
constexpr int kBfOut = kBfThreads * kBfPer;      // elements per workgroup
// Mask bytes per thread and chunk (and so list entries per chunk and thread):
// 16 for keys, and for ranks 2 and 3 while every workgroup runs at once (LDS holds
// three of rank 2 per compute unit, two of rank 3); else 12, which leaves room
// for five and three and loads four-byte words.  Sampled, us per call, with
// chunks of 1024 bytes, 16 and 12 per thread: 16 x 24 x 40 x 41, 624 workgroups,
// half background 2877, 3577, 2758, 1 % 108, 99, 75; 32 x 256^2, 2048 workgroups,
// half background 7863, 8222, 7858; 8 x 256^2, 512 workgroups, 1 % 129, 75, 80.
constexpr int kBfBytes = 16, kBfBytesMany = 12;
__host__ constexpr bool bf_many(int nd, uint64_t groups) { return groups > 256u * (nd == 2 ? 3u : 2u); }
constexpr int kBfKeyBits = 10;                   // KEY: bits of the number in a key
constexpr int kBfRun = 1 << kBfKeyBits;          // KEY: list entries between two merges
constexpr uint64_t kBfKeySum = uint64_t(1) << (31 - kBfKeyBits);   // KEY: most the squared extents sum to

struct BfArgs {
    const uint8_t *in;      // [batch][vox]
    float *dist;            // [batch][vox] or null
    int32_t *idx;           // [batch][ndim][vox] or null
    uint32_t vox;
    uint32_t bps;           // workgroups per sample
    int32_t ndim;
    Div32 div_shape[kMaxDim];
    float s[kMaxDim];       // sampling per axis (ones for unit)
    double sd[kMaxDim];     // the same in double (virtual element)
};

template <int METRIC, bool SAMP, int ND, bool KEY = false, int PB = (ND > 0) ? kBfBytes : 4>
__global__ void __launch_bounds__(kBfThreads) k_dt_bf(BfArgs a) {
    using V = typename std::conditional<SAMP, float, int32_t>::type;
    constexpr int MAXND = ND > 0 ? ND : kMaxDim;
    static_assert(!KEY || (METRIC == 0 && !SAMP && ND > 0), "keys: exact euclidean, rank 2 or 3");
    static_assert(PB % 4 == 0 && kBfThreads * PB <= 65536, "16-bit offsets within a chunk");
    constexpr int kBfChunk = kBfThreads * PB;
    __shared__ V zc[KEY ? 1 : kBfChunk][MAXND];   // background coordinates of the chunk
    // KEY: coordinates << kBfKeyBits and (sum of their squares << kBfKeyBits | number)
    __shared__ int4 zk[KEY ? kBfChunk + 4 : 1];
    __shared__ uint16_t zflat[KEY ? 1 : kBfChunk];   // their flat indices less the chunk's first
    __shared__ uint32_t wave_tot[kBfThreads / kWave];
    const int nd = ND > 0 ? ND : a.ndim;
    const int t = threadIdx.x;
    const int lane = t & (kWave - 1), wv = t / kWave;
    const uint32_t b = blockIdx.x / a.bps;          // sample
    const uint32_t blk = blockIdx.x - b * a.bps;    // workgroup within the sample
    const uint8_t *m = a.in + uint64_t(b) * a.vox;

    // decode a flat index into coordinates
    auto decode = [&](uint32_t f, int32_t *c) {
#pragma unroll
        for (int k = MAXND - 1; k >= 0; --k) {
            if (k < nd) {
                const uint32_t q = a.div_shape[k].div(f);
                c[k] = int32_t(f - q * a.div_shape[k].d);
                f = q;
            }
        }
    };
    // this thread's elements
    uint32_t e[kBfPer];
    V x[kBfPer][MAXND];
    V best[kBfPer];
    uint32_t arg[kBfPer];
    int32_t xx[kBfPer];                     // KEY: squared length of the coordinates
#pragma unroll
    for (int j = 0; j < kBfPer; ++j) {
        e[j] = blk * uint32_t(kBfOut) + uint32_t(j * kBfThreads + t);
        int32_t c[MAXND];
        decode(min(e[j], a.vox - 1), c);
#pragma unroll
        for (int k = 0; k < MAXND; ++k)
            if (k < nd) x[j][k] = KEY ? V(-2 * c[k]) : SAMP ? V(float(c[k]) * a.s[k]) : V(c[k]);
        xx[j] = 0;
        if constexpr (KEY) {
#pragma unroll
            for (int k = 0; k < MAXND; ++k) xx[j] += c[k] * c[k];
        }
        if constexpr (SAMP) best[j] = __builtin_inff();
        else best[j] = 0x7fffffff;
        arg[j] = 0xffffffffu;
    }

    // PB mask bytes from p (foreground past the end), and their zeros
    struct Bytes {
        uint32_t w[PB / 4];
    };
    auto fetch = [&](Bytes &y, uint32_t p) {
        if (PB == 16 && p + PB <= a.vox && (uintptr_t(m) + p) % 16 == 0) {
            const uint4 w = *reinterpret_cast<const uint4 *>(m + p);
            const uint32_t d4[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int j = 0; j < PB / 4; ++j) y.w[j] = d4[j];
        } else if (PB == kBfBytesMany && p + PB <= a.vox && (uintptr_t(m) + p) % 4 == 0) {
#pragma unroll
            for (int j = 0; j < PB / 4; ++j) y.w[j] = reinterpret_cast<const uint32_t *>(m + p)[j];
        } else {
#pragma unroll
            for (int j = 0; j < PB / 4; ++j) y.w[j] = 0;
#pragma unroll
            for (int j = 0; j < PB; ++j) y.w[j / 4] |= uint32_t(m[min(p + j, a.vox - 1)]) << (8 * (j % 4));
        }
    };
    auto zero_flags = [&](const Bytes &y, uint32_t p) {
        uint32_t flags = 0;
#pragma unroll
        for (int j = 0; j < PB; ++j)
            if (p + j < a.vox && ((y.w[j / 4] >> (8 * (j % 4))) & 0xffu) == 0) flags |= 1u << j;
        return flags;
    };
    Bytes cur;
    fetch(cur, uint32_t(t) * PB);
    for (uint32_t c0 = 0; c0 < a.vox; c0 += kBfChunk) {
        // ---- compact the chunk's background elements, in row-major order ----
        const uint32_t p0 = c0 + uint32_t(t) * PB;
        uint32_t flags = zero_flags(cur, p0);
        // the next chunk's bytes, on their way while this one's list runs
        if (c0 + kBfChunk < a.vox) fetch(cur, p0 + kBfChunk);
        uint32_t upto = __popc(flags);
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const uint32_t u = __shfl_up(upto, d, kWave);
            upto += lane >= d ? u : 0u;
        }
        if (lane == kWave - 1) wave_tot[wv] = upto;
        __syncthreads();
        uint32_t base = 0, count = 0;
#pragma unroll
        for (int w = 0; w < kBfThreads / kWave; ++w) {
            if (w < wv) base += wave_tot[w];
            count += wave_tot[w];
        }
        uint32_t pos = base + upto - __popc(flags);
        for (; flags; flags &= flags - 1) {
            const uint32_t f = p0 + uint32_t(__ffs(flags) - 1);
            int32_t c[MAXND];
            decode(f, c);
            if constexpr (KEY) {
                int32_t yy = 0;
#pragma unroll
                for (int k = 0; k < MAXND; ++k) yy += c[k] * c[k];
                zk[pos] = make_int4(c[0] << kBfKeyBits, c[1] << kBfKeyBits, MAXND > 2 ? c[MAXND - 1] << kBfKeyBits : 0,
                                    int32_t((uint32_t(yy) << kBfKeyBits) | pos % kBfRun));
            } else {
#pragma unroll
                for (int k = 0; k < MAXND; ++k)
                    if (k < nd) zc[pos][k] = SAMP ? V(float(c[k]) * a.s[k]) : V(c[k]);
            }
            if (!KEY) zflat[pos] = uint16_t(f - c0);
            ++pos;
        }
        if (KEY && t < 4) zk[count + t] = make_int4(0, 0, 0, 0x7fffffff);   // whole fours
        __syncthreads();
        if constexpr (KEY) {
            for (uint32_t z0 = 0; z0 < count; z0 += kBfRun) {
                const uint32_t z1 = min(count, z0 + kBfRun);
                int32_t key[kBfPer];
#pragma unroll
                for (int j = 0; j < kBfPer; ++j) key[j] = 0x7fffffff;
                for (uint32_t z = z0; z < z1; z += 4) {
                    int4 y[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) y[i] = zk[z + i];
#pragma unroll
                    for (int j = 0; j < kBfPer; ++j) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            // (unsigned: partial sums wrap modulo 2^32; the key itself fits)
                            uint32_t v = uint32_t(__mul24(x[j][0], y[i].x)) + uint32_t(y[i].w);
                            v = uint32_t(__mul24(x[j][1], y[i].y)) + v;
                            if (MAXND > 2) v = uint32_t(__mul24(x[j][MAXND - 1], y[i].z)) + v;
                            key[j] = min(key[j], int32_t(v));
                        }
                    }
                }
#pragma unroll
                for (int j = 0; j < kBfPer; ++j) {
                    const int32_t v = (key[j] >> kBfKeyBits) + xx[j];
                    if (v < best[j]) {
                        best[j] = v;
                        const int4 y = zk[z0 + uint32_t(key[j] & (kBfRun - 1))];
                        uint32_t f = uint32_t(y.x >> kBfKeyBits) * a.div_shape[1].d + uint32_t(y.y >> kBfKeyBits);
                        if (MAXND > 2) f = f * a.div_shape[MAXND - 1].d + uint32_t(y.z >> kBfKeyBits);
                        arg[j] = 0x80000000u | f;
                    }
                }
            }
            __syncthreads();
            continue;
        }
        // ---- run the list against this thread's elements ----------------------
        for (uint32_t z = 0; z < count; ++z) {
            V y[MAXND];
#pragma unroll
            for (int k = 0; k < MAXND; ++k)
                if (k < nd) y[k] = zc[z][k];
#pragma unroll
            for (int j = 0; j < kBfPer; ++j) {
                V v = V(0);
#pragma unroll
                for (int k = 0; k < MAXND; ++k) {
                    if (k < nd) {
                        const V d = x[j][k] - y[k];
                        if (METRIC == 0) v += d * d;
                        else if (METRIC == 1) v += d < V(0) ? -d : d;
                        else v = max(v, d < V(0) ? -d : d);
                    }
                }
                if (v < best[j]) {
                    best[j] = v;
                    arg[j] = z;
                }
            }
        }
        // remember the winners' flat indices before the list is rewritten
#pragma unroll
        for (int j = 0; j < kBfPer; ++j)
            if (arg[j] != 0xffffffffu && arg[j] < 0x80000000u) arg[j] = 0x80000000u | (c0 + zflat[arg[j]]);
        __syncthreads();
    }

    // ---- outputs -------------------------------------------------------------
#pragma unroll
    for (int j = 0; j < kBfPer; ++j) {
        if (e[j] >= a.vox) continue;
        int32_t c[MAXND], y[MAXND];
        decode(e[j], c);
        double value;
        if (arg[j] == 0xffffffffu) {
            // no background in the sample: the virtual element (-1, 0, ..., 0)
            double v = 0.0;
#pragma unroll
            for (int k = 0; k < MAXND; ++k) {
                if (k < nd) {
                    y[k] = k == 0 ? -1 : 0;
                    const double d = a.sd[k] * double(c[k] - y[k]);
                    if (METRIC == 0) v += d * d;
                    else if (METRIC == 1) v += d;
                    else v = v > d ? v : d;
                }
            }
            value = v;
        } else {
            decode(arg[j] & 0x7fffffffu, y);
            value = double(best[j]);
        }
        if (a.dist) {
            float dv;
            if (METRIC != 0) dv = float(value);
            else if (!SAMP && value < 16777216.0) dv = sqrtf(float(value));
            else dv = float(sqrt(value));
            a.dist[uint64_t(b) * a.vox + e[j]] = dv;
        }
        if (a.idx) {
#pragma unroll
            for (int k = 0; k < MAXND; ++k)
                if (k < nd) a.idx[(uint64_t(b) * uint32_t(nd) + uint32_t(k)) * a.vox + e[j]] = y[k];
        }
    }
}

}  // namespace tmedt
