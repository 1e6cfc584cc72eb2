// The next layer's change list by stream compaction (PlanArgs): one workgroup
// per tile of rows, inside a layer kernel's launch (all but sparse backbones and
// very large grids, whose lists come from the tiles).
//
// Method (SSCATeR, arXiv 2512.08557, Alg. 1): every output site touched by the
// scatter of a changed site is changed; with 3x3 kernels that is a dilation of
// the change map by one cell, downsampled for stride 2.  On bitmaps of 32
// cells per word a word of the target is the OR of the nine taps' shifted
// source words, and the scatter's (input, output) pairs are their bit counts.
// The tile's words are counted and scanned, the tile takes its places in the
// list's segments with one atomic each, and its cells are written in row-major order,
// a lane per cell, with their stamps and the nine bits that say which inputs
// changed.  The layer that consumes the list then needs no stamps, and tiles
// of it are neighbouring cells.
//
// What bounds it: its chain of round trips (source bits, the segments'
// counters, the writes), about 5 us, beside the launch's own tiles; so the
// tiles are small (128 words), and only words with something in them reach the
// write phase (with 256-word tiles, every word visited and its neighbours
// gathered again per cell, the plan took 12 us and outlasted every launch it
// was in).  Before, every layer's tiles stamped the next layer's footprint with
// nine device-scope atomics per cell and appended what was new: two dependent
// round trips beyond the XCD's L2 in every tile, and a third for the consumer
// to look up its inputs' stamps.  Measured on the 432x496 backbone, fp32: the
// 64->64 launches 9.3 -> 8.0 us, 128->128 10.7 -> 10.0; bf16 7.5 -> 5.8, 8.7 ->
// 7.5, 256->256 10.4 -> 9.7; per stride with its reads fp32 204 -> 199, bf16
// 161 -> 143 us; first window 559 -> 521.
#pragma once

#include "device_common.h"

namespace ssc {

// The 16 even bits of x.
__device__ __forceinline__ uint32_t even_bits(uint32_t x) {
    x &= 0x55555555u;
    x = (x | (x >> 1)) & 0x33333333u;
    x = (x | (x >> 2)) & 0x0F0F0F0Fu;
    x = (x | (x >> 4)) & 0x00FF00FFu;
    return (x | (x >> 8)) & 0x0000FFFFu;
}

// A target word with something in it, as the write phase reads it.
struct alignas(16) PlanWord {
    uint32_t tap[9];          // bit b: the input under tap t of cell b changed
    uint32_t any;             // their OR: the changed cells
    int pos;                  // cells of the tile before it
    int cell;                 // grid cell of bit 0
};
static_assert(sizeof(PlanWord) == 48, "three 16-byte LDS reads");

// lin: PLAN_IN words; rec: PLAN_WORDS records; wsum: 2 * NW + 2 words.  Every
// thread of the workgroup calls it.
template <int NW>
__device__ __forceinline__ void plan_tile(const PlanArgs& t, uint32_t epoch, int id, uint32_t* lin, PlanWord* rec,
                                          int* wsum) {
    constexpr int NTH = 64 * NW;
    const int tid = (int)threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (id >= t.tiles) return;                             // uniform: padding workgroups
    const int per_img = t.bands * t.chunks;
    const int img = id / per_img, rest = id - img * per_img, band = rest / t.chunks;
    const int r0 = band * t.rows, nr = min(t.rows, t.Hout - r0);
    const int x0 = (rest - band * t.chunks) * t.cols, nx = min(t.cols, t.wpo - x0);
    const int nwo = nr * nx;
    // source rows i0 .. i0 + ni - 1 and words j0 .. j0 + nj - 1 (one beyond the
    // tile on every side; outside the image they are zero)
    const int i0 = t.stride * r0 - 1, ni = t.stride * (nr - 1) + 3;
    const int j0 = t.stride * x0 - 1, nj = t.stride * nx + 2;
    const int nwi = ni * nj;

    if (t.bits_in) {
        const uint32_t* src = t.bits_in + (size_t)img * t.Hin * t.wpi;
        for (int k = tid; k < nwi; k += NTH) {
            const int r = (int)t.dnj[nx == t.cols ? 0 : 1]((uint32_t)k);
            const int i = i0 + r, j = j0 + k - r * nj;
            const bool in = i >= 0 && i < t.Hin && j >= 0 && j < t.wpi;
            const uint32_t v = src[min(max(i, 0), t.Hin - 1) * t.wpi + min(max(j, 0), t.wpi - 1)];
            lin[k] = in ? v : 0u;
        }
    } else {
        // by cell index: a row's word straddles two
        for (int k = tid; k < nwi; k += NTH) {
            const int r = (int)t.dnj[nx == t.cols ? 0 : 1]((uint32_t)k);
            const int i = i0 + r, j = j0 + k - r * nj;
            const bool in = i >= 0 && i < t.Hin && j >= 0 && j < t.wpi;
            const int at = (img * t.Hin + min(max(i, 0), t.Hin - 1)) * t.Win + 32 * min(max(j, 0), t.wpi - 1);
            const uint64_t v = (uint64_t)t.flat_in[at >> 5] | ((uint64_t)t.flat_in[(at >> 5) + 1] << 32);
            const int left = t.Win - 32 * j;
            const uint32_t keep = left >= 32 ? ~0u : (1u << (left & 31)) - 1u;
            lin[k] = in ? (uint32_t)(v >> (at & 31)) & keep : 0u;
        }
    }
    __syncthreads();

    // the target words, a thread each (passes of NTH words, in order), and
    // their cells' places: words with something in them get a record
    int nrec = 0, total = 0, pairs = 0;
    for (int k0 = 0; k0 < nwo; k0 += NTH) {
        const int k = k0 + tid;
        PlanWord p = {};
        int r = 0, x = 0;
        if (k < nwo) {
            r = (int)t.dnx[nx == t.cols ? 0 : 1]((uint32_t)k);
            x = k - r * nx;
            const int left = t.Wout - 32 * (x0 + x);
            const uint32_t keep = left >= 32 ? ~0u : (1u << left) - 1u;
#pragma unroll
            for (int m = 0; m < 3; ++m) {
                // source columns -1, 0, +1 of every target column
                const uint32_t* s = lin + (t.stride * r + m) * nj + t.stride * x;
                uint32_t tl, tc, tr;
                if (t.stride == 1) {
                    const uint32_t l = s[0], c = s[1], n = s[2];
                    tl = (c << 1) | (l >> 31);
                    tc = c;
                    tr = (c >> 1) | (n << 31);
                } else {
                    const uint32_t l = s[0], c = s[1], n = s[2];
                    tc = even_bits(c) | (even_bits(n) << 16);
                    tr = even_bits(c >> 1) | (even_bits(n >> 1) << 16);
                    tl = (tr << 1) | (l >> 31);
                }
                p.tap[3 * m] = tl & keep;
                p.tap[3 * m + 1] = tc & keep;
                p.tap[3 * m + 2] = tr & keep;
            }
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                p.any |= p.tap[q];
                pairs += (int)__popc(p.tap[q]);
            }
            t.bits_out[((size_t)img * t.Hout + r0 + r) * t.wpo + x0 + x] = p.any;
        }
        const int mine = (int)__popc(p.any);
        int incl = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(incl, d);
            if (lane >= d) incl += y;
        }
        const unsigned long long has = __ballot(p.any != 0u);
        if (lane == 63) {
            wsum[w] = incl;
            wsum[NW + w] = (int)__popcll(has);
        }
        __syncthreads();
        int cells = total + incl - mine, recs = nrec + (int)__popcll(has & ((1ull << lane) - 1ull));
#pragma unroll
        for (int q = 0; q < NW; ++q) {
            cells += q < w ? wsum[q] : 0;
            recs += q < w ? wsum[NW + q] : 0;
            total += wsum[q];
            nrec += wsum[NW + q];
        }
        if (p.any) {
            p.pos = cells;
            p.cell = (img * t.Hout + r0 + r) * t.Wout + 32 * (x0 + x);
            rec[recs] = p;
        }
        __syncthreads();                                   // the records; wsum is free for the next pass
    }
    // the tile's places in the list segments, an equal share of its cells in
    // each (a small grid is one tile, and half of the consumer's workgroups
    // walk either segment)
    if (total == 0) return;                                // uniform
    static_assert(NSHARD == 2, "two halves");
    const int half = (total + 1) / 2;
    if (tid < 2 && (tid == 0 || total > 1))
        wsum[2 * NW + tid] = atomicAdd(t.count + tid * CSTRIDE, tid == 0 ? half : total - half);
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) pairs += __shfl_xor(pairs, d);
    if (lane == 0 && pairs) atomicAdd(t.pairs + ((w & 1) * PSPREAD + (int)(blockIdx.x & (PSPREAD - 1))) * CSTRIDE, pairs);
    __syncthreads();
    const int at0 = wsum[2 * NW], at1 = t.seg + wsum[2 * NW + 1] - half;

    // the cells, a lane each: two words per wavefront pass
    const int b = lane & 31;
    for (int k0 = 2 * w; k0 < nrec; k0 += 2 * NW) {
        const int k = k0 + (lane >> 5);
        const PlanWord p = rec[min(k, nrec - 1)];
        if (k >= nrec || !((p.any >> b) & 1u)) continue;
        uint32_t mask = 0u;
#pragma unroll
        for (int q = 0; q < 9; ++q) mask |= ((p.tap[q] >> b) & 1u) << q;
        const int nth = p.pos + (int)__popc(p.any & ((1u << b) - 1u));
        const size_t pos = (size_t)((nth < half ? at0 : at1) + nth);
        t.list[pos] = p.cell + b;
        t.taps[pos] = (uint16_t)mask;
        t.stamp[p.cell + b] = epoch;
    }
}

}  // namespace ssc
