// Device helpers shared by the kernels: wavefront-aggregated list appends and
// the structural change-list propagation rule.
#pragma once

#include "sscater_internal.h"

namespace ssc {

typedef float f4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63u); }

// Structural propagation of changed cells to the next layer's list, in two
// phases for latency hiding.  Cell (i, j) of the grid (t.Hin x t.Win) feeds
// output ((i - m + 1)/s, (j - n + 1)/s) through tap (m, n) when both quotients
// are integral and inside (t.Hout x t.Wout): the scatter target of Eq. 2
// generalised to stride s, and the downsampling rule of Alg. 1 for s = 2.
// Each cell is handled by G lanes that share its 9 tap slots (slot = sub +
// it*G).  prop_issue stamps every target with `epoch` (atomicMax: the lane
// that moves a stamp owns the target); prop_finish (later, after unrelated
// work) counts the pairs and appends the owned targets of the wavefront to
// list segment `shard` with a single atomic.
// Both must be reached by every lane of the wavefront.
template <int G>
struct PropBatch {
    static constexpr int ITERS = (9 + G - 1) / G;
    int q[ITERS];
    uint32_t old[ITERS];   // stamp before this lane's atomic (owner iff < epoch)
};

// cell: a valid cell of the source grid (used for addressing even when
// inactive); active: whether the cell really changed.  Inactive lanes issue
// nothing.
template <int G>
__device__ __forceinline__ void prop_issue(const PropTarget& t, int cell, bool active, int sub, uint32_t epoch,
                                           PropBatch<G>& pb) {
    const int img = cell / (t.Hin * t.Win), loc = cell - img * (t.Hin * t.Win);
    const int i = loc / t.Win, j = loc - (loc / t.Win) * t.Win;
    const int obase = img * (t.Hout * t.Wout);
#pragma unroll
    for (int it = 0; it < PropBatch<G>::ITERS; ++it) {
        const int k = sub + it * G;
        const int m = k / 3, n = k - 3 * (k / 3);
        int rn = i - m + 1, cn = j - n + 1;
        bool ok = active && k < 9;
        if (t.stride == 2) {
            ok = ok && ((rn | cn) & 1) == 0;
            rn >>= 1;
            cn >>= 1;
        }
        ok = ok && rn >= 0 && rn < t.Hout && cn >= 0 && cn < t.Wout;
        const int q = obase + min(max(rn, 0), t.Hout - 1) * t.Wout + min(max(cn, 0), t.Wout - 1);
        pb.q[it] = ok ? q : -1;
        // pb.old is read only where q >= 0; leaving it unset on the other path
        // avoids a register copy that would wait for the atomic
        if (ok) pb.old[it] = atomicMax(&t.stamp[q], epoch);
    }
}

template <int G>
__device__ __forceinline__ void prop_finish(const PropTarget& t, uint32_t epoch, int shard, PropBatch<G>& pb) {
    constexpr int IT = PropBatch<G>::ITERS;
    const int lane = lane_id();
    const unsigned long long lt = (1ull << lane) - 1ull;
    unsigned long long ob[IT];
    bool own[IT];
    int pairs = 0, tot = 0;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        own[it] = pb.q[it] >= 0 && pb.old[it] < epoch;
        pairs += (int)__popcll(__ballot(pb.q[it] >= 0));
        ob[it] = __ballot(own[it]);
        tot += (int)__popcll(ob[it]);
    }
    int base = 0;
    if (lane == 0) {
        if (tot) base = atomicAdd(t.count + shard * CSTRIDE, tot);
        if (pairs) atomicAdd(t.pairs + (shard * PSPREAD + (int)(blockIdx.x & (PSPREAD - 1))) * CSTRIDE, pairs);
    }
    if (tot == 0) return;
    base = __shfl(base, 0);
    int32_t* seg = t.list + (size_t)shard * t.seg;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        if (own[it]) {
            seg[base + (int)__popcll(ob[it] & lt)] = pb.q[it];
            if (t.bits) atomicOr(&t.bits[pb.q[it] >> 5], 1u << (pb.q[it] & 31));
        }
        base += (int)__popcll(ob[it]);
    }
}

// Active-set words (sparse backbones): see MembTarget.
__device__ __forceinline__ bool memb_now(uint64_t w) { return (uint32_t)w != 0u; }

__device__ __forceinline__ bool memb_prev(uint64_t w, uint32_t epoch) {
    return (uint32_t)(w >> 33) == (epoch & 0x7FFFFFFFu) ? ((w >> 32) & 1ull) != 0ull : memb_now(w);
}

// Counts of the next regular layer: +-1 at every output site whose receptive
// field holds `cell` (the same stride rule as the change lists), in two
// halves like the propagation: memb_issue computes the targets and loads
// their words (from clamped, always valid addresses, also where `on` is
// false, so that no branch joins on the loads), memb_finish compare-and-swaps
// them.  A swap that lost to another lane or workgroup goes round again; all
// of a lane's pending targets go round together, so a round costs one round
// trip however many of them collided.
struct MembBatch {
    unsigned long long old[9];   // the targets' words as loaded
    uint32_t todo;               // bit k: target k exists and is to be updated
};

// Target k of `cell` (clamped to the grid) and whether it exists.
__device__ __forceinline__ unsigned long long* memb_target(const MembTarget& t, int cell, int hin, int win, int k,
                                                            bool& ok) {
    const int img = cell / (hin * win), loc = cell - img * (hin * win);
    const int i = loc / win, j = loc - (loc / win) * win;
    int rn = i - k / 3 + 1, cn = j - k % 3 + 1;
    ok = true;
    if (t.stride == 2) {
        ok = ((rn | cn) & 1) == 0;
        rn >>= 1;
        cn >>= 1;
    }
    ok = ok && rn >= 0 && rn < t.Hout && cn >= 0 && cn < t.Wout;
    return reinterpret_cast<unsigned long long*>(t.memb) + (size_t)img * t.Hout * t.Wout +
           (size_t)min(max(rn, 0), t.Hout - 1) * t.Wout + min(max(cn, 0), t.Wout - 1);
}

__device__ __forceinline__ void memb_issue(const MembTarget& t, int cell, int hin, int win, bool on, MembBatch& mb) {
    mb.todo = 0u;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        bool ok;
        unsigned long long* p = memb_target(t, cell, hin, win, k, ok);
        if (on && ok) mb.todo |= 1u << k;
        mb.old[k] = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// The word after adding `delta` to the count; the first change of a stride
// (epoch ep) records whether the site was active before it.
__device__ __forceinline__ unsigned long long memb_next(unsigned long long w, int delta, unsigned long long ep) {
    const uint32_t cnt = (uint32_t)w;
    const unsigned long long was = ((w >> 33) == ep) ? ((w >> 32) & 1ull) : (cnt != 0u ? 1ull : 0ull);
    return (ep << 33) | (was << 32) | (unsigned long long)(uint32_t)(cnt + (uint32_t)delta);
}

// memb_finish in two halves, so that the first swaps' round trip can overlap
// another (memb_swap issues them, memb_settle retries the lost ones); cell,
// hin, win: as given to memb_issue.
__device__ __forceinline__ void memb_swap(const MembTarget& t, int cell, int hin, int win, const MembBatch& mb,
                                          int delta, uint32_t epoch, unsigned long long (&got)[9]) {
    const unsigned long long ep = epoch & 0x7FFFFFFFu;
#pragma unroll
    for (int k = 0; k < 9; ++k) got[k] = mb.old[k];
    if (mb.todo == 0u) return;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        bool ok;
        unsigned long long* p = memb_target(t, cell, hin, win, k, ok);
        if ((mb.todo >> k) & 1u) got[k] = atomicCAS(p, mb.old[k], memb_next(mb.old[k], delta, ep));
    }
}

__device__ __forceinline__ void memb_settle(const MembTarget& t, int cell, int hin, int win, MembBatch& mb, int delta,
                                            uint32_t epoch, const unsigned long long (&got0)[9]) {
    const unsigned long long ep = epoch & 0x7FFFFFFFu;
    uint32_t todo = 0u;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        if (((mb.todo >> k) & 1u) && got0[k] != mb.old[k]) todo |= 1u << k;   // lost: retry from the word it found
        mb.old[k] = got0[k];
    }
    if (todo == 0u) return;
    unsigned long long* ptr[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        bool ok;
        ptr[k] = memb_target(t, cell, hin, win, k, ok);
    }
    while (todo) {
        unsigned long long got[9];
#pragma unroll
        for (int k = 0; k < 9; ++k)
            got[k] = (todo >> k) & 1u ? atomicCAS(ptr[k], mb.old[k], memb_next(mb.old[k], delta, ep)) : 0ull;
        uint32_t lost = 0u;
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            if (((todo >> k) & 1u) && got[k] != mb.old[k]) lost |= 1u << k;
            mb.old[k] = got[k];
        }
        todo = lost;
    }
}

// cell, hin, win: as given to memb_issue.
__device__ __forceinline__ void memb_finish(const MembTarget& t, int cell, int hin, int win, MembBatch& mb, int delta,
                                            uint32_t epoch) {
    unsigned long long got[9];
    memb_swap(t, cell, hin, win, mb, delta, epoch, got);
    memb_settle(t, cell, hin, win, mb, delta, epoch, got);
}

// prop_finish in two halves, so that the counter's round trip overlaps other
// work: prop_reserve counts the owned targets and takes their list positions
// (the atomic's result is not waited for), prop_write stores the entries.
template <int G>
struct PropSlots {
    static constexpr int IT = PropBatch<G>::ITERS;
    unsigned long long ob[IT];
    bool own[IT];
    int base, tot;
};

template <int G>
__device__ __forceinline__ void prop_reserve(const PropTarget& t, uint32_t epoch, int shard, const PropBatch<G>& pb,
                                             PropSlots<G>& ps) {
    constexpr int IT = PropBatch<G>::ITERS;
    int pairs = 0;
    ps.tot = 0;
    ps.base = 0;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        ps.own[it] = pb.q[it] >= 0 && pb.old[it] < epoch;
        pairs += (int)__popcll(__ballot(pb.q[it] >= 0));
        ps.ob[it] = __ballot(ps.own[it]);
        ps.tot += (int)__popcll(ps.ob[it]);
    }
    if (lane_id() == 0) {
        if (ps.tot) ps.base = atomicAdd(t.count + shard * CSTRIDE, ps.tot);
        if (pairs) atomicAdd(t.pairs + (shard * PSPREAD + (int)(blockIdx.x & (PSPREAD - 1))) * CSTRIDE, pairs);
    }
}

template <int G>
__device__ __forceinline__ void prop_write(const PropTarget& t, int shard, const PropBatch<G>& pb, PropSlots<G>& ps) {
    constexpr int IT = PropBatch<G>::ITERS;
    if (ps.tot == 0) return;
    const unsigned long long lt = (1ull << lane_id()) - 1ull;
    int base = __shfl(ps.base, 0);
    int32_t* seg = t.list + (size_t)shard * t.seg;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
        if (ps.own[it]) {
            seg[base + (int)__popcll(ps.ob[it] & lt)] = pb.q[it];
            if (t.bits) atomicOr(&t.bits[pb.q[it] >> 5], 1u << (pb.q[it] & 31));
        }
        base += (int)__popcll(ps.ob[it]);
    }
}

// fp32 -> bf16 bits, round to nearest even (finite values).
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return u >> 16;
}

// Clears n 16-byte values, spread over the grid.
__device__ __forceinline__ void clear_grid(uint4* p, int n) {
    for (int i = (int)(blockIdx.x * blockDim.x + threadIdx.x); i < n; i += (int)(gridDim.x * blockDim.x))
        p[i] = make_uint4(0u, 0u, 0u, 0u);
}

// ---- delta rows ----
//
// A delta row is stored at its cell, 4 bytes per channel in either dtype:
//   fp32: the fp32 deltas phi(Z_new) - phi(Z_old), consecutive channels.
//   bf16: per 32 channels 64 bytes of bf16(phi(Z_new)), then 64 bytes of
//         bf16(phi(Z_old)) (16 channels: 32 bytes each); the consumers
//         contract the difference of the two exactly.
// Consumers take a row in units of 32 channels (a row of 16 is one unit), 128
// bytes, which is one K = 32 matrix instruction's range.
//
// fp32 on the bf16 matrix cores.  A consumer splits its fp32 values in
// registers into three bf16 planes, h = bf16(v), m = bf16(v - h),
// l = v - h - m: 8 significant bits each, so the three hold all 24 bits, and
// with fp32's exponents, so values of any size stand beside each other (only
// bits below 2^-133 are lost).  Weights come split the same way.  Six of the
// nine products are formed; the other three are at most 2 * 2^-8 * 2^-17 +
// 2^-34 of the whole, the size of an fp32 multiplication's one rounding.  Six bf16 instructions take 96 cycles for 32
// channels where the fp32 kind takes 256.  The five smaller products of a unit
// (at most 2^-7 of the first) are summed by themselves and added once, so a
// unit costs the large sum two roundings, as little as it can on 16 registers
// (a second set of sums for them took 32 and spilled).
// Measured against fp16 planes under a power of two shared by 32 channels
// (three products, but the planes hold 22 bits, and fewer for a channel far
// below the unit's largest), error over a 64->64 layer against 64 bits: random
// features 1.0e-7, here 6.7e-8; single products 9.7e-8, 2.9e-8; channels 2^30
// apart with weights the other way round 3.1e-4, 6.7e-8; one channel 10^9 times
// the others with weights of 0 5.5e-4, 6.6e-8 (fp32 matrix instructions 2.7e-7
// in all but the second, 2.7e-8).
constexpr int UNIT_BYTES = 128;
__host__ __device__ constexpr int units_of(int channels) { return channels > 32 ? channels / 32 : 1; }
__host__ __device__ constexpr int delta_row_bytes(int channels) { return 4 * channels; }
// bytes from a bf16 row's new values to the old ones of the same channels
__host__ __device__ constexpr int plane_bytes(int channels) { return channels < 32 ? 2 * channels : 64; }

typedef float f2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf2v __attribute__((ext_vector_type(2)));

// Two values rounded to bf16 (nearest even), x in the low half.
__device__ __forceinline__ uint32_t bf16_pair(float x, float y) {
    const bf2v h = __builtin_convertvector((f2v{x, y}), bf2v);
    uint32_t b;
    __builtin_memcpy(&b, &h, 4);
    return b;
}

// The three planes of two values.  An infinity, and a finite value that rounds
// to one in bf16, leave a NaN in the lower planes, so the sums they enter are
// NaN.  SPECIAL does those right: an infinity goes to `inf` alone, and the
// planes of such a large value are cut off instead of rounded (h + m stays
// below it).  Every other value's planes are the same either way.
template <bool SPECIAL>
__device__ __forceinline__ void split_pair(float x, float y, uint32_t& h, uint32_t& m, uint32_t& l, uint32_t& inf) {
    if constexpr (SPECIAL) {
        const uint32_t xb = __float_as_uint(x), yb = __float_as_uint(y);
        const bool xi = (xb & 0x7FFFFFFFu) == 0x7F800000u, yi = (yb & 0x7FFFFFFFu) == 0x7F800000u;
        inf = (xi ? xb >> 16 : 0u) | (yi ? yb & 0xFFFF0000u : 0u);
        x = xi ? 0.f : x;
        y = yi ? 0.f : y;
    }
    h = bf16_pair(x, y);
    bool xl = false, yl = false;
    if constexpr (SPECIAL) {
        xl = (h & 0x7FFFu) == 0x7F80u;
        yl = (h & 0x7FFF0000u) == 0x7F800000u;
        if (xl) h = (h & 0xFFFF0000u) | (__float_as_uint(x) >> 16);
        if (yl) h = (h & 0xFFFFu) | (__float_as_uint(y) & 0xFFFF0000u);
    }
    const float rx = x - __uint_as_float(h << 16), ry = y - __uint_as_float(h & 0xFFFF0000u);
    m = bf16_pair(rx, ry);
    if constexpr (SPECIAL) {
        if (xl) m = (m & 0xFFFF0000u) | (__float_as_uint(rx) >> 16);
        if (yl) m = (m & 0xFFFFu) | (__float_as_uint(ry) & 0xFFFF0000u);
    }
    l = bf16_pair(rx - __uint_as_float(m << 16), ry - __uint_as_float(m & 0xFFFF0000u));
}

// The matrix operands of one lane's fp32 values of a unit: the four channels
// 4*g .. +3 (a) and, of 32 channels, 16 + 4*g .. +3 (b).  Of 16 channels K
// holds two planes side by side: x = [h | m], y = [h | l], and three
// instructions form the six products.
struct Planes {
    uint4 x, y, z;            // h, m, l (16 channels: x and y as above)
    uint4 inf;
};
template <int CIN, bool SPECIAL>
__device__ __forceinline__ Planes split_unit(const uint4 a, const uint4 b) {
    Planes p = {};
    uint32_t h[4], m[4], l[4], f[4] = {};
    const uint32_t v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    constexpr int N = CIN < 32 ? 2 : 4;
#pragma unroll
    for (int j = 0; j < N; ++j)
        split_pair<SPECIAL>(__uint_as_float(v[2 * j]), __uint_as_float(v[2 * j + 1]), h[j], m[j], l[j], f[j]);
    if constexpr (CIN < 32) {
        p.x = make_uint4(h[0], h[1], m[0], m[1]);
        p.y = make_uint4(h[0], h[1], l[0], l[1]);
    } else {
        p.x = make_uint4(h[0], h[1], h[2], h[3]);
        p.y = make_uint4(m[0], m[1], m[2], m[3]);
        p.z = make_uint4(l[0], l[1], l[2], l[3]);
    }
    p.inf = make_uint4(f[0], f[1], f[2], f[3]);
    return p;
}

__device__ __forceinline__ f4v mfma_bf16(const uint4 w, const uint4 v, const f4v c) {
    bf8v W, V;
    __builtin_memcpy(&W, &w, 16);
    __builtin_memcpy(&V, &v, 16);
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(W, V, c, 0, 0, 0);
}

// One unit of one operand for NB blocks of 16 output channels; w0, w1, w2: the
// weight planes Wh, Wm, Wl of every block (of 16 channels [Wh | Wh], [Wm |
// Wh], [Wl | Wm]).  Products outer, blocks inner: an accumulator's
// instructions are NB apart.
template <int CIN, int NB, bool SPECIAL>
__device__ __forceinline__ void mfma_unit(f4v (&acc)[NB], const uint4* w0, const uint4* w1, const uint4* w2,
                                          const Planes& p) {
    f4v lo[NB];
#pragma unroll
    for (int k = 0; k < NB; ++k) lo[k] = f4v{0.f, 0.f, 0.f, 0.f};
    auto all = [&](f4v (&c)[NB], const uint4* w, const uint4 v) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < NB; ++k) c[k] = mfma_bf16(w[k], v, c[k]);
    };
    if constexpr (CIN < 32) {
        all(lo, w2, p.x);
        all(lo, w1, p.y);
        all(acc, w0, p.x);
    } else {
        all(lo, w2, p.x);
        all(lo, w1, p.y);
        all(lo, w0, p.z);
        all(lo, w1, p.x);
        all(lo, w0, p.y);
        all(acc, w0, p.x);
    }
#pragma unroll
    for (int k = 0; k < NB; ++k)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[k][e] += lo[k][e];
    if constexpr (SPECIAL) all(acc, w0, p.inf);
}

// Z update and next-layer delta row of one lane: output cell q, NBL blocks of
// 16 output channels from channel c0 on, of which the lane holds the four at
// 4*g (Z_new = Z_old + D; delta phi(Z_new) - phi(Z_old), see above).
// Sparse backbones: now / prev say whether the site is active in this and
// in the previous stride; an inactive site's output is zero.
template <int COUT, bool BF16, int NBL>
__device__ __forceinline__ void epilogue_unit(const LayerArgs& a, int q, int c0, int g, const f4v (&o)[NBL],
                                              const f4v (&d)[NBL], bool now, bool prev) {
    char* drow = static_cast<char*>(a.delta_out) + (size_t)q * delta_row_bytes(COUT);
#pragma unroll
    for (int i = 0; i < NBL; ++i) {
        const int co = c0 + i * 16 + 4 * g;
        f4v zn;
#pragma unroll
        for (int k = 0; k < 4; ++k) zn[k] = o[i][k] + d[i][k];
        *reinterpret_cast<f4v*>(a.Z + (size_t)q * COUT + co) = zn;
        if (!a.delta_out) continue;                       // uniform
        f4v yo = o[i], yn = zn;
        if (a.relu) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                yo[k] = fmaxf(yo[k], 0.f);
                yn[k] = fmaxf(yn[k], 0.f);
            }
        }
        if (!prev) yo = f4v{0.f, 0.f, 0.f, 0.f};
        if (!now) yn = f4v{0.f, 0.f, 0.f, 0.f};
        if constexpr (BF16) {
            uint2 pn, po;
            pn.x = f32_to_bf16_bits(yn.x) | (f32_to_bf16_bits(yn.y) << 16);
            pn.y = f32_to_bf16_bits(yn.z) | (f32_to_bf16_bits(yn.w) << 16);
            po.x = f32_to_bf16_bits(yo.x) | (f32_to_bf16_bits(yo.y) << 16);
            po.y = f32_to_bf16_bits(yo.z) | (f32_to_bf16_bits(yo.w) << 16);
            char* u = drow + co / 32 * UNIT_BYTES + co % 32 * 2;
            *reinterpret_cast<uint2*>(u) = pn;
            *reinterpret_cast<uint2*>(u + plane_bytes(COUT)) = po;
        } else {
            f4v dy;
#pragma unroll
            for (int k = 0; k < 4; ++k) dy[k] = yn[k] - yo[k];
            *reinterpret_cast<f4v*>(drow + co * 4) = dy;
        }
    }
}

// ---- rings of LDS stages filled by asynchronous global->LDS copies ----

// s_waitcnt with only the vector-memory count limited to n.
template <int n>
__device__ __forceinline__ void wait_vm() {
    static_assert(n >= 0 && n < 64, "vmcnt");
    __builtin_amdgcn_s_waitcnt((n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14));
}

// Workgroup barrier without a memory fence.  __syncthreads() also drains
// every outstanding global access and LDS copy (vmcnt(0)), which would wait
// for the copies of the later chunks too.  Here each thread first waits for
// its own copies of the chunk it needs (wait_vm), and its LDS reads of the
// previous chunk have completed before their matrix instructions ran, so the
// hardware barrier makes the stage safe once this wavefront's own LDS reads
// have completed; the empty asm statements keep the compiler from moving
// memory accesses across it.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");
    // this wavefront's LDS reads are complete (lgkmcnt(0), no vmcnt limit)
    __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// wait_vm for a count that is a constant once its loop is unrolled (at most N)
template <int N>
__device__ __forceinline__ void wait_vm_n(int n) {
    if (n >= N) wait_vm<N>();
    else if constexpr (N > 0) wait_vm_n<N - 1>(n);
}

typedef __attribute__((address_space(3))) char lds_char;

// 16 bytes per lane from global memory straight into LDS (lane l to lds + 16*l)
__device__ __forceinline__ void copy16(const void* src, lds_char* lds) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                     (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}

__device__ __forceinline__ uint4 lds16(const lds_char* p) {
    typedef uint32_t u4v __attribute__((ext_vector_type(4)));
    const u4v v = *reinterpret_cast<const __attribute__((address_space(3))) u4v*>(p);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// The value is needed here: nothing that makes it may be moved past this point.
__device__ __forceinline__ void pin(uint4& v) {
    asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
}

__device__ __forceinline__ void flag_error(int32_t* err, int bit) {
    *(volatile int32_t*)err = bit;
}

}  // namespace ssc
