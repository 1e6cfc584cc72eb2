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
// inactive); active: whether the cell really changed.
// UNCOND = true: every lane issues its atomic unconditionally so that no
// branch joins on the returned value (a join would make the compiler wait for
// it right there).  A slot without a target stamps a clamped cell next to
// `cell` with 0, which never changes a stamp (stamps only grow and epochs
// start at 1); the addresses stay spread over the grid.  Use it where most
// lanes are active.  UNCOND = false: inactive lanes issue nothing.
template <int G, bool UNCOND>
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
        if (UNCOND) {
            pb.old[it] = atomicMax(&t.stamp[q], ok ? epoch : 0u);
        } else if (ok) {
            // pb.old is read only where q >= 0; leaving it unset on the other
            // path avoids a register copy that would wait for the atomic
            pb.old[it] = atomicMax(&t.stamp[q], epoch);
        }
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

__device__ __forceinline__ void memb_spread(const MembTarget& t, int cell, int hin, int win, int delta,
                                            uint32_t epoch) {
    MembBatch mb;
    memb_issue(t, cell, hin, win, true, mb);
    memb_finish(t, cell, hin, win, mb, delta, epoch);
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
// A delta row is stored at its cell in units of 32 channels, 128 bytes each:
// two planes of 32 16-bit values, so that one unit is both planes of one
// K = 32 matrix instruction and a row has 4 bytes per channel in either dtype.
// Rows of fewer than 32 channels take one unit whose other values stay zero.
//   bf16: plane 0 holds bf16(phi(Z_new)), plane 1 bf16(phi(Z_old)); the
//         consumers contract the difference of the two exactly.
//   fp32: plane 0 holds hi = fp16(v * s), plane 1 lo = fp16(v * s - hi), where
//         v is the fp32 delta and s the power of two that brings the unit's
//         largest |v| into [2^14, 2^15); the unit's 1/s is kept beside the
//         rows as a bf16 value (a power of two, so exact).  hi + lo carries v
//         to 2^-24 of itself, half an fp32 ulp (2^-39 of the unit's largest
//         value where that is more), and the weights are split the same way
//         with a scale per output channel, so hi*hi + lo*hi + hi*lo on the
//         fp16 matrix cores stands for the fp32 product at 3 matrix
//         instructions per 32 channels instead of 8 of the fp32 kind.  Scales
//         multiply fp32 sums only, by powers of two.
//         A row of 16 channels leaves half of its unit free, which takes what
//         the split leaves over (rest = v * s - hi - lo, at no cost to the
//         consumers): plane 0 = [hi | rest], plane 1 = [lo | hi], against the
//         weights' planes [Whi | Wrest] and [Wlo | Whi].  The short sums of 16
//         channels are the ones where the split's error would show (3e-8 of
//         the result beside the 9e-8 of the fp32 arithmetic around it).
// A unit that holds a NaN or an infinity gets that as its 1/s (and +-1 at the
// infinite values), so that what it contributes is not finite either.
constexpr int UNIT_BYTES = 128;
__host__ __device__ constexpr int units_of(int channels) { return channels > 32 ? channels / 32 : 1; }
__host__ __device__ constexpr int delta_row_bytes(int channels) { return units_of(channels) * UNIT_BYTES; }

typedef _Float16 h8v __attribute__((ext_vector_type(8)));
typedef _Float16 h4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t abs_bits4(const f4v v) {
    return max(max(__float_as_uint(v.x) & 0x7FFFFFFFu, __float_as_uint(v.y) & 0x7FFFFFFFu),
               max(__float_as_uint(v.z) & 0x7FFFFFFFu, __float_as_uint(v.w) & 0x7FFFFFFFu));
}

// Scale of a unit whose largest |value| has the bits mb: the factor s, and
// the bf16 bits of 1/s.
struct UnitScale {
    float s;
    uint16_t inv;
    bool finite;
};
__device__ __forceinline__ UnitScale unit_scale(uint32_t mb) {
    UnitScale u;
    const int e = (int)(mb >> 23);                    // biased exponent of the largest value
    u.finite = e != 255;
    const int se = min(268 - e, 253);                 // s = 2^(se - 127), 1/s a normal number
    u.s = __uint_as_float((uint32_t)se << 23);
    u.inv = (uint16_t)(u.finite ? (254 - se) << 7 : (mb > 0x7F800000u ? 0x7FC0 : 0x7F80));
    return u;
}

// hi, lo and rest of a value under its unit's scale.
__device__ __forceinline__ void split1(float v, const UnitScale& u, _Float16& hi, _Float16& lo, _Float16& rest) {
    float t = v * u.s;
    if (!u.finite) t = __builtin_isinf(v) ? copysignf(1.f, v) : 0.f;
    hi = (_Float16)t;
    lo = (_Float16)(t - (float)hi);
    rest = (_Float16)(t - (float)hi - (float)lo);
}

// Four consecutive channels of a row of C channels into their places (p: the
// first one's in plane 0).
template <int C>
__device__ __forceinline__ void store_split4(char* p, const f4v v, const UnitScale& u, bool store) {
    h4v h, l, r;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        _Float16 x, y, z;
        split1(v[k], u, x, y, z);
        h[k] = x;
        l[k] = y;
        r[k] = z;
    }
    if (!store) return;
    *reinterpret_cast<h4v*>(p) = h;
    *reinterpret_cast<h4v*>(p + 64) = l;
    if constexpr (C == 16) {
        *reinterpret_cast<h4v*>(p + 32) = r;
        *reinterpret_cast<h4v*>(p + 96) = h;
    }
}

__device__ __forceinline__ float bf16_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

// Z update and next-layer delta row of one lane: output cell q, NBL blocks of
// 16 output channels from channel c0 on, of which the lane holds the four at
// 4*g (Z_new = Z_old + D; delta phi(Z_new) - phi(Z_old), see above).  The NBL
// blocks are one unit (or all of a row of fewer than 32 channels), and the
// lanes l, l^16, l^32, l^48 hold its channels of one cell: every lane of the
// wavefront calls this, `store` says whether its cell and channels exist.
// Sparse backbones: now / prev say whether the site is active in this and
// in the previous stride; an inactive site's output is zero.
template <int COUT, bool BF16, int NBL>
__device__ __forceinline__ void epilogue_unit(const LayerArgs& a, int q, int c0, int g, const f4v (&o)[NBL],
                                              const f4v (&d)[NBL], bool store, bool now, bool prev) {
    f4v yo[NBL], yn[NBL];
#pragma unroll
    for (int i = 0; i < NBL; ++i) {
        f4v zn;
#pragma unroll
        for (int k = 0; k < 4; ++k) zn[k] = o[i][k] + d[i][k];
        if (store) *reinterpret_cast<f4v*>(a.Z + (size_t)q * COUT + c0 + i * 16 + 4 * g) = zn;
        yo[i] = o[i];
        yn[i] = zn;
        if (a.relu) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                yo[i][k] = fmaxf(yo[i][k], 0.f);
                yn[i][k] = fmaxf(yn[i][k], 0.f);
            }
        }
        if (!prev) yo[i] = f4v{0.f, 0.f, 0.f, 0.f};
        if (!now) yn[i] = f4v{0.f, 0.f, 0.f, 0.f};
    }
    if (!a.delta_out) return;                         // uniform
    const int u = c0 / 32;
    char* unit = static_cast<char*>(a.delta_out) + (size_t)q * delta_row_bytes(COUT) + u * UNIT_BYTES +
                 (c0 % 32) * 2 + g * 8;
    if constexpr (BF16) {
#pragma unroll
        for (int i = 0; i < NBL; ++i) {
            uint2 pn, po;
            pn.x = f32_to_bf16_bits(yn[i].x) | (f32_to_bf16_bits(yn[i].y) << 16);
            pn.y = f32_to_bf16_bits(yn[i].z) | (f32_to_bf16_bits(yn[i].w) << 16);
            po.x = f32_to_bf16_bits(yo[i].x) | (f32_to_bf16_bits(yo[i].y) << 16);
            po.y = f32_to_bf16_bits(yo[i].z) | (f32_to_bf16_bits(yo[i].w) << 16);
            if (store) {
                *reinterpret_cast<uint2*>(unit + i * 32) = pn;
                *reinterpret_cast<uint2*>(unit + 64 + i * 32) = po;
            }
        }
    } else {
        f4v dy[NBL];
        uint32_t mb = 0u;
#pragma unroll
        for (int i = 0; i < NBL; ++i) {
#pragma unroll
            for (int k = 0; k < 4; ++k) dy[i][k] = yn[i][k] - yo[i][k];
            mb = max(mb, abs_bits4(dy[i]));
        }
        mb = max(mb, (uint32_t)__shfl_xor((int)mb, 16));
        mb = max(mb, (uint32_t)__shfl_xor((int)mb, 32));
        const UnitScale us = unit_scale(mb);
#pragma unroll
        for (int i = 0; i < NBL; ++i) store_split4<COUT>(unit + i * 32, dy[i], us, store);
        if (store && g == 0) a.scale_out[(size_t)q * units_of(COUT) + u] = us.inv;
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
