// One convolution layer of a stride, on the changed cells only.
//
// Method (SSCATeR, arXiv 2512.08557, Eq. 2 and Alg. 1 backbone part): every
// changed input site scatters (I_curr - I_prev) x W[m, n] into the persistent
// output map; the touched output sites form the layer's change list; the next
// layer's input delta at a changed site is phi(Z_new) - phi(Z_old).
//
// Dataflow on gfx950 (output-stationary, one launch per layer, no atomics on
// the maps):
//   * the change list A_l of this layer's OUTPUT grid was built by an earlier
//     launch (scatter rule), so every output cell that receives a scatter
//     contribution is known up front;
//   * a workgroup owns TM = 16 or 32 consecutive cells of one segment of A_l
//     and up to 64 output channels.  It writes the changed ones of the 9 x TM
//     input cells under the tile's taps to LDS, from the list entries' tap bits
//     (plan.h) or by their change stamps (an unchanged input reads the zero
//     row);
//   * the contraction D[cout x 32 cells] += W_t^T[cout x cin] . dY^T over the
//     9 taps x cin channels is split over the NW wavefronts of the workgroup
//     by units of 32 channels of one tap: wavefront w takes the units w,
//     w + NW, ... for the whole TM x 64 tile.  No two wavefronts need the same
//     operand, so there is no barrier between the tile's table and its sums:
//     each loads its own weights straight into registers (packed in operand
//     order) and copies its own delta rows global->LDS asynchronously (an
//     operand's 16 rows lie 16 bytes per lane apart in memory, which the
//     vector memory path serves at a quarter of its rate; eight lanes per
//     128-byte unit go at the full rate).  The partial sums are added through
//     LDS in wavefront order.  Summing the 9 taps per output cell in a fixed order
//     is exactly the sum the scatter of Eq. 2 adds into that cell, so the
//     result is deterministic (it does not depend on the other cells of the
//     tile) and each Z row is read and written once per stride;
//   * up to 64 input channels (128 in bf16; STAT) a wavefront's weights stay in
//     its registers for all the tiles of its workgroup, loaded before the list
//     is known; wider layers stream them;
//   * epilogue in registers: Z_new = Z_old + D; store Z_new; write the next
//     layer's delta row at the cell;
//   * the next layer's change list (the structural rule, including stride-2
//     downsampling) is built by the launch's first workgroups (plan.h), or in
//     sparse backbones, where it depends on the active sets, by the tiles.
//
// MFMA operand layout (v_mfma_f32_16x16x32_f16 / _bf16):
//   src0 = weights, lane l supplies row cout = l%16, k = 8*(l/16) .. +7;
//   src1 = deltas,  lane l supplies cell l%16,       k = 8*(l/16) .. +7;
//   D: lane l, register j holds cout 4*(l/16)+j of cell l%16.
// A unit (32 channels, 128 bytes: two 64-byte planes, device_common.h) is
// exactly one such k range of both planes.
//   fp32: P = hi.Whi + hi.Wlo + lo.Whi over the unit, acc += P / s(unit);
//         the output channel's weight scale is applied once at the end;
//   bf16: acc += new.W - old.W (the sign bits of the old plane flipped:
//         exact), so the weights move once.
//
// What bounds it: at one sensor's sparsity the chain launch -> list entry ->
// stamps -> operands -> sums -> Z; on long lists the copies, at 64 bytes per
// clock and compute unit (a 32 x 64 tile of a 256-channel layer takes 864 KB,
// 5.8 us).  Measured per launch against what ran before (fp32 matrix
// instructions; the wide layers as a contraction plus a tap sum), 432x496
// backbone, ~4300 / 2300 / 1000 output cells: 64->64 11.5 -> 6.8 us, 128->128
// 9.9 + 5.8 -> 10.0, 256->256 14.5 + 5.6 -> 13.9; the first window (all cells)
// 48 -> 27, 38 + 20 -> 30.5, 40 + 10 -> 27.7; four 1024x1024 images 64->64
// 70.7 -> 37.7.  With the
// same tile as a workgroup-wide ring of LDS stages instead (both operands
// shared, a barrier per stage) a 256->256 launch took 21.9 us, and with the
// delta rows loaded in operand order straight into registers 17.6.
//
// Sparse backbones (SPARSE = true): a site inactive in this and in the
// previous stride neither changes nor propagates; an inactive site's output is
// zero in the delta epilogue; the first layer of a block passes its sites'
// membership changes to the next block's active-set counts (SPREAD).  Z is
// updated at every site of the list, active or not, so a site that joins the
// active set already holds its sum.
#include "plan.h"

#include <algorithm>

namespace ssc {

template <int CIN, int COUT, bool BF16, int TM = 32>
struct LayerShape {
    static constexpr int U = units_of(CIN);              // units of a delta row
    static constexpr int MH = TM / 16;
    static constexpr int CPU = TM / 8;                   // copies of a unit (1 KB each)
    static constexpr int ROWB = U * UNIT_BYTES;
    static constexpr int NT = COUT >= 64 ? 64 : (COUT + 15) / 16 * 16;   // output channels per workgroup
    static constexpr int NBN = COUT > 64 ? COUT / 64 : 1;                // workgroups per tile
    static constexpr int NB = NT / 16;                   // 16-channel blocks
    static constexpr int PL = BF16 ? 1 : 2;              // weight planes
    static constexpr int WU = NT * 64 * PL;              // bytes of a weight unit
    static constexpr int NU = 9 * U;                     // units of a tile
    static constexpr int NW = U >= 4 ? 8 : 6;            // wavefronts
    static constexpr int CNT = (NU + NW - 1) / NW;       // units of a wavefront, at most
    static constexpr int FULL = NU / NW;                 // units every wavefront has
    static constexpr bool STAT = U <= (BF16 ? 4 : 2);    // weights stay in registers
    static constexpr int D = CNT < 3 ? CNT : 3;          // units whose loads are in flight
    // vector loads certainly issued after the copies of unit i and before it
    // is awaited: the copies of the next D - 1 units and the streamed weights
    // of those of them that every wavefront has (the weights of the first D
    // units come before all copies; a unit's own weights and those of a unit
    // that only some wavefronts compute are not counted, the compiler may place
    // them on either side of the wait).  A smaller count waits for more.
    static constexpr int younger(int i) {
        int n = 0;
        for (int j = i + 1; j < i + D && j < CNT; ++j) n += CPU + (!STAT && j >= D && j < FULL ? PL * NB : 0);
        return n;
    }
    static constexpr int MAXW = (D - 1) * (CPU + PL * NB);
    // finishing wavefronts: 16 cells and one unit of output channels each (all
    // the channels of a tile of fewer than 64)
    static constexpr int OB = NB == 4 ? 2 : NB;          // blocks
    static constexpr int FW = MH * (NB / OB);
    static constexpr int SLOT = TM * UNIT_BYTES;         // a wavefront's unit in LDS
    static constexpr int SB = SLOT / 1024;               // blocks of partial sums that fit in it
    static constexpr int PLAN_LDS = PLAN_IN * 4 + PLAN_WORDS * (int)sizeof(PlanWord);
};

// The tiles of TM cells of one workgroup; b: its number among the grid's
// workgroups that walk tiles, nwg: how many those are.
template <int CIN, int COUT, int S, bool BF16, bool SPARSE, bool SPREAD, int TM>
__device__ __forceinline__ void layer_tiles(const int32_t* __restrict__ plist, const uint16_t* __restrict__ ptaps,
                                            const char* __restrict__ pweights, int pcap, int n0, int n1, int b, int nwg,
                                            const LayerArgs& a) {
    using L = LayerShape<CIN, COUT, BF16, TM>;
    constexpr int U = L::U, NB = L::NB, NBN = L::NBN, OB = L::OB, NW = L::NW, CNT = L::CNT, D = L::D, PL = L::PL;
    constexpr int NTH = 64 * NW, MH = L::MH, SLOT = L::SLOT, SB = L::SB;
    static_assert(9 * TM <= NTH, "one table entry per thread");
    __shared__ int rowcell[9][TM];                                      // changed input cell, or -1
    __shared__ __attribute__((aligned(16))) uint16_t rowsc[BF16 ? 1 : 9][TM][U];     // its units' 1/s (bf16), or 0
    // the wavefronts' delta units in flight (one LDS array per slot: the
    // compiler then tracks the copies into each slot separately); at the end
    // slots 0 and 1 take the partial sums
    __shared__ __attribute__((aligned(1024))) char as0[NW * SLOT];
    __shared__ __attribute__((aligned(1024))) char as1[NW * SLOT];
    __shared__ __attribute__((aligned(1024))) char as2[D > 2 ? NW * SLOT : 16];
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cl = lane & 15, g = lane >> 4;

    // workgroup b runs on XCD b % 8: an XCD's workgroups share one group of 64
    // output channels, so its L2 holds that group's weights only; segment and
    // tile follow
    const int xcd = b & 7, nb = xcd % NBN, idx = b >> 3;
    const int shard = idx & 1;
    const int GT = nwg / (2 * NBN);
    int tile = (idx >> 1) * (8 / NBN) + xcd / NBN;
    const int32_t* seg = plist + (size_t)shard * pcap;
    const int n = shard ? n1 : n0;

    // the finishing role of this wavefront: cells 16*fm.., channels c0..
    const int fm = w % MH, fb = w / MH * OB;
    const bool fin = w < L::FW;
    const bool lead = SPARSE && nb == 0 && w < MH;       // propagates its 16 cells
    const int c0 = nb * 64 + fb * 16;

    // table entry of this thread
    const int tr = tid % TM, tt = tid / TM;
    const uint16_t* tseg = ptaps ? ptaps + (size_t)shard * pcap : nullptr;
    int qt = seg[min(tile * TM + tr, pcap - 1)];
    uint32_t mk = tseg ? tseg[min(tile * TM + tr, pcap - 1)] : 0u;

    // copies: lane l takes the 16-byte piece of row 8k + l/8 that belongs in
    // slot l % 8 of it (piece ^ (row / 2) % 8: the 16 rows read together then
    // fall in different banks); reads: rows 16m + cl, piece g of either plane
    const int cr = lane >> 3;
    const uint32_t cp0 = (uint32_t)(((lane & 7) ^ (cr >> 1)) * 16), cp1 = cp0 ^ 64u;   // even and odd k
    const int sa = (cl >> 1) & 7;
    int a_hi = w * SLOT + cl * UNIT_BYTES + ((g ^ sa) << 4), a_lo = a_hi ^ 64;
    // (single values: the compiler's copy tracking follows only a short
    // address chain from the slot's array)
    asm("" : "+v"(a_hi), "+v"(a_lo));
    auto slot = [&](int k) -> lds_char* { return (lds_char*)(k == 0 ? as0 : (k == 1 ? as1 : as2)); };
    const char* dbase = static_cast<const char*>(a.delta_in);
    const char* zrow = static_cast<const char*>(a.zero);
    const char* wbase = pweights + (size_t)nb * L::NU * L::WU;   // uniform
    const uint32_t wl16 = (uint32_t)lane * 16u;
    // weights of unit un
    auto load_w = [&](int un, uint4 (&bw)[PL * NB]) __attribute__((always_inline)) {
        const char* p = wbase + (size_t)un * L::WU;
#pragma unroll
        for (int k = 0; k < PL * NB; ++k) bw[k] = *reinterpret_cast<const uint4*>(p + k * 1024 + wl16);
    };
    // unit i of wavefront ww (a wavefront without an i-th unit loads the last)
    auto unit = [&](int ww, int i) __attribute__((always_inline)) { return min(ww + NW * i, L::NU - 1); };
    constexpr int NBUF = L::STAT ? CNT : D;
    uint4 bw[NBUF][PL * NB];
    if (tile * TM < n) {
#pragma unroll
        for (int i = 0; i < NBUF; ++i) load_w(unit(w, i), bw[i]);
    }

    if (a.cum_dst && b == 0)
        for (int i = tid; i < a.n_cum; i += NTH) a.cum_dst[(size_t)i * CSTRIDE] += a.cum_src[(size_t)i * CSTRIDE];

    for (; tile * TM < n; tile += GT) {
        const int t0 = tile * TM;
        // (opaque: what follows from it is computed where it is used, not
        // kept in registers over all tiles)
        int wt = w;
        asm volatile("" : "+s"(wt));
        const int ef = t0 + 16 * fm + cl;                // the lane's cell of the epilogue
        const int qf = seg[min(ef, n - 1)];
        const bool vt = t0 + tr < n, vrow = ef < n;
        const int q = qf;                                // a valid cell also past the segment's end

        // this thread's input cell, whether it changed, and its units' scales
        // (loads from clamped, always valid addresses)
        const int q0 = __builtin_amdgcn_readfirstlane(qt);   // row 0, always valid
        const int p = vt ? qt : q0;
        int cell = 0;
        bool ch = vt && tt < 9;
        uint32_t ev = a.epoch;
        const int dr = tt / 3 - 1, dc = tt - 3 * (tt / 3) - 1;
        if (S == 1 && tseg) {
            ch = ch && ((mk >> tt) & 1u);
            cell = ch ? p + dr * a.Win + dc : p;
        } else {
            const int img = (int)a.dimg((uint32_t)p), pl = p - img * (a.Hout * a.Wout);
            const int pr = (int)a.drow((uint32_t)pl), pc = pl - pr * a.Wout;
            const int ir = S * pr + dr, ic = S * pc + dc;
            ch = ch && ir >= 0 && ir < a.Hin && ic >= 0 && ic < a.Win;
            if (tseg) ch = ch && ((mk >> tt) & 1u);
            cell = img * (a.Hin * a.Win) + min(max(ir, 0), a.Hin - 1) * a.Win + min(max(ic, 0), a.Win - 1);
            if (!tseg) ev = a.stamp_in[cell];
        }
        uint32_t sc[BF16 ? 1 : (U + 1) / 2];
        if constexpr (!BF16) {
            const uint16_t* sp = a.scale_in + (size_t)cell * U;
            if constexpr (U == 1) {
                sc[0] = *sp;
            } else {
#pragma unroll
                for (int i = 0; i < U / 2; ++i) sc[i] = reinterpret_cast<const uint32_t*>(sp)[i];
            }
        }
        f4v zo[OB], wsc[OB];
        // sparse backbones: only a site active now or before can change, and
        // only such sites go to the next layer's list
        bool now = true, prev = true;
        PropBatch<4> pb;
        MembBatch mbt;
        if (fin) {
#pragma unroll
            for (int i = 0; i < OB; ++i) {
                const int co = min(c0 + i * 16 + 4 * g, COUT - 4);
                zo[i] = *reinterpret_cast<const f4v*>(a.Z + (size_t)q * COUT + co);
                if constexpr (!BF16) wsc[i] = *reinterpret_cast<const f4v*>(a.wscale + co);
            }
            if constexpr (SPARSE) {
                const uint64_t mw = a.memb[q];
                now = memb_now(mw);
                prev = memb_prev(mw, a.epoch);
            }
        }
        ch = ch && ev == a.epoch;
        if (tt < 9) rowcell[tt][tr] = ch ? cell : -1;
        auto put_scales = [&]() __attribute__((always_inline)) {
            if constexpr (!BF16) {
                if (tt < 9) {
                    uint16_t* sp = &rowsc[tt][tr][0];
                    if constexpr (U == 1) {
                        *sp = ch ? (uint16_t)sc[0] : 0;
                    } else {
#pragma unroll
                        for (int i = 0; i < U / 2; ++i) reinterpret_cast<uint32_t*>(sp)[i] = ch ? sc[i] : 0u;
                    }
                }
            }
        };
        if constexpr (SPARSE) put_scales();              // they came with the stamps
        // the next tile's entry
        qt = seg[min((tile + GT) * TM + tr, pcap - 1)];
        if (tseg) mk = tseg[min((tile + GT) * TM + tr, pcap - 1)];
        lds_barrier();

        // delta units of the 32 rows
        auto load_a = [&](int i, lds_char* st) __attribute__((always_inline)) {
            const int un = unit(wt, i), t = un / U, u = un - t * U;
#pragma unroll
            for (int k = 0; k < L::CPU; ++k) {
                const int rc = rowcell[t][8 * k + cr];
                const char* src = rc >= 0 ? dbase + (size_t)rc * L::ROWB + u * UNIT_BYTES : zrow;
                copy16(src + (k & 1 ? cp1 : cp0), st + wt * SLOT + k * 1024);
            }
        };
#pragma unroll
        for (int i = 0; i < D; ++i) load_a(i, slot(i));
        if constexpr (!BF16 && !SPARSE) {                // the scales arrive while the copies are in flight
            put_scales();
            lds_barrier();
        }
        // sparse: the next layer's footprint stamps go out behind the first
        // operands, its list positions are taken once those have arrived (the
        // counter's round trip overlaps the contraction); a regular layer
        // followed by another one (SPREAD) loads the next regular layer's
        // words of the sites whose activity flips now, so that only their
        // swaps end the tile
        if (lead && a.has_next) prop_issue<4, false>(a.next, q, vrow && (now || prev), g, a.epoch, pb);
        if (SPREAD && lead) memb_issue(a.mnext, q, a.Hout, a.Wout, g == 0 && vrow && now != prev, mbt);
        PropSlots<4> ps;

        f4v acc[MH][NB];
#pragma unroll
        for (int m = 0; m < MH; ++m)
#pragma unroll
            for (int i = 0; i < NB; ++i) acc[m][i] = f4v{0.f, 0.f, 0.f, 0.f};
        auto compute = [&](int i, const lds_char* st, const uint4 (&bv)[PL * NB]) __attribute__((always_inline)) {
            const int un = unit(wt, i), t = un / U, u = un - t * U;
            uint4 av[2 * MH];
#pragma unroll
            for (int m = 0; m < MH; ++m) {
                av[2 * m] = lds16(st + a_hi + m * 2048);
                av[2 * m + 1] = lds16(st + a_lo + m * 2048);
            }
#pragma unroll
            for (int m = 0; m < MH; ++m) {
                if constexpr (BF16) {
                    const uint4 v = av[2 * m], o = av[2 * m + 1];
                    const uint32_t sg = 0x80008000u;
                    const uint4 ov = make_uint4(o.x ^ sg, o.y ^ sg, o.z ^ sg, o.w ^ sg);
                    bf8v A, O, B;
                    __builtin_memcpy(&A, &v, 16);
                    __builtin_memcpy(&O, &ov, 16);
#pragma unroll
                    for (int k = 0; k < NB; ++k) {
                        __builtin_memcpy(&B, &bv[k], 16);
                        acc[m][k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(B, A, acc[m][k], 0, 0, 0);
                    }
#pragma unroll
                    for (int k = 0; k < NB; ++k) {
                        __builtin_memcpy(&B, &bv[k], 16);
                        acc[m][k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(B, O, acc[m][k], 0, 0, 0);
                    }
                } else {
                    const float s = bf16_to_f32(rowsc[t][16 * m + cl][u]);
                    h8v A, O, B;
                    __builtin_memcpy(&A, &av[2 * m], 16);
                    __builtin_memcpy(&O, &av[2 * m + 1], 16);
                    f4v P[NB];
#pragma unroll
                    for (int k = 0; k < NB; ++k) {
                        __builtin_memcpy(&B, &bv[NB + k], 16);
                        P[k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(B, A, f4v{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                    }
#pragma unroll
                    for (int k = 0; k < NB; ++k) {
                        __builtin_memcpy(&B, &bv[k], 16);
                        P[k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(B, O, P[k], 0, 0, 0);
                    }
#pragma unroll
                    for (int k = 0; k < NB; ++k) {
                        __builtin_memcpy(&B, &bv[k], 16);
                        P[k] = __builtin_amdgcn_mfma_f32_16x16x32_f16(B, A, P[k], 0, 0, 0);
                    }
#pragma unroll
                    for (int k = 0; k < NB; ++k)
#pragma unroll
                        for (int j = 0; j < 4; ++j) acc[m][k][j] = fmaf(P[k][j], s, acc[m][k][j]);
                }
            }
        };
#pragma unroll
        for (int i = 0; i < CNT; ++i) {
            // this wavefront's copies of the unit have landed: everything but
            // what was issued after them (the younger units' copies and
            // weights; more than that in flight only waits for more).  What
            // is read below rests on this count, whatever waits the compiler
            // adds for the LDS reads
            wait_vm_n<L::MAXW>(L::younger(i));
            asm volatile("" ::: "memory");
            if constexpr (!L::STAT)
                if (i >= L::FULL) {
                    // a use outside the branch: the loads of a unit that only
                    // some wavefronts compute stay where they were issued
#pragma unroll
                    for (int k = 0; k < PL * NB; ++k) pin(bw[i % D][k]);
                }
            if (i < L::FULL || wt + NW * i < L::NU) compute(i, slot(i % D), bw[L::STAT ? i : i % D]);
            if (i + D < CNT) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the slot has been read
                load_a(i + D, slot(i % D));
                if constexpr (!L::STAT) load_w(unit(wt, i + D), bw[i % D]);
            }
            if (i == 0 && lead && a.has_next) prop_reserve<4>(a.next, a.epoch, shard, pb, ps);
            // keep the scheduler from hoisting later loads past this unit
            __builtin_amdgcn_sched_barrier(0);
        }

        // partial sums, added in wavefront order by the finishing wavefronts
        auto red = [&](int ww, int j) __attribute__((always_inline)) {   // block j of wavefront ww
            return reinterpret_cast<f4v*>((j / SB == 0 ? as0 : as1) + ww * SLOT + (j % SB) * 1024) + lane;
        };
        static_assert(MH * NB <= 2 * SB, "partial sums");
#pragma unroll
        for (int m = 0; m < MH; ++m)
#pragma unroll
            for (int k = 0; k < NB; ++k) *red(w, m * NB + k) = acc[m][k];
        lds_barrier();
        if (fin) {
            f4v d[OB];
#pragma unroll
            for (int i = 0; i < OB; ++i) {
                const int j = fm * NB + fb + i;
                d[i] = *red(0, j);
#pragma unroll
                for (int k = 1; k < NW; ++k) {
                    const f4v x = *red(k, j);
#pragma unroll
                    for (int e = 0; e < 4; ++e) d[i][e] += x[e];
                }
                if constexpr (!BF16)
#pragma unroll
                    for (int j = 0; j < 4; ++j) d[i][j] *= wsc[i][j];
            }
            epilogue_unit<COUT, BF16, OB>(a, q, c0, g, zo, d, vrow && (COUT % 16 == 0 || 4 * g < COUT), now, prev);
        }
        if (SPREAD && lead) memb_finish(a.mnext, q, a.Hout, a.Wout, mbt, now ? 1 : -1, a.epoch);
        if (lead && a.has_next) prop_write<4>(a.next, shard, pb, ps);
        // the next tile's table may be written now (its barrier orders the
        // sums: a wavefront writes red only after the barrier that every
        // finishing wavefront reaches after reading it)
        if constexpr (!L::STAT) {
            if ((tile + GT) * TM < n) {
#pragma unroll
                for (int i = 0; i < D; ++i) load_w(unit(wt, i), bw[i]);
            }
        }
    }
}

// The leading scalar arguments repeat what the struct holds: the build preloads
// them into SGPRs, so that the loads that open every tile (list entries, tap
// bits, counts, weights) and the branch to the plan need not wait for the
// argument fetch, a round trip of its own.
//
// Tile height: 32 cells, so that a tile's share of the weights is small; up to
// 64 input channels 16 where the list then still has a workgroup for every
// tile, on twice the compute units with half the operands and sums each.
// Measured on a 432x496 stride, 16 against 32 cells: 64->128 stride-2 launch
// (45 32-cell tiles) 6.3 against 7.7 us, 64->64 (100 to 140 tiles) 7.0 against
// 8.0 us; on lists of more tiles than workgroups 16 cells lose (four 1024x1024
// images, 1500 tiles: 45 against 33 us, two workgroups per compute unit).
template <int CIN, int COUT, int S, bool BF16, bool SPARSE, bool SPREAD>
__global__ __launch_bounds__((64 * LayerShape<CIN, COUT, BF16>::NW)) void layer_kernel(
    const int32_t* __restrict__ plist, const int32_t* __restrict__ pcount, const uint16_t* __restrict__ ptaps,
    const char* __restrict__ pweights, int pcap, int pplan, LayerArgs a) {
    using L = LayerShape<CIN, COUT, BF16>;
    if constexpr (!SPARSE) {
        if ((int)blockIdx.x < pplan) {
            __shared__ __attribute__((aligned(16))) char planlds[L::PLAN_LDS];
            __shared__ int plansum[2 * L::NW + 2];
            plan_tile<L::NW>(a.plan, a.epoch, (int)blockIdx.x, reinterpret_cast<uint32_t*>(planlds),
                             reinterpret_cast<PlanWord*>(planlds + PLAN_IN * 4), plansum);
            return;
        }
    }
    const int nplan = SPARSE ? 0 : pplan;
    const int b = (int)blockIdx.x - nplan, nwg = (int)gridDim.x - nplan;
    const int n0 = pcount[0], n1 = pcount[CSTRIDE];
    if constexpr (L::U <= 2) {
        if (max(n0, n1) <= 16 * (nwg / (2 * L::NBN))) {
            layer_tiles<CIN, COUT, S, BF16, SPARSE, SPREAD, 16>(plist, ptaps, pweights, pcap, n0, n1, b, nwg, a);
            return;
        }
    }
    layer_tiles<CIN, COUT, S, BF16, SPARSE, SPREAD, 32>(plist, ptaps, pweights, pcap, n0, n1, b, nwg, a);
}

// ---------------------------------------------------------------------------
// instantiation table
// ---------------------------------------------------------------------------
// (a build may give a shorter table of its own)
#ifndef SSC_ALL_SHAPES
#define SSC_CH_LIST(X, CIN, S) X(CIN, 8, S) X(CIN, 16, S) X(CIN, 32, S) X(CIN, 64, S) X(CIN, 128, S) X(CIN, 256, S)
#define SSC_ALL_SHAPES(X)                                                                            \
    SSC_CH_LIST(X, 16, 1) SSC_CH_LIST(X, 32, 1) SSC_CH_LIST(X, 64, 1) SSC_CH_LIST(X, 128, 1)         \
    SSC_CH_LIST(X, 256, 1) SSC_CH_LIST(X, 16, 2) SSC_CH_LIST(X, 32, 2) SSC_CH_LIST(X, 64, 2)         \
    SSC_CH_LIST(X, 128, 2) SSC_CH_LIST(X, 256, 2)
#endif

bool layer_supported(int cin, int cout, int stride, bool /*bf16*/) {
#define SSC_SUP(CI, CO, S) if (cin == CI && cout == CO && stride == S) return true;
    SSC_ALL_SHAPES(SSC_SUP)
#undef SSC_SUP
    return false;
}

template <int CI, int CO, int S, bool BF16, bool SPARSE>
static hipError_t launch_shape(const LayerArgs& a, const LaunchCtx& c) {
    using L = LayerShape<CI, CO, BF16>;
    // one workgroup per compute unit (a longer list loops over its remaining
    // tiles), at most the tiles of a full list
    const long long most = ((long long)a.cap + 15) / 16 * 2 * L::NBN;
    const int grid = (int)std::max(16LL, std::min(256LL, (most + 15) / 16 * 16)) + (SPARSE ? 0 : a.plan.wgs);
    const int plan = SPARSE ? 0 : a.plan.wgs;
    const char* w = static_cast<const char*>(a.wpack);
    if constexpr (SPARSE)
        if (a.mnext.memb)
            return launch_kernel(c, layer_kernel<CI, CO, S, BF16, true, true>, dim3(grid), dim3(64 * L::NW), a.list,
                                 a.count, a.taps, w, a.cap, plan, a);
    return launch_kernel(c, layer_kernel<CI, CO, S, BF16, SPARSE, false>, dim3(grid), dim3(64 * L::NW), a.list, a.count,
                         a.taps, w, a.cap, plan, a);
}

hipError_t launch_layer(const LayerArgs& a, int cin, int cout, int stride, bool bf16, bool sparse, const LaunchCtx& c) {
#define SSC_LAUNCH(CI, CO, S)                                                                               \
    if (cin == CI && cout == CO && stride == S) {                                                           \
        if (sparse)                                                                                         \
            return bf16 ? launch_shape<CI, CO, S, true, true>(a, c) : launch_shape<CI, CO, S, false, true>(a, c); \
        return bf16 ? launch_shape<CI, CO, S, true, false>(a, c) : launch_shape<CI, CO, S, false, false>(a, c);  \
    }
    SSC_ALL_SHAPES(SSC_LAUNCH)
#undef SSC_LAUNCH
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// weight repacking (device; the caller's weights uploaded as they are)
// ---------------------------------------------------------------------------
// Both kernels' packed weights: [output groups][unit][plane][block of 16
// output channels][lane l][8], lane l holding output channel l%16 of the block
// and the unit's input channels 8*(l/16) .. +7 (zero past cin, except as
// device_common.h says for 16 fp32 channels).  bf16: one
// plane (two for an upsampler: W and -W, an exact sign flip); fp32: the hi
// plane, then the lo plane, of the weights scaled per output channel by the
// power of two that brings the largest into [2^14, 2^15), as delta units are;
// scale[co] is its inverse (or the NaN or infinity among the weights).

// One wavefront per output channel: the scale of its n weights, the j-th at
// w[(j / run) * step + co * run + j % run] (run consecutive values each).
__global__ __launch_bounds__(64) void weight_scale_kernel(const float* __restrict__ w, int n, int run, int step,
                                                          float* __restrict__ fwd, float* __restrict__ inv) {
    const int co = (int)blockIdx.x;
    uint32_t mb = 0u;
    for (int j = (int)threadIdx.x; j < n; j += 64)
        mb = max(mb, __float_as_uint(w[(size_t)(j / run) * step + (size_t)co * run + j % run]) & 0x7FFFFFFFu);
#pragma unroll
    for (int k = 1; k < 64; k <<= 1) mb = max(mb, (uint32_t)__shfl_xor((int)mb, k));
    if (threadIdx.x == 0) {
        const UnitScale u = unit_scale(mb);
        fwd[co] = u.finite ? u.s : 0.f;
        inv[co] = bf16_to_f32(u.inv);
    }
}

// Plane values at input channel k of a unit (k = 0..31) of an fp32 weight w
// under its channel's scale s (0: the channel holds a value that is not
// finite).  cin = 16: k >= 16 stands for channel k - 16 (device_common.h).
__device__ __forceinline__ void split_weight(float w, float s, bool upper, uint16_t& p0, uint16_t& p1) {
    const UnitScale u{s, 0, s != 0.f};
    _Float16 hi, lo, rest;
    split1(w, u, hi, lo, rest);
    const _Float16 a = upper ? rest : hi, b = upper ? hi : lo;
    __builtin_memcpy(&p0, &a, 2);
    __builtin_memcpy(&p1, &b, 2);
}

// OIHW [cout][cin][3][3]; groups of up to 64 output channels, units [tap][32
// input channels].  One thread per packed position of a plane; positions of no
// channel (cout = 8, cin = 16) keep the buffer's zeros.
__global__ __launch_bounds__(256) void pack_weights_kernel(const void* __restrict__ w, int cin, int cout, int bf16,
                                                           const float* __restrict__ fwd, uint16_t* __restrict__ out) {
    const int nu = units_of(cin), coutp = (cout + 15) / 16 * 16, nt = min(coutp, 64);
    const int plane = nt * 32;                            // values of a plane of a unit
    const int n = 9 * nu * coutp * 32;
    for (int i = (int)(blockIdx.x * 256 + threadIdx.x); i < n; i += (int)gridDim.x * 256) {
        const int e = i & 7, l = (i >> 3) & 63, blk = i % plane / 512, ug = i / plane;   // ug: group and unit
        const int group = ug / (9 * nu), un = ug - group * (9 * nu), t = un / nu, u = un - t * nu;
        const int co = group * nt + blk * 16 + (l & 15);
        int ci = u * 32 + (l >> 4) * 8 + e;
        const bool upper = !bf16 && cin == 16 && ci >= 16;
        if (upper) ci -= 16;
        if (co >= cout || ci >= cin) continue;
        const size_t from = ((size_t)co * cin + ci) * 9 + t;
        const size_t to = (size_t)ug * plane * (bf16 ? 1 : 2) + (i % plane);
        if (bf16) out[to] = static_cast<const uint16_t*>(w)[from];
        else split_weight(static_cast<const float*>(w)[from], fwd[co], upper, out[to], out[to + plane]);
    }
}

// [cin][cout][S][S]; one group, units [32 input channels], blocks [sub-cell
// a*S + b][16 output channels].
__global__ __launch_bounds__(256) void pack_up_weights_kernel(const void* __restrict__ w, int cin, int cout, int s2,
                                                              int bf16, const float* __restrict__ fwd,
                                                              uint16_t* __restrict__ out) {
    const int ncbt = cout / 16, plane = s2 * cout * 32;
    const int n = units_of(cin) * plane;
    for (int i = (int)(blockIdx.x * 256 + threadIdx.x); i < n; i += (int)gridDim.x * 256) {
        const int e = i & 7, l = (i >> 3) & 63, ob = i % plane / 512, u = i / plane;
        const int ab = ob / ncbt, co = (ob - ab * ncbt) * 16 + (l & 15);
        int ci = u * 32 + (l >> 4) * 8 + e;
        const bool upper = !bf16 && cin == 16 && ci >= 16;
        if (upper) ci -= 16;
        if (ci >= cin) continue;
        const size_t from = ((size_t)ci * cout + co) * s2 + ab;
        const size_t to = (size_t)u * plane * 2 + (i % plane);
        if (bf16) {
            const uint16_t v = static_cast<const uint16_t*>(w)[from];
            out[to] = v;
            out[to + plane] = v ^ 0x8000u;
        } else {
            split_weight(static_cast<const float*>(w)[from], fwd[co], upper, out[to], out[to + plane]);
        }
    }
}

size_t wpack_bytes(int cin, int cout, bool bf16) {
    return (size_t)9 * units_of(cin) * (size_t)((cout + 15) / 16 * 16) * (bf16 ? 64 : 128);
}

size_t up_wpack_bytes(int cin, int cout, int stride) {
    return (size_t)units_of(cin) * 2 * (size_t)cout * stride * stride * 64;
}

static unsigned pack_grid(size_t values) { return (unsigned)std::min<size_t>(1024, (values + 255) / 256); }

hipError_t launch_pack_weights(const void* w, int cin, int cout, bool bf16, float* fwd, float* inv, void* out) {
    if (!bf16) hipLaunchKernelGGL(weight_scale_kernel, dim3(cout), dim3(64), 0, nullptr, static_cast<const float*>(w),
                                  9 * cin, 9 * cin, 0, fwd, inv);
    hipLaunchKernelGGL(pack_weights_kernel, dim3(pack_grid(wpack_bytes(cin, cout, true) / 2)), dim3(256), 0, nullptr, w,
                       cin, cout, bf16 ? 1 : 0, fwd, static_cast<uint16_t*>(out));
    return hipGetLastError();
}

hipError_t launch_pack_up_weights(const void* w, int cin, int cout, int stride, bool bf16, float* fwd, float* inv,
                                  void* out) {
    const int s2 = stride * stride;
    if (!bf16) hipLaunchKernelGGL(weight_scale_kernel, dim3(cout), dim3(64), 0, nullptr, static_cast<const float*>(w),
                                  cin * s2, s2, cout * s2, fwd, inv);
    hipLaunchKernelGGL(pack_up_weights_kernel, dim3(pack_grid(up_wpack_bytes(cin, cout, stride) / 4)), dim3(256), 0,
                       nullptr, w, cin, cout, s2, bf16 ? 1 : 0, fwd, static_cast<uint16_t*>(out));
    return hipGetLastError();
}

}  // namespace ssc
