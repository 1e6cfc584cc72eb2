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
//     downsampling) is built by the launch's first workgroups (plan.h), or by
//     the tiles: in sparse backbones, where it depends on the active sets, and
//     on very large grids (the host's plan_lists).
//
// MFMA operand layout (v_mfma_f32_16x16x32_bf16):
//   src0 = weights, lane l supplies row cout = l%16, k = 8*(l/16) .. +7;
//   src1 = deltas,  lane l supplies cell l%16,       k = 8*(l/16) .. +7;
//   D: lane l, register j holds cout 4*(l/16)+j of cell l%16.
// A unit (32 channels, 128 bytes) is one such k range, of which a lane reads
// the 16-byte pieces l/16 and 4 + l/16:
//   fp32: channels 4*(l/16) .. +3 and 16 more, split in registers into three
//         bf16 planes, six products (device_common.h);
//   bf16: acc += new.W - old.W (the sign bits of the old plane flipped:
//         exact), so the weights move once.
//
// What bounds it: at one sensor's sparsity the chain launch -> list entry ->
// stamps -> operands -> sums -> Z; on long lists the copies, at 64 bytes per
// clock and compute unit, and in fp32 the matrix instructions beside them (a
// 32 x 64 tile of a 256-channel fp32 layer takes 1.2 MB, 7.7 us, and 5.8 us of
// instructions).  Measured per fp32 launch against what ran before (fp32 matrix
// instructions; the wide layers as a contraction plus a tap sum), 432x496
// backbone, ~4300 / 2300 / 1000 output cells: 64->64 11.5 -> 7.8 us, 128->128
// 9.9 + 5.8 -> 10.6, 256->256 14.5 + 5.6 -> 14.2; the first window (all cells)
// 48 -> 28, 38 + 20 -> 31.4, 40 + 10 -> 34.1; four 1024x1024 images 64->64
// 70.7 -> 36.8.  Two fp16 planes and three products, which hold fewer bits
// (device_common.h), took 6.5, 9.9 and 13.4 us for the first three.  With the
// same tile as a workgroup-wide ring of LDS stages instead (both operands
// shared, a barrier per stage) a 256->256 launch took 8.5 us more, and with
// the delta rows loaded in operand order straight into registers 4.2.
//
// Sparse backbones (SPARSE = true, a.memb set): a site inactive in this and in the
// previous stride neither changes nor propagates; an inactive site's output is
// zero in the delta epilogue; the first layer of a block passes its sites'
// membership changes to the next block's active-set counts (SPREAD).  Z is
// updated at every site of the list, active or not, so a site that joins the
// active set already holds its sum.
#include "plan.h"

#include <algorithm>

namespace ssc {

typedef __attribute__((address_space(3))) f4v lds_f4v;

template <int CIN, int COUT, bool BF16, bool SPARSE, int TM = 32>
struct LayerShape {
    static constexpr int U = units_of(CIN);              // units of a delta row
    static constexpr int MH = TM / 16;
    static constexpr int CPU = TM / 8;                   // copies of a unit (1 KB each)
    static constexpr int ROWB = delta_row_bytes(CIN);
    static constexpr int NT = COUT >= 64 ? 64 : (COUT + 15) / 16 * 16;   // output channels per workgroup
    static constexpr int NBN = COUT > 64 ? COUT / 64 : 1;                // workgroups per tile
    static constexpr int NB = NT / 16;                   // 16-channel blocks
    static constexpr int PL = BF16 ? 1 : 3;              // weight planes
    static constexpr int WU = NT * 64 * PL;              // bytes of a weight unit
    static constexpr int NU = 9 * U;                     // units of a tile
    // wavefronts: 64 dense fp32 channels' 18 units leave a SIMD at most 5 of
    // them with 8 wavefronts, 6 with 6 (four 1024x1024 images 278 -> 270 us a
    // stride); the sparse kernels spill more registers with 8 (253 -> 259 us)
    static constexpr int NW = U >= 4 || (U == 2 && !BF16 && !SPARSE) ? 8 : 6;
    static constexpr int CNT = (NU + NW - 1) / NW;       // units of a wavefront, at most
    static constexpr int FULL = NU / NW;                 // units every wavefront has
    static constexpr bool STAT = U <= (BF16 ? 4 : 2);    // weights stay in registers
    // units whose copies are in flight (two where LDS takes eight wavefronts'
    // and a weight plane)
    static constexpr int D = U == 2 && !BF16 && !SPARSE ? 2 : (CNT < 3 ? CNT : 3);
    // units whose weights are: of three fp32 planes two units' are what the
    // registers hold beside the sums
    static constexpr int DW = STAT ? CNT : (BF16 || D < 2 ? D : 2);
    // 64 fp32 channels: the planes Wl of a wavefront's three units stay in LDS
    // (72 KB a workgroup), Wh and Wm in registers (96); five of the six
    // products are formed from those
    static constexpr bool WLDS = STAT && !BF16 && U == 2;
    static constexpr int RP = WLDS ? 2 : PL;             // weight planes in registers
    static constexpr int WL_LDS = WLDS ? NU * NB * 1024 : 16;
    // vector loads certainly issued after the copies of unit i, and after its
    // streamed weights, and before it is awaited: first the copies of units 0 ..
    // D - 1 (the weights of units 0 .. DW - 1 come before them), then, behind
    // each unit x, the copies of unit x + D and the streamed weights of unit
    // x + DW.  Weights of a unit that only some wavefronts compute are not
    // counted, the compiler may place them on either side of the wait.  A
    // smaller count waits for more.  The unit's weights are waited for with its
    // copies because the compiler's own wait for them, while copies are in
    // flight too, is for everything.
    static constexpr int younger(int i) {
        const bool own = !STAT && i >= DW;
        int n = 0;
        for (int j = i + 1; j < D && !own; ++j) n += CPU;
        for (int x = own ? i - DW + 1 : (i < D ? 0 : i - D); x < i; ++x) {
            if (x + D > i && x + D < CNT) n += CPU;
            if (!STAT && x + DW < FULL) n += PL * NB;
        }
        return n;
    }
    static constexpr int MAXW = (D - 1) * CPU + (STAT ? 0 : D * PL * NB);
    // finishing wavefronts: 16 cells and one unit of output channels each (all
    // the channels of a tile of fewer than 64)
    static constexpr int OB = NB == 4 ? 2 : NB;          // blocks
    static constexpr int FW = MH * (NB / OB);
    static constexpr int SLOT = TM * UNIT_BYTES;         // a wavefront's unit in LDS
    static constexpr int SB = SLOT / 1024;               // blocks of partial sums that fit in it
    // LDS of the workgroup: the plan and tiles of either height take the same
    static constexpr int AS = NW * SLOT, AS2 = D > 2 ? AS : 16;   // a slot of every wavefront
    static_assert(TM < 32 || (AS >= PLAN_IN * 4 && AS >= PLAN_WORDS * (int)sizeof(PlanWord)), "the plan fits");
};

// The tiles of TM cells of one workgroup; b: its number among the grid's
// workgroups that walk tiles, nwg: how many those are.
template <int CIN, int COUT, int S, bool BF16, bool SPARSE, bool SPREAD, int TM>
__device__ __forceinline__ void layer_tiles(const int32_t* __restrict__ plist, const uint16_t* __restrict__ ptaps,
                                            const char* __restrict__ pweights, int pcap, int n0, int n1, int b, int nwg,
                                            const LayerArgs& a, int (&rowcell)[9][32], lds_char* as0, lds_char* as1,
                                            lds_char* as2, lds_char* wl) {
    // rowcell: changed input cell, or -1.  as0, as1, as2: the wavefronts' delta
    // units in flight (one LDS array per slot: the compiler then tracks the
    // copies into each slot separately); at the end slots 0 and 1 take the
    // partial sums.  wl: weight planes (WLDS).
    using L = LayerShape<CIN, COUT, BF16, SPARSE, TM>;
    constexpr int U = L::U, NB = L::NB, NBN = L::NBN, OB = L::OB, NW = L::NW, CNT = L::CNT, D = L::D, PL = L::PL;
    constexpr int NTH = 64 * NW, MH = L::MH, SLOT = L::SLOT, SB = L::SB;
    constexpr int DW = L::DW, RP = L::RP;
    static_assert(9 * TM <= NTH, "one table entry per thread");
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
    uint32_t cp0 = (uint32_t)(((lane & 7) ^ (cr >> 1)) * 16), cp1 = cp0 ^ 64u;   // even and odd k
    // rows of 16 channels hold 64 bytes: fp32 reads pieces 0 to 3 only, bf16
    // pieces 0, 1 (new) and 4, 5 (old) with zeros in the others
    const bool half = BF16 && CIN < 32 && (cp0 & 32u) != 0u;
    if constexpr (CIN < 32) {
        cp0 = BF16 ? (cp0 & 64u) / 2 + (cp0 & 16u) : cp0 & 63u;
        cp1 = BF16 ? (cp1 & 64u) / 2 + (cp1 & 16u) : cp1 & 63u;
    }
    const int sa = (cl >> 1) & 7;
    int a_hi = w * SLOT + cl * UNIT_BYTES + ((g ^ sa) << 4), a_lo = a_hi ^ 64;
    // (single values: the compiler's copy tracking follows only a short
    // address chain from the slot's array)
    asm("" : "+v"(a_hi), "+v"(a_lo));
    auto slot = [&](int k) -> lds_char* { return k == 0 ? as0 : (k == 1 ? as1 : as2); };
    const char* dbase = static_cast<const char*>(a.delta_in);
    const char* zrow = static_cast<const char*>(a.zero);
    const char* wbase = pweights + (size_t)nb * L::NU * L::WU;   // uniform
    const uint32_t wl16 = (uint32_t)lane * 16u;
    // weights of unit un
    auto load_w = [&](int un, uint4 (&bw)[RP * NB]) __attribute__((always_inline)) {
        const char* p = wbase + (size_t)un * L::WU;
#pragma unroll
        for (int k = 0; k < RP * NB; ++k) bw[k] = *reinterpret_cast<const uint4*>(p + k * 1024 + wl16);
    };
    // unit i of wavefront ww (a wavefront without an i-th unit loads the last)
    auto unit = [&](int ww, int i) __attribute__((always_inline)) { return min(ww + NW * i, L::NU - 1); };
    uint4 bw[DW][RP * NB];
    if (tile * TM < n) {
#pragma unroll
        for (int i = 0; i < DW; ++i)
            if (!L::STAT || i < L::FULL || w + NW * i < L::NU) load_w(unit(w, i), bw[i]);
        if constexpr (L::WLDS) {
#pragma unroll
            for (int i = 0; i < CNT; ++i)
                if (i < L::FULL || w + NW * i < L::NU)
#pragma unroll
                    for (int k = 0; k < NB; ++k)
                        copy16(wbase + (size_t)unit(w, i) * L::WU + (2 * NB + k) * 1024 + wl16,
                               wl + (unit(w, i) * NB + k) * 1024);
        }
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
        const int q = seg[min(ef, n - 1)];               // a valid cell also past the segment's end
        const bool vt = t0 + tr < n, vrow = ef < n;

        // this thread's input cell and whether it changed (loads from clamped,
        // always valid addresses)
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
        f4v zo[OB];
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
            }
            if constexpr (SPARSE)
                if (a.memb) {                            // uniform
                    const uint64_t mw = a.memb[q];
                    now = memb_now(mw);
                    prev = memb_prev(mw, a.epoch);
                }
        }
        ch = ch && ev == a.epoch;
        if (tt < 9) rowcell[tt][tr] = ch ? cell : -1;
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
                const char* src = rc >= 0 && !half ? dbase + (size_t)rc * L::ROWB + u * UNIT_BYTES : zrow;
                copy16(src + (k & 1 ? cp1 : cp0), st + wt * SLOT + k * 1024);
            }
        };
#pragma unroll
        for (int i = 0; i < D; ++i) load_a(i, slot(i));
        // sparse: the next layer's footprint stamps go out behind the first
        // operands, its list positions are taken once those have arrived (the
        // counter's round trip overlaps the contraction); a regular layer
        // followed by another one (SPREAD) loads the next regular layer's
        // words of the sites whose activity flips now, so that only their
        // swaps end the tile (bf16; in fp32 the 18 registers would spill over
        // the contraction, so they are loaded behind it: the sparse backbone's
        // stride is the same either way, 234 us)
        if (lead && a.has_next) prop_issue<4>(a.next, q, vrow && (now || prev), g, a.epoch, pb);
        if (BF16 && SPREAD && lead) memb_issue(a.mnext, q, a.Hout, a.Wout, g == 0 && vrow && now != prev, mbt);
        PropSlots<4> ps;

        f4v acc[MH][NB];
        auto clear_sums = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int m = 0; m < MH; ++m)
#pragma unroll
                for (int i = 0; i < NB; ++i) acc[m][i] = f4v{0.f, 0.f, 0.f, 0.f};
        };
        clear_sums();
        auto compute = [&](int i, const lds_char* st, const uint4 (&bv)[RP * NB]) __attribute__((always_inline)) {
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
                    uint4 w3[NB];
#pragma unroll
                    for (int k = 0; k < NB; ++k) {
                        if constexpr (L::WLDS) w3[k] = lds16(wl + (unit(wt, i) * NB + k) * 1024 + wl16);
                        else w3[k] = bv[2 * NB + k];
                    }
                    mfma_unit<CIN, NB, false>(acc[m], bv, bv + NB, w3,
                                              split_unit<CIN, false>(av[2 * m], av[2 * m + 1]));
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
                    for (int k = 0; k < PL * NB; ++k) pin(bw[i % DW][k]);
                }
            if (i < L::FULL || wt + NW * i < L::NU) compute(i, slot(i % D), bw[i % DW]);
            if (i + D < CNT) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the slot has been read
                load_a(i + D, slot(i % D));
            }
            if constexpr (!L::STAT)
                if (i + DW < CNT) load_w(unit(wt, i + DW), bw[i % DW]);
            if (i == 0 && lead && a.has_next) prop_reserve<4>(a.next, a.epoch, shard, pb, ps);
            // keep the scheduler from hoisting later loads past this unit
            __builtin_amdgcn_sched_barrier(0);
        }

        if constexpr (!BF16) {
            // a value that the planes don't carry (an infinity, or a finite one
            // that rounds to it in bf16) left a NaN in all of its cell's sums:
            // the wavefront's units again, with such values done right
            bool nan = false;
#pragma unroll
            for (int m = 0; m < MH; ++m) nan = nan || acc[m][0][0] != acc[m][0][0];
            if (__ballot(nan) != 0ull) {
                clear_sums();
#pragma unroll 1
                for (int un = wt; un < L::NU; un += NW) {
                    const int t = un / U, u = un - t * U;
#pragma unroll
                    for (int m = 0; m < MH; ++m) {
                        const int rc = rowcell[t][16 * m + cl];
                        const char* src = rc >= 0 ? dbase + (size_t)rc * L::ROWB + u * UNIT_BYTES : zrow;
                        const uint4 v = *reinterpret_cast<const uint4*>(src + g * 16);
                        const uint4 x = *reinterpret_cast<const uint4*>(src + g * 16 + (CIN < 32 ? 0 : 64));
                        const Planes pl = split_unit<CIN, true>(v, x);
#pragma unroll
                        for (int k = 0; k < NB; ++k) {
                            uint4 wk[PL];
#pragma unroll
                            for (int p = 0; p < PL; ++p)
                                wk[p] = *reinterpret_cast<const uint4*>(wbase + (size_t)un * L::WU +
                                                                        (p * NB + k) * 1024 + wl16);
                            f4v s[1] = {acc[m][k]};
                            mfma_unit<CIN, 1, true>(s, wk, wk + 1, wk + 2, pl);
                            acc[m][k] = s[0];
                        }
                    }
                }
                // (the resident weights are fetched again rather than kept across
                // this: fewer registers in the kernels that run short of them)
                if constexpr (L::STAT) {
#pragma unroll
                    for (int i = 0; i < DW; ++i) load_w(unit(wt, i), bw[i]);
                }
            }
        }

        // partial sums, added in wavefront order by the finishing wavefronts
        auto red = [&](int ww, int j) __attribute__((always_inline)) {   // block j of wavefront ww
            return reinterpret_cast<lds_f4v*>((j / SB == 0 ? as0 : as1) + ww * SLOT + (j % SB) * 1024) + lane;
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
            }
            if (vrow && (COUT % 16 == 0 || 4 * g < COUT)) epilogue_unit<COUT, BF16, OB>(a, q, c0, g, zo, d, now, prev);
        }
        if (!BF16 && SPREAD && lead) memb_issue(a.mnext, q, a.Hout, a.Wout, g == 0 && vrow && now != prev, mbt);
        if (SPREAD && lead) memb_finish(a.mnext, q, a.Hout, a.Wout, mbt, now ? 1 : -1, a.epoch);
        if (lead && a.has_next) prop_write<4>(a.next, shard, pb, ps);
        // the next tile's table may be written now (its barrier orders the
        // sums: a wavefront writes red only after the barrier that every
        // finishing wavefront reaches after reading it)
        if constexpr (!L::STAT) {
            if ((tile + GT) * TM < n) {
#pragma unroll
                for (int i = 0; i < DW; ++i) load_w(unit(wt, i), bw[i]);
            }
        }
    }
}

// The leading scalar arguments repeat what the struct holds: the build preloads
// them into SGPRs, so that the loads that open every tile (list entries, tap
// bits, counts, weights) and the branch to the plan need not wait for the
// argument fetch, a round trip of its own.
//
// Tile height: 32 cells, so that a tile's share of the weights is small; 16
// where the list then still has a workgroup for every tile, on twice the
// compute units with half the operands and sums each (bf16 up to 64 input
// channels: wider bf16 tiles are all weight copies).  Measured on a 432x496
// fp32 stride, 16 against 32 cells: 128->128 10.6 against 10.7 us, 256->256
// 14.2 against 16.6, 128->256 stride 2 8.9 against 10.8, the backbone 205.6
// against 222.6; with two fp16 planes 64->128 stride 2 (45 32-cell tiles) 6.3
// against 7.7 us, 64->64 (100 to 140 tiles) 7.0 against 8.0.  On lists of more
// tiles than workgroups 16 cells lose (four 1024x1024 images, 1500 tiles: 45
// against 33 us, two workgroups per compute unit).
template <int CIN, int COUT, int S, bool BF16, bool SPARSE, bool SPREAD>
__global__ __launch_bounds__((64 * LayerShape<CIN, COUT, BF16, SPARSE>::NW)) void layer_kernel(
    const int32_t* __restrict__ plist, const int32_t* __restrict__ pcount, const uint16_t* __restrict__ ptaps,
    const char* __restrict__ pweights, int pcap, int pplan, LayerArgs a) {
    using L = LayerShape<CIN, COUT, BF16, SPARSE>;
    __shared__ int rowcell[9][32];
    __shared__ __attribute__((aligned(1024))) char as0[L::AS];
    __shared__ __attribute__((aligned(1024))) char as1[L::AS];
    __shared__ __attribute__((aligned(1024))) char as2[L::AS2];
    __shared__ __attribute__((aligned(1024))) char wl[L::WL_LDS];
    if constexpr (!SPARSE) {
        if ((int)blockIdx.x < pplan) {
            plan_tile<L::NW>(a.plan, a.epoch, (int)blockIdx.x, reinterpret_cast<uint32_t*>(as0),
                             reinterpret_cast<PlanWord*>(as1), &rowcell[0][0]);
            return;
        }
    }
    const int nplan = SPARSE ? 0 : pplan;
    const int b = (int)blockIdx.x - nplan, nwg = (int)gridDim.x - nplan;
    const int n0 = pcount[0], n1 = pcount[CSTRIDE];
    if constexpr (L::U <= 2 || !BF16) {
        if (max(n0, n1) <= 16 * (nwg / (2 * L::NBN))) {
            layer_tiles<CIN, COUT, S, BF16, SPARSE, SPREAD, 16>(plist, ptaps, pweights, pcap, n0, n1, b, nwg, a, rowcell,
                                                                (lds_char*)as0, (lds_char*)as1, (lds_char*)as2,
                                                                (lds_char*)wl);
            return;
        }
    }
    layer_tiles<CIN, COUT, S, BF16, SPARSE, SPREAD, 32>(plist, ptaps, pweights, pcap, n0, n1, b, nwg, a, rowcell,
                                                        (lds_char*)as0, (lds_char*)as1, (lds_char*)as2, (lds_char*)wl);
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
    using L = LayerShape<CI, CO, BF16, SPARSE>;
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
// and, at e = 0 .. 7, the unit's input channel
//   bf16: 8*(l/16) + e (zero past cin); one plane (two for an upsampler: W and
//         -W, an exact sign flip);
//   fp32: 4*(l/16) + e%4, and 16 more for e >= 4, the order in which a lane
//         takes its delta row (split_unit); planes Wh, Wm, Wl, or of 16
//         channels [Wh | Wh], [Wm | Wh], [Wl | Wm] over the halves of e.
__device__ __forceinline__ int packed_channel(int cin, int unit, int l, int e, int bf16) {
    if (bf16) return unit * 32 + (l >> 4) * 8 + e;
    return unit * 32 + (l >> 4) * 4 + (e & 3) + (cin >= 32 ? (e >> 2) * 16 : 0);
}

// An fp32 weight's planes at position e of a unit.
__device__ __forceinline__ void split_weight(float w, int cin, int e, uint16_t (&p)[3]) {
    uint32_t h, m, l, inf;
    split_pair<true>(w, 0.f, h, m, l, inf);
    const uint16_t H = (uint16_t)(h | inf), M = (uint16_t)m;
    const bool upper = cin < 32 && e >= 4;
    p[0] = H;
    p[1] = upper ? H : M;
    p[2] = upper ? M : (uint16_t)l;
}

// OIHW [cout][cin][3][3]; groups of up to 64 output channels, units [tap][32
// input channels].  One thread per packed position of a plane; positions of no
// channel (cout = 8, bf16 cin = 16) keep the buffer's zeros.
__global__ __launch_bounds__(256) void pack_weights_kernel(const void* __restrict__ w, int cin, int cout, int bf16,
                                                           uint16_t* __restrict__ out) {
    const int nu = units_of(cin), coutp = (cout + 15) / 16 * 16, nt = min(coutp, 64);
    const int plane = nt * 32;                            // values of a plane of a unit
    const int n = 9 * nu * coutp * 32;
    for (int i = (int)(blockIdx.x * 256 + threadIdx.x); i < n; i += (int)gridDim.x * 256) {
        const int e = i & 7, l = (i >> 3) & 63, blk = i % plane / 512, ug = i / plane;   // ug: group and unit
        const int group = ug / (9 * nu), un = ug - group * (9 * nu), t = un / nu, u = un - t * nu;
        const int co = group * nt + blk * 16 + (l & 15), ci = packed_channel(cin, u, l, e, bf16);
        if (co >= cout || ci >= cin) continue;
        const size_t from = ((size_t)co * cin + ci) * 9 + t;
        const size_t to = (size_t)ug * plane * (bf16 ? 1 : 3) + (i % plane);
        if (bf16) {
            out[to] = static_cast<const uint16_t*>(w)[from];
        } else {
            uint16_t p[3];
            split_weight(static_cast<const float*>(w)[from], cin, e, p);
            for (int k = 0; k < 3; ++k) out[to + (size_t)k * plane] = p[k];
        }
    }
}

// [cin][cout][S][S]; one group, units [32 input channels], blocks [sub-cell
// a*S + b][16 output channels].
__global__ __launch_bounds__(256) void pack_up_weights_kernel(const void* __restrict__ w, int cin, int cout, int s2,
                                                              int bf16, uint16_t* __restrict__ out) {
    const int ncbt = cout / 16, plane = s2 * cout * 32;
    const int n = units_of(cin) * plane;
    for (int i = (int)(blockIdx.x * 256 + threadIdx.x); i < n; i += (int)gridDim.x * 256) {
        const int e = i & 7, l = (i >> 3) & 63, ob = i % plane / 512, u = i / plane;
        const int ab = ob / ncbt, co = (ob - ab * ncbt) * 16 + (l & 15), ci = packed_channel(cin, u, l, e, bf16);
        if (ci >= cin) continue;
        const size_t from = ((size_t)ci * cout + co) * s2 + ab;
        const size_t to = (size_t)u * plane * (bf16 ? 2 : 3) + (i % plane);
        if (bf16) {
            const uint16_t v = static_cast<const uint16_t*>(w)[from];
            out[to] = v;
            out[to + plane] = v ^ 0x8000u;
        } else {
            uint16_t p[3];
            split_weight(static_cast<const float*>(w)[from], cin, e, p);
            for (int k = 0; k < 3; ++k) out[to + (size_t)k * plane] = p[k];
        }
    }
}

size_t wpack_bytes(int cin, int cout, bool bf16) {
    return (size_t)9 * units_of(cin) * (size_t)((cout + 15) / 16 * 16) * 64 * (bf16 ? 1 : 3);
}

size_t up_wpack_bytes(int cin, int cout, int stride, bool bf16) {
    return (size_t)units_of(cin) * (size_t)cout * stride * stride * 64 * (bf16 ? 2 : 3);
}

static unsigned pack_grid(size_t values) { return (unsigned)std::min<size_t>(1024, (values + 255) / 256); }

hipError_t launch_pack_weights(const void* w, int cin, int cout, bool bf16, void* out) {
    hipLaunchKernelGGL(pack_weights_kernel, dim3(pack_grid(wpack_bytes(cin, cout, true) / 2)), dim3(256), 0, nullptr, w,
                       cin, cout, bf16 ? 1 : 0, static_cast<uint16_t*>(out));
    return hipGetLastError();
}

hipError_t launch_pack_up_weights(const void* w, int cin, int cout, int stride, bool bf16, void* out) {
    hipLaunchKernelGGL(pack_up_weights_kernel, dim3(pack_grid(up_wpack_bytes(cin, cout, stride, true) / 4)), dim3(256),
                       0, nullptr, w, cin, cout, stride * stride, bf16 ? 1 : 0, static_cast<uint16_t*>(out));
    return hipGetLastError();
}

}  // namespace ssc
