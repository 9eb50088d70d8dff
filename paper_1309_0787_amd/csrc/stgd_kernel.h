// Stochastic tensor gradient descent on the implicit whitened third moment
// (Section 3.2, Lemma "update"), in the stacked matrix form of Section 4.3:
//
//   G  = Phi^T Phi,  O = Phi (G * G)               (matrix cores)
//   PA = YA Phi, PB = YB Phi                       (batch x k, matrix cores)
//   mA = Phi^T ybarA, mB = Phi^T ybarB
//   H  = PA * PB,  s = column sums of H
//   Q  = a H - b PA diag(mB) - b diag(mA) PB
//   D  = YC^T Q / B + ybarC (c mA*mB - b s / B)^T  (matrix cores)
//   Phi <- Phi + beta (D - kappa O)
//
// One workgroup of 8 waves runs one whole online run (all steps); the tensor
// is never formed.  The FP32 master copy of Phi (and its Kahan compensation)
// stays in registers, a copy in the operand type in LDS.
//
// Column ownership.  Every quantity above is made column by column: column i
// of G, O, P, Q and D needs only phi_i and the whole of Phi and of the batch.
// A wave owns 16 columns (one tile column) and carries them through both
// chains, Phi^T Phi -> G*G -> O and P -> Q -> D, in registers: the matrix
// cores return a tile with rows 4 (lane / 16) + r of column lane % 16, which
// two lane-group swaps per register pair turn into the second operand of the
// product that contracts over those rows.  So neither G*G nor Q passes through
// LDS, the column sums and the means stay inside a wave, and the waves meet
// only when Phi changes: one barrier per step where LDS holds the Phi copy and
// the batch twice, two where it holds them once.  LDS serves the first operands
// only (Phi and the batch, rows or transposed reads), which every wave reads
// whole.
//
// What bounds a step (k = 100, one view, 100 rows: 3.6 us, 8600 cycles): 7
// working waves on 4 SIMDs.  Matrix instructions fill 36% of the three SIMDs
// that carry two waves; LDS delivers 0.9 MB a step (7 waves x Phi and the batch,
// both ways), 60% of its rate; the rest is the chain G -> O -> (means) -> Q -> D
// with two or three LDS trips that nothing covers.  The kernel that split every
// product over a grid of waves and took G*G and Q through LDS (four barriers a
// step) measured, before and after, us per step: k = 100 one view 4.2 -> 3.6
// (compensated 4.9 -> 3.9), three views 16.2 -> 5.0 (compensated 16.5 -> 5.9;
// there the views did not fit beside the exchange buffer and were read from
// global memory inside the products), k = 128 5.8 -> 4.8, k = 80 3.6 -> 2.9,
// k = 64 2.3 -> 1.8, k = 48 2.0 -> 1.6, k = 32 1.3 -> 1.2.  Two columns per wave
// pair (5.3) and two per wave at one wave per SIMD (5.2) were slower at k = 100.
//
// With NT = ceil(k / 16) < 8 columns the waves left over stage the batch
// (kSpec); waves 4 .. 7, which share a SIMD with the older waves 0 .. 3 and lose
// the arbitration to them, raise their priority through the batch products,
// so that both end together (k = 100: 3.85 -> 3.63 us).
#pragma once

#include "stgd_args.h"

namespace otm {
namespace {

// ---------------------------------------------------------------------------
// Matrix-core operands (16x16x32 BF16).  Lane l (q = l / 16, c = l % 16) of a
// product over one K block of KB rows supplies the first operand's row c and the
// second operand's column c, both at rows 8 q + e, e < 8, of the block, and
// receives rows 4 q + r, r < 4, of column c of the 16 x 16 result.
// ---------------------------------------------------------------------------
struct Mma {
    using Y = __bf16;
    using Op = __bf16;
    using Frag = bf16x8;
    using Chunk = bf16x8;
    static constexpr int KB = 32;
    // LDS row padding: rows 8 x odd dwords apart (96, 160, 224 or 288 bytes).
    // Of the pitches 256 to 336 bytes only 288 let a 16-byte row read (lane l:
    // row l % 16, chunk l / 16) run without bank conflicts (4 cycles per wave
    // against 8 to 32, measured on gfx950)
    static constexpr int SPAD = 16;
    static constexpr int CH = 8;
    __device__ static f32x4 mma(Frag a, Frag b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
    __device__ static Op to_op(float x) { return f32_to_bf16(x); }
    // sw: the row's column permutation (Phi copy), 0 for the batch
    __device__ static Frag row(const Op* x, int q, int sw) {
        return *reinterpret_cast<const bf16x8*>(x + ((8 * q) ^ sw));
    }
    // Column permutation of row r of the Phi copy: rows with bit 2 set swap
    // their 16-byte chunks in pairs.  At the 288-byte pitch the 8-byte stores
    // of a result tile (lane l: row l % 16, piece l / 16) otherwise hit each
    // bank twice as often as they need to (16 cycles per wave); with the
    // permutation they take 8 (a contiguous 8-byte store takes 6.6), while the
    // row reads stay conflict-free (measured on gfx950).
    __device__ static constexpr int sw(int r) { return ((r >> 2) & 1) << 3; }
    // Column reads: lane l receives X[8 (l/16) + e][l % 16], e < 8, where
    // X[r][c] = x[r * stride + c] in LDS.  Two transposing 8-byte reads (rows
    // 0-3 and 4-7 of the lane's group): lane s addresses columns 4 (s % 4) ..
    // + 3 of row 8 (s/16) + (s % 16)/4, and element i of lane l comes from
    // element l % 4 of lane 16 (l/16) + (l % 16)/4 + 4 i.  x and stride keep
    // every address 8-byte aligned.
    __device__ static Frag col(const Op* x, int stride, int lane) { return col_t<0>(x, stride, lane); }
    // on a permuted array (sw above), x at a row that is a multiple of 8 and a
    // column that is a multiple of 16: the first read's rows keep their order,
    // the second read's rows (bit 2 set) have their chunks swapped
    __device__ static Frag col_sw(const Op* x, int stride, int lane) { return col_t<8>(x, stride, lane); }
    template <int SW>
    __device__ static Frag col_t(const Op* x, int stride, int lane) {
        typedef short s16x4 __attribute__((ext_vector_type(4)));
        typedef short s16x8 __attribute__((ext_vector_type(8)));
        typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
        const Op* p = x + (8 * (lane >> 4) + ((lane >> 2) & 3)) * stride;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * (lane & 3)));
        const s16x4 hi =
            __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * stride + ((4 * (lane & 3)) ^ SW)));
        const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(Frag, v);
    }
    // Second operand of the product that contracts over the 32 rows of two
    // result tiles t[0], t[1]: lane group q holds rows 4 q .. 4 q + 3 of each
    // and needs rows 8 q .. 8 q + 7 of the pair.  Swapping the upper half of
    // t[0] with the lower half of t[1], then the odd 16-lane rows of the first
    // with the even ones of the second, leaves rows 8 q .. + 3 in the first
    // and 8 q + 4 .. + 7 in the second.
    __device__ static Frag second(const f32x4* t) {
        u32x4 f;
        bf16x4 x, y;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            x[r] = f32_to_bf16(t[0][r]);
            y[r] = f32_to_bf16(t[1][r]);
        }
        typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
        const u32x2 px = __builtin_bit_cast(u32x2, x), py = __builtin_bit_cast(u32x2, y);
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const auto h = __builtin_amdgcn_permlane32_swap(px[d], py[d], false, false);
            const auto o = __builtin_amdgcn_permlane16_swap(h[0], h[1], false, false);
            f[d] = o[0];
            f[2 + d] = o[1];
        }
        return __builtin_bit_cast(Frag, f);
    }
    // The same for a block whose second tile is empty: 16x16x16 instructions,
    // rows 4 q .. 4 q + 3 of one tile as they are
    typedef short Half __attribute__((ext_vector_type(4)));
    __device__ static Half col_half(const Op* x, int stride, int lane, int sw) {
        typedef __attribute__((address_space(3))) Half lds_half;
        const Op* p = x + (4 * (lane >> 4) + ((lane >> 2) & 3)) * stride;
        return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_half*)(p + ((4 * (lane & 3)) ^ sw)));
    }
    __device__ static Half second_half(f32x4 t) {
        bf16x4 x;
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = f32_to_bf16(t[r]);
        return __builtin_bit_cast(Half, x);
    }
    __device__ static f32x4 mma_half(Half a, Half b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
    }
    __device__ static float elem(Frag f, int e) { return bf16_to_f32(f[e]); }
    __device__ static u32x4 chunk_mask(int valid) {
        u32x4 m;
#pragma unroll
        for (int d = 0; d < 4; ++d)
            m[d] = ((2 * d < valid) ? 0x0000ffffu : 0u) | ((2 * d + 1 < valid) ? 0xffff0000u : 0u);
        return m;
    }
    __device__ static void store4(Op* p, f32x4 v) {
        bf16x4 o;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = f32_to_bf16(v[r]);
        *reinterpret_cast<bf16x4*>(p) = o;
    }
};

// LDS of one run.  NV: views held at once (1 or 3); NBUF, NBY: copies of Phi and of
// the batch (2: the next step's are written while this step's are read).
template <int NT, int NV, int NBUF, int NBY>
struct SgdSmem {
    using Op = Mma::Op;
    static constexpr int TPB = Mma::KB / 16;             // tiles per K block
    static constexpr int NKB = (NT + TPB - 1) / TPB;   // K blocks of a contraction over k
    static constexpr int KPW = NKB * Mma::KB;            // stored row width (and rows of the Phi copy)
    static constexpr int SP = KPW + Mma::SPAD;           // row pitch
    alignas(16) Op phi[NBUF][KPW * SP];
    alignas(16) Op y[NBY][NV * MB * SP];
    alignas(16) float ybar[3 * KPW];
    alignas(16) int32_t idx[2][MB];                          // row indices of the coming steps (by step parity)
};

// Views and copies that fit: one barrier per step with two copies of Phi and of
// the batch, else two.
template <int NT, bool ALIASED>
struct SgdMode {
    static constexpr int V = ALIASED ? 1 : 3;
    template <int NBUF, int NBY>
    static constexpr bool fits = sizeof(SgdSmem<NT, V, NBUF, NBY>) <= kLdsLimit;
    static constexpr bool kTwo = fits<2, 2>;
    static constexpr int NV = V;
    static constexpr int NBUF = kTwo ? 2 : 1;
    static constexpr int NBY = fits<1, 2> ? 2 : 1;
    using SM = SgdSmem<NT, NV, NBUF, NBY>;
    static_assert(sizeof(SM) <= kLdsLimit, "STGD shared memory exceeds 160 KB");
};

// Position of a step: its pass, its batch in the pass, its rows (0 past the last step).
struct StepPos {
    int pass, s, nb;
};

// One whole run of restart r_id by the calling workgroup.  COMP = false (BF16
// only, for runs without compensation) keeps no compensation terms.
template <int NT, bool ALIASED, bool COMP>
__device__ __forceinline__ void sgd_body(const SgdArgs& g, const int r_id, typename SgdMode<NT, ALIASED>::SM& sm) {
    using Mode = SgdMode<NT, ALIASED>;
    using SM = typename Mode::SM;
    using Op = Mma::Op;
    using Y = Mma::Y;
    using Frag = Mma::Frag;
    constexpr int TPB = SM::TPB, NKB = SM::NKB, KPW = SM::KPW, SP = SM::SP, KB = Mma::KB;
    constexpr int NV = Mode::NV, NBUF = Mode::NBUF, NBY = Mode::NBY;
    constexpr int NCH = MB / KB;                       // chunks of KB batch rows
    constexpr int SG = NT < 4 ? NT : 4, NSG = (NT + SG - 1) / SG;   // row tiles of O and D whose operands are read ahead together
    // BF16 blocks take two tiles: with an odd number of tiles the last block of O
    // is half empty and takes the 16-row instruction (half the LDS reads)
    constexpr bool kHalfO = NT % 2 == 1;
    // Up to three tile columns (one view: four) a wave has a SIMD to itself and the
    // registers for it: the chunks of a batch run side by side, and the rows of ybar
    // stay in registers (k = 40, 128 rows: 1.84 -> 1.60 us a step, k = 64, 100 rows
    // 2.05 -> 1.84; at k = 64 with three views and past it the registers run out)
    constexpr bool kWide = NT <= 3 || (NT == 4 && ALIASED);

    const int tid = threadIdx.x;
    const int lane = tid & 63, l16 = lane & 15, q = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6) & (kWaves - 1);
    // (waves w and w + 4 run on one SIMD: with NT = 7 only one of the four has a
    // single working wave)
    const bool act = w < NT;
    const int c = act ? w : 0;

    const int k = g.k, n = g.n, ldy = g.ldy, B = g.batch;
    const int i = c * 16 + l16;                        // this lane's component
    const bool lane_live = act && i < k;
    const float live = lane_live ? 1.0f : 0.0f;
    const float* Phi0 = g.Phi0 + (size_t)r_id * k * k;
    float* Phi = g.Phi + (size_t)r_id * k * k;
    float* Comp = g.Phi_comp ? g.Phi_comp + (size_t)r_id * k * k : nullptr;
    float* Snap = g.snapshots ? g.snapshots + (size_t)r_id * g.passes * k * k : nullptr;
    const int32_t* perms = g.perms ? g.perms + (size_t)r_id * g.perm_stride : nullptr;
    const Y* Yv[3] = {static_cast<const Y*>(g.YA), static_cast<const Y*>(g.YB), static_cast<const Y*>(g.YC)};
    bool bad = false;
    // mA = Phi^T ybarA and mB = Phi^T ybarB ride along in Phi^T Phi when a wave
    // has all rows of its column and two padding rows are free: rows k, k + 1 of
    // the Phi copy hold ybarA, ybarB, so G[k][i] = mA[i], G[k + 1][i] = mB[i]
    // (both rows of G*G are cleared before O).  Otherwise the vector ALU sums
    // them from the wave's second operand.
    const bool mfold = k + 2 <= NT * 16;
    const int swl = Mma::sw(l16);

    // ---- master copy: the wave's column
    f32x4 phi_r[NT], comp[COMP ? NT : 1];
#pragma unroll
    for (int mt = 0; mt < NT; ++mt) {
        f32x4 v = {0.f, 0.f, 0.f, 0.f}, cv = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int a = mt * 16 + 4 * q + r;
            if (lane_live && a < k) {
                v[r] = Phi0[(size_t)i * k + a];
                if (COMP && Comp) cv[r] = Comp[(size_t)i * k + a];
            }
        }
        phi_r[mt] = v;
        if constexpr (COMP) comp[mt] = cv;
    }

    // ---- batch staging: thread -> 16-byte column piece a0t of rows tr0 + RPP j.
    // Loads of scattered rows stall the waves that issue them (45 cycles each in
    // BF16), so where waves are left over (kSpec) those stage the batch alone,
    // LB rows per thread at a time, and the others run the products.
    constexpr bool kSpec = NBY == 2 && NT < kWaves;
    // With two copies of the batch the rows loaded during a step are written to
    // LDS at the start of the next one (AHEAD = 2 steps before they are used:
    // a step of small k is shorter than a trip to memory), else at the end.
    constexpr int NL = kSpec ? 64 * (kWaves - NT) : kThreads;
    const int lt = kSpec ? tid - 64 * NT : tid;
    const bool stager = !kSpec || !act;
    constexpr int cpr = KPW / Mma::CH;
    constexpr int CPRP = cpr <= 4 ? 4 : cpr <= 8 ? 8 : cpr <= 16 ? 16 : 32;   // a power of two
    constexpr int RPP = NL / CPRP;
    constexpr int NPT = (MB + RPP - 1) / RPP;
    constexpr int AHEAD = NBY == 2 && (!kSpec || NV * NPT <= 12) ? 2 : 1;
    constexpr bool kPart = kSpec && AHEAD == 1;        // rows go through LB at a time, within a step
    constexpr int LB = kPart ? 16 : NPT;
    constexpr int NIX = (MB + NL - 1) / NL;            // row indices per thread
    const int a0t = (lt & (CPRP - 1)) * Mma::CH, tr0 = lt / CPRP;
    const bool loader = a0t < k;                       // columns past k are never written: they stay zero
    const u32x4 a0mask = Mma::chunk_mask(k - a0t);
    Mma::Chunk pbuf[NV][LB];
    auto at_step = [&](int t) -> StepPos {
        StepPos p{};
        p.pass = t / g.spp;
        p.s = t - p.pass * g.spp;
        p.nb = t < g.end_step ? min(B, n - p.s * B) : 0;
        return p;
    };
    auto next_step = [&](const StepPos& p, int t) -> StepPos {   // position of step t, one past p
        StepPos o = p;
        o.s = p.s + 1;
        if (o.s == g.spp) {
            o.s = 0;
            o.pass = p.pass + 1;
        }
        o.nb = t < g.end_step ? min(B, n - o.s * B) : 0;
        return o;
    };
    // The loads below are unconditional (lanes without a row read one that
    // exists): a load under a condition makes the compiler wait for the
    // previous load of its registers, one memory round trip each.
    int32_t nidx[NIX];                                 // this thread's rows of the step after next
    auto fetch_index = [&](const StepPos& p) {
        if (perms) {
            const int32_t* pp = perms + (p.nb > 0 ? (size_t)p.pass * n + (size_t)p.s * B : 0);
#pragma unroll
            for (int e = 0; e < NIX; ++e) nidx[e] = pp[lt + NL * e < p.nb ? lt + NL * e : 0];
        }
    };
    auto put_index = [&](const StepPos& p, int t, const int32_t (&from)[NIX]) {   // row 0 past nb
#pragma unroll
        for (int e = 0; e < NIX; ++e) {
            const int at = lt + NL * e;
            int32_t r = perms ? from[e] : p.s * B + at;
            if (at < p.nb && (r < 0 || r >= n)) {   // out-of-range permutation entry: reads row 0, reported
                r = 0;
                bad = true;
            }
            if (at < MB) sm.idx[t & 1][at] = at < p.nb ? r : 0;
        }
    };
    const int a0c = loader ? a0t : 0;
    auto read_index = [&](int (&r)[NPT], int t) {
#pragma unroll
        for (int j = 0; j < NPT; ++j) r[j] = sm.idx[t & 1][MB % RPP ? min(tr0 + j * RPP, MB - 1) : tr0 + j * RPP];
    };
    // Rows r of views v0 .. v0 + NV - 1 into pbuf: the share x of X, so that the
    // loads spread over the products of a step
    auto issue_rows = [&](int v0, const int (&r)[NPT], int x, int X) {
        if constexpr (!kPart) {
#pragma unroll
            for (int e = 0; e < NV * NPT; ++e)
                if (e >= x * NV * NPT / X && e < (x + 1) * NV * NPT / X) {
                    const int v = e / NPT, j = e % NPT;
                    pbuf[v][j] = *reinterpret_cast<const Mma::Chunk*>(Yv[v0 + v] + ((size_t)r[j] * ldy + a0c));
                }
        }
    };
    auto store_row = [&](Op* y, int nb, int v, int j, const Mma::Chunk& c16) {
        const int tr = tr0 + j * RPP;                  // rows nb .. B - 1 of a short batch are cleared
        const u32x4 x = __builtin_bit_cast(u32x4, c16) & a0mask;
        const u32x4 z = {0u, 0u, 0u, 0u};
        if (tr < B) *reinterpret_cast<u32x4*>(&y[(v * MB + tr) * SP + a0t]) = tr < nb ? x : z;
    };
    auto commit_rows = [&](Op* y, int nb) {
        if constexpr (!kPart) {
            if (loader) {
#pragma unroll
                for (int j = 0; j < NPT; ++j)
#pragma unroll
                    for (int v = 0; v < NV; ++v) store_row(y, nb, v, j, pbuf[v][j]);
            }
        }
    };
    // all rows of step t into y, LB at a time (kPart)
    auto stage_rows = [&](Op* y, int nb, int t) {
        if constexpr (kPart) {
#pragma unroll
            for (int j0 = 0; j0 < NPT; j0 += LB) {
                int r[LB];
#pragma unroll
                for (int j = 0; j < LB; ++j) r[j] = sm.idx[t & 1][min(tr0 + (j0 + j) * RPP, MB - 1)];
#pragma unroll
                for (int j = 0; j < LB; ++j)
                    if (j0 + j < NPT)
#pragma unroll
                        for (int v = 0; v < NV; ++v)
                            pbuf[v][j] = *reinterpret_cast<const Mma::Chunk*>(Yv[v] + ((size_t)r[j] * ldy + a0c));
                if (loader) {
#pragma unroll
                    for (int j = 0; j < LB; ++j)
                        if (j0 + j < NPT)
#pragma unroll
                            for (int v = 0; v < NV; ++v) store_row(y, nb, v, j0 + j, pbuf[v][j]);
                }
            }
        }
    };
    StepPos p0 = at_step(g.start_step), p1 = next_step(p0, g.start_step + 1), p2 = next_step(p1, g.start_step + 2);
    int ridx[NPT];
    // first steps: the indices of all of them in one trip, then the rows
    int32_t first[2][NIX];
    if (stager) {
        fetch_index(p0);
#pragma unroll
        for (int e = 0; e < NIX; ++e) first[0][e] = nidx[e];
        fetch_index(p1);
#pragma unroll
        for (int e = 0; e < NIX; ++e) first[1][e] = nidx[e];
        fetch_index(p2);
    }
    // ---- LDS: Phi copy (phi_i in row i), zero past k and (batch) everywhere else
    {
        const u32x4 z = {0u, 0u, 0u, 0u};
        constexpr int NP = sizeof(sm.phi) / 16, NY = sizeof(sm.y) / 16;
        static_assert(sizeof(sm.phi) % 16 == 0 && sizeof(sm.y) % 16 == 0, "cleared 16 bytes at a time");
        for (int e = tid; e < NP; e += kThreads) reinterpret_cast<u32x4*>(&sm.phi[0][0])[e] = z;
        for (int e = tid; e < NY; e += kThreads) reinterpret_cast<u32x4*>(&sm.y[0][0])[e] = z;
    }
    __syncthreads();
    for (int e = tid; e < (mfold ? k + 2 : k) * k; e += kThreads) {
        const int r = e / k, a = e - r * k;
        const float v = r < k ? Phi0[e] : g.ybar[e - k * k];
#pragma unroll
        for (int b = 0; b < NBUF; ++b) sm.phi[b][r * SP + (a ^ Mma::sw(r))] = Mma::to_op(v);
    }
    for (int e = tid; e < 3 * KPW; e += kThreads) {
        const int v = e / KPW, a = e % KPW;
        sm.ybar[e] = (a < k) ? g.ybar[v * k + a] : 0.0f;
    }
    if (stager) {
        put_index(p0, g.start_step, first[0]);
        put_index(p1, g.start_step + 1, first[1]);
    }
    __syncthreads();
    if (stager) {
        if constexpr (kPart) {
            stage_rows(sm.y[0], p0.nb, g.start_step);
        } else {
            read_index(ridx, g.start_step);
            issue_rows(0, ridx, 0, 1);
            if constexpr (AHEAD == 2) read_index(ridx, g.start_step + 1);
            commit_rows(sm.y[0], p0.nb);
            if constexpr (AHEAD == 2) issue_rows(0, ridx, 0, 1);
        }
    }
    __syncthreads();
    if constexpr (AHEAD == 2) {
        if (stager) {
            put_index(p2, g.start_step + 2, nidx);
            fetch_index(next_step(p2, g.start_step + 3));
        }
        __syncthreads();
    }
    // the loads of the master copy land here: a wait inside the loop would also
    // wait for the batch rows in flight
    __builtin_amdgcn_s_waitcnt(0);
    int cur = 0;                           // copies in use
    StepPos p3 = next_step(p2, g.start_step + 3);
    // scalars of a step: worked out at the end of the step before it, where a wave
    // waits for its LDS writes
    float beta, invB;
    const float invBatch = 1.0f / static_cast<float>(B);
    auto scalars = [&](const StepPos& p, int t) {
        beta = g.beta0 / (1.0f + static_cast<float>(t) * g.inv_tau);
        invB = p.nb == B ? invBatch : 1.0f / static_cast<float>(p.nb);
    };
    scalars(p0, g.start_step);
    if (kSpec && NT <= 4 && act) __builtin_amdgcn_s_setprio(2);   // before the stagers
    f32x4 ybw[kWide ? 2 * NKB * 2 : 1], ycw[kWide ? NT : 1];
    if constexpr (kWide) {
#pragma unroll
        for (int b = 0; b < NKB; ++b)
#pragma unroll
            for (int e4 = 0; e4 < 2; ++e4)
#pragma unroll
                for (int v = 0; v < 2; ++v)
                    ybw[(b * 2 + e4) * 2 + v] = *reinterpret_cast<const f32x4*>(&sm.ybar[v * KPW + b * KB + 8 * q + 4 * e4]);
#pragma unroll
        for (int mt = 0; mt < NT; ++mt)
            ycw[mt] = *reinterpret_cast<const f32x4*>(&sm.ybar[2 * KPW + mt * 16 + 4 * q]);
    }
    for (int t = g.start_step; t < g.end_step; ++t) {
        const int nb = p0.nb;
        const Op* phi = sm.phi[NBUF == 2 ? cur : 0];
        const Op* y = sm.y[NBY == 2 ? cur : 0];
        Op* phi_n = sm.phi[NBUF == 2 ? cur ^ 1 : 0];
        Op* y_n = sm.y[NBY == 2 ? cur ^ 1 : 0];
        // rows of step t + AHEAD and the row indices of the step after start their
        // trip from global memory
        const StepPos pf = AHEAD == 2 ? next_step(p3, t + 4) : p2;
        if (!kPart && stager) {
            if constexpr (AHEAD == 2) {    // (nidx: fetched during the last step)
                commit_rows(y_n, p1.nb);
                put_index(p3, t + 3, nidx);
            }
            read_index(ridx, t + AHEAD);
        }

        Frag bphi[NKB];                    // second operand: this column of Phi
        f32x4 dacc[NT];
        float mA = 0.f, mB = 0.f, colsum = 0.f;
        float al = 0.f, bmA = 0.f, bmB = 0.f;
        const float f3 = beta * live * g.kappa;
        f32x4 oacc[NT];
        // batch rows of a chunk: first operands of P
        Frag fp[TPB][NKB];
        auto load_p = [&](const Op* yv, int ch) {
#pragma unroll
            for (int b = 0; b < NKB; ++b)
#pragma unroll
                for (int u = 0; u < TPB; ++u)
                    if (u == 0 || kWide || ch * KB + 16 < nb)   // a chunk with at most 16 rows is half a chunk
                        fp[u][b] = Mma::row(yv + (ch * KB + u * 16 + l16) * SP + b * KB, q, 0);
        };
        if (act) {
#pragma unroll
            for (int b = 0; b < NKB; ++b) bphi[b] = Mma::row(phi + i * SP + b * KB, q, swl);
            // first operands of O: columns of Phi, SG row tiles (group e) at a time
            Frag fo[2][SG];
            Mma::Half foh[2][kHalfO ? SG : 1];
            auto load_o = [&](int e) {
                const int ob = e / NSG;
                const bool half = kHalfO && ob == NKB - 1;
#pragma unroll
                for (int u = 0; u < SG; ++u) {
                    const int mt = (e % NSG) * SG + u;
                    if (mt >= NT) continue;
                    const Op* x = phi + ob * KB * SP + mt * 16;
                    if (half) {   // rows 4 q + .. : bit 2 is set where q is odd
                        if constexpr (kHalfO) foh[e & 1][u] = Mma::col_half(x, SP, lane, (q & 1) << 3);
                    } else {
                        fo[e & 1][u] = Mma::col_sw(x, SP, lane);
                    }
                    }
            };
            // ---- G = Phi^T Phi: In every
            // product the first operands of the next group of instructions are
            // read from LDS before the current group is issued (the scheduling
            // barriers keep the compiler from sinking the reads to their uses).
            constexpr int GT = NKB * TPB, GG = SG, NGG = NSG;   // GG row tiles at a time
            f32x4 gacc[GT];
            Frag fg[2][GG];
            auto load_g = [&](int e) {
#pragma unroll
                for (int j = 0; j < GG; ++j) {
                    const int u = (e % NGG) * GG + j;
                    if (u < NT)
                        fg[e & 1][j] = Mma::row(phi + (u * 16 + l16) * SP + (e / NGG) * KB, q, swl);
                }
            };
            load_g(0);
            if constexpr (!kSpec) fetch_index(pf);
#pragma unroll
            for (int u = 0; u < GT; ++u) gacc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < NKB * NGG; ++e) {
                if (e + 1 < NKB * NGG) load_g(e + 1);
                else load_o(0);
                if (!kSpec && e % NGG == 0) issue_rows(0, ridx, e / NGG, NKB + NKB);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < GG; ++j) {
                    const int u = (e % NGG) * GG + j;
                    if (u < NT) gacc[u] = Mma::mma(fg[e & 1][j], bphi[e / NGG], gacc[u]);
                }
            }
            // ---- the means, then G*G (rows past k cleared)
            if (mfold) {
                const int kk = k & 15, r = kk & 3, r1 = (kk + 1) & 3;
                const f32x4 gv = gacc[NT - 1];
                const float x0 = r == 0 ? gv[0] : r == 1 ? gv[1] : r == 2 ? gv[2] : gv[3];
                const float x1 = r1 == 0 ? gv[0] : r1 == 1 ? gv[1] : r1 == 2 ? gv[2] : gv[3];
                mA = add_xor32(add_xor16(q == kk >> 2 ? x0 : 0.0f));
                mB = add_xor32(add_xor16(q == (kk + 1) >> 2 ? x1 : 0.0f));
            } else {
#pragma unroll
                for (int b = 0; b < NKB; ++b)
#pragma unroll
                    for (int e4 = 0; e4 < KB / 16; ++e4) {
                        const int a = b * KB + 8 * q + 4 * e4;
                        f32x4 ya, yb;
                        if constexpr (kWide) {
                            ya = ybw[(b * 2 + e4) * 2];
                            yb = ybw[(b * 2 + e4) * 2 + 1];
                        } else {
                            ya = *reinterpret_cast<const f32x4*>(&sm.ybar[a]);
                            yb = *reinterpret_cast<const f32x4*>(&sm.ybar[KPW + a]);
                        }
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float x = Mma::elem(bphi[b], 4 * e4 + e);
                            mA = fmaf(x, ya[e], mA);
                            mB = fmaf(x, yb[e], mB);
                        }
                    }
                mA = add_xor32(add_xor16(mA));
                mB = add_xor32(add_xor16(mB));
            }
#pragma unroll
            for (int ob = 0; ob < NKB; ++ob)
#pragma unroll
                for (int u = 0; u < TPB; ++u) {
                    f32x4& gv = gacc[ob * TPB + u];
                    gv = gv * gv;
                    if (ob * TPB + u == NT - 1) {   // the rows that hold the means
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if ((NT - 1) * 16 + 4 * q + r >= k) gv[r] = 0.0f;
                    }
                }
            // ---- O = Phi (G*G)
#pragma unroll
            for (int mt = 0; mt < NT; ++mt) oacc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < NKB * NSG; ++e) {
                const int ob = e / NSG;
                if (e + 1 < NKB * NSG) load_o(e + 1);
                else load_p(y, 0);
                if (!kSpec && e % NSG == 0) issue_rows(0, ridx, NKB + ob, NKB + NKB);
                __builtin_amdgcn_sched_barrier(0);
                if (kHalfO && ob == NKB - 1) {
                    const Mma::Half fb = Mma::second_half(gacc[ob * TPB]);
#pragma unroll
                    for (int u = 0; u < SG; ++u) {
                        const int mt = (e % NSG) * SG + u;
                        if constexpr (kHalfO)
                            if (mt < NT) oacc[mt] = Mma::mma_half(foh[e & 1][u], fb, oacc[mt]);
                    }
                } else {
                    const Frag fb = Mma::second(&gacc[ob * TPB]);
#pragma unroll
                    for (int u = 0; u < SG; ++u) {
                        const int mt = (e % NSG) * SG + u;
                        if (mt < NT) oacc[mt] = Mma::mma(fo[e & 1][u], fb, oacc[mt]);
                    }
                }
            }
            // -beta kappa O enters the compensation term (c <- c + beta kappa O) or,
            // without one, the master copy at once, so O is not live through the
            // batch products
#pragma unroll
            for (int mt = 0; mt < NT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if constexpr (COMP) comp[mt][r] = fmaf(f3, oacc[mt][r], comp[mt][r]);
                    else phi_r[mt][r] = fmaf(-f3, oacc[mt][r], phi_r[mt][r]);
                }
            if (NT > 4 && w >= 4) __builtin_amdgcn_s_setprio(1);
            al = g.a * live;
            bmA = g.b * live * mA;
            bmB = g.b * live * mB;
#pragma unroll
            for (int mt = 0; mt < NT; ++mt) dacc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        } else {
            fetch_index(pf);
            if constexpr (kPart) stage_rows(y_n, p1.nb, t + 1);
            else issue_rows(0, ridx, 0, 1);
            if constexpr (kPart) put_index(pf, t + 2, nidx);
        }

        auto hold = [&]() {
            if constexpr (!kWide) __builtin_amdgcn_sched_barrier(0);
        };
        auto coeff = [&](f32x4& pa, const f32x4& pb) {   // Q in place of PA, and the column sums
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float xa = pa[r];
                if constexpr (ALIASED) {   // one view: xb = xa
                    colsum = fmaf(xa, xa, colsum);
                    pa[r] = xa * fmaf(al, xa, -(bmA + bmB));
                } else {
                    const float xb = pb[r];
                    colsum = fmaf(xa, xb, colsum);
                    pa[r] = fmaf(xa, fmaf(al, xb, -bmB), -bmA * xb);
                }
            }
        };
        // ---- the batch, KB rows at a time: P -> Q -> D (the rows of a chunk past
        // nb are zero)
        auto product = [&](const Op* yv, int ch, f32x4 (&pt)[TPB], auto tiles) {
            constexpr int T = decltype(tiles)::value;
#pragma unroll
            for (int u = 0; u < T; ++u) pt[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int b = 0; b < NKB; ++b) {
#pragma unroll
                for (int u = 0; u < T; ++u) pt[u] = Mma::mma(fp[u][b], bphi[b], pt[u]);
            }
        };
        // first operands of D: batch columns of a chunk, SG row tiles (group e) at a time
        Frag fd[2][SG];
        auto load_d = [&](const Op* yv, int ch, int e) {
#pragma unroll
            for (int u = 0; u < SG; ++u)
                if (e * SG + u < NT) fd[e & 1][u] = Mma::col(yv + ch * KB * SP + (e * SG + u) * 16, SP, lane);
        };
        auto direction = [&](const Op* yv, int ch, const f32x4* qt) {   // group 0 is there
            const Frag fb = Mma::second(qt);
#pragma unroll
            for (int e = 0; e < NSG; ++e) {
                if (e + 1 < NSG) load_d(yv, ch, e + 1);
                hold();
#pragma unroll
                for (int u = 0; u < SG; ++u)
                    if (e * SG + u < NT) dacc[e * SG + u] = Mma::mma(fd[e & 1][u], fb, dacc[e * SG + u]);
            }
        };
        auto chunk = [&](int ch, auto tiles) {
            constexpr int T = decltype(tiles)::value;
            const Op* yd = y + (NV == 3 ? 2 * MB * SP : 0);
            f32x4 pa[TPB], pb[TPB];
            Mma::Half fdh[T < TPB ? NT : 1];
            auto load_dt = [&]() {
                if constexpr (T < TPB) {
#pragma unroll
                    for (int mt = 0; mt < NT; ++mt) fdh[mt] = Mma::col_half(yd + ch * KB * SP + mt * 16, SP, lane, 0);
                } else {
                    load_d(yd, ch, 0);
                }
            };
            if constexpr (!ALIASED) {
                product(y, ch, pa, tiles);
                load_p(y + MB * SP, ch);
                hold();
            }
            load_dt();
            hold();
            if constexpr (ALIASED) product(y, ch, pa, tiles);
            else product(y + MB * SP, ch, pb, tiles);
            if constexpr (T == TPB) load_p(y, min(ch + 1, NCH - 1));   // the next chunk's (past the last: unused)
            hold();
#pragma unroll
            for (int u = 0; u < T; ++u) coeff(pa[u], ALIASED ? pa[u] : pb[u]);
            if constexpr (T < TPB) {
                const Mma::Half fb = Mma::second_half(pa[0]);
#pragma unroll
                for (int mt = 0; mt < NT; ++mt) dacc[mt] = Mma::mma_half(fdh[mt], fb, dacc[mt]);
            } else {
                direction(yd, ch, pa);
            }
        };
        if (act) {
            int ch = 0;
            if (kWide && nb > MB - 2 * KB) {   // (the rows past nb are zero)
#pragma unroll
                for (int x = 0; x < NCH; ++x) chunk(x, IntC<TPB>{});
                ch = NCH;
            }
#pragma unroll 1
            for (; ch * KB + 16 < nb; ++ch) chunk(ch, IntC<TPB>{});
            if (ch * KB < nb) chunk(ch, IntC<1>{});
        }

        if constexpr (NT > 4) __builtin_amdgcn_s_setprio(0);
        const float bl = beta * live, cb = g.b * invB;
        colsum = add_xor32(add_xor16(colsum));
        const float f1 = bl * invB, cmm = g.c * mA * mB;
        if constexpr (NBUF == 1) __syncthreads();      // every read of Phi and of the batch is done
        const float rv = cmm - cb * colsum;
        const float f2 = bl * rv;
        const bool pass_end = (p0.s == g.spp - 1 || t + 1 == g.end_step);
        if (act) {
            f32x4 yc[NT];
#pragma unroll
            for (int mt = 0; mt < NT; ++mt)   // (a row tile past NT is not used)
                yc[mt] = kWide ? ycw[kWide ? mt : 0] : *reinterpret_cast<const f32x4*>(&sm.ybar[2 * KPW + mt * 16 + 4 * q]);
#pragma unroll
            for (int mt = 0; mt < NT; ++mt) {
                const f32x4 ybc = yc[mt];
                const f32x4 d = dacc[mt];
                f32x4 v = phi_r[mt];
                if constexpr (COMP) {
                    f32x4 cv = comp[mt];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        // Kahan step
                        const float u = fmaf(f1, d[r], fmaf(f2, ybc[r], -cv[r]));
                        const float s = v[r] + u;
                        cv[r] = (s - v[r]) - u;
                        v[r] = s;
                    }
                    comp[mt] = cv;
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] += fmaf(f1, d[r], f2 * ybc[r]);
                }
                phi_r[mt] = v;
            }
            if (lane_live) {
#pragma unroll
                for (int mt = 0; mt < NT; ++mt) {
                        Mma::store4(&phi_n[i * SP + ((mt * 16 + 4 * q) ^ swl)], phi_r[mt]);
                }
            }
            if (pass_end) {
                // non-finite values propagate through every later step, so one
                // check per pass (and at the end of the run) sees any of them
#pragma unroll
                for (int mt = 0; mt < NT; ++mt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) bad |= !isfinite(phi_r[mt][r]);
            }
            if (Snap != nullptr && p0.s == g.spp - 1) {   // Phi to the snapshot of this pass
#pragma unroll
                for (int mt = 0; mt < NT; ++mt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int a = mt * 16 + 4 * q + r;
                        if (lane_live && a < k)
                            Snap[(size_t)p0.pass * k * k + (size_t)i * k + a] = phi_r[mt][r];
                    }
            }
        }
        if constexpr (!kSpec) {
            if constexpr (AHEAD == 1) commit_rows(y_n, p1.nb);
            if constexpr (AHEAD == 1) put_index(pf, t + 2, nidx);
        }
        scalars(p1, t + 1);
        __syncthreads();
        p0 = p1;
        p1 = p2;
        p2 = p3;
        p3 = AHEAD == 2 ? pf : next_step(p3, t + 4);
        cur ^= 1;
    }

    // ---- write back the master copy (and compensation)
#pragma unroll
    for (int mt = 0; mt < NT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int a = mt * 16 + 4 * q + r;
            if (lane_live && a < k) {
                Phi[(size_t)i * k + a] = phi_r[mt][r];
                if (Comp) {
                    if constexpr (COMP) Comp[(size_t)i * k + a] = comp[mt][r];
                    else Comp[(size_t)i * k + a] = 0.0f;
                }
            }
        }
    if (bad && g.nonfinite) *g.nonfinite = 1;
}

}  // namespace
}  // namespace otm
