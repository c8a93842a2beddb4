// The enumeration kernel of folded properties (instantiated in enum_fold_*.hip).
#pragma once

#include "enum_q8_impl.h"
#include "kernels_fold.h"

namespace ibmc {

typedef int v2i __attribute__((ext_vector_type(2)));

// First-layer activations of 16 points as the B operand: DW dwords per lane.
// Units per lane: KW / 4; K-block kb of 64 holds positions 64 kb + 16 g + b,
// the 32-wide form positions 8 g + b.
template <int KW>
struct FoldShape {
    static constexpr bool K32 = KW == 32;
    static constexpr int KB = K32 ? 1 : KW / 64;      // MFMAs per 16 x 16 tile
    static constexpr int DW = KW / 16;                // dwords of activations per lane
    static constexpr int WV = KW / 32;                // 16-byte weight vectors per lane and point
    static constexpr int TILE = K32 ? 512 : 1024;     // bytes of one A tile
    static constexpr int NT = KW <= 64 ? 4 : 2;
    // position of int16 vector v (8 units) of lane group g
    __device__ static constexpr int pos(int v, int g) { return K32 ? g * 8 : (v >> 1) * 64 + g * 16 + (v & 1) * 8; }
};

// Eight units of one point: u = base + e w in 16-bit halves, saturated to the
// requantiser's window by doubling, whose byte 1 is then 2 (a - 64) plus a low
// bit that is masked off.  Two dwords of four units each.
// WIDE: the products may leave the room that the clamped base keeps, so the
// sum saturates, and halvings extra doublings bring the window to 16 bits.
template <bool WIDE>
__device__ __forceinline__ void fold_units(const v4i &b, const v4i &w, short2_t e2, int halvings, int &d0, int &d1) {
    int r[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        short2_t u;
        if constexpr (WIDE) {
            u = __builtin_elementwise_add_sat(as_s2(b[t]), (short2_t)(e2 * as_s2(w[t])));
            for (int h = 0; h < halvings; ++h) u = __builtin_elementwise_add_sat(u, u);
        } else {
            u = as_s2(b[t]) + e2 * as_s2(w[t]);
        }
        r[t] = as_int(__builtin_elementwise_add_sat(u, u));
    }
    d0 = (int)(__builtin_amdgcn_perm(r[1], r[0], 0x07050301u) & 0xfefefefeu);
    d1 = (int)(__builtin_amdgcn_perm(r[3], r[2], 0x07050301u) & 0xfefefefeu);
}

template <int KW>
__device__ __forceinline__ v4i fold_mfma(const int8_t *tile, const int (&a)[KW / 16], v4i acc, int lane) {
    if constexpr (KW == 32) {
        const long A = *reinterpret_cast<const long *>(tile + lane * 8);
        const v2i b = {a[0], a[1]};
        return __builtin_amdgcn_mfma_i32_16x16x32_i8(A, __builtin_bit_cast(long, b), acc, 0, 0, 0);
    } else {
#pragma unroll
        for (int kb = 0; kb < KW / 64; ++kb) {
            const v4i A = *reinterpret_cast<const v4i *>(tile + kb * 1024 + lane * 16);
            const v4i b = {a[4 * kb], a[4 * kb + 1], a[4 * kb + 2], a[4 * kb + 3]};
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(A, b, acc, 0, 0, 0);
        }
        return acc;
    }
}

// Last job whose first chunk is at or before `chunk`: two rounds of 64-way
// comparison instead of a serial search (n_jobs <= 4096).
__device__ __forceinline__ int fold_find_job(const EnumJob *jobs, int n_jobs, int64_t chunk, int lane) {
    const int step = (n_jobs + 63) >> 6;
    int i = lane * step;
    bool le = i < n_jobs && gld(&jobs[min(i, n_jobs - 1)].chunk_begin) <= chunk;
    const int blk = __popcll(__ballot(le)) - 1;          // job 0 starts at chunk 0
    int lo = blk * step;
    if (step > 1) {
        i = lo + lane;
        le = lane < step && i < n_jobs && gld(&jobs[min(i, n_jobs - 1)].chunk_begin) <= chunk;
        lo += __popcll(__ballot(le)) - 1;
    }
    return wave_uniform(lo);
}

// Enumeration over folded properties.  L: weight layers; KW: padded live
// units of layer 1; WIDE: see fold_units; EPI: layer 2's requantiser shift is
// 7 (saturating epilogue), else any.  A workgroup takes tickets of 4 * batch
// chunks of one job, a quarter per wave, and stages the property's later
// layers in LDS when the property changes.  A chunk is 16 NT last-element
// positions for each segment of a group; where a segment has fewer positions
// left, the tiles of one step take several segments.
//
// Why: on the 784-256-256-10 blob images 20-89 of 256 first-layer units and
// 84-217 of 256 second-layer units can change, so a point needs 7 to 30 of the
// 68 MFMAs and a quarter of the first-layer work of the unreduced network.
// Measured (64 images, 707 M points, one launch each): 41.5 -> 13.2 ms of
// enumeration.  Bound: the vector ALU (per 64 points about 96 instructions of
// first layer and 20 per 16-row tile of layer 2); three workgroups per CU
// hide the chunk set-up's loads, so nothing is prefetched across chunks.
//
// The output layer computes, for every class c, the difference to the clean
// label's logit E_c = z_c - z_label + [c < label] (scaled by 2 for two-layer
// networks): a point is a counterexample iff some E_c > 0.
template <int L, int KW, bool WIDE, int EPI>
__global__ void __launch_bounds__(256, KW <= 64 ? 3 : 2) enum_fold_kernel(FoldParams P) {
    using S = FoldShape<KW>;
    constexpr int NT = S::NT, CH = 16 * NT, DW = S::DW, WV = S::WV;
    constexpr int SIG = L == 2 ? 2 : 1;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63, wave = wave_uniform((int)(threadIdx.x >> 6));
    const int j16 = lane & 15, g = lane >> 4;
    char *wbase = smem + P.stage_max + wave * (kFoldGroup * KW * 2 + kFoldGroup * 8);
    int16_t *const base16 = reinterpret_cast<int16_t *>(wbase);
    int64_t *const r0s = reinterpret_cast<int64_t *>(wbase + kFoldGroup * KW * 2);
    volatile int64_t *const ticket_s =
        reinterpret_cast<volatile int64_t *>(smem + P.stage_max + 4 * (kFoldGroup * KW * 2 + kFoldGroup * 8));
    const int8_t *const st = reinterpret_cast<const int8_t *>(smem);

    int cur_prop = -1, fetches = 0;
    // of the current property
    const int16_t *W1 = nullptr, *etab = nullptr;
    const int32_t *v0 = nullptr;
    int mt2 = 0, kbo = 0, two = 0, s2 = 0, halvings = 0, vlo = 0, vhi = 0, label = 0;
    int off_b2 = 0, off_wo = 0, off_y = 0;
    int lowm = 0;   // bit t: this lane's class 4 g + t has a lower index than the label
    v4i bo4 = v4i{0, 0, 0, 0};
    int lo2 = -64, hi2 = 63;
    asm("" : "+v"(lo2));
    asm("" : "+v"(hi2));
    // records: slots come in blocks of kRecBlock from one atomic
    int64_t rnext = 0, rend = 0;

    while (true) {
        if (threadIdx.x == 0) {
            int64_t t = -1;
            if (!(P.abort_host && (++fetches & 7) == 0 && *P.abort_host)) t = (int64_t)atomicAdd(P.queue, 1ull);
            *ticket_s = t;
        }
        __syncthreads();
        const int64_t ticket = (int64_t)wave_uniform((unsigned long long)*ticket_s);
        const int64_t start = ticket * 4 * P.batch;
        if (ticket < 0 || start >= P.total_chunks) break;
        const int job = fold_find_job(P.jobs, P.n_jobs, start, lane);
        const int prop = wave_uniform(P.jobs[job].prop);
        if (prop != cur_prop) {
            cur_prop = prop;
            const FoldRun &R = P.runs[prop];
            const int bytes = R.stage_bytes;
            const v4i *src = reinterpret_cast<const v4i *>(R.stage);
            for (int t = threadIdx.x; t < bytes / 16; t += 256) reinterpret_cast<v4i *>(smem)[t] = gld(src + t);
            W1 = R.W1;
            etab = R.etab;
            v0 = R.v0;
            mt2 = wave_uniform(R.mt2);
            kbo = wave_uniform(R.kbo);
            two = wave_uniform(R.two);
            s2 = wave_uniform(R.s2);
            halvings = wave_uniform(R.halvings);
            vlo = wave_uniform(R.vlo);
            vhi = wave_uniform(R.vhi);
            label = wave_uniform(R.label);
            constexpr int OT = L == 2 ? S::KB * S::TILE : 1024;   // bytes of the output tiles of one K-block
            off_b2 = mt2 * S::KB * S::TILE;
            off_wo = off_b2 + mt2 * 64;
            off_y = off_wo + kbo * OT;
            lowm = 0;
#pragma unroll
            for (int t = 0; t < 4; ++t) lowm |= (4 * g + t < label ? 1 : 0) << t;
            __syncthreads();
            const int4 b = *reinterpret_cast<const int4 *>(st + off_y + (two ? kbo * OT : 0) + g * 16);
            bo4 = v4i{b.x, b.y, b.z, b.w};
        } else {
            __syncthreads();
        }
        Cursor c;
        const int64_t c0 = start + (int64_t)wave * P.batch;
        const int64_t c1 = min(c0 + P.batch, (int64_t)wave_uniform((unsigned long long)P.jobs[job].chunk_end));
        if (c0 >= c1) continue;
        cursor_job_start<CH, FoldParams>(c, P, job);
        cursor_decode_in_job<CH, FoldParams>(c, P, job, c0);
        unsigned ncex = 0, nties = 0;
        bool seg = true, r0ok = false;
        while (true) {
            if (seg) {
                // bases of the group's segments
                r0ok = false;
                Cursor ct = c;
                for (int w = 0; w < c.nw; ++w) {
                    int pp[kMaxK], ee[kMaxK];
#pragma unroll
                    for (int j = 0; j < kMaxK; ++j) {
                        pp[j] = ee[j] = 0;
                        if (j < ct.k - 1) {
                            pp[j] = ct.pre[j];
                            ee[j] = wave_uniform((int)gld(etab + ct.pre[j] * ct.m + ct.dg[j]));
                        }
                    }
#pragma unroll
                    for (int r = 0; r < (KW + 63) / 64; ++r) {
                        const int q = (lane & (KW - 1)) + 64 * r;
                        int v = gld(v0 + q);
#pragma unroll
                        for (int j = 0; j < kMaxK; ++j)
                            if (j < ct.k - 1) v += ee[j] * (int)gld(W1 + pp[j] * KW + q);
                        base16[w * KW + q] = (int16_t)min(max(v, vlo), vhi);
                    }
                    if (w + 1 < c.nw) seg_step(ct);
                }
                __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): LDS writes done
                __builtin_amdgcn_wave_barrier();
            }
            // positions of the chunk's tiles
            const int obase = (int)c.ch * CH;
            const int left = ((int)c.seglen - obase + 15) >> 4;      // >= 1 tiles left in the segment
            const int lp = left >= NT ? (NT == 4 ? 2 : 1) : (left > 2 ? 2 : left - 1);   // log2 of the position tiles
            const int np = 1 << lp, sp = NT >> lp;                   // position tiles, segments per step
            const int nw = c.nw;
            int cand[NT], plast[NT];
            unsigned ok = 0;   // bit t: this lane's position of tile t exists
            short2_t e2[NT];
            v4i wv[NT][WV];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                int o = obase + (t & (np - 1)) * 16 + j16;
                if (o < (int)c.seglen) ok |= 1u << t;
                else o = 0;
                plast[t] = c.q + 1 + (int)div_m(c, (unsigned)o);
                cand[t] = (c.q + 1) * c.m + o;
                const short e = gld(etab + cand[t]);
                e2[t] = short2_t{e, e};
                const int16_t *wp = W1 + plast[t] * KW;
#pragma unroll
                for (int v = 0; v < WV; ++v) wv[t][v] = gld(reinterpret_cast<const v4i *>(wp + S::pos(v, g)));
            }
            for (int w = 0; w < nw; w += sp) {
                // ---- layer 1
                int a1[NT][DW];
                if (sp == 1) {
#pragma unroll
                    for (int v = 0; v < WV; ++v) {
                        const v4i b = *reinterpret_cast<const v4i *>(base16 + w * KW + S::pos(v, g));
#pragma unroll
                        for (int t = 0; t < NT; ++t)
                            fold_units<WIDE>(b, wv[t][v], e2[t], halvings, a1[t][2 * v], a1[t][2 * v + 1]);
                    }
                } else {
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        const int ws = min(w + (t >> lp), nw - 1);
#pragma unroll
                        for (int v = 0; v < WV; ++v) {
                            const v4i b = *reinterpret_cast<const v4i *>(base16 + ws * KW + S::pos(v, g));
                            fold_units<WIDE>(b, wv[t][v], e2[t], halvings, a1[t][2 * v], a1[t][2 * v + 1]);
                        }
                    }
                }
                // ---- later layers
                v4i E[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t) E[t] = bo4;
                if constexpr (L == 2) {
#pragma unroll
                    for (int t = 0; t < NT; ++t) E[t] = fold_mfma<KW>(st + off_wo, a1[t], E[t], lane);
                    if (two) {
#pragma unroll
                        for (int t = 0; t < NT; ++t) E[t] = fold_mfma<KW>(st + off_y, a1[t], E[t], lane);
                    }
                } else {
                    auto tile = [&](int mt, v4i (&acc)[NT]) __attribute__((always_inline)) {
                        const int4 b = *reinterpret_cast<const int4 *>(st + off_b2 + mt * 64 + g * 16);
#pragma unroll
                        for (int t = 0; t < NT; ++t)
                            acc[t] = fold_mfma<KW>(st + mt * S::KB * S::TILE, a1[t], v4i{b.x, b.y, b.z, b.w}, lane);
                    };
                    auto requant = [&](const v4i &acc) __attribute__((always_inline)) -> int {
                        return EPI ? requant4_sat(acc) : requant4_clamp(acc, s2, lo2, hi2);
                    };
                    auto output = [&](int kb, const v4i (&a2)[NT]) __attribute__((always_inline)) {
                        const v4i A = *reinterpret_cast<const v4i *>(st + off_wo + kb * 1024 + lane * 16);
#pragma unroll
                        for (int t = 0; t < NT; ++t) E[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A, a2[t], E[t], 0, 0, 0);
                        if (two) {
                            const v4i Y = *reinterpret_cast<const v4i *>(st + off_y + kb * 1024 + lane * 16);
#pragma unroll
                            for (int t = 0; t < NT; ++t)
                                E[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(Y, a2[t], E[t], 0, 0, 0);
                        }
                    };
                    const int full = mt2 >> 2;
                    for (int kb = 0; kb < full; ++kb) {
                        v4i a2[NT], acc[NT], accn[NT];
                        tile(4 * kb, acc);
#pragma unroll
                        for (int z = 0; z < 4; ++z) {
                            if (z < 3) tile(4 * kb + z + 1, accn);
#pragma unroll
                            for (int t = 0; t < NT; ++t) {
                                a2[t][z] = requant(acc[t]);
                                acc[t] = accn[t];
                            }
                        }
                        output(kb, a2);
                    }
                    if (mt2 & 3) {
                        // the last one to three tiles; the others' weights are zero in the output layer
                        v4i a2[NT], acc[NT];
#pragma unroll
                        for (int t = 0; t < NT; ++t) a2[t] = v4i{0, 0, 0, 0};
#pragma unroll
                        for (int z = 0; z < 3; ++z) {
                            if (z < (mt2 & 3)) {
                                tile(4 * full + z, acc);
#pragma unroll
                                for (int t = 0; t < NT; ++t) a2[t][z] = requant(acc[t]);
                            }
                        }
                        output(full, a2);
                    }
                }
                // ---- decisions
                unsigned long long hot = 0;
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    hot |= __ballot(max(max(E[t][0], E[t][1]), max(E[t][2], E[t][3])) >= 0);
                if (hot) {
                    unsigned viol[NT];
                    int lab[NT], n = 0;
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        const bool here = ((ok >> t) & 1u) && w + (t >> lp) < nw;
                        const unsigned vmask = (unsigned)(__ballot(here) & 0xffffull);
                        unsigned long long pos = 0, eq = 0;
                        v4i d;
#pragma unroll
                        for (int z = 0; z < 4; ++z) {
                            pos |= __ballot(E[t][z] > 0);
                            d[z] = E[t][z] - (((lowm >> z) & 1) ? SIG : 0);
                            eq |= __ballot(d[z] == 0);
                        }
                        viol[t] = fold_groups(pos) & vmask;
                        nties += __popc(fold_groups(eq) & vmask & ~viol[t]);
                        lab[t] = 0;
                        if (viol[t]) {
                            int bv = INT32_MIN, bi = 0x7fffffff, bc = 0;
                            argmax_tile<false>(d, 0, g, 16, bv, bi, bc);
                            argmax_combine(bv, bi, bc);
                            lab[t] = bi;
                            // the label itself stands at difference 0
                            const bool tie = bc + (bv == 0 ? 1 : 0) > 1;
                            nties += (unsigned)__popcll(__ballot(g == 0 && ((viol[t] >> j16) & 1u) && tie));
                            n += __popc(viol[t]);
                        }
                    }
                    if (n) {
                        if (!r0ok) {
                            r0ok = true;
                            Cursor ct = c;
                            for (int v = 0; v < c.nw; ++v) {
                                const EmitInfo ei = make_emit_info<FoldParams>(ct, P);
                                if (lane == 0) r0s[v] = ei.r0;
                                if (v + 1 < c.nw) seg_step(ct);
                            }
                            __builtin_amdgcn_s_waitcnt(0xc07f);
                            __builtin_amdgcn_wave_barrier();
                        }
                        ncex += n;
                        const int64_t room = rend - rnext;
                        int64_t nb = 0;
                        if (n > room) {
                            unsigned long long s = 0;
                            if (lane == 0) s = atomicAdd(P.rec_count, (unsigned long long)kRecBlock);
                            nb = (int64_t)wave_uniform(s);
                        }
                        int64_t mk = 1;
                        for (int j = 0; j < c.k; ++j) mk *= c.m;
                        int before = 0;
#pragma unroll
                        for (int t = 0; t < NT; ++t) {
                            if (g == 0 && ((viol[t] >> j16) & 1u)) {
                                const int at = before + __popc(viol[t] & ((1u << j16) - 1u));
                                const int64_t idx = at < room ? rnext + at : nb + (at - room);
                                if (idx < P.rec_cap) {
                                    DevRec r;
                                    r.rank = r0s[w + (t >> lp)] + (int64_t)plast[t] * mk + (cand[t] - plast[t] * c.m);
                                    r.prop = c.prop;
                                    r.klab = (c.k << 24) | (lab[t] & 0xffffff);
                                    P.recs[idx] = r;
                                }
                            }
                            before += __popc(viol[t]);
                        }
                        if (n > room) {
                            rnext = nb + (n - room);
                            rend = nb + kRecBlock;
                        } else {
                            rnext += n;
                        }
                    }
                }
            }
            if (c.chunk + 1 >= c1) break;
            seg = cursor_next<CH, FoldParams>(c, P);
        }
        if (lane == 0) {
            if (ncex) atomicAdd(P.slot_cex + c.slot, (unsigned long long)ncex);
            if (nties) atomicAdd(P.slot_ties + c.slot, (unsigned long long)nties);
        }
    }
    // sentinels into the unused slots of the wave's last block
    const int64_t idx = rnext + lane;
    if (idx < rend && idx < P.rec_cap) {
        DevRec r;
        r.rank = -1;
        r.prop = -1;
        r.klab = 0;
        P.recs[idx] = r;
    }
}

#define IBMC_FOLD(L_, KW_, WIDE_, EPI_) \
    {L_, KW_, WIDE_, EPI_, FoldShape<KW_>::NT, reinterpret_cast<const void *>(&enum_fold_kernel<L_, KW_, WIDE_, EPI_>)}

}  // namespace ibmc
