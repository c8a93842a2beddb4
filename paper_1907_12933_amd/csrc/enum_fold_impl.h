// The enumeration kernel of folded properties (instantiated in enum_fold_*.hip).
#pragma once

#include "enum_q8_impl.h"
#include "fold_search.h"
#include "kernels_fold.h"

namespace ibmc {

typedef int v2i __attribute__((ext_vector_type(2)));

// First-layer positions of a folded property: KB K-blocks, in each of which
// lane group g of the B operand holds UB units, positions kb * 4 UB + g UB + b
// (UB = 8: the 32-wide MFMA; 12 and 16: the 64-wide one, whose last four bytes
// per lane stay zero for 12).
template <int KW>
struct FoldShape {
    static constexpr int KB = fold_blocks(KW), UB = fold_units_per_block(KW);
    static constexpr bool K32 = UB == 8;
    static constexpr int U = KB * UB;                 // units per lane
    static constexpr int DB = K32 ? 2 : 4;            // dwords of a K-block's B operand per lane
    static constexpr int DW = KB * DB;
    static constexpr int TILE = K32 ? 512 : 1024;     // bytes of one A tile
    static constexpr int NT = KW <= 64 ? 4 : 2;
    // position of unit group v (four units) of lane group g
    __device__ static constexpr int pos(int v, int g) {
        return v / (UB / 4) * 4 * UB + g * UB + v % (UB / 4) * 4;
    }
    // its dword in the B operand
    __device__ static constexpr int dword(int v) { return v / (UB / 4) * DB + v % (UB / 4); }
};

// Base + 32-bit byte offset: a scalar base and one vector offset register.
template <class T>
__device__ __forceinline__ T gld_at(const void *base, unsigned off) {
    typedef const __attribute__((address_space(1))) char *gptr;
    return *(const __attribute__((address_space(1))) T *)((gptr)base + off);
}

// Four units of one point: u = base + e w in 16-bit halves, saturated to the
// requantiser's window by doubling, whose byte 1 is then 2 (a - 64) plus a low
// bit that is masked off.
// WIDE: the products may leave the room that the clamped base keeps, so the
// sum saturates, and halvings extra doublings bring the window to 16 bits.
template <bool WIDE>
__device__ __forceinline__ int fold_units(const v2i &b, const v2i &w, short2_t e2, int halvings) {
    int r[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        short2_t u;
        if constexpr (WIDE) {
            u = __builtin_elementwise_add_sat(as_s2(b[t]), (short2_t)(e2 * as_s2(w[t])));
            for (int h = 0; h < halvings; ++h) u = __builtin_elementwise_add_sat(u, u);
        } else {
            u = as_s2(b[t]) + e2 * as_s2(w[t]);
        }
        r[t] = as_int(__builtin_elementwise_add_sat(u, u));
    }
    return (int)(__builtin_amdgcn_perm(r[1], r[0], 0x07050301u) & 0xfefefefeu);
}

// Requantiser of four accumulators whose activation cannot leave the int16
// saturation's ends: 2 u - 32768 never above -1 (byte a - 128), or 2 u never
// below 0 (byte a).
__device__ __forceinline__ int requant4_sat_uncapped(v4i acc) {
    const short2_t p0 = __builtin_amdgcn_cvt_pk_i16(acc[0], acc[1]), p1 = __builtin_amdgcn_cvt_pk_i16(acc[2], acc[3]);
    return (int)__builtin_amdgcn_perm(__builtin_bit_cast(unsigned, p1), __builtin_bit_cast(unsigned, p0), 0x07050301u);
}

template <int KW>
__device__ __forceinline__ v4i fold_mfma(const int8_t *tile, const int (&a)[FoldShape<KW>::DW], v4i acc, int lane) {
    if constexpr (FoldShape<KW>::K32) {
        const long A = *reinterpret_cast<const long *>(tile + lane * 8);
        const v2i b = {a[0], a[1]};
        return __builtin_amdgcn_mfma_i32_16x16x32_i8(A, __builtin_bit_cast(long, b), acc, 0, 0, 0);
    } else {
#pragma unroll
        for (int kb = 0; kb < FoldShape<KW>::KB; ++kb) {
            const v4i A = *reinterpret_cast<const v4i *>(tile + kb * 1024 + lane * 16);
            const v4i b = {a[4 * kb], a[4 * kb + 1], a[4 * kb + 2], a[4 * kb + 3]};
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(A, b, acc, 0, 0, 0);
        }
        return acc;
    }
}

// Maximum over the four lane groups of a point.
__device__ __forceinline__ int rows_max(int x) {
    const LanePair a = swap16(x);
    const LanePair b = swap32(max(a.lo, a.hi));
    return max(b.lo, b.hi);
}

// Last job whose first chunk is at or before `chunk` (job 0 starts at chunk 0):
// 64-way comparison instead of a serial search.
__device__ __forceinline__ int fold_find_job(const EnumJob *jobs, int n_jobs, int64_t chunk, int lane) {
    return wave_uniform(fold_search(n_jobs, [&](int first, int step, int n) __attribute__((always_inline)) {
        const int i = lane * step;
        return __popcll(__ballot(i < n && gld(&jobs[first + min(i, n - 1)].chunk_begin) <= chunk));
    }));
}

// LDS of one wave.
template <int KW>
struct FoldWave {
    int16_t base[kFoldGroup * KW];       // first-layer bases of the group's segments
    int64_t r0[kFoldGroup], mk;          // their rank offsets, m^k (written when a point is recorded)
    int64_t pad_;
    int32_t pc[64];                      // prefix element j of segment w at 8 w + j: candidate,
    int16_t pp[64], pe[64];              // pixel, effective delta
};

__device__ __forceinline__ void fold_lds_sync() {
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave's LDS writes are done
    __builtin_amdgcn_wave_barrier();
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
// 89-176 of 256 second-layer units can change, so a point needs 12 to 36 of
// the 68 MFMAs and an eighth to a third of the first-layer work of the
// unreduced network.  Measured (64 images, 707 M points): enumeration 41.5 ->
// 12.0 ms; 78 G points/s on images without counterexamples (48 wide), 50 on
// the others.  Bound: the vector ALU, busy 77 % of the cycles (per 64 points
// of the 48-wide form 350 instructions: 72 of first layer, 24 to 40 per pair
// of layer-2 tiles, about 25 of chunk set-up).  Three workgroups per CU hide
// the chunk set-up's loads, so nothing is prefetched across chunks; the next
// pair's weight tiles are read from LDS under the current pair's
// requantisation (unprefetched single tiles: 13.1 ms).
//
// Layer 2 runs its tiles in pairs, whose packed activations are one 32-wide
// B operand of the output layer.  Under the saturating epilogue (shift 7) a
// unit that never exceeds 127 needs no cap (2 u - 32768 stays below 0), nor
// does one that never falls below 0 if it enters as 2 u (byte a, saturated at
// 127); such units fill the leading pairs, two instructions in five saved.
//
// The output layer computes, for every class c, the difference to the clean
// label's logit E_c = z_c - z_label + [c < label] (scaled by 2 for two-layer
// networks): a point is a counterexample iff some E_c > 0.
template <int L, int KW, bool WIDE, int EPI>
__global__ void __launch_bounds__(256, KW <= 64 ? 3 : 2) enum_fold_kernel(FoldParams P) {
    using S = FoldShape<KW>;
    constexpr int NT = S::NT, CH = 16 * NT, DW = S::DW, UG = S::U / 4;
    constexpr int SIG = L == 2 ? 2 : 1;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63, wave = wave_uniform((int)(threadIdx.x >> 6));
    const int j16 = lane & 15, g = lane >> 4;
    FoldWave<KW> &ws = *reinterpret_cast<FoldWave<KW> *>(smem + P.stage_max + wave * sizeof(FoldWave<KW>));
    volatile int64_t *const ticket_s =
        reinterpret_cast<volatile int64_t *>(smem + P.stage_max + 4 * sizeof(FoldWave<KW>));
    const int8_t *const st = reinterpret_cast<const int8_t *>(smem);

    int cur_prop = -1, fetches = 0;
    // of the current property
    const void *W1 = nullptr, *etab = nullptr;
    const int32_t *v0 = nullptr;
    int npair = 0, free_pairs = 0, two = 0, s2 = 0, halvings = 0, vlo = 0, vhi = 0;
    int off_b2 = 0, off_wo = 0, off_y = 0;
    v4i bo4 = v4i{0, 0, 0, 0};
    v4i adj = v4i{0, 0, 0, 0};   // SIG where this lane's class 4 g + z has a lower index than the label
    int lo2 = -64, hi2 = 63;
    asm("" : "+v"(lo2));
    asm("" : "+v"(hi2));
    // records: slots come in blocks from one atomic, 8 at first (a wave with a
    // few records leaves few unused), then twice as many, up to kRecBlock
    int64_t rnext = 0, rend = 0;
    int rblock = 8;

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
            W1 = reinterpret_cast<const void *>(wave_uniform((unsigned long long)R.W1));
            etab = reinterpret_cast<const void *>(wave_uniform((unsigned long long)R.etab));
            v0 = R.v0;
            npair = wave_uniform(R.npair);
            free_pairs = wave_uniform(R.free_pairs);
            two = wave_uniform(R.two);
            s2 = wave_uniform(R.s2);
            halvings = wave_uniform(R.halvings);
            vlo = wave_uniform(R.vlo);
            vhi = wave_uniform(R.vhi);
            const int out_bytes = L == 2 ? S::KB * S::TILE : npair * 512, label = wave_uniform(R.label);
            off_b2 = 2 * npair * S::KB * S::TILE;
            off_wo = off_b2 + npair * 128;
            off_y = off_wo + out_bytes;
#pragma unroll
            for (int z = 0; z < 4; ++z) adj[z] = 4 * g + z < label ? SIG : 0;
            __syncthreads();
            const int4 b = *reinterpret_cast<const int4 *>(st + off_y + (two ? out_bytes : 0) + g * 16);
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
                // bases of the group's segments: their prefix elements first (lane
                // 8 w + j: element j of segment w), then every base at once
                r0ok = false;
                const int np = c.k - 1, nw = c.nw;
                if (np > 0) {
                    Cursor ct = c;
                    int cnd = 0, pix = 0;
                    for (int w = 0; w < nw; ++w) {
#pragma unroll
                        for (int j = 0; j < kMaxK - 1; ++j)
                            if (j < np && lane == 8 * w + j) {
                                cnd = ct.pre[j] * ct.m + ct.dg[j];
                                pix = ct.pre[j];
                            }
                        if (w + 1 < nw) seg_step(ct);
                    }
                    ws.pe[lane] = gld_at<int16_t>(etab, (unsigned)cnd * 2u);
                    ws.pc[lane] = cnd;
                    ws.pp[lane] = (int16_t)pix;
                    fold_lds_sync();
                }
                constexpr int IT = kFoldGroup * KW / 64;   // bases of 64 positions
                // (KW = 256: in two rounds, for the registers)
                constexpr int RN = IT > 16 ? 16 : IT;
                for (int r0 = 0; r0 < IT; r0 += RN) {
                    if (64 * r0 / KW >= nw) break;
                    int v[RN];
#pragma unroll
                    for (int r = 0; r < RN; ++r) v[r] = gld(v0 + (lane + 64 * (r0 + r)) % KW);
                    for (int j = 0; j < np; ++j) {
#pragma unroll
                        for (int r = 0; r < RN; ++r) {
                            const int at = lane + 64 * (r0 + r), w = at / KW, q = at - w * KW;
                            v[r] += (int)ws.pe[8 * w + j] *
                                    (int)gld_at<int16_t>(W1, (unsigned)((int)ws.pp[8 * w + j] * KW + q) * 2u);
                        }
                    }
#pragma unroll
                    for (int r = 0; r < RN; ++r) ws.base[lane + 64 * (r0 + r)] = (int16_t)min(max(v[r], vlo), vhi);
                }
                fold_lds_sync();
            }
            // positions of the chunk's tiles
            const int obase = (int)c.ch * CH;
            const int left = ((int)c.seglen - obase + 15) >> 4;      // >= 1 tiles left in the segment
            const int lp = left >= NT ? (NT == 4 ? 2 : 1) : (left > 2 ? 2 : left - 1);   // log2 of the position tiles
            const int npt = 1 << lp, sp = NT >> lp;                  // position tiles, segments per step
            const int nw = c.nw;
            int plast[NT], ilast[NT];
            unsigned ok = 0;   // bit t: this lane's position of tile t exists
            short2_t e2[NT];
            v2i wv[NT][UG];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                int o = obase + (t & (npt - 1)) * 16 + j16;
                if (o < (int)c.seglen) ok |= 1u << t;
                else o = 0;
                const int dp = (int)div_m(c, (unsigned)o);
                plast[t] = c.q + 1 + dp;
                ilast[t] = o - dp * c.m;
                const short e = gld_at<short>(etab, (unsigned)((c.q + 1) * c.m + o) * 2u);
                e2[t] = short2_t{e, e};
                const unsigned wo = (unsigned)(plast[t] * KW) * 2u;
                if constexpr (S::UB % 8 == 0) {
#pragma unroll
                    for (int v = 0; v < UG; v += 2) {
                        const v4i x = gld_at<v4i>(W1, wo + (unsigned)S::pos(v, g) * 2u);
                        wv[t][v] = v2i{x[0], x[1]};
                        wv[t][v + 1] = v2i{x[2], x[3]};
                    }
                } else {
#pragma unroll
                    for (int v = 0; v < UG; ++v) wv[t][v] = gld_at<v2i>(W1, wo + (unsigned)S::pos(v, g) * 2u);
                }
            }
            for (int w = 0; w < nw; w += sp) {
                // ---- layer 1
                int a1[NT][DW];
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int d = 0; d < DW; ++d) a1[t][d] = 0;
                if (sp == 1) {
#pragma unroll
                    for (int v = 0; v < UG; ++v) {
                        const v2i b = *reinterpret_cast<const v2i *>(&ws.base[w * KW + S::pos(v, g)]);
#pragma unroll
                        for (int t = 0; t < NT; ++t) a1[t][S::dword(v)] = fold_units<WIDE>(b, wv[t][v], e2[t], halvings);
                    }
                } else {
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        const int wt = min(w + (t >> lp), nw - 1);
#pragma unroll
                        for (int v = 0; v < UG; ++v) {
                            const v2i b = *reinterpret_cast<const v2i *>(&ws.base[wt * KW + S::pos(v, g)]);
                            a1[t][S::dword(v)] = fold_units<WIDE>(b, wv[t][v], e2[t], halvings);
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
                    // pairs of 16-row tiles: the next pair's weights and init are read
                    // from LDS ahead, the second tile's MFMAs run beside the
                    // first's requantisation
                    struct Pair {
                        v4i A[2][S::K32 ? 1 : S::KB], b[2];
                    };
                    auto fetch = [&](int p, Pair &x) __attribute__((always_inline)) {
#pragma unroll
                        for (int z = 0; z < 2; ++z) {
                            x.b[z] = *reinterpret_cast<const v4i *>(st + off_b2 + (2 * p + z) * 64 + g * 16);
                            const int8_t *at = st + (2 * p + z) * S::KB * S::TILE;
                            if constexpr (S::K32) {
                                const v2i a = *reinterpret_cast<const v2i *>(at + lane * 8);
                                x.A[z][0] = v4i{a[0], a[1], 0, 0};
                            } else {
#pragma unroll
                                for (int kb = 0; kb < S::KB; ++kb) x.A[z][kb] = *reinterpret_cast<const v4i *>(at + kb * 1024 + lane * 16);
                            }
                        }
                    };
                    Pair cur;
                    fetch(0, cur);
                    auto pair = [&](int p, bool cap) __attribute__((always_inline)) {
                        const long W = *reinterpret_cast<const long *>(st + off_wo + p * 512 + lane * 8);
                        v4i acc[2][NT];
#pragma unroll
                        for (int z = 0; z < 2; ++z)
#pragma unroll
                            for (int t = 0; t < NT; ++t) {
                                acc[z][t] = cur.b[z];
                                if constexpr (S::K32) {
                                    acc[z][t] = __builtin_amdgcn_mfma_i32_16x16x32_i8(
                                        __builtin_bit_cast(long, v2i{cur.A[z][0][0], cur.A[z][0][1]}),
                                        __builtin_bit_cast(long, v2i{a1[t][0], a1[t][1]}), acc[z][t], 0, 0, 0);
                                } else {
#pragma unroll
                                    for (int kb = 0; kb < S::KB; ++kb)
                                        acc[z][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(
                                            cur.A[z][kb], v4i{a1[t][4 * kb], a1[t][4 * kb + 1], a1[t][4 * kb + 2], a1[t][4 * kb + 3]},
                                            acc[z][t], 0, 0, 0);
                                }
                            }
                        fetch(min(p + 1, npair - 1), cur);
                        v2i a2[NT];
#pragma unroll
                        for (int z = 0; z < 2; ++z)
#pragma unroll
                            for (int t = 0; t < NT; ++t)
                                a2[t][z] = !EPI ? requant4_clamp(acc[z][t], s2, lo2, hi2)
                                           : cap ? requant4_sat(acc[z][t]) : requant4_sat_uncapped(acc[z][t]);
#pragma unroll
                        for (int t = 0; t < NT; ++t)
                            E[t] = __builtin_amdgcn_mfma_i32_16x16x32_i8(W, __builtin_bit_cast(long, a2[t]), E[t], 0, 0, 0);
                        if (two) {
                            const long Y = *reinterpret_cast<const long *>(st + off_y + p * 512 + lane * 8);
#pragma unroll
                            for (int t = 0; t < NT; ++t)
                                E[t] = __builtin_amdgcn_mfma_i32_16x16x32_i8(Y, __builtin_bit_cast(long, a2[t]), E[t], 0, 0, 0);
                        }
                    };
                    int p = 0;
                    if constexpr (EPI)
                        for (; p < free_pairs; ++p) pair(p, false);
                    for (; p < npair; ++p) pair(p, true);
                }
                // ---- decisions: nothing to do while every difference is negative
                int top[NT];
                unsigned long long hot = 0;
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    top[t] = max(max(E[t][0], E[t][1]), max(E[t][2], E[t][3]));
                    hot |= __ballot(top[t] >= 0);
                }
                if (hot == 0) continue;
                // lane 16 t + j16 reports point j16 of tile t
                unsigned long long vmask = 0;   // its counterexamples
                int lab = 0;
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const unsigned here = w + (t >> lp) < nw ? (unsigned)(__ballot((ok >> t) & 1u) & 0xffffull) : 0u;
                    const int mx = rows_max(top[t]);
                    const unsigned viol = (unsigned)__ballot(mx > 0) & here;
                    const unsigned even = (unsigned)__ballot(mx == 0) & here;
                    if (even) {   // a tie unless the classes at 0 stand just below the label's logit
                        unsigned long long eq = 0;
#pragma unroll
                        for (int z = 0; z < 4; ++z) eq |= __ballot(E[t][z] == adj[z]);
                        nties += __popc(fold_groups(eq) & even);
                    }
                    if (!viol) continue;
                    const v4i d = E[t] - adj;
                    const int best = rows_max(max(max(d[0], d[1]), max(d[2], d[3])));
                    int first = 0x7fffffff;   // lowest class index that reaches it
                    unsigned once = (unsigned)__ballot(best == 0) & 0xffffu, again = 0;   // points by how many do
#pragma unroll
                    for (int z = 3; z >= 0; --z) {
                        const bool is = d[z] == best;
                        const unsigned long long m = __ballot(is);
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const unsigned b = (unsigned)(m >> (16 * r)) & 0xffffu;
                            again |= once & b;
                            once |= b;
                        }
                        first = is ? 4 * g + z : first;
                    }
                    nties += __popc(again & viol);
                    first = -rows_max(-first);
                    lab = g == t ? first : lab;
                    vmask |= (unsigned long long)viol << (16 * t);
                }
                if (vmask == 0) continue;
                if (!r0ok) {
                    // rank offsets of the group's segments, lane w: segment w
                    r0ok = true;
                    if (lane < nw) {
                        int64_t s = 0, dg = 0;
                        const int k = c.k;
                        for (int j = 0; j < k - 1; ++j) {
                            const int px = ws.pp[8 * lane + j];
                            s += binom_small(c.n - 1 - px, k - j);
                            dg = dg * c.m + (ws.pc[8 * lane + j] - px * c.m);
                        }
                        int64_t mk = 1;
                        for (int j = 0; j < k; ++j) mk *= c.m;
                        ws.r0[lane] = (binom_small(c.n, k) - 1 - s - (c.n - 1)) * mk + dg * c.m;
                        if (lane == 0) ws.mk = mk;
                    }
                    fold_lds_sync();
                }
                const int n = __popcll(vmask);
                ncex += n;
                const int64_t room = rend - rnext;
                int64_t nb = 0;
                int got = 0;
                if (n > room) {
                    got = max(rblock, (int)(n - room));
                    rblock = min(2 * rblock, kRecBlock);
                    unsigned long long s = 0;
                    if (lane == 0) s = atomicAdd(P.rec_count, (unsigned long long)got);
                    nb = (int64_t)wave_uniform(s);
                }
                int pl = plast[0], il = ilast[0];
#pragma unroll
                for (int t = 1; t < NT; ++t) {
                    pl = g == t ? plast[t] : pl;
                    il = g == t ? ilast[t] : il;
                }
                if ((vmask >> lane) & 1ull) {
                    const int at = __popcll(vmask & ((1ull << lane) - 1ull));
                    const int64_t idx = at < room ? rnext + at : nb + (at - room);
                    if (idx < P.rec_cap) {
                        DevRec r;
                        r.rank = ws.r0[w + (g >> lp)] + (int64_t)pl * ws.mk + il;
                        r.prop = c.prop;
                        r.klab = (c.k << 24) | (lab & 0xffffff);
                        P.recs[idx] = r;
                    }
                }
                if (n > room) {
                    rnext = nb + (n - room);
                    rend = nb + got;
                } else {
                    rnext += n;
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
    {L_, KW_, WIDE_, EPI_, FoldShape<KW_>::NT, (int)sizeof(FoldWave<KW_>), reinterpret_cast<const void *>(&enum_fold_kernel<L_, KW_, WIDE_, EPI_>)}

}  // namespace ibmc
