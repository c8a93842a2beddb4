// Device code of the float (sigmoid variant) enumeration, shared by the
// kernel instances: the per-point forward pass with the incremental first
// layer (Sec. II-A, Eqs. (1)-(2)), the decision against the clean label
// (Sec. III-C) with near ties flagged, and wave-aggregated records.
//
// Both kernel families evaluate a point in one fixed sequence of FP32
// operations, which the eval kernels repeat exactly for listed points:
//   v_j = u0_j; v_j = fma(e_t, W1[p_t][j], v_j) for the prefix pixels in
//   ascending order, then for the last pixel; a_j = sigmoid(v_j);
//   every later layer: total = bias; per block of kF32SumBlock inputs a
//   partial sum accumulated from zero by fma in input order, added to the
//   total; hidden layers apply the sigmoid, the last layer gives the logits.
// e_t = (clamp(x[p_t] + d_t, 0, 255) - x[p_t]) / 256 is exact in FP32.
#pragma once

#include "enum_common.h"
#include "kernels_f32.h"

namespace ibmc {

typedef float v4f __attribute__((ext_vector_type(4)));

// Load through the constant address space: a wave-uniform address becomes
// one scalar-cache load for the whole wave (weights, biases and the clean
// potentials are read-only while the kernels run).
template <class T>
__device__ __forceinline__ T cld(const T *p) {
    return *(const __attribute__((address_space(4))) T *)p;
}

// A pointer the compiler may not treat as loop-invariant: the weight loads
// behind it stay at their use instead of being hoisted out of the chunk loop
// into (spilled) scalar registers.
template <class T>
__device__ __forceinline__ const T *opaque(const T *p) {
    asm volatile("" : "+s"(p));
    return p;
}

// 1 / (1 + e^-u) with the hardware base-2 exponential of -u log2(e) and the
// hardware reciprocal (each about 1 ulp); saturates to 0 and 1 for large |u|.
__device__ __forceinline__ float sigmoid_f32(float u) {
    const float e = __builtin_amdgcn_exp2f(-u * 1.4426950408889634f);
    return __builtin_amdgcn_rcpf(1.0f + e);
}

// The table sigmoid: knots u_i = -8 + i/16 holding sigma(u_i) in FP32 (tab,
// kLutIntervals + 1 values), linear between knots, the end values outside.
__device__ __forceinline__ float table_sigmoid(float u, const float *tab) {
    const float t = (u + 8.0f) * 16.0f;
    if (!(t > 0.0f)) return tab[0];
    if (t >= (float)kLutIntervals) return tab[kLutIntervals];
    const int i = (int)t;
    const float a = tab[i];
    return fmaf(t - (float)i, tab[i + 1] - a, a);
}

// Hidden-layer activation: the exponential form, or the table (use_tab).
__device__ __forceinline__ float act_f32(float u, bool use_tab, const float *tab) {
    return use_tab ? table_sigmoid(u, tab) : sigmoid_f32(u);
}

// Stage the table sigmoid's knots in LDS (every thread of the block takes
// part; tab: the block's LDS copy).  Returns whether the table is used.
__device__ __forceinline__ bool stage_table(const float *lut, float *tab) {
    if (!lut) return false;
    for (int i = threadIdx.x; i <= kLutIntervals; i += blockDim.x) tab[i] = lut[i];
    __syncthreads();
    return true;
}

// Cross-lane exchange through this wave's LDS: earlier writes complete
// before later reads.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float eff_delta(int xv, int d) {
    return (float)(clamp_pixel(xv + d) - xv) * (1.0f / 256.0f);
}

// Lowest-index largest logit, its value and the margin to the runner-up
// (infinite with one class).  Classes past the network's hold -infinity.
template <int NCP>
__device__ __forceinline__ void decide_f32(const float (&z)[NCP], int &best, float &top, float &margin) {
    best = 0;
    top = z[0];
    float second = -INFINITY;
#pragma unroll
    for (int j = 1; j < NCP; ++j) {
        const bool gt = z[j] > top;
        second = gt ? top : (z[j] > second ? z[j] : second);
        top = gt ? z[j] : top;
        best = gt ? j : best;
    }
    margin = top - second;
}

__device__ __forceinline__ unsigned lane_rank(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// The near ties among one wave's points.
__device__ __forceinline__ void emit_near(const FEnumParams &P, const Cursor &c, bool near, int p, int i, int best) {
    const int lane = __lane_id();
    const unsigned long long mn = __ballot(near);
    if (mn) {
        unsigned long long base = 0;
        if (lane == 0) {
            base = atomicAdd(P.tie_count, (unsigned long long)__popcll(mn));
            atomicAdd(P.slot_ties + c.slot, (unsigned long long)__popcll(mn));
        }
        base = wave_uniform(base);
        if (near) {
            const unsigned long long idx = base + lane_rank(mn);
            if ((int64_t)idx < P.tie_cap) {
                DevRec r;
                r.rank = point_rank<FEnumParams>(c, P, p, i);
                r.prop = c.prop;
                r.klab = (c.k << 24) | best;
                P.ties[idx] = r;
            }
        }
    }
}

// Counterexample and near-tie records of one wave's points: one atomic per
// wave and kind for the slots, one for the level counter; lanes write their
// own records at base + their rank among the set lanes.
__device__ __forceinline__ void emit_f32(const FEnumParams &P, const Cursor &c, bool viol, bool near, int p, int i,
                                         int best) {
    const int lane = __lane_id();
    const unsigned long long mv = __ballot(viol);
    if (mv) {
        unsigned long long base = 0;
        if (lane == 0) {
            base = atomicAdd(P.rec_count, (unsigned long long)__popcll(mv));
            atomicAdd(P.slot_cex + c.slot, (unsigned long long)__popcll(mv));
        }
        base = wave_uniform(base);
        if (viol) {
            const unsigned long long idx = base + lane_rank(mv);
            if ((int64_t)idx < P.rec_cap) {
                DevRec r;
                r.rank = point_rank<FEnumParams>(c, P, p, i);
                r.prop = c.prop;
                r.klab = (c.k << 24) | best;
                P.recs[idx] = r;
            }
        }
    }
    emit_near(P, c, near, p, i, best);
}

// Tickets between two reads of the host's abort request by one wave (a read
// of host memory crosses PCIe; one per ticket from every wave saturated it).
constexpr int kAbortPollTickets = 64;

// Next queue ticket of a persistent wave: [start, end) of at most P.batch
// chunks from the wave's current slice q; a drained slice sends the wave to
// the next one (tries counts the slices visited).  Returns -1 when every
// slice is drained or a stop / abort was requested.  The device stop flag is
// read per ticket, the host abort request every kAbortPollTickets tickets
// (polls counts them; never at a wave's first ticket, where every wave of the
// grid would read host memory at once); a wave that sees the abort raises
// the stop flag.
template <class PT>
__device__ __forceinline__ int64_t f32_ticket(const PT &P, int &q, int &tries, int64_t &end, int &polls) {
    while (tries < kF32Queues) {
        const int64_t lo = (int64_t)q * P.slice;
        const int64_t hi = min(lo + P.slice, P.total_chunks);
        unsigned long long t = 0;
        int stop = 0;
        const bool poll_host = P.abort_host && (++polls % kAbortPollTickets) == 0;
        if (__lane_id() == 0) {
            if (lo < hi) t = atomicAdd(P.queue + (int64_t)q * kQueueStride, (unsigned long long)P.batch);
            stop = *P.stop_flag;
            if (poll_host && *P.abort_host) {
                stop = 1;
                *P.stop_flag = 1;
            }
        }
        if (wave_uniform(stop)) return -1;
        const int64_t start = lo + (int64_t)wave_uniform(t);
        if (lo < hi && start < hi) {
            end = min(start + (int64_t)P.batch, hi);
            return start;
        }
        q = q + 1 == kF32Queues ? 0 : q + 1;
        tries++;
    }
    return -1;
}

// The first slice of a wave: waves are spread evenly over the slices.
__device__ __forceinline__ int f32_first_slice() {
    const int w = (int)((blockIdx.x * (blockDim.x >> 6)) + (threadIdx.x >> 6));
    return w % kF32Queues;
}

// Decode point (k, rank) of a property: ascending pixels and delta indices.
__device__ __forceinline__ void decode_point_dev(int n, int m, int k, int64_t rank, int (&pix)[kMaxK],
                                                 int (&dig)[kMaxK]) {
    int64_t mk = 1;
    for (int j = 0; j < k; ++j) mk *= m;
    lex_unrank_subset_fixed(rank / mk, k, n, pix);
    int64_t d = rank % mk;
#pragma unroll
    for (int j = kMaxK - 1; j >= 0; --j) {
        dig[j] = 0;
        if (j < k) { dig[j] = (int)(d % m); d /= m; }
    }
}

// ---------------------------------------------------------------------------
// one point per lane
// ---------------------------------------------------------------------------

constexpr int kLaneWaves = 4;  // waves per workgroup of the lane kernels

// A wave's position for the lane kernels.  The whole cursor lives in the
// wave's LDS; the fields that a chunk needs are kept as scalars.  (All of it in
// registers, with the code that moves it inlined around the point's own work,
// took 182 vector registers for sixteen units, two waves a SIMD, or spilled.)
// These kernels take plain jobs only (SEG_PLAIN).
struct LaneCursor {
    Cursor *S;
    int q, m, seglen, ch, nch, prop, slot, k;
    unsigned mmagic, m1;
    const uint8_t *img;
    const int16_t *dl;
    __device__ __forceinline__ void refresh() {
        ranked = false;
        q = wave_uniform(S->q);
        m = wave_uniform(S->m);
        seglen = wave_uniform((int)S->seglen);
        ch = wave_uniform((int)S->ch);
        nch = wave_uniform((int)S->nch);
        prop = wave_uniform(S->prop);
        slot = wave_uniform(S->slot);
        k = wave_uniform(S->k);
        mmagic = (unsigned)wave_uniform((int)S->mmagic);
        m1 = (unsigned)wave_uniform((int)S->m1);
        img = reinterpret_cast<const uint8_t *>(wave_uniform((unsigned long long)S->img));
        dl = reinterpret_cast<const int16_t *>(wave_uniform((unsigned long long)S->dl));
    }
    template <int CH, class PT>
    __device__ __forceinline__ void decode(const PT &P, int64_t chunk) {
        Cursor c;
        cursor_decode<CH, PT>(c, P, chunk);
        *S = c;
        refresh();
    }
    // To chunk `chunk`, the next one; true when the segment changed.
    template <int CH, class PT>
    __device__ __forceinline__ bool next(const PT &P, int64_t chunk) {
        if (++ch < nch) return false;
        Cursor c = *S;
        c.mode = SEG_PLAIN;
        c.ch = c.nch - 1;
        c.chunk = chunk - 1;
        cursor_next<CH, PT>(c, P);
        *S = c;
        refresh();
        return true;
    }
    // last_element32
    __device__ __forceinline__ bool last_element(int o, int &p, int &i) const {
        const bool ok = o < seglen;
        const unsigned uo = ok ? (unsigned)o : 0u;
        const unsigned qd = __umulhi(uo, mmagic) + uo * m1;
        p = q + 1 + (int)qd;
        i = (int)(uo - qd * (unsigned)m);
        return ok;
    }
    // A point's rank is linear in its last pixel and delta: r0 + p mk + i, r0 of
    // the segment worked out at its first record.
    int64_t r0, mk;
    bool ranked;
    template <class PT>
    __device__ __forceinline__ int64_t rank(const PT &P, int p, int i) {
        if (!ranked) {
            Cursor c = *S;
            c.mode = SEG_PLAIN;
            mk = 1;
            for (int j = 0; j < k; ++j) mk *= m;
            const int64_t first = point_rank<PT>(c, P, q + 1, 0) - (int64_t)(q + 1) * mk;
            r0 = (int64_t)wave_uniform((unsigned long long)first);
            ranked = true;
        }
        return r0 + (int64_t)p * mk + i;
    }
};

// The wave's records, gathered in LDS: one atomic on the call's record count
// and one coalesced store per 65 records or more.  An atomic per chunk made
// every wave wait for the one address: ten glyphs' L2 balls (27 million points,
// 1.8 million records) took 3.4 ms; with this, the skipped prefixes, longer
// tickets and the matrix cores 1.5.
constexpr int kLaneRecs = 128;

struct LaneRecords {
    DevRec *buf;   // [kLaneRecs]
    int n;         // (wave-uniform)
    // the records of the lanes in mask, mine among them (viol)
    template <class PT>
    __device__ __forceinline__ void put(const PT &P, unsigned long long mask, bool viol, int64_t rank, int prop, int klab,
                                        int lane) {
        if (viol) {
            DevRec r;
            r.rank = rank;
            r.prop = prop;
            r.klab = klab;
            buf[n + lane_rank(mask)] = r;
        }
        n += __popcll(mask);
        if (n > kLaneRecs - 64) flush(P, lane);
    }
    template <class PT>
    __device__ __forceinline__ void flush(const PT &P, int lane) {
        unsigned long long rb = 0;
        if (lane == 0) rb = atomicAdd(P.rec_count, (unsigned long long)n);
        rb = wave_uniform(rb);
        wave_lds_sync();
        for (int t = lane; t < n; t += 64)
            if ((int64_t)(rb + t) < P.rec_cap) P.recs[rb + t] = buf[t];
        wave_lds_sync();
        n = 0;
    }
};

// One layer of the lanes' points on the matrix cores: the 4x4x1 FP32 product
// of sixteen blocks gives every lane, from its own activation (B: point
// 4b + j of block b in lane 4b + j), four outputs of its own point (D: one
// output per register), and the broadcast of one block's A lets one register
// hold the weights of sixteen inputs: lane 4b + i has input 16 kb + b, output
// 4 q + i.  Each product is one fma per output (also for subnormal values),
// so the order of operations is the one stated above.  The scalar form, four
// fma with weights from the scalar cache, took twice the matrix pipe's time
// and all of it on the vector unit, which the sigmoids need: 196-128-64-10
// 2.5 -> 4.5, 100-64-10 14 -> 21, 35-32-16-5 24 -> 32, 35-16-5 67 -> 77
// billion points per second; the vector unit bounds it still (sigmoids, and
// for the small networks the decision and the chunk's set-up).
// w[kb * QS + q]: QS quads of outputs; the first Q are computed.
template <int K, int QS>
__device__ __forceinline__ void lane_weights(const float *W, int ld, int lane, float (&w)[K / 16 * QS]) {
    const unsigned at = (unsigned)((lane >> 2) * ld + (lane & 3));
#pragma unroll
    for (int kb = 0; kb < K / 16; ++kb)
#pragma unroll
        for (int q = 0; q < QS; ++q) w[kb * QS + q] = gld(W + (16 * kb * ld + 4 * q) + at);
}

template <int K, int Q, int QS>
__device__ __forceinline__ void lane_rows(const float (&w)[K / 16 * QS], const float (&a)[K], v4f (&tot)[Q]) {
#pragma unroll
    for (int ib = 0; ib < K; ib += kF32SumBlock) {
        v4f part[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) part[q] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int kb = ib / 16; kb < (ib + kF32SumBlock) / 16 && kb < K / 16; ++kb) {
#define IBMC_ROW(k)                                                                                           \
    _Pragma("unroll") for (int q = 0; q < Q; ++q) part[q] =                                                   \
        __builtin_amdgcn_mfma_f32_4x4x1f32(w[kb * QS + q], a[16 * kb + k], part[q], 4, k, 0)
            IBMC_ROW(0);  IBMC_ROW(1);  IBMC_ROW(2);  IBMC_ROW(3);  IBMC_ROW(4);  IBMC_ROW(5);  IBMC_ROW(6);  IBMC_ROW(7);
            IBMC_ROW(8);  IBMC_ROW(9);  IBMC_ROW(10); IBMC_ROW(11); IBMC_ROW(12); IBMC_ROW(13); IBMC_ROW(14); IBMC_ROW(15);
#undef IBMC_ROW
        }
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) tot[q][i] += part[q][i];
    }
}

// The last layer's weights stay in registers (NCP / 4 per sixteen inputs).
template <int H1, int H2, int NCP>
struct LaneOut {
    static constexpr int K = H2 > 0 ? H2 : H1, QS = NCP / 4;
    float w[K / 16 * QS];
    __device__ __forceinline__ void load(const FNetDev &net, int lane) {
        lane_weights<K, QS>(net.WP[H2 > 0 ? 3 : 2], NCP, lane, w);
    }
};

// Layers >= 2 of the lane's point from its first-layer activations a1; z of
// the first 4 Q classes, -infinity past the network's.  a2w: this wave's LDS
// columns [H2][64] of the second hidden layer; each lane touches only its own.
template <int H1, int H2, int NCP, int Q>
__device__ __forceinline__ void lane_upper(const FNetDev &net, const LaneOut<H1, H2, NCP> &out,
                                           const float (&a1)[H1], float *a2w, int lane, float (&z)[NCP], bool use_tab,
                                           const float *tab) {
    constexpr int QS = NCP / 4;
    const float *B = opaque(net.bP[H2 > 0 ? 3 : 2]);
    v4f tot[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) tot[q][i] = cld(B + 4 * q + i);
    if constexpr (H2 == 0) {
        lane_rows<H1, Q, QS>(out.w, a1, tot);
    } else {
        const float *W2 = opaque(net.WP[2]);
        const float *B2 = opaque(net.bP[2]);
        // second hidden layer, sixteen units per step, into this lane's LDS column
#pragma unroll 1
        for (int jb = 0; jb < H2; jb += 16) {
            float w2[H1 / 16 * 4];
            lane_weights<H1, 4>(W2 + jb, H2, lane, w2);
            v4f t2[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) t2[q][i] = cld(B2 + jb + 4 * q + i);
            lane_rows<H1, 4, 4>(w2, a1, t2);
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) a2w[(jb + 4 * q + i) * 64 + lane] = act_f32(t2[q][i], use_tab, tab);
        }
        float a2[H2];
#pragma unroll
        for (int j = 0; j < H2; ++j) a2[j] = a2w[j * 64 + lane];
        lane_rows<H2, Q, QS>(out.w, a2, tot);
    }
#pragma unroll
    for (int j = 0; j < NCP; ++j) z[j] = j < 4 * Q ? tot[j / 4 < Q ? j / 4 : 0][j & 3] : -INFINITY;
}

// The same with the quads that nc classes need, and the decision.
template <int H1, int H2, int NCP>
__device__ __forceinline__ void lane_decide(const FNetDev &net, const LaneOut<H1, H2, NCP> &out, int nc,
                                            const float (&a1)[H1], float *a2w, int lane, float (&z)[NCP], bool use_tab,
                                            const float *tab, int &best, float &top, float &margin) {
    if (NCP == 16 && nc <= 12) lane_upper<H1, H2, NCP, NCP == 16 ? 3 : 2>(net, out, a1, a2w, lane, z, use_tab, tab);
    else lane_upper<H1, H2, NCP, NCP / 4>(net, out, a1, a2w, lane, z, use_tab, tab);
    decide_f32<NCP>(z, best, top, margin);
}

// First-layer potentials before the last pixel: v_j = u0_j, then one fma
// per prefix element in ascending pixel order.
__device__ __forceinline__ float prefix_potential_rt(const FNetDev &net, int h1p, const float *u0, int np,
                                                     const int (&pp)[kMaxK], const float (&ee)[kMaxK], int j) {
    float v = u0[j];
#pragma unroll
    for (int t = 0; t < kMaxK - 1; ++t)
        if (t < np) v = fmaf(ee[t], net.W1P[(int64_t)pp[t] * h1p + j], v);
    return v;
}

template <int H1>
__device__ __forceinline__ float prefix_potential(const FNetDev &net, const float *u0, int np, const int (&pp)[kMaxK],
                                                  const float (&ee)[kMaxK], int j) {
    return prefix_potential_rt(net, H1, u0, np, pp, ee, j);
}

// The prefix of the cursor's segment: pixels and effective deltas (their
// loads issued together).
__device__ __forceinline__ void segment_prefix(const Cursor &c, int (&pp)[kMaxK], float (&ee)[kMaxK]) {
    const int np = c.k - 1;
    int xs[kMaxK], ds[kMaxK];
#pragma unroll
    for (int t = 0; t < kMaxK; ++t) {
        xs[t] = 0;
        ds[t] = 0;
        if (t < np) { xs[t] = gld(c.img + c.pre[t]); ds[t] = gld(c.dl + c.dg[t]); }
    }
#pragma unroll
    for (int t = 0; t < kMaxK; ++t) {
        pp[t] = t < np ? c.pre[t] : 0;
        ee[t] = t < np ? eff_delta(xs[t], ds[t]) : 0.0f;
    }
}

// Persistent enumeration, one point per lane; chunks of 64 consecutive
// last-element positions of one segment.  Per segment (all prefix pixels
// fixed) the wave computes v_j before the last pixel once into its LDS slot;
// per property it keeps the clean label in a register; a chunk then loads
// only its own pixels, deltas and first-layer rows.
// (The waves per SIMD keep the registers that the compiler would spend on
// addresses in check: 128-64 took 416 and ran one wave.  Ten table instances spill
// under it, those of 128 units up to 480 registers; their calls take a fifth to
// two thirds of what they took with scalar weights and no bound, 128-64-10 4.81 ->
// 1.16 ms, 16-16-10 without scratch before 1.02 -> 0.95.)
template <int H1, int H2, int NCP, bool TAB>
__global__ void __launch_bounds__(256, H1 <= 16 ? 4 : H1 <= 32 ? 3 : 2) enum_f32_lane_kernel(FEnumParams P) {
    constexpr int CH = kF32LaneChunk;
    __shared__ float a2s[kLaneWaves][H2 > 0 ? H2 : 1][64];
    __shared__ __attribute__((aligned(16))) float bases[kLaneWaves][H1];
    __shared__ float tab[kLutIntervals + 1];
    // TAB is a compile-time switch: a run-time choice inside the unrolled
    // layer loops keeps both activations live and spills the 128-wide ones
    const bool use_tab = TAB && stage_table(P.lut, tab);
    const int lane = __lane_id();
    float *a2w = &a2s[threadIdx.x >> 6][0][0];
    float *base = &bases[threadIdx.x >> 6][0];
    const int nc = P.net.dims[P.net.L];
    LaneOut<H1, H2, NCP> out;
    out.load(P.net, lane);
    __shared__ __attribute__((aligned(16))) DevRec rbuf[kLaneWaves][kLaneRecs];
    __shared__ __attribute__((aligned(16))) Cursor cursors[kLaneWaves];
    LaneRecords recs{&rbuf[threadIdx.x >> 6][0], 0};
    LaneCursor c;
    c.S = &cursors[threadIdx.x >> 6];
    int tslot = -1;
    unsigned long long tcex = 0;
    auto tally = [&]() __attribute__((always_inline)) {
        if (tcex && lane == 0) atomicAdd(P.slot_cex + tslot, tcex);
        tcex = 0;
    };
    int64_t cur = 0, end = 0;
    bool seg_new = true;
    int prop_seen = -1, label0 = 0;
    int q = f32_first_slice(), tries = 0, polls = 0;
    while (true) {
        if (cur >= end) {
            const int64_t start = f32_ticket(P, q, tries, end, polls);
            if (start < 0) break;
            cur = start;
            c.decode<CH, FEnumParams>(P, cur);
            seg_new = true;
        }
        if (c.slot != tslot) {
            tally();
            tslot = c.slot;
        }
        // the lane's point: its loads go out first
        int p = 0, i = 0;
        const bool valid = c.last_element(c.ch * CH + lane, p, i);
        const int xv = gld(c.img + p), dv = gld(c.dl + i);
        float4 wrow[H1 / 4];
        const float4 *w1 = reinterpret_cast<const float4 *>(P.net.W1P + (int64_t)p * H1);
#pragma unroll
        for (int j4 = 0; j4 < H1 / 4; ++j4) wrow[j4] = w1[j4];
        if (c.prop != prop_seen) {
            prop_seen = c.prop;
            label0 = wave_uniform(gld(&P.props[c.prop].label0));
        }
        if (seg_new) {
            int pp[kMaxK];
            float ee[kMaxK];
            segment_prefix(*c.S, pp, ee);
            const float *u0 = P.u0f + (int64_t)c.prop * P.u0_stride;
#pragma unroll
            for (int j0 = 0; j0 < H1; j0 += 64)
                if (j0 + lane < H1) base[j0 + lane] = prefix_potential<H1>(P.net, u0, c.k - 1, pp, ee, j0 + lane);
            wave_lds_sync();
            seg_new = false;
        }
        const float e = eff_delta(xv, dv);
        float a1[H1];
#pragma unroll
        for (int j4 = 0; j4 < H1 / 4; ++j4) {
            const float4 b = *reinterpret_cast<const float4 *>(base + 4 * j4);
            a1[4 * j4 + 0] = act_f32(fmaf(e, wrow[j4].x, b.x), use_tab, tab);
            a1[4 * j4 + 1] = act_f32(fmaf(e, wrow[j4].y, b.y), use_tab, tab);
            a1[4 * j4 + 2] = act_f32(fmaf(e, wrow[j4].z, b.z), use_tab, tab);
            a1[4 * j4 + 3] = act_f32(fmaf(e, wrow[j4].w, b.w), use_tab, tab);
        }
        float z[NCP];
        int best;
        float top, margin;
        lane_decide<H1, H2, NCP>(P.net, out, nc, a1, a2w, lane, z, use_tab, tab, best, top, margin);
        bool near = valid && margin <= P.tie_rel * fmaxf(1.0f, fabsf(top));
        bool viol = valid && best != label0;
        if (P.literal) {
            // (opaque: the compiler would compute this for every point and select)
#pragma unroll
            for (int j = 0; j < NCP; ++j) asm volatile("" : "+v"(z[j]));
            // the threshold literal: the desired (clean) class below V, another above
            float zd = z[0], other = -INFINITY;
#pragma unroll
            for (int j = 0; j < NCP; ++j) {
                if (j == label0) zd = z[j];
                else if (j < nc) other = fmaxf(other, z[j]);
            }
            const float V = P.lit_v;
            viol = valid && zd < V && other > V;
            near = valid && fminf(fabsf(zd - V), fabsf(other - V)) <= P.tie_rel * fmaxf(1.0f, fabsf(V));
        }
        const unsigned long long mv = __ballot(viol);
        if (mv) {
            tcex += (unsigned long long)__popcll(mv);
            recs.put(P, mv, viol, c.rank<FEnumParams>(P, p, i), c.prop, (c.k << 24) | best, lane);
        }
        if (__ballot(near)) emit_near(P, *c.S, near, p, i, best);
        cur++;
        if (cur < end) seg_new = c.next<CH, FEnumParams>(P, cur);
    }
    tally();
    if (recs.n) recs.flush(P, lane);
}

// Listed points (or the clean images of listed properties), one per lane,
// in the same sequence of operations.
template <int H1, int H2, int NCP, bool TAB>
__global__ void __launch_bounds__(256) eval_f32_lane_kernel(F32EvalParams E) {
    __shared__ float a2s[kLaneWaves][H2 > 0 ? H2 : 1][64];
    __shared__ float tab[kLutIntervals + 1];
    const bool use_tab = TAB && stage_table(E.lut, tab);
    const int lane = __lane_id();
    float *a2w = &a2s[threadIdx.x >> 6][0][0];
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool ok = t < E.n;
    const int64_t tt = ok ? t : 0;
    const int prop = E.prop_of ? E.prop_of[tt] : 0;
    const PropDev &pr = E.props[prop];
    const int k = E.label_props ? 0 : E.ks[tt];
    const int64_t rank = E.label_props ? 0 : E.ranks[tt];
    int pix[kMaxK], dig[kMaxK];
    decode_point_dev(pr.n, pr.m, k, rank, pix, dig);
    int pp[kMaxK];
    float ee[kMaxK];
    const int np = k > 0 ? k - 1 : 0;
    int p = 0;
    float e = 0.0f;
#pragma unroll
    for (int j = 0; j < kMaxK; ++j) {
        pp[j] = 0;
        ee[j] = 0.0f;
        if (j < np) { pp[j] = pix[j]; ee[j] = eff_delta(pr.image[pix[j]], pr.deltas[dig[j]]); }
        if (k > 0 && j == k - 1) { p = pix[j]; e = eff_delta(pr.image[pix[j]], pr.deltas[dig[j]]); }
    }
    const float *u0 = E.u0f + (int64_t)prop * E.u0_stride;
    const float *w1 = E.net.W1P + (int64_t)p * H1;
    float a1[H1];
#pragma unroll
    for (int j = 0; j < H1; ++j)
        a1[j] = act_f32(fmaf(e, w1[j], prefix_potential<H1>(E.net, u0, np, pp, ee, j)), use_tab, tab);
    float z[NCP];
    const int nc = E.net.dims[E.net.L];
    LaneOut<H1, H2, NCP> out;
    out.load(E.net, lane);
    int best;
    float top, margin;
    lane_decide<H1, H2, NCP>(E.net, out, nc, a1, a2w, lane, z, use_tab, tab, best, top, margin);
    if (!ok) return;
    if (E.label_props) {
        E.label_props[prop].label0 = best;
        E.label_props[prop].tie0 = 0;
        return;
    }
    if (E.logits)
#pragma unroll
        for (int j = 0; j < NCP; ++j)
            if (j < nc) E.logits[tt * nc + j] = z[j];
    if (E.labels) E.labels[tt] = best;
    if (E.margins) E.margins[tt] = margin;
}

// A compiled lane instance: L weight layers, padded widths, its kernels.
// enum_fn[t] / eval_fn[t]: the exponential sigmoid (t = 0) or the table (t = 1).
struct F32LaneVariant {
    int L, h1, h2, ncp;
    const void *enum_fn[2];
    const void *eval_fn[2];
};

#define IBMC_F32_LANE(H1, H2, NCP)                                                                 \
    F32LaneVariant { (H2) > 0 ? 3 : 2, H1, H2, NCP,                                                \
                     {reinterpret_cast<const void *>(&enum_f32_lane_kernel<H1, H2, NCP, false>),    \
                      reinterpret_cast<const void *>(&enum_f32_lane_kernel<H1, H2, NCP, true>)},    \
                     {reinterpret_cast<const void *>(&eval_f32_lane_kernel<H1, H2, NCP, false>),    \
                      reinterpret_cast<const void *>(&eval_f32_lane_kernel<H1, H2, NCP, true>)} }

// Instance tables (one per source file, to split compilation).
const F32LaneVariant *f32_lane_variants_l2(int *n);
const F32LaneVariant *f32_lane_variants_l3(int *n);

}  // namespace ibmc
