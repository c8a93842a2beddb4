// Integer enumeration with one point per lane, for small networks (one or
// two hidden layers of at most 64 units, at most 16 classes), where a 16x16
// matrix-core tile would be mostly padding.  Per point: the incremental
// first layer (Sec. II-A, Eq. (1): base + e W1[:, p], then the integer
// requantiser), the later layers on the matrix instruction of sixteen 4 x 4
// blocks (each lane gets four outputs of its own point; one register holds the
// weights of sixteen words of inputs for all lanes), the lowest-index argmax
// and the decision against the clean label (Sec. III-C).  The domain is either the
// delta set (offsets clamped to [0, 255]) or the L2 ball of Sec. III-C,
// Eq. (9): digits map to offsets -rd..-1, 1..rd, and a point belongs to the
// ball when every pixel stays in [0, 255] and the squared length of its
// offsets is at most r2.
//
// What bounds it: latency, for the most part; a chunk is about 200 vector
// instructions and waits for its pixel and weight row.  (The next chunk's loads
// ahead of the current one's work spilled and took 2.0 ms where this takes 1.5.)
#include <type_traits>

#include "f32_impl.h"
#include "kernels_lane.h"

namespace ibmc {

// Four activations clamp(u >> s, 0, 127) of one 32-bit word of first-layer
// weights (units 4w..4w+3), packed as bytes.
__device__ __forceinline__ int lane_act4(const int32_t *b, int w, int e, int s) {
    int a[4];
#pragma unroll
    for (int z = 0; z < 4; ++z) {
        const int u = b[z] + __mul24(e, (w << (24 - 8 * z)) >> 24);   // (a plain product takes a 64-bit one)
        a[z] = min(max(u >> s, 0), 127);
    }
    return a[0] | (a[1] << 8) | (a[2] << 16) | (a[3] << 24);
}

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// A layer's weights for the matrix instruction of sixteen 4 x 4 blocks: the
// word of inputs 4 i .. 4 i + 3 and outputs 4 q .. 4 q + 3 is block
// (q NI / 4 + i) % 16 of register (q NI / 4 + i) / 16, an output per lane.
// (W: layout [NO / 8][NI / 4][8].)
template <int NI, int NO>
struct LaneWeights {
    static constexpr int NW = NI / 4, REGS = NO / 4 * NW / 16;
    int w[REGS];
    __device__ __forceinline__ void load(const int32_t *W, int lane) {
#pragma unroll
        for (int r = 0; r < REGS; ++r) {
            const int blk = 16 * r + (lane >> 2), q = blk / NW, i = blk % NW, j = 4 * q + (lane & 3);
            w[r] = W[((j >> 3) * NW + i) * 8 + (j & 7)];
        }
    }
    // acc[r] += the outputs 4 Q + r of the lane's own point: its input word goes in
    // as one column of its block's B, one block's weights go to all blocks
    template <int Q>
    __device__ __forceinline__ void quad(const int (&in)[NW], v4i &acc) const {
        static_for<0, NW>([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value, blk = Q * NW + i;
            acc = __builtin_amdgcn_mfma_i32_4x4x4i8(w[blk / 16], in[i], acc, 4, blk % 16, 0);
        });
    }
};

// Hidden layer: requantised and packed.
template <int NI, int NO>
__device__ __forceinline__ void lane_hidden(const int (&in)[NI / 4], const LaneWeights<NI, NO> &W, const int32_t *B, int s,
                                            int (&out)[NO / 4]) {
    static_for<0, NO / 4>([&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        v4i acc;
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] = cld(B + 4 * q + r);
        W.template quad<q>(in, acc);
        int a[4];
#pragma unroll
        for (int z = 0; z < 4; ++z) a[z] = min(max(acc[z] >> s, 0), 127);
        out[q] = a[0] | (a[1] << 8) | (a[2] << 16) | (a[3] << 24);
    });
}

// Output layer, the first 4 Q classes: their logits (of classes past the
// network's: the lowest value), the lowest-index argmax and whether another
// class reaches it.
template <int NI, int Q>
__device__ __forceinline__ void lane_decide(const int (&in)[NI / 4], const LaneWeights<NI, 16> &W, const int32_t *B,
                                            int (&z)[16], int &best, bool &tie) {
    static_for<0, Q>([&](auto qc) __attribute__((always_inline)) {
        constexpr int q = decltype(qc)::value;
        v4i acc;
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[r] = cld(B + 4 * q + r);
        W.template quad<q>(in, acc);
#pragma unroll
        for (int r = 0; r < 4; ++r) z[4 * q + r] = acc[r];
    });
    best = 0;
    int top = z[0];
    tie = false;
#pragma unroll
    for (int j = 1; j < 4 * Q; ++j) {
        const bool gt = z[j] > top;
        tie = gt ? false : (tie || z[j] == top);
        best = gt ? j : best;
        top = max(top, z[j]);
    }
}

// Persistent enumeration: chunks of 64 consecutive last-element positions
// of one segment from the sliced queue.  Per segment the wave keeps the
// first-layer potentials before the last pixel in its LDS slot (and, for the
// ball, whether the prefix stays in [0, 255] and its squared length, and skips
// the segment's chunks if it doesn't); per chunk it tallies counterexamples,
// exact ties and visited points of the level.
// Three waves a SIMD: four spill a few registers, and the scratch memory alone
// costs a short call 50 us (16-20-9, one image, 300,000 positions: 320 us a call
// against 256).
template <int H1, int H2>
__global__ void __launch_bounds__(256, 3) enum_lane_kernel(LaneParams P) {
    constexpr int CH = kLaneChunk;
    constexpr int HL = H2 > 0 ? H2 : H1;
    __shared__ __attribute__((aligned(16))) int32_t bases[kLaneWaves][H1];
    __shared__ __attribute__((aligned(16))) DevRec rbuf[kLaneWaves][kLaneRecs];
    const int lane = __lane_id();
    __shared__ __attribute__((aligned(16))) Cursor cursors[kLaneWaves];
    LaneRecords out{&rbuf[threadIdx.x >> 6][0], 0};
    LaneWeights<H1, (H2 > 0 ? H2 : 16)> w2;
    LaneWeights<HL, 16> wo;
    if constexpr (H2 > 0) w2.load(P.net.W2S, lane);
    wo.load(P.net.WOS, lane);
    int32_t *base = &bases[threadIdx.x >> 6][0];
    const int nc = P.net.nc, s1 = P.net.s1, s2 = P.net.s2;
    LaneCursor c;
    c.S = &cursors[threadIdx.x >> 6];
    int64_t cur = 0, end = 0;
    bool seg_new = true;
    int prop_seen = -1, label0 = 0, ball = 0, rd = 0, r2 = 0;
    int pre_ok = 1, pre_sq = 0;
    int q = f32_first_slice(), tries = 0, polls = 0;
    int tslot = -1;
    unsigned long long tcex = 0, tties = 0, tpts = 0;
    auto flush = [&]() __attribute__((always_inline)) {
        if (tslot >= 0 && lane == 0) {
            if (tcex) atomicAdd(P.slot_cex + tslot, tcex);
            if (tties) atomicAdd(P.slot_ties + tslot, tties);
            if (tpts) atomicAdd(P.slot_points + tslot, tpts);
        }
        tcex = tties = tpts = 0;
    };
    while (true) {
        if (cur >= end) {
            const int64_t start = f32_ticket(P, q, tries, end, polls);
            if (start < 0) break;
            cur = start;
            c.decode<CH, LaneParams>(P, cur);
            seg_new = true;
        }
        if (c.slot != tslot) {
            flush();
            tslot = c.slot;
        }
        if (c.prop != prop_seen) {
            prop_seen = c.prop;
            const PropDev &pr = P.props[c.prop];
            label0 = wave_uniform(gld(&pr.label0));
            ball = wave_uniform(gld(&pr.ball));
            rd = wave_uniform(gld(&pr.ball_rd));
            r2 = wave_uniform(gld(&pr.ball_r2));
        }
        // the lane's point
        int p = 0, i = 0;
        bool valid = c.last_element(c.ch * CH + lane, p, i);
        const int xv = gld(c.img + p);
        const int dv = ball ? ball_offset(i, rd) : (int)gld(c.dl + i);
        v4i wcol[H1 / 16];
        const v4i *w1 = reinterpret_cast<const v4i *>(P.net.W1C + (int64_t)p * H1);
#pragma unroll
        for (int t = 0; t < H1 / 16; ++t) wcol[t] = w1[t];
        if (seg_new) {
            const int np = c.k - 1;
            int pp[kMaxK], ee[kMaxK];
            int ok = 1, sq = 0;
#pragma unroll
            for (int t = 0; t < kMaxK; ++t) {
                pp[t] = 0;
                ee[t] = 0;
                if (t < np) {
                    pp[t] = c.S->pre[t];
                    const int xs = wave_uniform((int)gld(c.img + pp[t]));
                    if (ball) {
                        const int d = ball_offset(c.S->dg[t], rd);
                        ok &= (xs + d >= 0 && xs + d <= 255) ? 1 : 0;
                        sq += d * d;
                        ee[t] = d;
                    } else {
                        ee[t] = clamp_pixel(xs + wave_uniform((int)gld(c.dl + c.S->dg[t]))) - xs;
                    }
                }
            }
            pre_ok = ok;
            pre_sq = sq;
            const int32_t *u0 = P.u0 + (int64_t)c.prop * P.u0_stride;
            for (int j = lane; j < H1; j += 64) {
                const int qj = P.net.q1[j];
                int v = qj >= 0 ? u0[qj] : 0;
#pragma unroll
                for (int t = 0; t < kMaxK - 1; ++t)
                    if (t < np) v += ee[t] * (int)P.net.W1C[(int64_t)pp[t] * H1 + j];
                base[j] = v;
            }
            wave_lds_sync();
            seg_new = false;
        }
        int e;
        if (ball) {
            const int v = xv + dv;
            valid = valid && pre_ok && v >= 0 && v <= 255 && pre_sq + dv * dv <= r2;
            e = dv;
        } else {
            e = clamp_pixel(xv + dv) - xv;
        }
        const unsigned long long vmask = __ballot(valid);
        if (vmask) {
            // first layer from the segment base, requantised and packed
            int a1[H1 / 4];
#pragma unroll
            for (int t = 0; t < H1 / 16; ++t) {
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const int4 b = *reinterpret_cast<const int4 *>(base + 16 * t + 4 * w);
                    const int32_t bb[4] = {b.x, b.y, b.z, b.w};
                    a1[4 * t + w] = lane_act4(bb, wcol[t][w], e, s1);
                }
            }
            int z[16], best;
            bool tied;
            auto decide = [&](const int(&in)[HL / 4]) __attribute__((always_inline)) {
                const int32_t *B = opaque(P.net.bo);
                if (nc <= 8) lane_decide<HL, 2>(in, wo, B, z, best, tied);
                else if (nc <= 12) lane_decide<HL, 3>(in, wo, B, z, best, tied);
                else lane_decide<HL, 4>(in, wo, B, z, best, tied);
            };
            if constexpr (H2 > 0) {
                int a2[H2 / 4];
                lane_hidden<H1, H2>(a1, w2, opaque(P.net.b2), s2, a2);
                decide(a2);
            } else {
                decide(a1);
            }
            bool viol = valid && best != label0;
            bool tie = valid && tied;
            if (P.literal) {
                // the threshold literal: the desired (clean) class below V,
                // another above; ties: one of the two equals V
                int zd = z[0], other = INT32_MIN;
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    if (j >= nc) continue;
                    if (j == label0) zd = z[j];
                    else other = max(other, z[j]);
                }
                viol = valid && zd < P.lit_v && other > P.lit_v;
                tie = valid && (zd == P.lit_v || other == P.lit_v);
            }
            const unsigned long long mv = __ballot(viol);
            if (mv) out.put(P, mv, viol, c.rank<LaneParams>(P, p, i), c.prop, (c.k << 24) | best, lane);
            tcex += (unsigned long long)__popcll(mv);
            tties += (unsigned long long)__popcll(__ballot(tie));
            tpts += (unsigned long long)__popcll(vmask);
        }
        if (!pre_ok) {
            // no point of the ball has this prefix: on to its last chunk of the ticket
            const int skip = (int)min((int64_t)(c.nch - c.ch), end - cur) - 1;
            c.ch += skip;
            cur += skip;
        }
        cur++;
        if (cur < end) seg_new = c.next<CH, LaneParams>(P, cur);
    }
    flush();
    if (out.n) out.flush(P, lane);
}

struct LaneInst {
    int h1, h2;
    const void *fn;
};

#define IBMC_LANE(H1, H2) LaneInst { H1, H2, reinterpret_cast<const void *>(&enum_lane_kernel<H1, H2>) }

static const LaneInst kLaneInst[] = {
    IBMC_LANE(16, 0),  IBMC_LANE(32, 0),  IBMC_LANE(64, 0),  IBMC_LANE(16, 16), IBMC_LANE(16, 32), IBMC_LANE(16, 64),
    IBMC_LANE(32, 16), IBMC_LANE(32, 32), IBMC_LANE(32, 64), IBMC_LANE(64, 16), IBMC_LANE(64, 32), IBMC_LANE(64, 64),
};

int lane_width(int h) { return h <= 16 ? 16 : h <= 32 ? 32 : h <= 64 ? 64 : 0; }

bool lane_eligible(const int *dims, int L) {
    if (L != 2 && L != 3) return false;
    if (dims[1] < 1 || dims[1] > 64 || dims[L] > 16) return false;
    return L == 2 || (dims[2] >= 1 && dims[2] <= 64);
}

static const LaneInst *find_lane(const LaneNetDev &net) {
    for (const LaneInst &v : kLaneInst)
        if (v.h1 == net.LH1 && v.h2 == net.LH2) return &v;
    return nullptr;
}

const void *lane_enum_kernel(const LaneNetDev &net) {
    const LaneInst *v = net.ok ? find_lane(net) : nullptr;
    return v ? v->fn : nullptr;
}

int lane_enum_grid(const LaneNetDev &net, int n_cu) {
    const LaneInst *v = net.ok ? find_lane(net) : nullptr;
    if (!v) return 0;
    int occ = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, v->fn, 256, 0) != hipSuccess || occ < 1) return 0;
    return n_cu * occ;
}

hipError_t launch_enum_lane(int grid, const LaneParams &P, hipStream_t s) {
    const LaneInst *v = find_lane(P.net);
    if (!v || grid < 1) return hipErrorInvalidValue;
    void *args[] = {const_cast<LaneParams *>(&P)};
    return hipLaunchKernel(v->fn, dim3(grid), dim3(256), args, 0, s);
}

}  // namespace ibmc
