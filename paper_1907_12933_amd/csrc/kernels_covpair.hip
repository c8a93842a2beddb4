// Pair coverage in one pass (the SS / DS / SV / DV covers of Sec. III-B,
// Eqs. (3)-(6), over input pairs (x1, x2)): a workgroup takes 16 NX pairs,
// runs both images of every pair through the network on int8 MFMA and tests
// every neuron of every layer on the fly, so that no potential ever goes to
// memory.
//
// Columns of the MFMA B operand: N-tiles 0 .. NX-1 hold x1 of the pairs, the
// next NX x2 of the same pairs, so the accumulators of a pair's two images
// for the same four neurons sit in the same lane.  Every wave (sixteen per
// workgroup) owns up to four 16-row M-tiles of each layer and keeps their
// accumulators for all N-tiles in registers: each weight tile loaded once
// feeds 2 NX MFMAs, each activation fragment read from LDS up to four.
//
// What bounds it: a tile reads the whole network, 3 MB for
// 784-1024-1024-1024-10, so the L2's 64 bytes per cycle and CU set the pace
// at 16 pairs and matrix cores and L2 take about the same time at 32.  x2's
// first layer, which differs from x1's by a few pixels, runs on the matrix
// cores like x1's, on the weight tiles already there: the rank-r update from
// lists of changed pixels gathered its weights a word at a time, each load
// waited for.  65,536 pairs of 784-1024-1024-1024-10: 1,612 us with eight
// waves, the update and 64-bit tests, 687 us now; the tests on the vector unit
// (about 25 instructions per neuron and pair) come next, the matrix cores are
// busy for 155 us.
//
// After a layer: the sign / value changes of every neuron as 4-bit
// nibbles per pair in LDS, the squared distance as per-wave partial sums,
// and (hidden layers) the requantised activations written back over the
// layer's inputs.  At the end every pair's counts, first sign change and
// distance decide its covered rows, which are OR-ed into the device masks
// as the potential-based predicate kernel does (the all-rows masks of DS /
// DV, which every pair with a distance change ORs into the same few words,
// are gathered per tile in LDS and flushed with one atomic per word).
#include <algorithm>

#include "kernels_cov.h"

namespace ibmc {

constexpr int kPairWaves = 16;

__device__ __forceinline__ unsigned long long sat_add(unsigned long long a, unsigned long long b) {
    const unsigned long long s = a + b;
    return s < a ? ~0ull : s;
}

__device__ __forceinline__ int pair_requant_byte(int acc_minus_off, int s) {
    const int lim = 64 << s;
    const int v = min(max(acc_minus_off, -lim), lim - 1);
    return (v >> s) & 0xff;
}

// One layer of a tile: the potentials of all columns, their tests, and (hidden
// layers) the next inputs.  Wave w owns M-tiles w, w + kPairWaves, ..., NMT of
// them at most (past the layer's last it repeats that one and drops it), whose
// accumulators live here alone: one function per count, because conditions on
// them made the compiler keep copies in memory.  Four waves a SIMD cover the
// weight tiles' loads.
template <int NX, int NMT>
__device__ __forceinline__ void pair_layer(const CovPairParams &P, int l, int8_t *act, uint8_t *nib,
                                           unsigned long long *dist, int wave, int lane) {
    constexpr int NC = 2 * NX, NP = 16 * NX;
    const QNetDev &net = P.net;
    const FwdExtra &fx = P.fx;
    const int KB = (l == 1) ? fx.K0 / 64 : net.H[l - 1] / 64, MT = net.H[l] / 16, RS = P.act_stride;
    const int8_t *tiles = (l == 1) ? net.W1tile : fx.Wn[l];
    const bool hidden = l < net.L, on = wave < MT;
    const int s = hidden ? net.shift[l - 1] : 0;
    const int off = hidden ? (64 << s) : 0;
    int j16 = lane & 15, g = lane >> 4;
    // (opaque: the addresses made of them would be kept over all layers)
    asm volatile("" : "+v"(j16), "+v"(g));
    v4i acc[NMT][NC];
    if (on) {
#pragma unroll
        for (int i = 0; i < NMT; ++i) {
            const int4 b = *reinterpret_cast<const int4 *>(fx.init[l] + min(wave + kPairWaves * i, MT - 1) * 16 + g * 4);
#pragma unroll
            for (int c = 0; c < NC; ++c) acc[i][c] = v4i{b.x, b.y, b.z, b.w};
        }
        const unsigned at = (unsigned)lane * 16u;
        const int8_t *b = act + j16 * RS + g * 16;
        for (int kb = 0; kb < KB; ++kb) {
            v4i A[NMT];
#pragma unroll
            for (int i = 0; i < NMT; ++i) {
                // the tile's address as a scalar: vector address pairs would spill
                const int8_t *t = tiles + (unsigned)((min(wave + kPairWaves * i, MT - 1) * KB + kb) * 1024);
                asm("" : "+s"(t));
                A[i] = *reinterpret_cast<const __attribute__((address_space(1))) v4i *>((const __attribute__((address_space(1))) int8_t *)t + at);
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const v4i B = *reinterpret_cast<const v4i *>(b + c * 16 * RS + kb * 64);
#pragma unroll
                for (int i = 0; i < NMT; ++i) acc[i][c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[i], B, acc[i][c], 0, 0, 0);
            }
        }
    }
    __syncthreads();   // every wave has read this layer's inputs
    if (!on) {
        // (its part of the distance)
        for (int t = lane; t < NP; t += 64) dist[((l - 1) * NP + t) * kPairWaves + wave] = 0;
        return;
    }
    // the layer's tests: nibbles of sign / value changes, distance partials
    const int nout = net.dims[l];
    const int nbo = P.nib_off[l];
    if (P.small >> l & 1) {
        // 24-bit products, no carry out of the 64-bit distance; rows past
        // the layer count as equal zeros
#pragma unroll
        for (int c = 0; c < NX; ++c) {
            unsigned long long dsum = 0;
#pragma unroll
            for (int i = 0; i < NMT; ++i) {
                const int mt = wave + kPairWaves * i;
                if (mt < MT) {
                    const bool full = mt * 16 + 16 <= nout;   // (the wave's)
                    uint32_t nb = 0;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        int a = acc[i][c][t] + off, b = acc[i][c + NX][t] + off;
                        if (!full && mt * 16 + g * 4 + t >= nout) a = b = 0;
                        const uint32_t sc = (uint32_t)(a ^ b) >> 31;
                        const uint32_t aa = (uint32_t)abs(a), bb = (uint32_t)abs(b);
                        const uint32_t mx = max(aa, bb), mn = min(aa, bb);
                        const bool vc = mx > 0 && __umul24(P.cp.ratio_den, mx) >= __umul24(P.cp.ratio_num, mn);
                        const uint32_t ad = (uint32_t)abs(a - b);
                        dsum += (unsigned long long)ad * ad;
                        nb |= sc << t | (vc ? 16u << t : 0u);
                    }
                    // a value change excludes a sign change
                    nib[(c * 16 + j16) * P.nib_stride + nbo + mt * 4 + g] = (uint8_t)(nb & ~(nb << 4));
                }
            }
            dsum += __shfl_xor(dsum, 16);
            dsum += __shfl_xor(dsum, 32);
            if (g == 0) dist[((l - 1) * NP + c * 16 + j16) * kPairWaves + wave] = dsum;
        }
    } else {
#pragma unroll
    for (int c = 0; c < NX; ++c) {
        // the squared distance as a 64-bit sum plus a count of its
        // carries (saturated once, after the layer)
        unsigned long long dlo = 0;
        uint32_t dhi = 0;
#pragma unroll
        for (int i = 0; i < NMT; ++i) {
            const int mt = wave + kPairWaves * i;
            if (mt < MT) {
                int sn = 0, vn = 0;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int r = mt * 16 + g * 4 + t;
                    if (r < nout) {
                        // potentials fit int32 (the loader's headroom check);
                        // |a - b| < 2^32 is |a| + |b| across a sign change,
                        // else max - min of the magnitudes
                        const int a = acc[i][c][t] + off, b = acc[i][c + NX][t] + off;
                        const bool sc = (a ^ b) < 0;   // the signs differ (sign(0) = 1)
                        const uint32_t aa = a < 0 ? 0u - (uint32_t)a : (uint32_t)a;
                        const uint32_t bb = b < 0 ? 0u - (uint32_t)b : (uint32_t)b;
                        const uint32_t mx = aa > bb ? aa : bb, mn = aa > bb ? bb : aa;
                        const bool vc = !sc && mx > 0 &&
                                        (uint64_t)(uint32_t)P.cp.ratio_den * mx >=
                                            (uint64_t)(uint32_t)P.cp.ratio_num * mn;
                        const uint32_t ad = sc ? aa + bb : mx - mn;
                        const unsigned long long nl = dlo + (unsigned long long)ad * ad;
                        dhi += nl < dlo;
                        dlo = nl;
                        sn |= (int)sc << t;
                        vn |= (int)vc << t;
                    }
                }
                nib[(c * 16 + j16) * P.nib_stride + nbo + mt * 4 + g] = (uint8_t)(sn | (vn << 4));
            }
        }
        unsigned long long dsum = dhi ? ~0ull : dlo;
        dsum = sat_add(dsum, __shfl_xor(dsum, 16));
        dsum = sat_add(dsum, __shfl_xor(dsum, 32));
        if (g == 0) dist[((l - 1) * NP + c * 16 + j16) * kPairWaves + wave] = dsum;
    }
    }
    if (hidden) {
#pragma unroll
        for (int i = 0; i < NMT; ++i) {
            const int mt = wave + kPairWaves * i;
            if (mt < MT) {
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    int packed = 0;
#pragma unroll
                    for (int t = 0; t < 4; ++t) packed |= pair_requant_byte(acc[i][c][t], s) << (8 * t);
                    *reinterpret_cast<int *>(act + (c * 16 + j16) * RS + mt * 16 + g * 4) = packed;
                }
            }
        }
    }
}

template <int NX>
__global__ void __launch_bounds__(64 * kPairWaves) cov_pair_kernel(CovPairParams P) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int NC = 2 * NX;          // N-tiles
    constexpr int NP = 16 * NX;         // pairs per tile
    const QNetDev &net = P.net;
    const FwdExtra &fx = P.fx;
    const CovLayout &lay = P.lay;
    const int L = net.L, n = net.dims[0];
    const int RS = P.act_stride;        // bytes per activation row
    int8_t *act = reinterpret_cast<int8_t *>(smem);                       // [NC * 16][RS]
    uint8_t *nib = reinterpret_cast<uint8_t *>(smem + P.off_nib);         // [NP][nib_stride]
    unsigned long long *dist = reinterpret_cast<unsigned long long *>(smem + P.off_dist);  // [L][NP][waves]
    // the tile's OR of the all-rows (DS, DV) masks, flushed once per tile
    uint32_t *tds = reinterpret_cast<uint32_t *>(smem + P.off_all);        // [all_words]
    uint32_t *tdv = tds + lay.all_words;                                   // [all_words]
    // the wave index as a scalar: the compiler then sees every M-tile
    // condition as wave-uniform (no exec-masked MFMAs, loads run ahead)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int K0 = fx.K0;               // <= kMaxWidth: one 16-byte load a lane covers a row
    const bool wide = ((n | (int)(uintptr_t)P.x1 | (int)(uintptr_t)P.x2) & 15) == 0;
    for (int64_t tile = blockIdx.x; tile * NP < P.n_pairs; tile += gridDim.x) {
        const int64_t pair0 = tile * NP;
        for (int t = threadIdx.x; t < 2 * lay.all_words; t += blockDim.x) tds[t] = 0u;
        __syncthreads();
        // stage x - 128 of both images (zeros past the last pair and past n):
        // wave w takes rows w, w + waves, ...
        if (wide) {
            // sixteen pixels a lane, all rows of the wave in flight
            v4i px[NC * 16 / kPairWaves];
#pragma unroll
            for (int r = 0; r < NC * 16 / kPairWaves; ++r) {
                const int col = wave + kPairWaves * r;
                const int64_t pg = pair0 + col % NP;
                px[r] = v4i{0, 0, 0, 0};
                if (pg < P.n_pairs && lane * 16 < n) {
                    const v4i x = *reinterpret_cast<const v4i *>((col < NP ? P.x1 : P.x2) + pg * n + lane * 16);
#pragma unroll
                    for (int e = 0; e < 4; ++e) px[r][e] = x[e] ^ (int)0x80808080;
                }
            }
#pragma unroll
            for (int r = 0; r < NC * 16 / kPairWaves; ++r)
                if (lane * 16 < K0) *reinterpret_cast<v4i *>(act + (wave + kPairWaves * r) * RS + lane * 16) = px[r];
        } else {
            for (int col = wave; col < NC * 16; col += kPairWaves) {
                const int64_t pg = pair0 + col % NP;
                const uint8_t *src = (col < NP ? P.x1 : P.x2) + pg * n;
                const bool live = pg < P.n_pairs;
                for (int p4 = lane * 4; p4 < K0; p4 += 256) {
                    uint32_t w = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int pix = p4 + e;
                        const uint32_t v = (live && pix < n) ? (uint32_t)(uint8_t)((int)src[pix] - 128) : 0u;
                        w |= v << (8 * e);
                    }
                    *reinterpret_cast<uint32_t *>(act + col * RS + p4) = w;
                }
            }
        }
        __syncthreads();
        for (int l = 1; l <= L; ++l) {
            const int mt = (net.H[l] / 16 + kPairWaves - 1) / kPairWaves;
            if (mt == 1) pair_layer<NX, 1>(P, l, act, nib, dist, wave, lane);
            else if (mt == 2) pair_layer<NX, 2>(P, l, act, nib, dist, wave, lane);
            else if (mt == 3) pair_layer<NX, 3>(P, l, act, nib, dist, wave, lane);
            else pair_layer<NX, 4>(P, l, act, nib, dist, wave, lane);
            __syncthreads();
        }
        // per pair: counts, first sign change and distance of every layer, then
        // the covered rows (one wave per pair)
        for (int pr = wave; pr < NP; pr += kPairWaves) {
            if (pair0 + pr >= P.n_pairs) continue;
            const uint8_t *nb = nib + pr * P.nib_stride;
            // layer by layer: this layer's count, first sign change and
            // distance; then block l - 1 (rows of layer l - 1, bits of layer l)
            int pcnt = 0, pfirst = 0;
            bool pdc = false;
            for (int l = 0; l < lay.nl; ++l) {
                const int nbytes = net.H[l + 1] / 4, nbo = P.nib_off[l + 1];
                if (l > 0 && (pcnt == 1 || pdc)) {
                    const int W = lay.words[l];
                    for (int t = lane; t < W; t += 64) {
                        uint32_t sw = 0, vw = 0;
#pragma unroll
                        for (int k = 0; k < 8; ++k) {
                            const int b = 8 * t + k;
                            const int v = b < nbytes ? nb[nbo + b] : 0;
                            sw |= (uint32_t)(v & 15) << (4 * k);
                            vw |= (uint32_t)(v >> 4) << (4 * k);
                        }
                        if (pcnt == 1) {
                            const int64_t row = lay.rowoff[l - 1] + (int64_t)pfirst * W;
                            if (sw) atomicOr(P.bits.rows_ss + row + t, sw);
                            if (vw) atomicOr(P.bits.rows_sv + row + t, vw);
                        }
                        if (pdc) {
                            // every pair of the tile ORs the same words: gather in LDS
                            if (sw) atomicOr(tds + lay.alloff[l - 1] + t, sw);
                            if (vw) atomicOr(tdv + lay.alloff[l - 1] + t, vw);
                        }
                    }
                }
                int cnt = 0, first = 0x7fffffff;
                for (int b0 = 0; b0 < nbytes; b0 += 64) {
                    const int b = b0 + lane;
                    const int v = b < nbytes ? (nb[nbo + b] & 15) : 0;
                    cnt += __popc(v);
                    if (v) first = min(first, 4 * b + __ffs(v) - 1);
                }
                unsigned long long dsum = lane < kPairWaves ? dist[(l * NP + pr) * kPairWaves + lane] : 0ull;
#pragma unroll
                for (int sh = 32; sh >= 1; sh >>= 1) {
                    cnt += __shfl_xor(cnt, sh);
                    first = min(first, __shfl_xor(first, sh));
                    dsum = sat_add(dsum, __shfl_xor(dsum, sh));
                }
                pcnt = cnt;
                pfirst = first;
                pdc = cnt == 0 && dsum >= (unsigned long long)P.cp.dist_sq_min;
            }
        }
        __syncthreads();
        for (int t = threadIdx.x; t < lay.all_words; t += blockDim.x) {
            if (tds[t]) atomicOr(P.bits.all_ds + t, tds[t]);
            if (tdv[t]) atomicOr(P.bits.all_dv + t, tdv[t]);
        }
        __syncthreads();
    }
}

static bool cov_pair_plan(const QNetDev &net, const FwdExtra &fx, int nx, CovPairParams &P, size_t &lds) {
    int hmax = fx.K0;
    for (int l = 1; l < net.L; ++l) hmax = std::max(hmax, net.H[l]);
    P.act_stride = hmax + 16;
    int nbo = 0;
    P.nib_off[0] = 0;
    for (int l = 1; l <= net.L; ++l) {
        P.nib_off[l] = nbo;
        nbo += net.H[l] / 4;
    }
    P.nib_off[net.L + 1] = nbo;
    P.nib_stride = (nbo + 3) & ~3;
    const int NP = 16 * nx;
    size_t o = (size_t)2 * NP * P.act_stride;
    o = (o + 15) & ~(size_t)15;
    P.off_nib = (int)o;
    o += (size_t)NP * P.nib_stride;
    o = (o + 15) & ~(size_t)15;
    P.off_dist = (int)o;
    o += (size_t)net.L * NP * kPairWaves * 8;
    P.off_all = (int)o;
    o += (size_t)2 * std::max(P.lay.all_words, 1) * 4;
    lds = o;
    return lds <= (size_t)160 * 1024;
}

// 32 pairs a tile where 16 would give a CU a second one, if the LDS holds it
// (784-1024-1024-1024-10, 65,536 pairs: 687 us against 1,016, that is 86 and 63
// us a tile); fewer pairs spread over the chip better by 16.
hipError_t launch_cov_pair(CovPairParams P, int n_cu, hipStream_t s) {
    if (P.n_pairs <= 0) return hipSuccess;
    size_t lds = 0;
    const int nx = P.n_pairs > (int64_t)n_cu * 16 && cov_pair_plan(P.net, P.fx, 2, P, lds) ? 2 : 1;
    if (nx == 1 && !cov_pair_plan(P.net, P.fx, 1, P, lds)) return hipErrorInvalidValue;
    const int64_t tiles = (P.n_pairs + 16 * nx - 1) / (16 * nx);
    const int grid = (int)std::min<int64_t>(tiles, (int64_t)n_cu * 16);
    if (nx == 2) hipLaunchKernelGGL(cov_pair_kernel<2>, dim3(grid), dim3(64 * kPairWaves), lds, s, P);
    else hipLaunchKernelGGL(cov_pair_kernel<1>, dim3(grid), dim3(64 * kPairWaves), lds, s, P);
    return hipGetLastError();
}

}  // namespace ibmc
