// Coverage-guided test generation (the test generation from the covers of
// Sec. III-B that the paper leaves open, Sec. IV-C): every point of one
// level of the delta-set domain is a candidate test x' for the clean image
// x; one wave per candidate computes the potentials of x' (the first layer
// as the rank-k update of x's potentials, Eq. (1), the later layers densely),
// the sign / value / distance changes against x of every non-input layer and
// the neuron pairs (i, j) of adjacent layers that the pair (x, x') covers
// under one criterion, as a bitset in the layout of ibmc_coverage's
// covered_bits.  A greedy loop then picks, one test at a time, the candidate
// covering the most pairs not yet covered (the host queues the steps in
// batches and reads their winners back once per batch).  Networks whose non-input layers
// have at most 64 units (one lane per unit).
#include <climits>

#include "kernels_covsearch.h"
#include "enum_common.h"

namespace ibmc {

// lex_unrank_subset by a wave: the values of one element side by side, where
// one after another, two 64-bit divisions each, they took most of the kernel.
__device__ __forceinline__ void wave_unrank_subset(int64_t rank, int k, int n, int lane, int (&p)[kMaxK]) {
    int64_t R = binom_small(n, k) - 1 - rank;
    int c = n;
#pragma unroll
    for (int j = 0; j < kMaxK; ++j) {
        if (j >= k) break;
        const int r = k - j;
        // the largest cj < c with binom(cj, r) <= R, or r - 1
        int cj = r - 1;
        int64_t bj = 0;
        for (int base = r; base < c; base += 64) {
            const int v = base + lane;
            const int64_t b = binom_small(min(v, c - 1), r);
            const int cnt = __popcll(__ballot(v < c && b <= R));
            if (cnt == 0) break;
            cj = base + cnt - 1;
            bj = __shfl(b, cnt - 1);
            if (cnt < 64) break;
        }
        R -= bj;
        p[j] = n - 1 - cj;
        c = cj;
    }
}

// A wave keeps its unit's weights of layers 2 .. L in registers, packed for
// four-way dot products, over all of its candidates; bound by latency (one wave
// per candidate, a few thousand candidates).  With a byte load and a wait per
// weight and unranking by lane loops 3,915 candidates of 30-40-30-6 took 116 us,
// now 49 us (the weights alone changed nothing; the unranking above did).
__global__ void __launch_bounds__(64) cov_cand_kernel(CovCandParams P) {
    __shared__ __attribute__((aligned(16))) int act[16];   // 64 activations, a byte each
    __shared__ unsigned long long mask[kCovSearchMaxWords];
    const int lane = threadIdx.x;
    const QNetDev &net = P.net;
    const int L = net.L, n = net.dims[0], m = P.m;
    int wr[kMaxLayers - 1][16], br[kMaxLayers - 1];
#pragma unroll
    for (int l = 2; l <= kMaxLayers; ++l) {
        br[l - 2] = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) wr[l - 2][w] = 0;
        if (l > L) continue;
        const int h = net.dims[l], hin = net.dims[l - 1], j = min(lane, h - 1);
        br[l - 2] = net.bd[l][j];
        const int8_t *row = net.Wd[l] + (int64_t)j * hin;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            uint32_t v = 0;
#pragma unroll
            for (int z = 0; z < 4; ++z) {
                const int b = (uint8_t)row[min(4 * w + z, hin - 1)];
                v |= (uint32_t)(4 * w + z < hin ? b : 0) << (8 * z);
            }
            wr[l - 2][w] = (int)v;
        }
    }
    for (int64_t c = blockIdx.x; c < P.n_cand; c += gridDim.x) {
        // the candidate's pixels and offsets (ascending pixels, digits base m)
        const int64_t rank = P.rank0 + c;
        int64_t mk = 1;
        for (int t = 0; t < P.k; ++t) mk *= m;
        int pix[kMaxK], off[kMaxK];
        wave_unrank_subset(rank / mk, P.k, n, lane, pix);
        int64_t d = rank % mk;
        for (int t = P.k - 1; t >= 0; --t) {
            const int di = (int)(d % m);
            d /= m;
            const int xv = P.image[pix[t]];
            off[t] = clamp_pixel(xv + P.deltas[di]) - xv;
        }
        for (int w = lane; w < P.words; w += 64) mask[w] = 0ull;
        unsigned long long sc[kMaxLayers], vc[kMaxLayers];
        int dc[kMaxLayers];
        int label = 0;
        int uoff = 0;
#pragma unroll
        for (int l = 1; l <= kMaxLayers; ++l) {
            if (l > L) break;
            const int h = net.dims[l];
            int u = 0;
            if (l == 1) {
                if (lane < h) {
                    u = P.pot0[lane];
                    for (int t = 0; t < P.k; ++t) u += off[t] * (int)net.Wd[1][(int64_t)lane * n + pix[t]];
                }
            } else {
                u = br[l - 2];
#pragma unroll
                for (int w = 0; w < 16; ++w) u = __builtin_amdgcn_sdot4(act[w], wr[l - 2][w], u, false);
            }
            // changes against the clean image's potentials of this layer
            const int a = lane < h ? P.pot0[uoff + lane] : 0;
            const bool sa = a >= 0, sb = u >= 0;   // sign(0) = 1
            const bool s_ch = lane < h && sa != sb;
            const int64_t aa = a < 0 ? -(int64_t)a : a, bb = u < 0 ? -(int64_t)u : u;
            const int64_t mx = aa > bb ? aa : bb, mn = aa > bb ? bb : aa;
            const bool v_ch = lane < h && !s_ch && mx > 0 &&
                              (int64_t)P.cp.ratio_den * mx >= (int64_t)P.cp.ratio_num * mn;
            // squared distance, saturating (as the coverage predicates count it)
            const int64_t dd = (int64_t)a - u;
            const unsigned long long ad = (unsigned long long)(dd < 0 ? -dd : dd);
            unsigned long long d2 = lane < h ? ((ad >> 32) ? ~0ull : ad * ad) : 0ull;
            for (int sh = 32; sh >= 1; sh >>= 1) {
                const unsigned long long o = __shfl_xor(d2, sh), t = d2 + o;
                d2 = t < d2 ? ~0ull : t;
            }
            sc[l - 1] = __ballot(s_ch);
            vc[l - 1] = __ballot(v_ch);
            dc[l - 1] = sc[l - 1] == 0 && d2 >= (unsigned long long)P.cp.dist_sq_min;
            uoff += h;
            // this layer's activations for the next one; the label from the last
            __syncthreads();
            if (l < L) {
                reinterpret_cast<int8_t *>(act)[lane] = lane < h ? (int8_t)min(max(u >> net.shift[l - 1], 0), 127) : (int8_t)0;
            } else {
                // lowest-index argmax
                long long key = lane < h ? ((long long)u << 6) | (63 - lane) : LLONG_MIN;
#pragma unroll
                for (int sh = 32; sh >= 1; sh >>= 1) {
                    const long long o = __shfl_xor(key, sh);
                    key = o > key ? o : key;
                }
                label = 63 - (int)(key & 63);
            }
            __syncthreads();
        }
        // covered pairs: block l pairs layer l (rows i) with layer l + 1
        int64_t boff = 0;
        for (int l = 1; l < L; ++l) {
            const int h0 = net.dims[l], h1 = net.dims[l + 1];
            const unsigned long long single = (P.crit == 0 || P.crit == 2) ? sc[l - 1] : 0ull;
            const bool one = __popcll(single) == 1;
            const bool dist = (P.crit == 1 || P.crit == 3) && dc[l - 1];
            const unsigned long long pat = (P.crit == 0 || P.crit == 1) ? sc[l] : vc[l];
            // row lane: one sign change at that row (SS / SV), or every row (DS / DV)
            const bool row_on = lane < h0 && pat && ((one && ((single >> lane) & 1ull)) || dist);
            if (row_on) {
                const int64_t b = boff + (int64_t)lane * h1;
                const int w = (int)(b >> 6), sh = (int)(b & 63);
                atomicOr(&mask[w], pat << sh);
                if (sh && sh + h1 > 64) atomicOr(&mask[w + 1], pat >> (64 - sh));
            }
            boff += (int64_t)h0 * h1;
        }
        __syncthreads();
        for (int w = lane; w < P.words; w += 64) P.masks[c * P.words + w] = mask[w];
        if (lane == 0) P.labels[c] = label;
        __syncthreads();
    }
}

// The candidate of a key.
__device__ __forceinline__ unsigned long long cov_key_index(unsigned long long key) {
    return ((1ull << 40) - 1ull) - (key & ((1ull << 40) - 1ull));
}

// One greedy step: the gain of every candidate (pairs it covers beyond the
// covered ones), reduced to the largest gain, lowest candidate index first: key
// = gain 2^40 + (2^40 - 1 - index).  prev: the last step's covered set; with
// prev_key, that step's winner is added to it first, by every workgroup for
// itself, and the first one writes the sum (next) and the winner's label (-1:
// no winner).  A launch of its own for that took 2.3 us a step and its gap.
__global__ void __launch_bounds__(256) cov_step_kernel(const unsigned long long *masks, int64_t n_cand, int words,
                                                       const unsigned long long *prev, const unsigned long long *prev_key,
                                                       unsigned long long *next, const int32_t *labels,
                                                       int32_t *prev_label, unsigned long long *best_key) {
    __shared__ unsigned long long cov[kCovSearchMaxWords];
    __shared__ unsigned long long red[4];
    const unsigned long long last = prev_key ? *prev_key : 0ull;
    for (int w = threadIdx.x; w < words; w += blockDim.x) {
        cov[w] = prev[w] | (last ? masks[cov_key_index(last) * words + w] : 0ull);
        if (prev_key && blockIdx.x == 0) next[w] = cov[w];
    }
    if (prev_key && blockIdx.x == 0 && threadIdx.x == 0) *prev_label = last ? labels[cov_key_index(last)] : -1;
    if (!best_key) return;
    __syncthreads();
    unsigned long long key = 0;
    for (int64_t c = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; c < n_cand;
         c += (int64_t)gridDim.x * blockDim.x) {
        int gain = 0;
        for (int w = 0; w < words; ++w) gain += __popcll(masks[c * words + w] & ~cov[w]);
        const unsigned long long k =
            ((unsigned long long)gain << 40) | (((1ull << 40) - 1ull) - (unsigned long long)c);
        if (gain > 0 && k > key) key = k;
    }
    for (int sh = 32; sh >= 1; sh >>= 1) {
        const unsigned long long o = __shfl_xor(key, sh);
        key = o > key ? o : key;
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = key;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long b = red[0];
        for (int t = 1; t < (int)(blockDim.x >> 6); ++t) b = red[t] > b ? red[t] : b;
        if (b) atomicMax(best_key, b);
    }
}

hipError_t launch_cov_cand(const CovCandParams &P, hipStream_t s) {
    if (P.n_cand <= 0) return hipSuccess;
    const int grid = (int)std::min<int64_t>(P.n_cand, 4096);
    hipLaunchKernelGGL(cov_cand_kernel, dim3(grid), dim3(64), 0, s, P);
    return hipGetLastError();
}

hipError_t launch_cov_step(const unsigned long long *masks, int64_t n_cand, int words, const unsigned long long *prev,
                           const unsigned long long *prev_key, unsigned long long *next, const int32_t *labels,
                           int32_t *prev_label, unsigned long long *best_key, hipStream_t s) {
    const int grid = best_key ? (int)std::max<int64_t>(1, std::min<int64_t>((n_cand + 255) / 256, 2048)) : 1;
    hipLaunchKernelGGL(cov_step_kernel, dim3(grid), dim3(256), 0, s, masks, n_cand, words, prev, prev_key, next, labels,
                       prev_label, best_key);
    return hipGetLastError();
}

}  // namespace ibmc
