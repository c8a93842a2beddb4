// Integer-network kernels for gfx950: plain dense forward (clean pass,
// replay, forward), and the exhaustive enumeration of the bounded
// perturbation domain with incremental first layer and int8 MFMA later layers.
#include <vector>

#include "kernels_q8.h"
#include "kernels_fold.h"
#include "enum_common.h"

namespace ibmc {

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------

__device__ __forceinline__ int requant_relu(int u, int s) {
    // floor(u / 2^s) (arithmetic shift), then clamp to [0, 127]
    return min(max(u >> s, 0), 127);
}

__device__ __forceinline__ int pack4(int a0, int a1, int a2, int a3) {
    return a0 | (a1 << 8) | (a2 << 16) | (a3 << 24);
}


// ---------------------------------------------------------------------------
// plain dense forward of one image held in LDS (one workgroup of kFwdThreads)
// ---------------------------------------------------------------------------

constexpr int kFwdThreads = 1024;
constexpr int kFwdSplit = 4;  // every dot product is split over this many threads

__device__ void dense_tail_block(const QNetDev &net, int *act0, int *act1, int (*part)[kMaxWidth], int32_t *pot,
                                 int *label_out, int *tie_out);

// xs: n pixel values; act0/act1: scratch of kMaxWidth ints each; part:
// kFwdSplit x kMaxWidth ints of partial sums.  Every layer's dot products are
// split over the inputs (short dependent chains, coalesced weight reads).
// The transposed first layer is read four neurons per 32-bit load, its
// inputs split as many ways as the partial sums allow (16 for up to 256
// neurons); the row-major later layers are read 16 weights per load when a
// row is a multiple of 16 bytes, split kFwdSplit ways over the row.
// Writes potentials (natural order, layers concatenated) if pot != nullptr,
// layer-1 potentials in sigma order if u0s != nullptr; returns the label
// (thread 0 holds the valid value) and the exact-tie flag.
__device__ void dense_forward_block(const QNetDev &net, const int *xs, int *act0, int *act1,
                                    int (*part)[kMaxWidth], int32_t *pot, int32_t *u0s, int *label_out,
                                    int *tie_out) {
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int n = net.dims[0], H1 = net.H[1];
    int *const pf = &part[0][0];                     // [S1][H1] for the first layer
    // layer 1 through the transposed first layer, sigma order
    const int G1 = H1 / 4;                           // groups of four neurons
    const int S1 = max(1, min(16, kFwdSplit * kMaxWidth / H1));
    const int seg1 = (n + S1 - 1) / S1;
    for (int t = tid; t < G1 * S1; t += nthr) {
        const int grp = t % G1, sp = t / G1;
        const int i0 = sp * seg1, i1 = min(n, i0 + seg1);
        const int *w4 = reinterpret_cast<const int *>(net.W1T) + grp;   // row stride H1 / 4 words
        int u0 = 0, u1 = 0, u2 = 0, u3 = 0;
#pragma unroll 8
        for (int i = i0; i < i1; ++i) {
            const int w = w4[(int64_t)i * G1];
            const int x = xs[i];
            u0 += (int)(int8_t)w * x;
            u1 += (int)(int8_t)(w >> 8) * x;
            u2 += (int)(int8_t)(w >> 16) * x;
            u3 += (w >> 24) * x;
        }
        int *dst = pf + sp * H1 + 4 * grp;
        dst[0] = u0;
        dst[1] = u1;
        dst[2] = u2;
        dst[3] = u3;
    }
    __syncthreads();
    for (int q = tid; q < H1; q += nthr) {
        int u = net.b1s[q];
        for (int sp = 0; sp < S1; ++sp) u += pf[sp * H1 + q];
        const int neuron = sigma64(q);
        if (u0s) u0s[q] = u;
        if (neuron < net.dims[1]) {
            if (pot) pot[neuron] = u;
            act0[neuron] = (net.L > 1) ? requant_relu(u, net.shift[0]) : u;
        }
    }
    __syncthreads();
    dense_tail_block(net, act0, act1, part, pot, label_out, tie_out);
}

// Layers 2..L and the label of one image whose first-layer activations
// (natural order, requantised unless the net has one layer) are in act0.
// act1 and part are scratch as above; pot as above (layers >= 2).
__device__ void dense_tail_block(const QNetDev &net, int *act0, int *act1, int (*part)[kMaxWidth], int32_t *pot,
                                 int *label_out, int *tie_out) {
    const int tid = threadIdx.x, nthr = blockDim.x;
    int *in = act0, *out = act1;
    int po = net.dims[1];
    for (int l = 2; l <= net.L; ++l) {
        const int nin = net.dims[l - 1], nout = net.dims[l];
        const int8_t *W = net.Wd[l];
        const bool wide = (nin % 16) == 0 && (reinterpret_cast<uintptr_t>(W) % 16) == 0;
        // every dot product split sp ways, as many as the block's threads
        // allow (one task each where possible: the loads of a task are issued
        // together, so a layer costs about one memory round trip), at most
        // one 16-weight load per split point and within the partial sums
        const int units = wide ? nin / 16 : nin;
        const int split = max(1, min(min(nthr / nout, units), kFwdSplit * kMaxWidth / nout));
        // split points on 16-weight boundaries when the rows are read 16 at a time
        const int seg = wide ? (units + split - 1) / split * 16 : (nin + split - 1) / split;
        int *const pf = &part[0][0];                     // [split][nout]
        for (int t = tid; t < nout * split; t += nthr) {
            const int j = t / split, sp = t % split;
            const int i0 = sp * seg, i1 = min(nin, i0 + seg);
            const int8_t *row = W + (int64_t)j * nin;
            int u = 0;
            if (wide) {
#pragma unroll 4
                for (int i = i0; i < i1; i += 16) {
                    const int4 w = *reinterpret_cast<const int4 *>(row + i);
                    const int ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        u += (int)(int8_t)ww[c] * in[i + 4 * c] + (int)(int8_t)(ww[c] >> 8) * in[i + 4 * c + 1] +
                             (int)(int8_t)(ww[c] >> 16) * in[i + 4 * c + 2] + (ww[c] >> 24) * in[i + 4 * c + 3];
                    }
                }
            } else {
#pragma unroll 8
                for (int i = i0; i < i1; ++i) u += (int)row[i] * in[i];
            }
            pf[sp * nout + j] = u;
        }
        __syncthreads();
        for (int j = tid; j < nout; j += nthr) {
            int u = net.bd[l][j];
            for (int sp = 0; sp < split; ++sp) u += pf[sp * nout + j];
            if (pot) pot[po + j] = u;
            out[j] = (l < net.L) ? requant_relu(u, net.shift[l - 1]) : u;
        }
        po += nout;
        __syncthreads();
        int *t = in; in = out; out = t;
    }
    if (tid == 0) {
        const int nc = net.dims[net.L];
        int best = 0;
        for (int j = 1; j < nc; ++j) if (in[j] > in[best]) best = j;
        int cnt = 0;
        for (int j = 0; j < nc; ++j) cnt += in[j] == in[best];
        *label_out = best;
        *tie_out = cnt > 1;
    }
}

__global__ void __launch_bounds__(kFwdThreads) forward_q8_kernel(QNetDev net, const uint8_t *images,
                                                                 int64_t n_images, int32_t *labels,
                                                                 int32_t *pots, int64_t pot_stride) {
    __shared__ int xs[kMaxWidth];
    __shared__ int a0[kMaxWidth], a1[kMaxWidth];
    __shared__ int part[kFwdSplit][kMaxWidth];
    __shared__ int lab, tie;
    for (int64_t img = blockIdx.x; img < n_images; img += gridDim.x) {
        const uint8_t *x = images + img * net.dims[0];
        for (int i = threadIdx.x; i < net.dims[0]; i += blockDim.x) xs[i] = x[i];
        __syncthreads();
        dense_forward_block(net, xs, a0, a1, part, pots ? pots + img * pot_stride : nullptr, nullptr, &lab, &tie);
        __syncthreads();
        if (threadIdx.x == 0 && labels) labels[img] = lab;
        __syncthreads();
    }
}

// Clean pass of the properties listed in prop_ids: first-layer potentials in
// sigma order (the base of every incremental update, stored at the property's
// index) and the clean label.  Block b of the grid takes property
// prop_ids[b / S] and the first-layer neurons of slice b % S (S = H1 /
// clean_slice(H1)) over all pixels; the last of a property's S blocks to
// finish (counted in its clean_done, which starts at a multiple of S) runs
// the later layers from the stored potentials and writes the label.  One
// property thus spreads over S compute units instead of one.
__host__ __device__ inline int clean_slice(int H1) { return H1 % 64 == 0 ? 64 : 16; }
constexpr int kCleanThreads = 1024;
// a slice's partial sums, segs x slice = 4 kCleanThreads ints, fit in part
static_assert(4 * kCleanThreads <= kFwdSplit * kMaxWidth, "clean pass partial sums");

__global__ void __launch_bounds__(kCleanThreads) clean_q8_kernel(QNetDev net, PropDev *props,
                                                                 const int32_t *prop_ids, int32_t n_ids,
                                                                 int32_t *u0_store, int64_t u0_stride) {
    __shared__ int a0[kMaxWidth], a1[kMaxWidth];
    __shared__ int part[kFwdSplit][kMaxWidth];
    __shared__ int lab, tie, last;
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int n = net.dims[0], H1 = net.H[1];
    const int slice = clean_slice(H1), S = H1 / slice;
    const int G = slice / 4;                             // four neurons per 32-bit weight word
    const int segs = nthr / G;                           // pixel segments (segs * slice <= 4 kMaxWidth)
    const int G1 = H1 / 4;
    for (int64_t b = blockIdx.x; b < (int64_t)n_ids * S; b += gridDim.x) {
        const int pid = prop_ids[b / S];
        const int w = (int)(b % S);
        const uint8_t *x = props[pid].image;
        int32_t *u0s = u0_store + (int64_t)pid * u0_stride;
        // partial sums of the slice over this thread's pixel segment
        const int grp = tid % G, sg = tid / G;
        const int seg = (n + segs - 1) / segs;
        const int i0 = sg * seg, i1 = min(n, i0 + seg);
        const int *w4 = reinterpret_cast<const int *>(net.W1T) + w * G + grp;   // row stride G1 words
        int u0 = 0, u1 = 0, u2 = 0, u3 = 0;
#pragma unroll 8
        for (int i = i0; i < i1; ++i) {
            const int wv = w4[(int64_t)i * G1];
            const int xv = x[i];
            u0 += (int)(int8_t)wv * xv;
            u1 += (int)(int8_t)(wv >> 8) * xv;
            u2 += (int)(int8_t)(wv >> 16) * xv;
            u3 += (wv >> 24) * xv;
        }
        int *pf = &part[0][0];                            // [segs][slice]
        pf[sg * slice + 4 * grp + 0] = u0;
        pf[sg * slice + 4 * grp + 1] = u1;
        pf[sg * slice + 4 * grp + 2] = u2;
        pf[sg * slice + 4 * grp + 3] = u3;
        __syncthreads();
        if (tid < slice) {
            const int q = w * slice + tid;
            int u = net.b1s[q];
            for (int t = 0; t < segs; ++t) u += pf[t * slice + tid];
            u0s[q] = u;
        }
        // publish the slice, then count it (release); the block that
        // completes the count sees every slice (acquire)
        __threadfence();
        __syncthreads();
        if (tid == 0) last = (atomicAdd(&props[pid].clean_done, 1) + 1) % S == 0;
        __syncthreads();
        if (last) {
            __threadfence();
            for (int q = tid; q < H1; q += nthr) {
                const int neuron = sigma64(q);
                if (neuron < net.dims[1]) {
                    const int u = u0s[q];
                    a0[neuron] = (net.L > 1) ? requant_relu(u, net.shift[0]) : u;
                }
            }
            __syncthreads();
            dense_tail_block(net, a0, a1, part, nullptr, &lab, &tie);
            __syncthreads();
            if (tid == 0) { props[pid].label0 = lab; props[pid].tie0 = tie; }
        }
        __syncthreads();
    }
}

// Scan of the folded properties: the clean pass of clean_q8_kernel with, per
// first-layer unit, the largest and smallest change that one perturbed pixel
// can make (every delta between the smallest and the largest, clamped to
// [0, 255] with the pixel).  k of them bound the potential over the whole
// domain; the block that completes a property's slices turns the bounds into
// activation intervals and lists the live units (intervals of more than one
// value).  Latency-bound: one weight pass over the first layer (as the clean
// pass) and the clean label's forward pass.
constexpr int kScanSlice = 64;

// Appends value to list for every thread of the block whose flag is set, in
// thread order; returns how many (cnt: one int per wave).
__device__ int fold_compact(bool flag, int value, int32_t *list, int *cnt) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const unsigned long long m = __ballot(flag);
    if (lane == 0) cnt[wv] = __popcll(m);
    __syncthreads();
    int before = 0, all = 0;
    for (int t = 0; t < nw; ++t) {
        before += t < wv ? cnt[t] : 0;
        all += cnt[t];
    }
    if (flag) list[before + __popcll(m & ((1ull << lane) - 1ull))] = value;
    __syncthreads();
    return all;
}

// Output layer of a folded property, a wave per row: bias with the constant
// inputs, and the live inputs' weights times their offsets; then into `two`
// (0 before) whether a weight difference to the label's row leaves int8 on a
// live input (1) or is 127 - (-128) = 255, which no two int8 add up to (2).
// iv(i): input i's interval as lowest | highest << 8; off(i): its offset.
template <class IV, class OFF>
__device__ void fold_output(const QNetDev &net, int lab, int32_t *bo, int32_t *rso, int *two, IV iv, OFF off) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int L = net.L, nin = net.dims[L - 1], nc = net.dims[L];
    for (int r = wv; r < nc; r += nw) {
        const int8_t *row = net.Wd[L] + (int64_t)r * nin, *lrow = net.Wd[L] + (int64_t)lab * nin;
        int cs = 0, sum = 0, wide = 0;
#pragma unroll 4
        for (int i = lane; i < nin; i += 64) {
            const int c = row[i], d = c - (int)lrow[i], v = iv(i), a = v & 0xff;
            const bool fixed = a == ((v >> 8) & 0xff);
            cs += fixed ? c * a : 0;
            sum += fixed ? 0 : c * off(i);
            wide |= fixed ? 0 : (d < -128 || d > 127) | (d > 254) << 1;
        }
        for (int d = 32; d > 0; d >>= 1) {
            cs += __shfl_xor(cs, d);
            sum += __shfl_xor(sum, d);
        }
        if (wide) atomicOr(two, wide);
        if (lane == 0) {
            bo[r] = net.bd[L][r] + cs;
            rso[r] = sum;
        }
    }
    __syncthreads();
}

__global__ void __launch_bounds__(kCleanThreads) fold_scan_kernel(const QNetDev *nets, const FoldProp *fps,
                                                                  PropDev *props, const int32_t *block_map,
                                                                  int32_t *u0_store, int64_t u0_stride) {
    __shared__ int a0[kMaxWidth], a1[kMaxWidth];
    __shared__ int part[3 * 64][kScanSlice];
    static_assert(sizeof(part) >= sizeof(int) * kFwdSplit * kMaxWidth, "dense tail scratch");
    __shared__ int lab, tie, last, cnt[16], two;
    const int tid = threadIdx.x, lane = tid & 63;
    const FoldProp F = fps[block_map[blockIdx.x] >> 8];
    const int w = block_map[blockIdx.x] & 0xff;
    const QNetDev &net = nets[F.net];
    const int n = net.dims[0], H1 = net.H[1], L = net.L, h1 = net.dims[1];
    const int S = H1 / kScanSlice, G1 = H1 / 4;
    const FoldWs ws = fold_ws(H1, L == 3 ? net.H[2] : 0);
    const uint8_t *x = props[F.pid].image;
    int32_t *u0s = u0_store + (int64_t)F.pid * u0_stride;
    {
        // 16 groups of four units, 64 pixel segments
        const int grp = tid & 15, sg = tid >> 4;
        const int seg = (n + 63) / 64;
        const int i0 = sg * seg, i1 = min(n, i0 + seg);
        const int *w4 = reinterpret_cast<const int *>(net.W1T) + w * 16 + grp;
        int u[4] = {0, 0, 0, 0}, up[4] = {0, 0, 0, 0}, dn[4] = {0, 0, 0, 0};
#pragma unroll 8
        for (int i = i0; i < i1; ++i) {
            const int wd = w4[(int64_t)i * G1];
            const int xv = x[i];
            const int eh = min(xv + F.dhi, 255) - xv, el = max(xv + F.dlo, 0) - xv;   // eh >= 0 >= el
#pragma unroll
            for (int z = 0; z < 4; ++z) {
                const int c = (int)(int8_t)(wd >> (8 * z));
                u[z] += c * xv;
                const int p = c * eh, q = c * el;
                up[z] = max(up[z], max(p, q));
                dn[z] = min(dn[z], min(p, q));
            }
        }
#pragma unroll
        for (int z = 0; z < 4; ++z) {
            part[sg][4 * grp + z] = u[z];
            part[64 + sg][4 * grp + z] = up[z];
            part[128 + sg][4 * grp + z] = dn[z];
        }
        __syncthreads();
        if (tid < 3 * kScanSlice) {
            const int what = tid >> 6, q = w * kScanSlice + lane;
            int v = what == 0 ? net.b1s[q] : 0;
            for (int t = 0; t < 64; ++t) {
                const int pv = part[64 * what + t][lane];
                v = what == 0 ? v + pv : what == 1 ? max(v, pv) : min(v, pv);
            }
            if (what == 0) u0s[q] = v;
            else F.ws[(what == 1 ? ws.ub : ws.lb) + q] = v;
        }
    }
    // publish the slice, then count it (release); the block that completes
    // the count sees every slice (acquire)
    __threadfence();
    __syncthreads();
    if (tid == 0) last = (atomicAdd(&props[F.pid].clean_done, 1) + 1) % S == 0;
    __syncthreads();
    if (!last) return;
    __threadfence();
    // intervals of layer 1 (H1 <= 1024 threads): 64-bit bounds, they may
    // leave int32
    bool live = false;
    if (tid < H1) {
        const int neuron = sigma64(tid);
        if (neuron < h1) {
            const int64_t u = u0s[tid];
            const int64_t hi = (u + (int64_t)F.k * F.ws[ws.ub + tid]) >> net.shift[0];
            const int64_t lo = (u + (int64_t)F.k * F.ws[ws.lb + tid]) >> net.shift[0];
            const int ih = (int)min((int64_t)127, max((int64_t)0, hi)), il = (int)min((int64_t)127, max((int64_t)0, lo));
            const int a = requant_relu((int)u, net.shift[0]);
            a0[neuron] = a;
            F.ws[ws.iv1 + neuron] = il | ih << 8 | a << 16;
            live = ih != il;
        }
    }
    const int live1 = fold_compact(live, tid, F.ws + ws.list1, cnt);
    dense_tail_block(net, a0, a1, reinterpret_cast<int (*)[kMaxWidth]>(&part[0][0]), nullptr, &lab, &tie);
    __syncthreads();
    if (tid == 0) {
        props[F.pid].label0 = lab;
        props[F.pid].tie0 = tie;
        F.ws[ws.done] = 0;
        F.counts[0] = live1;
        F.counts[3] = lab;
        two = 0;
    }
    __syncthreads();
    if (L == 2) {
        fold_output(net, lab, F.ws + ws.bo, F.ws + ws.rso, &two, [&](int i) { return F.ws[ws.iv1 + i]; },
                    [](int) { return 64; });
        if (tid == 0) {
            F.counts[1] = 0;
            F.counts[2] = two;
        }
    }
}

// Second hidden layer of the scanned three-layer properties.  A block takes
// 64 rows of one property: per row the bias with the constant inputs, the
// live weights' sum, and bounds of the potential over the domain, the
// tighter of
//   - the inputs' intervals, and
//   - the joint bound: one pixel's change d of the first-layer potentials
//     moves the row by at most sum_j max(0, w_j d_j) / 2^s (the requantiser is
//     monotone and contracts by 2^s), and with d_j = e W_jp
//     sum_j max(0, w_j W_jp) = (sum |w_j| |W_jp| + sum w_j W_jp) / 2: two int8
//     matrix products over the pixels.  k times the largest over the pixels,
//     plus the live weights' |w| for the floors.
// On blob images with k = 2 it leaves about two thirds of the units that the
// intervals alone leave live, and half of the ones with both ends in reach.
// The block that completes a property lists the live rows in the order of
// their forms (FoldForm) and does the output layer.
constexpr int kBoundPix = 256;   // pixels per round of the joint bound

__global__ void __launch_bounds__(256) fold_bound_kernel(const QNetDev *nets, const FoldProp *fps, const PropDev *props,
                                                         const int32_t *row_map) {
    __shared__ __attribute__((aligned(16))) int8_t wb[kBoundPix / 16 * 1024];   // one K-block of pixel columns
    __shared__ int l1[kFoldMaxWidth];
    __shared__ int res[64][6];
    __shared__ int cnt[4], last, two;
    __shared__ int iv2[kMaxWidth];
    __shared__ int16_t offs[kMaxWidth];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int j16 = lane & 15, g = lane >> 4;
    const FoldProp F = fps[row_map[blockIdx.x] >> 8];
    const int r0 = (row_map[blockIdx.x] & 0xff) * 64;
    const QNetDev &net = nets[F.net];
    const int n = net.dims[0], H1 = net.H[1], h1 = net.dims[1], h2 = net.dims[2];
    const FoldWs ws = fold_ws(H1, net.H[2]);
    const int live1 = F.counts[0];
    const int8_t *W2 = net.Wd[2];
    // row sums, a row per lane and a quarter of the columns per wave: constant
    // part, live weights, interval below and above the constant part, live
    // |w|, live clean part
    for (int t = tid; t < kMaxWidth; t += 256) iv2[t] = t < h1 ? F.ws[ws.iv1 + t] : 0;
    for (int t = tid; t < kFoldMaxWidth; t += 256) l1[t] = t < live1 ? F.ws[ws.list1 + t] : -1;
    for (int t = tid; t < 64 * 6; t += 256) (&res[0][0])[t] = 0;
    __syncthreads();
    {
        const int row = min(r0 + lane, h2 - 1);
        const int8_t *wr = W2 + (int64_t)row * h1;
        const int per = ((h1 + 15) / 16) * 4, c0 = wv * per, c1 = min(c0 + per, h1);   // columns, in fours
        const bool words = h1 % 4 == 0;
        int v[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll 4
        for (int i = c0; i < c1; i += 4) {
            unsigned wd = 0;
            if (words) {
                wd = *reinterpret_cast<const unsigned *>(wr + i);
            } else {
#pragma unroll
                for (int z = 0; z < 4; ++z) wd |= (unsigned)(uint8_t)wr[min(i + z, h1 - 1)] << (8 * z);
            }
#pragma unroll
            for (int z = 0; z < 4; ++z) {
                // (past the end: interval 0..0)
                const int iv = iv2[i + z], lo = iv & 0xff, hi = (iv >> 8) & 0xff, a = iv >> 16;
                const int c = (int)(int8_t)(wd >> (8 * z));
                const bool live = lo != hi;
                v[0] += live ? 0 : c * lo;
                v[1] += live ? c : 0;
                v[2] += live ? min(c * lo, c * hi) : 0;
                v[3] += live ? max(c * lo, c * hi) : 0;
                v[4] += live ? abs(c) : 0;
                v[5] += live ? c * a : 0;
            }
        }
#pragma unroll
        for (int z = 0; z < 6; ++z) atomicAdd(&res[lane][z], v[z]);
    }
    __syncthreads();
    // joint bound of the wave's 16 rows: lane (j16, g) holds rows 4 g + z
    const bool joint = F.joint && live1 > 0 && live1 <= kFoldMaxWidth;
    int mu[4] = {0, 0, 0, 0}, md[4] = {0, 0, 0, 0};
    if (joint) {
        const uint8_t *x = props[F.pid].image;
        const int KB = (live1 + 63) / 64;
        for (int p0 = 0; p0 < n; p0 += kBoundPix) {
            v4i sp[kBoundPix / 16], sq[kBoundPix / 16];   // sum w W and sum |w| |W| per pixel tile
#pragma unroll
            for (int t = 0; t < kBoundPix / 16; ++t) sp[t] = sq[t] = v4i{0, 0, 0, 0};
            for (int kb = 0; kb < KB; ++kb) {
                __syncthreads();
                // this K-block's columns of the pixels: thread (pixel tid / 16 + 16 r,
                // dword tid % 16), every byte load of eight pixels in flight together
                {
                    const int ln = tid & 15, px = tid >> 4;      // dword (ln / 4 = lane group, ln % 4)
                    int q[4];
#pragma unroll
                    for (int z = 0; z < 4; ++z) q[z] = l1[kb * 64 + ln * 4 + z];
                    for (int r = 0; r < kBoundPix / 16; r += 8) {
                        unsigned v[8];
#pragma unroll
                        for (int h = 0; h < 8; ++h) {
                            const int p = p0 + (r + h) * 16 + px;
                            const int8_t *col = net.W1T + (int64_t)min(p, n - 1) * H1;
                            v[h] = 0;
#pragma unroll
                            for (int z = 0; z < 4; ++z) {
                                const unsigned c = (unsigned)(uint8_t)col[max(q[z], 0)];
                                v[h] |= (q[z] >= 0 ? c : 0u) << (8 * z);
                            }
                            if (p >= n) v[h] = 0;
                        }
#pragma unroll
                        for (int h = 0; h < 8; ++h)   // tile r + h, lane px + 16 (ln / 4), dword ln % 4
                            reinterpret_cast<unsigned *>(wb)[(r + h) * 256 + (px + 16 * (ln >> 2)) * 4 + (ln & 3)] = v[h];
                    }
                }
                v4i A, B;
                const int row = r0 + wv * 16 + j16;
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    unsigned v = 0, u = 0;
#pragma unroll
                    for (int z = 0; z < 4; ++z) {
                        const int q = l1[kb * 64 + g * 16 + d * 4 + z];
                        const int w = (int)W2[(int64_t)min(row, h2 - 1) * h1 + (q >= 0 ? sigma64(q) : 0)];
                        const int c = row < h2 && q >= 0 ? w : 0;
                        v |= (unsigned)(uint8_t)c << (8 * z);
                        u |= (unsigned)abs(c) << (8 * z);
                    }
                    A[d] = (int)v;
                    B[d] = (int)u;
                }
                __syncthreads();
#pragma unroll
                for (int t = 0; t < kBoundPix / 16; ++t) {
                    const v4i W = *reinterpret_cast<const v4i *>(wb + t * 1024 + lane * 16);
                    v4i N;
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        // |byte| = (byte ^ s) - s with s = -1 for negative bytes, no borrow between bytes
                        const unsigned s = (((unsigned)W[d] >> 7) & 0x01010101u);
                        N[d] = (int)(((unsigned)W[d] ^ (s * 0xffu)) + s);
                    }
                    sp[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A, W, sp[t], 0, 0, 0);
                    sq[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(B, N, sq[t], 0, 0, 0);
                }
            }
#pragma unroll
            for (int t = 0; t < kBoundPix / 16; ++t) {
                const int p = p0 + t * 16 + j16;
                const int xv = p < n ? x[p] : 0;
                const int eh = p < n ? min(xv + F.dhi, 255) - xv : 0, el = p < n ? xv - max(xv + F.dlo, 0) : 0;
#pragma unroll
                for (int z = 0; z < 4; ++z) {
                    const int pos = (sq[t][z] + sp[t][z]) >> 1, neg = (sq[t][z] - sp[t][z]) >> 1;
                    // (24-bit products: pos, neg < 2^23)
                    mu[z] = max(mu[z], max(__mul24(pos, eh), __mul24(neg, el)));
                    md[z] = max(md[z], max(__mul24(neg, eh), __mul24(pos, el)));
                }
            }
        }
        for (int d = 8; d > 0; d >>= 1)
#pragma unroll
            for (int z = 0; z < 4; ++z) {
                mu[z] = max(mu[z], __shfl_xor(mu[z], d));
                md[z] = max(md[z], __shfl_xor(md[z], d));
            }
    }
    if (j16 < 4) {
        const int lr = wv * 16 + 4 * g + j16, row = r0 + lr;
        const int up = j16 == 0 ? mu[0] : j16 == 1 ? mu[1] : j16 == 2 ? mu[2] : mu[3];
        const int dn = j16 == 0 ? md[0] : j16 == 1 ? md[1] : j16 == 2 ? md[2] : md[3];
        if (row < h2) {
            const int b = net.bd[2][row] + res[lr][0];
            int64_t lo = (int64_t)b + res[lr][2], hi = (int64_t)b + res[lr][3];
            if (joint) {
                const int64_t c = (int64_t)b + res[lr][5];
                hi = min(hi, c + res[lr][4] + 1 + ((int64_t)F.k * up >> net.shift[0]));
                lo = max(lo, c - res[lr][4] - 1 - ((int64_t)F.k * dn >> net.shift[0]));
            }
            const int s2 = net.shift[1];
            const int form = lo >= 0 ? FOLD_UPPER : (hi >> s2) <= 127 ? FOLD_LOWER : FOLD_BOTH;
            const int al = (int)min((int64_t)127, max((int64_t)0, lo >> s2));
            const int ah = (int)min((int64_t)127, max((int64_t)0, hi >> s2));
            F.ws[ws.b2 + row] = b;
            F.ws[ws.rs2 + row] = res[lr][1];
            F.ws[ws.iv2 + row] = al | ah << 8 | form << 16;
        }
    }
    __threadfence();
    __syncthreads();
    if (tid == 0) last = atomicAdd(&F.ws[ws.done], 1) + 1 == (h2 + 63) / 64;
    __syncthreads();
    if (!last) return;
    __threadfence();
    // live rows by form; with the saturating epilogue (shift 7) the pairs of
    // tiles that hold no row with both ends in reach need no cap, and their FOLD_UPPER
    // rows take offset 0 instead of 128
    const bool sat = net.shift[1] == 7;
    for (int t = tid; t < h2; t += 256) iv2[t] = F.ws[ws.iv2 + t];
    if (tid == 0) two = 0;
    __syncthreads();
    int total = 0, n_free = 0;
    for (int f = FOLD_UPPER; f <= FOLD_BOTH; ++f) {
        for (int b = 0; b < h2; b += 256) {
            const int row = b + tid;
            const int iv = row < h2 ? iv2[row] : 0;
            const bool on = row < h2 && (iv & 0xff) != ((iv >> 8) & 0xff) && (iv >> 16) == f;
            total += fold_compact(on, row, F.ws + ws.list2 + total, cnt);
        }
        if (f <= FOLD_LOWER) n_free = total;
    }
    // (with every live row free of the cap, the last, partly filled pair is too)
    const int free_pairs = !sat ? 0 : n_free == total ? (total + 31) / 32 : n_free / 32;
    for (int t = tid; t < total; t += 256) {
        const int row = F.ws[ws.list2 + t];
        offs[row] = (int16_t)(!sat ? 64 : t / 32 < free_pairs && (iv2[row] >> 16) == FOLD_UPPER ? 0 : 128);
    }
    __syncthreads();
    fold_output(net, F.counts[3], F.ws + ws.bo, F.ws + ws.rso, &two, [&](int i) { return iv2[i]; },
                [&](int i) { return (int)offs[i]; });
    if (tid == 0) {
        F.counts[1] = total | free_pairs << 16;
        F.counts[2] = two;
    }
}

// Replay: rebuild each perturbed image from its record and run the plain
// forward pass.
__global__ void __launch_bounds__(kFwdThreads) replay_q8_kernel(QNetDev net, const uint8_t *clean,
                                                                const int16_t *deltas, int m,
                                                                const CexRec *recs, int64_t n_recs,
                                                                int32_t *labels) {
    __shared__ int xs[kMaxWidth];
    __shared__ int a0[kMaxWidth], a1[kMaxWidth];
    __shared__ int part[kFwdSplit][kMaxWidth];
    __shared__ int lab, tie;
    __shared__ int pix[kMaxK], dig[kMaxK];
    const int n = net.dims[0];
    for (int64_t r = blockIdx.x; r < n_recs; r += gridDim.x) {
        const int k = recs[r].k;
        if (threadIdx.x == 0) {
            int64_t mk = 1;
            for (int j = 0; j < k; ++j) mk *= m;
            int64_t srank = recs[r].rank / mk, drank = recs[r].rank % mk;
            int p[kMaxK];
            lex_unrank_subset(srank, k, n, p);
            for (int j = k - 1; j >= 0; --j) { dig[j] = (int)(drank % m); drank /= m; }
            for (int j = 0; j < k; ++j) pix[j] = p[j];
        }
        for (int i = threadIdx.x; i < n; i += blockDim.x) xs[i] = clean[i];
        __syncthreads();
        if (threadIdx.x == 0)
            for (int j = 0; j < k; ++j) xs[pix[j]] = clamp_pixel(xs[pix[j]] + deltas[dig[j]]);
        __syncthreads();
        dense_forward_block(net, xs, a0, a1, part, nullptr, nullptr, &lab, &tie);
        __syncthreads();
        if (threadIdx.x == 0) labels[r] = lab;
        __syncthreads();
    }
}

__global__ void fill_u64_kernel(unsigned long long *p, int64_t n, unsigned long long v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// ---------------------------------------------------------------------------
// enumeration
// ---------------------------------------------------------------------------

// ---------------------------------------------------------------------------
// instantiation table (the instances live in enum_q8_*.hip, compiled in parallel)
// ---------------------------------------------------------------------------

const EnumVariant *enum_variants(int *count) {
    static std::vector<EnumVariant> all;
    if (all.empty()) {
        int n = 0;
        const EnumVariant *v = enum_variants_l2(&n);
        all.insert(all.end(), v, v + n);
        v = enum_variants_l3a(&n);
        all.insert(all.end(), v, v + n);
        v = enum_variants_l3b(&n);
        all.insert(all.end(), v, v + n);
        v = enum_variants_l3a_fast(&n);
        all.insert(all.end(), v, v + n);
        v = enum_variants_l3b_fast(&n);
        all.insert(all.end(), v, v + n);
        v = enum_variants_general(&n);
        all.insert(all.end(), v, v + n);
    }
    *count = (int)all.size();
    return all.data();
}

// ---------------------------------------------------------------------------
// host launch wrappers
// ---------------------------------------------------------------------------

hipError_t launch_forward_q8(const QNetDev &net, const uint8_t *images, int64_t n_images,
                             int32_t *labels, int32_t *pots, int64_t pot_stride, hipStream_t s) {
    if (n_images <= 0) return hipSuccess;
    const int grid = (int)std::min<int64_t>(n_images, 4096);
    hipLaunchKernelGGL(forward_q8_kernel, dim3(grid), dim3(kFwdThreads), 0, s, net, images, n_images,
                       labels, pots, pot_stride);
    return hipGetLastError();
}

hipError_t launch_clean_q8(const QNetDev &net, PropDev *props, const int32_t *prop_ids,
                           int32_t n_ids, int32_t *u0_store, int64_t u0_stride, hipStream_t s) {
    if (n_ids <= 0) return hipSuccess;
    if (net.H[1] % 16) return hipErrorInvalidValue;
    const int grid = (int)std::min<int64_t>((int64_t)n_ids * (net.H[1] / clean_slice(net.H[1])), 8192);
    hipLaunchKernelGGL(clean_q8_kernel, dim3(grid), dim3(kCleanThreads), 0, s, net, props, prop_ids, n_ids,
                       u0_store, u0_stride);
    return hipGetLastError();
}

hipError_t launch_fold_scan(const QNetDev *nets, const FoldProp *fps, PropDev *props, const int32_t *block_map,
                            int n_blocks, int32_t *u0_store, int64_t u0_stride, hipStream_t s) {
    if (n_blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(fold_scan_kernel, dim3(n_blocks), dim3(kCleanThreads), 0, s, nets, fps, props, block_map,
                       u0_store, u0_stride);
    return hipGetLastError();
}

hipError_t launch_fold_bound(const QNetDev *nets, const FoldProp *fps, const PropDev *props, const int32_t *row_map,
                             int n_blocks, hipStream_t s) {
    if (n_blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(fold_bound_kernel, dim3(n_blocks), dim3(256), 0, s, nets, fps, props, row_map);
    return hipGetLastError();
}

hipError_t launch_replay_q8(const QNetDev &net, const uint8_t *clean, const int16_t *deltas, int m,
                            const CexRec *recs, int64_t n_recs, int32_t *labels, hipStream_t s) {
    if (n_recs <= 0) return hipSuccess;
    const int grid = (int)std::min<int64_t>(n_recs, 8192);
    hipLaunchKernelGGL(replay_q8_kernel, dim3(grid), dim3(kFwdThreads), 0, s, net, clean, deltas, m, recs,
                       n_recs, labels);
    return hipGetLastError();
}

hipError_t launch_fill_u64(unsigned long long *p, int64_t n, unsigned long long v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int grid = (int)std::min<int64_t>((n + 255) / 256, 1024);
    hipLaunchKernelGGL(fill_u64_kernel, dim3(grid), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

int64_t enum_lds_bytes(const EnumVariant &v, const QNetDev &net) {
    int64_t w = 0;
    if (v.wlds) {
        if (v.L == 3) w += (int64_t)(net.H[2] / 16) * v.kb1 * 1024;
        const int kbl = (v.L == 3) ? v.kb2 : v.kb1;
        w += (int64_t)(net.H[v.L] / 16) * kbl * 1024;
    }
    const int64_t biases = 4LL * ((v.L == 3 ? (int64_t)v.kb2 * 64 : 0) + net.H[v.L]);
    // per wave (4 per workgroup): one int32 or kSegGroup int16 first-layer
    // bases, and the cursor record
    const int64_t h1 = (int64_t)v.kb1 * 64;
    return w + biases + 4LL * std::max<int64_t>(h1 * 4, (int64_t)kSegGroup * h1 * 2) + 4LL * (int64_t)sizeof(Cursor);
}

hipError_t launch_enum_q8(const EnumVariant &v, int grid, const EnumParams &P,
                          const int32_t *u0_store, int64_t u0_stride, const int32_t *u0_index,
                          hipStream_t s) {
    const int64_t lds = enum_lds_bytes(v, P.net);
    EnumParams Q = P;
    Q.notify = (P.stop_on_first || P.track_first || P.hit_host) ? 1 : 0;
    void *args[] = {&Q, &u0_store, &u0_stride, &u0_index};
    return hipLaunchKernel(v.fn, dim3(grid), dim3(256), args, (size_t)lds, s);
}

}  // namespace ibmc
