// Training kernels of the float (sigmoid) networks, two launches per step.
//
// The pass: a workgroup takes four samples through the forward pass (a_0 =
// x / 256, sigmoid hidden layers, linear logits, Eq. (2)), the softmax
// cross-entropy against the label and the deltas of the backward pass.  Every
// layer product runs on the FP32 matrix instruction of sixteen 4 x 4 blocks,
// whose blocks are sixteen groups of four rows and whose columns are the four
// samples: a wave covers 64 rows, one input per instruction, so that every
// output is one chain of fma over the inputs in order.  Four samples a
// workgroup, because a batch of 256 then spreads over 64 compute units where
// tiles of sixteen would leave it on sixteen; what remains is latency, so a
// layer's first weights are loaded before the barrier that its inputs wait for
// and 32 inputs' weights stay in flight along the chain.
//
// The weights: a workgroup per 16 x 16 tile of a layer's gradient
// sum_s delta_s a_s^T (the bias as one more input that is 1), up to 256
// samples' rows staged in LDS in one go; a lane sums one entry, group by group
// of samples (train_group), and takes its Adam step in place, so no gradient
// goes through memory.  A workgroup of its own sums the loss beside them.
//
// Fixed summation order, no atomics: a training run is the same on every call.
// Measured, 35-256-128-10 at batch 256, per step: pass 25 us, weights 8 us (a
// tile of eight samples per workgroup on the vector ALU with partial
// gradients, their sum and the Adam step as launches of their own: 88 + 10 +
// 5 us); an epoch of 20,000 samples 8.5 -> 3.1 ms, with the same bits.  Bound
// by latency: the products' operations take about 1 us.  Small networks are at
// the kernels' own latency (35-16-5, batch 1: 7 + 2.4 us a step, where the former
// launches took 6.3 + 1.2 + 1.5; 5,000 samples in one pass: a serial sum over 20
// stages, 91 us).  (Inputs and samples
// split over waves and added at the end took 19 + 5 us, but rounded otherwise:
// an epoch's loss moved by 2e-9.)
#include "kernels_train.h"

namespace ibmc {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v4f_u __attribute__((ext_vector_type(4), aligned(4)));

TrainNetDev train_layout(int L, const int *dims) {
    TrainNetDev N{};
    N.L = L;
    int64_t t = 0;
    int a = 0;
    for (int l = 0; l <= L; ++l) {
        N.dims[l] = dims[l];
        N.aoff[l] = a;
        a += round_up(dims[l], 4);
        N.widest = std::max(N.widest, round_up(dims[l], 4));
        if (l == 0) continue;
        N.toff[l] = t;
        t += (int64_t)dims[l] * dims[l - 1] + dims[l];
    }
    N.n_params = t;
    N.units = a;
    return N;
}

int train_group(const TrainNetDev &N, int wanted) {
    int64_t units = 0;
    for (int l = 0; l <= N.L; ++l) units += N.dims[l];
    int g = std::max(1, std::min(wanted, kTrainMaxGroup));
    while (g > 1 && g * (2 * units - N.dims[0] + 1) * 4 > 64 * 1024) --g;
    return g;
}

// A barrier for data in LDS alone: loads from memory stay in flight over it.
__device__ __forceinline__ void train_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// acc += sum over k < K of M[row][k] in[sample][k], in order.  ROWS: M is W
// (row-major, a row per lane); else M is W transposed (W[k][row]).
template <bool ROWS>
struct TrainChain {
    static constexpr int AHEAD = 8;   // groups of four inputs in flight
    const float *W;
    int R, K, row;
    v4f cur[AHEAD];

    __device__ __forceinline__ void load(v4f (&w)[AHEAD], int k) const {
#pragma unroll
        for (int h = 0; h < AHEAD; ++h) {
            const int at = k + 4 * h;
            if (at + 4 > K) continue;
            if constexpr (ROWS) {
                w[h] = *reinterpret_cast<const v4f_u *>(W + (int64_t)row * K + at);
            } else {
#pragma unroll
                for (int z = 0; z < 4; ++z) w[h][z] = W[(int64_t)(at + z) * R + row];
            }
        }
    }
    __device__ __forceinline__ void start(const float *W_, int R_, int K_, int row_) {
        W = W_;
        R = R_;
        K = K_;
        row = min(row_, R_ - 1);
        load(cur, 0);
    }
    __device__ __forceinline__ void run(const float *x, v4f &acc) {
        int k = 0;
        for (; k + 4 * AHEAD <= K; k += 4 * AHEAD) {
            v4f nxt[AHEAD];
            load(nxt, k + 4 * AHEAD);
#pragma unroll
            for (int h = 0; h < AHEAD; ++h) step(cur[h], x + k + 4 * h, acc);
#pragma unroll
            for (int h = 0; h < AHEAD; ++h) cur[h] = nxt[h];
        }
#pragma unroll
        for (int h = 0; h < AHEAD; ++h)
            if (k + 4 * h + 4 <= K) step(cur[h], x + k + 4 * h, acc);
        for (k = K & ~3; k < K; ++k)
            acc = __builtin_amdgcn_mfma_f32_4x4x1f32(ROWS ? W[(int64_t)row * K + k] : W[(int64_t)k * R + row], x[k], acc, 0, 0, 0);
    }
    static __device__ __forceinline__ void step(const v4f &w, const float *x, v4f &acc) {
        const v4f b = *reinterpret_cast<const v4f *>(x);
#pragma unroll
        for (int z = 0; z < 4; ++z) acc = __builtin_amdgcn_mfma_f32_4x4x1f32(w[z], b[z], acc, 0, 0, 0);
    }
};

// (lane 4 b + c, register r of a chain: row 4 b + r of the wave's 64, sample c)
__global__ void __launch_bounds__(1024) train_pass_kernel(TrainPassParams P) {
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const TrainNetDev &N = P.net;
    const int tid = threadIdx.x, nt = blockDim.x, L = N.L, n = N.dims[0], U = N.units, D = N.widest;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), c = lane & 3, r0 = wave * 64 + (lane & ~3);
    const int64_t first = (int64_t)blockIdx.x * kTrainTile;
    const int S = (int)min((int64_t)kTrainTile, P.count - first);
    float *act = lds;                               // [4][U]
    float *del = act + 4 * U;                       // [2][4][D]: this layer's deltas and the next
    // zeros for the missing samples
    for (int t = tid; t < 4 * n; t += nt) {
        const int s = t / n, i = t - s * n;
        float v = 0.f;
        if (s < S) {
            const int64_t e = P.e0 + first + s;
            const int64_t img = P.order ? P.order[e] : e;
            v = (float)P.images[img * n + i] * (1.f / 256.f);
        }
        act[s * U + i] = v;
    }
    for (int l = 1; l <= L; ++l) {
        const int nin = N.dims[l - 1], nout = N.dims[l];
        const float *W = P.theta + N.toff[l], *b = W + (int64_t)nout * nin;
        TrainChain<true> ch;
        v4f acc = v4f{0.f, 0.f, 0.f, 0.f};
        const bool on = wave * 64 < nout;
        if (on) {
            ch.start(W, nout, nin, wave * 64 + lane);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] = b[min(r0 + r, nout - 1)];
        }
        train_barrier();
        if (on) {
            ch.run(act + c * U + N.aoff[l - 1], acc);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (r0 + r < nout) act[c * U + N.aoff[l] + r0 + r] = (l < L) ? 1.f / (1.f + expf(-acc[r])) : acc[r];
        }
    }
    train_barrier();
    // softmax cross-entropy of each sample's logits; dL/du of the logits
    const int nc = N.dims[L];
    if (tid < 4) {
        if (tid < S) {
            const int64_t e = P.e0 + first + tid;
            const int y = P.labels[P.order ? P.order[e] : e];
            const float *z = act + tid * U + N.aoff[L];
            float zmax = z[0];
            for (int q = 1; q < nc; ++q) zmax = fmaxf(zmax, z[q]);
            float sum = 0.f;
            for (int q = 0; q < nc; ++q) sum += expf(z[q] - zmax);
            P.loss[first + tid] = logf(sum) - (z[y] - zmax);
            const float inv = 1.f / sum;
            for (int q = 0; q < nc; ++q) del[tid * D + q] = (expf(z[q] - zmax) * inv - (q == y ? 1.f : 0.f)) * P.inv_n;
        } else {
            for (int q = 0; q < nc; ++q) del[tid * D + q] = 0.f;
        }
    }
    // the activations out, while the deltas are under way
    float *ga = P.acts + first * U, *gd = P.dels + first * U;
    for (int t = tid; t < 4 * N.aoff[L]; t += nt) {
        const int s = t / N.aoff[L], i = t - s * N.aoff[L];
        ga[(int64_t)s * U + i] = act[s * U + i];
    }
    for (int l = L; l >= 1; --l) {
        const int nin = N.dims[l - 1], nout = N.dims[l];
        float *cur = del + ((L - l) & 1) * 4 * D, *nxt = del + ((L - l + 1) & 1) * 4 * D;
        TrainChain<false> ch;
        const bool on = l > 1 && wave * 64 < nin;
        if (on) ch.start(P.theta + N.toff[l], nin, nout, wave * 64 + lane);
        train_barrier();
        for (int t = tid; t < 4 * nout; t += nt) {
            const int s = t / nout, j = t - s * nout;
            gd[(int64_t)s * U + N.aoff[l] + j] = cur[s * D + j];
        }
        if (on) {
            // dL/du_{l-1} = (W_l^T dL/du_l) a (1 - a)
            v4f acc = v4f{0.f, 0.f, 0.f, 0.f};
            ch.run(cur + c * D, acc);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (r0 + r < nin) {
                    const float a = act[c * U + N.aoff[l - 1] + r0 + r];
                    nxt[c * D + r0 + r] = acc[r] * a * (1.f - a);
                }
        }
    }
}

constexpr int kTrainStage = 256, kTrainStride = kTrainStage + 4;   // (rows 16 bytes apart: sixteen on 64 banks)

__global__ void __launch_bounds__(256) train_weights_kernel(TrainPassParams P, TrainUpdate A) {
    __shared__ __attribute__((aligned(16))) float ds[16 * kTrainStride], as[16 * kTrainStride];
    const TrainNetDev &N = P.net;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int U = N.units, T = P.group;
    if (blockIdx.x == gridDim.x - 1) {
        // the pass's loss in a fixed order: a lane per 64th group, then the lanes
        if (wave) return;
        double acc = 0.0;
        for (int64_t g = lane; g * T < P.count; g += 64) {
            float v[kTrainMaxGroup], part = 0.f;
#pragma unroll
            for (int z = 0; z < kTrainMaxGroup; ++z) v[z] = P.loss[min(g * T + min(z, T - 1), P.count - 1)];
#pragma unroll
            for (int z = 0; z < kTrainMaxGroup; ++z)
                if (z < T && g * T + z < P.count) part += v[z];
            acc += (double)part;
        }
        for (int s = 32; s > 0; s >>= 1) acc += __shfl_xor(acc, s);
        if (lane == 0) *A.loss_acc += acc;
        return;
    }
    int blk = blockIdx.x, l = 1, ti = 1;
    for (; l <= N.L; ++l) {
        ti = (N.dims[l - 1] + 16) / 16;                       // the inputs and one for the bias
        const int tiles = ((N.dims[l] + 15) / 16) * ti;
        if (blk < tiles) break;
        blk -= tiles;
    }
    const int nin = N.dims[l - 1], nout = N.dims[l];
    const int j0 = blk / ti * 16, i0 = blk % ti * 16;
    // staged by this thread: samples s0, s0 + 16, .. of column q
    const int q = tid & 15, s0 = tid >> 4;
    const float *d = P.dels + N.aoff[l] + min(j0 + q, nout - 1), *a = P.acts + N.aoff[l - 1] + min(i0 + q, nin - 1);
    const bool one = i0 + q == nin;
    // summed by this thread
    const int jr = j0 + (tid >> 4), ic = i0 + (tid & 15);
    const bool mine = jr < nout && ic <= nin;
    const int64_t at = N.toff[l] + (ic < nin ? (int64_t)jr * nin + ic : (int64_t)nout * nin + jr);
    float total = mine && A.grad && A.accumulate ? A.grad[at] : 0.f;
    float th = 0.f, mo = 0.f, ve = 0.f;                       // (read ahead of the sum)
    if (mine && !A.grad) {
        th = A.theta[at];
        mo = A.mom[at];
        ve = A.vel[at];
    }
    const float *dr = ds + (tid >> 4) * kTrainStride, *ar = as + (tid & 15) * kTrainStride;
    const int per = kTrainStage / T * T;
    for (int64_t b = 0; b < P.count; b += per) {
        const int m = (int)min((int64_t)per, P.count - b);
        float dv[16], av[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if (16 * r >= m) break;
            const int64_t s = b + min(s0 + 16 * r, m - 1);
            dv[r] = d[s * U];
            av[r] = a[s * U];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if (16 * r >= m) break;
            const int s = s0 + 16 * r;
            ds[q * kTrainStride + s] = s < m ? dv[r] : 0.f;
            as[q * kTrainStride + s] = s < m ? (one ? 1.f : av[r]) : 0.f;
        }
        __syncthreads();
        float acc = 0.f;
        int in = 0;                                           // samples of the running group
        if (T % 4 == 0) {
#pragma unroll 4
            for (int s = 0; s < m; s += 4) {
                const v4f x = *reinterpret_cast<const v4f *>(dr + s), y = *reinterpret_cast<const v4f *>(ar + s);
#pragma unroll
                for (int z = 0; z < 4; ++z) acc = fmaf(x[z], y[z], acc);
                if ((in += 4) == T) {
                    total += acc;
                    acc = 0.f;
                    in = 0;
                }
            }
        } else {
            for (int s = 0; s < m; ++s) {
                acc = fmaf(dr[s], ar[s], acc);
                if (++in == T) {
                    total += acc;
                    acc = 0.f;
                    in = 0;
                }
            }
        }
        if (in) total += acc;
    }
    if (mine) {
        if (A.grad) {
            A.grad[at] = total;
        } else {
            // (rounded as in prop_adam_kernel, wherever the loads stand)
            const float m = fmaf(1.f - A.b1, total, A.b1 * mo);
            const float v = fmaf(total, (1.f - A.b2) * total, A.b2 * ve);
            A.mom[at] = m;
            A.vel[at] = v;
            A.theta[at] = th - A.lr * (m / A.c1) / (sqrtf(v / A.c2) + A.eps);
        }
    }
}

hipError_t launch_train_pass(const TrainPassParams &P, hipStream_t s) {
    if (P.count <= 0) return hipSuccess;
    const int64_t wgs = (P.count + kTrainTile - 1) / kTrainTile;
    const size_t lds = ((size_t)4 * P.net.units + 8 * P.net.widest) * sizeof(float);
    const int waves = std::max(4, (P.net.widest + 63) / 64);   // a wave per 64 rows
    hipLaunchKernelGGL(train_pass_kernel, dim3((unsigned)wgs), dim3(64 * waves), lds, s, P);
    return hipGetLastError();
}

hipError_t launch_train_weights(const TrainPassParams &P, const TrainUpdate &U, hipStream_t s) {
    if (P.count <= 0) return hipSuccess;
    unsigned blocks = 0;
    for (int l = 1; l <= P.net.L; ++l) blocks += ((P.net.dims[l] + 15) / 16) * ((P.net.dims[l - 1] + 16) / 16);
    hipLaunchKernelGGL(train_weights_kernel, dim3(blocks + 1), dim3(256), 0, s, P, U);   // (and one for the loss)
    return hipGetLastError();
}

}  // namespace ibmc
