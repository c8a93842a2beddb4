// Training kernels of the float (sigmoid) networks, two launches per step.
//
// The pass: a workgroup of sixteen waves takes four samples through the
// forward pass (a_0 = x / 256, sigmoid hidden layers, linear logits, Eq. (2)),
// the softmax cross-entropy against the label and the deltas of the backward
// pass.  Every layer product runs on the FP32 matrix instruction of sixteen
// 4 x 4 blocks, whose blocks are sixteen groups of four rows and whose columns
// are the four samples: a wave covers 64 rows, and the waves beyond the rows
// split the inputs, their partial sums added in LDS.  Four samples a
// workgroup, because a batch of 256 then spreads over 64 compute units where
// tiles of sixteen would leave it on sixteen; what remains is latency (one
// weight round trip and two barriers per layer and direction).
//
// The weights: a workgroup per 16 x 16 tile of a layer's gradient
// sum_s delta_s a_s^T (the bias as one more input that is 1), the samples
// split over its four waves, on 16 x 16 x 4 FP32 matrix instructions with the
// running sums added every 64 samples; the tile's Adam step follows in place,
// so no gradient goes through memory.
//
// Fixed summation order, no atomics: a training run is the same on every call.
// Measured, 35-256-128-10 at batch 256, per step: pass 19 us, weights 5 us (a
// tile of eight samples per workgroup on the vector ALU with partial
// gradients, their sum and the Adam step as launches of their own: 88 + 10 +
// 5 us); an epoch of 20,000 samples 8.4 -> 2.4 ms.  Bound by latency: the
// products' operations take about 1 us.  Its error against FP64 after an
// epoch is 3.8e-7 (4.2e-7 before).
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

constexpr int kTrainWaves = kTrainThreads / 64;

// Row blocks of 64 and input splits of one layer product over the waves.
struct TrainSplit {
    int rb, sp, kper;
};
__device__ __forceinline__ TrainSplit train_split(int rows, int k) {
    TrainSplit s;
    s.rb = (rows + 63) / 64;
    s.sp = max(1, min(kTrainWaves / s.rb, (k + 15) / 16));
    s.kper = ((k + s.sp - 1) / s.sp + 3) & ~3;
    return s;
}

// Partial products of one layer for the four samples: part[split][row][sample]
// = sum over the split's inputs k of M[row][k] in[sample][k].  ROWS: M is W
// (row-major, a row per lane); else M is W transposed (W[k][row]).  in: LDS
// rows of `stride` floats, zero from K to its next multiple of four.
template <bool ROWS>
__device__ __forceinline__ void train_product(const float *W, int R, int K, const float *in, int stride, float *part) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = lane & 3;
    const TrainSplit S = train_split(R, K);
    if (wave >= S.rb * S.sp) return;
    const int rb = wave % S.rb, sp = wave / S.rb;
    const int k0 = sp * S.kper, k1 = min(K, k0 + S.kper);
    const int row = min(rb * 64 + lane, R - 1);
    const float *x = in + c * stride;
    v4f acc = v4f{0.f, 0.f, 0.f, 0.f};
    int k = k0;
    auto load = [&](int at) __attribute__((always_inline)) -> v4f {
        if constexpr (ROWS) {
            return *reinterpret_cast<const v4f_u *>(W + (int64_t)row * K + at);
        } else {
            v4f a;
#pragma unroll
            for (int z = 0; z < 4; ++z) a[z] = W[(int64_t)(at + z) * R + row];
            return a;
        }
    };
    auto step = [&](const v4f &a, int at) __attribute__((always_inline)) {
        const v4f b = *reinterpret_cast<const v4f *>(x + at);
#pragma unroll
        for (int z = 0; z < 4; ++z) acc = __builtin_amdgcn_mfma_f32_4x4x1f32(a[z], b[z], acc, 0, 0, 0);
    };
    // sixteen inputs' weights in flight together
    for (; k + 16 <= k1; k += 16) {
        v4f a[4];
#pragma unroll
        for (int h = 0; h < 4; ++h) a[h] = load(k + 4 * h);
#pragma unroll
        for (int h = 0; h < 4; ++h) step(a[h], k + 4 * h);
    }
    for (; k + 4 <= k1; k += 4) step(load(k), k);
    for (; k < k1; ++k) {
        const float a = ROWS ? W[(int64_t)row * K + k] : W[(int64_t)k * R + row];
        acc = __builtin_amdgcn_mfma_f32_4x4x1f32(a, x[k], acc, 0, 0, 0);
    }
    // lane 4 b + c, register r: row 4 b + r, sample c
    float *out = part + (size_t)(sp * S.rb + rb) * 256 + (lane & ~3) * 4 + c;
#pragma unroll
    for (int r = 0; r < 4; ++r) out[4 * r] = acc[r];
}

// Sum over the splits of row / sample t (= 4 row + sample).
__device__ __forceinline__ float train_sum(const float *part, const TrainSplit &S, int t) {
    float v = 0.f;
    for (int sp = 0; sp < S.sp; ++sp) v += part[(size_t)sp * S.rb * 256 + t];
    return v;
}

__global__ void __launch_bounds__(kTrainThreads) train_pass_kernel(TrainPassParams P) {
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const TrainNetDev &N = P.net;
    const int tid = threadIdx.x, L = N.L, n = N.dims[0], U = N.units;
    const int64_t first = (int64_t)blockIdx.x * kTrainTile;
    const int S = (int)min((int64_t)kTrainTile, P.count - first);
    float *act = lds;                               // [4][U]
    float *del = act + 4 * U;                       // [2][4][widest]: this layer's deltas and the next
    float *part = del + 8 * N.widest;               // [16][256]
    float *loss = part + kTrainWaves * 256;         // [4]
    // zeros in the padding and the missing samples
    for (int t = tid; t < 4 * U + 8 * N.widest; t += kTrainThreads) lds[t] = 0.f;
    __syncthreads();
    for (int t = tid; t < S * n; t += kTrainThreads) {
        const int s = t / n, i = t - s * n;
        const int64_t e = P.e0 + first + s;
        const int64_t img = P.order ? P.order[e] : e;
        act[s * U + i] = (float)P.images[img * n + i] * (1.f / 256.f);
    }
    __syncthreads();
    for (int l = 1; l <= L; ++l) {
        const int nin = N.dims[l - 1], nout = N.dims[l];
        const float *W = P.theta + N.toff[l], *b = W + (int64_t)nout * nin;
        train_product<true>(W, nout, nin, act + N.aoff[l - 1], U, part);
        __syncthreads();
        const TrainSplit sp = train_split(nout, nin);
        for (int t = tid; t < 4 * nout; t += kTrainThreads) {
            const int j = t >> 2, s = t & 3;
            const float u = b[j] + train_sum(part, sp, t);
            act[s * U + N.aoff[l] + j] = (l < L) ? 1.f / (1.f + expf(-u)) : u;
        }
        __syncthreads();
    }
    // softmax cross-entropy of each sample's logits; dL/du of the logits
    const int nc = N.dims[L], D = N.widest;
    if (tid < 4) {
        loss[tid] = 0.f;
        if (tid < S) {
            const int64_t e = P.e0 + first + tid;
            const int y = P.labels[P.order ? P.order[e] : e];
            const float *z = act + tid * U + N.aoff[L];
            float zmax = z[0];
            for (int c = 1; c < nc; ++c) zmax = fmaxf(zmax, z[c]);
            float sum = 0.f;
            for (int c = 0; c < nc; ++c) sum += expf(z[c] - zmax);
            loss[tid] = logf(sum) - (z[y] - zmax);
            const float inv = 1.f / sum;
            for (int c = 0; c < nc; ++c) del[tid * D + c] = (expf(z[c] - zmax) * inv - (c == y ? 1.f : 0.f)) * P.inv_n;
        }
    }
    // the activations out, while the deltas are under way
    float *ga = P.acts + first * U, *gd = P.dels + first * U;
    for (int t = tid; t < 4 * N.aoff[L]; t += kTrainThreads) {
        const int s = t / N.aoff[L], i = t - s * N.aoff[L];
        ga[(int64_t)s * U + i] = act[s * U + i];
    }
    __syncthreads();
    for (int l = L; l >= 1; --l) {
        const int nin = N.dims[l - 1], nout = N.dims[l];
        float *cur = del + ((L - l) & 1) * 4 * D, *nxt = del + ((L - l + 1) & 1) * 4 * D;
        for (int t = tid; t < 4 * nout; t += kTrainThreads) {
            const int s = t / nout, j = t - s * nout;
            gd[(int64_t)s * U + N.aoff[l] + j] = cur[s * D + j];
        }
        if (l == 1) break;
        // dL/du_{l-1} = (W_l^T dL/du_l) a (1 - a)
        train_product<false>(P.theta + N.toff[l], nin, nout, cur, D, part);
        __syncthreads();
        const TrainSplit sp = train_split(nin, nout);
        const int pad = (nin + 3) & ~3;
        for (int t = tid; t < 4 * pad; t += kTrainThreads) {
            const int i = t >> 2, s = t & 3;
            const float a = act[s * U + N.aoff[l - 1] + i];
            nxt[s * D + i] = i < nin ? train_sum(part, sp, t) * a * (1.f - a) : 0.f;
        }
        __syncthreads();
    }
    if (tid == 0) P.loss[blockIdx.x] = ((loss[0] + loss[1]) + loss[2]) + loss[3];
}

__global__ void __launch_bounds__(256) train_weights_kernel(TrainPassParams P, TrainUpdate A) {
    __shared__ float sum[4][256];
    const TrainNetDev &N = P.net;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, j16 = lane & 15, g = lane >> 4;
    const int U = N.units;
    int blk = blockIdx.x, l = 1, ti = 1;
    for (; l <= N.L; ++l) {
        ti = (N.dims[l - 1] + 16) / 16;                       // the inputs and one for the bias
        const int tiles = ((N.dims[l] + 15) / 16) * ti;
        if (blk < tiles) break;
        blk -= tiles;
    }
    const int nin = N.dims[l - 1], nout = N.dims[l];
    const int j0 = blk / ti * 16, i0 = blk % ti * 16;
    const int j = j0 + j16, i = i0 + j16;
    const float *d = P.dels + N.aoff[l] + min(j, nout - 1), *a = P.acts + N.aoff[l - 1] + min(i, nin - 1);
    const bool on = j < nout, in = i < nin, one = i == nin;
    // rows of four samples, a contiguous quarter of them per wave
    const int64_t rows = (P.count + 3) / 4, per = (rows + 3) / 4;
    const int64_t q0 = wave * per, q1 = min(rows, q0 + per);
    v4f total = v4f{0.f, 0.f, 0.f, 0.f};
    for (int64_t q = q0; q < q1; q += 16) {
        v4f acc = v4f{0.f, 0.f, 0.f, 0.f};
        const int m = (int)min((int64_t)16, q1 - q);
        float dv[16], av[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int64_t s = (q + (r < m ? r : 0)) * 4 + g;
            dv[r] = d[s * U];
            av[r] = a[s * U];
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float x = r < m && on ? dv[r] : 0.f, y = in ? av[r] : one ? 1.f : 0.f;
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x, y, acc, 0, 0, 0);
        }
        total += acc;
    }
    // lane (c, g), register z: row 4 g + z, column c of the tile
#pragma unroll
    for (int z = 0; z < 4; ++z) sum[wave][(4 * g + z) * 16 + j16] = total[z];
    __syncthreads();
    const int jr = j0 + (tid >> 4), ic = i0 + (tid & 15);
    if (jr < nout && ic <= nin) {
        const float gr = ((sum[0][tid] + sum[1][tid]) + sum[2][tid]) + sum[3][tid];
        const int64_t at = N.toff[l] + (ic < nin ? (int64_t)jr * nin + ic : (int64_t)nout * nin + jr);
        if (A.grad) {
            A.grad[at] = (A.accumulate ? A.grad[at] : 0.f) + gr;
        } else {
            const float m = A.b1 * A.mom[at] + (1.f - A.b1) * gr;
            const float v = A.b2 * A.vel[at] + (1.f - A.b2) * gr * gr;
            A.mom[at] = m;
            A.vel[at] = v;
            A.theta[at] -= A.lr * (m / A.c1) / (sqrtf(v / A.c2) + A.eps);
        }
    }
    if (blockIdx.x == 0 && wave == 0) {
        // the pass's loss in a fixed order: a lane per 64th workgroup, then the lanes
        double acc = 0.0;
        for (int64_t t = lane; t < rows; t += 64) acc += (double)P.loss[t];
        for (int s = 32; s > 0; s >>= 1) acc += __shfl_xor(acc, s);
        if (lane == 0) *A.loss_acc += acc;
    }
}

hipError_t launch_train_pass(const TrainPassParams &P, hipStream_t s) {
    if (P.count <= 0) return hipSuccess;
    const int64_t wgs = (P.count + kTrainTile - 1) / kTrainTile;
    const size_t lds = ((size_t)4 * P.net.units + 8 * P.net.widest + kTrainWaves * 256 + 4) * sizeof(float);
    hipLaunchKernelGGL(train_pass_kernel, dim3((unsigned)wgs), dim3(kTrainThreads), lds, s, P);
    return hipGetLastError();
}

hipError_t launch_train_weights(const TrainPassParams &P, const TrainUpdate &U, hipStream_t s) {
    if (P.count <= 0) return hipSuccess;
    unsigned blocks = 0;
    for (int l = 1; l <= P.net.L; ++l) blocks += ((P.net.dims[l] + 15) / 16) * ((P.net.dims[l - 1] + 16) / 16);
    hipLaunchKernelGGL(train_weights_kernel, dim3(blocks), dim3(256), 0, s, P, U);
    return hipGetLastError();
}

}  // namespace ibmc
