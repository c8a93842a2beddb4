// Gather of the folded properties' reduced networks, and the launch side of
// their enumeration.
#include <vector>

#include "kernels_fold.h"
#include "enum_common.h"

namespace ibmc {

// Bytes of a 16-row tile over kw first-layer positions.
static int tile_bytes(int kw) { return kw == 32 ? 512 : fold_blocks(kw) * 1024; }

int fold_stage_bytes(int L, int kw, int npair, int two) {
    const int out = L == 3 ? npair * 512 : tile_bytes(kw);
    return 2 * npair * (tile_bytes(kw) + 64) + out * (two ? 2 : 1) + 64;
}

int64_t fold_lds_bytes(const FoldVariant &v, int stage_max) {
    return stage_max + 4LL * v.wave_bytes + 16;
}

const FoldVariant *fold_variants(int *count) {
    static const std::vector<FoldVariant> all = [] {
        std::vector<FoldVariant> a;
        for (auto f : {fold_variants_l2a, fold_variants_l2b, fold_variants_l2c,
                       fold_variants_l3fa, fold_variants_l3fb, fold_variants_l3fc,
                       fold_variants_l3ga, fold_variants_l3gb, fold_variants_l3gc}) {
            int n = 0;
            const FoldVariant *v = f(&n);
            a.insert(a.end(), v, v + n);
        }
        return a;
    }();
    *count = (int)all.size();
    return all.data();
}

// Position of byte b of lane group g in K-block kb of an A tile over kw
// first-layer positions (-1: none).
__device__ __forceinline__ int fold_kpos(int kw, int kb, int g, int b) {
    const int ub = fold_units_per_block(kw);
    return b < ub ? kb * 4 * ub + g * ub + b : -1;
}

// Block (part, build): writes its share of the build's first-layer columns,
// effective deltas, weight tiles and inits.  Byte gathers from L2-resident
// weights; a few microseconds, bound by latency.
__global__ void __launch_bounds__(256) fold_gather_kernel(const QNetDev *nets, const FoldBuild *builds, int parts,
                                                          const PropDev *props, const int32_t *u0_store,
                                                          int64_t u0_stride, FoldRun *runs) {
    __shared__ int l1[kFoldMaxWidth], l2[kMaxWidth];
    const FoldBuild &B = builds[blockIdx.y];
    const QNetDev &net = nets[B.net];
    const PropDev &pr = props[B.pid];
    const FoldRun R = B.run;
    const int KW = B.kw, L = net.L, H1 = net.H[1], n = net.dims[0], m = pr.m;
    const FoldWs ws = fold_ws(H1, L == 3 ? net.H[2] : 0);
    for (int t = threadIdx.x; t < KW; t += 256) l1[t] = t < B.live1 ? B.ws[ws.list1 + t] : -1;
    if (L == 3)
        for (int t = threadIdx.x; t < R.npair * 32; t += 256) l2[t] = t < B.live2 ? B.ws[ws.list2 + t] : -1;
    __syncthreads();
    const int nt = parts * 256, t0 = blockIdx.x * 256 + threadIdx.x;
    // first-layer columns, four units per step
    int2 *W1 = reinterpret_cast<int2 *>(const_cast<int16_t *>(R.W1));
    const int q4 = KW / 4;
    for (int t = t0; t < n * q4; t += nt) {
        const int p = t / q4, u = (t % q4) * 4;
        int v[4];
#pragma unroll
        for (int z = 0; z < 4; ++z) v[z] = l1[u + z] >= 0 ? (int)net.W1T[(int64_t)p * H1 + l1[u + z]] * B.f : 0;
        W1[t] = make_int2((v[0] & 0xffff) | (v[1] << 16), (v[2] & 0xffff) | (v[3] << 16));
    }
    int16_t *et = const_cast<int16_t *>(R.etab);
    for (int t = t0; t < n * m; t += nt) {
        const int p = t / m, xv = pr.image[p];
        et[t] = (int16_t)(clamp_pixel(xv + pr.deltas[t - p * m]) - xv);
    }
    const int32_t *u0s = u0_store + (int64_t)B.pid * u0_stride;
    int32_t *v0 = const_cast<int32_t *>(R.v0);
    for (int t = t0; t < KW; t += nt) v0[t] = l1[t] >= 0 ? u0s[l1[t]] * B.f - (1 << (14 - R.halvings)) : -(1 << (14 - R.halvings));
    // later layers: dwords of the staged block
    int *stage = reinterpret_cast<int *>(const_cast<int8_t *>(R.stage));
    const int kbs = fold_blocks(KW), tdw = KW == 32 ? 128 : 256;      // K-blocks and dwords per tile
    const int per = KW == 32 ? 2 : 4;                                        // dwords per lane and tile
    const int o_b2 = 2 * R.npair * kbs * tdw, o_wo = o_b2 + R.npair * 32;
    const int out = L == 3 ? R.npair * 128 : kbs * tdw, o_y = o_wo + out, o_bo = R.two ? o_y + out : o_y;
    const int h1 = net.dims[1];
    for (int t = t0; t < o_b2; t += nt) {
        const int tile = t / (kbs * tdw), r = t % (kbs * tdw), kb = r / tdw, ln = (r % tdw) / per, d = r % per;
        const int row = l2[tile * 16 + (ln & 15)];
        unsigned v = 0;
#pragma unroll
        for (int z = 0; z < 4; ++z) {
            const int kp = fold_kpos(KW, kb, ln >> 4, d * 4 + z), q = kp >= 0 ? l1[kp] : -1;
            const int wv = (row >= 0 && q >= 0) ? (int)net.Wd[2][(int64_t)row * h1 + sigma64(q)] : 0;
            v |= (unsigned)(uint8_t)wv << (8 * z);
        }
        stage[t] = (int)v;
    }
    // layer-2 init: inputs 2 (a1 - 64); the saturating epilogue takes
    // 2 u2 - 32768 (2 u2 for the units of uncapped pairs that stay above 0),
    // the general one 2 (u2 - 64 * 2^s2)
    for (int t = t0; t < R.npair * 32; t += nt) {
        const int row = l2[t];
        int v = 0;
        if (row >= 0) {
            const bool upper = t / 32 < R.free_pairs && (B.ws[ws.iv2 + row] >> 16) == FOLD_UPPER;
            v = 2 * (B.ws[ws.b2 + row] + 64 * B.ws[ws.rs2 + row]) - (!B.epi ? 128 << net.shift[1] : upper ? 0 : 32768);
        }
        stage[o_b2 + t] = v;
    }
    // output layer: rows W_c - W_label in one or two bytes
    const int hl = net.dims[L - 1], lab = R.label;
    for (int t = t0; t < out; t += nt) {
        // three layers: a 32-wide block per pair of layer-2 tiles, whose byte
        // 4 d + z of lane group g is row 16 d + 4 g + z of the pair
        const int pl = L == 3 ? 2 : per;
        const int td = L == 3 ? 128 : tdw;
        const int kb = t / td, ln = (t % td) / pl, d = t % pl, c = ln & 15;
        unsigned x = 0, y = 0;
#pragma unroll
        for (int z = 0; z < 4; ++z) {
            int unit = -1;
            if (L == 3) {
                unit = l2[kb * 32 + 16 * d + 4 * (ln >> 4) + z];
            } else {
                const int kp = fold_kpos(KW, kb, ln >> 4, d * 4 + z), q = kp >= 0 ? l1[kp] : -1;
                unit = q >= 0 ? sigma64(q) : -1;
            }
            if (unit >= 0 && c < R.nc && c != lab) {
                const int df = (int)net.Wd[L][(int64_t)c * hl + unit] - (int)net.Wd[L][(int64_t)lab * hl + unit];
                const int a = min(max(df, -128), 127);
                x |= (unsigned)(uint8_t)a << (8 * z);
                y |= (unsigned)(uint8_t)(df - a) << (8 * z);
            }
        }
        stage[o_wo + t] = (int)x;
        if (R.two) stage[o_y + t] = (int)y;
    }
    // output init: z_c - z_label + [c < label], doubled for two-layer nets
    // (whose inputs are 2 (a - 64))
    for (int c = t0; c < 16; c += nt) {
        int v = -(1 << 30);
        if (c < R.nc && c != lab) {
            const int db = B.ws[ws.bo + c] - B.ws[ws.bo + lab], dr = B.ws[ws.rso + c] - B.ws[ws.rso + lab];
            v = db + dr + (c < lab ? 1 : 0);
            if (L == 2) v *= 2;
        }
        stage[o_bo + c] = v;
    }
    if (t0 == 0) runs[B.pid] = R;
}

hipError_t launch_fold_gather(const QNetDev *nets, const FoldBuild *builds, int n, int parts, const PropDev *props,
                              const int32_t *u0_store, int64_t u0_stride, FoldRun *runs, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fold_gather_kernel, dim3(parts, n), dim3(256), 0, s, nets, builds, parts, props, u0_store,
                       u0_stride, runs);
    return hipGetLastError();
}

hipError_t launch_enum_fold(const FoldVariant &v, int grid, const FoldParams &P, hipStream_t s) {
    if (grid < 1) return hipErrorInvalidValue;
    void *args[] = {const_cast<FoldParams *>(&P)};
    return hipLaunchKernel(v.fn, dim3(grid), dim3(256), args, (size_t)fold_lds_bytes(v, P.stage_max), s);
}

}  // namespace ibmc
