// Gather of the folded properties' reduced networks, and the launch side of
// their enumeration.
#include <vector>

#include "kernels_fold.h"
#include "enum_common.h"

namespace ibmc {

static int out_tile_bytes(int L, int kw) { return L == 3 ? 1024 : kw == 32 ? 512 : kw / 64 * 1024; }

int fold_stage_bytes(int L, int kw, int mt2, int two) {
    const int kbo = L == 3 ? (mt2 + 3) / 4 : 1;
    const int t2 = kw == 32 ? 512 : kw / 64 * 1024;
    return mt2 * t2 + mt2 * 64 + kbo * out_tile_bytes(L, kw) * (two ? 2 : 1) + 64;
}

int64_t fold_lds_bytes(const FoldVariant &v, int stage_max) {
    return stage_max + 4LL * (kFoldGroup * v.kw * 2 + kFoldGroup * 8) + 16;
}

const FoldVariant *fold_variants(int *count) {
    static const std::vector<FoldVariant> all = [] {
        std::vector<FoldVariant> a;
        for (auto f : {fold_variants_l2, fold_variants_l3f, fold_variants_l3g}) {
            int n = 0;
            const FoldVariant *v = f(&n);
            a.insert(a.end(), v, v + n);
        }
        return a;
    }();
    *count = (int)all.size();
    return all.data();
}

// Position of byte b of lane group g in K-block kb of an A tile over KW
// first-layer positions.
__device__ __forceinline__ int fold_kpos(int kw, int kb, int g, int b) { return kw == 32 ? g * 8 + b : kb * 64 + g * 16 + b; }

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
        for (int t = threadIdx.x; t < R.mt2 * 16; t += 256) l2[t] = t < B.live2 ? B.ws[ws.list2 + t] : -1;
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
    const int kbs = KW == 32 ? 1 : KW / 64, tdw = KW == 32 ? 128 : 256;      // K-blocks and dwords per tile
    const int per = KW == 32 ? 2 : 4;                                        // dwords per lane and tile
    const int o_b2 = R.mt2 * kbs * tdw, o_wo = o_b2 + R.mt2 * 16;
    const int otd = L == 3 ? 256 : kbs * tdw, o_y = o_wo + R.kbo * otd, o_bo = R.two ? o_y + R.kbo * otd : o_y;
    const int h1 = net.dims[1];
    for (int t = t0; t < o_b2; t += nt) {
        const int tile = t / (kbs * tdw), r = t % (kbs * tdw), kb = r / tdw, ln = (r % tdw) / per, d = r % per;
        const int row = l2[tile * 16 + (ln & 15)];
        unsigned v = 0;
#pragma unroll
        for (int z = 0; z < 4; ++z) {
            const int q = l1[fold_kpos(KW, kb, ln >> 4, d * 4 + z)];
            const int wv = (row >= 0 && q >= 0) ? (int)net.Wd[2][(int64_t)row * h1 + sigma64(q)] : 0;
            v |= (unsigned)(uint8_t)wv << (8 * z);
        }
        stage[t] = (int)v;
    }
    // layer-2 init: inputs 2 (a1 - 64); the saturating epilogue takes
    // 2 u2 - 32768, the general one 2 (u2 - 64 * 2^s2)
    for (int t = t0; t < R.mt2 * 16; t += nt) {
        const int row = l2[t];
        int v = 0;
        if (row >= 0)
            v = 2 * (B.ws[ws.b2 + row] + 64 * B.ws[ws.rs2 + row]) - (B.epi ? 32768 : 128 << net.shift[1]);
        stage[o_b2 + t] = v;
    }
    // output layer: rows W_c - W_label in one or two bytes
    const int hl = net.dims[L - 1], lab = R.label;
    for (int t = t0; t < R.kbo * otd; t += nt) {
        const int pl = L == 3 ? 4 : per;
        const int td = L == 3 ? 256 : tdw;
        const int kb = t / td, ln = (t % td) / pl, d = t % pl, c = ln & 15;
        unsigned x = 0, y = 0;
#pragma unroll
        for (int z = 0; z < 4; ++z) {
            int unit = -1;
            if (L == 3) {
                const int r = kb * 64 + sigma64(16 * (ln >> 4) + 4 * d + z);
                unit = r < R.mt2 * 16 ? l2[r] : -1;
            } else {
                const int q = l1[fold_kpos(KW, kb, ln >> 4, d * 4 + z)];
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
    // output init: z_c - z_label + [c < label], doubled for two-layer nets;
    // inputs are 2 (a - 64), a - 128 (saturating epilogue) or a - 64
    for (int c = t0; c < 16; c += nt) {
        int v = -(1 << 30);
        if (c < R.nc && c != lab) {
            const int db = B.ws[ws.bo + c] - B.ws[ws.bo + lab], dr = B.ws[ws.rso + c] - B.ws[ws.rso + lab];
            const int off = L == 3 && B.epi ? 128 : 64;
            v = db + off * dr + (c < lab ? 1 : 0);
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
