// Tree-masked attention without matrix cores: one wavefront per (sequence, node, query
// head). The on-device cross-check of the bf16 matrix-core kernels (VS_IMPL_GENERIC).
// Math: paper Eq. 1 with a softmax scale, restricted to the keys a node may see
// (all prefix tokens + the tree slots of its ancestor-or-self set, Section 3.1).
#include "vs_device.h"

namespace vs {

// grid = (T, Hq, B), block = 64. Lane j scores key j0 + j of each 64-key chunk; for the
// value product lane c owns channels c, c + 64, ...
template <int D>
__global__ __launch_bounds__(kWave) void attn_generic_kernel(const AttnParams p) {
    constexpr int CPL = D / kWave; // channels per lane
    __shared__ int32_t sp[VS_MAX_TREE];
    __shared__ int32_t sflag;
    __shared__ float sq[D];
    __shared__ float spj[kWave];
    __shared__ int64_t soff[kWave];

    const int node = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
    const int lane = threadIdx.x;
    const int kvh = h / p.group;

    int32_t tree_code = VS_STATUS_OK;
    if (p.tree_keys == 0) {
        if (lane == 0) sflag = 0;
        __syncthreads();
    } else {
        tree_code = load_tree(p.parent + (int64_t)b * p.T, p.T, sp, &sflag);
    }
    const int32_t S = p.prefix_len[b];
    const bool s_ok = prefix_ok(p, S);
    if (node == 0 && h == 0) report_status(p, b, tree_code, s_ok, S, &sflag);
    if (tree_code != VS_STATUS_OK || !s_ok) return;

    const uint64_t mask = p.tree_keys == 0 ? 0ull : (p.tree_mask ? p.tree_mask[(int64_t)b * p.T + node] : ancestor_mask(sp, node));
    const uint16_t* q = (const uint16_t*)p.q + (((int64_t)b * p.T + node) * p.Hq + h) * D;
    for (int c = lane; c < D; c += kWave) sq[c] = bf16_bits_to_float(q[c]);
    __syncthreads();

    const uint16_t* kbase = (const uint16_t*)p.k;
    const uint16_t* vbase = (const uint16_t*)p.v;
    const int n = S + p.tree_keys;
    float m = -INFINITY, l = 0.f;
    float acc[CPL];
#pragma unroll
    for (int i = 0; i < CPL; ++i) acc[i] = 0.f;

    for (int j0 = 0; j0 < n; j0 += kWave) {
        const int j = j0 + lane;
        bool vis = false;
        int64_t off = 0;
        float s = -INFINITY;
        if (j < n) {
            vis = (j < S) || ((mask >> (j - S)) & 1ull);
            if (vis) {
                off = token_offset(p, b, kvh, j);
                const uint16_t* kr = kbase + off;
                float dot = 0.f;
#pragma unroll 8
                for (int c = 0; c < D; ++c) dot = fmaf(sq[c], bf16_bits_to_float(kr[c]), dot);
                s = dot * p.scale;
            }
        }
        const float cm = wave_max(s);
        const float m_new = fmaxf(m, cm);
        float pj = 0.f, alpha = 1.f;
        if (m_new > -INFINITY) {
            pj = vis ? expf(s - m_new) : 0.f;
            alpha = expf(m - m_new); // m = -inf → 0
        }
        l = l * alpha + wave_sum(pj);
        m = m_new;
#pragma unroll
        for (int i = 0; i < CPL; ++i) acc[i] *= alpha;
        __syncthreads();
        spj[lane] = pj;
        soff[lane] = off;
        __syncthreads();
        const int cnt = min(kWave, n - j0);
        for (int jj = 0; jj < cnt; ++jj) {
            const float w = spj[jj];
            if (w != 0.f) { // invisible keys are skipped, never multiplied
                const uint16_t* vr = vbase + soff[jj];
#pragma unroll
                for (int i = 0; i < CPL; ++i) acc[i] = fmaf(w, bf16_bits_to_float(vr[lane + i * kWave]), acc[i]);
            }
        }
    }
    uint16_t* o = (uint16_t*)p.out + (((int64_t)b * p.T + node) * p.Hq + h) * D;
    const float inv = 1.f / l;
#pragma unroll
    for (int i = 0; i < CPL; ++i) o[lane + i * kWave] = float_to_bf16_bits(acc[i] * inv);
}

hipError_t launch_attention_generic(const AttnParams& p, hipStream_t s) {
    dim3 grid(p.T, p.Hq, p.B), block(kWave);
    if (p.d == 64) hipLaunchKernelGGL((attn_generic_kernel<64>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((attn_generic_kernel<128>), grid, block, 0, s, p);
    return hipGetLastError();
}

} // namespace vs
