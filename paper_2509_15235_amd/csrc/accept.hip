// Greedy acceptance over a draft tree (paper Section 3.1 at temperature 0): a draft token
// survives iff it equals the target's argmax at its parent; the deepest surviving node
// ends the accepted path and its own argmax is the bonus token.
//
// Two kernels (one for few logits, below): (1) a bandwidth-bound scan that reduces every chunk of a logits row to (max, first index), (2) one workgroup
// per sequence that finishes the row argmax and walks the tree.
#include <atomic>

#include "logits_scan.h"

// Scratch of vs_tree_accept_noalloc: the per-(row, chunk) results that vs_tree_accept keeps in the
// caller's workspace. One copy per GPU, held until the process ends. In host code the array's
// name is only a handle for hipGetSymbolAddress: the device address is asked for once per device
// and everything that touches the memory uses that address.
constexpr size_t kNoallocScratchBytes = VS_ACCEPT_NOALLOC_MAX_BYTES;
static __device__ __align__(256) unsigned char scratch[kNoallocScratchBytes];

namespace vs {

namespace {

struct Best {
    float v;
    int32_t i;
};

// Candidate (v, i) replaces the incumbent iff it is larger, or equal with a lower index.
// NaN candidates never win ('>' and '==' are false for NaN).
__device__ __forceinline__ void take(Best& b, float v, int32_t i) {
    if (v > b.v || (v == b.v && i < b.i)) {
        b.v = v;
        b.i = i;
    }
}

constexpr int kRowThreads = kScanThreads / VS_MAX_TREE; // threads of the walk that share a row's chunks
static_assert(kRowThreads == 8, "three steps of a butterfly");

// (max, first index) of the part of a chunk that a wave holds, in every lane. The maximum is found on values alone (one v_max
// per element); the index is recovered afterwards as the lowest position that equals the wave's maximum. NaN never equals
// anything and never survives fmaxf, -0 == +0.
template <int THREADS>
__device__ __forceinline__ Best chunk_best(const ScanChunk& c, int chunk, int tid) {
    float m = c.tail;
#pragma unroll
    for (int j = 0; j < kScanVec; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) m = fmaxf(m, c.a[j][e]);
    m = wave_max(m);
    int32_t idx = (c.tail_at != INT32_MAX && c.tail == m) ? c.tail_at : INT32_MAX;
#pragma unroll
    for (int j = kScanVec - 1; j >= 0; --j) {
        const int k = tid + j * THREADS;
#pragma unroll
        for (int e = 3; e >= 0; --e)
            if (k < c.nvec && c.a[j][e] == m) idx = c.begin + 4 * k + e;
    }
    // a left-to-right '>' scan never displaces a NaN in column 0
    const float first = c.nvec > 0 ? c.a[0][0] : c.tail;
    if (__any(chunk == 0 && tid == 0 && first != first)) return {INFINITY, 0};
    return {m, wave_min(idx)}; // lanes without the wave's maximum have INT32_MAX
}
__device__ __forceinline__ uint64_t pair_of(Best b) { return ((uint64_t)(uint32_t)b.i << 32) | __float_as_uint(b.v); }

// grid = B*T*chunks, block = THREADS.
template <int THREADS>
__global__ __launch_bounds__(THREADS, 8) void argmax_partial_kernel(const AcceptParams p) {
    __shared__ float sv[THREADS / kWave];
    __shared__ int32_t si[THREADS / kWave];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const ScanItem it = scan_item(p.by_chunks);
    const ScanChunk c = scan_load<THREADS>(p.logits + (int64_t)it.row * p.ld, it.chunk, p.V);
    Best best = chunk_best<THREADS>(c, it.chunk, tid);
    if (lane == 0) {
        sv[wave] = best.v;
        si[wave] = best.i;
    }
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int w = 1; w < THREADS / kWave; ++w) take(best, sv[w], si[w]);
        p.pairs[(int64_t)it.row * p.chunks + it.chunk] = pair_of(best);
    }
}

// The walk over sequence b's tree, `pairs` its rows' (all threads of a workgroup of 512 or more). Eight threads share a row's chunks,
// four pairs each in flight; the first wave holds the tree, a lane per node: asked for by `tree` behind the first pairs.
template <typename Tree>
__device__ __forceinline__ void accept_walk(const AcceptParams& p, int b, const uint64_t* pairs, Tree tree, int32_t* samax) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int T = p.T, i = tid / kRowThreads, sub = tid % kRowThreads;
    int32_t parent = -2, draft = -1;
    {
        constexpr int kPre = 4;
        pairs += (int64_t)min(i, T - 1) * p.chunks;
        uint64_t w[kPre];
        auto fetch = [&](int c0) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < kPre; ++q) w[q] = pairs[min(c0 + kRowThreads * q, p.chunks - 1)]; // (the last one again: no harm)
        };
        fetch(sub);
        tree(parent, draft);
        Best best = {-INFINITY, INT32_MAX};
        for (int c0 = sub; c0 < p.chunks; c0 += kRowThreads * kPre) {
            if (c0 != sub) fetch(c0);
#pragma unroll
            for (int q = 0; q < kPre; ++q) take(best, __uint_as_float((uint32_t)w[q]), (int32_t)(w[q] >> 32));
        }
        take(best, __uint_as_float(dpp<kDppXor1>(__float_as_uint(best.v))), (int32_t)dpp<kDppXor1>(best.i));
        take(best, __uint_as_float(dpp<kDppXor2>(__float_as_uint(best.v))), (int32_t)dpp<kDppXor2>(best.i));
        take(best, __uint_as_float(dpp<kDppXor7>(dpp<kDppXor3>(__float_as_uint(best.v)))), (int32_t)dpp<kDppXor7>(dpp<kDppXor3>(best.i)));
        if (i < T && sub == 0) {
            const int32_t idx = best.i == INT32_MAX ? 0 : best.i; // nothing above -inf: index 0
            samax[i] = idx;
            if (p.row_argmax) p.row_argmax[(int64_t)b * T + i] = idx;
        }
    }
    __syncthreads();
    if (tid >= kWave) return;
    const int32_t code = tree_check(parent, T);
    int node = 0, alen = 0;
    if (code == VS_STATUS_OK) {
        // level by level: a node is accepted iff its token is its parent's argmax and its parent is accepted. The deepest
        // accepted node ends the path, the lowest of several.
        const bool match = lane > 0 && lane < T && draft == samax[parent < 0 ? 0 : parent];
        uint64_t level = 1;
        for (;;) {
            level = __ballot(match && ((level >> (parent & 63)) & 1));
            if (level == 0) break;
            node = __builtin_ctzll(level);
            ++alen;
        }
    }
    const int32_t path = code == VS_STATUS_OK ? tree_path(parent, node, alen) : -1;
    if (lane < T) p.path[(int64_t)b * T + lane] = path;
    if (lane == 0) {
        if (p.status) p.status[b] = code;
        p.accepted_len[b] = alen;
        p.bonus[b] = code == VS_STATUS_OK ? samax[node] : -1;
    }
}

// grid = B, block = 512.
__global__ __launch_bounds__(kScanThreads) void accept_walk_kernel(const AcceptParams p) {
    __shared__ int32_t samax[VS_MAX_TREE];
    const int b = blockIdx.x;
    accept_walk(p, b, p.pairs + (int64_t)b * p.T * p.chunks, [&](int32_t& parent, int32_t& draft) __attribute__((always_inline)) {
        if (threadIdx.x >= kWave) return;
        parent = tree_lane(p.parent + (int64_t)b * p.T, p.T);
        draft = p.draft[(int64_t)b * p.T + min((int)threadIdx.x, p.T - 1)];
    }, samax);
}

// Both in one for few logits: a workgroup of sixteen waves per sequence scans all of its rows, a piece of 1024 logits a wave, and
// walks the tree. Bound by one trip to memory; the second launch and the trip for the pairs are gone (us, two kernels /
// one: 1 x 8 x 1000 5.7 / 4.3, 16 x 16 x 1024 6.7 / 5.5, 16 x 4 x 4000 7.0 / 5.4). With two pieces a wave it is no better (16 x 4 x 8000
// 7.1 / 7.1), with four worse (16 x 8 x 8000 7.3 / 10.6): the waves of one CU then take turns at the index search.
// grid = B, block = 1024.
constexpr int kSmallThreads = 1024, kSmallItems = kSmallThreads / kWave, kSmallPiece = kWave * kScanVec * 4;
__global__ __launch_bounds__(kSmallThreads) void accept_small_kernel(const AcceptParams p) {
    __shared__ uint64_t s_pairs[kSmallItems];
    __shared__ int32_t samax[VS_MAX_TREE];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int32_t parent = -2, draft = -1;
    if (wave == 0) {
        parent = tree_lane(p.parent + (int64_t)b * p.T, p.T);
        draft = p.draft[(int64_t)b * p.T + min(lane, p.T - 1)];
    }
    if (wave < p.T * p.chunks) { // uniform
        uint32_t piece;
        const uint32_t row = fast_div((uint32_t)wave, p.by_chunks, piece);
        const ScanChunk c = scan_load<kWave, kSmallPiece>(p.logits + ((int64_t)b * p.T + row) * p.ld, (int)piece, p.V, lane);
        const Best best = chunk_best<kWave>(c, (int)piece, lane);
        if (lane == 0) s_pairs[wave] = pair_of(best);
    }
    __syncthreads();
    accept_walk(p, b, s_pairs, [&](int32_t& to_parent, int32_t& to_draft) __attribute__((always_inline)) {
        to_parent = parent;
        to_draft = draft;
    }, samax);
}

constexpr int kMaxDevices = 64;
std::atomic<void*> scratch_of[kMaxDevices]; // device address of `scratch` on each device, null = not asked yet

// Device address of the current device's copy of `scratch`; asks the runtime on the first call
// per device. Returns null (and leaves no sticky error) when that fails.
void* scratch_address() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        return nullptr;
    }
    void* ptr = scratch_of[dev].load(std::memory_order_acquire);
    if (ptr) return ptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
        (void)hipGetLastError();
        return nullptr;
    }
    scratch_of[dev].store(ptr, std::memory_order_release);
    return ptr;
}

} // namespace

// workspace: 8 bytes per (row, chunk); sized by chunks half as long, it holds them with room to spare
hipError_t launch_accept(AcceptParams p, void* workspace, hipStream_t s) {
    const int64_t pieces = ((int64_t)p.V + kSmallPiece - 1) / kSmallPiece;
    if (pieces * p.T <= kSmallItems) { // (figures at the kernel)
        p.chunks = (int32_t)pieces;
        p.by_chunks = fast_div_by(p.chunks);
        hipLaunchKernelGGL(accept_small_kernel, dim3(p.B), dim3(kSmallThreads), 0, s, p);
        return hipGetLastError();
    }
    const bool short_chunks = scan_short_chunks(p.V, (int64_t)p.B * p.T);
    const int chunk = short_chunks ? kScanChunk / 2 : kScanChunk;
    p.chunks = (int32_t)(((int64_t)p.V + chunk - 1) / chunk);
    p.by_chunks = fast_div_by(p.chunks);
    p.pairs = (uint64_t*)workspace;
    const dim3 grid((unsigned)((int64_t)p.chunks * p.B * p.T));
    if (short_chunks) hipLaunchKernelGGL(argmax_partial_kernel<kScanThreads / 2>, grid, dim3(kScanThreads / 2), 0, s, p);
    else hipLaunchKernelGGL(argmax_partial_kernel<kScanThreads>, grid, dim3(kScanThreads), 0, s, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(accept_walk_kernel, dim3(p.B), dim3(kScanThreads), 0, s, p);
    return hipGetLastError();
}

} // namespace vs

extern "C" int32_t vs_tree_accept_noalloc(const float* logits, int64_t ld_logits, int32_t V, const int32_t* draft_tokens,
                                          const int32_t* parent, int32_t B, int32_t T, int32_t* accepted_len,
                                          int32_t* path, int32_t* bonus_token, int32_t* row_argmax, int32_t* status,
                                          void* stream) {
    using namespace vs;
    if (!logits || !draft_tokens || !parent || !accepted_len || !path || !bonus_token) return VS_ERR_NULL;
    if (B < 1 || T < 1 || T > VS_MAX_TREE || V < 1 || ld_logits < V) return VS_ERR_SHAPE;
    const size_t need = vs_accept_workspace_bytes(B, T, V);
    if (need == 0 || need > kNoallocScratchBytes) return VS_ERR_WORKSPACE; // beyond the static scratch: use vs_tree_accept
    if (const int32_t dc = check_device()) return dc;
    unsigned char* ws = (unsigned char*)scratch_address();
    if (!ws) return VS_ERR_HIP;
    AcceptParams p{};
    p.logits = logits;
    p.ld = ld_logits;
    p.V = V;
    p.draft = draft_tokens;
    p.parent = parent;
    p.B = B;
    p.T = T;
    p.accepted_len = accepted_len;
    p.path = path;
    p.bonus = bonus_token;
    p.row_argmax = row_argmax;
    p.status = status;
    return launch_accept(p, ws, (hipStream_t)stream) == hipSuccess ? VS_OK : VS_ERR_HIP;
}
