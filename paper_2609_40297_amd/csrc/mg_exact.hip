// Exact marginal gain with voxel sets on the device (eq. 2; the comparison the
// paper runs with voxel hash maps on the CPU, Sec. IV-E and V-A).
//
// For node n at window k_n, I(n) is the set of unknown voxels its window's
// rays meet. A set is a bit per voxel of the map in the path masks' layout, and
// a node with children keeps the union U(n) = U(parent) | I(n) of its own and
// its ancestors' sets as its path mask, with the code words: what conditions its
// children is "the voxel is in U(parent)", which is the question the trace asks
// of a path mask, so the incidences outside the ancestors' sets are counted by
// the trace itself, uniform blocks in one step. Level by level (k_exact_set,
// k_exact_merge):
//   - the trace counts incidences outside U(parent): over the window's rays
//     (X_ray at given windows), or over the panorama's per bin, from which the
//     node's window is chosen (own yaw);
//   - every window ray's unknown voxels are set in the node's own set;
//   - the own set is merged with U(parent): its size (A_set), its members
//     outside U(parent) (X_set), and U(n) with its code words for a node with
//     children; the own set is cleared for the next node that takes its place.
// Bounded by the walk of single unknown voxels and by the atomic ors of the sets'
// words: a lane gathers the bits of a word along its ray, a workgroup those of its
// 64 rays in LDS (the rays near the node, and neighbours far from it, meet the same
// words), and small levels give a ray to several lanes. Own-yaw gains and then the
// three counts at their windows, on a 500-node tree (360 x 60 rays, 200 x 200 x 60
// grid): 2.66 ms with each lane's words sent to memory (2.62 eight at a time), 2.47
// with rays split, 2.07 with the words gathered in LDS; 16.8 ms with hash sets
// (32-bit ids, open addressing, every ancestor's table probed for every incidence).
#pragma clang fp contract(off)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <set>
#include <vector>

#include "mg_batch.h"

using namespace mgk;

namespace mgx {

// One wave: a block of kRayBlockCols x kRayBlockRows window rays. Its LDS words: with
// 2^8, 2^9 and 2^10 of them 2.10, 2.08 and 2.13 ms; four waves that share 2^11: 2.11.
constexpr int kSetThreads = 64, kSetWordsLog = 9, kSetWords = 1 << kSetWordsLog;
// Lanes a ray while the launch has at most this many waves: a small level lasts as
// long as its longest ray's chain of steps. With one lane 2.28 ms; limits of 8192,
// 16384, 32768, 65536 and 131072 waves: 2.10, 2.11, 2.07, 2.13 and 2.15.
constexpr int64_t kSetWaves = 32768;
constexpr int kMergeThreads = 256;           // one thread per brick
constexpr size_t kPoolBytes = size_t(1) << 30;   // own sets held at once (at least one node's)

// The unknown voxels met by the rays of each listed node's window, set in
// own[item * mask_words ...] (all clear before). Work item = (node, block of
// window rays); free blocks are crossed in one step. kSeg lanes share a ray: each
// walks the stretch between two parameters, equal parts of the way to the ray's
// first hit (which the level's trace has stored), the last one to the ray's end.
// A stretch starts in the voxel that the walk stands in when every boundary with a
// parameter below its start is crossed; the stretch before sets the same bit.
template <int kSeg>
__global__ __launch_bounds__(kSetThreads) void k_exact_set(MapDev M, SensorDev S, TreeDev Tr,
                                                           const int32_t* __restrict__ nodes,
                                                           const int32_t* __restrict__ yaw, int32_t blocks,
                                                           uint32_t* own) {
    constexpr int32_t kCols = kRayBlockCols / kSeg, kPix = kSetThreads / kSeg;
    __shared__ uint32_t s_word[kSetWords], s_bits[kSetWords];
    for (int32_t k = (int32_t)threadIdx.x; k < kSetWords; k += kSetThreads) {
        s_word[k] = ~0u;
        s_bits[k] = 0u;
    }
    __syncthreads();
    const int32_t item = (int32_t)(blockIdx.x / (uint32_t)blocks), blk = (int32_t)blockIdx.x - item * blocks;
    const int32_t node = nodes[item];
    const int32_t cb = (int32_t)divide((uint32_t)blk, (uint32_t)S.nrb, S.nrb_mul), lane = (int32_t)threadIdx.x, seg = lane / kPix;
    const int32_t i = cb * kCols + (lane & (kCols - 1));
    const int32_t j = (blk - cb * S.nrb) * kRayBlockRows + (lane & (kPix - 1)) / kCols;
    uint32_t* mine = own + (size_t)item * M.mask_words;
    // the bits of a word: into its slot, or to memory where another word holds the slot
    auto put = [&](uint32_t word, uint32_t bits) {
        const uint32_t at = (word * 0x9e3779b1u) >> (32 - kSetWordsLog);
        const uint32_t was = atomicCAS(&s_word[at], ~0u, word);
        if (was == ~0u || was == word)
            atomicOr(&s_bits[at], bits);
        else
            atomicOr(&mine[word], bits);
    };
    auto walk = [&]() {
        int32_t c = S.c0_of_win[yaw[node]] + i;
        c = c >= S.W ? c - S.W : c;
        const int32_t r = c * S.H + j;
        RayWalk w;
        w.start(Tr.q4[node], S.d4[r], S.iv4[r], M);
        float end = S.rv;
        if (kSeg > 1) {
            // (a ray of less than a voxel a stretch is left to its first lane)
            const float h = Tr.dpan[(size_t)node * S.R + r];
            const bool split = h >= (float)kSeg;
            if (seg > 0) {
                if (!split) return;
                const float most = __uint_as_float(__float_as_uint(h * ((float)seg / (float)kSeg)) - 1u);
                w.pass(most, most, most, most);
                if (!w.in_grid(M)) return;
            }
            if (split && seg < kSeg - 1) end = h * ((float)(seg + 1) / (float)kSeg);
        }
        const int32_t before = (int32_t)__float_as_uint(end) - 1;
        const float most = fminf(__uint_as_float((uint32_t)before), end);
        uint32_t word = 0u, bits = 0u;           // bits of one word gathered along the ray
        uint32_t st = M.bricks[w.addr(M)];
        while ((st & 2u) == 0u) {                // (occupied, or outside the grid: the ray ends)
            uint32_t e1 = __builtin_amdgcn_ubfe(kEdgeOfLevel, st & (kLevelMask << kLevelShift), 4u);
            if (is_unknown(st)) {
                const uint32_t to = mask_word(w.x(), w.y(), w.z(), M);
                if (to != word) {
                    if (bits) put(word, bits);
                    word = to;
                    bits = 0u;
                }
                bits |= 1u << mask_bit(w.x(), w.y());
                e1 = 0u;
            }
            if (!(w.cross(e1, before, most) < end)) break;
            st = M.bricks[w.addr(M)];
        }
        if (bits) put(word, bits);
    };
    if (i < S.WB && j < S.H) walk();
    __syncthreads();
#pragma unroll
    for (int32_t k = (int32_t)threadIdx.x; k < kSetWords; k += kSetThreads)
        if (s_word[k] != ~0u) atomicOr(&mine[s_word[k]], s_bits[k]);
}

// The code word of a brick's 512 bits without its block's code (mg_internal.h).
__device__ __forceinline__ uint32_t code_of_words(const uint32_t (&q)[16]) {
    uint32_t cw = 0u;
    bool none = true, all = true;
#pragma unroll
    for (uint32_t qd = 0; qd < 8; ++qd) {
        const uint32_t m = (qd & 1u) ? 0xf0f0f0f0u : 0x0f0f0f0fu;     // x half; words: rows' half and z-slices
        uint32_t any = 0u, every = ~0u;
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t v = q[2u * (4u * (qd >> 2) + k) + ((qd >> 1) & 1u)];
            any |= v & m;
            every &= v | ~m;
        }
        const bool qn = any == 0u, qa = every == ~0u;
        none = none && qn;
        all = all && qa;
        cw |= (qn ? (uint32_t)kMaskNone : (qa ? (uint32_t)kMaskAll : (uint32_t)kMaskMixed)) << (2u + 2u * qd);
    }
    return cw | (none ? (uint32_t)kMaskNone : (all ? (uint32_t)kMaskAll : (uint32_t)kMaskMixed));
}

// Merges each listed node's own set with its parent's union, a thread per brick
// (in blocks of 2x2x2 bricks, as the mask builder visits them): counts (may be
// null) and, for a node with children, its union and code words, of which only
// what can be read is written (mg_internal.h). The own set is left clear. Bricks
// that the node's rays cannot reach hold nothing of its set, which is not read there
// (and a leaf has no union to write there): 300 nodes, 128 x 24 rays of 50 voxels, on a
// 1024 x 1024 x 200 grid, the three counts at given windows: 1715 -> 808 us (1225 with
// the hash sets, whose cost did not grow with the grid); 500 nodes of rays that reach
// most of their grid (200 x 200 x 60): 1166 and 1166 us.
__global__ __launch_bounds__(kMergeThreads) void k_exact_merge(MapDev M, TreeDev Tr, const int32_t* __restrict__ nodes,
                                                               int32_t chunks, uint32_t* __restrict__ own,
                                                               uint32_t* __restrict__ a_set,
                                                               uint32_t* __restrict__ x_set, float rv) {
    const int32_t item = (int32_t)(blockIdx.x / (uint32_t)chunks);
    const uint32_t sl = (blockIdx.x - (uint32_t)item * (uint32_t)chunks) * kMergeThreads + threadIdx.x;
    const int32_t node = nodes[item];
    const int2 slots = Tr.mask_slot[node];
    const int32_t slot = slots.x, ps = slots.y;      // (the parent's union)
    const uint32_t nb = M.mask_words >> 4;
    const uint3 at = slot_brick(sl, M);
    const uint32_t bx = at.x, by = at.y, bz = at.z;
    const bool in_map = bx < M.mbx && by < M.mby && bz < M.mbz;
    const uint32_t b = in_map ? bx + M.mbx * (by + M.mby * bz) : 0u;
    // distance of the brick's box from the node: a voxel entered before the range lies
    // within it but for rounding, far below the voxel added
    const float4 p = Tr.q4[node];
    const float x0 = (float)(8u * bx), y0 = (float)(8u * by), z0 = (float)(8u * bz);
    const float dx = fmaxf(fmaxf(x0 - p.x, p.x - (x0 + 8.f)), 0.f), dy = fmaxf(fmaxf(y0 - p.y, p.y - (y0 + 8.f)), 0.f),
                dz = fmaxf(fmaxf(z0 - p.z, p.z - (z0 + 8.f)), 0.f);
    const bool reach = dx * dx + dy * dy + dz * dz <= (rv + 1.f) * (rv + 1.f);
    const uint32_t bu = in_map & (reach | (slot >= 0)) ? (M.brick_unk[b] & 3u) : (uint32_t)kBrickKnown;
    uint32_t cw = 0u, members = 0u, fresh = 0u;
    if (bu != kBrickKnown) {
        uint32_t q[16];
        uint4* o = reinterpret_cast<uint4*>(own + (size_t)item * M.mask_words + (size_t)b * 16u);
        uint32_t any = 0u;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint4 v = reach ? o[k] : make_uint4(0u, 0u, 0u, 0u);
            q[4 * k] = v.x; q[4 * k + 1] = v.y; q[4 * k + 2] = v.z; q[4 * k + 3] = v.w;
            any |= v.x | v.y | v.z | v.w;
        }
        const uint32_t pcw = ps >= 0 ? Tr.mcode[(size_t)ps * nb + b] : uniform_code_word(kMaskNone);
        const uint32_t pc = pcw & 3u;
        cw = pcw;
        if (any != 0u) {
#pragma unroll
            for (int k = 0; k < 4; ++k) o[k] = make_uint4(0u, 0u, 0u, 0u);
        }
        // (a brick the node adds nothing to keeps the parent's code, and its words where they can be read)
        if (any != 0u || (slot >= 0 && (pc == kMaskMixed || bu == kBrickSomeUnknown))) {
            const uint4* par = reinterpret_cast<const uint4*>(Tr.masks + (size_t)(ps >= 0 ? ps : 0) * M.mask_words + (size_t)b * 16u);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t u = pc == kMaskAll ? ~0u : 0u;
                const uint4 v = pc == kMaskMixed ? par[k] : make_uint4(u, u, u, u);
                const uint32_t pv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    members += (uint32_t)__popc(q[4 * k + e]);
                    fresh += (uint32_t)__popc(q[4 * k + e] & ~pv[e]);
                    q[4 * k + e] |= pv[e];
                }
            }
            if (any != 0u) cw = code_of_words(q);
            if (slot >= 0 && ((cw & 3u) == kMaskMixed || bu == kBrickSomeUnknown)) {
                uint4* out = reinterpret_cast<uint4*>(Tr.masks + (size_t)slot * M.mask_words + (size_t)b * 16u);
#pragma unroll
                for (int k = 0; k < 4; ++k) out[k] = make_uint4(q[4 * k], q[4 * k + 1], q[4 * k + 2], q[4 * k + 3]);
            }
        }
    }
    // the code of the block of 2x2x2 bricks: uniform when its bricks are wholly unknown and all clear, or all set
    const uint32_t lane8 = threadIdx.x & 56u;
    const bool unk = bu == kBrickAllUnknown;
    const uint32_t n8 = (uint32_t)(__builtin_amdgcn_ballot_w64(unk && (cw & 3u) == kMaskNone) >> lane8) & 0xffu;
    const uint32_t s8 = (uint32_t)(__builtin_amdgcn_ballot_w64(unk && (cw & 3u) == kMaskAll) >> lane8) & 0xffu;
    if (slot >= 0 && bu != kBrickKnown) {
        const uint32_t bc = n8 == 0xffu ? (uint32_t)kMaskNone : (s8 == 0xffu ? (uint32_t)kMaskAll : (uint32_t)kMaskMixed);
        Tr.mcode[(size_t)slot * nb + b] = (cw & 0x3ffffu) | (bc << 18);
    }
    for (int32_t off = 32; off > 0; off >>= 1) {
        members += __shfl_xor(members, off, 64);
        fresh += __shfl_xor(fresh, off, 64);
    }
    if ((threadIdx.x & 63u) == 0u) {
        if (a_set && members) atomicAdd(&a_set[node], members);
        if (x_set && fresh) atomicAdd(&x_set[node], fresh);
    }
}

// Own sets of one device, which its trees' calls take in turn (they hold the lock
// and return after the work): all clear between calls but after one that failed,
// whose voxels may still be in them. Freed with the last tree that used them.
struct State {
    uint32_t* own = nullptr;
    size_t words = 0;
    size_t asked = 0;                            // words a call wanted when they were allocated: more than `words` if memory was short
    bool clear = false;
    std::set<mg_tree> users;
};

std::mutex g_mu;
std::map<int, State> g_state;                    // by device

int fail_hip(hipError_t e, const char* what) {
    return mgb::set_error(e == hipErrorOutOfMemory ? MG_E_NOMEM : MG_E_DEVICE, what);
}

// Own sets for the widest of the levels' lists (*nodes of them), at most kPoolBytes
// and fewer where device memory is short, for a call that says itself when it has
// left them clear.
int own_sets(State& st, mg_tree t, const MapDev& M, const std::vector<int32_t>& level_ptr, hipStream_t s, int32_t* nodes) {
    const size_t per = M.mask_words;
    size_t want = 1;
    for (size_t d = 0; d + 1 < level_ptr.size(); ++d) want = std::max(want, (size_t)(level_ptr[d + 1] - level_ptr[d]));
    want = std::min(want, std::max<size_t>(1, kPoolBytes / (sizeof(uint32_t) * per)));
    st.users.insert(t);
    if (st.clear && st.words >= per && std::max(st.words, st.asked) >= per * want) {
        *nodes = (int32_t)std::min(want, st.words / per);
        st.clear = false;
        return MG_OK;
    }
    st.clear = false;
    (void)hipFree(st.own);                       // (after the work of a call that failed)
    st.own = nullptr;
    st.words = 0;
    st.asked = per * want;
    hipError_t e = mgb::device_alloc(&st.own, sizeof(uint32_t) * per * want);
    while (e == hipErrorOutOfMemory && want > 1) {
        want = (want + 1) / 2;
        e = mgb::device_alloc(&st.own, sizeof(uint32_t) * per * want);
    }
    if (e == hipSuccess) e = launch_zero_u32(st.own, per * want, s);
    if (e != hipSuccess) {
        (void)hipFree(st.own);
        st.own = nullptr;
        return fail_hip(e, "exact-gain sets");
    }
    st.words = per * want;
    *nodes = (int32_t)want;
    return MG_OK;
}

// Own sets, counts and unions of the listed nodes (of one level), as many at a time as there are sets (held).
hipError_t merge_level(const State& st, int32_t held, const mgb::TreeView& v, const int32_t* nodes, int32_t n, const int32_t* yaw,
                       uint32_t* a_set, uint32_t* x_set, hipStream_t s) {
    const SensorDev& S = *v.sd;
    const int32_t chunks = (int32_t)((v.map->build_slots + kMergeThreads - 1) / kMergeThreads);
    for (int32_t at = 0; at < n; at += held) {
        const int32_t cnt = std::min(held, n - at);
        const int64_t waves = (int64_t)cnt * ((S.WB + kRayBlockCols - 1) / kRayBlockCols) * S.nrb;
        int seg = 8;
        while (seg > 1 && waves * seg > kSetWaves) seg >>= 1;
        const int32_t cols = kRayBlockCols / seg, blocks = (S.WB + cols - 1) / cols * S.nrb;
        const dim3 grid((unsigned)cnt * (unsigned)blocks);
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid, dim3(kSetThreads), 0, s, *v.map, S, *v.td, nodes + at, yaw, blocks, st.own);
        };
        if (seg == 8)
            go(k_exact_set<8>);
        else if (seg == 4)
            go(k_exact_set<4>);
        else if (seg == 2)
            go(k_exact_set<2>);
        else
            go(k_exact_set<1>);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_exact_merge, dim3((unsigned)cnt * (unsigned)chunks), dim3(kMergeThreads), 0, s, *v.map,
                           *v.td, nodes + at, chunks, st.own, a_set, x_set, S.rv);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace mgx

namespace mgb {
void forget_exact(mg_tree t) {
    std::lock_guard<std::mutex> lk(mgx::g_mu);
    for (auto& d : mgx::g_state) {
        mgx::State& st = d.second;
        if (st.users.erase(t) == 0 || !st.users.empty()) continue;
        (void)hipFree(st.own);
        st.own = nullptr;
        st.words = 0;
        st.clear = false;
    }
}
}  // namespace mgb

extern "C" int mg_eval_exact(mg_tree t, void* hip_stream, const int32_t* yaw_bin, uint32_t* x_ray, uint32_t* x_set,
                             uint32_t* a_set) {
    using namespace mgx;
    if (!t || !yaw_bin || !x_ray) return mgb::set_error(MG_E_INVALID, "tree/yaw_bin/x_ray is NULL");
    mgb::TreeView v;
    int rc = mgb::tree_view(t, &v);
    if (rc != MG_OK) return rc;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
    if (dev != v.device) return mgb::set_error(MG_E_INVALID, "the tree lives on another device");
    hipStream_t s = (hipStream_t)hip_stream;
    const SensorDev& S = *v.sd;
    const TreeDev& Tr = *v.td;
    const int32_t n = v.n;
    {
        // windows are indices into the sensor's tables: check them on the host
        std::vector<int32_t> k(n);
        e = hipMemcpyAsync(k.data(), yaw_bin, sizeof(int32_t) * n, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return fail_hip(e, "exact-gain windows");
        for (int32_t i = 0; i < n; ++i)
            if (k[i] < 0 || k[i] >= S.B) return mgb::set_error(MG_E_INVALID, "a window index is outside [0, yaw_bins)");
    }
    std::lock_guard<std::mutex> lk(g_mu);
    State& st = g_state[dev];
    int32_t held = 0;
    const bool sets = x_set || a_set;        // (without them only a union of ancestors is asked for)
    rc = own_sets(st, t, *v.map, sets ? *v.level_ptr : *v.mask_level_ptr, s, &held);
    if (rc != MG_OK) return rc;
    e = launch_zero_u32(x_ray, (size_t)n, s);
    if (e == hipSuccess && x_set) e = launch_zero_u32(x_set, (size_t)n, s);
    if (e == hipSuccess && a_set) e = launch_zero_u32(a_set, (size_t)n, s);
    for (int32_t d = 0; d < v.levels && e == hipSuccess; ++d) {
        const int32_t b = (*v.level_ptr)[d], cnt = (*v.level_ptr)[d + 1] - b;
        const int32_t mb = (*v.mask_level_ptr)[d], mcnt = (*v.mask_level_ptr)[d + 1] - mb;
        e = launch_trace_window(*v.map, S, Tr, Tr.level_nodes + b, cnt, yaw_bin, x_ray, sets, s);
        if (e == hipSuccess)
            e = sets ? merge_level(st, held, v, Tr.level_nodes + b, cnt, yaw_bin, a_set, x_set, s)
                     : merge_level(st, held, v, Tr.mask_nodes + mb, mcnt, yaw_bin, nullptr, nullptr, s);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail_hip(e, "exact-gain kernels");
    st.clear = true;
    return MG_OK;
}

extern "C" int mg_eval_exact_marginal(mg_tree t, void* hip_stream, uint32_t* gain, int32_t* yaw_bin) {
    using namespace mgx;
    if (!t || !gain || !yaw_bin) return mgb::set_error(MG_E_INVALID, "tree/gain/yaw_bin is NULL");
    mgb::TreeView v;
    int rc = mgb::tree_view(t, &v);
    if (rc != MG_OK) return rc;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
    if (dev != v.device) return mgb::set_error(MG_E_INVALID, "the tree lives on another device");
    hipStream_t s = (hipStream_t)hip_stream;
    const SensorDev& S = *v.sd;
    const TreeDev& Tr = *v.td;
    std::lock_guard<std::mutex> lk(g_mu);
    State& st = g_state[dev];
    int32_t held = 0;
    rc = own_sets(st, t, *v.map, *v.mask_level_ptr, s, &held);
    if (rc != MG_OK) return rc;
    // level by level: new incidences per bin, window, then the set at that window
    e = launch_zero_u32(Tr.bins, (size_t)S.B * v.n, s);
    for (int32_t d = 0; d < v.levels && e == hipSuccess; ++d) {
        const int32_t b = (*v.level_ptr)[d], cnt = (*v.level_ptr)[d + 1] - b;
        const int32_t mb = (*v.mask_level_ptr)[d], mcnt = (*v.mask_level_ptr)[d + 1] - mb;
        const int32_t* nodes = Tr.level_nodes + b;
        e = launch_trace(*v.map, S, Tr, nodes, cnt, true, false, s);
        if (e == hipSuccess) e = launch_finish(S, Tr, nodes, cnt, true, gain, yaw_bin, s);
        if (e == hipSuccess)
            e = merge_level(st, held, v, Tr.mask_nodes + mb, mcnt, (const int32_t*)yaw_bin, nullptr, nullptr, s);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail_hip(e, "exact marginal gain");
    st.clear = true;
    return MG_OK;
}
