// gfx950 kernels of the marginal-gain path.
//
// Exactness: every decision (which voxels a ray visits, whether an ancestor
// sees a voxel, which window wins) is taken in IEEE binary32 with the
// operation order of the definitions below and without contraction into
// fused multiply-adds. Approximate arithmetic (hardware reciprocal and
// reciprocal square root) appears only in *estimates* of a pixel index that
// are then corrected by the exact boundary tests, so it never changes a result.
#pragma clang fp contract(off)

#include <hip/hip_ext.h>

#include "mg_internal.h"

namespace mgk {

// Global-memory views of pointers that reach a kernel through a descriptor in
// memory: the compiler then issues global (not flat) loads for them.
typedef const __attribute__((address_space(1))) uint8_t* gbytes_t;
typedef const __attribute__((address_space(1))) float* gfloats_t;
typedef const __attribute__((address_space(1))) uint32_t* gwords_t;
__device__ __forceinline__ gbytes_t as_global(const uint8_t* p) { return (gbytes_t)p; }
__device__ __forceinline__ gfloats_t as_global(const float* p) { return (gfloats_t)p; }
__device__ __forceinline__ gwords_t as_global(const uint32_t* p) { return (gwords_t)p; }

// A workgroup-uniform pointer moved to scalar registers (loads through it then
// take a scalar base and a 32-bit vector offset).
template <class T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (T*)(((uint64_t)hi << 32) | lo);
}

// Wave ballot of a boolean (no widening of the predicate to an integer).
__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// ---------------------------------------------------------------- map layout

// Dense [nz][ny][nx] -> bricks; padding voxels (beyond the true extent) are
// set to kOutside, which ends a traversal that reaches them.
__global__ void k_brick(const uint8_t* __restrict__ dense, uint8_t* __restrict__ bricks, MapDev m) {
    const uint32_t total = (uint32_t)m.nbx * m.nby * m.nbz * 512u;
    for (uint32_t o = blockIdx.x * blockDim.x + threadIdx.x; o < total; o += gridDim.x * blockDim.x) {
        uint32_t b = o >> 9, in = o & 511u;
        int32_t bx = (int32_t)(b % (uint32_t)m.nbx);
        int32_t by = (int32_t)((b / (uint32_t)m.nbx) % (uint32_t)m.nby);
        int32_t bz = (int32_t)(b / ((uint32_t)m.nbx * (uint32_t)m.nby));
        int32_t x = bx * 8 + (int32_t)(in & 7u), y = by * 8 + (int32_t)((in >> 3) & 7u),
                z = bz * 8 + (int32_t)(in >> 6);
        uint8_t v = kOutside;
        if (x < m.nx && y < m.ny && z < m.nz)
            v = dense[(size_t)x + (size_t)m.nx * ((size_t)y + (size_t)m.ny * (size_t)z)];
        bricks[o] = v;
    }
}

// Per-brick summaries, after any write of the states: brick_unk[b] says whether
// brick b holds no, some or only unknown voxels, and every unknown and free
// voxel gets the level of the largest block around it that holds its state
// only (mark_brick_row). One wave per brick, each lane reading 8 of its 512
// bytes and writing them back only if a mark changes (padding voxels past the
// grid hold kOutside, so a block that reaches past the grid is never marked).
__global__ void k_brick_flags(MapDev m) {
    const uint32_t nb = m.mask_words >> 4;
    const uint32_t lane = threadIdx.x & 63u;
    uint8_t* grid = const_cast<uint8_t*>(m.bricks);
    for (uint32_t b = (blockIdx.x * blockDim.x + threadIdx.x) >> 6; b < nb; b += (gridDim.x * blockDim.x) >> 6) {
        const uint32_t bx = b % m.mbx, by = (b / m.mbx) % m.mby, bz = b / (m.mbx * m.mby);
        const uint32_t base = voxel_addr((int32_t)(bx * 8u), (int32_t)(by * 8u), (int32_t)(bz * 8u), m);
        uint64_t* p = reinterpret_cast<uint64_t*>(grid + base + lane * 8u);
        const uint64_t v = *p;
        bool any_unk, all_unk, all_free;
        const uint64_t w = mark_brick_row(v, lane, &any_unk, &all_unk, &all_free);
        if (lane == 0) m.brick_unk[b] = brick_summary(any_unk, all_unk, all_free);
        if (w != v) *p = w;
    }
}

// 16x16x16 blocks, after the bricks' summaries: where an aligned block of 2x2x2
// bricks lies in the grid's bricks and holds only wholly free (or only wholly
// unknown) bricks, their voxels are marked at level 1. A wave takes 8 blocks, a
// lane per brick to look at the summaries, then all its lanes write each such
// block's 4 KiB. 512 x 512 x 128, 80 % unknown: 7.6 us (a thread per brick
// that writes its own 512 bytes: 13.9 us).
__global__ void k_blocks16(MapDev m) {
    const uint32_t cx = m.mbx >> 1, cy = m.mby >> 1, cz = m.mbz >> 1, n = cx * cy * cz;     // whole blocks
    const uint32_t lane = threadIdx.x & 63u, k = lane & 7u;
    uint8_t* grid = const_cast<uint8_t*>(m.bricks);
    for (uint32_t g = ((blockIdx.x * blockDim.x + threadIdx.x) >> 6) * 8u; g < n; g += ((gridDim.x * blockDim.x) >> 6) * 8u) {
        const uint32_t c = g + (lane >> 3);
        const uint32_t bx = 2u * (c % cx) + (k & 1u), by = 2u * ((c / cx) % cy) + ((k >> 1) & 1u), bz = 2u * (c / (cx * cy)) + (k >> 2);
        const uint32_t own = c < n ? m.brick_unk[bx + m.mbx * (by + m.mby * bz)] : 0u;
        const uint64_t f = ballot((own & kBrickAllFree) != 0u), u = ballot((own & 3u) == kBrickAllUnknown);
        for (uint32_t i = 0; i < 8u; ++i) {
            const bool free_b = ((f >> (8u * i)) & 0xffu) == 0xffu, unk_b = ((u >> (8u * i)) & 0xffu) == 0xffu;
            if (!free_b && !unk_b) continue;
            const uint32_t ci = g + i;       // (a lane's 64 bytes: brick lane / 8 of the block)
            const uint32_t x = 2u * (ci % cx) + ((lane >> 3) & 1u), y = 2u * ((ci / cx) % cy) + ((lane >> 4) & 1u),
                           z = 2u * (ci / (cx * cy)) + (lane >> 5);
            const uint32_t base = voxel_addr((int32_t)(x * 8u), (int32_t)(y * 8u), (int32_t)(z * 8u), m);
            const uint32_t w = ((free_b ? kFree : kUnknown) | (1u << kLevelShift)) * 0x01010101u;
            uint4* p = reinterpret_cast<uint4*>(grid + base) + (lane & 7u);       // (a brick is 512 contiguous, aligned bytes)
#pragma unroll
            for (int q = 0; q < 4; ++q) p[8 * q] = make_uint4(w, w, w, w);
        }
    }
}

__global__ void k_zero_u32(uint32_t* __restrict__ p, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

// ---------------------------------------------------------------- window geometry

// A node's position (voxel units) and its window: first column and the unit
// vectors of its left and right boundaries.
struct WindowGeom {
    float qx, qy, qz;
    int32_t c0;
    float b0x, b0y;       // left boundary of the window
    float b1x, b1y;       // right boundary (left boundary of column c0 + w_buf)
};

__device__ __forceinline__ int32_t wrap(int32_t c, int32_t W) { return c >= W ? c - W : c; }

// r lies at or to the left (counter-clockwise side) of boundary direction b.
__device__ __forceinline__ bool left_of(float2 b, float rx, float ry) { return b.x * ry - b.y * rx >= 0.f; }

// Workgroups are dealt to the chip's 8 XCDs (each with its own L2) in turn:
// this permutation of the grid gives each XCD runs of kRun consecutive work
// units (neighbouring pixel blocks, or bricks, of one node) while the runs
// still alternate over the whole grid; the grid's last partial round keeps
// the identity. Runs of 8 in the per-tree trace: 500 nodes 893 to 898 us in plain
// order, 881 to 889 so, 333 odd ones 638 to 643 and 624 to 634 (four processes each;
// runs of 16 and 64 are within that spread); its builder gains nothing. Multi-tree launches take
// 16 (128.9 ms against 136 in plain order, 24000 nodes).
constexpr uint32_t kTreeRun = 8, kBatchRun = 16;
template <uint32_t kRun>
__device__ __forceinline__ uint32_t xcd_grouped(uint32_t g, uint32_t n) {
    const uint32_t full = (n / (8u * kRun)) * (8u * kRun);
    return g < full ? ((g >> 3) / kRun) * (8u * kRun) + (g & 7u) * kRun + (g >> 3) % kRun : g;
}

// ---------------------------------------------------------------- path masks

// Mask builder launch shapes (rays per workgroup of the trace kernel, bricks
// per workgroup of the builder), all compiled; shape 0 is the default.
struct Shape {
    int threads, bricks;
};
constexpr Shape kShapes[] = {{256, 64}, {128, 64}, {512, 64}, {256, 128}, {256, 32}, {256, 256}, {128, 128}, {128, 256}, {512, 128}, {128, 512}, {128, 1024}, {64, 1024}, {64, 256}};
constexpr int kNumShapes = sizeof(kShapes) / sizeof(kShapes[0]);
constexpr int kMaxBuildBricks = 1024;
// the builder's fixed LDS beside its tables: a flag byte, a code word and a brick index per slot, and a word
constexpr size_t kBuildFixedLds = (size_t)kMaxBuildBricks * 9u + 16u;
constexpr int kBuildThreads = 256;
constexpr int kFewThreads = 512, kFewLanes = 8;   // of a launch of few workgroups (few_chunks)

struct TableLDS {
    float2* bv;
    float* ts;
    uint16_t* lut_col;
    uint16_t* lut_row;
};

// LDS carve-up of the builder, for one node: the column boundaries of its
// window (boundary k of the window = column c0 + k, k = 0 .. W_buf + 1) | row
// table | guess tables.
__device__ __forceinline__ TableLDS carve_tables(char* smem, const SensorDev& S) {
    TableLDS L;
    L.bv = reinterpret_cast<float2*>(smem);                 // [W_buf + 2]
    L.ts = reinterpret_cast<float*>(L.bv + S.WB + 2);
    L.lut_col = reinterpret_cast<uint16_t*>(L.ts + S.H + 1);
    L.lut_row = L.lut_col + S.n_lut_col;
    return L;
}

__device__ __forceinline__ void load_tables(const TableLDS& L, const SensorDev& S, int32_t c0) {
    for (int32_t i = threadIdx.x; i < S.WB + 2; i += blockDim.x) {
        int32_t c = c0 + i;
        c = c >= S.W ? c - S.W : c;
        c = c >= S.W ? c - S.W : c;
        L.bv[i] = S.bv[c];
    }
    for (int32_t i = threadIdx.x; i <= S.H; i += blockDim.x) L.ts[i] = S.ts[i];
    for (int32_t i = threadIdx.x; i < S.n_lut_col; i += blockDim.x) L.lut_col[i] = S.lut_col[i];
    for (int32_t i = threadIdx.x; i < S.n_lut_row; i += blockDim.x) L.lut_row[i] = S.lut_row[i];
}

// What the node can observe of brick (bx, by, bz), from below: the pixels that
// the brick's voxel centres can fall in lie inside a rectangle of the window
// (azimuth from the corners of the centres' box seen from outside, elevation
// from its nearest and farthest horizontal distance; both widened by a pixel,
// so float angles cannot drop a pixel), and every centre lies between the
// box's nearest and farthest distances. Returns kViewNone when the largest
// first hit over the tiles that cover the rectangle is below the nearest
// distance (no voxel is observed); kViewAll when the rectangle lies inside the
// window and its row band with a pixel to spare and the farthest distance is
// within the range and below the smallest first hit over those tiles (every
// voxel centre passes the per-voxel test, with margins for rounding); else
// kViewSome (the node is within a voxel of the box horizontally, the rectangle
// covers more than 64 tiles, or the voxels must be tested one by one).
// tm: the node's tile maxima, then its tile minima.
// `kLanes` neighbouring lanes (a power of two) hold the same brick and share its
// tiles; lane g is one of them.
enum : int { kViewNone = 0, kViewSome = 1, kViewAll = 2 };
template <int kLanes>
__device__ int brick_view(const SensorDev& S, const float* __restrict__ tm, float4 q, int32_t c0, uint32_t bx,
                          uint32_t by, uint32_t bz, int32_t g) {
    const float x0 = (float)(bx * 8u) + 0.5f - q.x, x1 = x0 + 7.f;
    const float y0 = (float)(by * 8u) + 0.5f - q.y, y1 = y0 + 7.f;
    const float z0 = (float)(bz * 8u) + 0.5f - q.z, z1 = z0 + 7.f;
    if (x0 <= 1.f && x1 >= -1.f && y0 <= 1.f && y1 >= -1.f) return kViewSome;
    // window columns of the four corners, unwrapped around the window
    const float W = (float)S.W, sh = 0.5f * (float)(S.W - S.WB);
    float lo = 1e30f, hi = -1e30f;
    const float cx[4] = {x0, x1, x0, x1}, cy[4] = {y0, y0, y1, y1};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float v = (atan2f(cy[k], cx[k]) - S.az0) * S.daz_inv - (float)c0;
        v -= W * floorf((v + sh) / W);
        lo = fminf(lo, v);
        hi = fmaxf(hi, v);
    }
    if (hi - lo > 0.5f * W) return kViewSome;
    if (hi + 1.f < 0.f || lo - 1.f >= (float)S.WB) return kViewNone;
    const float fc_lo = floorf(lo) - 1.f, fc_hi = floorf(hi) + 1.f;
    const int32_t c_lo = (int32_t)fmaxf(fc_lo, 0.f);
    const int32_t c_hi = (int32_t)fminf(fc_hi, (float)(S.WB - 1));
    const float dx = x0 > 0.f ? x0 : (x1 < 0.f ? -x1 : 0.f);
    const float dy = y0 > 0.f ? y0 : (y1 < 0.f ? -y1 : 0.f);
    const float dz = z0 > 0.f ? z0 : (z1 < 0.f ? -z1 : 0.f);
    const float rmin = sqrtf(dx * dx + dy * dy);
    const float rmax = sqrtf(fmaxf(x0 * x0, x1 * x1) + fmaxf(y0 * y0, y1 * y1));
    const float e_hi = atan2f(z1, z1 >= 0.f ? rmin : rmax);
    const float e_lo = atan2f(z0, z0 >= 0.f ? rmax : rmin);
    const float r_lo = floorf((e_lo - S.el0) * S.del_inv) - 1.f, r_hi = floorf((e_hi - S.el0) * S.del_inv) + 1.f;
    if (r_hi < 0.f || r_lo > (float)(S.H - 1)) return kViewNone;
    const int32_t j_lo = (int32_t)fmaxf(r_lo, 0.f), j_hi = (int32_t)fminf(r_hi, (float)(S.H - 1));
    const int32_t tc0 = c_lo / kTileCols, tc1 = c_hi / kTileCols, tr0 = j_lo / kTileRows, tr1 = j_hi / kTileRows;
    const int32_t rows = tr1 - tr0 + 1, tiles = (tc1 - tc0 + 1) * rows;
    if (tiles > 64) return kViewSome;
    float m = 0.f, mn = __builtin_inff();
    const float per_row = 1.0f / (float)rows;
    for (int32_t k = g; k < tiles; k += 4 * kLanes) {
#pragma unroll
        for (int32_t e = 0; e < 4; ++e) {                    // four tiles' loads in flight (500 nodes, four processes: 896 to 900 us one by one, 881 to 889)
            const int32_t t = min(k + e * kLanes, tiles - 1);
            const int32_t c = (int32_t)(((float)t + 0.5f) * per_row);   // t / rows: t < 64
            const int32_t at = (tc0 + c) * S.trows + tr0 + (t - c * rows);
            m = fmaxf(m, tm[at]);
            mn = fminf(mn, tm[S.n_tiles + at]);
        }
    }
#pragma unroll
    for (int32_t off = 1; off < kLanes; off <<= 1) {
        m = fmaxf(m, __shfl_xor(m, off, 64));
        mn = fminf(mn, __shfl_xor(mn, off, 64));
    }
    const float dmin2 = dx * dx + dy * dy + dz * dz;
    if (!(m * m * 1.0001f + 0.01f >= dmin2)) return kViewNone;
    const bool inside = (fc_lo >= 0.f) & (fc_hi <= (float)(S.WB - 1)) & (r_lo >= 0.f) & (r_hi <= (float)(S.H - 1));
    const float dmax2 = fmaxf(x0 * x0, x1 * x1) + fmaxf(y0 * y0, y1 * y1) + fmaxf(z0 * z0, z1 * z1);
    return (inside && dmax2 * 1.0001f + 0.01f <= fminf(S.rv2, mn * mn)) ? kViewAll : kViewSome;
}

// Path mask of node `node` over bricks [chunk * bricks, ...) of the mask grid:
// the parent's path mask (none at the root, and none with anc_cap = 1) ORed
// with the voxels the node itself observes. A voxel is observed when its
// centre lies in a pixel cell of the node's window (azimuth between two column
// boundaries by exact left-of tests, elevation between two row boundaries by
// r_z|r_z| against rho^2 times the tabulated t|t| of the boundary; cells
// half-open) and its squared range is at most the squared first hit stored for
// that pixel: the test its descendants would make against it. A brick keeps
// the parent's bits (and code) without testing when it lies beyond the range,
// wholly outside the node's azimuth wedge (margins cover the brick's voxel
// centres, within 3.5 sqrt(3) of its centre and 3.5 sqrt(2) across in x and
// y, and rounding), holds no unknown voxel, has every bit set already, or
// fails the depth cull (brick_view); a brick whose voxels the node observes
// all (brick_view again) gets every bit set without testing. Of these bricks
// only what can be read is written (the code, and the words when they can be
// read). The window's tables are loaded into LDS only when some
// brick of the chunk is tested (kFew: at the start). One wave tests one brick: each lane one (x, y)
// column of 8 voxels. Whole workgroup; chunks past the map's last brick do
// nothing (a batch launch covers its largest map).
__device__ __forceinline__ void build_live(const MapDev& M, const SensorDev& S, const TreeDev& Tr, int32_t node,
                                           const WindowGeom& A, float4 q, const uint32_t* par, uint32_t* out,
                                           char* smem, const uint8_t* s_live, uint32_t* s_cw, const uint32_t* s_b,
                                           uint32_t lo, int32_t cnt, bool loaded);

template <bool kFew>
__device__ __forceinline__ void build_chunk(const MapDev& M, const SensorDev& S, const TreeDev& Tr, int32_t node,
                                            int32_t chunk, int32_t bricks, char* smem, uint8_t* s_live,
                                            uint32_t* s_cw, uint32_t* s_b, int32_t* s_any) {
    const int32_t tid = threadIdx.x;
    const int2 slots = Tr.mask_slot[node];
    const int32_t slot = slots.x, ps = slots.y;
    const uint32_t nb = M.mask_words >> 4;
    const uint32_t lo = (uint32_t)chunk * (uint32_t)bricks;  // first build slot (bricks is a multiple of 8)
    if (slot < 0 || lo >= M.build_slots) return;             // a leaf (nothing reads its mask), or past the map
    uint32_t* out = Tr.masks + (size_t)slot * M.mask_words;
    const uint32_t* par = nullptr;
    const uint32_t* pcode = nullptr;
    if (Tr.anc_cap > 1 && ps >= 0) {
        par = Tr.masks + (size_t)ps * M.mask_words;
        pcode = Tr.mcode + (size_t)ps * nb;
    }
    const float4 q = Tr.q4[node];
    const int32_t c0 = Tr.c0[node];
    int32_t c1 = c0 + S.WB;
    c1 = c1 >= S.W ? c1 - S.W : c1;
    WindowGeom A;
    A.qx = q.x; A.qy = q.y; A.qz = q.z; A.c0 = c0;
    const float2 b0 = S.bv[c0], b1 = S.bv[c1];
    A.b0x = b0.x; A.b0y = b0.y; A.b1x = b1.x; A.b1y = b1.y;
    const int32_t cnt = bricks;
    constexpr int32_t kLanes = kFew ? kFewLanes : 1;         // lanes that share a brick's view
    if (tid == 0) *s_any = 0;
    if (kFew) load_tables(carve_tables(smem, S), S, c0);
    // The chunk's slots, a block of 2x2x2 bricks per 8 slots: s_b holds each slot's
    // brick (~0 for a slot past the grid's bricks).
    for (int32_t i = tid; i < cnt; i += (int32_t)blockDim.x) {
        const uint3 at = slot_brick(lo + (uint32_t)i, M);
        const uint32_t bx = at.x, by = at.y, bz = at.z;
        s_b[i] = (bx < M.mbx && by < M.mby && bz < M.mbz) ? bx + M.mbx * (by + M.mby * bz) : ~0u;
    }
    __syncthreads();
    // per brick of the chunk (s_live): bit 4 live, bits 2-3 its brick_unk value,
    // bits 0-1 the parent's code (kMaskNone at the root); a slot past the grid's
    // bricks holds no unknown voxel
    for (int32_t i = tid / kLanes; i < cnt; i += (int32_t)blockDim.x / kLanes) {
        const uint32_t b = s_b[i];
        if (b == ~0u) {                                      // (its lanes write the same)
            s_live[i] = (uint8_t)(kBrickKnown << 2);
            continue;
        }
        const uint3 at = slot_brick(lo + (uint32_t)i, M);
        const uint32_t bx = at.x, by = at.y, bz = at.z;
        const float rx = (float)(bx * 8u) + 4.0f - q.x, ry = (float)(by * 8u) + 4.0f - q.y,
                    rz = (float)(bz * 8u) + 4.0f - q.z;
        const float reach = S.rv + 6.6f;                     // 3.5 sqrt(3) = 6.06, plus rounding
        const bool near = rx * rx + ry * ry + rz * rz <= reach * reach;
        const float w0 = A.b0x * ry - A.b0y * rx, w1 = A.b1x * ry - A.b1y * rx;
        const bool wedge = (w0 >= -5.5f) & (w1 < 5.5f);      // 3.5 sqrt(2) = 4.95, plus rounding
        const uint32_t bu = M.brick_unk[b] & 3u;            // (without the all-free bit)
        const uint32_t pcw = par ? pcode[b] : uniform_code_word(kMaskNone);   // the parent's code word
        const uint32_t pc = pcw & 3u;
        // (a brick without unknown voxels needs no bits: only unknown voxels' bits
        // are read; nor does one whose voxels an ancestor all observes)
        const int view = (near && wedge && bu != kBrickKnown && pc != kMaskAll)
                             ? brick_view<kLanes>(S, Tr.tmax + (size_t)slot * 2 * S.n_tiles, q, c0, bx, by, bz,
                                                  tid & (kLanes - 1))
                             : kViewNone;
        // (a brick whose voxels the node observes all gets every bit set, as the
        // per-voxel test would give it)
        const bool live = view == kViewSome;
        s_live[i] = (uint8_t)(((uint32_t)live << 4) | (bu << 2) | (view == kViewAll ? (uint32_t)kMaskAll : pc));
        s_cw[i] = view == kViewAll ? uniform_code_word(kMaskAll) : pcw;
        if (live) *s_any = 1;
    }
    __syncthreads();
    // Bricks that cannot hold a newly observed voxel keep the parent's code and
    // the bits that can be read: its words when they are mixed, constant words
    // for a brick that also holds known voxels, none for a wholly unknown brick
    // with a uniform code; bricks without unknown voxels are left alone.
    for (int32_t w = tid; w < cnt * 16; w += blockDim.x) {
        const uint32_t f = s_live[w >> 4];
        const uint32_t pc = f & 3u, bu = (f >> 2) & 3u;
        if ((f & 16u) || bu == kBrickKnown || (bu == kBrickAllUnknown && pc != kMaskMixed)) continue;
        const uint32_t wi = s_b[w >> 4] * 16u + (uint32_t)(w & 15);
        out[wi] = pc == kMaskMixed ? par[wi] : (pc == kMaskAll ? ~0u : 0u);
    }
    uint32_t* code = Tr.mcode + (size_t)slot * nb;
    if (*s_any) build_live(M, S, Tr, node, A, q, par, out, smem, s_live, s_cw, s_b, lo, cnt, kFew);
    __syncthreads();
    // Code words of the chunk's bricks that hold an unknown voxel, with the code
    // of their block of 2x2x2 bricks (bits 18-19): uniform when the block's 8
    // bricks are all wholly unknown and their codes all clear or all set.
    for (int32_t i = tid; i < cnt; i += (int32_t)blockDim.x) {
        const uint32_t f = s_live[i];
        if (((f >> 2) & 3u) != kBrickKnown) {
            const int32_t g = i & ~7;
            uint32_t all_none = 1u, all_set = 1u;
#pragma unroll
            for (int32_t k = 0; k < 8; ++k) {
                const uint32_t fk = s_live[g + k], ck = s_cw[g + k] & 3u;
                const bool unk = ((fk >> 2) & 3u) == kBrickAllUnknown;
                all_none &= (unk && ck == kMaskNone) ? 1u : 0u;
                all_set &= (unk && ck == kMaskAll) ? 1u : 0u;
            }
            const uint32_t bc = all_none ? (uint32_t)kMaskNone : (all_set ? (uint32_t)kMaskAll : (uint32_t)kMaskMixed);
            code[s_b[i]] = (s_cw[i] & 0x3ffffu) | (bc << 18);
        }
    }
}

// The live bricks of a chunk (build_chunk): one wave tests one brick, each lane
// one (x, y) column of 8 voxels; the brick's code word goes to s_cw.
__device__ __forceinline__ void build_live(const MapDev& M, const SensorDev& S, const TreeDev& Tr, int32_t node,
                                           const WindowGeom& A, float4 q, const uint32_t* par, uint32_t* out,
                                           char* smem, const uint8_t* s_live, uint32_t* s_cw, const uint32_t* s_b,
                                           uint32_t lo, int32_t cnt, bool loaded) {
    const int32_t tid = threadIdx.x;
    const int32_t c0 = A.c0;
    const TableLDS L = carve_tables(smem, S);
    if (!loaded) {
        load_tables(L, S, c0);
        __syncthreads();
    }
    const int32_t lane = tid & 63;
    const float ts0 = L.ts[0], tsH = L.ts[S.H];
    const gfloats_t dnode = as_global(uniform_ptr(Tr.dpan + (size_t)node * S.R));   // the node's panorama
    // (the wave's brick is wave-uniform: its index arithmetic stays scalar)
    const int32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int32_t i = wave; i < cnt; i += (int32_t)(blockDim.x >> 6)) {
        const uint32_t f = s_live[i];
        if (!(f & 16u)) continue;
        const uint32_t b = s_b[i];
        const uint3 at = slot_brick(lo + (uint32_t)i, M);
        const int32_t bx = (int32_t)at.x, by = (int32_t)at.y, bz = (int32_t)at.z;
        const int32_t x = bx * 8 + (lane & 7), y = by * 8 + (lane >> 3);
        const float cx = (float)x + 0.5f, cy = (float)y + 0.5f;
        const uint32_t wbase = b << 4;
        uint32_t pw = 0u;                 // the parent's bits (a live brick's parent code is not all set)
        if ((f & 3u) == kMaskMixed && lane < 16) pw = par[wbase + (uint32_t)lane];
        // The lane's column of the brick: the azimuth column of its pixels (the
        // same for the 8 voxels, which share x and y), the row of each voxel,
        // then the 8 depths, loaded together. The voxels' states are not read: only unknown voxels' bits are ever looked
        // up, so bits of known voxels (and of voxels past the grid) do not matter.
        const float rx = cx - A.qx, ry = cy - A.qy;
        const float w0 = A.b0x * ry - A.b0y * rx;
        const float w1 = A.b1x * ry - A.b1y * rx;
        const bool wedge = (w0 >= 0.f) & (w1 < 0.f);
        const float rho2 = rx * rx + ry * ry;
        // column (computed for every lane; only lanes in the wedge use it, and the
        // clamps keep every table index inside its table)
        const float u0 = A.b0x * rx + A.b0y * ry;
        float pa = w0 * __builtin_amdgcn_rcpf(fabsf(u0) + w0);
        pa = u0 < 0.f ? 2.f - pa : pa;
        const int32_t gc =
            L.lut_col[(int32_t)__builtin_amdgcn_fmed3f(pa * S.lut_col_scale, 0.f, (float)(S.n_lut_col - 1))];
        const float2 v0 = L.bv[gc], v1 = L.bv[gc + 1], v2 = L.bv[gc + 2];
        const bool l0 = (gc == 0) | left_of(v0, rx, ry);
        const bool l1 = (gc + 1 < S.WB) & left_of(v1, rx, ry);
        const bool l2 = (gc + 2 < S.WB) & left_of(v2, rx, ry);
        int32_t col = gc + (int32_t)l1;
        if (wedge & !(l0 & !l2)) {      // (rare: a guess at a bucket edge)
            for (;;) {
                if (col + 1 >= S.WB || !left_of(L.bv[col + 1], rx, ry)) break;
                ++col;
            }
            for (;;) {
                if (col == 0 || left_of(L.bv[col], rx, ry)) break;
                --col;
            }
        }
        // (column < 4096 and H <= 2048: the product fits the 24-bit multiplier; the
        // index is into the node's own panorama, R < 2^22 entries)
        const uint32_t colbase = __umul24((uint32_t)wrap(A.c0 + col, S.W), (uint32_t)S.H);
        const float irho = __builtin_amdgcn_rsqf(rho2);
        // Rows: the row of a voxel is the number of inner row boundaries j in
        // 1..H-1 with sz >= rho2 * ts[j] (ts and hence rho2 * ts[j] grow with j,
        // so they form a prefix). Within the lane's column sz grows with z, so
        // the count never falls from one slice to the next: slice 0 takes the
        // guess table and its settle (exact for any sz: the table's clamped ends
        // give 0 and H - 1 outside the band), each later slice checks the next
        // two boundaries and walks on only when both are passed (steep voxels
        // near the node). Lanes outside the wedge never use their rows.
        uint32_t idx[8];
        float r2[8];
        bool ok[8];
        int32_t row = 0;
#pragma unroll
        for (int32_t pz = 0; pz < 8; ++pz) {
            const float rz = ((float)(bz * 8 + pz) + 0.5f) - A.qz;
            const float range2 = rho2 + rz * rz;
            const float sz = rz * fabsf(rz);
            ok[pz] = wedge & (range2 <= S.rv2) & (sz >= rho2 * ts0) & (sz < rho2 * tsH);
            r2[pz] = range2;
            if (pz == 0) {
                const float tg = rz * irho;
                const int32_t gr = L.lut_row[(int32_t)__builtin_amdgcn_fmed3f((tg - S.lut_row_lo) * S.lut_row_scale,
                                                                             0.f, (float)(S.n_lut_row - 1))];
                const float e0 = L.ts[gr], e1 = L.ts[gr + 1], e2 = L.ts[min(gr + 2, S.H)];
                const bool q0 = (gr == 0) | (sz >= rho2 * e0);
                const bool q1 = (gr + 1 < S.H) & (sz >= rho2 * e1);
                const bool q2 = (gr + 2 < S.H) & (sz >= rho2 * e2);
                row = gr + (int32_t)q1;
                if (wedge & !(q0 & !q2)) {   // (rare: a guess at a bucket edge)
                    for (;;) {
                        if (row + 1 >= S.H || !(sz >= rho2 * L.ts[row + 1])) break;
                        ++row;
                    }
                    for (;;) {
                        if (row == 0 || sz >= rho2 * L.ts[row]) break;
                        --row;
                    }
                }
            } else {
                const float e1 = L.ts[min(row + 1, S.H)], e2 = L.ts[min(row + 2, S.H)];
                const bool a1 = (row + 1 < S.H) & (sz >= rho2 * e1);
                const bool a2 = (row + 2 < S.H) & (sz >= rho2 * e2);
                row += (int32_t)a1;
                if (wedge & a2) {            // (two or more boundaries between neighbouring voxels)
                    for (;;) {
                        if (row + 1 >= S.H || !(sz >= rho2 * L.ts[row + 1])) break;
                        ++row;
                    }
                }
            }
            idx[pz] = ok[pz] ? colbase + (uint32_t)row : 0u;
        }
        float D[8];
#pragma unroll
        for (int32_t pz = 0; pz < 8; ++pz) D[pz] = *(gfloats_t)((gbytes_t)dnode + (idx[pz] << 2));
        // observed: the centre's squared range is at most its pixel's squared depth;
        // lane l < 16 collects mask word l of the brick (slice l / 2) and stores it
        uint32_t word = 0u;
#pragma unroll
        for (int32_t pz = 0; pz < 8; ++pz) {
            const uint64_t bal = ballot(ok[pz] & (r2[pz] <= D[pz] * D[pz]));
            word = lane == 2 * pz ? (uint32_t)bal : word;
            word = lane == 2 * pz + 1 ? (uint32_t)(bal >> 32) : word;
        }
        word |= pw;
        if (lane < 16) out[wbase + (uint32_t)lane] = word;
        // the brick's code word: its 512 bits and each quarter's 64 all clear, all
        // set, or mixed (word l holds slice l / 2, rows 4 (l & 1) .. + 3, x in its
        // bytes' low and high nibbles)
        const bool w_ok = lane < 16;
        const uint64_t nz_lo = ballot(w_ok & ((word & 0x0f0f0f0fu) != 0u)), nz_hi = ballot(w_ok & ((word & 0xf0f0f0f0u) != 0u));
        const uint64_t nf_lo = ballot(w_ok & ((word | 0xf0f0f0f0u) != ~0u)), nf_hi = ballot(w_ok & ((word | 0x0f0f0f0fu) != ~0u));
        uint32_t cw = (nz_lo | nz_hi) == 0ull ? (uint32_t)kMaskNone : ((nf_lo | nf_hi) == 0ull ? (uint32_t)kMaskAll : (uint32_t)kMaskMixed);
#pragma unroll
        for (uint32_t qd = 0; qd < 8; ++qd) {
            const uint64_t lq = 0x55ull << (8u * (qd >> 2) + ((qd >> 1) & 1u));   // words of the quarter's slices and rows
            const uint64_t nz = (qd & 1u) ? nz_hi : nz_lo, nf = (qd & 1u) ? nf_hi : nf_lo;
            const uint32_t qc = (nz & lq) == 0ull ? (uint32_t)kMaskNone : ((nf & lq) == 0ull ? (uint32_t)kMaskAll : (uint32_t)kMaskMixed);
            cw |= qc << (2u + 2u * qd);
        }
        if (lane == 0) s_cw[i] = cw;
    }
}

template <bool kFew>
__global__ __launch_bounds__(kFew ? kFewThreads : kBuildThreads) void k_mask_build(MapDev M, SensorDev S, TreeDev Tr,
                                                              const int32_t* __restrict__ nodes, int32_t chunks,
                                                              int32_t bricks, uint32_t chunks_mul) {
    extern __shared__ char smem[];
    __shared__ uint8_t s_live[kMaxBuildBricks];
    __shared__ uint32_t s_cw[kMaxBuildBricks];
    __shared__ uint32_t s_b[kMaxBuildBricks];
    __shared__ int32_t s_any;
    const uint32_t item = divide(blockIdx.x, (uint32_t)chunks, chunks_mul);
    build_chunk<kFew>(M, S, Tr, nodes[item], (int32_t)(blockIdx.x - item * (uint32_t)chunks), bricks, smem, s_live, s_cw,
                      s_b, &s_any);
}

// ---------------------------------------------------------------- ray traversal

// Lane shuffles without LDS: within rows of 16 lanes (DPP), and between the rows.
template <int kCtrl>
__device__ __forceinline__ uint32_t dpp(uint32_t v, uint32_t outside) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)outside, (int)v, kCtrl, 0xf, 0xf, false);
}
constexpr int kRowShl = 0x100, kRowShr = 0x110, kRowRor = 0x120;
__device__ __forceinline__ uint32_t add_halves(uint32_t v) {       // lanes l and l ^ 32
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return r[0] + r[1];
}
__device__ __forceinline__ uint32_t add_row_pairs(uint32_t v) {    // lanes l and l ^ 16
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return r[0] + r[1];
}

// Adds one wave's counts to its node's bins. Lane l holds count n and the bin of
// its column, column l mod kCols of the wave's block (bins never fall with the
// column): the counts of a column are summed over the lanes that share it, then
// over the columns of a bin by a segmented scan, and the last column of each bin
// makes one atomic add. A wave's columns touch a bin or a few, so this replaces an
// LDS histogram over all bins with its clearing, barriers and read-out; with one
// count per node and bin instead of two, and first hits stored only where they
// are read, it took 2 % off the large launches (12000 nodes 51.7 -> 50.7 ms).
template <int kCols>
__device__ __forceinline__ void add_to_bins(uint32_t n, uint32_t bin, uint32_t* __restrict__ bins) {
    if (ballot(n != 0u) == 0ull) return;
    n = add_row_pairs(add_halves(n));
    if (kCols <= 8) n += dpp<kRowRor + 8>(n, 0u);
    if (kCols <= 4) n += dpp<kRowRor + 4>(n, 0u);
    if (kCols <= 2) n += dpp<kRowRor + 2>(n, 0u);
    const uint32_t col = threadIdx.x & (kCols - 1);
    const bool last = (col == kCols - 1) | (dpp<kRowShl + 1>(bin, ~0u) != bin);
#define MG_SCAN(off)                                                                               \
    if (off < kCols) {                                                                             \
        const uint32_t o = dpp<kRowShr + off>(n, 0u), b = dpp<kRowShr + off>(bin, ~0u);            \
        n += (b == bin && col >= off) ? o : 0u;                                                   \
    }
    MG_SCAN(1)
    MG_SCAN(2)
    MG_SCAN(4)
    MG_SCAN(8)
#undef MG_SCAN
    if ((threadIdx.x & 63u) < kCols && last && n != 0u) atomicAdd(&bins[bin], n);
}

// One workgroup = kTh / 64 pixel blocks (tile `tile`) of one node, one block of
// kRayBlockCols x kRayBlockRows rays per wave: neighbouring pixels have rays of
// similar length, so a wave's lanes run for similar numbers of steps. A lane walks
// its ray with the Amanatides-Woo 3D DDA (face-crossing parameters recomputed
// as (boundary - q) * (1/d); ties step x, then y, then z; a voxel is visited
// while its entry parameter is below the range and it is inside the grid). An
// occupied voxel ends the ray and its entry parameter (or the range) is the
// ray's first hit (written when keep_hits: only a node with children, whose mask is
// built from them, and a caller that asked for depth buffers read them).
// Unknown voxels count into the bin of the ray's column: all of them in the
// absolute pass; in marginal mode those that the parent's path mask does not
// hold (no ancestor observes them); the root has no ancestor, so all its
// unknown voxels count. The grid byte of the next voxel is
// requested before the step ends, and a mask word is used one step after it
// was requested, so both loads have a step of work to hide behind. Ends with
// each wave's counts added to the node's bins.
//
// Steps are RayWalk's: one exact probe an axis decides which boundaries a block
// crossing passes, in place of the three or four of a search over the block's
// boundaries, and a single voxel takes the same path, so a wave does too: this
// loop is bound by instruction issue, and by the latency of its chain where a
// level has few nodes. Against the search: 59.8 -> 48.1 ms a batch of 4 trees of
// 3000 nodes (720 x 120 rays, 512 x 512 x 128 grid), 2.93 -> 2.12 ms the
// absolute pass of 1000 of these nodes, 1.21 -> 1.01 ms one tree of 500 nodes
// (360 x 60 rays, 200 x 200 x 60 grid).
//
// kSeg > 1 gives each ray to kSeg lanes, each walking the stretch of the ray
// between two parameters (kSeg equal parts of the range; a wave then holds a
// kSeg times narrower block of pixels), for launches too small to fill the chip:
// they last as long as the longest ray's chain of dependent steps, which the
// split divides. A stretch starts in the voxel that the walk stands in when every
// boundary with a parameter below the stretch's start is crossed (found as a
// step finds it), whose visit the stretch before has counted, and ends as the
// range ends; stretches after the ray's first hit count nothing, and a ray that
// has left the grid starts its later stretches outside.
//
// kWindow walks the rays of one yaw window only (WB columns from column c0) and
// adds their counts to *total.
template <bool kMarginal, int kTh, int kSeg = 1, bool kWindow = false>
__device__ __forceinline__ void trace_tile(const MapDev& M, const SensorDev& S, const TreeDev& Tr, int32_t node,
                                           int32_t tile, bool keep_hits, int32_t c0 = 0, uint32_t* total = nullptr) {
    const int32_t tid = threadIdx.x;
    const uint32_t* pmask = nullptr;     // the parent's path mask
    const uint32_t* pcode = nullptr;     // and its bricks' code words
    if (kMarginal) {
        const int32_t ps = Tr.mask_slot[node].y;
        if (Tr.anc_cap > 0 && ps >= 0) {
            pmask = Tr.masks + (size_t)ps * M.mask_words;
            pcode = Tr.mcode + (size_t)ps * (M.mask_words >> 4);
        }
    }
    const gwords_t pm = as_global(uniform_ptr(pmask));
    const gwords_t pc = as_global(uniform_ptr(pcode));
    // this wave's pixel block and this lane's pixel in it (column c, row j)
    const int32_t blk = __builtin_amdgcn_readfirstlane(tile * (kTh / 64) + (tid >> 6));
    const int32_t cb = __builtin_amdgcn_readfirstlane((int32_t)divide((uint32_t)blk, (uint32_t)S.nrb, S.nrb_mul));
    constexpr int32_t kCols = kRayBlockCols / kSeg, kPix = 64 / kSeg;
    const int32_t seg = (tid & 63) / kPix;               // this lane's stretch of its ray
    const int32_t i = cb * kCols + (tid & (kCols - 1));
    const int32_t c = kWindow ? wrap(c0 + i, S.W) : i;
    const int32_t j = (blk - cb * S.nrb) * kRayBlockRows + ((tid & (kPix - 1)) / kCols);
    const bool has_ray = (blk < S.n_blocks) & (i < (kWindow ? S.WB : S.W)) & (j < S.H);
    const int32_t r = c * S.H + j;
    const int32_t rr = has_ray ? r : 0;
    const uint32_t bin = kWindow ? 0u : (uint32_t)S.bin_of_col[has_ray ? c : 0];
    const float4 p = Tr.q4[node];
    const float4 d = S.d4[rr];
    const float4 iv = S.iv4[rr];
    RayWalk w;
    w.start(p, d, iv, M);
    // the stretch's start and end parameters, and the float below its end (> 0);
    // a range of less than a voxel a stretch is left to the ray's first lane
    const bool split = kSeg > 1 && S.rv >= (float)kSeg;
    const float t0 = split ? S.rv * ((float)seg / (float)kSeg) : 0.f;
    const float t1 = split && seg < kSeg - 1 ? S.rv * ((float)(seg + 1) / (float)kSeg) : S.rv;
    const int32_t t1_before = (int32_t)__float_as_uint(t1) - 1;
    const float t1_most = fminf(__uint_as_float((uint32_t)t1_before), t1);
    bool inside = has_ray & (split | (seg == 0));   // (the node lies inside the grid)
    bool counted = false;                // the current voxel's visit is the stretch before's
    if (split && seg > 0) {
        const float most = __uint_as_float(__float_as_uint(t0) - 1u);
        w.pass(most, most, most, most);
        inside = has_ray & w.in_grid(M);
        counted = true;
    }
    int32_t usum = w.ux + w.uy + w.uz + (counted ? 1 : 0);
    // lanes holding the earlier stretches of this lane's ray, and those that hit
    constexpr uint64_t kRayLanes = kSeg == 4 ? 0x0001000100010001ull : (kSeg == 2 ? 0x0000000100000001ull : 0x0101010101010101ull);
    const uint64_t earlier = kSeg > 1 ? ((kRayLanes << (tid & (kPix - 1))) & ((1ull << (tid & 63)) - 1ull)) : 0ull;
    uint64_t hits = 0ull;
    // h is kept negated (and t starts at -0): a hit at parameter 0 is +0 in the
    // node's own voxel and -0 in a voxel entered at once, since only an axis the
    // ray moves down has a boundary at the node, with parameter 0 * (1/d), d < 0
    float t = kSeg > 1 && seg > 0 ? t0 : -0.f, h = -S.rv;
    uint32_t n = 0;                      // the ray's count
    const gbytes_t grid = as_global(M.bricks);
    // a lane without a ray (or whose ray has left the grid) reads a padding byte
    // and is done at once
    uint32_t addr = inside ? w.addr(M) : M.outside;   // address of the current voxel
    // (this first byte is read through the generic pointer and the loop's through
    // the global one, so the compiler keeps the loop's load at the end of the
    // step instead of merging the two into one load at the top of the loop)
    uint32_t st = M.bricks[addr];
    uint32_t mw = 0u, mb = 0u;          // mask word of the last unknown voxel, and its bit
    bool pend = false;                  // (a word requested in the previous step)
    uint32_t cb_idx = ~0u, cw = 0u;     // the last unknown block's brick and its code word
    if (ballot(has_ray)) {
        uint64_t alive;
        do {
            // The mask word requested in the previous step and the current voxel's
            // byte are used first, then the next voxel is found and its byte
            // requested. A lane that has finished (or left the grid) reads a
            // padding byte, which is neither unknown nor occupied.
            if (kMarginal) {
                n += (pend & !((mw >> mb) & 1u)) ? 1u : 0u;
                pend = false;
            }
            h = st == kOccupied ? -t : h;
            if (kSeg > 1) hits |= ballot(st == kOccupied);
            // The block crossed in this step (e1: its edge - 1): the marked block
            // around a free voxel; for an unknown voxel the largest marked block
            // over which the parent's mask is uniform (every bit clear, or every
            // bit set), else the voxel itself, whose mask bit is looked up. The
            // absolute pass and the root see nothing observed.
            const bool unk = is_unknown(st);
            uint32_t e1 = __builtin_amdgcn_ubfe(kEdgeOfLevel, st & (kLevelMask << kLevelShift), 4u);
            bool fresh = unk;           // the voxels crossed are unknown and no ancestor observes them
            if (kMarginal && pm != nullptr) {
                fresh = false;
                if (unk) {
                    const int32_t x = w.x(), y = w.y(), z = w.z();
                    const uint32_t b = mask_brick(x, y, z, M);
                    uint32_t code = kMaskMixed;
                    // (a wholly unknown block with a uniform code is always crossed by its
                    // code: the words of its brick need not exist)
                    if (e1 != 0u) {
                        if (b != cb_idx) {
                            cw = *(gwords_t)((gbytes_t)pc + (b << 2));
                            cb_idx = b;
                        }
                        // the code of its block of 2x2x2 bricks (a 16-voxel block), else the
                        // brick's (a brick at most), else its quarter's (a quarter at most)
                        const uint32_t qs = 2u + ((((uint32_t)x >> 1) & 2u) | ((uint32_t)y & 4u) | (((uint32_t)z << 1) & 8u));
                        const uint32_t bc = (cw >> 18) & 3u, kc = cw & 3u, qc = (cw >> qs) & 3u;
                        const bool block_uniform = (e1 == 15u) & (bc != kMaskMixed);
                        const bool brick_uniform = kc != kMaskMixed;
                        code = block_uniform ? bc : (brick_uniform ? kc : qc);
                        const uint32_t most = block_uniform ? 15u : (brick_uniform ? 7u : 3u);
                        e1 = code == kMaskMixed ? 0u : (e1 < most ? e1 : most);
                    }
                    fresh = code == kMaskNone;
                    pend = (code == kMaskMixed) & !counted;
                    if (pend) {
                        const uint32_t off = ((b << 4) | ((uint32_t)(z & 7) << 1) | ((uint32_t)(y & 4) >> 2)) << 2;  // < 2^29 bytes
                        mw = *(gwords_t)((gbytes_t)pm + off);
                        mb = mask_bit(x, y);
                    }
                }
            }
            const float T = w.cross(e1, t1_before, t1_most);
            // voxels of the block visited: one per boundary crossed, and the last one of a ray that ends
            const int32_t unew = w.ux + w.uy + w.uz;
            const uint32_t count = (uint32_t)(unew - usum) + (T < t1 ? 0u : 1u);
            usum = unew;
            n += fresh ? count : 0u;
            if (kSeg > 1) counted = false;
            // a lane that stops here (occupied, finished or outside) compares +inf
            // with the range: one comparison gives the mask the ballot takes
            const float tn_go = (st & 2u) == 0u ? T : __builtin_inff();
            const bool next_ok = (tn_go < t1) & (kSeg == 1 || (hits & earlier) == 0ull);
            alive = ballot(next_ok);
            addr = next_ok ? w.addr(M) : M.outside;
            st = grid[addr];
            t = T;
        } while (alive);
    }
    // (stretches past the ray's first hit count nothing; one lane of a ray writes its
    // first hit: that of the hit, else its last stretch's)
    const bool first = kSeg == 1 || (hits & earlier) == 0ull;
    if (kMarginal) {
        n += (pend & !((mw >> mb) & 1u)) ? 1u : 0u;
        if (keep_hits & has_ray & first & (kSeg == 1 || (h > -S.rv) | (seg == kSeg - 1)))
            Tr.dpan[(size_t)node * S.R + r] = h == 0.f ? h : -h;
    }
    add_to_bins<kCols>(first ? n : 0u, bin, kWindow ? total : Tr.bins + (size_t)node * S.B);
}

// Per-tree levels: one-wave workgroups (as the batch autotuner picks for the
// large workloads).
constexpr int kTreeTraceThreads = 64;
template <bool kMarginal, int kSeg>
__global__ __launch_bounds__(kTreeTraceThreads) void k_trace(MapDev M, SensorDev S, TreeDev Tr,
                                                             const int32_t* __restrict__ nodes, bool depth) {
    // (workgroup-uniform values kept in scalar registers)
    const uint32_t g = xcd_grouped<kTreeRun>(blockIdx.x, gridDim.x);
    const int32_t item = __builtin_amdgcn_readfirstlane((int32_t)divide(g, (uint32_t)S.T, S.T_mul));
    const int32_t tile = __builtin_amdgcn_readfirstlane((int32_t)g - item * S.T);
    const int32_t node = nodes[item];
    trace_tile<kMarginal, kTreeTraceThreads, kSeg>(M, S, Tr, node, tile, depth || Tr.mask_slot[node].x >= 0);
}

// The rays of each node's window yaw[node], counted into total[node].
template <int kSeg>
__global__ __launch_bounds__(kTreeTraceThreads) void k_trace_window(MapDev M, SensorDev S, TreeDev Tr,
                                                                    const int32_t* __restrict__ nodes,
                                                                    const int32_t* __restrict__ yaw,
                                                                    uint32_t* __restrict__ total, bool hits) {
    const uint32_t g = xcd_grouped<kTreeRun>(blockIdx.x, gridDim.x);
    const int32_t item = __builtin_amdgcn_readfirstlane((int32_t)divide(g, (uint32_t)S.T, S.T_mul));
    const int32_t tile = __builtin_amdgcn_readfirstlane((int32_t)g - item * S.T);
    const int32_t node = nodes[item];
    trace_tile<true, kTreeTraceThreads, kSeg, true>(M, S, Tr, node, tile, hits || Tr.mask_slot[node].x >= 0, S.c0_of_win[yaw[node]], total + node);
}

// ---------------------------------------------------------------- window selection

// A level's window selection stands between its trace and its mask builder, so
// its time is the latency of one workgroup's chain of loads: bins, then the
// window's first hits. Hence every load that does not depend on the window is
// requested at once, the scan takes three barriers, a tile's 16 first hits are
// in flight together, and a small level deals a node's tiles (and depth image)
// to several workgroups, which all repeat the selection. With a scan of a
// barrier pair per step and tiles read value by value, 500 nodes in 9 levels took
// 957 us, 920 us so; 20 nodes in 5 levels 97.5 and 89.3 us.
struct FinishLds {
    uint32_t p[2 * kMaxBins + 1];
    uint32_t tot[kThreads / 64];
    unsigned long long best[kThreads / 64];
    int32_t c0[kMaxBins];
};

// Window sums from a prefix sum over the bins taken circularly
// (P[i+1] = P[i] + bins[i mod B], S(k) = P[k+w] - P[k]), then the largest sum
// with the smallest k. Whole workgroup; returns (sum << 32) | (B - 1 - k) to
// every thread, and the window's first column in *c0. Bins are read with atomic
// loads (they were accumulated with device-scope atomics, possibly by other
// workgroups). The workgroup synchronises before it uses `s` again.
__device__ __forceinline__ unsigned long long select_window(const uint32_t* bins, const SensorDev& S, FinishLds& s,
                                                            int32_t* c0) {
    static_assert(2 * kThreads >= 2 * kMaxBins, "two bins a thread");
    const int32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int32_t L = S.B + S.w;   // extended length <= 2 * S.B
    uint32_t v[2];
#pragma unroll
    for (int32_t e = 0; e < 2; ++e) {
        const int32_t i = 2 * tid + e;
        v[e] = i < L ? __hip_atomic_load(&bins[i < S.B ? i : i - S.B], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    }
    if (tid < S.B) s.c0[tid] = S.c0_of_win[tid];
    uint32_t x = v[0] + v[1];
    for (int32_t off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_up(x, off, 64);
        x += lane >= off ? o : 0u;
    }
    if (lane == 63) s.tot[wave] = x;
    __syncthreads();
    for (int32_t i = 0; i < kThreads / 64 - 1; ++i) x += i < wave ? s.tot[i] : 0u;
    if (tid == 0) s.p[0] = 0u;
    s.p[2 * tid + 1] = x - v[1];
    s.p[2 * tid + 2] = x;
    __syncthreads();
    unsigned long long key = 0ull;
    if (tid < S.B) key = ((unsigned long long)(s.p[tid + S.w] - s.p[tid]) << 32) | (uint32_t)(S.B - 1 - tid);
    for (int32_t off = 32; off > 0; off >>= 1) {
        const unsigned long long o = __shfl_xor(key, off, 64);
        key = o > key ? o : key;
    }
    if (lane == 0) s.best[wave] = key;
    __syncthreads();
    unsigned long long best = s.best[0];
    for (int32_t i = 1; i < kThreads / 64; ++i) best = s.best[i] > best ? s.best[i] : best;
    *c0 = s.c0[S.B - 1 - (int32_t)(uint32_t)(best & 0xffffffffull)];
    return best;
}

// The largest and the smallest first hit of each tile of a node's window
// (kTileCols x kTileRows pixels, partial at the window's edges), for the mask
// builder's whole-brick tests of the node's bricks; only nodes with children
// (slot >= 0) have a path mask to build.
// Consecutive threads take consecutive tiles of a tile column, so their reads
// of the column-major panorama are contiguous. A partial tile reads its last
// column and row again instead of stopping early.
__device__ __forceinline__ void tile_max(const SensorDev& S, const TreeDev& Tr, int32_t node, int32_t slot, int32_t c0,
                                         int32_t part, int32_t parts) {
    if (slot < 0) return;
    const float* src = Tr.dpan + (size_t)node * S.R;
    float* dst = Tr.tmax + (size_t)slot * 2 * S.n_tiles;
    for (int32_t t = part * kThreads + (int32_t)threadIdx.x; t < S.n_tiles; t += parts * kThreads) {
        const int32_t tc = t / S.trows, j0 = (t - tc * S.trows) * kTileRows;
        float f[kTileCols][kTileRows];
#pragma unroll
        for (int32_t i = 0; i < kTileCols; ++i) {
            const float* col = src + (size_t)wrap(c0 + min(tc * kTileCols + i, S.WB - 1), S.W) * S.H;
#pragma unroll
            for (int32_t j = 0; j < kTileRows; ++j) f[i][j] = col[min(j0 + j, S.H - 1)];
        }
        float m = 0.f, mn = __builtin_inff();
#pragma unroll
        for (int32_t i = 0; i < kTileCols; ++i)
#pragma unroll
            for (int32_t j = 0; j < kTileRows; ++j) {
                m = fmaxf(m, f[i][j]);
                mn = fminf(mn, f[i][j]);
            }
        dst[t] = m;
        dst[S.n_tiles + t] = mn;
    }
}

// `parts` workgroups per node of a level: gain and window; in marginal mode also
// the node's window start column for its descendants.
__global__ __launch_bounds__(kThreads) void k_finish(SensorDev S, TreeDev Tr, const int32_t* __restrict__ nodes,
                                                     int marginal, uint32_t* __restrict__ gain,
                                                     int32_t* __restrict__ yaw, int32_t parts) {
    __shared__ FinishLds s;
    const int32_t item = (int32_t)(blockIdx.x / (uint32_t)parts), part = (int32_t)blockIdx.x - item * parts;
    const int32_t node = nodes[item];
    const int32_t slot = marginal ? Tr.mask_slot[node].x : -1;
    int32_t c0;
    const unsigned long long best = select_window(Tr.bins + (size_t)node * S.B, S, s, &c0);
    if (threadIdx.x == 0 && part == 0) {
        gain[node] = (uint32_t)(best >> 32);
        yaw[node] = S.B - 1 - (int32_t)(uint32_t)(best & 0xffffffffull);
        if (marginal) Tr.c0[node] = c0;
    }
    tile_max(S, Tr, node, slot, c0, part, parts);
}

// ---------------------------------------------------------------- multi-tree, level by level

// Clears the bins of every tree in a batch. Grid: (blocks, n_trees).
__global__ void k_batch_zero(const BatchTree* __restrict__ trees, int32_t B) {
    const BatchTree& T = trees[blockIdx.y];
    const size_t nb = (size_t)T.td.n * (size_t)B;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < nb; i += (size_t)gridDim.x * blockDim.x)
        T.td.bins[i] = 0u;
}

// One depth level of all trees at once: work item = (tree, node) from
// `items` (tree << 32 | node), T workgroups per item.
template <int kTh, int kSeg>
__global__ __launch_bounds__(kTh) void k_trace_multi(const BatchTree* __restrict__ trees,
                                                     const unsigned long long* __restrict__ items, SensorDev S,
                                                     bool depth) {
    // (workgroup-uniform values kept in scalar registers)
    const uint32_t g = xcd_grouped<kBatchRun>(blockIdx.x, gridDim.x);
    const int32_t item = __builtin_amdgcn_readfirstlane((int32_t)divide(g, (uint32_t)S.T, S.T_mul));
    const int32_t tile = __builtin_amdgcn_readfirstlane((int32_t)g - item * S.T);
    const unsigned long long it = items[item];
    const BatchTree& BT = trees[(uint32_t)(it >> 32)];
    if (BT.status != nullptr && *BT.status != 0) return;      // (the request has failed)
    SensorDev St = S;
    St.rv = BT.rv;
    St.rv2 = BT.rv2;
    const MapDev M = BT.map;     // copies: loaded once, not re-read through the descriptor
    const TreeDev Tr = BT.td;
    const int32_t node = (int32_t)(uint32_t)it;
    trace_tile<true, kTh, kSeg>(M, St, Tr, node, tile, depth || Tr.mask_slot[node].x >= 0);
}

// Path masks of one depth level's nodes with children, all trees at once:
// `chunks` workgroups per item, `bricks` bricks each.
template <bool kFew>
__global__ __launch_bounds__(kFew ? kFewThreads : kBuildThreads) void k_mask_build_multi(const BatchTree* __restrict__ trees,
                                                                    const unsigned long long* __restrict__ items,
                                                                    SensorDev S, int32_t chunks, int32_t bricks, uint32_t chunks_mul) {
    extern __shared__ char smem[];
    __shared__ uint8_t s_live[kMaxBuildBricks];
    __shared__ uint32_t s_cw[kMaxBuildBricks];
    __shared__ uint32_t s_b[kMaxBuildBricks];
    __shared__ int32_t s_any;
    const uint32_t g = xcd_grouped<kBatchRun>(blockIdx.x, gridDim.x);
    const uint32_t item = divide(g, (uint32_t)chunks, chunks_mul);
    const unsigned long long it = items[item];
    const BatchTree& BT = trees[(uint32_t)(it >> 32)];
    if (BT.status != nullptr && *BT.status != 0) return;      // (the request has failed)
    SensorDev St = S;
    St.rv = BT.rv;
    St.rv2 = BT.rv2;
    const MapDev M = BT.map;
    const TreeDev Tr = BT.td;
    build_chunk<kFew>(M, St, Tr, (int32_t)(uint32_t)it, (int32_t)(g - item * (uint32_t)chunks), bricks, smem, s_live, s_cw,
                      s_b, &s_any);
}

// Window selection of one (tree, node) item of a batch: gain, window, the
// window's first column, the depth-cull tile maxima and, when asked for, the
// node's depth buffer. Workgroup `part` of the `parts` that share the item.
__device__ __forceinline__ void finish_item(const BatchTree* __restrict__ trees, unsigned long long it,
                                            const SensorDev& S, const BatchOut& out, FinishLds& s, int32_t part,
                                            int32_t parts) {
    const BatchTree& BT = trees[(uint32_t)(it >> 32)];
    if (BT.status != nullptr && *BT.status != 0) return;      // (the request has failed)
    const int32_t node = (int32_t)(uint32_t)it;
    const int32_t slot = BT.td.mask_slot[node].x;
    int32_t c0;
    const unsigned long long best = select_window(BT.td.bins + (size_t)node * S.B, S, s, &c0);
    if (threadIdx.x == 0 && part == 0) {
        const int32_t k = S.B - 1 - (int32_t)(uint32_t)(best & 0xffffffffull);
        (out.gain ? out.gain + BT.out_off : BT.td.gain)[node] = (uint32_t)(best >> 32);
        (out.gain ? out.yaw + BT.out_off : BT.td.yaw)[node] = k;
        BT.td.c0[node] = c0;
    }
    tile_max(S, BT.td, node, slot, c0, part, parts);
    if (out.depth) {
        const int32_t per = S.H * S.WB;
        const float* src = BT.td.dpan + (size_t)node * S.R;
        float* dst = out.depth + ((size_t)BT.out_off + (size_t)node) * per;
        for (int32_t o = part * kThreads + (int32_t)threadIdx.x; o < per; o += parts * kThreads) {
            const int32_t j = o / S.WB, ii = o - j * S.WB;
            int32_t c = c0 + ii;
            c = c >= S.W ? c - S.W : c;
            dst[o] = src[c * S.H + j];
        }
    }
}

// Window selection for one depth level of all trees: `parts` workgroups per item.
__global__ __launch_bounds__(kThreads) void k_finish_multi(const BatchTree* __restrict__ trees,
                                                           const unsigned long long* __restrict__ items, SensorDev S,
                                                           BatchOut out, int32_t parts) {
    __shared__ FinishLds s;
    const int32_t item = (int32_t)(blockIdx.x / (uint32_t)parts);
    finish_item(trees, items[item], S, out, s, (int32_t)blockIdx.x - item * parts, parts);
}

// ---------------------------------------------------------------- persistent batch

// Barrier over the whole grid of the persistent batch kernel, whose workgroups
// are all resident at once (the cooperative launch refuses a grid that cannot
// be). sync[0] counts arrivals and only grows: after k barriers it reaches
// k * gridDim.x, which each workgroup tracks in *target. A wait that polls
// `spin_limit` times without every workgroup arriving sets sync[1], and every
// workgroup then leaves at its next barrier, so the kernel always ends; the
// host reads sync[1] afterwards. An agent-scope release fence before the
// arrival and an acquire fence after the wait make each phase's writes visible
// to the next phase on every XCD; the polls themselves are relaxed loads, which
// leave the caches of the workgroups still working alone. Returns false once a
// wait has given up.
__device__ bool grid_barrier(uint32_t* sync, uint32_t* target, uint32_t spin_limit, int32_t* s_ok) {
    __syncthreads();
    if (threadIdx.x == 0) {
        *target += gridDim.x;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __hip_atomic_fetch_add(&sync[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int32_t ok = 1;
        for (uint32_t polls = 0;; ++polls) {
            const uint32_t a = __hip_atomic_load(&sync[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((int32_t)(a - *target) >= 0) break;
            if (__hip_atomic_load(&sync[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u || polls >= spin_limit) {
                __hip_atomic_store(&sync[1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ok = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(8);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        *s_ok = ok;
    }
    __syncthreads();
    return *s_ok != 0;
}

// The whole batch in one launch (Sec. IV-C's depth order across all trees):
// for each depth level, every (node, ray tile) is traced, then every node's
// window is chosen, then the path masks of the level's nodes with children
// are built, with a grid barrier after each phase. Work units of a phase are
// dealt to the workgroups in turn (unit = blockIdx.x + k * gridDim.x); every
// workgroup passes every barrier, whether it had units or not.
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_batch_persistent(
    const BatchTree* __restrict__ trees, const unsigned long long* __restrict__ items,
    const int32_t* __restrict__ level_ptr, const unsigned long long* __restrict__ mitems,
    const int32_t* __restrict__ mlevel_ptr, int32_t levels, SensorDev S, BatchOut out, int32_t chunks, int32_t bricks,
    uint32_t* sync, uint32_t spin_limit) {
    extern __shared__ char smem[];
    __shared__ uint8_t s_live[kMaxBuildBricks];
    __shared__ union {                       // (a phase each, a barrier between them)
        FinishLds fin;
        struct { uint32_t cw[kMaxBuildBricks], b[kMaxBuildBricks]; } build;
    } s_u;
    __shared__ int32_t s_any, s_ok;
    uint32_t target = 0;
    const uint32_t G = gridDim.x;
    for (int32_t d = 0; d < levels; ++d) {
        const int32_t i0 = level_ptr[d], n = level_ptr[d + 1] - i0;
        const uint32_t units = (uint32_t)n * (uint32_t)S.T;
        for (uint32_t u = blockIdx.x; u < units; u += G) {
            const int32_t item = __builtin_amdgcn_readfirstlane((int32_t)divide(u, (uint32_t)S.T, S.T_mul));
            const int32_t tile = __builtin_amdgcn_readfirstlane((int32_t)u - item * S.T);
            const unsigned long long it = items[i0 + item];
            const BatchTree& BT = trees[(uint32_t)(it >> 32)];
            if (BT.status == nullptr || *BT.status == 0) {
                SensorDev St = S;
                St.rv = BT.rv;
                St.rv2 = BT.rv2;
                const MapDev M = BT.map;
                const TreeDev Tr = BT.td;
                const int32_t node = (int32_t)(uint32_t)it;
                trace_tile<true, kThreads>(M, St, Tr, node, tile, out.depth != nullptr || Tr.mask_slot[node].x >= 0);
            }
        }
        if (!grid_barrier(sync, &target, spin_limit, &s_ok)) return;
        for (uint32_t u = blockIdx.x; u < (uint32_t)n; u += G) {
            finish_item(trees, items[i0 + (int32_t)u], S, out, s_u.fin, 0, 1);
            __syncthreads();
        }
        if (!grid_barrier(sync, &target, spin_limit, &s_ok)) return;
        const int32_t m0 = mlevel_ptr[d];
        const uint32_t bunits = (uint32_t)(mlevel_ptr[d + 1] - m0) * (uint32_t)chunks;
        for (uint32_t u = blockIdx.x; u < bunits; u += G) {
            const int32_t item = __builtin_amdgcn_readfirstlane((int32_t)(u / (uint32_t)chunks));
            const int32_t chunk = __builtin_amdgcn_readfirstlane((int32_t)u - item * chunks);
            const unsigned long long it = mitems[m0 + item];
            const BatchTree& BT = trees[(uint32_t)(it >> 32)];
            if (BT.status == nullptr || *BT.status == 0) {
                SensorDev St = S;
                St.rv = BT.rv;
                St.rv2 = BT.rv2;
                const MapDev M = BT.map;
                const TreeDev Tr = BT.td;
                build_chunk<false>(M, St, Tr, (int32_t)(uint32_t)it, chunk, bricks, smem, s_live, s_u.build.cw, s_u.build.b, &s_any);
            }
            __syncthreads();
        }
        if (d + 1 < levels && !grid_barrier(sync, &target, spin_limit, &s_ok)) return;
    }
}

// depth[n][j][i] = first hit of ray ((c0[n] + i) mod W, j)
__global__ void k_depth_out(SensorDev S, TreeDev Tr, float* __restrict__ depth) {
    const size_t per = (size_t)S.H * S.WB;
    const size_t total = per * (size_t)Tr.n;
    for (size_t o = blockIdx.x * (size_t)blockDim.x + threadIdx.x; o < total; o += (size_t)gridDim.x * blockDim.x) {
        const int32_t node = (int32_t)(o / per);
        const int32_t rem = (int32_t)(o - (size_t)node * per);
        const int32_t j = rem / S.WB, i = rem - j * S.WB;
        int32_t c = Tr.c0[node] + i;
        c = c >= S.W ? c - S.W : c;
        depth[o] = Tr.dpan[(size_t)node * S.R + (size_t)c * S.H + j];
    }
}

// ---------------------------------------------------------------- launchers

static int grid_for(size_t n, int threads) {
    size_t g = (n + threads - 1) / threads;
    return (int)(g > 65536 ? 65536 : (g < 1 ? 1 : g));
}

hipError_t launch_brick(const uint8_t* dense, uint8_t* bricks, const MapDev& m, hipStream_t s) {
    size_t total = (size_t)m.nbx * m.nby * m.nbz * 512u;
    hipLaunchKernelGGL(k_brick, dim3(grid_for(total, 256)), dim3(256), 0, s, dense, bricks, m);
    return hipGetLastError();
}

hipError_t launch_brick_flags(const MapDev& m, hipStream_t s) {
    const size_t threads = (size_t)(m.mask_words >> 4) * 64u;
    hipLaunchKernelGGL(k_brick_flags, dim3(grid_for(threads, 256)), dim3(256), 0, s, m);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? launch_blocks16(m, s) : e;
}

hipError_t launch_blocks16(const MapDev& m, hipStream_t s) {
    const size_t threads = ((size_t)(m.mbx / 2) * (m.mby / 2) * (m.mbz / 2) + 7) / 8 * 64;    // a wave per 8 blocks
    if (threads == 0) return hipSuccess;
    hipLaunchKernelGGL(k_blocks16, dim3(grid_for(threads, 256)), dim3(256), 0, s, m);
    return hipGetLastError();
}

hipError_t launch_zero_u32(uint32_t* p, size_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero_u32, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

int shape_count() { return kNumShapes; }

// The server's launch shape: one-wave trace workgroups and 256-brick builder
// chunks (its levels hold a few nodes of each request in flight, so small
// trace workgroups and few builder workgroups suit it; measured on 16 robots'
// requests: 9.25 -> 10.3 G rays/s saturated against shape 0).
static constexpr int find_shape(int threads, int bricks) {
    for (int i = 0; i < kNumShapes; ++i)
        if (kShapes[i].threads == threads && kShapes[i].bricks == bricks) return i;
    return 0;
}
int serve_shape() {
    constexpr int k = find_shape(64, 256);
    static_assert(kShapes[k].threads == 64 && kShapes[k].bricks == 256, "the server's shape is compiled");
    return k;
}

void shape_of(int shape, int* threads, int* bricks) {
    *threads = kShapes[shape].threads;
    *bricks = kShapes[shape].bricks;
}

size_t build_lds_bytes(const SensorDev& sd) {
    return sizeof(float2) * (sd.WB + 2) + sizeof(float) * (sd.H + 1) +
           sizeof(uint16_t) * (sd.n_lut_col + sd.n_lut_row);
}

size_t build_lds_total(const SensorDev& sd) { return build_lds_bytes(sd) + kBuildFixedLds; }

size_t lds_limit() {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || v <= 0)
        return 64u * 1024u;
    return (size_t)v;
}

// Lanes per ray of a trace launch: the most that keep it at kSplitWaves waves
// (two rounds of the chip's 8192 wave slots; beyond, the chip is full and the
// stretches after first hits are work lost). Measured (1 lane -> this rule): a
// 20-node tree 121 -> 98 us, 100 nodes 545 -> 510, 333 nodes of short rays
// 623 -> 608, 500 nodes 1006 -> 971, 29000 nodes even; limits of 8192, 12288 and
// 24576 waves: 517, 517 and 520 us for the 100 nodes, 985, 976 and 974 for the 500.
constexpr int64_t kSplitWaves = 16384;
static int trace_segments(const SensorDev& sd, int32_t n_nodes, int32_t columns) {
    const int64_t waves = (int64_t)n_nodes * ((columns + kRayBlockCols - 1) / kRayBlockCols) * sd.nrb;
    for (int seg = 8; seg > 1; seg >>= 1)
        if (waves * seg <= kSplitWaves) return seg;
    return 1;
}

// The sensor as a trace launch over `columns` columns takes it, with `threads`
// lanes a workgroup and `seg` lanes a ray.
static SensorDev trace_sensor(const SensorDev& sd, int seg, int32_t threads, int32_t columns) {
    SensorDev st = sd;
    const int32_t cols = kRayBlockCols / seg;
    st.n_blocks = (columns + cols - 1) / cols * sd.nrb;
    st.T = (st.n_blocks * 64 + threads - 1) / threads;
    st.T_mul = divisor_mul((uint32_t)st.T);
    return st;
}

int32_t tiles_per_node(const SensorDev& sd, int shape) {
    return (sd.n_blocks * 64 + kShapes[shape].threads - 1) / kShapes[shape].threads;
}

hipError_t launch_trace(const MapDev& m, const SensorDev& sd, const TreeDev& td, const int32_t* nodes,
                        int32_t n_nodes, bool marginal, bool depth, hipStream_t s) {
    if (n_nodes <= 0) return hipSuccess;
    const int seg = trace_segments(sd, n_nodes, sd.W);
    const SensorDev st = trace_sensor(sd, seg, kTreeTraceThreads, sd.W);
    const dim3 grid((unsigned)n_nodes * (unsigned)st.T);
    if (marginal) {
        if (seg == 8)
            hipLaunchKernelGGL((k_trace<true, 8>), grid, dim3(kTreeTraceThreads), 0, s, m, st, td, nodes, depth);
        else if (seg == 4)
            hipLaunchKernelGGL((k_trace<true, 4>), grid, dim3(kTreeTraceThreads), 0, s, m, st, td, nodes, depth);
        else if (seg == 2)
            hipLaunchKernelGGL((k_trace<true, 2>), grid, dim3(kTreeTraceThreads), 0, s, m, st, td, nodes, depth);
        else
            hipLaunchKernelGGL((k_trace<true, 1>), grid, dim3(kTreeTraceThreads), 0, s, m, st, td, nodes, depth);
    } else {
        if (seg == 8)
            hipLaunchKernelGGL((k_trace<false, 8>), grid, dim3(kTreeTraceThreads), 0, s, m, st, td, nodes, depth);
        else if (seg == 4)
            hipLaunchKernelGGL((k_trace<false, 4>), grid, dim3(kTreeTraceThreads), 0, s, m, st, td, nodes, depth);
        else if (seg == 2)
            hipLaunchKernelGGL((k_trace<false, 2>), grid, dim3(kTreeTraceThreads), 0, s, m, st, td, nodes, depth);
        else
            hipLaunchKernelGGL((k_trace<false, 1>), grid, dim3(kTreeTraceThreads), 0, s, m, st, td, nodes, depth);
    }
    return hipGetLastError();
}

hipError_t launch_trace_window(const MapDev& m, const SensorDev& sd, const TreeDev& td, const int32_t* nodes,
                               int32_t n_nodes, const int32_t* yaw, uint32_t* total, bool hits,
                               hipStream_t s) {
    if (n_nodes <= 0) return hipSuccess;
    const int seg = trace_segments(sd, n_nodes, sd.WB);
    const SensorDev st = trace_sensor(sd, seg, kTreeTraceThreads, sd.WB);
    const dim3 grid((unsigned)n_nodes * (unsigned)st.T);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(kTreeTraceThreads), 0, s, m, st, td, nodes, yaw, total, hits); };
    if (seg == 8)
        go(k_trace_window<8>);
    else if (seg == 4)
        go(k_trace_window<4>);
    else if (seg == 2)
        go(k_trace_window<2>);
    else
        go(k_trace_window<1>);
    return hipGetLastError();
}

// Bricks per builder workgroup of one launch: `most`, halved while the launch
// has fewer than kBuildFill workgroups (16 per CU: two rounds of the eight
// resident ones), down to one block of 2x2x2 bricks. A level of few nodes is
// bound by the longest workgroup's serial brick tests, so it takes many short
// workgroups; a level of many nodes by work per workgroup. Measured against 64
// bricks for all small launches: a 20-node tree 145 -> 121 us, 100 nodes
// 564 -> 545, 500 nodes 1031 -> 1004 (fills of 1024, 2048 and 8192: 1098, 1018
// and 1028), 12000 nodes even.
constexpr int64_t kBuildFill = 4096;
static int32_t build_bricks(uint32_t slots, int32_t n_nodes, int32_t most) {
    int32_t bricks = most;
    while (bricks > 8 && (int64_t)n_nodes * ((slots + (uint32_t)bricks - 1u) / (uint32_t)bricks) < kBuildFill) bricks >>= 1;
    return bricks;
}
// A launch of chunks of one block of bricks whose workgroups are all resident at
// once even with a wave per brick (1024 of 8 waves fill the chip): bound by one
// workgroup's chain of loads, so each brick gets a wave of its own, 8 lanes share
// a brick's view, and the tables are requested at the start, needed or not. 20
// nodes in 4 levels (up to 160 workgroups a launch): 109 to 112 us with four waves,
// 97 to 104 so (four processes each; lanes 16 or 1024 threads are even); 500 nodes,
// of whose levels one is that small, are even (887 and 884). Larger launches lose by it: with chunks of up
// to 16 and 32 bricks in 8 waves the 500 nodes take 954 and 971 us against 920.
constexpr uint64_t kFewChunks = 1024;
static bool few_chunks(uint64_t chunks, int32_t bricks) { return bricks == 8 && chunks <= kFewChunks; }
constexpr int32_t kTreeBuildBricks = 256;     // the most a per-tree level takes

hipError_t launch_mask_build(const MapDev& m, const SensorDev& sd, const TreeDev& td, const int32_t* nodes,
                             int32_t n_nodes, hipStream_t s) {
    if (n_nodes <= 0) return hipSuccess;
    const int32_t bricks = build_bricks(m.build_slots, n_nodes, kTreeBuildBricks);
    const int32_t chunks = (int32_t)((m.build_slots + (uint32_t)bricks - 1u) / (uint32_t)bricks);
    const size_t lds = build_lds_bytes(sd);
    if (lds + kBuildFixedLds > lds_limit()) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)n_nodes * (unsigned)chunks);
    const uint32_t mul = divisor_mul((uint32_t)chunks);
    if (few_chunks(grid.x, bricks))
        hipLaunchKernelGGL(k_mask_build<true>, grid, dim3(kFewThreads), lds, s, m, sd, td, nodes, chunks, bricks, mul);
    else
        hipLaunchKernelGGL(k_mask_build<false>, grid, dim3(kBuildThreads), lds, s, m, sd, td, nodes, chunks, bricks, mul);
    return hipGetLastError();
}

// Workgroups that share a node's window selection: one tile a thread, while the
// launch stays within kFinishFill workgroups. 500 nodes of 345 tiles (two
// workgroups for levels of up to 512): 887 to 893 us with one each, 881 to 889 so,
// 100 nodes 560 to 562 and 554 to 558 (four processes each), 20 nodes even; up to
// 4096 workgroups gains nothing more and repeats selections that fill the chip anyway
// (16 trees of up to 2000 nodes: 8.45 and 8.54 ms).
constexpr int32_t kFinishFill = 1024;
static int32_t finish_parts(const SensorDev& sd, int32_t n_items, bool tiles) {
    const int32_t work = tiles ? (sd.n_tiles + kThreads - 1) / kThreads : 1;
    return std::max(std::min(work, kFinishFill / n_items), 1);
}

hipError_t launch_finish(const SensorDev& sd, const TreeDev& td, const int32_t* nodes, int32_t n_nodes,
                         bool marginal, uint32_t* gain, int32_t* yaw, hipStream_t s) {
    if (n_nodes <= 0) return hipSuccess;
    const int32_t parts = finish_parts(sd, n_nodes, marginal);
    hipLaunchKernelGGL(k_finish, dim3((unsigned)(n_nodes * parts)), dim3(kThreads), 0, s, sd, td, nodes,
                       marginal ? 1 : 0, gain, yaw, parts);
    return hipGetLastError();
}

hipError_t launch_depth_out(const SensorDev& sd, const TreeDev& td, float* depth, hipStream_t s) {
    size_t total = (size_t)sd.H * sd.WB * td.n;
    hipLaunchKernelGGL(k_depth_out, dim3(grid_for(total, 256)), dim3(256), 0, s, sd, td, depth);
    return hipGetLastError();
}

// ---------------------------------------------------------------- path score (eq. 3, eq. 4)

// Traversal cost (eq. 3) and exponential objective (eq. 4) of one node, summed
// from the root down its ancestor list (nearest first, so walked backwards) in
// the order the recursions take: c += |p_m - p_prev| and
// o += g(m) v^3 exp(-lambda c), in float64 on the float32 positions in metres.
__device__ __forceinline__ void score_node(const BatchTree& T, const uint32_t* __restrict__ g, int32_t node,
                                           double lambda, double* c_out, double* o_out) {
    const int32_t a0 = T.td.anc_ptr[node], a1 = T.td.anc_ptr[node + 1];
    int32_t prev = a1 > a0 ? T.td.anc_ids[a1 - 1] : node;      // the root
    double c = 0.0;
    double o = (double)g[prev] * T.vox3;
    for (int32_t k = a1 - 2; k >= a0 - 1; --k) {
        const int32_t m = k >= a0 ? T.td.anc_ids[k] : node;
        const float4 pa = T.td.pm[prev], pb = T.td.pm[m];
        const double dx = (double)pb.x - (double)pa.x;
        const double dy = (double)pb.y - (double)pa.y;
        const double dz = (double)pb.z - (double)pa.z;
        c = c + sqrt(dx * dx + dy * dy + dz * dz);
        o = o + (double)g[m] * T.vox3 * exp(-lambda * c);
        prev = m;
    }
    *c_out = c;
    *o_out = o;
}

// One thread per node of one tree (grid: blocks x trees).
__global__ void k_score(const BatchTree* __restrict__ trees, const uint32_t* __restrict__ gain, double lambda,
                        double* __restrict__ cost, double* __restrict__ obj) {
    const BatchTree& T = trees[blockIdx.y];
    const int32_t node = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
    if (node >= T.td.n) return;
    double c, o;
    score_node(T, gain + T.out_off, node, lambda, &c, &o);
    if (cost) cost[T.out_off + node] = c;
    obj[T.out_off + node] = o;
}

// Whole workgroup: the node of largest objective among the threads'
// candidates (bo, bi), smallest id on ties, written to best[tree]; and (if
// asked) its root path, root first, padded with -1.
__device__ __forceinline__ void best_and_branch(const BatchTree& T, double bo, int32_t bi, int32_t tree,
                                                int32_t* __restrict__ best, int32_t* __restrict__ branch) {
    __shared__ double s_o[kThreads];
    __shared__ int32_t s_i[kThreads];
    s_o[threadIdx.x] = bo;
    s_i[threadIdx.x] = bi;
    __syncthreads();
    for (int32_t off = kThreads / 2; off > 0; off >>= 1) {
        if ((int32_t)threadIdx.x < off) {
            const double po = s_o[threadIdx.x + off];
            const int32_t pi = s_i[threadIdx.x + off];
            const double mo = s_o[threadIdx.x];
            const int32_t mi = s_i[threadIdx.x];
            if (pi >= 0 && (mi < 0 || po > mo || (po == mo && pi < mi))) {
                s_o[threadIdx.x] = po;
                s_i[threadIdx.x] = pi;
            }
        }
        __syncthreads();
    }
    const int32_t b = s_i[0];
    if (threadIdx.x == 0) best[tree] = b;
    if (branch && threadIdx.x < kMaxAnc + 1) {
        const int32_t a0 = T.td.anc_ptr[b], d = T.td.anc_ptr[b + 1] - a0;     // ancestors, nearest first
        const int32_t t = (int32_t)threadIdx.x;
        branch[(size_t)tree * (kMaxAnc + 1) + t] = t < d ? T.td.anc_ids[a0 + d - 1 - t] : t == d ? b : -1;
    }
}

// One workgroup per tree: argmax over the objectives k_score wrote.
__global__ __launch_bounds__(kThreads) void k_best(const BatchTree* __restrict__ trees,
                                                   const double* __restrict__ obj, int32_t* __restrict__ best,
                                                   int32_t* __restrict__ branch) {
    const BatchTree& T = trees[blockIdx.x];
    const double* o = obj + T.out_off;
    double bo = 0.0;
    int32_t bi = -1;
    for (int32_t i = threadIdx.x; i < T.td.n; i += kThreads)
        if (bi < 0 || o[i] > bo) {           // ids ascend, so a later equal value never wins
            bo = o[i];
            bi = i;
        }
    best_and_branch(T, bo, bi, (int32_t)blockIdx.x, best, branch);
}

// Small trees: score and argmax in one launch, one workgroup per tree.
__global__ __launch_bounds__(kThreads) void k_score_best(const BatchTree* __restrict__ trees,
                                                         const uint32_t* __restrict__ gain, double lambda,
                                                         double* __restrict__ cost, double* __restrict__ obj,
                                                         int32_t* __restrict__ best, int32_t* __restrict__ branch) {
    const BatchTree& T = trees[blockIdx.x];
    double bo = 0.0;
    int32_t bi = -1;
    for (int32_t i = threadIdx.x; i < T.td.n; i += kThreads) {
        double c, o;
        score_node(T, gain + T.out_off, i, lambda, &c, &o);
        if (cost) cost[T.out_off + i] = c;
        obj[T.out_off + i] = o;
        if (bi < 0 || o > bo) {
            bo = o;
            bi = i;
        }
    }
    best_and_branch(T, bo, bi, (int32_t)blockIdx.x, best, branch);
}

// Trees of up to kFuseNodes nodes take the single-launch kernel.
constexpr uint32_t kFuseNodes = 8192;

hipError_t launch_score(const BatchTree* trees, int32_t n_trees, uint32_t max_nodes, const uint32_t* gain,
                        double lambda, double* cost, double* obj, int32_t* best, int32_t* branch, hipStream_t s) {
    if (max_nodes <= kFuseNodes) {
        hipLaunchKernelGGL(k_score_best, dim3((unsigned)n_trees), dim3(kThreads), 0, s, trees, gain, lambda, cost, obj,
                           best, branch);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_score, dim3((unsigned)grid_for(max_nodes, 256), (unsigned)n_trees), dim3(256), 0, s, trees,
                       gain, lambda, cost, obj);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_best, dim3((unsigned)n_trees), dim3(kThreads), 0, s, trees, obj, best, branch);
    return hipGetLastError();
}

}  // namespace mgk

namespace mgk {

hipError_t launch_batch_zero(const BatchTree* trees, int32_t n_trees, uint32_t max_nodes, const SensorDev& sd,
                             hipStream_t s) {
    const uint32_t blocks = (uint32_t)grid_for((size_t)max_nodes * sd.B, 256);
    hipLaunchKernelGGL(k_batch_zero, dim3(blocks, (unsigned)n_trees), dim3(256), 0, s, trees, sd.B);
    return hipGetLastError();
}

namespace {

template <int kTh>
void launch_multi(const BatchTree* trees, const unsigned long long* items, int32_t n_items, const SensorDev& sd,
                  bool depth, hipStream_t s, hipEvent_t t0, hipEvent_t t1) {
    const int seg = trace_segments(sd, n_items, sd.W);
    const SensorDev st = trace_sensor(sd, seg, seg > 1 ? 64 : kTh, sd.W);
    const dim3 grid((unsigned)n_items * (unsigned)st.T);
    auto go = [&](auto kernel, int threads) {
        if (t0 && t1)
            hipExtLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, t0, t1, 0u, trees, items, st, depth);
        else
            hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, trees, items, st, depth);
    };
    if (seg == 8)
        go(k_trace_multi<64, 8>, 64);
    else if (seg == 4)
        go(k_trace_multi<64, 4>, 64);
    else if (seg == 2)
        go(k_trace_multi<64, 2>, 64);
    else
        go(k_trace_multi<kTh, 1>, kTh);
}

template <int I>
void launch_multi_shape(int shape, const BatchTree* trees, const unsigned long long* items, int32_t n_items,
                        const SensorDev& sd, bool depth, hipStream_t s, hipEvent_t t0, hipEvent_t t1) {
    if constexpr (I < kNumShapes) {
        if (shape == I)
            launch_multi<kShapes[I].threads>(trees, items, n_items, sd, depth, s, t0, t1);
        else
            launch_multi_shape<I + 1>(shape, trees, items, n_items, sd, depth, s, t0, t1);
    }
}

}  // namespace

hipError_t launch_batch_level(const BatchTree* trees, const unsigned long long* items, int32_t n_items,
                              const unsigned long long* mitems, int32_t n_mitems, uint32_t mask_bricks,
                              const SensorDev& sd, const BatchOut& out, hipStream_t s, int shape, hipEvent_t t0, hipEvent_t t1,
                              hipEvent_t b0, hipEvent_t b1) {
    if (n_items <= 0) return hipSuccess;
    if (shape < 0 || shape >= kNumShapes) return hipErrorInvalidValue;
    const size_t lds = build_lds_bytes(sd);
    if (lds + kBuildFixedLds > lds_limit()) return hipErrorInvalidConfiguration;
    launch_multi_shape<0>(shape, trees, items, n_items, sd, out.depth != nullptr, s, t0, t1);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int32_t parts = finish_parts(sd, n_items, n_mitems > 0);
    hipLaunchKernelGGL(k_finish_multi, dim3((unsigned)(n_items * parts)), dim3(kThreads), 0, s, trees, items, sd, out,
                       parts);
    e = hipGetLastError();
    if (e != hipSuccess || n_mitems <= 0) return e;
    const int32_t bricks = build_bricks(mask_bricks, n_mitems, kShapes[shape].bricks);
    const int32_t chunks = (int32_t)((mask_bricks + (uint32_t)bricks - 1) / (uint32_t)bricks);
    if ((uint64_t)n_mitems * (uint64_t)chunks >= (1ull << 32)) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)n_mitems * (unsigned)chunks);
    const uint32_t mul = divisor_mul((uint32_t)chunks);
    const bool few = few_chunks(grid.x, bricks);
    const auto kernel = few ? k_mask_build_multi<true> : k_mask_build_multi<false>;
    const dim3 threads(few ? kFewThreads : kBuildThreads);
    if (b0 && b1)
        hipExtLaunchKernelGGL(kernel, grid, threads, lds, s, b0, b1, 0u, trees, mitems, sd, chunks, bricks, mul);
    else
        hipLaunchKernelGGL(kernel, grid, threads, lds, s, trees, mitems, sd, chunks, bricks, mul);
    return hipGetLastError();
}

hipError_t persistent_grid(const SensorDev& sd, int32_t* grid) {
    int dev = 0, cus = 0, coop = 0, per_cu = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev);
    if (e != hipSuccess) return e;
    if (!coop) return hipErrorNotSupported;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_batch_persistent, kThreads, build_lds_bytes(sd));
    if (e != hipSuccess) return e;
    if (per_cu < 1 || cus < 1) return hipErrorInvalidConfiguration;
    *grid = per_cu * cus;
    return hipSuccess;
}

hipError_t launch_batch_persistent(const BatchTree* trees, const unsigned long long* items, const int32_t* level_ptr,
                                   const unsigned long long* mitems, const int32_t* mlevel_ptr, int32_t levels,
                                   uint32_t mask_bricks, const SensorDev& sd, const BatchOut& out, uint32_t* sync,
                                   uint32_t spin_limit, hipStream_t s) {
    if (levels <= 0) return hipSuccess;
    const size_t lds = build_lds_bytes(sd);
    if (lds + kBuildFixedLds > lds_limit()) return hipErrorInvalidConfiguration;
    int32_t grid = 0;
    hipError_t e = persistent_grid(sd, &grid);
    if (e != hipSuccess) return e;
    SensorDev st = sd;
    st.T = tiles_per_node(sd, 0);
    st.T_mul = divisor_mul((uint32_t)st.T);
    int32_t bricks = kShapes[0].bricks;
    int32_t chunks = (int32_t)((mask_bricks + (uint32_t)bricks - 1) / (uint32_t)bricks);
    e = launch_zero_u32(sync, 2, s);
    if (e != hipSuccess) return e;
    void* args[] = {(void*)&trees, (void*)&items, (void*)&level_ptr, (void*)&mitems, (void*)&mlevel_ptr,
                    (void*)&levels, (void*)&st, (void*)&out, (void*)&chunks, (void*)&bricks, (void*)&sync, (void*)&spin_limit};
    e = hipLaunchCooperativeKernel((const void*)k_batch_persistent, dim3((unsigned)grid), dim3(kThreads), args, lds, s);
    if (e != hipSuccess) return e;
    return hipGetLastError();
}

}  // namespace mgk
