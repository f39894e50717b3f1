// Internal device-side descriptors shared by the kernels and the host API.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace mgk {

constexpr int kThreads = 256;      // rays per workgroup (4 wave64)
constexpr int kMaxAnc = 64;        // deepest supported ancestor chain
constexpr int kMaxBins = 256;      // yaw bins
constexpr int kMaxAz = 4096;       // panorama columns (LDS holds their boundaries)
constexpr int kMaxEl = 2048;
constexpr int kRayBlockCols = 16;  // pixel block of one wave of the trace kernels: 16 columns
constexpr int kRayBlockRows = 4;   // by 4 rows
constexpr int kTileCols = 4;       // depth-cull tiles of a node's window: 4 columns
constexpr int kTileRows = 4;       // by 4 rows

// kOutside marks the padding around the grid: a traversal that reaches it
// has left the grid. The low two bits of a byte are the state, and bit 1 set
// (kOccupied, kOutside) ends a traversal. Bits 2-4 of an unknown or a free
// voxel name the largest aligned block around it that holds that state only
// (the traversal may cross such a block in one step): 1 its 16x16x16 block
// of 8 bricks, 2 its 8x8x8 brick (kUnknownBrick, kFreeBrick), 3 its 4x4x4
// quarter brick, 4 (free voxels only) its 2x2x2 block, 0 none; the block's
// edge is 32 >> level voxels.
enum : uint8_t { kUnknown = 0, kFree = 1, kOccupied = 2, kOutside = 3, kUnknownBrick = 8, kFreeBrick = 9 };
constexpr uint32_t kLevelShift = 2, kLevelMask = 7;
// (block edge - 1) of level l in bits 4 l .. 4 l + 3: 0, 15, 7, 3, 1 (a byte's
// level field, in place at bit 2, is the shift)
constexpr uint32_t kEdgeOfLevel = 0x137f0u;
__host__ __device__ inline bool is_unknown(uint32_t s) { return (s & 3u) == 0u; }

// The block levels of one brick's voxels up to the brick (levels 2 to 4; the
// 16x16x16 blocks are marked afterwards, from the bricks' summaries), by one
// wave: each lane holds the 8 voxels (x = 0..7, bytes 0..7 of v) of row
// (y, z) = (lane & 7, lane >> 3) of the brick, as states or as marked bytes;
// returns them marked. any_unk, all_unk, all_free: whether the brick holds an
// unknown voxel, only unknown voxels, only free voxels.
__device__ __forceinline__ uint64_t mark_brick_row(uint64_t v, uint32_t lane, bool* any_unk, bool* all_unk,
                                                   bool* all_free_out) {
    const uint64_t ones = 0x0101010101010101ull;
    const uint64_t s8 = v & (3ull * ones);                       // the states, a byte each
    // (a byte is unknown when it is zero: states are below 0x80, so the borrow test is exact)
    const bool row_unk = ((s8 - ones) & ~s8 & (0x80ull * ones)) != 0ull;
    const bool all_free = __builtin_amdgcn_ballot_w64(s8 != ones) == 0ull;
    *all_free_out = all_free;
    *all_unk = __builtin_amdgcn_ballot_w64(s8 != 0ull) == 0ull;
    *any_unk = __builtin_amdgcn_ballot_w64(row_unk) != 0ull;
    if (all_free | *all_unk) return s8 | ((uint64_t)(2u << kLevelShift) * ones);   // (the whole brick: level 2)
    uint32_t fb = 0u, ub = 0u;          // per byte: free, unknown
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t s = (uint32_t)(s8 >> (8 * k)) & 0xffu;
        fb |= (s == kFree ? 1u : 0u) << k;
        ub |= (s == kUnknown ? 1u : 0u) << k;
    }
    // quarter bricks: x halves of the row, over the 4x4 rows (y, z) of the lane's quarter
    const uint32_t y = lane & 7u, z = lane >> 3;
    const uint64_t quarter = (0x0f0f0f0full << (y & 4u)) << (8u * (z & 4u));
    const uint64_t nf_lo = __builtin_amdgcn_ballot_w64((fb & 0x0fu) != 0x0fu), nf_hi = __builtin_amdgcn_ballot_w64((fb & 0xf0u) != 0xf0u);
    const uint64_t nu_lo = __builtin_amdgcn_ballot_w64((ub & 0x0fu) != 0x0fu), nu_hi = __builtin_amdgcn_ballot_w64((ub & 0xf0u) != 0xf0u);
    // 2x2x2 blocks: x pairs of the row, over the 2x2 rows of the lane's pair of rows
    const uint64_t pairs = 0x303ull << ((y & 6u) + 8u * (z & 6u));
    uint32_t f2 = 0u;                   // bit p: x pair p of this row lies in a wholly free block
#pragma unroll
    for (int p = 0; p < 4; ++p)
        f2 |= ((__builtin_amdgcn_ballot_w64(((fb >> (2 * p)) & 3u) != 3u) & pairs) == 0ull ? 1u : 0u) << p;
    const bool f4lo = (nf_lo & quarter) == 0ull, f4hi = (nf_hi & quarter) == 0ull;
    const bool u4lo = (nu_lo & quarter) == 0ull, u4hi = (nu_hi & quarter) == 0ull;
    uint64_t out = 0ull;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint32_t s = (uint32_t)(v >> (8 * k)) & 3u;
        const bool f4 = k < 4 ? f4lo : f4hi, u4 = k < 4 ? u4lo : u4hi;
        uint32_t lv = 0u;
        if (s == kFree) lv = f4 ? 3u : (((f2 >> (k >> 1)) & 1u) ? 4u : 0u);
        if (s == kUnknown) lv = u4 ? 3u : 0u;
        out |= (uint64_t)(s | (lv << kLevelShift)) << (8 * k);
    }
    return out;
}

// Per brick of a path mask (one byte): its 512 bits are mixed, all clear (no
// voxel of the brick observed) or all set. Only unknown voxels' bits are ever
// read, so a mask keeps its code current for every brick that holds an
// unknown voxel, and its 16 words for such a brick whenever they can be read:
// the code is mixed, or the brick also holds known voxels (unknown voxels of
// such a brick are looked up by word, without the code). Words of bricks
// without unknown voxels, and of wholly unknown bricks with a uniform code,
// are never written.
enum : uint8_t { kMaskMixed = 0, kMaskNone = 1, kMaskAll = 2 };
// A brick's code word: bits 0-1 the code of its 512 bits, bits 2 + 2q and
// 3 + 2q the code of its quarter q (the 4x4x4 voxels with (x & 4, y & 4, z & 4)
// = 4 * (q & 1, (q >> 1) & 1, q >> 2)), bits 18-19 the code of its block of
// 2x2x2 bricks when those are all wholly unknown (else mixed).
__host__ __device__ inline uint32_t uniform_code_word(uint32_t c) { return c * 0x15555u; }
// brick_unk values (bits 0-1): no unknown voxel, some, all 512 (the
// kUnknownBrick marks); bit 2 (kBrickAllFree) set when all 512 are free
enum : uint8_t { kBrickKnown = 0, kBrickSomeUnknown = 1, kBrickAllUnknown = 2, kBrickAllFree = 4 };
__device__ __forceinline__ uint8_t brick_summary(bool any_unk, bool all_unk, bool all_free) {
    return (uint8_t)((any_unk ? (all_unk ? kBrickAllUnknown : kBrickSomeUnknown) : kBrickKnown) |
                     (all_free ? kBrickAllFree : 0));
}

// Division by a count that the host knows, exact for every n: `mul` falls short of
// 2^32 / d by less than 1, so the product's high word is the quotient or one less. (A
// variable divisor costs a wave some 30 instructions before its first step.)
inline uint32_t divisor_mul(uint32_t d) { return d > 1u ? (uint32_t)((1ull << 32) / d) : ~0u; }
__device__ __forceinline__ uint32_t divide(uint32_t n, uint32_t d, uint32_t mul) {
    const uint32_t q = __umulhi(n, mul);
    return q + (n - q * d >= d ? 1u : 0u);
}

// Occupancy grid in 8x8x8-voxel bricks (512 B each, x fastest inside a
// brick, bricks x fastest): a ray stays inside one brick for several steps,
// so its gathers hit few cache lines. Brick counts are powers of two with at
// least one padding voxel past the grid on every axis, so a voxel's byte
// address is a bit-field merge of its coordinates; coordinate -1 wraps to the
// last padding voxel of its axis, which holds kOutside like all padding.
struct MapDev {
    const uint8_t* bricks;
    int32_t nx, ny, nz;     // true extent in voxels
    int32_t nbx, nby, nbz;  // bricks per axis (powers of two, 8 * nb > n)
    uint32_t xm, ym, zm;    // brick-index bits of a coordinate: (8 * nb - 1) & ~7
    uint32_t shy, shz;      // left shifts placing (y & ym) and (z & zm) in the address
    uint32_t outside;       // address of a padding byte (kOutside)
    // Path masks (one bit per voxel, see mask_word): bricks per axis holding
    // the grid, ceil(n / 8), and 32-bit words per mask (16 per brick).
    uint32_t mbx, mby, mbz;
    uint32_t mask_words;
    // The mask builder visits bricks by blocks of 2x2x2 (ceil(mb / 2) blocks per
    // axis, x fastest; in a block x, then y, then z): slots = 8 * blocks.
    uint32_t build_slots;
    uint32_t mbx2, mby2, mbx2_mul, mby2_mul;   // blocks along x and y, and their divisor_mul
    // [mbx * mby * mbz] per mask brick: kBrickKnown, kBrickSomeUnknown or
    // kBrickAllUnknown, with kBrickAllFree (kept current, with the block
    // marks, by every write of the map's states)
    uint8_t* brick_unk;
};

// Byte address of voxel (x, y, z) in the bricked grid, for -1 <= x <= nx
// (likewise y, z): bits 0-8 are the position inside the brick, then the brick
// index x-fastest.
__host__ __device__ inline uint32_t voxel_addr(int32_t x, int32_t y, int32_t z, const MapDev& M) {
    const uint32_t ux = (uint32_t)x, uy = (uint32_t)y, uz = (uint32_t)z;
    return (ux & 7u) | ((uy & 7u) << 3) | ((uz & 7u) << 6) | ((ux & M.xm) << 6) | ((uy & M.ym) << M.shy) |
           ((uz & M.zm) << M.shz);
}

// Path masks: one bit per voxel of the grid, in 8x8x8 bricks of 512 bits (16
// words), bricks x fastest with tight counts mbx = ceil(nx / 8) etc. Voxel
// (x, y, z) is bit (x & 7) | (y & 3) << 3 of word (z & 7) << 1 | (y & 7) >> 2
// of its brick, i.e. bit (x & 7) | (y & 7) << 3 | (z & 7) << 6 of the brick's
// 512 bits: a z-slice of a brick is 64 consecutive bits, two words.
__device__ __forceinline__ uint32_t mask_word(int32_t x, int32_t y, int32_t z, const MapDev& M) {
    const uint32_t b = (uint32_t)(x >> 3) + __umul24(M.mbx, (uint32_t)(y >> 3) + __umul24(M.mby, (uint32_t)(z >> 3)));
    return (b << 4) | ((uint32_t)(z & 7) << 1) | ((uint32_t)(y & 4) >> 2);
}
__device__ __forceinline__ uint32_t mask_bit(int32_t x, int32_t y) { return (uint32_t)(x & 7) | ((uint32_t)(y & 3) << 3); }
__device__ __forceinline__ uint32_t mask_brick(int32_t x, int32_t y, int32_t z, const MapDev& M) {
    return (uint32_t)(x >> 3) + __umul24(M.mbx, (uint32_t)(y >> 3) + __umul24(M.mby, (uint32_t)(z >> 3)));
}

// The mask brick of build slot `sl` (past the grid's bricks in a partial block).
__device__ __forceinline__ uint3 slot_brick(uint32_t sl, const MapDev& M) {
    const uint32_t blk = sl >> 3, row = divide(blk, M.mbx2, M.mbx2_mul), bz = divide(row, M.mby2, M.mby2_mul);
    return make_uint3(2u * (blk - row * M.mbx2) + (sl & 1u), 2u * (row - bz * M.mby2) + ((sl >> 1) & 1u),
                      2u * bz + ((sl >> 2) & 1u));
}

// A ray walked by the Amanatides-Woo 3D DDA (face-crossing parameters recomputed
// as (boundary - q) * (1/d); ties step x, then y, then z), an aligned block at a
// time.
//
// Mirrored coordinates: on an axis the ray moves down, the coordinate is
// negated (voxel index x becomes ~x, boundary b becomes -b), so every ray moves
// up on every axis. The parameter (boundary - q) * (1/d) is the same float
// either way (negating both factors is exact), but for the sign of a zero. A
// voxel's byte address merges bit fields of its coordinates, so the mirroring is
// undone by one exclusive or of the merged address.
//
// One step leaves the aligned block of `edge` voxels around the voxel (edge 1:
// the voxel itself), through the face whose boundary parameter T comes first
// (ties x, y, z), and then every axis has crossed the boundaries that come
// before that crossing in the DDA's order: those with parameter below T, or
// equal to T on the exit axis and the axes before it. An axis's position at T
// is q + T d; the error of that sum is below 0.01 voxel (|q| <= 8192, T at most
// the grid's diagonal, three roundings of T and one of the sum), so every
// boundary but the one nearest to it lies at least 0.49 voxel away and its side
// of T is not in doubt, and the nearest one is decided by its own parameter,
// computed as the single step computes it. (A boundary the ray starts on or has
// passed is never crossed again: the coordinate does not fall.) A single voxel is
// the same step with edge 1. Where states change from voxel to voxel and no block
// is marked, that is more work than a step of one axis: 200 nodes on states drawn
// voxel by voxel, the absolute pass, 412 us with a single-voxel step of its own and
// 640 so (with ancestors 1306 and 1385); a branch for waves of single voxels takes
// 535 and 1267 there and 1 to 3 % longer on maps of rooms and walls.
struct RayWalk {
    int32_t mx, my, mz;      // 0, or ~0 on an axis the ray moves down
    float qx, qy, qz;        // the node, mirrored
    float dx, dy, dz;        // the direction's magnitudes
    float fx, fy, fz;        // their inverses; +inf on an axis the ray does not move along: its
                             // next boundary lies past the node, so its parameter is +inf
    int32_t ux, uy, uz;      // the voxel, mirrored
    uint32_t mirror;         // the address bits of the mirrored axes
    __device__ __forceinline__ void start(float4 p, float4 d, float4 iv, const MapDev& M) {
        const float inf = __builtin_inff();
        mx = d.x < 0.f ? -1 : 0; my = d.y < 0.f ? -1 : 0; mz = d.z < 0.f ? -1 : 0;
        qx = mx ? -p.x : p.x; qy = my ? -p.y : p.y; qz = mz ? -p.z : p.z;
        dx = fabsf(d.x); dy = fabsf(d.y); dz = fabsf(d.z);
        fx = dx != 0.f ? fabsf(iv.x) : inf; fy = dy != 0.f ? fabsf(iv.y) : inf; fz = dz != 0.f ? fabsf(iv.z) : inf;
        ux = (int32_t)floorf(p.x) ^ mx; uy = (int32_t)floorf(p.y) ^ my; uz = (int32_t)floorf(p.z) ^ mz;
        mirror = voxel_addr(mx, my, mz, M);
    }
    __device__ __forceinline__ int32_t x() const { return ux ^ mx; }
    __device__ __forceinline__ int32_t y() const { return uy ^ my; }
    __device__ __forceinline__ int32_t z() const { return uz ^ mz; }
    __device__ __forceinline__ uint32_t addr(const MapDev& M) const { return voxel_addr(ux, uy, uz, M) ^ mirror; }
    __device__ __forceinline__ bool in_grid(const MapDev& M) const {
        return (uint32_t)x() < (uint32_t)M.nx && (uint32_t)y() < (uint32_t)M.ny && (uint32_t)z() < (uint32_t)M.nz;
    }
    // Crosses, from the ray's start or from where it stands, every boundary whose
    // parameter is at most ax, ay, az on its axis, those near the parameter `at`.
    __device__ __forceinline__ void pass(float at, float ax, float ay, float az) {
        const float ex = __builtin_rintf(__builtin_fmaf(at, dx, qx));
        const float ey = __builtin_rintf(__builtin_fmaf(at, dy, qy));
        const float ez = __builtin_rintf(__builtin_fmaf(at, dz, qz));
        ux = max(ux, (int32_t)ex - ((ex - qx) * fx <= ax ? 0 : 1));
        uy = max(uy, (int32_t)ey - ((ey - qy) * fy <= ay ? 0 : 1));
        uz = max(uz, (int32_t)ez - ((ez - qz) * fz <= az ? 0 : 1));
    }
    // The parameter at which the aligned block of e1 + 1 voxels a side is left.
    __device__ __forceinline__ float exit(uint32_t e1) const {
        const float Tx = ((float)((ux | (int32_t)e1) + 1) - qx) * fx;
        const float Ty = ((float)((uy | (int32_t)e1) + 1) - qy) * fy;
        const float Tz = ((float)((uz | (int32_t)e1) + 1) - qz) * fz;
        return fminf(fminf(Tx, Ty), Tz);
    }
    // Leaves the aligned block of e1 + 1 voxels a side and returns the parameter T
    // at which it is left. Where the walk's end lies inside the block (T is not
    // below it), only boundaries with a parameter below the end are crossed. before
    // and most: the float below the end (> 0), as bits and as a float.
    __device__ __forceinline__ float cross(uint32_t e1, int32_t before, float most) {
        // the block's exit boundary and its parameter on each axis; the first one
        const float Tx = ((float)((ux | (int32_t)e1) + 1) - qx) * fx;
        const float Ty = ((float)((uy | (int32_t)e1) + 1) - qy) * fy;
        const float Tz = ((float)((uz | (int32_t)e1) + 1) - qz) * fz;
        const float Txy = fminf(Tx, Ty), T = fminf(Txy, Tz);
        // (T >= +0; below 0 there is no parameter: a NaN, which none is at most)
        const float at = fminf(T, most);
        const int32_t tb = (int32_t)__float_as_uint(T) - 1;
        const float below = __uint_as_float((uint32_t)(tb < before ? tb : before));
        pass(at, at, Tx == T ? below : at, Txy == T ? below : at);
        return T;
    }
};

// Panorama ray tables and yaw-window geometry (built on the host, see mg_api).
struct SensorDev {
    const float4* d4;          // [R] unit direction (w unused)
    const float4* iv4;         // [R] 1/d per component, 0 where d == 0
    const int32_t* bin_of_col; // [W]
    const float2* bv;          // [W] left boundary unit vector of each column
    const float* ts;           // [H+1] tan(e)|tan(e)| at the row boundaries
    const int32_t* c0_of_win;  // [B] first column of window k
    int32_t W, H, B, w, WB, R, T;   // R = W*H rays, T = workgroups per node
    // The trace kernels give each wave a block of kRayBlockCols x kRayBlockRows
    // pixels (rays of one block have similar lengths, so a wave's lanes finish
    // at similar steps); blocks are numbered row block fastest.
    int32_t nrb;               // row blocks, ceil(H / kRayBlockRows)
    int32_t n_blocks;          // ceil(W / kRayBlockCols) * nrb
    uint32_t T_mul, nrb_mul;   // divisor_mul of T and nrb
    // Depth cull of the path-mask builder: a window's pixels in tiles of
    // kTileCols x kTileRows (tcols x trows tiles, column-major), and float
    // angles that place a direction's pixel to within a pixel: azimuth of
    // column 0's left boundary and columns per radian, elevation of row 0's
    // lower boundary and rows per radian.
    int32_t tcols, trows, n_tiles;
    float az0, daz_inv, el0, del_inv;
    float rv;                  // range in voxel units
    float rv2;                 // rv*rv (no depth can exceed it)
    // Guess tables for the pixel lookup (a guess only picks where the exact
    // boundary comparisons start): column from a pseudo-angle past the
    // window's left boundary, row from the elevation tangent.
    const uint16_t* lut_col;   // [n_lut_col]
    const uint16_t* lut_row;   // [n_lut_row]
    int32_t n_lut_col, n_lut_row;
    float lut_col_scale;       // pseudo-angle -> lut_col index
    float lut_row_lo;          // tangent at the bottom of the band
    float lut_row_scale;       // tangent -> lut_row index
};

// One tree's device state. Depth buffers are kept as full panoramas: the
// first-hit parameter of every ray of node n lives at dpan[n*R + r] and the
// node's buffer is the window slice starting at column c0[n]. Every node with
// children has a path mask (mask_slot[n].x >= 0): the set of voxels that n or
// one of its ancestors observes (with anc_cap = 1: that n observes), which is
// what conditions n's children.
struct TreeDev {
    const float4* q4;          // [n] position in voxel units
    const float4* pm;          // [n] position in metres, as given
    const int32_t* anc_ptr;    // [n+1] CSR into anc_ids
    const int32_t* anc_ids;    // ancestors, nearest first
    const int32_t* level_nodes;// [n] nodes sorted by depth
    uint32_t* gain;            // [n] scratch outputs
    int32_t* yaw;
    uint32_t* bins;            // [n][B]: the evaluation's counts (absolute, or marginal)
    float* dpan;               // [n][R]
    int32_t* c0;               // [n]
    uint32_t* masks;           // [nodes with children][mask_words]
    const int2* mask_slot;     // [n] index into masks: the node's (-1 for a leaf) and its parent's (-1 for the root);
                               // side by side: found through the ancestor list the parent's took three dependent loads
    const int32_t* mask_nodes; // nodes with children, by depth level
    float* tmax;               // [nodes with children][2][n_tiles]: largest, then smallest first hit of each tile of the window
    uint32_t* mcode;           // [nodes with children][mask bricks]: code words
    int32_t n;
    int32_t anc_cap;           // ancestors that condition a node: kMaxAnc (all) or 1 (the parent only)
};

// One tree of a multi-tree launch: its map and node data, its range in voxel
// units (maps may differ in voxel size) and where its outputs go.
struct BatchTree {
    MapDev map;
    TreeDev td;
    float rv, rv2;
    double vox3;               // voxel volume (m^3): a gain count times this is a volume
    uint32_t out_off;          // first node of this tree in the launch's outputs (BatchOut)
    // Device status word of the tree's request, or NULL: nonzero marks the
    // request failed, and every later kernel of it returns at once.
    const int32_t* status;
};

// Where a multi-tree launch puts its results (a launch argument, so a plan does
// not depend on the buffers): node i of tree t at t's out_off + i. At gain NULL
// every tree's results go to its own scratch arrays (TreeDev::gain, yaw).
struct BatchOut {
    uint32_t* gain;
    int32_t* yaw;
    float* depth;              // [node][H][WB] or NULL
};

// Launchers (mg_kernels.hip).
hipError_t launch_brick(const uint8_t* dense, uint8_t* bricks, const MapDev& m, hipStream_t s);
hipError_t launch_zero_u32(uint32_t* p, size_t n, hipStream_t s);
// Map contents (mg_map.hip): TSDF conversion of the whole grid or of a box,
// listed voxel updates, and a dense copy of the states.
hipError_t launch_tsdf_grid(const float* dist, const float* weight, const MapDev& m, float surface, float min_weight,
                            hipStream_t s);
hipError_t launch_tsdf_box(const float* dist, const float* weight, const MapDev& m, const int32_t lo[3],
                           const int32_t size[3], float surface, float min_weight, hipStream_t s);
hipError_t launch_map_scatter(const uint32_t* ids, const uint8_t* states, uint32_t count, const MapDev& m,
                              uint32_t* rejected, hipStream_t s);
hipError_t launch_unbrick(const MapDev& m, uint8_t* dense, hipStream_t s, bool marks = false);
hipError_t launch_fill_outside(const MapDev& m, hipStream_t s);
// Recomputes brick_unk and the block marks from the states (after any write
// of the states): the bricks' summaries, then the 16x16x16 blocks.
hipError_t launch_brick_flags(const MapDev& m, hipStream_t s);
// The 16x16x16 blocks alone (after a conversion that took the bricks' summaries itself).
hipError_t launch_blocks16(const MapDev& m, hipStream_t s);
hipError_t launch_trace(const MapDev& m, const SensorDev& sd, const TreeDev& td, const int32_t* nodes,
                        int32_t n_nodes, bool marginal, bool depth, hipStream_t s);   // depth: keep every node's first hits
// Unknown voxels met by the rays of each listed node's window yaw[node] and not
// in its parent's path mask, added to total[node]. The window's first hits are kept
// for nodes with children, with `hits` for every node.
hipError_t launch_trace_window(const MapDev& m, const SensorDev& sd, const TreeDev& td, const int32_t* nodes,
                               int32_t n_nodes, const int32_t* yaw, uint32_t* total, bool hits, hipStream_t s);
// Path masks of the listed nodes (all with children), after their windows are chosen.
hipError_t launch_mask_build(const MapDev& m, const SensorDev& sd, const TreeDev& td, const int32_t* nodes,
                             int32_t n_nodes, hipStream_t s);
hipError_t launch_finish(const SensorDev& sd, const TreeDev& td, const int32_t* nodes, int32_t n_nodes,
                         bool marginal, uint32_t* gain, int32_t* yaw, hipStream_t s);
hipError_t launch_depth_out(const SensorDev& sd, const TreeDev& td, float* depth, hipStream_t s);
// Launch shapes (shape 0 = default): rays per workgroup of the trace kernel
// and bricks per workgroup of the mask builder.
int shape_count();
void shape_of(int shape, int* threads, int* bricks);
int serve_shape();                         // the launch shape the server's level launches use
int32_t tiles_per_node(const SensorDev& sd, int shape);
size_t lds_limit();                        // LDS bytes one workgroup may use on the current device
size_t build_lds_bytes(const SensorDev& sd);   // LDS of the mask builder (sensor tables)
size_t build_lds_total(const SensorDev& sd);   // and with its fixed arrays
// Path score of every node of the trees (eq. 3, eq. 4) and each tree's best node.
hipError_t launch_score(const BatchTree* trees, int32_t n_trees, uint32_t max_nodes, const uint32_t* gain,
                        double lambda, double* cost, double* obj, int32_t* best, int32_t* branch, hipStream_t s);
hipError_t launch_batch_zero(const BatchTree* trees, int32_t n_trees, uint32_t max_nodes, const SensorDev& sd,
                             hipStream_t s);
// One depth level of many trees: trace with launch shape `shape`, window
// selection, then the path masks of the level's nodes with children
// (`mitems`, a subset of `items`). t0/t1 and b0/b1 (may be null): events the
// trace and the builder dispatches themselves record at their start and end.
// mask_bricks: build slots (MapDev::build_slots) of the largest map among the launch's trees.
hipError_t launch_batch_level(const BatchTree* trees, const unsigned long long* items, int32_t n_items,
                              const unsigned long long* mitems, int32_t n_mitems, uint32_t mask_bricks,
                              const SensorDev& sd, const BatchOut& out, hipStream_t s, int shape = 0, hipEvent_t t0 = nullptr,
                              hipEvent_t t1 = nullptr, hipEvent_t b0 = nullptr, hipEvent_t b1 = nullptr);
// The whole batch in one cooperative launch of co-resident workgroups: for each
// depth level d, the trace of items[level_ptr[d] .. level_ptr[d + 1]), their
// windows, then the path masks of mitems[mlevel_ptr[d] .. mlevel_ptr[d + 1]),
// with grid barriers between the phases. sync: 2 device words (zeroed here);
// sync[1] != 0 afterwards when a barrier wait gave up after spin_limit polls.
hipError_t launch_batch_persistent(const BatchTree* trees, const unsigned long long* items, const int32_t* level_ptr,
                                   const unsigned long long* mitems, const int32_t* mlevel_ptr, int32_t levels,
                                   uint32_t mask_bricks, const SensorDev& sd, const BatchOut& out, uint32_t* sync,
                                   uint32_t spin_limit, hipStream_t s);
// Workgroups of the persistent launch: the co-resident capacity of the device.
hipError_t persistent_grid(const SensorDev& sd, int32_t* grid);

}  // namespace mgk
