// Device-side building blocks shared by the EMST kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace emst {

constexpr uint32_t kLeafFlag = 0x80000000u;   // child ref: leaf (low 31 bits = original index)
constexpr uint32_t kInvalid = 0xFFFFFFFFu;    // label of a subtree that spans several components
constexpr uint32_t kNone = 0xFFFFFFFFu;       // "no candidate" / "no parent"
constexpr uint32_t kInfBits = 0x7F800000u;    // +inf as float32 bits
constexpr uint64_t kKeyMax = ~0ull;
constexpr int kWave = 64;

// ---------------------------------------------------------------------------
// Node record of the binary LBVH.  One record per internal node holds
// everything a traversal needs about BOTH children, in two parts: the two
// boxes (48 bytes in 3D, 32 in 2D), which never change after the build, and
// one 16-byte entry with each child's reference (internal node index, or
// kLeafFlag | original point index) and component label, the labels
// rewritten every round.  With one point per leaf a leaf child's box is the
// point itself.  A node visit is one 16-byte gather per 16 bytes: the
// traversal is bound by the number of gather instructions (the texture
// addresser takes 19 to 20 cycles for one, whatever its width, and was busy
// 88 % of the second round at 2M points), so labels in an array of their own
// cost it a fifth gather: all rounds' traversals of 37M points took 30.4 ms
// that way and take 28.4, of 2M points 1.83 and 1.64 ms; k_round_prep, which
// writes the labels into 16-byte entries, takes 615 instead of 540 us a launch
// at 37M points.
//
//   3D: child c at floats [6c, 6c + 6): lo.x, lo.y, lo.z, hi.x, hi.y, hi.z
//   2D: child c at floats [4c, 4c + 4): lo.x, lo.y, hi.x, hi.y
//   entry: ref of child 0, ref of child 1, label of child 0, label of child 1
template <int DIM> struct Rec;

template <> struct alignas(16) Rec<3> {
    float4 a, b, c;
};
template <> struct alignas(16) Rec<2> {
    float4 box0, box1;
};

static_assert(sizeof(Rec<3>) == 48, "3D boxes are 48 bytes");
static_assert(sizeof(Rec<2>) == 32, "2D boxes are 32 bytes");

// Upward-walk metadata of an internal node (32 B): the node's Morton cell
// shrunk by a safety margin (every point whose coordinates lie inside it is
// a leaf of the node; an empty cell, lo = +inf, for nodes that split equal
// codes by index), and the link to its parent ((parent << 1) | side, or
// kNone at the root).
struct alignas(16) Up {
    float4 a;  // cell lo x, y, z, parent link (bits)
    float4 b;  // cell hi x, y, z, unused
};

template <int DIM> struct Child {
    float lo[DIM], hi[DIM];
    uint32_t lab, ref;  // label, reference (from the entry)
};

__device__ __forceinline__ uint32_t fbits(float f) { return __float_as_uint(f); }
__device__ __forceinline__ float bitsf(uint32_t u) { return __uint_as_float(u); }

// The boxes of both children.
template <int DIM>
__device__ __forceinline__ void unpack(const Rec<DIM>& r, Child<DIM>& c0, Child<DIM>& c1);

template <>
__device__ __forceinline__ void unpack<3>(const Rec<3>& r, Child<3>& c0, Child<3>& c1) {
    c0.lo[0] = r.a.x; c0.lo[1] = r.a.y; c0.lo[2] = r.a.z;
    c0.hi[0] = r.a.w; c0.hi[1] = r.b.x; c0.hi[2] = r.b.y;
    c1.lo[0] = r.b.z; c1.lo[1] = r.b.w; c1.lo[2] = r.c.x;
    c1.hi[0] = r.c.y; c1.hi[1] = r.c.z; c1.hi[2] = r.c.w;
}

template <>
__device__ __forceinline__ void unpack<2>(const Rec<2>& r, Child<2>& c0, Child<2>& c1) {
    c0.lo[0] = r.box0.x; c0.lo[1] = r.box0.y; c0.hi[0] = r.box0.z; c0.hi[1] = r.box0.w;
    c1.lo[0] = r.box1.x; c1.lo[1] = r.box1.y; c1.hi[0] = r.box1.z; c1.hi[1] = r.box1.w;
}

// ---------------------------------------------------------------------------
// Distances.  The float32 squared distance D is evaluated in one fixed
// order -- d = a0 - b0; s = d*d; then s = s + (ak - bk)^2 for k = 1.. --
// with every step rounded separately (no contraction into FMA).  The box
// distance uses the same order on the per-coordinate gap
// g = max(lo - p, 0, p - hi); rounding is monotone, so it never exceeds D(p, q)
// for a q inside the box, and for a degenerate box (a leaf, lo = hi = q) it
// equals D(p, q) bit for bit because |fl(q - p)| = |fl(p - q)|.

#pragma clang fp contract(off)

template <int DIM>
__device__ __forceinline__ float sqdist(const float* a, const float* b) {
    float d = a[0] - b[0];
    float s = d * d;
#pragma unroll
    for (int k = 1; k < DIM; ++k) {
        d = a[k] - b[k];
        s = s + d * d;
    }
    return s;
}

template <int DIM>
__device__ __forceinline__ float boxdist(const float* p, const float* lo, const float* hi) {
    float g = fmaxf(fmaxf(lo[0] - p[0], p[0] - hi[0]), 0.0f);
    float s = g * g;
#pragma unroll
    for (int k = 1; k < DIM; ++k) {
        g = fmaxf(fmaxf(lo[k] - p[k], p[k] - hi[k]), 0.0f);
        s = s + g * g;
    }
    return s;
}

// The reported weight of an edge of squared length d2: its square root,
// correctly rounded (the library is built with correctly rounded float32
// square roots).
__device__ __forceinline__ float edge_weight(float d2) { return sqrtf(d2); }

// ---------------------------------------------------------------------------
// atomics with explicit scope / ordering

__device__ __forceinline__ uint32_t load_relaxed(const uint32_t* p) {
    return __hip_atomic_load(const_cast<uint32_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t load_relaxed64(const uint64_t* p) {
    return __hip_atomic_load(const_cast<uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int lane_id() { return __lane_id(); }

// gfx950 hands workgroups to its 8 XCDs round-robin (workgroup w runs on
// XCD w % 8), and every XCD has its own L2.  For a grid whose size is a
// multiple of 8 this maps the hardware workgroup id to a logical one so
// that each XCD sweeps one contiguous eighth of the logical range: queries
// that are neighbours in Morton order then share one L2.
constexpr int kXcds = 8;
__device__ __forceinline__ int64_t xcd_block(int64_t hw, int64_t grid) {
    const int64_t per = grid / kXcds;
    return (hw % kXcds) * per + hw / kXcds;
}

// Lane moves inside the vector unit (no LDS): the value of the lane CTRL
// names, or the lane's own value where there is none.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_move(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, CTRL, ROWS, 0xF, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp_move(uint64_t x) {
    return ((uint64_t)dpp_move<CTRL, ROWS>((uint32_t)(x >> 32)) << 32) | dpp_move<CTRL, ROWS>((uint32_t)x);
}

// Segmented inclusive min-scan over the lanes of a wave, segments = runs of
// equal `lab` in lane order.  Lanes only ever combine values carrying the
// same label, and the last lane of a run ends up with the minimum of the
// whole run; *run_end tells whether this lane is that last lane.  Every lane
// of the wave must call it.  The six steps move values by DPP (1, 2, 4 and 8
// lanes inside a row of 16, then the last lane of a row to the next rows); a
// lane takes part in a step if its run reaches back to the lanes it gets
// values from.  (Through LDS, two or three
// ds_bpermute a step, k_round_prep took 621 instead of 615 us a launch at 37M
// points and 39.6 instead of 37.8 us at 2M.)
template <typename T>
__device__ __forceinline__ T wave_seg_min(uint32_t lab, T v, bool* run_end) {
    const int lane = lane_id();
    // (every lane moves its label: a lane left out would give its neighbour 0)
    const uint32_t before = (uint32_t)__shfl_up((int)lab, 1);
    const uint64_t heads = __ballot((lane == 0) | (before != lab));
    const int start = 63 - __clzll(heads & (~0ull >> (63 - lane)));  // first lane of the run
    T o = dpp_move<0x111, 0xF>(v);  // row_shr:1
    if (lane - 1 >= start && o < v) v = o;
    o = dpp_move<0x112, 0xF>(v);
    if (lane - 2 >= start && o < v) v = o;
    o = dpp_move<0x114, 0xF>(v);
    if (lane - 4 >= start && o < v) v = o;
    o = dpp_move<0x118, 0xF>(v);
    if (lane - 8 >= start && o < v) v = o;
    o = dpp_move<0x142, 0xA>(v);  // row_bcast:15 to rows 1 and 3
    if ((lane & ~15) > start && o < v) v = o;
    o = dpp_move<0x143, 0xC>(v);  // row_bcast:31 to rows 2 and 3
    if (start < 32 && o < v) v = o;
    *run_end = lane == 63 || ((heads >> (lane + 1)) & 1ull);
    return v;
}

}  // namespace emst
