// Small clouds without a tree.
//
// Up to kFlatMax points the hierarchy costs more than it saves: its build is
// a chain of some twenty dependent launches, and a search from its root a
// chain of dependent record loads.  Such a cloud is only put in Morton order
// and cut into tiles of 64 consecutive points with their boxes.  A
// workgroup searches for the 64 points of one tile: its waves share the
// tiles whose box lies within the largest radius among the 64 points, and
// compare every pair of points of such a tile (Algorithm 2 of the paper with
// a flat list of subtrees; the labels of Optimization 1 skip a tile that
// lies in the searching points' component).
//
// With so few points the whole edge key (D bits, min index, max index)
// fits 64 bits, so one atomicMin per component decides its edge, and the
// bound of Optimization 2 is the D of the shortest edge offered so far:
// Morton-adjacent pairs and the points' candidates of earlier rounds that
// still lie outside are offered as edges before the search of a round.
//
// One round: k_flat_search, then k_flat_merge (one workgroup) or, above
// kFlatOne points, k_flat_parent, k_flat_jump and k_flat_relabel.
// All rounds a cloud of its size usually takes are queued without waiting;
// the kernels of a round that finds one component left return at once.
#pragma once

#include "emst_kernels.h"

namespace emst {

// The rule: a cloud of up to 16,384 points is solved this way.  Measured
// against the tree (us a build, tree / flat): uniform 2D 4,000 points 480 /
// 208, 16,384 581 / 342; clustered 3D 4,000 542 / 243, 16,384 628 / 381;
// skewed 3D, whose points share a few codes so that no tile is skipped,
// 8,000 843 / 633, 12,000 868 / 838 and 16,384 950 / 1,243, the only form of
// cloud that the tree solves faster below the line (it took 1,530 when the
// line was drawn).  At 20,000 points that form takes 2,638 without a tree.
constexpr int64_t kFlatMax = 16384;
constexpr int kFlatTile = 64;         // one query per lane
static_assert(kFlatMax <= 65536, "two indices and D fill the key");

struct FlatArgs {
    int64_t n;
    int tiles;
    const float4* pts;      // sorted: x, y, z, original index; NaN up to the end of the last tile
    const uint32_t* inv;    // sorted position of every original index
    const float4* box;      // two per tile: lo, hi
    uint32_t* labels;
    uint32_t* tile_label;   // the one label of a tile's points, else kInvalid
    uint32_t* cand_d;       // as TraverseArgs
    uint32_t* cand_p;
    uint64_t* compkey;      // shortest edge offered to each component: (D, min, max)
    uint32_t* par;
    uint64_t* ekeys;        // edge of each component id once it has merged
    Ctrl* ctrl;
};

// A round's kernels have nothing to do once the round before has left one
// component, or for a cloud that fails validation.
__device__ __forceinline__ bool flat_over(const Ctrl* ctrl, int round) {
    return ctrl->flat_bad || (round > 0 && ctrl->flat_comps[round - 1] <= 1u);
}

__device__ __forceinline__ uint64_t flat_key(uint32_t d, uint32_t a, uint32_t b) {
    return ((uint64_t)d << 32) | (min(a, b) << 16) | max(a, b);
}

// The number of keys below `mine` (keys are distinct), counted by the
// workgroup's waves in slices: wave w of W compares one key per lane with
// the keys [w n / W, (w + 1) n / W), which are the same for all lanes and
// come through scalar loads.  All n^2 comparisons of 10,000 keys take 17 us,
// the eight passes of a radix sort of 20,000 keys 87 us.
template <int W>
__device__ __forceinline__ uint32_t flat_rank(const uint64_t* __restrict__ keys, int n, uint64_t mine, int w,
                                              uint32_t (*s_cnt)[64]) {
    const int lo = (int)((int64_t)n * w / W), hi = (int)((int64_t)n * (w + 1) / W);
    uint32_t cnt = 0;
#pragma unroll 32
    for (int k = lo; k < hi; ++k) cnt += keys[k] < mine;
    s_cnt[w][lane_id()] = cnt;
    __syncthreads();
    uint32_t r = 0;
    if (w == 0)
        for (int v = 0; v < W; ++v) r += s_cnt[v][lane_id()];
    return r;
}

// Box distance between two boxes, in the order of D (rounding is monotone,
// so it never exceeds D of a point of each).
template <int DIM>
__device__ __forceinline__ float box_box(const float4& alo, const float4& ahi, const float4& blo, const float4& bhi) {
    float g = fmaxf(fmaxf(blo.x - ahi.x, alo.x - bhi.x), 0.0f);
    float s = g * g;
    g = fmaxf(fmaxf(blo.y - ahi.y, alo.y - bhi.y), 0.0f);
    s = s + g * g;
    if (DIM > 2) {
        g = fmaxf(fmaxf(blo.z - ahi.z, alo.z - bhi.z), 0.0f);
        s = s + g * g;
    }
    return s;
}

template <int DIM>
__device__ __forceinline__ float box_point(const float4& p, const float4& lo, const float4& hi) {
    const float a[3] = {p.x, p.y, p.z}, l[3] = {lo.x, lo.y, lo.z}, h[3] = {hi.x, hi.y, hi.z};
    return boxdist<DIM>(a, l, h);
}

template <int DIM>
__device__ __forceinline__ float sqdist4(const float4& a, const float4& b) {
    const float x[3] = {a.x, a.y, a.z}, y[3] = {b.x, b.y, b.z};
    return sqdist<DIM>(x, y);
}

// Memory that no thread of the launch writes, read at addresses that are the
// same for all lanes of a wave: scalar loads.
__device__ __forceinline__ uint32_t uniform_load(const uint32_t* p, int at) {
    return ((const __attribute__((address_space(4))) uint32_t*)(uintptr_t)p)[at];
}
__device__ __forceinline__ float4 uniform_load(const float4* p, int at) {
    typedef float vec __attribute__((ext_vector_type(4)));
    const vec v = ((const __attribute__((address_space(4))) vec*)(uintptr_t)p)[at];
    return make_float4(v.x, v.y, v.z, v.w);
}

// COUNT consecutive points from `first` on as candidates of one query per
// lane: (D, j) order among the points outside component c within the
// radius.  The points arrive by scalar loads, all in flight together, and
// enter the distances as scalar operands.
template <int DIM, int COUNT>
__device__ __forceinline__ void flat_scan(const FlatArgs& a, int first, const float4& me, uint32_t c, float& radius,
                                          uint64_t& best) {
    float4 o[COUNT];
    uint32_t l[COUNT];
#pragma unroll
    for (int q = 0; q < COUNT; ++q) {
        o[q] = uniform_load(a.pts, first + q);
        l[q] = uniform_load(a.labels, first + q);
    }
#pragma unroll
    for (int q = 0; q < COUNT; ++q) {
        const float d = sqdist4<DIM>(me, o[q]);
        if (d <= radius && l[q] != c) {
            const uint64_t k = ((uint64_t)fbits(d) << 32) | fbits(o[q].w);
            if (k < best) {
                best = k;
                radius = d;
            }
        }
    }
}

// The search of one round.  The reuse rules are those of k_traverse_fast
// (variant 13); a kept candidate was offered by k_flat_relabel.  The
// workgroup's waves hold the same 64 queries and share the candidates:
// first those of the queries' own tile, then, if a query still has none,
// those of the nearest tile, which gives every query a radius; then the
// tiles within the largest radius, listed in LDS and handed out in parts of
// 16 points.  Improvements pass through LDS after every part.  Bound by
// the latency of these steps at 10,000 points and below, above by the
// distance evaluations of the tiles that cannot be skipped.
constexpr int kFlatPart = 16;
constexpr int kFlatWaves = 16;

template <int DIM>
__global__ __launch_bounds__(64 * kFlatWaves) void k_flat_search(FlatArgs a, int round) {
    constexpr int W = kFlatWaves;
    if (flat_over(a.ctrl, round)) return;
    __shared__ unsigned long long s_best[kFlatTile];
    __shared__ uint32_t s_list[kFlatMax / kFlatTile];
    __shared__ unsigned long long s_near, s_active;
    __shared__ uint32_t s_count;
    const int lane = lane_id(), w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = blockIdx.x;
    const int64_t i = (int64_t)tile * kFlatTile + lane;
    const bool valid = i < a.n;
    float4 me = make_float4(0.f, 0.f, 0.f, 0.f);
    uint32_t c = kNone, miss = kInfBits, pd = 0u;
    bool active = valid, drop = false;
    if (valid) {
        me = a.pts[i];
        c = a.labels[i];
    }
    // The state of the queries is read by one wave: other workgroups lower
    // the components' keys meanwhile, and all waves must agree.
    if (w == 0) {
        if (valid && round > 0) {
            const uint64_t key = load_relaxed64(&a.compkey[c]);
            if (key != kKeyMax) miss = (uint32_t)(key >> 32);
            pd = a.cand_d[i];
            const uint32_t pp = a.cand_p[i];
            if (pp != kNone) {
                if (a.labels[pp] != c) active = false;                 // kept
                else if (pd > miss) active = false, drop = true;       // absorbed beyond the radius
            } else if (miss <= pd) {
                active = false;                                        // nothing within pd
            }
        }
        const uint64_t am = __ballot(active);
        s_best[lane] = ((uint64_t)miss << 32) | kNone;
        if (lane == 0) {
            s_active = am;
            s_near = kKeyMax;
            s_count = 0u;
        }
    }
    __syncthreads();
    if (s_active == 0ull) {
        if (w == 0 && drop) {
            a.cand_d[i] = pd - 1u;
            a.cand_p[i] = kNone;
        }
        return;
    }
    active = (s_active >> lane) & 1ull;
    uint64_t best = s_best[lane];
    float radius = active ? bitsf((uint32_t)(best >> 32)) : -1.f;
    __syncthreads();  // (improvements come only after every wave has read the start)
    auto refresh = [&]() {
        if (!active) return;
        best = s_best[lane];
        radius = bitsf((uint32_t)(best >> 32));
    };
    constexpr int kShare = kFlatTile / W;
    flat_scan<DIM, kShare>(a, tile * kFlatTile + w * kShare, me, c, radius, best);
    if (active) atomicMin(&s_best[lane], (unsigned long long)best);
    __syncthreads();
    refresh();
    // one tile per thread: its box distance; +inf for a tile that needs no look
    const uint32_t own = round > 0 ? uniform_load(a.tile_label, tile) : kInvalid;
    const int tt = threadIdx.x;
    static_assert(kFlatMax / kFlatTile <= 64 * W, "a thread per tile");
    float dist = INFINITY;
    if (tt < a.tiles && tt != tile && (own == kInvalid || a.tile_label[tt] != own))
        dist = box_box<DIM>(uniform_load(a.box, 2 * tile), uniform_load(a.box, 2 * tile + 1), a.box[2 * tt],
                            a.box[2 * tt + 1]);
    if (__ballot(active && (uint32_t)best == kNone) != 0ull) {  // (the same in every wave)
        uint64_t near = dist < INFINITY ? ((uint64_t)fbits(dist) << 32) | (uint32_t)tt : kKeyMax;
        if (w * 64 < a.tiles) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1)
                near = min(near, (uint64_t)__shfl_xor((unsigned long long)near, off));
            if (lane == 0) atomicMin(&s_near, (unsigned long long)near);
        }
        __syncthreads();
        near = s_near;
        if (near != kKeyMax) {
            const int u = __builtin_amdgcn_readfirstlane((uint32_t)near);
            flat_scan<DIM, kShare>(a, u * kFlatTile + w * kShare, me, c, radius, best);
            if (active) atomicMin(&s_best[lane], (unsigned long long)best);
        }
        __syncthreads();
        refresh();
    }
    float far = radius;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) far = fmaxf(far, __shfl_xor(far, off));
    {
        const bool go = dist <= far && dist < INFINITY;
        const uint64_t m = __ballot(go);
        if (m) {
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&s_count, (uint32_t)__popcll(m));
            at = __builtin_amdgcn_readfirstlane(at);
            if (go) s_list[at + __popcll(m & ((1ull << lane) - 1ull))] = (uint32_t)tt;
        }
    }
    __syncthreads();
    constexpr int kParts = kFlatTile / kFlatPart;
    const int items = __builtin_amdgcn_readfirstlane(s_count) * kParts;
    for (int k = w; k < items; k += W) {
        const int u = __builtin_amdgcn_readfirstlane(s_list[k / kParts]);
        if (__ballot(box_point<DIM>(me, uniform_load(a.box, 2 * u), uniform_load(a.box, 2 * u + 1)) <= radius) == 0ull)
            continue;
        flat_scan<DIM, kFlatPart>(a, u * kFlatTile + (k % kParts) * kFlatPart, me, c, radius, best);
        if (active) {
            const uint64_t old = atomicMin(&s_best[lane], (unsigned long long)best);
            best = min(best, old);
            radius = bitsf((uint32_t)(best >> 32));
        }
    }
    __syncthreads();
    if (w != 0) return;
    best = s_best[lane];
    const uint32_t j = (uint32_t)best, d = (uint32_t)(best >> 32), oi = fbits(me.w);
    const bool found = active && j != kNone;
    if (active) {
        a.cand_d[i] = found ? d : miss;
        a.cand_p[i] = found ? a.inv[j] : kNone;
    } else if (drop) {
        a.cand_d[i] = pd - 1u;
        a.cand_p[i] = kNone;
    }
    uint64_t key = found ? flat_key(d, oi, j) : kKeyMax;
    if (round == 0) {
        if (valid) a.compkey[c] = key;
        return;
    }
    bool run_end;
    key = wave_seg_min<uint64_t>(c, key, &run_end);
    if (valid && run_end && key != kKeyMax && key < load_relaxed64(&a.compkey[c]))
        atomicMin((unsigned long long*)&a.compkey[c], (unsigned long long)key);
}

// Merge, step 1, for every component (a position that is its own label):
// the component at the other end of its edge becomes its parent, except
// that of the two components that share one edge the smaller label becomes
// a root.  Two components share an edge exactly when their keys are equal.
__global__ __launch_bounds__(256) void k_flat_parent(FlatArgs a, int round) {
    if (flat_over(a.ctrl, round)) return;
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool root = false;
    if (c < a.n && a.labels[c] == (uint32_t)c) {
        const uint64_t key = a.compkey[c];
        uint32_t s = (uint32_t)c;
        if (key != kKeyMax) {
            const uint32_t lu = a.labels[a.inv[(uint32_t)(key >> 16) & 0xFFFFu]], lv = a.labels[a.inv[(uint32_t)key & 0xFFFFu]];
            s = lu == (uint32_t)c ? lv : lu;
            root = (uint32_t)c < s && a.compkey[s] == key;
        } else {  // (a cloud that fails validation may find no edge)
            root = true;
        }
        a.par[c] = root ? (uint32_t)c : s;
        a.ekeys[c] = root ? kKeyMax : key;
    }
    const int roots = __syncthreads_count(root);
    if (threadIdx.x == 0 && roots) atomicAdd(&a.ctrl->flat_comps[round], (uint32_t)roots);
}

// Merge, step 2: pointer jumping (see merge_jump_one); roots start the next
// round without an edge.
__global__ __launch_bounds__(256) void k_flat_jump(FlatArgs a, int round) {
    if (flat_over(a.ctrl, round)) return;
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= a.n || a.labels[c] != (uint32_t)c) return;
    uint32_t p = load_relaxed(&a.par[c]);
    if (p == (uint32_t)c) a.compkey[c] = kKeyMax;
    for (int it = 0; it < (int)kFlatMax; ++it) {
        const uint32_t pp = load_relaxed(&a.par[p]);
        if (pp == p) return;
        __hip_atomic_store(&a.par[c], pp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        p = pp;
    }
}

// Merge, step 3, and the offers of the next round: every point takes its
// root as its label; a pair of Morton neighbours in different components,
// and a point's candidate that still lies outside its component, are edges
// of theirs.  Labels read while their block rewrites them lead to the same
// root, old or new.
template <int DIM>
__global__ __launch_bounds__(256) void k_flat_relabel(FlatArgs a, int round) {
    if (flat_over(a.ctrl, round) || a.ctrl->flat_comps[round] <= 1u) return;
    __shared__ uint32_t s_l[258];
    const int t = threadIdx.x;
    const int64_t i0 = (int64_t)blockIdx.x * 256, i = i0 + t;
    auto root_of = [&](int64_t p) { return a.par[a.labels[p]]; };
    const bool valid = i < a.n;
    const uint32_t r = valid ? root_of(i) : kNone;
    s_l[t + 1] = r;
    if (t < 2) {
        const int64_t p = t == 0 ? i0 - 1 : i0 + 256;
        s_l[t == 0 ? 0 : 257] = p >= 0 && p < a.n ? root_of(p) : kNone;
    }
    uint64_t key = kKeyMax;
    float4 me = make_float4(0.f, 0.f, 0.f, 0.f);
    if (valid) {
        me = a.pts[i];
        const uint32_t pp = a.cand_p[i];
        if (pp != kNone && root_of(pp) != r) key = flat_key(a.cand_d[i], fbits(me.w), fbits(a.pts[pp].w));
    }
    __syncthreads();
    if (valid) {
        if (i > 0 && s_l[t] != r) {
            const float4 o = a.pts[i - 1];
            key = min(key, flat_key(fbits(sqdist4<DIM>(o, me)), fbits(o.w), fbits(me.w)));
        }
        if (i + 1 < a.n && s_l[t + 2] != r) {
            const float4 o = a.pts[i + 1];
            key = min(key, flat_key(fbits(sqdist4<DIM>(me, o)), fbits(o.w), fbits(me.w)));
        }
        a.labels[i] = r;
    }
    const uint32_t first = __builtin_amdgcn_readfirstlane(r);
    const bool one = __ballot(valid && r != first) == 0ull;
    if (valid && lane_id() == 0) a.tile_label[i / kFlatTile] = one ? first : kInvalid;
    bool run_end;
    key = wave_seg_min<uint64_t>(r, key, &run_end);
    if (valid && run_end && key != kKeyMax && key < load_relaxed64(&a.compkey[r]))
        atomicMin((unsigned long long*)&a.compkey[r], (unsigned long long)key);
}

// The three merge steps and the offers in one workgroup, for clouds of at
// most kFlatOne points: labels, parents and keys stay in LDS, and offers are
// LDS atomics.  At 1,000 points the three launches take 12 us, this one
// 6 us; at 16,384 the one workgroup would be slower than three launches of
// many.
constexpr int kFlatOne = 4096;

template <int DIM>
__global__ __launch_bounds__(1024) void k_flat_merge(FlatArgs a, int round) {
    if (flat_over(a.ctrl, round)) return;
    constexpr int kPer = kFlatOne / 1024;
    __shared__ uint32_t s_lab[kFlatOne], s_par[kFlatOne];
    __shared__ unsigned long long s_key[kFlatOne];
    __shared__ uint32_t s_roots;
    const int t = threadIdx.x, n = (int)a.n;
    if (t == 0) s_roots = 0u;
    uint32_t lab[kPer];
    uint64_t key[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int p = q * 1024 + t;
        lab[q] = p < n ? a.labels[p] : kNone;
        key[q] = p < n ? a.compkey[p] : kKeyMax;  // (of a component only where p is one)
        s_lab[p] = lab[q];
        s_key[p] = key[q];
    }
    __syncthreads();
    uint32_t roots = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const uint32_t c = (uint32_t)(q * 1024 + t);
        bool root = false;
        if (lab[q] == c) {
            uint32_t s = c;
            if (key[q] != kKeyMax) {
                const uint32_t lu = s_lab[a.inv[(uint32_t)(key[q] >> 16) & 0xFFFFu]];
                const uint32_t lv = s_lab[a.inv[(uint32_t)key[q] & 0xFFFFu]];
                s = lu == c ? lv : lu;
                root = c < s && s_key[s] == key[q];
            } else {
                root = true;
            }
            s_par[c] = root ? c : s;
            a.ekeys[c] = root ? kKeyMax : key[q];
        }
        roots += (uint32_t)__popcll(__ballot(root));
    }
    if (lane_id() == 0 && roots) atomicAdd(&s_roots, roots);
    __syncthreads();
    if (t == 0) a.ctrl->flat_comps[round] = s_roots;
    if (s_roots <= 1u) return;
    for (int it = 0; it < kFlatOne; ++it) {  // (halves the longest chain every time)
        bool more = false;
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const uint32_t c = (uint32_t)(q * 1024 + t);
            if (lab[q] != c) continue;
            const uint32_t p = s_par[c], pp = s_par[p];
            if (pp != p) {
                s_par[c] = pp;
                more = true;
            }
        }
        if (!__syncthreads_or(more)) break;
    }
    uint32_t r[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int p = q * 1024 + t;
        r[q] = kNone;
        if (p >= n) continue;
        r[q] = s_par[lab[q]];
        if (r[q] == (uint32_t)p) s_key[p] = kKeyMax;
        a.labels[p] = r[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) s_lab[q * 1024 + t] = r[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int p = q * 1024 + t;
        const uint32_t first = __builtin_amdgcn_readfirstlane(r[q]);
        const bool one = __ballot(p < n && r[q] != first) == 0ull;
        if (p >= n) continue;
        if (lane_id() == 0) a.tile_label[p / kFlatTile] = one ? first : kInvalid;
        const uint32_t pp = a.cand_p[p];
        const bool kept = pp != kNone && s_lab[pp] != r[q];
        const bool left = p > 0 && s_lab[p - 1] != r[q], right = p + 1 < n && s_lab[p + 1] != r[q];
        if (!(kept || left || right)) continue;
        const float4 me = a.pts[p];
        uint64_t k = kKeyMax;
        if (kept) k = flat_key(a.cand_d[p], fbits(me.w), fbits(a.pts[pp].w));
        if (left) {
            const float4 o = a.pts[p - 1];
            k = min(k, flat_key(fbits(sqdist4<DIM>(o, me)), fbits(o.w), fbits(me.w)));
        }
        if (right) {
            const float4 o = a.pts[p + 1];
            k = min(k, flat_key(fbits(sqdist4<DIM>(me, o)), fbits(o.w), fbits(me.w)));
        }
        atomicMin(&s_key[r[q]], (unsigned long long)k);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int p = q * 1024 + t;
        if (p < n && r[q] == (uint32_t)p) a.compkey[p] = s_key[p];
    }
}

// The box of every tile (one wave each), the padding of the last one, and the
// labels of the start.
template <int DIM>
__global__ __launch_bounds__(256) void k_flat_tiles(FlatArgs a, float4* spts, float4* box) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    if (i < a.n) {
        const float4 me = spts[i];
        const float p[3] = {me.x, me.y, me.z};
#pragma unroll
        for (int k = 0; k < DIM; ++k) lo[k] = hi[k] = p[k];
        a.labels[i] = (uint32_t)i;
    } else if (i < (int64_t)a.tiles * kFlatTile) {
        const float nan = bitsf(0x7FC00000u);  // no distance to it is within any radius
        spts[i] = make_float4(nan, nan, nan, bitsf(kNone));
    }
#pragma unroll
    for (int k = 0; k < DIM; ++k)
        for (int off = 32; off > 0; off >>= 1) {
            lo[k] = fminf(lo[k], __shfl_xor(lo[k], off));
            hi[k] = fmaxf(hi[k], __shfl_xor(hi[k], off));
        }
    if (lane_id() == 0 && i < a.n) {
        box[2 * (i / kFlatTile)] = make_float4(lo[0], lo[1], lo[2], 0.f);
        box[2 * (i / kFlatTile) + 1] = make_float4(hi[0], hi[1], hi[2], 0.f);
    }
}

template <int DIM>
__device__ __forceinline__ float4 flat_point(const float* __restrict__ pts, uint32_t o) {
    return make_float4(pts[(int64_t)o * DIM], pts[(int64_t)o * DIM + 1], DIM > 2 ? pts[(int64_t)o * DIM + 2 % DIM] : 0.f,
                       bitsf(o));
}

// Morton order by counting smaller keys: keys[i] = code << 16 | i.
template <int DIM>
__global__ __launch_bounds__(1024) void k_flat_order(const uint64_t* __restrict__ keys,
                                                     const float* __restrict__ pts, int n,
                                                     float4* __restrict__ spts, uint32_t* __restrict__ inv) {
    __shared__ uint32_t s_cnt[16][64];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i = blockIdx.x * 64 + lane_id();
    const uint64_t mine = i < n ? keys[i] : 0ull;
    const uint32_t r = flat_rank<16>(keys, n, mine, w, s_cnt);
    if (w != 0 || i >= n) return;
    spts[r] = flat_point<DIM>(pts, (uint32_t)i);
    inv[i] = r;
}

// The edges of the merged components in canonical order: the rank of a key
// among all keys is its place (the last root's slot holds the largest key).
__global__ __launch_bounds__(1024) void k_flat_edges(const uint64_t* __restrict__ ekeys, int n, const Ctrl* ctrl,
                                                     int last, int32_t* __restrict__ edges, float* __restrict__ wt,
                                                     float* __restrict__ d2) {
    if (ctrl->flat_bad || ctrl->flat_comps[last] > 1u) return;
    __shared__ uint32_t s_cnt[16][64];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i = blockIdx.x * 64 + lane_id();
    const uint64_t mine = i < n ? ekeys[i] : kKeyMax;
    const uint32_t r = flat_rank<16>(ekeys, n, mine, w, s_cnt);
    if (w != 0 || mine == kKeyMax) return;
    const float d = bitsf((uint32_t)(mine >> 32));
    reinterpret_cast<int2*>(edges)[r] = make_int2((int)((uint32_t)(mine >> 16) & 0xFFFFu), (int)((uint32_t)mine & 0xFFFFu));
    wt[r] = edge_weight(d);
    if (d2) d2[r] = d;
}

}  // namespace emst
