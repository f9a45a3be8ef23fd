// Chain engine: every pass of a render in a single persistent launch.
//
// The recursion I_n(u,v) = F(I_{n-1}(u,v), S) is pointwise (Section 2), so a
// pixel's K passes form a chain that needs nothing from other pixels.  A work
// item is one pixel of one view (64-pixel tiles in super-tiles per view,
// views back to back, taken through one band of items per XCD); a lane
// carries its pixel through the view's passes -- trace, shade,
// write image k, and, if the inputs of the next ray changed, displace the
// camera and trace again -- and takes a new pixel as soon as the chain ends
// (after K passes, or when the colour, and in the depth and normal modes the
// hit data, stopped changing: the next ray would be identical, so the result
// is written to the remaining images at once).  No pass barrier and no
// per-pass state in HBM are needed, and views of any size, pass count and
// mode share one launch and its tail.
//
// The work that is not traversal -- finishing a traced pass (shade, write,
// decide) and setting up rays (new pixels, next passes) -- runs in setup
// rounds, when at least refill_min lanes of the wave wait for it, so that it
// runs with most of the wave's lanes instead of a few at a time.  A setup
// round also sets the wave's issue priority from the passes still ahead of
// its youngest chain: longest work first, which shortens the launch's tail
// (the last pixels handed out start chains of up to K passes).
//
// Between setup rounds the wave's rays start in their tile group's entry list
// (below) and put the leaves they reach into a queue that all lanes work off
// (trav_queue).  The instrumented kernel, and launches that have no room for the
// lists or would not gain by them, start at the root and test each leaf in its
// ray's lane (trav_step).
//
// The same kernel serves rcp_render and rcp_render_batch.  Views are read
// from a device table, by each lane, or with scalar loads when the launch
// holds one view; a single render's one-entry table is written by a setup
// kernel from its by-value argument, so a captured graph holds the view and
// rcp_graph_update can change it.  (A view passed as a kernel argument lets
// the compiler hoist its uniform float math into vector registers for the
// whole loop, costing occupancy.)
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>

#include "traverse.hpp"

namespace rcp {
namespace {

struct ViewDev {
    Camera cam;
    int W, H, K, tiles_x, tile_log2w;
    int super_log2;        // log2 of the super-tile side in tiles (0: plain tile rows)
    int super_rows;        // super-tiles per column (batches take them column by column)
    float hw;              // half_width(cam.th, W, H)
    float le, ld, z0;
    float* out;            // [K][H][W][3]
    int32_t* ids;          // [K][H][W] or NULL
    // entry lists (below): one per group of 2^kGroupLog2 x 2^kGroupLog2 tiles
    uint32_t entry_base;   // the view's first list
    uint32_t entries_x;    // groups per row
    float spread_dir;      // bounds of lambda_dir w and lambda_eye w along each camera axis over
    float spread_eye;      // all passes; spread_dir < 0: no useful bound, the lists cull nothing
    float z_reach;         // the largest |z - z0| they hold for (depth mode)
};

static_assert(sizeof(ViewDev) + 2 * sizeof(uint32_t) + 64 <= kViewBytes, "one-entry view table");

// a single render's band counters live in the scene's counter array
static_assert(kFetchWords <= 2 * kMaxPasses + 8, "band counters of a single render");

struct ChainArgs {
    DevScene sc;
    const ViewDev* views;     // [n_views]
    const uint32_t* begin;    // [n_views + 1] first work item of each view
    int n_views;
    uint32_t n_items;         // work items of the launch
    uint32_t* fetch;          // kFetchParts work counters kFetchStride words apart, zero at launch
    int refill_min;
    uint32_t take;               // most pixels a wave holds at once (64, or fewer so that a small launch fills the chip)
    bool whole;                  // waves take whole tiles and keep what is left for their next idle lanes
    uint32_t exit_lanes;
    int32_t* spill;
    uint32_t spill_stride;
    unsigned long long* stats;   // [K][kStatCols] (STATS): rays, inner nodes, triangles, rays continued,
                                 // LDS node reads, stack entries spilled
    const uint32_t* order;       // single view, or NULL: item i is pixel (i & 63) of tile order[i >> 6]
    const float4* entries;       // entry lists of the views' tile groups (ENTRY kernels)
};

// ---- Entry lists --------------------------------------------------------------
// All rays of a tile group's pixels, in every pass, lie in one narrow pyramid:
// the group's rectangle of the image plane, widened by the largest
// displacement (at most lambda_dir along each camera axis in the colour
// mode), seen from the eye (moved by at most lambda_eye).  Every one of those
// rays would walk the same top levels of the tree, past boxes that the
// pyramid misses anyway.  So before the launch each group gets a list of
// up to kEntryItems subtrees: those that the pyramid meets, opened as far
// as that many items allow, nearest first.  A ray tests all items of its
// group's list when it is set up -- a setup round runs with most lanes of the
// wave, and they read the same LDS words -- keeps a bit mask of those it
// meets, and takes its next subtree from the mask whenever its stack is
// empty.  The items' boxes are the exact boxes of the tree's nodes, and only
// boxes that no ray of the group can meet are left out, so the closest hit
// stays the same.  (A pixel whose displacement turns out beyond the bound goes
// on from the root; see the kernel.)  Which launches have lists: lists_pay.
//
// Measured on the 1080p terrain frame (1M triangles, K = 6; ms): 16 items 1.09; 32
// items 1.18 (twice the tests, and a workgroup less per CU); groups of 2 x 2
// tiles 1.09, one tile 1.14, 8 x 8 tiles 1.10; two lists per wave 1.11 (more
// rays without one).
constexpr int kEntryItems = 16;
// A list in HBM (kEntryStride float4): the six planes of four items (as in a
// node) each, the links, then the number of used quads of items.
constexpr uint32_t kEntryF4 = 7 * kEntryItems / 4;     // planes and links, the part held in LDS
constexpr uint32_t kEntryLinks = 6 * kEntryItems / 4;  // first float4 of the links
static_assert(kEntryF4 < kEntryStride && kEntryStride <= 64, "one load per lane copies a list");
constexpr int kGroupLog2 = 2;             // groups of 4 x 4 tiles
constexpr int kEntrySlots = 3;            // lists a wave holds in LDS
static_assert(kNoUnitNormal >= (uint32_t)kEntrySlots, "or'ed to a slot, the mark must name none");
constexpr int kEntryStack = kQueueStack;  // LDS stack entries next to them

// Lanes waiting for a setup round that start one once the bands are used up
// (measured on the terrain frame: 1 -- a round for every waiting lane --
// 0.6% slower; 4 and 12 within 0.2%; 16 and 24 slower again).
constexpr uint32_t kDrainedRound = 8;

// ONE: the launch holds a single view.  Its entry is then read with scalar
// loads (the table is constant during the launch), not per lane through the
// vector-memory path, which the traversal keeps busy.
typedef __attribute__((address_space(4))) ViewDev ConstView;

template <bool STATS, int MODE, bool ONE, bool ENTRY, int STACK, int BLOCK, bool PAIR>
__device__ inline void chain_body(const ChainArgs& a) {
    constexpr bool AUX = MODE != RCP_MODE_COLOR;
    // LDS: the waves' entry lists, or the staged top levels (128-byte nodes, as
    // in HBM, so the same plane offsets serve both), then the stack area, the
    // stats and the view starts
    extern __shared__ float4 smem[];
    float4* top = smem;
    // the traversal reads staged node i at LDS byte address 128 i: the
    // dynamic LDS must begin at address 0, as it does while the kernel
    // declares no LDS of its own (otherwise the launch does nothing and
    // raises the scene's error flag)
    if ((uint32_t)(size_t)(const LdsV4*)top != 0u) {
        if (threadIdx.x == 0) __hip_atomic_store(a.sc.err_flag, kErrLdsLayout, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        return;
    }
    // (the stack directly after the nodes: its column addresses then carry no
    // constant offset, which the paired LDS writes of a push could not encode)
    char* lds = (char*)(smem + (ENTRY ? (BLOCK / 64) * kEntrySlots * kEntryF4 : 8u * a.sc.top_count));
    int32_t* stack_area = (int32_t*)lds;                                  // STACK * BLOCK
    lds += sizeof(int32_t) * STACK * BLOCK;
    // ENTRY: the wave's ray records and leaf queue
    const uint32_t wave_lds =
        __builtin_amdgcn_readfirstlane((uint32_t)(size_t)(const LdsI32*)(int32_t*)lds + (threadIdx.x >> 6) * kQueueBytes);
    if (ENTRY) lds += (BLOCK / 64) * kQueueBytes;
    unsigned long long* lstats = (unsigned long long*)lds;                // STATS: kStatCols * kMaxPasses
    if (STATS) lds += sizeof(unsigned long long) * kStatCols * kMaxPasses;
    uint32_t* vbegin = (uint32_t*)lds;                                    // n_views + 1

    const ConstView* views = (const ConstView*)a.views;
    if (!ONE)
        for (int i = threadIdx.x; i <= a.n_views; i += BLOCK) vbegin[i] = a.begin[i];
    if (!ENTRY)
        for (uint32_t i = threadIdx.x; i < 8u * a.sc.top_count; i += BLOCK)
            if ((i & 7u) != 7u) top[i] = a.sc.nodes[i];   // the zero padding is never read
    if (STATS)
        for (int i = threadIdx.x; i < kStatCols * kMaxPasses; i += BLOCK) lstats[i] = 0ull;
    __syncthreads();

    int v = 0;                 // the lane's view

    const uint32_t gtid = blockIdx.x * BLOCK + threadIdx.x;
    StackT<STACK, BLOCK> st;
    st.lds = stack_area + threadIdx.x;
    st.spill = a.spill + gtid;
    st.stride = a.spill_stride;
    const uint32_t n_items = a.n_items;

    bool alive = false;        // tracing a ray
    bool ended = false;        // its pass is traced, waiting for a setup round to be finished
    bool pending = false;      // holds the inputs of its next pass, waiting for a setup round
    bool drained = false;      // wave-uniform
    uint32_t part = blockIdx.x % kFetchParts;   // wave-uniform: the band fetched from
    uint32_t parts_done = 0;                    // wave-uniform: bands found used up
    uint32_t cur = 0, end = 0;                  // wave-uniform: items taken from a band and not handed out yet
    int k = 0, x = 0, y = 0;
    // ENTRY: slot i of the wave's LDS holds the list of group tag[i], with
    // quads[i] used quads (wave-uniform); `slot` is the lane's slot
    // (kEntrySlots: none, its rays start at the root)
    const uint32_t slot0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * (kEntrySlots * kEntryF4 * 16u);
    uint32_t tag[kEntrySlots], quads[kEntrySlots];
#pragma unroll
    for (int i = 0; i < kEntrySlots; ++i) {
        tag[i] = 0xFFFFFFFFu;
        quads[i] = 0u;
    }
    uint32_t slot = kEntrySlots;
    float pr = 0.5f, pg = 0.5f, pb = 0.5f;              // previous colour (the seed I_0 at pass 0)
    float pa[4] = {INFINITY, 0.0f, 0.0f, 0.0f};         // previous hit data: view depth, unit normal
    TravCount cnt;                                      // STATS: counters of the current ray
    Trav tv;
    tv.node = -1;

    for (;;) {
        // ---- setup round, when enough lanes wait: finish the traced passes,
        // fetch new pixels for idle lanes, and set up the rays of new pixels and
        // of next passes together (work done by a few lanes alone wastes the wave)
        // Once the bands are used up, lanes waiting for their next pass no
        // longer wait for refill_min idle lanes (their chains decide when the
        // launch ends), but for kDrainedRound of them, or for the wave's last
        // ray to end: a round costs the same for 1 lane as for 64.
        const unsigned long long need = wave_ballot(!alive);
        const unsigned long long waiting = wave_ballot(ended || pending);
        const uint32_t n_need = popc_u32(need), n_wait = popc_u32(waiting);
        if (n_need >= (uint32_t)a.refill_min ||
            (drained && cur == end && n_wait != 0u && (n_wait >= kDrainedRound || n_need == 64u))) {
            // lanes whose pass is traced: shade, write, and keep the inputs
            // of the next pass or end the chain
            if (ended) {
                {
                    const ConstView& vw = views[ONE ? 0 : v];
                    float rgb[3];
                    float na[4] = {INFINITY, 0.0f, 0.0f, 0.0f};
                    int32_t hid = -1;
                    if (ENTRY) recorded_hit(tv.h, wave_lds);
                    if (tv.h.id != INT_MAX) {
                        const float4 c = a.sc.shade[2 * (size_t)tv.h.slot + (tv.h.front ? 0 : 1)];
                        rgb[0] = c.x; rgb[1] = c.y; rgb[2] = c.z;
                        hid = tv.h.id;
                        if (AUX) {
                            // view depth of P = o + t d along the camera's forward axis; the
                            // ray is rebuilt (bit-identical) rather than kept in registers
                            float ro[3], rd[3];
                            make_ray<MODE>(vw.cam, vw.hw, vw.W, vw.H, x, y, pr, pg, pb, pa, vw.z0, vw.le, vw.ld, ro,
                                           rd);
                            float P3[3];
#pragma unroll
                            for (int c3 = 0; c3 < 3; ++c3) P3[c3] = ro[c3] + tv.h.t * rd[c3];
                            na[0] = ((P3[0] - vw.cam.eye[0]) * vw.cam.forward[0] +
                                     (P3[1] - vw.cam.eye[1]) * vw.cam.forward[1]) +
                                    (P3[2] - vw.cam.eye[2]) * vw.cam.forward[2];
                            const float4 nv = a.sc.normals[tv.h.slot];
                            na[1] = nv.x; na[2] = nv.y; na[3] = nv.z;
                            // The lists hold for displacements within the view's bounds.  The
                            // test's t of a triangle seen edge on is rounding error, and may put
                            // the hit outside the scene's box; the normal of one whose area is
                            // near the least float may be longer than 1: then the pixel's next
                            // rays start at the root.  (The normal's mark is a slot that no
                            // wave has: a test of the mark costs the 801 x 451 normal frame 2%.)
                            if (ENTRY && MODE == RCP_MODE_DEPTH && !(fabsf(na[0] - vw.z0) <= vw.z_reach))
                                slot = kEntrySlots;
                            if (ENTRY && MODE == RCP_MODE_NORMAL) slot |= __float_as_uint(nv.w);
                        }
                    } else {
                        rgb[0] = a.sc.bg[0]; rgb[1] = a.sc.bg[1]; rgb[2] = a.sc.bg[2];
                    }
                    const size_t P = (size_t)vw.W * (size_t)vw.H;
                    const size_t pix = (size_t)y * (size_t)vw.W + (size_t)x;
                    // the next ray is a function of the colour (and, in the depth and
                    // normal modes, of the hit data): unchanged inputs, unchanged result
                    bool changed = __float_as_uint(rgb[0]) != __float_as_uint(pr) ||
                                   __float_as_uint(rgb[1]) != __float_as_uint(pg) ||
                                   __float_as_uint(rgb[2]) != __float_as_uint(pb);
                    if (AUX)
                        changed = changed || __float_as_uint(na[0]) != __float_as_uint(pa[0]) ||
                                  __float_as_uint(na[1]) != __float_as_uint(pa[1]) ||
                                  __float_as_uint(na[2]) != __float_as_uint(pa[2]) ||
                                  __float_as_uint(na[3]) != __float_as_uint(pa[3]);
                    // image k, and every later image when nothing changed
                    const int k_end = changed ? k + 1 : vw.K;
                    for (int kk = k; kk < k_end; ++kk) {
                        float* q = vw.out + ((size_t)kk * P + pix) * 3;
                        q[0] = rgb[0]; q[1] = rgb[1]; q[2] = rgb[2];
                        if (vw.ids) vw.ids[(size_t)kk * P + pix] = hid;
                    }
                    bool next = changed && k + 1 < vw.K;
                    if (ENTRY && !AUX && next && k >= 2) {
                        // The colour of two or three passes ago again: that pass's
                        // successor follows, and so on, so the remaining images
                        // repeat with that period.  The colours of those passes
                        // are read back from the pixel's own images.  (Terrain
                        // frames: 9% of the rays at 1M triangles and K = 6; 4K
                        // frame of 16M triangles, K = 8: 7.73 -> 5.96 ms.  The
                        // depth and normal modes would need their hit data of
                        // those passes as well: kept in registers, no faster at
                        // 1080p and 4% slower on a small frame.)
                        const float* q2 = vw.out + ((size_t)(k - 2) * P + pix) * 3;
                        const float* q3 = k >= 3 ? vw.out + ((size_t)(k - 3) * P + pix) * 3 : q2;
                        const float c2[3] = {q2[0], q2[1], q2[2]}, c3[3] = {q3[0], q3[1], q3[2]};
                        int period = 0;
                        if (__float_as_uint(c2[0]) == __float_as_uint(rgb[0]) && __float_as_uint(c2[1]) == __float_as_uint(rgb[1]) &&
                            __float_as_uint(c2[2]) == __float_as_uint(rgb[2]))
                            period = 2;
                        else if (k >= 3 && __float_as_uint(c3[0]) == __float_as_uint(rgb[0]) &&
                                 __float_as_uint(c3[1]) == __float_as_uint(rgb[1]) &&
                                 __float_as_uint(c3[2]) == __float_as_uint(rgb[2]))
                            period = 3;
                        if (period != 0) {
                            next = false;
                            for (int kk = k + 1; kk < vw.K; ++kk) {
                                const size_t to = (size_t)kk * P + pix, from = to - (size_t)period * P;
                                const float r0 = vw.out[3 * from], r1 = vw.out[3 * from + 1], r2 = vw.out[3 * from + 2];
                                vw.out[3 * to] = r0;
                                vw.out[3 * to + 1] = r1;
                                vw.out[3 * to + 2] = r2;
                                if (vw.ids) vw.ids[to] = vw.ids[from];
                            }
                        }
                    }
                    if (STATS) {
                        unsigned long long* sk = lstats + kStatCols * k;
                        atomicAdd(&sk[0], 1ull);
                        atomicAdd(&sk[1], (unsigned long long)cnt.nodes);
                        atomicAdd(&sk[2], (unsigned long long)cnt.tris);
                        if (next) atomicAdd(&sk[3], 1ull);
                        atomicAdd(&sk[4], (unsigned long long)cnt.lds);
                        atomicAdd(&sk[5], (unsigned long long)cnt.spill);
                        cnt = TravCount();
                    }
                    if (next) {
                        ++k;
                        pr = rgb[0]; pg = rgb[1]; pb = rgb[2];
                        if (AUX) { pa[0] = na[0]; pa[1] = na[1]; pa[2] = na[2]; pa[3] = na[3]; }
                        pending = true;
                    }
                }
                ended = false;
            }
            const unsigned long long idle = wave_ballot(!alive && !pending);
            // (a wave that holds fewer pixels than lanes fills up to `take`)
            const uint32_t held = 64u - popc_u32(idle);
            const uint32_t n_idle = held < a.take ? a.take - held : 0u;
            // items for the idle lanes: what is left of those taken last, then
            // a whole tile or as many as there are idle lanes left
            const uint32_t left = end - cur;
            uint32_t base = 0, lim = 0;
            if (left < n_idle && !drained) {
                const uint32_t want = a.whole ? a.take : n_idle - left;
                wave_fetch(a.fetch, n_items, want, part, parts_done, drained, base, lim);
                lim = base + want < lim ? base + want : lim;
            }
            const uint32_t nth = lanes_below(idle);
            const uint32_t item = nth < left ? cur + nth : base + (nth - left);
            const bool get = !alive && !pending && nth < n_idle && (nth < left || item < lim);
            if (n_idle <= left) {
                cur += n_idle;
            } else {
                cur = base + (n_idle - left);
                end = lim;
                if (cur > end) cur = end;
            }
            bool init = pending;
            uint32_t group = 0xFFFFFFFFu;   // ENTRY: tile group of a new pixel
            {
                if (get) {
                    // the view holding this item: last begin <= item
                    if (!ONE) {
                        int lo = 0, hi = a.n_views;
                        while (hi - lo > 1) {
                            const int mid = (lo + hi) >> 1;
                            if (vbegin[mid] <= item) lo = mid; else hi = mid;
                        }
                        v = lo;
                    }
                    const uint32_t local = ONE ? (a.order ? (a.order[item >> 6] << 6) | (item & 63u) : item)
                                               : item - vbegin[v];
                    {
                        const ConstView& vw = views[ONE ? 0 : v];
                        tile_pixel(local, (uint32_t)vw.tiles_x, (uint32_t)vw.tile_log2w, (uint32_t)vw.super_log2, x, y,
                                   ONE ? 0u : (uint32_t)vw.super_rows);
                        if (x < vw.W && y < vw.H) {
                            k = 0;
                            pr = 0.5f; pg = 0.5f; pb = 0.5f;
                            pa[0] = INFINITY; pa[1] = 0.0f; pa[2] = 0.0f; pa[3] = 0.0f;
                            init = true;
                            if (ENTRY) {
                                const uint32_t gx = (uint32_t)x >> (vw.tile_log2w + kGroupLog2);
                                const uint32_t gy = (uint32_t)y >> (6 - vw.tile_log2w + kGroupLog2);
                                group = vw.entry_base + gy * vw.entries_x + gx;
                            }
                        }
                    }
                }
            }
            if (ENTRY) {
                // the entry lists of the new pixels' groups (the tiles of a round
                // may come from anywhere in the band, when they go out by cost or
                // what was left is topped up): already in a slot, or copied into
                // one that no live lane uses.  Without a free slot the pixels
                // start at the scene's root.
                unsigned long long todo = wave_ballot(group != 0xFFFFFFFFu);
                if (todo != 0ull) {
                    uint32_t busy = 0;
#pragma unroll
                    for (int i = 0; i < kEntrySlots; ++i)
                        if (wave_ballot((alive || pending) && slot == (uint32_t)i) != 0ull) busy |= 1u << i;
                    do {
                        const uint32_t g = (uint32_t)__builtin_amdgcn_readlane((int)group, __builtin_ctzll(todo));
                        uint32_t got = kEntrySlots;
#pragma unroll
                        for (int i = 0; i < kEntrySlots; ++i)
                            if (got == kEntrySlots && tag[i] == g) got = i;
                        if (got == kEntrySlots) {
                            const uint32_t l = threadIdx.x & 63u;
#pragma unroll
                            for (int i = 0; i < kEntrySlots; ++i)
                                if (got == kEntrySlots && ((busy >> i) & 1u) == 0u) {
                                    got = i;
                                    tag[i] = g;
                                    const float4 q = a.entries[(size_t)g * kEntryStride + (l < kEntryStride ? l : kEntryF4)];
                                    quads[i] = (uint32_t)__builtin_amdgcn_readlane(__float_as_int(q.x), kEntryF4);
                                    const V4 qv = {q.x, q.y, q.z, q.w};
                                    if (l < kEntryF4) *(LdsV4*)(size_t)(slot0 + (kEntryF4 * i + l) * 16u) = qv;
                                }
                        }
                        if (got != kEntrySlots) busy |= 1u << got;
                        const bool mine = group == g;
                        if (mine) slot = got;
                        todo &= ~wave_ballot(mine);
                    } while (todo != 0ull);
                    wave_lds_fence();
                }
            }
            {
                // Longest remaining work first: the wave's issue priority follows
                // the passes still ahead of its youngest chain (at most K - k),
                // so that the chains started last, which decide when the launch
                // ends, are not slowed down by waves about to finish.
                // (Measured on the terrain frame: 3.7% faster; applied only once
                // the bands are used up, 3.0%.)
                const int kk = views[ONE ? 0 : v].K;
                const bool live = alive || init;
                const int rem = kk - k;
                if (wave_ballot(live && 3 * rem >= 2 * kk) != 0ull) __builtin_amdgcn_s_setprio(3);
                else if (wave_ballot(live && 2 * rem >= kk) != 0ull) __builtin_amdgcn_s_setprio(2);
                else if (wave_ballot(live && 3 * rem >= kk) != 0ull) __builtin_amdgcn_s_setprio(1);
                else __builtin_amdgcn_s_setprio(0);
            }
            if (init) {
                const ConstView& vw = views[ONE ? 0 : v];
                float o[3], d[3];
                make_ray<MODE>(vw.cam, vw.hw, vw.W, vw.H, x, y, pr, pg, pb, pa, vw.z0, vw.le, vw.ld, o, d);
                trav_init(tv, a.sc, o, d, st);
                tv.todo = 0u;
                tv.items = 0u;
                if (ENTRY) record_ray(tv.rw, wave_lds);
                if (ENTRY && slot < (uint32_t)kEntrySlots) {
                    // the items the ray meets, in the order of the list
                    uint32_t n = 0;
#pragma unroll
                    for (int i = 0; i < kEntrySlots; ++i) n = slot == (uint32_t)i ? quads[i] : n;
                    uint32_t at = slot0 + slot * (kEntryF4 * 16u);
                    tv.items = at + kEntryLinks * 16u;
                    for (uint32_t j = 0; j < n; ++j, at += 96u) tv.todo |= meet4(tv, at) << (4u * j);
                    tv.node = next_node<true>(tv, st);
                }
                if (STATS) cnt = TravCount();
                alive = true;
                pending = false;
            }
        }
        if (wave_ballot(alive) == 0ull) {
            if (drained && cur == end && wave_ballot(pending || ended) == 0ull) break;
            continue;
        }

        // ---- one traversal step -------------------------------------------------
        if (ENTRY) {
            // until the next setup round can start
            const uint32_t dead = popc_u32(wave_ballot(!alive));
            const uint32_t enough = drained && cur == end ? (dead + kDrainedRound < 64u ? dead + kDrainedRound : 64u) : (uint32_t)a.refill_min;
            trav_queue<true, PAIR>(tv, a.sc, st, wave_lds, a.exit_lanes, enough);
        } else if (alive && tv.node != -1) {
            trav_step<STATS, false>(tv, a.sc, st, a.exit_lanes, cnt);
        }

        if (alive && tv.node == -1) {   // the pass is traced: finish it in the next round
            alive = false;
            ended = true;
        }
    }

    if (STATS) {
        __syncthreads();
        for (int i = threadIdx.x; i < kStatCols * kMaxPasses; i += BLOCK)
            if (lstats[i]) atomicAdd(&a.stats[i], lstats[i]);
    }
}

// Colour mode, the default: asking for 6 waves per SIMD (at most 80 VGPRs)
// was measured faster than the 5 the compiler picks alone; 7 and 8 spill and
// are slower.  The depth and normal modes keep the compiler's choice (6
// spills there and measured 1% slower).  STACK (LDS stack entries per lane)
// and BLOCK (workgroup size) are launch parameters the autotuner chooses
// among for the colour mode's timed kernel; the instrumented kernel and the
// depth and normal modes use kStack and kBlock.
// PAIR (the launches that few_pixels names): the leaves' triangles are read in
// pairs, which a chain waits for once instead of twice, and a wave fewer per
// SIMD makes room for them.
template <bool STATS, bool ONE, bool ENTRY, int STACK, int BLOCK, bool PAIR>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(PAIR ? 5 : 6))) void k_chain(ChainArgs a) {
    chain_body<STATS, RCP_MODE_COLOR, ONE, ENTRY, STACK, BLOCK, PAIR>(a);
}

template <bool STATS, int MODE, bool ONE, bool ENTRY, bool PAIR>
__global__ __launch_bounds__(kBlock) void k_chain_aux(ChainArgs a) {
    chain_body<STATS, MODE, ONE, ENTRY, ENTRY ? kEntryStack : kStack, kBlock, PAIR>(a);
}

// ---- Small scenes: every triangle tested ----------------------------------------
// A frame of few pixels leaves the chip idle while its chains wait on one
// dependent node or triangle load after another, and a small scene of large,
// overlapping triangles has a tree that prunes little.  Then the pixel's rays
// are tested against all triangles by G lanes side by side, 64 / G pixels per
// wave, each pixel's passes in a loop: no tree, no stack, no work queue, and
// nothing before the launch.  The nearest hit is the least (t, triangle index)
// word of the group, as in the leaf queue.
template <int MODE, int G>
__global__ __launch_bounds__(kBlock) void k_direct(DevScene sc, ViewDev v) {
    constexpr bool AUX = MODE != RCP_MODE_COLOR;
    const uint32_t P = (uint32_t)v.W * (uint32_t)v.H;
    const uint32_t pixel = (blockIdx.x * kBlock + threadIdx.x) / G, sub = threadIdx.x % G;
    const bool live = pixel < P;
    const int y = (int)(pixel / (uint32_t)v.W), x = (int)(pixel - (uint32_t)y * (uint32_t)v.W);
    float prev[3] = {0.5f, 0.5f, 0.5f};
    float pa[4] = {INFINITY, 0.0f, 0.0f, 0.0f};
    int k = live ? 0 : v.K;    // the pixel's pass; v.K: its chain has ended
    // a ray that tests every triangle takes as many steps as there are full
    // leaves of them: more than its budget, and it ends as in the traversal
    const bool spent = (sc.n_tris + (uint32_t)kMaxLeaf - 1u) / (uint32_t)kMaxLeaf > sc.step_budget;
    if (spent && threadIdx.x == 0)
        __hip_atomic_store(sc.err_flag, kErrStepBudget, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    while (wave_ballot(k < v.K) != 0ull) {
        float o[3], d[3];
        make_ray<MODE>(v.cam, v.hw, v.W, v.H, x, y, prev[0], prev[1], prev[2], pa, v.z0, v.le, v.ld, o, d);
        const RayW r = ray_setup(o, d, dominant_axis(d), sc.n_tris);
        unsigned long long best = ~0ull;
        uint32_t slot = 0;
        if (k < v.K && !spent) {
            const float4* tp = sc.tris + 3 * (size_t)r.tri_base;
            const uint32_t last = sc.n_tris - 1u;
            uint32_t i = sub;
            const float4* a = tp + 3 * (size_t)min(i, last);
            float4 v0 = a[0], v1 = a[1], v2 = a[2];
            for (; i < sc.n_tris; i += G) {
                // the next triangle is loaded while this one is tested
                const float4* b = tp + 3 * (size_t)min(i + G, last);
                const float4 n0 = b[0], n1 = b[1], n2 = b[2];
                float t;
                bool front;
                if (hit_triangle(r, v0, v1, v2, t, front)) {
                    const unsigned long long key = ((unsigned long long)__float_as_uint(t) << 32) | __float_as_uint(v0.w);
                    if (key < best) {
                        best = key;
                        slot = i | (front ? 0x80000000u : 0u);
                    }
                }
                v0 = n0; v1 = n1; v2 = n2;
            }
        }
#pragma unroll
        for (int m = G / 2; m >= 1; m >>= 1) {
            const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(best >> 32), m, 64);
            const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)best, m, 64);
            const uint32_t os = (uint32_t)__shfl_xor((int)slot, m, 64);
            const unsigned long long other = ((unsigned long long)hi << 32) | lo;
            if (other < best) {
                best = other;
                slot = os;
            }
        }
        if (k >= v.K) continue;
        // shade, write, and keep the inputs of the next pass or end the chain
        float rgb[3] = {sc.bg[0], sc.bg[1], sc.bg[2]};
        float na[4] = {INFINITY, 0.0f, 0.0f, 0.0f};
        int32_t hid = -1;
        if (best != ~0ull) {
            const uint32_t tri = slot & 0x7FFFFFFFu;
            const float4 c = sc.shade[2 * (size_t)tri + ((slot >> 31) ? 0 : 1)];
            rgb[0] = c.x; rgb[1] = c.y; rgb[2] = c.z;
            hid = (int32_t)(uint32_t)best;
            if (AUX) {
                const float t = __uint_as_float((uint32_t)(best >> 32));
                float p3[3];
#pragma unroll
                for (int c3 = 0; c3 < 3; ++c3) p3[c3] = o[c3] + t * d[c3];
                na[0] = ((p3[0] - v.cam.eye[0]) * v.cam.forward[0] + (p3[1] - v.cam.eye[1]) * v.cam.forward[1]) +
                        (p3[2] - v.cam.eye[2]) * v.cam.forward[2];
                const float4 nv = sc.normals[tri];
                na[1] = nv.x; na[2] = nv.y; na[3] = nv.z;
            }
        }
        bool changed = false;
#pragma unroll
        for (int c = 0; c < 3; ++c) changed = changed || __float_as_uint(rgb[c]) != __float_as_uint(prev[c]);
        if (AUX)
#pragma unroll
            for (int c = 0; c < 4; ++c) changed = changed || __float_as_uint(na[c]) != __float_as_uint(pa[c]);
        const int k_end = changed ? k + 1 : v.K;
        for (int kk = k + (int)sub; kk < k_end; kk += G) {
            float* q = v.out + ((size_t)kk * P + pixel) * 3;
            q[0] = rgb[0]; q[1] = rgb[1]; q[2] = rgb[2];
            if (v.ids) v.ids[(size_t)kk * P + pixel] = hid;
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) prev[c] = rgb[c];
#pragma unroll
        for (int c = 0; c < 4; ++c) pa[c] = na[c];
        k = k_end;
    }
}

// Zero the work counters (kFetchParts per launch) and the stats.
__global__ void k_clear_chain(uint32_t* fetch, int n, unsigned long long* stats) {
    for (int i = threadIdx.x; i < (int)kFetchWords * n; i += blockDim.x) fetch[i] = 0u;
    if (stats)
        for (int i = threadIdx.x; i < kStatCols * kMaxPasses; i += blockDim.x) stats[i] = 0ull;
}

// Setup of a one-view launch (a single render, or a batch of one view): its
// one-entry view table, item range, zeroed band counters and stats.
__device__ inline void setup_single(const ViewDev& v, ViewDev* table, uint32_t* begin, uint32_t n_items,
                                    uint32_t* fetch, unsigned long long* stats) {
    if (threadIdx.x == 0) {
        *table = v;
        begin[0] = 0u;
        begin[1] = n_items;
        for (uint32_t p = 0; p < kFetchParts; ++p) fetch[kFetchStride * p] = 0u;
    }
    if (stats)
        for (int i = threadIdx.x; i < kStatCols * kMaxPasses; i += blockDim.x) stats[i] = 0ull;
}

// ---- Cost order of a single render's tiles -----------------------------------
// A tile's score is the largest number of occupied cells of the scene's
// occupancy grid that one of four undisplaced rays crosses, through the
// centres of the tile's quadrants (a voxel walk after Amanatides and Woo, "A
// Fast Voxel Traversal Algorithm for Ray Tracing", Eurographics 1987): a
// tile's wave is as slow as its slowest lane.  Each ray's segment inside the
// grid is walked in two halves by two threads, which halves the longest walk,
// the one that sets the kernel's time.  Rays that skim many occupied cells
// tend to start long chains; within each band the tiles are handed out by
// decreasing score, so that those chains start first and the launch's tail,
// set by the chains started last, gets shorter.  The order decides only when
// a pixel is rendered, never its result.
constexpr uint32_t kScoreBins = 256;

constexpr uint32_t kScoreBlock = 256;

__device__ inline void tile_scores(const ViewDev& v, const OccGrid& g, uint32_t n_tiles, uint32_t* score, uint32_t block,
                                   uint32_t* occ) {
    for (uint32_t i = threadIdx.x; i < g.words; i += kScoreBlock) occ[i] = g.bits[i];
    __syncthreads();
    // eight neighbouring threads per tile: the quadrant in the low two bits,
    // the half of the ray's walk in the third; every thread reaches the
    // shuffles at the end
    const uint32_t gt = block * kScoreBlock + threadIdx.x;
    const uint32_t t = gt >> 3, sub = gt & 3u, half = (gt >> 2) & 1u;
    const uint32_t tw = 1u << (uint32_t)v.tile_log2w, th = 64u >> (uint32_t)v.tile_log2w;
    int x0 = 0, y0 = 0, x = 0, y = 0;
    if (t < n_tiles) tile_pixel(t << 6, (uint32_t)v.tiles_x, (uint32_t)v.tile_log2w, (uint32_t)v.super_log2, x0, y0);
    const bool live = t < n_tiles && x0 < v.W && y0 < v.H;
    const uint32_t sx = (sub & 1u) ? (3u * tw) / 4u : tw / 4u, sy = (sub & 2u) ? (3u * th) / 4u : th / 4u;
    tile_pixel((t << 6) + sy * tw + sx, (uint32_t)v.tiles_x, (uint32_t)v.tile_log2w,
               (uint32_t)v.super_log2, x, y);
    x = x < v.W ? x : v.W - 1;
    y = y < v.H ? y : v.H - 1;
    const float fx = (float)(2 * x + 1) / (float)v.W - 1.0f;
    const float fy = 1.0f - (float)(2 * y + 1) / (float)v.H;
    float o[3], d[3], inv[3];
    float tmin = 0.0f, tmax = INFINITY;
    bool miss = false;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        o[a] = v.cam.eye[a];
        d[a] = v.cam.forward[a] + fx * v.hw * v.cam.right[a] + fy * v.cam.th * v.cam.up[a];
        const float lo = g.lo[a], hi = g.lo[a] + g.cell[a] * (float)g.n[a];
        if (d[a] == 0.0f) {
            inv[a] = INFINITY;
            miss = miss || o[a] < lo || o[a] > hi;
        } else {
            inv[a] = 1.0f / d[a];
            const float t0 = (lo - o[a]) * inv[a], t1 = (hi - o[a]) * inv[a];
            tmin = fmaxf(tmin, fminf(t0, t1));
            tmax = fminf(tmax, fmaxf(t0, t1));
        }
    }
    uint32_t count = 0;
    if (live && !miss && tmin <= tmax) {
        const float tmid = 0.5f * (tmin + tmax);
        const float tbeg = half ? tmid : tmin, tend = half ? tmax : tmid;
        // per axis: the next boundary's t, its spacing, the cell index stride
        // of a step and the steps left inside the grid
        float tnext[3], tdelta[3];
        int stride[3];
        uint32_t left[3];
        int cell = 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float p = o[a] + tbeg * d[a];
            int q = (int)floorf((p - g.lo[a]) / g.cell[a]);
            q = q < 0 ? 0 : (q >= g.n[a] ? g.n[a] - 1 : q);
            const int step = d[a] > 0.0f ? 1 : (d[a] < 0.0f ? -1 : 0);
            tnext[a] = step == 0 ? INFINITY
                                 : (g.lo[a] + (float)(q + (step > 0 ? 1 : 0)) * g.cell[a] - o[a]) * inv[a];
            tdelta[a] = step == 0 ? INFINITY : g.cell[a] * fabsf(inv[a]);
            const int unit = a == 0 ? 1 : (a == 1 ? g.n[0] : g.n[0] * g.n[1]);
            stride[a] = step * unit;
            left[a] = step > 0 ? (uint32_t)(g.n[a] - 1 - q) : (step < 0 ? (uint32_t)q : 0u);
            cell += q * unit;
        }
        // one step per iteration, without branches: the axis whose boundary
        // comes first (x, then y, then z among equal ones); the walk ends past
        // tend or at the grid's side.  The second half's first cell is the
        // first half's last, counted there.
        const int steps = g.n[0] + g.n[1] + g.n[2];
        for (int it = 0; it < steps; ++it) {
            count += (it > 0 || half == 0u) ? (occ[(uint32_t)cell >> 5] >> ((uint32_t)cell & 31u)) & 1u : 0u;
            const bool ax = tnext[0] <= tnext[1] && tnext[0] <= tnext[2];
            const bool ay = !ax && tnext[1] <= tnext[2];
            const bool az = !ax && !ay;
            const float tn = ax ? tnext[0] : (ay ? tnext[1] : tnext[2]);
            const uint32_t l = ax ? left[0] : (ay ? left[1] : left[2]);
            if (tn > tend || l == 0u) break;
            cell += ax ? stride[0] : (ay ? stride[1] : stride[2]);
            tnext[0] += ax ? tdelta[0] : 0.0f;
            tnext[1] += ay ? tdelta[1] : 0.0f;
            tnext[2] += az ? tdelta[2] : 0.0f;
            left[0] -= ax ? 1u : 0u;
            left[1] -= ay ? 1u : 0u;
            left[2] -= az ? 1u : 0u;
        }
    }
    count += (uint32_t)__shfl_xor((int)count, 4);   // the ray's two halves
    count = max(count, (uint32_t)__shfl_xor((int)count, 1));
    count = max(count, (uint32_t)__shfl_xor((int)count, 2));
    if (sub == 0u && half == 0u && t < n_tiles) score[t] = count;
}

// The entry list of a tile group, by one wave.  The items are opened in
// rounds, all of the list at once: four lanes load one item's node and test a
// child each against the group's pyramid, and the openings are accepted in
// the order of the items' box areas (those that do not add items first)
// while at most kEntryItems items result.  About six rounds of one dependent
// node load each on the terrain frame.
// A full list can still shrink its items (openings that add none).  A single
// view's launch waits for its lists and leaves that out (k_prepare 22.3 -> 17.6
// us at 1080p, 801 x 451 frame 311 -> 305); a batch, whose views share one
// launch, gains more from it than it costs (3.38 -> 3.35 ms for 16 views).
constexpr uint32_t kEntryGroups = kScoreBlock / 64;   // lists per workgroup
constexpr int kEntryChunks = kEntryItems / 16;        // items per group of four lanes

struct EntryLds {
    // items in two buffers: six planes of 32, links; the list is then laid
    // out in the buffer not in use
    float buf[2][7 * kEntryItems];
    uint32_t key[kEntryItems];
};

// Four planes through the pyramid's sides and one through the eye, as
// n . P >= c for points P that any of the group's rays may reach.
struct Pyramid {
    float n[5][3], c[5];
    bool cull;

    // Whether the box may hold such a point: its farthest corner along each
    // plane's normal.  False for the NaN planes of an unused slot.
    __device__ inline bool meets(const float lo[3], const float hi[3]) const {
        bool in = lo[0] <= hi[0];
        if (cull) {
#pragma unroll
            for (int p = 0; p < 5; ++p) {
                float e = n[p][0] * (n[p][0] > 0.0f ? hi[0] : lo[0]);
                e = __builtin_fmaf(n[p][1], n[p][1] > 0.0f ? hi[1] : lo[1], e);
                e = __builtin_fmaf(n[p][2], n[p][2] > 0.0f ? hi[2] : lo[2], e);
                in = in && e >= c[p];
            }
        }
        return in;
    }
};

template <class View>
__device__ inline Pyramid group_pyramid(const View& v, uint32_t local, float radius) {
    // the group's rectangle of pixels, and its pyramid's slopes along right
    // and up, widened for the displacement and for the rounding of the rays
    // and of the camera's basis (at most 1e-5 from orthonormal)
    const int gw = 1 << (v.tile_log2w + kGroupLog2), gh = 1 << (6 - v.tile_log2w + kGroupLog2);
    const int x0 = (int)(local % v.entries_x) * gw, y0 = (int)(local / v.entries_x) * gh;
    const int x1 = min(x0 + gw, v.W) - 1, y1 = min(y0 + gh, v.H) - 1;
    Pyramid r;
    r.cull = v.spread_dir >= 0.0f;
    const float ds = r.cull ? v.spread_dir : 0.0f;
    const float th = v.cam.th;
    const float eps = 4e-5f * (1.0f + v.hw + th) / (1.0f - ds);
    float lo_s = ((float)(2 * x0 + 1) / (float)v.W - 1.0f) * v.hw - ds;
    float hi_s = ((float)(2 * x1 + 1) / (float)v.W - 1.0f) * v.hw + ds;
    float lo_t = (1.0f - (float)(2 * y1 + 1) / (float)v.H) * th - ds;
    float hi_t = (1.0f - (float)(2 * y0 + 1) / (float)v.H) * th + ds;
    const float near_s = 1.0f / (1.0f + ds), far_s = 1.0f / (1.0f - ds);   // 1 / (forward component)
    lo_s = fminf(lo_s * near_s, lo_s * far_s);
    lo_t = fminf(lo_t * near_s, lo_t * far_s);
    hi_s = fmaxf(hi_s * near_s, hi_s * far_s);
    hi_t = fmaxf(hi_t * near_s, hi_t * far_s);
    lo_s -= eps * (1.0f + fabsf(lo_s));
    lo_t -= eps * (1.0f + fabsf(lo_t));
    hi_s += eps * (1.0f + fabsf(hi_s));
    hi_t += eps * (1.0f + fabsf(hi_t));
    // margins: the eye's displacement, and 2^-16 of the largest coordinates
    // (the traversal widens its boxes by 2^-18 of them)
    const float eye_max = fmaxf(fmaxf(fabsf(v.cam.eye[0]), fabsf(v.cam.eye[1])), fabsf(v.cam.eye[2]));
    const float size = (radius + eye_max + 2.0f * v.spread_eye) * 1.52587890625e-5f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        r.n[0][a] = v.cam.right[a] - lo_s * v.cam.forward[a];
        r.n[1][a] = hi_s * v.cam.forward[a] - v.cam.right[a];
        r.n[2][a] = v.cam.up[a] - lo_t * v.cam.forward[a];
        r.n[3][a] = hi_t * v.cam.forward[a] - v.cam.up[a];
        r.n[4][a] = v.cam.forward[a];
    }
    const float slope[5] = {lo_s, hi_s, lo_t, hi_t, 0.0f};
#pragma unroll
    for (int p = 0; p < 5; ++p) {
        const float l1 = fabsf(r.n[p][0]) + fabsf(r.n[p][1]) + fabsf(r.n[p][2]);
        const float ne = r.n[p][0] * v.cam.eye[0] + r.n[p][1] * v.cam.eye[1] + r.n[p][2] * v.cam.eye[2];
        r.c[p] = ne - (v.spread_eye * 1.001f * (1.0f + fabsf(slope[p])) + size * l1);
    }
    return r;
}

template <bool SHRINK, class View>
__device__ inline void entry_list(const View& v, uint32_t local, const DevScene& sc, float4* __restrict__ out, EntryLds& m) {
    constexpr int N = kEntryItems, C = kEntryChunks;
    const int lane = (int)(threadIdx.x & 63u), child = lane & 3;
    const Pyramid py = group_pyramid(v, local, sc.radius);
    int cur = 0, count = 1;
    if (lane == 0) {   // the root
#pragma unroll
        for (int a = 0; a < 6; ++a) m.buf[0][N * a] = 0.0f;
        m.buf[0][6 * N] = __int_as_float(0);
    }
    for (int round = 0; round < 64 && (SHRINK || count < N); ++round) {
        wave_lds_fence();
        const float* b = m.buf[cur];
        float box[C][7];       // the lane's child of each of its items, with its link
        bool cand[C], in[C];
        uint32_t key[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int item = (lane >> 2) + 16 * c;
            const int32_t link = item < count ? __float_as_int(b[6 * N + item]) : -1;
            cand[c] = link >= 0;   // an inner node
            in[c] = false;
            float area = 0.0f;
            if (cand[c]) {
                const float* g = (const float*)(sc.nodes + 8 * (size_t)link) + child;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    box[c][a] = g[8 * a];
                    box[c][3 + a] = g[8 * a + 4];
                }
                box[c][6] = g[24];
                const float ex = b[3 * N + item] - b[item], ey = b[4 * N + item] - b[N + item],
                            ez = b[5 * N + item] - b[2 * N + item];
                area = ex * ey + ey * ez + ez * ex;
                in[c] = py.meets(box[c], box[c] + 3);
            }
            const uint32_t kids = (uint32_t)__builtin_popcount((uint32_t)(wave_ballot(in[c]) >> (lane & 60)) & 15u);
            // rank of the opening: its area's bits, above those the items it
            // adds plus one; the item's number breaks ties
            key[c] = cand[c] ? ((kids <= 1u ? 0x7F800000u : (__float_as_uint(area) & 0x7FFFFFFFu)) & ~7u) | kids : 1u;
            if (child == 0) m.key[item] = key[c];
        }
        wave_lds_fence();
        int sum[C];
#pragma unroll
        for (int c = 0; c < C; ++c) sum[c] = count + (int)(key[c] & 7u) - 1;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const uint32_t kj = m.key[j];
            const int add = (int)(kj & 7u) - 1;
#pragma unroll
            for (int c = 0; c < C; ++c)
                sum[c] += ((kj >> 3) > (key[c] >> 3) || ((kj >> 3) == (key[c] >> 3) && j < (lane >> 2) + 16 * c)) ? add : 0;
        }
        // the next round's items: the children in place of the opened ones
        float* w = m.buf[cur ^ 1];
        int next = 0;
        bool opened = false;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int item = (lane >> 2) + 16 * c;
            const bool accept = cand[c] && sum[c] <= N;
            opened = opened || accept;
            const bool give = accept ? in[c] : (item < count && child == 0);
            const unsigned long long all = wave_ballot(give);
            if (give) {
                const int pos = next + (int)lanes_below(all);
#pragma unroll
                for (int a = 0; a < 7; ++a) w[N * a + pos] = accept ? box[c][a] : b[N * a + item];
            }
            next += (int)popc_u32(all);
        }
        if (wave_ballot(opened) == 0ull) break;
        cur ^= 1;
        count = next;
    }
    wave_lds_fence();
    // the list, nearest item first: unused slots have NaN planes, which no ray meets
    const float nan = __int_as_float(0x7FC00000);
    float b[7] = {nan, nan, nan, nan, nan, nan, __int_as_float(-1)};
    float depth = INFINITY;
    if (lane < count) {
#pragma unroll
        for (int a = 0; a < 7; ++a) b[a] = m.buf[cur][a * N + lane];
        depth = v.cam.forward[0] * (b[0] + b[3]) + v.cam.forward[1] * (b[1] + b[4]) + v.cam.forward[2] * (b[2] + b[5]);
    }
    // (boxes of infinite extent are the only way to a NaN: then the order of arrival)
    if (wave_ballot(depth != depth) != 0ull) depth = (float)lane;
    if (lane < N) m.key[lane] = __float_as_uint(depth);
    wave_lds_fence();
    int rank = 0;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const float dj = __uint_as_float(m.key[j]);
        rank += (dj < depth || (dj == depth && j < lane)) ? 1 : 0;
    }
    float* w = m.buf[cur ^ 1];
    if (lane < N) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            w[24 * (rank >> 2) + 8 * a + (rank & 3)] = b[a];
            w[24 * (rank >> 2) + 8 * a + 4 + (rank & 3)] = b[3 + a];
        }
        w[6 * N + rank] = b[6];
    }
    wave_lds_fence();
    if (lane < (int)kEntryF4) out[lane] = ((const float4*)w)[lane];
    if (lane == 0) out[kEntryF4] = make_float4(__int_as_float((count + 3) / 4), 0.0f, 0.0f, 0.0f);
}

// Everything a single render needs before its chain launch that does not
// depend on the order: entry lists (workgroups below entry_blocks; they take
// longest, so they start first), tile scores (the next score_blocks) and,
// without a cost order, the setup (one more).
__global__ __launch_bounds__(kScoreBlock) void k_prepare(ViewDev v, OccGrid g, DevScene sc, uint32_t n_tiles, uint32_t* score,
                                                         uint32_t score_blocks, float4* entries, uint32_t n_entries,
                                                         uint32_t entry_blocks, ViewDev* table, uint32_t* begin,
                                                         uint32_t n_items, uint32_t* fetch, unsigned long long* stats) {
    extern __shared__ float4 prep_lds[];
    if (blockIdx.x < entry_blocks) {
        const uint32_t e = blockIdx.x * kEntryGroups + (threadIdx.x >> 6);
        if (e < n_entries)
            entry_list<false>(v, e, sc, entries + (size_t)e * kEntryStride, ((EntryLds*)prep_lds)[threadIdx.x >> 6]);
    } else if (blockIdx.x < entry_blocks + score_blocks) {
        tile_scores(v, g, n_tiles, score, blockIdx.x - entry_blocks, (uint32_t*)prep_lds);
    } else {
        setup_single(v, table, begin, n_items, fetch, stats);
    }
}

// The entry lists of a batch: one workgroup per kEntryGroups lists, the view
// of each found in the table.
__global__ __launch_bounds__(kScoreBlock) void k_batch_entries(const ViewDev* __restrict__ views, int n_views, DevScene sc,
                                                               float4* entries, uint32_t n_entries) {
    extern __shared__ float4 prep_lds[];
    const uint32_t sub = threadIdx.x >> 6, e = blockIdx.x * kEntryGroups + sub;
    if (e >= n_entries) return;
    int lo = 0, hi = n_views;   // the last view with entry_base <= e
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (views[mid].entry_base <= e) lo = mid; else hi = mid;
    }
    lo = __builtin_amdgcn_readfirstlane(lo);
    entry_list<true>(views[lo], e - views[lo].entry_base, sc, entries + (size_t)e * kEntryStride, ((EntryLds*)prep_lds)[sub]);
}

// One workgroup per band: a counting sort of the band's tiles by decreasing
// score (order within a score is the order of arrival, which only moves
// work in time).  Every tile of the band lands in exactly one slot of the
// band's range, so order[] is a permutation of the tiles.  One more
// workgroup does the launch's setup.
__global__ __launch_bounds__(1024) void k_band_order(const uint32_t* __restrict__ score, uint32_t n_items,
                                                     uint32_t* __restrict__ order, ViewDev v, ViewDev* table,
                                                     uint32_t* begin, uint32_t* fetch, unsigned long long* stats) {
    if (blockIdx.x == kFetchParts) {
        setup_single(v, table, begin, n_items, fetch, stats);
        return;
    }
    __shared__ uint32_t hist[kScoreBins];
    const uint32_t lo = part_begin(n_items, blockIdx.x) >> 6, hi = part_begin(n_items, blockIdx.x + 1u) >> 6;
    for (uint32_t i = threadIdx.x; i < kScoreBins; i += 1024) hist[i] = 0u;
    __syncthreads();
    for (uint32_t t = lo + threadIdx.x; t < hi; t += 1024) {
        const uint32_t b = score[t] < kScoreBins ? score[t] : kScoreBins - 1u;
        atomicAdd(&hist[b], 1u);
    }
    __syncthreads();
    // each bin's first slot: the tiles of all higher scores come before it
    // (a scan over the bins from the highest down, kScoreBins threads)
    __shared__ uint32_t scan[kScoreBins];
    const uint32_t own = threadIdx.x < kScoreBins ? hist[kScoreBins - 1u - threadIdx.x] : 0u;
    if (threadIdx.x < kScoreBins) scan[threadIdx.x] = own;
    __syncthreads();
    for (uint32_t off = 1; off < kScoreBins; off <<= 1) {
        const uint32_t add = (threadIdx.x < kScoreBins && threadIdx.x >= off) ? scan[threadIdx.x - off] : 0u;
        __syncthreads();
        if (threadIdx.x < kScoreBins) scan[threadIdx.x] += add;
        __syncthreads();
    }
    if (threadIdx.x < kScoreBins) hist[kScoreBins - 1u - threadIdx.x] = scan[threadIdx.x] - own;
    __syncthreads();
    for (uint32_t t = lo + threadIdx.x; t < hi; t += 1024) {
        const uint32_t b = score[t] < kScoreBins ? score[t] : kScoreBins - 1u;
        order[lo + atomicAdd(&hist[b], 1u)] = t;
    }
}

// A chain kernel instantiation with its workgroup size and stack depth.
struct ChainKernel {
    const void* fn;
    int block;
    int stack;
    bool entry;      // rays start in entry lists
};

// (the deeper of the two stacks is kEntryStack entries next to the entry
// lists: six workgroups still fit a CU's LDS)
template <bool STATS, bool ONE, bool ENTRY>
ChainKernel colour_kernel(int stack, int block) {
    constexpr int D = ENTRY ? kEntryStack : kStack;
    if constexpr (!STATS) {
        if (stack == 8 && block == 512) return {(const void*)k_chain<false, ONE, ENTRY, 8, 512, false>, 512, 8, ENTRY};
        if (stack == 8) return {(const void*)k_chain<false, ONE, ENTRY, 8, kBlock, false>, kBlock, 8, ENTRY};
        if (block == 512) return {(const void*)k_chain<false, ONE, ENTRY, D, 512, false>, 512, D, ENTRY};
    }
    return {(const void*)k_chain<STATS, ONE, ENTRY, D, kBlock, false>, kBlock, D, ENTRY};
}

template <bool STATS, int MODE, bool ONE, bool ENTRY, bool PAIR>
ChainKernel aux_kernel() {
    return {(const void*)k_chain_aux<STATS, MODE, ONE, ENTRY, PAIR>, kBlock, ENTRY ? kEntryStack : kStack, ENTRY};
}

template <bool STATS, bool ONE, bool ENTRY>
ChainKernel chain_kernel2(int mode, const Launch& lp) {
    switch (mode) {
        case RCP_MODE_DEPTH: return aux_kernel<STATS, RCP_MODE_DEPTH, ONE, ENTRY, false>();
        case RCP_MODE_NORMAL: return aux_kernel<STATS, RCP_MODE_NORMAL, ONE, ENTRY, false>();
        default: return colour_kernel<STATS, ONE, ENTRY>(lp.stack, lp.block);
    }
}

// The kernel of a launch over n_views views in `mode` (the single-view
// kernels when n_views == 1), with or without entry lists.
ChainKernel chain_kernel(bool stats, int n_views, int mode, const Launch& lp, bool entry) {
    // The instrumented kernel always starts at the root, so that its counts are
    // those of the tree, the same in both engines.
    if (stats)
        return n_views == 1 ? chain_kernel2<true, true, false>(mode, lp) : chain_kernel2<true, false, false>(mode, lp);
    if (entry) return n_views == 1 ? chain_kernel2<false, true, true>(mode, lp) : chain_kernel2<false, false, true>(mode, lp);
    return n_views == 1 ? chain_kernel2<false, true, false>(mode, lp) : chain_kernel2<false, false, false>(mode, lp);
}

// The kernel that reads triangles in pairs, in place of one with entry lists
// in workgroups of kBlock.
template <bool ONE>
ChainKernel pair_kernel(int mode) {
    switch (mode) {
        case RCP_MODE_DEPTH: return aux_kernel<false, RCP_MODE_DEPTH, ONE, true, true>();
        case RCP_MODE_NORMAL: return aux_kernel<false, RCP_MODE_NORMAL, ONE, true, true>();
        default: return {(const void*)k_chain<false, ONE, true, kEntryStack, kBlock, true>, kBlock, kEntryStack, true};
    }
}

// A launch whose time is that of its longest chains rather than of its work:
// up to four pixels per lane that the default kernel keeps resident (1.6M
// pixels in the colour mode, 1.3M in the others).  (1M-triangle terrain, K = 6,
// ms without / with pairs: colour 400 x 225 0.53 / 0.49, 640 x 360 0.60 / 0.55,
// 1440 x 810 0.84 / 0.78, 1600 x 900 0.88 / 0.87, 1920 x 1080 1.06 / 1.06, 3840 x
// 2160 K = 8 on 16M triangles 5.67 / 5.83; normal 560 x 315 0.62 / 0.58, 1440 x 810
// 0.81 / 0.78, 1600 x 900 0.87 / 0.90, 1920 x 1080 1.07 / 1.10.)
bool few_pixels(uint64_t items, uint32_t threads) { return items <= 4u * (uint64_t)threads; }

// LDS of a workgroup: the waves' entry lists or the staged top levels, the
// stack area and the view starts (and the stats).
size_t chain_smem(const Launch& lp, const ChainKernel& k, bool stats, int n_views) {
    size_t b = (k.entry ? (size_t)(k.block / 64) * kEntrySlots * kEntryF4 * 16 : kNodeBytes * (size_t)lp.top_count) +
               sizeof(int32_t) * (size_t)k.stack * (size_t)k.block +
               (k.entry ? (size_t)(k.block / 64) * kQueueBytes : 0) +
               sizeof(uint32_t) * (size_t)((n_views + 4) & ~3);
    if (stats) b += sizeof(unsigned long long) * kStatCols * kMaxPasses;
    return b;
}

}  // namespace

// Resident workgroups per CU and CU count of a kernel at an LDS size, on the
// current device.  The runtime's answers are cached: they cannot change in a
// process, and asking costs more than a launch.
rcp_status resident_blocks(const void* kernel, int block, size_t smem, int& per_cu, int& cus) {
    static std::mutex mu;
    static std::map<std::tuple<const void*, size_t, int>, std::pair<int, int>> cache;
    int dev = 0;
    RCP_HIP(hipGetDevice(&dev));
    const auto key = std::make_tuple(kernel, smem, dev);
    {
        std::lock_guard<std::mutex> lk(mu);
        const auto it = cache.find(key);
        if (it != cache.end()) {
            per_cu = it->second.first;
            cus = it->second.second;
            return RCP_OK;
        }
    }
    RCP_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block, smem));
    RCP_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    std::lock_guard<std::mutex> lk(mu);
    cache[key] = std::make_pair(per_cu, cus);
    return RCP_OK;
}

namespace {

// Kernel, grid and LDS size of a launch over n_views views in `mode`.
struct ChainGrid {
    ChainKernel k;
    int blocks = 0;
    size_t smem = 0;
    uint32_t lanes = 0;   // threads of a full grid of the default kernel
    uint32_t threads() const { return (uint32_t)blocks * (uint32_t)k.block; }
};

// Workgroups of kernel g.k that stay resident.
rcp_status resident_grid(const Launch& lp, bool stats, int n_views, ChainGrid& g) {
    g.smem = chain_smem(lp, g.k, stats, n_views);
    int per_cu = 0, cus = 0;
    const rcp_status st = resident_blocks(g.k.fn, g.k.block, g.smem, per_cu, cus);
    if (st != RCP_OK) return st;
    if (per_cu < 1) per_cu = 1;
    // blocks_per_cu counts workgroups of kBlock threads; a larger workgroup
    // counts as several
    if (lp.blocks_per_cu > 0) {
        const int cap = std::max(1, lp.blocks_per_cu * kBlock / g.k.block);
        if (cap < per_cu) per_cu = cap;
    }
    g.blocks = per_cu * cus;
    g.lanes = g.threads();
    return RCP_OK;
}

// Whether a ray visits a large part of the scene's triangles (a soup of large
// triangles about three quarters of their number in nodes and tests, a terrain
// 1 / 80 of it at 1000 triangles and less above).
bool visits_much(const rcp_scene* s) { return s->ray_work > (float)s->dev.n_tris / 16.0f; }

// Whether a launch's rays are better off in entry lists than at the root.  A ray
// that has a list tests its 16 boxes, whatever it meets of them, and saves the
// levels of the tree above them; how much that is depends on how narrow the
// groups' pyramids are (`spread`: the displacement in radians or so, see below)
// and on how many levels there are.  Terrains, colour mode, speed against the
// root start for spreads 0.01 / 0.03 / 0.05 / 0.1 / 0.2:
//   1920 x 1080, K = 6: 5000 triangles (9 levels) 1.13 / 1.03 / 0.96 / 0.89 / 0.87, 20,000
//     1.10 / 0.99 / 0.95 / 0.92 / 0.89, 100,000 (12) 1.11 / 1.00 / 0.96 / 0.94 / 0.95,
//     300,000 (14) 1.07 / 1.01 / 1.01 / 1.01 / 1.00, 1M 1.13 / 1.07 / 1.05 / 1.04 / 1.02;
//     K = 3: 5000 1.07 / 1.05 / 1.02 / 0.99 / 0.98, 100,000 1.05 / 1.04 / 1.03 / 1.02 / 0.97
//   1280 x 720, K = 6: 5000 1.15 / 1.04 / 0.99 / 0.90 / 0.88, 100,000 1.20 / 1.08 / 1.03 /
//     0.98 / 0.95, 1M 1.20 / 1.20 / 1.05 / 1.01 / 1.02; K = 3 more throughout
//   3840 x 2160, K = 6: 5000 1.22 / 1.16 / 1.11 / 1.03 / 0.94, 100,000 1.36 / 1.17 / 1.08 /
//     0.97 / 0.91, 1M 1.40 / 1.20 / 1.11 / 1.03 / 0.99
// The depth and normal modes lose less by wide pyramids: nothing up to 0.2, but
// for 1280 x 720 frames of 5000 triangles in the depth mode (0.04 1.00, 0.08 0.97,
// 0.12 0.94).
// Where a ray visits much of the scene most boxes are met; the lists pay by what
// comes with them, the leaf queue, and that for long chains and small frames
// (soups of 200 to 4000 triangles, six views: 3840 x 2160, K = 1 0.92-1.11, K = 3
// 0.93-1.16, K = 8 1.05-1.6; 1920 x 1080, K = 1 and 3 0.93-1.19, K = 6 1.2-1.6; 1280 x
// 720, all 1.1-1.8): a frame of up to three passes is no slower only from the root,
// but for the depth and normal modes from 635 triangles on (3840 x 2160, K = 2 and
// 3: 64 0.96, 256 1.00, 635 1.05, 1200 1.13, 2500 1.33).
bool lists_pay(const rcp_scene* s, int mode, double spread, int K, uint64_t items, uint32_t lanes) {
    const bool few = few_pixels(items, lanes), many = items >= 7u * (uint64_t)lanes;
    if (visits_much(s)) return few || K > 3 || (mode != RCP_MODE_COLOR && s->ray_work >= 400.0f);
    const uint32_t levels = s->dev.max_depth;
    double most = 0.2;
    if (mode != RCP_MODE_COLOR) {
        if (few && levels <= 9u) most = 0.06;
    } else if (many) {
        most = 0.1;
    } else if (levels > 12u || (few && K <= 3)) {
        return true;
    } else if (few) {
        most = levels > 10u ? 0.09 : 0.04;
    } else {
        most = K <= 3 ? 0.06 : 0.032;
    }
    return spread <= most;
}

// The grid of a launch over `items` pixels (with their tiles' padding).  It
// needs no more overflow area than one of more items: the kernel for few keeps
// as many stack entries per lane, and no more lanes.
rcp_status chain_grid(const Launch& lp, bool stats, int n_views, int mode, bool entry, uint64_t items, ChainGrid& g) {
    g.k = chain_kernel(stats, n_views, mode, lp, entry);
    RCP_TRY_STATUS(resident_grid(lp, stats, n_views, g));
    if (!stats && entry && g.k.block == kBlock && g.k.stack == kEntryStack && few_pixels(items, g.threads())) {
        ChainGrid p;
        p.k = n_views == 1 ? pair_kernel<true>(mode) : pair_kernel<false>(mode);
        RCP_TRY_STATUS(resident_grid(lp, stats, n_views, p));
        p.blocks = std::min(p.blocks, g.blocks);
        p.lanes = g.lanes;
        g = p;
    }
    return RCP_OK;
}

// Pixels a wave holds at once.  A launch of few pixels would leave most of
// the chip's waves without any while the others' rays wait for the slowest of
// 64: the smallest power of two is taken that gives each resident wave at most
// two handfuls.  (20,000-triangle terrain, K = 6, microseconds with 64 / the
// choice: 64 x 64 353 / 223 with 1, 320 x 200 396 / 327 with 8, 512 x 512
// 401 / 362 with 32; halving or doubling the choice is slower or the same.)
void set_take(const rcp_scene* s, ChainArgs& a, const ChainGrid& g, int K) {
    const uint64_t waves = (uint64_t)g.threads() / 64u;
    a.take = 1u;
    while (a.take < 64u && (uint64_t)a.n_items > 2u * waves * a.take) a.take *= 2u;
    // Whole tiles keep a tile's pixels in one wave and make a third of the
    // atomics, but a wave then keeps up to a tile that others could start when
    // the work runs out: taken from seven pixels per lane on.  (Frame ms,
    // exact / whole: 1920 x 1080, K = 6, 5 per lane 1.06 / 1.09; 2560 x 1440, 9
    // per lane 1.69 / 1.53; 3840 x 2160, K = 8, 21 per lane 4.33 / 3.38; 4 mixed
    // views, 6 per lane 1.39 / 1.35.  Pieces of 8, 16 or 32 pixels gain nothing:
    // the tiles then lie across waves as much as with exact counts.  The lanes are
    // those of a full grid: one cut down to its stack overflow area has more
    // pixels per lane and no more time to lose: 16M triangles, 1080p, K = 3 on
    // four workgroups per CU 1.66 / 1.83.)
    // Not where a ray visits much of the scene: the fetches are then a small part,
    // and what a wave keeps is long work (3840 x 2160, exact / whole: soups of 64
    // triangles, K = 8, 0.89 / 1.01, of 128 1.16 / 1.31, of 635, K = 3, 1.64 / 1.87, of
    // 2500 4.41 / 5.40; terrains of
    // 20,000 1.00 / 0.83, of 16M, K = 8, 4.33 / 3.38).
    // And from the root not in frames of one pass, nor in trees whose rays' work
    // is long (without lists, 3840 x 2160, exact / whole: K = 1, 20,000 triangles 0.51 /
    // 0.55, 1M 0.80 / 0.88; K = 2, 20,000 0.84 / 0.76, 1M 1.57 / 1.55, 4M, 74 of
    // ray_work, 1.94 / 2.03; 16 views, 5000 1.36 / 1.20, 1M, 36 of ray_work, 4.51 / 4.53, spread
    // 0.2 4.80 / 5.04).
    a.whole = a.n_items >= 7u * (uint64_t)g.lanes && !visits_much(s) && (g.k.entry || (K >= 2 && s->ray_work <= (a.n_views == 1 ? 50.0f : 30.0f)));
    // the refill threshold in idle lanes, in proportion
    a.refill_min = 64 - (int)a.take + (a.refill_min * (int)a.take + 63) / 64;
}

rcp_status launch_chain(const ChainGrid& g, hipStream_t stream, ChainArgs a) {
    void* args[] = {(void*)&a};
    RCP_HIP(hipLaunchKernel(g.k.fn, dim3((unsigned)g.blocks), dim3((unsigned)g.k.block), args, g.smem, stream));
    return RCP_OK;
}

size_t spill_depth_of(const rcp_scene* s, const ChainKernel& k) {
    return spill_per_thread(s->dev, k.stack);
}

// Groups of tiles of a view (one entry list each).
uint64_t view_entries(int W, int H, int tile_log2w, uint32_t* per_row = nullptr) {
    const uint64_t gw = 1ull << (tile_log2w + kGroupLog2), gh = 1ull << (6 - tile_log2w + kGroupLog2);
    const uint64_t x = ((uint64_t)W + gw - 1) / gw, y = ((uint64_t)H + gh - 1) / gh;
    if (per_row) *per_row = (uint32_t)x;
    return x * y;
}

// Bounds of the displacements lambda w of a view's rays along each camera
// axis, over all passes: |2c - 1| <= 1 for every shaded colour (clamped to
// [0, 1]) and as the background says; times the largest |z - z0| of a hit
// in the depth mode (z over the scene's box); 1 in the normal mode (a
// product of unit vectors).  spread_dir < 0 where the rays' pyramid would not
// be one (lambda_dir w as long as the focal distance) or the numbers leave
// the range in which single precision holds the test's margins.
// z_reach: the |z - z0| that is bounded by; a hit beyond it (see the kernel) ends
// the use of the lists.
void view_spread(const rcp_scene* s, const Camera& cam, float hw, const Disp& d, float& dir, float& eye,
                 float& z_reach) {
    double w = 1.0;
    if (d.mode != RCP_MODE_NORMAL)
        for (int a = 0; a < 3; ++a) w = std::max(w, std::fabs(2.0 * s->dev.bg[a] - 1.0));
    double far = s->dev.radius;
    for (int a = 0; a < 3; ++a) far = std::max(far, std::fabs((double)cam.eye[a]));
    if (d.mode == RCP_MODE_DEPTH) {
        double lo = 0.0, hi = 0.0;
        for (int a = 0; a < 3; ++a) {
            const double p = (double)s->occ.lo[a] - cam.eye[a];
            const double q = p + (double)s->occ.cell[a] * s->occ.n[a];
            lo += std::min(p * cam.forward[a], q * cam.forward[a]);
            hi += std::max(p * cam.forward[a], q * cam.forward[a]);
        }
        const double reach = std::max(std::fabs(lo - d.z0), std::fabs(hi - d.z0)) * 1.0001 + 1e-4 * far;
        z_reach = (float)reach;
        w *= reach;
    }
    w *= 1.0001;
    const double wd = w * d.ld, we = w * d.le;
    const bool fine = wd <= 0.5 && we <= 1e12 && far <= 1e12 && hw <= 1e4f && cam.th <= 1e4f;
    dir = fine ? (float)wd : -1.0f;
    eye = fine ? (float)we : 0.0f;
}

// The same as one number: how far a ray of the view may be turned, with the
// eye's displacement seen from half the scene's longest extent (which is about
// where a view of the whole scene is taken from).
double spread_angle(const rcp_scene* s, float dir, float eye) {
    if (dir < 0.0f) return HUGE_VAL;
    double extent = 1e-30;
    for (int a = 0; a < 3; ++a) extent = std::max(extent, 0.5 * s->occ.cell[a] * s->occ.n[a]);
    return dir + eye / extent;
}

double view_spread_angle(const rcp_scene* s, const Camera& cam, int W, int H, const Disp& d) {
    float dir, eye, reach;
    view_spread(s, cam, half_width(cam.th, W, H), d, dir, eye, reach);
    return spread_angle(s, dir, eye);
}

ViewDev view_of(const rcp_scene* s, const Camera& cam, int W, int H, int K, const Disp& d, float* out, int32_t* ids,
                int tile_log2w) {
    ViewDev v{};
    v.cam = cam;
    v.W = W; v.H = H; v.K = K;
    v.hw = half_width(cam.th, W, H);
    v.tile_log2w = tile_log2w;
    v.tiles_x = (W + (1 << tile_log2w) - 1) >> tile_log2w;
    v.super_log2 = super_log2_for(W, H, tile_log2w);
    const int tiles_y = (H + (64 >> tile_log2w) - 1) / (64 >> tile_log2w);
    v.super_rows = (tiles_y + (1 << v.super_log2) - 1) >> v.super_log2;
    v.le = d.le; v.ld = d.ld; v.z0 = d.z0;
    v.out = out;
    v.ids = ids;
    (void)view_entries(W, H, tile_log2w, &v.entries_x);
    view_spread(s, cam, v.hw, d, v.spread_dir, v.spread_eye, v.z_reach);
    return v;
}

uint64_t view_items(const ViewDev& v) {
    return view_tile_items(v.W, v.H, v.tile_log2w, v.super_log2);
}

uint64_t frame_items(int W, int H, int tile_log2w) {
    return view_tile_items(W, H, tile_log2w, super_log2_for(W, H, tile_log2w));
}

// Entries of a view's score and order buffer: two per tile.
size_t order_entries(int W, int H, int tile_log2w) { return 2 * (size_t)(frame_items(W, H, tile_log2w) >> 6); }

}  // namespace

rcp_status prepare_chain(rcp_scene* s, Workspace& ws, int W, int H, int mode, hipStream_t stream) {
    const Launch lp = launch_params(s, chain_ordered(s));
    size_t need = 0;
    for (const auto& [stats, entry] : {std::pair(false, false), std::pair(false, true), std::pair(true, false)}) {
        ChainGrid g;
        RCP_TRY_STATUS(chain_grid(lp, stats, 1, mode, entry, ~0ull, g));
        need = std::max(need, spill_depth_of(s, g.k) * g.threads());
    }
    rcp_status st = ensure_workspace(s, ws, 0, 0, need, stream);
    if (st != RCP_OK) return st;
    const uint64_t lists = view_entries(W, H, lp.tile_log2w);
    return ensure_tiles(ws, order_entries(W, H, lp.tile_log2w), lists <= kMaxBatchEntries ? lists : 0, stream);
}

namespace {

// The kernels before a one-view chain launch: tile scores and entry lists
// (where there is room for them), then the cost order, or the setup alone.
rcp_status launch_prepare(const rcp_scene* s, const ViewDev& view, uint32_t n_items, uint32_t* order, float4* entries,
                          ViewDev* table, uint32_t* begin, uint32_t* fetch, unsigned long long* stats,
                          hipStream_t stream) {
    const uint32_t n_tiles = n_items >> 6;
    // tile scores in the second half of the order buffer, the order in the first
    uint32_t* score = order ? order + n_tiles : nullptr;
    const uint32_t score_blocks = order ? (8 * n_tiles + kScoreBlock - 1) / kScoreBlock : 0u;
    const uint32_t n_entries = entries ? (uint32_t)view_entries(view.W, view.H, view.tile_log2w) : 0u;
    const uint32_t entry_blocks = (n_entries + kEntryGroups - 1) / kEntryGroups;
    size_t smem = order ? sizeof(uint32_t) * s->occ.words : 0;
    if (entries) smem = std::max(smem, sizeof(EntryLds) * kEntryGroups);
    hipLaunchKernelGGL(k_prepare, dim3(score_blocks + entry_blocks + (order ? 0u : 1u)), dim3(kScoreBlock), smem, stream,
                       view, s->occ, s->dev, n_tiles, score, score_blocks, entries, n_entries, entry_blocks, table, begin,
                       n_items, fetch, stats);
    if (order)
        hipLaunchKernelGGL(k_band_order, dim3(kFetchParts + 1), dim3(1024), 0, stream, (const uint32_t*)score, n_items,
                           order, view, table, begin, fetch, stats);
    RCP_CHECK_LAUNCH();
    return RCP_OK;
}

// Enqueue the setup kernels and the chain launch of one view on a workspace
// that already fits the grid.
rcp_status launch_one_view(rcp_scene* s, Workspace& w, const Launch& lp, const ChainGrid& g, const Camera& cam,
                           int W, int H, int K, const Disp& disp, float* out_images, int32_t* out_ids, bool stats,
                           hipStream_t stream) {
    const ViewDev view = view_of(s, cam, W, H, K, disp, out_images, out_ids, lp.tile_log2w);
    ChainArgs a{};
    a.sc = s->dev;
    a.sc.top_count = lp.top_count;
    a.views = (const ViewDev*)w.view;
    a.begin = (const uint32_t*)((char*)w.view + ((sizeof(ViewDev) + 63) & ~(size_t)63));
    a.n_views = 1;
    a.n_items = (uint32_t)view_items(view);
    a.fetch = w.counters;
    a.refill_min = lp.refill_min;
    set_take(s, a, g, K);
    a.exit_lanes = (uint32_t)lp.exit_lanes;
    a.spill = w.spill;
    a.spill_stride = g.threads();
    a.stats = stats ? w.stats : nullptr;
    const uint32_t n_tiles = a.n_items >> 6;
    const bool ordered = s->tuning.tile_order && s->occ.bits && w.order && w.order_cap >= 2 * (size_t)n_tiles && n_tiles > 0;
    a.order = ordered ? w.order : nullptr;
    a.entries = g.k.entry ? w.entries : nullptr;
    RCP_TRY_STATUS(launch_prepare(s, view, a.n_items, ordered ? w.order : nullptr, g.k.entry ? w.entries : nullptr,
                                  (ViewDev*)a.views, (uint32_t*)a.begin, w.counters, a.stats, stream));
    return launch_chain(g, stream, a);
}

// Whether a view's rays can start in entry lists held by a buffer of `cap`
// float4.
bool entries_fit(const rcp_scene* s, const float4* buf, size_t cap, uint64_t n) {
    return s->dev.n_nodes > 0 && buf && cap >= kEntryStride * n;
}

template <int MODE>
void launch_direct_mode(const rcp_scene* s, const ViewDev& v, int lanes, hipStream_t stream) {
    const uint64_t threads = (uint64_t)v.W * (uint64_t)v.H * (uint64_t)lanes;
    const dim3 grid((unsigned)((threads + kBlock - 1) / kBlock));
    switch (lanes) {
        case 64: hipLaunchKernelGGL((k_direct<MODE, 64>), grid, dim3(kBlock), 0, stream, s->dev, v); break;
        case 16: hipLaunchKernelGGL((k_direct<MODE, 16>), grid, dim3(kBlock), 0, stream, s->dev, v); break;
        default: hipLaunchKernelGGL((k_direct<MODE, 4>), grid, dim3(kBlock), 0, stream, s->dev, v); break;
    }
}

// Lanes per pixel of the direct kernel, or 0 where the tree is faster.
//
// Its time is that of the pixels times triangles it tests in the first pass
// (0.78 T tests/s; the later ones trace only what moves); the tree's is a chain
// of dependent loads per pass, the longer the more nodes and triangles a ray is
// expected to visit (ray_work, the SAH cost with all costs 1): 10-20 for a
// terrain of up to 100,000 triangles, about three quarters of the triangle
// count for a soup of large triangles.  Microseconds, direct / tree:
//   terrain, 1024 triangles (ray_work 12), K = 6: 64 x 64 42 / 190, 128 x 128
//     99 / 200, 320 x 200 246 / 200; 4096 triangles: 64 x 64 130 / 210, 128 x 128
//     375 / 230; 256 triangles: 320 x 200 85 / 190, 640 x 400 224 / 190
//   soup, 256 triangles (209), K = 6: 64 x 64 17 / 314, 720 x 480 156 / 668,
//     1280 x 720 412 / 779; 2500 (1888), 720 x 480: K = 1 1116 / 756, K = 6 1418 / 3584;
//     16384 (11959): 400 x 300 K = 1 2591 / 2585, 720 x 480 K = 2 7780 / 5981, K = 6
//     9580 / 16650; 65536: 320 x 200 K = 1 6019 / 6324; 262144: 160 x 100 K = 1
//     7947 / 11090, K = 6 16083 / 56382
// so it is taken for no more triangles than a group tests in the time the tree's
// passes take at least (4096, or 16 per unit of ray_work, up to the 262144 it was
// measured at), up to 20M tests in the first pass or half a million per unit of
// ray_work, and no more than the tree's K passes take: the last line, which
// grows more slowly than the ray_work, because a ray's closest hit ends it
// before most of the boxes that it would cross.
// 64 lanes per pixel leave few pixels per wave, which small frames want; 16
// are faster from about 32K pixels on, 4 for large frames of few triangles
// (128 triangles: 640 x 400 104 / 77 with 4 / 16 lanes, 1280 x 720 227 / 251).
int direct_lanes(const rcp_scene* s, int W, int H, int K) {
    const double tris = s->dev.n_tris, pixels = (double)W * H, work = s->ray_work;
    if (tris < 1.0 || tris > std::min(std::max(4096.0, 16.0 * work), 262144.0)) return 0;
    const double tests = pixels * tris;
    if (tests > std::max(20e6, 0.5e6 * work) || tests > 6.5e9) return 0;
    if (tests > K * std::min({0.125e9 + 0.19e6 * work, 1.2e9 + 0.065e6 * work, 5e9})) return 0;
    // (the hook that fails allocations is there for the paths that make some)
    if (alloc_hook_armed()) return 0;
    if (tris <= 64.0) return pixels <= 4e5 ? 16 : 4;
    return pixels <= 32768.0 ? 64 : (tris > 128.0 || pixels <= 4e5 ? 16 : 4);
}

// A direct launch of more tests than this is kept apart from a server's other
// launches (BatchWorkspace::alone).
constexpr double kAloneTests = 50e6;

rcp_status launch_direct(const rcp_scene* s, const Camera& cam, int W, int H, int K, const Disp& disp, float* out_images,
                         int32_t* out_ids, int lanes, hipStream_t stream) {
    const ViewDev v = view_of(s, cam, W, H, K, disp, out_images, out_ids, 3);
    switch (disp.mode) {
        case RCP_MODE_DEPTH: launch_direct_mode<RCP_MODE_DEPTH>(s, v, lanes, stream); break;
        case RCP_MODE_NORMAL: launch_direct_mode<RCP_MODE_NORMAL>(s, v, lanes, stream); break;
        default: launch_direct_mode<RCP_MODE_COLOR>(s, v, lanes, stream); break;
    }
    RCP_CHECK_LAUNCH();
    return RCP_OK;
}

}  // namespace

rcp_status render_chain(rcp_scene* s, Workspace& w, const Camera& cam, int W, int H, int K, const Disp& disp,
                        float* out_images, int32_t* out_ids, unsigned long long* host_counts, hipStream_t stream) {
    const bool stats = host_counts != nullptr;
    const int lanes = stats ? 0 : direct_lanes(s, W, H, K);
    if (lanes > 0) return launch_direct(s, cam, W, H, K, disp, out_images, out_ids, lanes, stream);
    const Launch lp = launch_params(s, chain_ordered(s));
    const uint64_t n_entries = view_entries(W, H, lp.tile_log2w), items = frame_items(W, H, lp.tile_log2w);
    ChainGrid g;
    bool entry = !stats && s->dev.n_nodes > 0 && n_entries <= kMaxBatchEntries;
    if (entry) {
        RCP_TRY_STATUS(chain_grid(lp, stats, 1, disp.mode, true, items, g));
        entry = lists_pay(s, disp.mode, view_spread_angle(s, cam, W, H, disp), K, items, g.lanes);
    }
    rcp_status st = ensure_tiles(w, order_entries(W, H, lp.tile_log2w), entry ? n_entries : 0, stream);
    if (st != RCP_OK) return st;
    if (!entry || !entries_fit(s, w.entries, w.entry_cap, n_entries))
        RCP_TRY_STATUS(chain_grid(lp, stats, 1, disp.mode, false, items, g));
    st = ensure_workspace(s, w, 0, 0, spill_depth_of(s, g.k) * g.threads(), stream);
    if (st != RCP_OK) return st;
    st = launch_one_view(s, w, lp, g, cam, W, H, K, disp, out_images, out_ids, stats, stream);
    if (st != RCP_OK) return st;
    if (stats) {
        RCP_HIP(hipMemcpyAsync(host_counts, w.stats, sizeof(unsigned long long) * kStatCols * K,
                               hipMemcpyDeviceToHost, stream));
        RCP_HIP(hipStreamSynchronize(stream));
        return take_device_error(s);
    }
    return RCP_OK;
}

rcp_status render_chain_fixed(rcp_scene* s, Workspace& w, const Camera& cam, int W, int H, int K,
                              const Disp& disp, float* out_images, int32_t* out_ids, hipStream_t stream) {
    // the cost order where the workspace's order area holds the view's tiles
    const bool ordered = chain_ordered(s) && w.order &&
                         w.order_cap >= order_entries(W, H, launch_params(s, true).tile_log2w);
    const Launch lp = launch_params(s, ordered);
    int dev = 0, cus = 0;
    RCP_HIP(hipGetDevice(&dev));
    RCP_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    // as many workgroups as the overflow area holds (the grid size changes
    // the speed only), but at least one per compute unit.  The kernel with
    // entry lists keeps fewer stack entries in LDS and needs more of the area:
    // it is taken where four workgroups per compute unit fit.
    // (The area for the lists lies right before the overflow area, and is
    // added to it when there are none.)
    ChainGrid g;
    size_t per_block = 0, fit = 0;
    const uint64_t items = frame_items(W, H, lp.tile_log2w);
    for (const bool entry : {true, false}) {
        if (entry && !entries_fit(s, w.entries, w.entry_cap, view_entries(W, H, lp.tile_log2w))) continue;
        if (!entry && w.entries) {
            w.spill = (int32_t*)w.entries;
            w.spill_cap += w.entry_cap * (sizeof(float4) / sizeof(int32_t));
        }
        RCP_TRY_STATUS(chain_grid(lp, false, 1, disp.mode, entry, items, g));
        if (entry && !lists_pay(s, disp.mode, view_spread_angle(s, cam, W, H, disp), K, items, g.lanes)) continue;
        per_block = spill_depth_of(s, g.k) * (size_t)g.k.block;
        fit = w.spill_cap / per_block;
        if (entry && fit * g.k.block >= 4 * (size_t)cus * kBlock) break;
    }
    if (fit < (size_t)cus) {
        set_error("the scene's traversal stack needs %zu bytes of overflow area per compute unit's workgroup; "
                  "the preallocated scratch holds %zu for %d compute units",
                  per_block * sizeof(int32_t), w.spill_cap * sizeof(int32_t), cus);
        return RCP_ERR_INVALID_ARGUMENT;
    }
    if (const int lanes = direct_lanes(s, W, H, K))
        return launch_direct(s, cam, W, H, K, disp, out_images, out_ids, lanes, stream);
    if ((size_t)g.blocks > fit) g.blocks = (int)fit;
    return launch_one_view(s, w, lp, g, cam, W, H, K, disp, out_images, out_ids, false, stream);
}

namespace {

// Grow a batch buffer in stream order.
template <typename T>
rcp_status grow(T** p, size_t& cap, size_t need, size_t bytes_each, hipStream_t stream) {
    if (need <= cap && *p) return RCP_OK;
    stream_free((void*)*p, stream);
    *p = nullptr;
    cap = 0;
    rcp_status st = stream_alloc((void**)p, bytes_each * need, stream);
    if (st != RCP_OK) return st;
    cap = need;
    return RCP_OK;
}

size_t view_table_bytes(size_t n_views) {
    return ((sizeof(ViewDev) * n_views + 255) & ~(size_t)255) + sizeof(uint32_t) * (n_views + 3);
}

}  // namespace

rcp_status prepare_batch_workspace(rcp_scene* s, BatchWorkspace& ws, int n_views, size_t lists, hipStream_t stream) {
    const bool with_staging = lists > 0;
    const Launch lp = launch_params(s);
    size_t spill_need = 0;
    for (int mode = 0; mode < 3; ++mode)
        for (int nv : {1, 2})
            for (const bool entry : {false, true}) {
                ChainGrid g;
                RCP_TRY_STATUS(chain_grid(lp, false, nv, mode, entry, ~0ull, g));
                spill_need = std::max(spill_need, spill_depth_of(s, g.k) * g.threads());
            }
    rcp_status st = RCP_OK;
    if ((size_t)n_views > ws.view_cap || !ws.views) {
        stream_free(ws.views, stream);
        ws.views = nullptr;
        ws.view_cap = 0;
        st = stream_alloc(&ws.views, view_table_bytes((size_t)n_views), stream);
        if (st == RCP_OK) ws.view_cap = (size_t)n_views;
    }
    size_t fetch_cap = ws.fetch ? kFetchWords * 3 : 0;
    if (st == RCP_OK) st = grow(&ws.fetch, fetch_cap, kFetchWords * 3, sizeof(uint32_t), stream);
    if (st == RCP_OK)
        st = grow(&ws.spill, ws.spill_cap, spill_need, sizeof(int32_t), stream);
    if (st == RCP_OK && with_staging && ws.order_cap < 2 * kServerOrderTiles)
        st = grow(&ws.order, ws.order_cap, 2 * kServerOrderTiles, sizeof(uint32_t), stream);
    if (st == RCP_OK && with_staging && !ws.staging) {
        if (alloc_hook_fails()) {
            set_error("pinned host allocation failed (test hook)");
            return RCP_ERR_OUT_OF_MEMORY;
        }
        RCP_HIP(hipHostMalloc(&ws.staging, view_table_bytes((size_t)n_views), hipHostMallocDefault));
    }
    if (st == RCP_OK && with_staging && ws.entry_cap < kEntryStride * lists) {
        // without room for entry lists the rays start at the root
        const rcp_status se = grow(&ws.entries, ws.entry_cap, kEntryStride * lists, sizeof(float4), stream);
        if (se != RCP_OK && se != RCP_ERR_OUT_OF_MEMORY) st = se;
    }
    return st;
}

namespace {

Camera camera_of(const rcp_view& v) {
    Camera c{};
    for (int a = 0; a < 3; ++a) {
        c.eye[a] = v.camera.eye[a];
        c.right[a] = v.camera.right[a];
        c.up[a] = v.camera.up[a];
        c.forward[a] = v.camera.forward[a];
    }
    c.th = v.camera.tan_half_fovy;
    return c;
}

Disp disp_of(const rcp_view& v) { return Disp{v.disp.lambda_eye, v.disp.lambda_dir, v.disp.z0, v.disp.mode}; }

// Whether the rays of a batch are better off in entry lists (see render_batch).
rcp_status views_want_lists(const rcp_scene* s, const Launch& lp, const rcp_view* views, int n_views, bool& want) {
    want = s->dev.n_nodes > 0;
    if (!want) return RCP_OK;
    const auto spread = [&](const rcp_view& v) { return view_spread_angle(s, camera_of(v), v.W, v.H, disp_of(v)); };
    if (n_views == 1) {
        const uint64_t items = frame_items(views->W, views->H, lp.tile_log2w);
        ChainGrid g;
        RCP_TRY_STATUS(chain_grid(lp, false, 1, views->disp.mode, true, items, g));
        want = lists_pay(s, views->disp.mode, spread(*views), views->K, items, g.lanes);
    } else if (!visits_much(s) && s->dev.max_depth <= 12u) {
        want = false;
        for (int i = 0; i < n_views && !want; ++i) want = spread(views[i]) <= 0.1;
    }
    return RCP_OK;
}

}  // namespace

rcp_status batch_route(const rcp_scene* s, const rcp_view* views, int n_views, Route& r) {
    if (n_views == 1 && direct_lanes(s, views->W, views->H, views->K) > 0) {
        r = Route::direct;
        return RCP_OK;
    }
    bool lists = false;
    RCP_TRY_STATUS(views_want_lists(s, launch_params(s), views, n_views, lists));
    r = lists ? Route::lists : Route::root;
    return RCP_OK;
}

rcp_status render_batch(rcp_scene* s, const rcp_view* views, int n_views, BatchWorkspace& ws, hipStream_t stream) {
    const Launch lp = launch_params(s);
    // views grouped by displacement mode, one launch per mode present
    std::vector<int> order((size_t)n_views);
    for (int i = 0; i < n_views; ++i) order[(size_t)i] = i;
    std::stable_sort(order.begin(), order.end(),
                     [&](int p, int q) { return views[p].disp.mode < views[q].disp.mode; });
    std::vector<ViewDev> hv((size_t)n_views);
    std::vector<uint32_t> hb((size_t)n_views + 3);   // begin arrays of the groups, back to back
    struct Group { int mode, first, count; size_t bofs; uint32_t items; int passes; };   // passes: the most of any view
    std::vector<Group> groups;
    uint64_t items = 0, n_entries = 0;
    size_t bofs = 0;
    for (int j = 0; j < n_views; ++j) {
        const rcp_view& vi = views[order[(size_t)j]];
        if (groups.empty() || groups.back().mode != vi.disp.mode) {
            if (!groups.empty()) {
                hb[bofs++] = (uint32_t)items;
                groups.back().items = (uint32_t)items;
            }
            groups.push_back(Group{vi.disp.mode, j, 0, bofs, 0, 0});
            items = 0;
        }
        hv[(size_t)j] = view_of(s, camera_of(vi), vi.W, vi.H, vi.K, disp_of(vi), vi.out_images, vi.out_ids, lp.tile_log2w);
        hv[(size_t)j].entry_base = (uint32_t)std::min<uint64_t>(n_entries, 0xFFFFFFFFull);
        n_entries += view_entries(vi.W, vi.H, lp.tile_log2w);
        hb[bofs++] = (uint32_t)items;
        items += view_items(hv[(size_t)j]);
        if (items >= (1ull << 32) - (1ull << 24)) {   // headroom for fetches past the end
            set_error("a batch of mode %d holds %llu work items (limit 2^32 - 2^24)", vi.disp.mode,
                      (unsigned long long)items);
            return RCP_ERR_INVALID_ARGUMENT;
        }
        groups.back().count++;
        groups.back().passes = std::max(groups.back().passes, vi.K);
    }
    hb[bofs++] = (uint32_t)items;
    groups.back().items = (uint32_t)items;

    ws.alone = false;
    if (n_views == 1)
        if (const int lanes = direct_lanes(s, views[0].W, views[0].H, views[0].K)) {
            ws.alone = (double)views[0].W * views[0].H * s->dev.n_tris > kAloneTests;
            return launch_direct(s, hv[0].cam, views[0].W, views[0].H, views[0].K, disp_of(views[0]), views[0].out_images,
                                 views[0].out_ids, lanes, stream);
        }

    // entry lists for all views, up to kMaxBatchEntries (a server slot: as many
    // as it was sized for); without room for them the rays start at the root, and
    // so they do where the lists of none would pay (several views share a launch,
    // which lists make faster even where a single one's do not: soups 1.1-2.2
    // times; 16 views of a terrain of 5000 triangles at a spread of 0.05 1.15, at
    // 0.2 1.02 with lists and 1.13 from the root, of 100,000 1.16, 0.99 and 0.98;
    // 4 views 0.97, 0.85 and 0.97, 0.96, 0.93 and 0.97)
    bool want = false;
    RCP_TRY_STATUS(views_want_lists(s, lp, views, n_views, want));
    if (want && !ws.staging && n_entries <= kMaxBatchEntries && ws.entry_cap < kEntryStride * n_entries) {
        const rcp_status se = grow(&ws.entries, ws.entry_cap, kEntryStride * (size_t)n_entries, sizeof(float4), stream);
        if (se != RCP_OK && se != RCP_ERR_OUT_OF_MEMORY) return se;
    }
    const bool entry = want && entries_fit(s, ws.entries, ws.entry_cap, n_entries);
    // From the root the views go out row by row.  (16 views of 1M triangles 4.50
    // ms against 4.68 by columns, of 4M 5.44 and 5.80.)
    if (!entry)
        for (ViewDev& v : hv) v.super_rows = 0;
    size_t spill_need = 0;
    std::vector<ChainGrid> grids(groups.size());
    for (size_t g = 0; g < groups.size(); ++g) {
        rcp_status st = chain_grid(lp, false, groups[g].count, groups[g].mode, entry, groups[g].items, grids[g]);
        if (st != RCP_OK) return st;
        spill_need = std::max(spill_need, spill_depth_of(s, grids[g].k) * grids[g].threads());
    }

    // buffers grow in stream order (a server's slots are sized at creation
    // and never grow here)
    if ((size_t)n_views > ws.view_cap || !ws.views) {
        if (ws.staging) {
            set_error("a batch of %d views exceeds the %zu views its workspace was sized for", n_views, ws.view_cap);
            return RCP_ERR_INTERNAL;
        }
        stream_free(ws.views, stream);
        ws.views = nullptr;
        ws.view_cap = 0;
        rcp_status st = stream_alloc(&ws.views, view_table_bytes((size_t)n_views), stream);
        if (st != RCP_OK) return st;
        ws.view_cap = (size_t)n_views;
    }
    if (ws.staging && spill_need > ws.spill_cap) {
        set_error("the batch needs more stack overflow area than its workspace was sized for (launch parameters "
                  "changed since)");
        return RCP_ERR_INTERNAL;
    }
    size_t fetch_cap = ws.fetch ? kFetchWords * 3 : 0;
    rcp_status st = grow(&ws.fetch, fetch_cap, kFetchWords * 3, sizeof(uint32_t), stream);
    if (st == RCP_OK) st = grow(&ws.spill, ws.spill_cap, spill_need, sizeof(int32_t), stream);
    if (st != RCP_OK) return st;
    ViewDev* d_views = (ViewDev*)ws.views;
    const size_t begin_ofs = (sizeof(ViewDev) * (size_t)n_views + 255) & ~(size_t)255;
    uint32_t* d_begin = (uint32_t*)((char*)ws.views + begin_ofs);
    // One view (a lone request of a server, say) is a single render: its
    // tiles go out in cost order, as rcp_render's do, with the launch
    // parameters of that order.  A server slot, whose buffers never grow,
    // keeps the screen order for a view beyond its order buffer.
    const uint32_t n_tiles1 = n_views == 1 ? groups[0].items >> 6 : 0u;
    bool ordered1 = n_views == 1 && s->tuning.tile_order && s->occ.bits && n_tiles1 > 0;
    if (ordered1 && 2 * (size_t)n_tiles1 > ws.order_cap) {
        if (ws.staging) ordered1 = false;
        else if ((st = grow(&ws.order, ws.order_cap, 2 * (size_t)n_tiles1, sizeof(uint32_t), stream)) != RCP_OK)
            return st;
    }
    const Launch lpr = ordered1 ? launch_params(s, true) : lp;
    if (n_views == 1) {
        // the view's table is written from the by-value argument, with no host copy
        RCP_TRY_STATUS(launch_prepare(s, hv[0], groups[0].items, ordered1 ? ws.order : nullptr,
                                      entry ? ws.entries : nullptr, d_views, d_begin, ws.fetch, nullptr, stream));
    } else if (ws.staging) {
        // a server slot: copy from its pinned table (the slot's previous
        // launch, the last reader, has finished)
        std::memcpy(ws.staging, hv.data(), sizeof(ViewDev) * (size_t)n_views);
        std::memcpy((char*)ws.staging + begin_ofs, hb.data(), sizeof(uint32_t) * bofs);
        RCP_HIP(hipMemcpyAsync(d_views, ws.staging, begin_ofs + sizeof(uint32_t) * bofs, hipMemcpyHostToDevice,
                               stream));
        hipLaunchKernelGGL(k_clear_chain, dim3(1), dim3(64), 0, stream, ws.fetch, (int)groups.size(),
                           (unsigned long long*)nullptr);
    } else {
        // pageable sources: the copies have read them when the calls return
        RCP_HIP(hipMemcpyAsync(d_views, hv.data(), sizeof(ViewDev) * (size_t)n_views, hipMemcpyHostToDevice,
                               stream));
        RCP_HIP(hipMemcpyAsync(d_begin, hb.data(), sizeof(uint32_t) * bofs, hipMemcpyHostToDevice, stream));
        hipLaunchKernelGGL(k_clear_chain, dim3(1), dim3(64), 0, stream, ws.fetch, (int)groups.size(),
                           (unsigned long long*)nullptr);
    }
    if (entry && n_views > 1)
        hipLaunchKernelGGL(k_batch_entries, dim3((unsigned)((n_entries + kEntryGroups - 1) / kEntryGroups)),
                           dim3(kScoreBlock), sizeof(EntryLds) * kEntryGroups, stream, (const ViewDev*)d_views, n_views,
                           s->dev, ws.entries, (uint32_t)n_entries);
    RCP_CHECK_LAUNCH();
    for (size_t g = 0; g < groups.size(); ++g) {
        ChainArgs a{};
        a.sc = s->dev;
        a.sc.top_count = lp.top_count;
        a.views = d_views + groups[g].first;
        a.begin = d_begin + groups[g].bofs;
        a.n_views = groups[g].count;
        a.n_items = groups[g].items;
        a.fetch = ws.fetch + kFetchWords * g;
        a.refill_min = lpr.refill_min;
        set_take(s, a, grids[g], groups[g].passes);
        a.exit_lanes = (uint32_t)lpr.exit_lanes;
        a.spill = ws.spill;
        a.spill_stride = grids[g].threads();
        a.order = ordered1 ? ws.order : nullptr;
        a.entries = entry ? ws.entries : nullptr;
        rcp_status st2 = launch_chain(grids[g], stream, a);
        if (st2 != RCP_OK) return st2;
    }
    return RCP_OK;
}

void free_batch_workspace(BatchWorkspace& ws, hipStream_t stream) {
    stream_free(ws.order, stream);
    stream_free(ws.entries, stream);
    stream_free(ws.views, stream);
    stream_free(ws.fetch, stream);
    stream_free(ws.spill, stream);
    if (ws.staging) (void)hipHostFree(ws.staging);
    ws = BatchWorkspace{};
}

}  // namespace rcp
