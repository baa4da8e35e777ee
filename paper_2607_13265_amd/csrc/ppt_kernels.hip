// ppt_kernels.hip -- wavefront kernels of the differentiable polarized path tracer (gfx950).
//
// Paths are processed in chunks of a flat index space that spans every view of a plan (the
// batch): path g = (view, crop pixel, sample), samples fastest.  Per chunk and bounce:
//   k_extend   closest-hit traversal of the queued rays (lean kernel, LDS traversal stack),
//              from the second bounce on together with the any-hit traversal of the previous
//              bounce's next-event rays,
//   k_compact  from the one-byte outcome that traversal leaves per slot: misses end their path,
//              hits go to the shading queue,
//   k_shade    vertex sampling and Mueller weights; appends continuing paths to the next ray
//              queue and next-event rays to the shadow queue (workgroup-staged queues, one
//              global atomic per flush).
// Render (Sec. 3.1, Eq. 2): the state carries the prefix Mueller product beta and the radiance
// sum; k_accum reduces the samples of each pixel.  Backward (Sec. 3.2, 4.3, Fig. 2): the primal
// pass keeps a hit record per vertex and carries the path's adjoint row forward; one walk from the last
// vertex to the first (k_adjoint_deep, k_adjoint_first) evaluates each vertex again (no second
// traversal), differentiates it against the suffix radiance L[b+1] it carries, and advances
// L[b] = E_b + W_b L[b+1].  The light-stage variants and the comparators cache W_b and E_b per vertex instead:
// k_fold folds them into suffixes and queues the paths, k_replay replays them forward.  No Mueller
// matrix is inverted.
// A chunk of few paths runs each path's bounces in one launch (k_paths, k_adjoint_paths).
#include "ppt_device.h"

#include <mutex>

namespace ppt {

// ============================================================================ wave helpers
// Workgroup-aggregated counters: one global atomic per workgroup and nonzero counter.  Every
// thread of the workgroup must call it (it synchronizes the workgroup).
struct Count {
    uint32_t c[ST_COUNT];
    DEV Count() {
#pragma unroll
        for (int k = 0; k < ST_COUNT; ++k) c[k] = 0u;
    }
};
DEV void flush_stats(Stats* st, const Count& n) {
    if (!st) return;
    __shared__ uint32_t part[ST_COUNT];
    if (threadIdx.x < ST_COUNT) part[threadIdx.x] = 0u;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ST_COUNT; ++k) {
        uint32_t v = wave_sum_u(n.c[k]);
        if (lane_id() == 0 && v) atomicAdd(&part[k], v);
    }
    __syncthreads();
    if (threadIdx.x < ST_COUNT && part[threadIdx.x]) atomicAdd(&st->c[threadIdx.x], (unsigned long long)part[threadIdx.x]);
}

// Workgroup queue in LDS: lanes append with one LDS atomic per wavefront; the buffer is copied
// to the global queue (one global atomic per flush) when another workgroup iteration might not
// fit, and at the end.
constexpr int QBUF = 2048;
struct BlockQueue {
    int n, base;
    int buf[QBUF];
};
DEV void bq_push(BlockQueue& q, bool pred, int slot) {
    unsigned long long m = __ballot(pred);
    int wb = 0;
    if (lane_id() == 0 && m) wb = atomicAdd(&q.n, (int)__popcll(m));
    wb = __shfl(wb, 0, WAVE);
    if (pred) q.buf[wb + (int)__popcll(m & ((1ull << lane_id()) - 1ull))] = slot;
}
// all threads of the workgroup call it after the pushes of an iteration
DEV void bq_flush(BlockQueue& q, int* gcount, int* gqueue, bool force) {
    __syncthreads();
    int n = q.n;
    if (n > 0 && (force || n > QBUF - BLOCK)) {
        if (threadIdx.x == 0) q.base = atomicAdd(gcount, n);
        __syncthreads();
        int b = q.base;
        for (int k = threadIdx.x; k < n; k += BLOCK) gqueue[b + k] = q.buf[k];
        __syncthreads();
        if (threadIdx.x == 0) q.n = 0;
        __syncthreads();
    }
}
DEV void sig_add(uint64_t& h, uint32_t x) {
#pragma unroll
    for (int i = 0; i < 4; ++i) { h ^= (x >> (8 * i)) & 0xffu; h *= 1099511628211ull; }
}

// Work distribution of the persistent kernels.  Only the first ceil(n / BLOCK) workgroups take
// part (fetch_active; the others leave at once).  Active wavefront w first takes the static batch
// [w * s, (w + 1) * s) with s = n / active wavefronts rounded up and kept in [FETCH_MIN, batch];
// positions beyond all static batches are handed out in batches through one atomic on a counter that an earlier
// kernel cleared, one of WORK_SHARDS: wavefront w takes from counter w mod WORK_SHARDS, whose t-th ticket is
// batch t WORK_SHARDS + (w + t) mod WORK_SHARDS, so that no counter's batches keep to one part of an image.  A
// wavefront stops at its counter's first ticket beyond the queue; fewer than WORK_SHARDS wavefronts share fewer counters.
// On a single counter the additions (10 ns each, one after the other) took most of a camera-ray launch and
// forced batches of 256; with 16 counters and batches of 64 (128 where each wavefront takes many) the
// camera rays of 4.2M paths take 181 us instead of 340, those of the 128-view batch 6.1 ms a step
// instead of 7.0, the walk of the 921,600 depth-128 paths 3.7 ms instead of 4.7, and launches end evenly.
// (The forward replay and the tape's sweep keep batches of FETCH_REPLAY: with the paths of a wavefront handed
// out together the hybrid replay's lanes meet their blocks together, 11.6 ms against 15.5.)
// A queue of up to one batch per wavefront is covered by the static batches alone, with no atomic.  A
// wavefront gives its positions, in order, to its lanes that have no work; every lane of the wavefront
// must call take().
//
// Traversal spreads a queue that does not fill the GPU (least > 0): with fewer rays than lanes, a launch
// lasts as long as its slowest wavefront, whose lanes wait for each other's descents and leaves, so
// a wavefront takes only n / SPREAD_WAVES positions, and at least `least`, 2, in a scene whose tree is deep
// enough for rays to differ.  A 5,917-path preview 304 -> 229 us, a 28,512-path step 1040 -> 873 us (launches per
// bounce); from SPREAD_WAVES full wavefronts on, two per SIMD, full wavefronts are the faster.  Not in a shallow one,
// whose rays take alike: with 8 rays a wavefront a traversal launch through 20 polarizer sheets took 18.9 us instead of
// 14.8 (P-RB of 47,616 paths in chunks of 1,024 30.5 ms against 25.5; P-PRB of 2,304 paths through 85 sheets 5.10
// against 4.91), 16,384 paths among 80 triangles gained 1 to 3 %.
constexpr int FETCH_MIN = WAVE, FETCH_BATCH = 2 * WAVE, FETCH_REPLAY = 4 * WAVE, FETCH_SHARE = 8;
constexpr int SPREAD_DEEP = 2, SPREAD_WAVES = 2048, SHALLOW_STACK = 10;
DEV int spread_least(const WArgs& A) { return A.stack_cap > SHALLOW_STACK ? SPREAD_DEEP : 0; }
DEV int fetch_min(int n, int least) { return least ? max(least, min(FETCH_MIN, (n + SPREAD_WAVES - 1) / SPREAD_WAVES)) : FETCH_MIN; }
DEV int fetch_blocks(int n, int per_wave) {
    const int per_block = per_wave * (BLOCK / WAVE);
    return max(1, min((int)gridDim.x, (n + per_block - 1) / per_block));
}
DEV bool fetch_active(int n, int least = 0) { return (int)blockIdx.x < fetch_blocks(n, fetch_min(n, least)); }
DEV int* work_counter(const PathState& S, int set, int shard) {
    return S.counts + WORK_FIRST + (set * WORK_SHARDS + shard) * WORK_LINE;
}
// the batch of the next ticket of the wavefront's counter, wave-uniform (every lane of the wavefront calls it);
// waves: the wavefronts that take tickets
DEV int work_ticket(const PathState& S, int set, int wave, int waves) {
    const int shards = work_shards(waves), shard = wave & (shards - 1);
    int t = 0;
    if (lane_id() == 0) t = atomicAdd(work_counter(S, set, shard), 1);
    return work_batch(__builtin_amdgcn_readfirstlane(t), shard, shards);
}
DEV int wave_number() { return blockIdx.x * (BLOCK / WAVE) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE)); }
struct WaveFetch {
    int c, cend;    // the wavefront's current batch [c, cend)
    int stat;       // positions covered by the static batches
    int batch;      // positions per ticket
    int waves;      // wavefronts that take part
    bool exhausted;
    DEV explicit WaveFetch(int n, int least = 0, bool replay = false) {
        const int smin = fetch_min(n, least);
        waves = fetch_blocks(n, smin) * (BLOCK / WAVE);
        const int w = wave_number();  // (known uniform: the fetch state stays in scalar registers)
        batch = replay ? FETCH_REPLAY : max(FETCH_MIN, min(FETCH_BATCH, n / (FETCH_SHARE * waves)));
        int sb = (n + waves - 1) / waves;
        sb = sb < smin ? smin : (sb > batch ? batch : sb);
        stat = waves * sb;
        c = min(w * sb, n);
        cend = min(c + sb, n);
        exhausted = n <= stat;
    }
    DEV int take(bool need, int n, const PathState& S, int set) {
        const unsigned long long m = __ballot(need);
        const int k = (int)__popcll(m), rank = (int)__popcll(m & ((1ull << lane_id()) - 1ull));
        const int rem = cend - c;
        int nb = -1;
        if (k > rem && !exhausted) nb = stat + work_ticket(S, set, wave_number(), waves) * batch;
        int idx = -1;
        if (need) {
            if (rank < rem) idx = c + rank;
            else if (nb >= 0 && nb + (rank - rem) < min(nb + batch, n)) idx = nb + (rank - rem);
        }
        if (nb >= 0) {
            if (nb >= n) { exhausted = true; c = cend = 0; }
            else { cend = min(nb + batch, n); c = min(nb + (k - rem), cend); }
        } else {
            c = min(c + k, cend);
        }
        return idx;
    }
    DEV bool more() const { return !exhausted || c < cend; }  // wave-uniform
};

// Path keys of a global path index of view V.  The index within a view fits 32 bits (checked when the
// plan is made).
struct PathId { int lx, ly; uint32_t smp, pix; };
// n / d for n < 2^31 and inv = 1 / d in double: (n + 1/2) / d lies at least 1 / (2 d) from an integer and the
// product is off by less than 2^-21 / d, so the quotient is exact (4 instructions instead of the about 25 of
// a 32-bit division).
DEV uint32_t div_by(uint32_t n, double inv) { return (uint32_t)(((double)n + 0.5) * inv); }
DEV PathId path_keys(const DevView& V, int64_t g) {
    PathId r;
    const uint32_t local = (uint32_t)(g - V.path_off);
    const uint32_t pl = div_by(local, V.inv_spp);
    r.smp = local - pl * (uint32_t)V.spp;
    r.ly = (int)div_by(pl, V.inv_cw);
    r.lx = (int)(pl - (uint32_t)r.ly * (uint32_t)V.crop_w);
    r.pix = (uint32_t)((V.crop_y0 + r.ly) * V.width + V.crop_x0 + r.lx);
    return r;
}
// The view of a wavefront's paths.  The lanes mostly hold consecutive paths of one view, and go on in
// that view, so the view found last is kept (v and its paths [lo, hi), wave-uniform, in scalar
// registers), and a new one is searched (binary, by scalar loads) only when a path lies outside it.
// A search per wavefront and step by vector loads was a chain of log2(views) round trips: the
// first-vertex kernel of the 128-view batch spent half of its time in it.
struct ViewRange { int v = 0; int64_t lo = 0, hi = 0; };
DEV int64_t read_lane64(int64_t x, int lane) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)x >> 32), lane);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
DEV void view_at(const WArgs& A, int64_t g, ViewRange& R) {  // g wave-uniform
    if (g >= R.lo && g < R.hi) return;
    int lo = 0, hi = A.n_views - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (cval(&A.views[mid].path_off, 0) <= g) lo = mid; else hi = mid - 1;
    }
    R.v = lo;
    R.lo = cval(&A.views[lo].path_off, 0);
    R.hi = lo + 1 < A.n_views ? cval(&A.views[lo + 1].path_off, 0) : INT64_MAX;
}
// The view of path g of an active lane: the wavefront's, or its own where its path lies in another one.
// Every lane of the wavefront calls find(), then an active lane view().
DEV void view_find(const WArgs& A, ViewRange& R, bool active, int64_t g) {
    const uint64_t m = __ballot(active);
    if (m != 0ull) view_at(A, read_lane64(g, __ffsll((long long)m) - 1), R);
}
DEV int lane_view(const WArgs& A, int64_t g) {  // (g of each lane its own)
    int lo = 0, hi = A.n_views - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (gval(&A.views[mid].path_off, 0) <= g) lo = mid; else hi = mid - 1;
    }
    return lo;
}
DEV DevView view_of(const WArgs& A, const ViewRange& R, int64_t g, int& v) {
    DevView V = cval(A.views, R.v);
    v = R.v;
    if (g < R.lo || g >= R.hi) {
        v = lane_view(A, g);
        V = gval(A.views, (size_t)v);
    }
    return V;
}
// f(v, V) for the active lanes, view by view: v and V are the wave-uniform view of the lanes that run it
// (one pass unless the lanes' paths g span views).  Every lane of the wavefront calls it, so that the
// range stays in scalar registers.  EACH: lanes left after VIEW_PASSES views look theirs up each for itself (a
// wavefront of 64 views of one path took 64 passes: render of 300,000 such views 245 -> 393 us).
constexpr int VIEW_PASSES = 4;
template <bool EACH = true, class F>
DEV void for_views(const WArgs& A, ViewRange& R, bool active, int64_t g, F f) {
    bool todo = active;
    for (int pass = 0;; ++pass) {
        const uint64_t m = __ballot(todo);
        if (m == 0ull) break;
        if (EACH && pass == VIEW_PASSES) {
            if (todo) {
                const int v = lane_view(A, g);
                f(v, gval(A.views, (size_t)v));
            }
            break;
        }
        view_at(A, read_lane64(g, __ffsll((long long)m) - 1), R);
        if (todo && g >= R.lo && g < R.hi) {
            const DevView V = cval(A.views, R.v);
            f(R.v, V);
            todo = false;
        }
    }
}

// The call table (parameter pointers, gradient routing) is read for every parameter access; a
// copy in LDS turns those dependent global loads into LDS reads.  All threads call it, followed by
// a workgroup barrier before first use.
DEV void table_to_lds(CallTable* dst, const CallTable* src) {
    const int n = (int)(sizeof(CallTable) / sizeof(int));
    for (int k = threadIdx.x; k < n; k += BLOCK) ((int*)dst)[k] = ((const int*)src)[k];
}

// Record accessors (layouts in ppt_internal.h).
DEV float4* ray_rec(const PathState& S, int i) { return S.ray + (size_t)i * RAY_F4; }
DEV float4* shd_rec(const PathState& S, int i) { return S.shd + (size_t)i * SHD_F4; }
DEV float4* acc_rec(const PathState& S, int i) { return S.acc + (size_t)i * ACC_F4; }
DEV float4* r1_rec(const PathState& S, int i) { return S.acc + (size_t)i * R1_F4; }  // (rank-one render)
// the rank-one render's shadow rays: a dense 32-byte record per slot behind the rank-one records
DEV float4* r1_shd(const PathState& S, int Q, int i) { return S.acc + (size_t)Q * R1_F4 + (size_t)i * 2; }
static_assert(R1_F4 + 2 <= ACC_F4, "the rank-one records and their shadow rays fit in the accumulator array");
// Except for the tape's, bounces use the shadow-record array as two dense arrays (a fold later writes whole
// 128-byte records there): a 32-byte shadow ray per slot, four to a cache line, and behind them the 48 bytes
// that an occluded light sample restores, the path's radiance (full render) or the E_b of an emitting vertex
// (comparators).  The hybrid replay's and the cached backward's bounces use the shadow rays alone.  (In
// whole 128-byte records with the pending next-event part, which traversal read for every ray and added to the
// radiance of the visible ones, the full render of 43M paths of 12 bounces cost 27.4 ms of traversal and 9.1 of shading
// instead of 25.0 and 8.6.)
static_assert(2 + 3 <= SHD_F4, "the dense shadow rays and what they restore fit in the shadow-record array");
DEV float4* shd1_rec(const PathState& S, int i) { return S.shd + (size_t)i * SHD1_F4; }
DEV float4* rest_rec(const PathState& S, int Q, int i) { return S.shd + (size_t)Q * 2 + (size_t)i * 3; }
// cached backward: a vertex's record, and the adjoint row of a vertex after the first (b0 >= 1)
DEV float4* vtx_rec(const PathState& S, int Q, int b0, int i) { return S.vtx + ((size_t)b0 * Q + i) * VTX_F4; }
template <bool R1>
DEV float4* row_rec(const PathState& S, int Q, int b0, int i) {
    return S.row + ((size_t)(b0 - 1) * Q + i) * (R1 ? ROW1_F4 : ROW_F4);
}
DEV float4* cache_rec(const PathState& S, int Q, int b0, int i) {  // b0: 0-based vertex index
    return S.cache + ((size_t)b0 * Q + i) * CACHE_F4;
}
DEV float4* hit_rec(const PathState& S, int Q, int b0, int i) { return S.hits + ((size_t)b0 * Q + i); }
DEV float4* tape_rec(const PathState& S, int Q, int b0, int i) {  // (the tape occupies the cache region)
    return S.cache + ((size_t)b0 * Q + i) * TAPE_F4;
}
DEV float4* ckpt_rec(const PathState& S, int Q, int blk, int i) { return S.ckpt + ((size_t)blk * Q + i) * CKPT_F4; }
DEV float4 f4(float a, float b, float c, float d) { return make_float4(a, b, c, d); }
DEV void ld12(const float4* r, float* v) {
#pragma unroll
    for (int k = 0; k < 3; ++k) { float4 t = r[k]; v[4 * k] = t.x; v[4 * k + 1] = t.y; v[4 * k + 2] = t.z; v[4 * k + 3] = t.w; }
}
DEV void st12(float4* r, const float* v) {
#pragma unroll
    for (int k = 0; k < 3; ++k) r[k] = f4(v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]);
}
// a + b of two rounded values (never contracted with the product that gave one of them)
DEV float add_rounded(float a, float b) {
#pragma clang fp contract(off)
    return a + b;
}
// ray record: origin and direction ([0], [1].xy); keys in [3]
DEV void ray_od(const float4* R, v3& o, v3& d) {
    float4 a = R[0], b = R[1];
    o = mk(a.x, a.y, a.z);
    d = mk(a.w, b.x, b.y);
}
DEV void ray_set(float4* R, v3 o, v3 d, float Cs = 0.0f, float Ss = 0.0f) {
    R[0] = f4(o.x, o.y, o.z, d.x);
    R[1] = f4(d.y, d.z, Cs, Ss);
}

constexpr int VTX_PREV_DELTA = 1 << 26;  // (vertex record: beside the primitive)
constexpr int INFO_DEAD = 1 << 9;
constexpr int INFO_EMIT = 1 << 10;  // (a cached-backward shadow ray's vertex emits: its E_b is kept)
DEV int info_make(int nverts, bool prev_delta, int view) { return nverts | (prev_delta ? 256 : 0) | (view << 12); }

// World of a view: in a scene of one world it comes from the launch arguments (wave-uniform
// scalar loads), otherwise from the world table through the view.
DEV DevWorld world_of(const WArgs& A, int view) {
    if (A.one_world) return A.world0;
    return gval(A.worlds, (size_t)gval(A.views, (size_t)view).world);
}
DEV DevWorld world_of(const WArgs& A, const DevView& V) { return A.one_world ? A.world0 : gval(A.worlds, (size_t)V.world); }

// ============================================================================ chunk start
#ifndef PPT_EXT_TU  // (non-template kernels: in the main compilation unit only)
__global__ void k_reset_counts(int* counts) {
    for (int k = threadIdx.x; k < COUNT_INTS; k += BLOCK) counts[k] = 0;
}

#endif  // PPT_EXT_TU

// ============================================================================ rays of a path
// Begin and end of the rays of path `slot`, between their record and the traversal state T.
//
// Camera ray: generated here, its record written when it is finished.  Returns whether it is traversed (not
// that of a masked path).
DEV bool camera_begin(const WArgs& A, const ViewRange& range, int slot, Trav& T, int& info, Count& cnt) {
    const PathState& S = A.S;
    const int64_t g = A.g0 + slot;
    int v;
    const DevView V = view_of(A, range, g, v);
    const bool live = !(A.mask && !A.mask[g]);
    const PathId id = path_keys(V, g);
    v3 o, d;
    camera_ray(V, V.crop_x0 + id.lx, V.crop_y0 + id.ly, id.smp, A.seed, o, d);
    info = info_make(0, false, v);
    trav_begin(T, world_of(A, V), o, d, 3.0e38f);
    if (A.sig) A.sig[g] = live ? 1469598103934665603ull : 0ull;
    if (live) {
        ++cnt.c[ST_PATHS];
        ++cnt.c[ST_RAYS];
    } else {
        S.hflag[slot] = 2;
        S.nv[slot] = 0;  // (no vertex)
    }
    return live;
}
// The camera ray's record if it hit a surface (ray, sensor rotation, hit, keys; the keys again from the slot
// and the view); of a ray that escaped only the bytes that say so.
DEV void camera_end(const WArgs& A, const ViewRange& range, int slot, const Trav& T, int info) {
    const PathState& S = A.S;
    const int64_t g = A.g0 + slot;
    int v;
    const DevView V = view_of(A, range, g, v);
    if (T.h.prim >= 0) {
        float4* R = ray_rec(S, slot);
        const PathId id = path_keys(V, g);
        // rotation from the canonical frame of the light arriving along -d to the
        // sensor frame, kept in the record's spare words for the pixel reduction
        const v3 kc = -T.d;
        float Cs, Ss;
        rot_cs(kc, canon_x(kc), normalize(ld3(V.r) - kc * dot(ld3(V.r), kc)), Cs, Ss);
        ray_set(R, T.o, T.d, Cs, Ss);
        R[2] = f4(T.tb, T.h.u, T.h.v, __int_as_float(T.h.prim));
        R[3] = f4(__int_as_float(info), __uint_as_float(id.pix), __uint_as_float(id.smp),
                  __uint_as_float(V.view_id));
    }
    S.hflag[slot] = T.h.prim >= 0 ? 1 : 0;
    // whether the path has a vertex (the shading kernels of the backward then count them)
    S.nv[slot] = T.h.prim >= 0 ? 1 : 0;
}
// Next-event ray: the ray and its vertex's info word in one record (no read of the ray record, whose line
// would be fetched for its 16-byte key word).
template <int SMODE>
DEV void shadow_begin(const WArgs& A, int slot, Trav& T, int& info) {
    const PathState& S = A.S;
    const float4* H = SMODE == 4 ? r1_shd(S, A.Q, slot) : SMODE == 3 ? shd_rec(S, slot) : shd1_rec(S, slot);
    const float4 s0 = H[0], s1 = H[1];
    info = __float_as_int(s1.w);
    trav_begin(T, world_of(A, info >> 12), mk(s0.x, s0.y, s0.z), mk(s1.x, s1.y, s1.z), s0.w);
}
// What the outcome of a next-event ray (occ: occluded) changes.
template <int SMODE>
DEV void shadow_end(const WArgs& A, int slot, int info, bool occ) {
    const PathState& S = A.S;
    const int Q = A.Q;
    if (SMODE == 4) {
        // rank-one render: the path's radiance words already hold the next-event part
        // (k_shade<4>); an occluded light sample restores them from word 3
        if (occ) {
            float4* AC = r1_rec(S, slot);
            AC[2] = AC[3];
        }
        if (A.sig) sig_add(A.sig[A.g0 + slot], (uint32_t)(occ ? NEE_OCCLUDED : NEE_VISIBLE));
    } else if (SMODE == 5) {
        // cached backward: the vertex's record reads visible; an occluded sample marks it
        if (occ) vtx_rec(S, Q, (info & 255) - 1, slot)[1].w = __int_as_float(1);
    } else if (SMODE == 0) {
        // the path's radiance already holds the next-event part (k_shade<0>); an occluded light sample
        // restores it from beside the shadow rays
        if (occ) {
            float4* dst = acc_rec(S, slot) + 5;
            const float4* Lw = rest_rec(S, Q, slot);
            const float4 l0 = Lw[0], l1 = Lw[1], l2 = Lw[2];
            dst[0] = l0; dst[1] = l1; dst[2] = l2;
        }
        if (A.sig) sig_add(A.sig[A.g0 + slot], (uint32_t)(occ ? NEE_OCCLUDED : NEE_VISIBLE));
    } else if (SMODE >= 0) {
        if (SMODE == 1) {
            // the cache record holds E_b plus the next-event part and a visible sample
            // (k_shade<1>); an occluded light sample sets the E words back to E_b (zero unless
            // the vertex emits, when it was kept beside the shadow rays) and its visibility word
            // (two whole 32-byte sectors); a visible one writes nothing
            if (occ) {
                float4* dst = cache_rec(S, Q, (info & 255) - 1, slot) + 4;
                if (info & INFO_EMIT) {
                    const float4* Eb = rest_rec(S, Q, slot);
#pragma unroll
                    for (int k = 0; k < 3; ++k) dst[k] = Eb[k];
                } else {  // (E_b is zero)
#pragma unroll
                    for (int k = 0; k < 3; ++k) dst[k] = f4(0.0f, 0.0f, 0.0f, 0.0f);
                }
                dst[3] = f4(__int_as_float(NEE_OCCLUDED), 0.0f, 0.0f, 0.0f);
            }
        } else if (SMODE != 2) {  // the hybrid replay recomputes the next-event part from the visibility bit
            // (the tape forward adds it to both the radiance and the vertex's E_b)
            const float4* H = shd_rec(S, slot);
            float4* dst = acc_rec(S, slot) + 5;
            if (!occ) {
                float4* te = tape_rec(S, Q, (info & 255) - 1, slot) + 4;
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    float4 a = dst[k], p = H[2 + k];
                    dst[k] = f4(a.x + p.x, a.y + p.y, a.z + p.z, a.w + p.w);
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    float4 a = te[k], p = H[5 + k];
                    te[k] = f4(a.x + p.x, a.y + p.y, a.z + p.z, a.w + p.w);
                }
            }
        }
        if (SMODE != 1) {  // in the hit word of the vertex whose light sample this is
            float* hwp = SMODE == 3 ? &tape_rec(S, Q, (info & 255) - 1, slot)[2].w
                                    : &hit_rec(S, Q, (info & 255) - 1, slot)->x;
            uint32_t hw = (uint32_t)__float_as_int(*hwp);
            hw = (hw & ~(7u << 26)) | ((uint32_t)(occ ? NEE_OCCLUDED : NEE_VISIBLE) << 26);
            *hwp = __int_as_float((int)hw);
        }
        if (A.sig) sig_add(A.sig[A.g0 + slot], (uint32_t)(occ ? NEE_OCCLUDED : NEE_VISIBLE));
    }
}

// Closest hits of the rays of one bounce: a persistent kernel in which a lane takes the next queued
// ray as soon as its own is finished.  SMODE >= 0: the same launch resolves the shadow rays of the
// previous bounce (positions [0, n_s) of one work list, any hit; SMODE is that bounce's mode: 0
// full render, 1 backward with cache records (light stage, comparators), 2 hybrid replay, 3 tape, 4 render with
// the rank-one record, 5 cached backward), so the two kinds of rays share one launch and its tail.
// SMODE -1: the first bounce of rays whose records are written (P-RB sub-paths); SMODE -2: the
// first bounce of a chunk's camera paths, each lane generating the camera ray of the path it takes
// (no separate ray-generation pass writing records that this launch would read back).
// STATS: the launch adds to the work counters (A.stats set); without them a lane holds no counter
// registers.
template <int SMODE, bool STATS>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(STATS ? 7 : 8, 8))) k_extend(WArgs A) {
    extern __shared__ int lds_stack[];
    int* stack = lds_stack + threadIdx.x;
    trav_stack_init(stack);
    PathState& S = A.S;
    if (blockIdx.x == 0 && threadIdx.x == 0) {  // the queues the following kernels append to
        S.counts[CNT_RAY(1 - A.qin)] = 0;
        S.counts[CNT_HIT] = 0;
        if (SMODE < 0) S.counts[CNT_SHADOW] = 0;  // (a launch with shadow rays reads it: compaction clears it)
    }
    const int* q = A.qin ? S.queue1 : S.queue0;
    const int ne = A.first ? A.n_chunk : S.counts[CNT_RAY(A.qin)];
    const int ns = SMODE >= 0 ? S.counts[CNT_SHADOW] : 0;
    const int n = ns + ne;
    const int least = spread_least(A);
    if (!fetch_active(n, least)) return;
    Count cnt;
    WaveFetch F(n, least);
    Trav T;
    bool alive = false, any = false;
    int slot = -1, info = 0;
    ViewRange range;  // (camera rays)
    while (true) {
        const int idx = F.take(!alive, n, S, WORK_TRAVERSAL);
        if constexpr (SMODE == -2) {
            view_find(A, range, idx >= 0, A.g0 + idx);
            if (idx >= 0) {
                slot = idx;
                alive = camera_begin(A, range, slot, T, info, cnt);
            }
        } else if (idx >= 0) {
            any = idx < ns;
            if (SMODE >= 0 && any) {
                slot = S.squeue[idx];
                shadow_begin<SMODE>(A, slot, T, info);
                alive = true;
                ++cnt.c[ST_SHADOW_RAYS];
            } else {
                slot = A.first ? idx : q[idx - ns];
                const float4* R = ray_rec(S, slot);
                // the ray and its info word in one round trip (a dead ray's record is set up
                // and not traversed); a queued continuing ray is live, so in a scene of one world
                // its info word is not needed
                v3 o, d;
                ray_od(R, o, d);
                const bool need_info = A.first || !A.one_world;
                info = need_info ? __float_as_int(R[3].x) : 0;
                trav_begin(T, world_of(A, info >> 12), o, d, 3.0e38f);
                alive = !(info & INFO_DEAD);
                if (alive) ++cnt.c[ST_RAYS];
            }
        }
        if (!__any(alive) && !F.more()) break;
        const bool refill = F.more();
        uint32_t nn = 0, np = 0;
        const bool done = alive && trav_round<STATS>(T, SMODE >= 0 && any, nn, np, stack, refill);
        if (STATS) {
            if (SMODE >= 0 && any) {
                cnt.c[ST_SHADOW_NODES] += nn; cnt.c[ST_SHADOW_PRIMS] += np;
            } else {
                cnt.c[ST_NODES] += nn; cnt.c[ST_PRIMS] += np;
            }
        }
        if constexpr (SMODE == -2) {
            view_find(A, range, done, A.g0 + slot);
            if (done) {
                alive = false;
                camera_end(A, range, slot, T, info);
            }
        } else if (done) {
            alive = false;
            if (SMODE >= 0 && any) {
                shadow_end<SMODE>(A, slot, info, T.h.prim >= 0);
            } else {
                float4* R = ray_rec(S, slot);
                // the hit in one aligned 16-byte store (a hit's distance is the final tb); a miss
                // writes only its outcome byte (its path ends: nothing reads the hit words)
                if (T.h.prim >= 0) R[2] = f4(T.tb, T.h.u, T.h.v, __int_as_float(T.h.prim));
                S.hflag[slot] = T.h.prim >= 0 ? 1 : 0;
            }
        }
    }
    if (STATS) flush_stats(A.stats, cnt);
}

#ifndef PPT_EXT_TU  // (in the main compilation unit only)
// ============================================================================ hit compaction
// Splits the rays of this bounce by the outcome byte traversal wrote for each slot: misses end their
// path here (signature; a camera ray that escapes keeps a vertex count of 0, which the pixel
// reduction reads as no radiance), hits go, in queue order, to the hit queue that the shading kernel
// reads, so its lanes all hold a vertex.
// A workgroup takes tiles of up to COMPACT_ITEMS positions per thread (COMPACT_TILES tiles while they are
// smaller) and adds to the hit queue's size once per
// tile: the additions of all workgroups to that one word pass one after the other, 10 ns each (with a flush
// per 1,800 hits and one at every workgroup's end they took most of the launch: 24 us for 0.9M rays,
// now 11 us).
constexpr int COMPACT_ITEMS = 16, COMPACT_TILES = 512;
__global__ void __launch_bounds__(BLOCK) k_compact(WArgs A) {
    PathState& S = A.S;
    const int* qin = A.qin ? S.queue1 : S.queue0;
    const int n = A.first ? A.n_chunk : S.counts[CNT_RAY(A.qin)];
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) S.counts[CNT_SHADOW] = 0;  // the shadow queue the shading kernel appends to (the traversal read it)
        if (threadIdx.x < WORK_SHARDS) *work_counter(S, WORK_TRAVERSAL, threadIdx.x) = 0;  // (of the next traversal launch)
    }
    constexpr int WAVES = BLOCK / WAVE;
    static_assert(COMPACT_ITEMS * WAVES <= WAVE, "one wavefront scans a tile's counts");
    __shared__ int at[WAVE];  // hits of (item, wavefront), then where they go
    const int wave = threadIdx.x / WAVE, lane = lane_id();
    const int items = max(1, min(COMPACT_ITEMS, (n + COMPACT_TILES * BLOCK - 1) / (COMPACT_TILES * BLOCK)));
    for (int t0 = blockIdx.x * items * BLOCK; t0 < n; t0 += gridDim.x * items * BLOCK) {
        int slot[COMPACT_ITEMS], rank[COMPACT_ITEMS];
        if (threadIdx.x < WAVE) at[threadIdx.x] = 0;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < COMPACT_ITEMS; ++k) {
            rank[k] = -1;
            if (k >= items) continue;
            const int i = t0 + k * BLOCK + threadIdx.x;
            bool hit = false;
            if (i < n) {
                slot[k] = A.first ? i : qin[i];
                const int f = S.hflag[slot[k]];  // (a byte per ray instead of the hit words of its record)
                hit = f == 1;
                if (f == 0 && A.sig) sig_add(A.sig[A.g0 + slot[k]], 0xffffffffu);
            }
            const uint64_t m = __ballot(hit);
            if (hit) rank[k] = (int)__popcll(m & ((1ull << lane) - 1ull));
            if (lane == 0) at[k * WAVES + wave] = (int)__popcll(m);
        }
        __syncthreads();
        if (wave == 0) {
            const int c = at[lane];
            int sum = c;
#pragma unroll
            for (int o = 1; o < WAVE; o <<= 1) {
                const int up = __shfl_up(sum, o, WAVE);
                if (lane >= o) sum += up;
            }
            const int total = __shfl(sum, WAVE - 1, WAVE);
            int base = 0;
            if (lane == 0 && total) base = atomicAdd(&S.counts[CNT_HIT], total);
            at[lane] = __shfl(base, 0, WAVE) + sum - c;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < COMPACT_ITEMS; ++k)
            if (rank[k] >= 0) S.hqueue[at[k * WAVES + wave] + rank[k]] = slot[k];
        __syncthreads();
    }
}

#endif  // PPT_EXT_TU

// ============================================================================ sensor adjoint
// dL/dI of a pixel (analyzer a, per sample) and the adjoint rows at the camera ray it gives:
// a_c = (sum_a delta_a,c^T A_a / spp) R_s, R_s the rotation (Cs, Ss) into the sensor frame.
DEV int64_t pixel_offset(const DevView& V, uint32_t pix) {  // (of its first analyzer, in the image)
    const int py = (int)div_by(pix, V.inv_w), px = (int)(pix - (uint32_t)py * (uint32_t)V.width);
    return V.out_off + ((int64_t)(py - V.crop_y0) * V.crop_w + (px - V.crop_x0)) * 12;
}
// (C2, S2) = (cos 2 theta, sin 2 theta) of a linear polarizer
DEV void sensor_rows(const WArgs& A, const DevView& V, int64_t px_off, float C2, float S2, float Cs, float Ss, float* av) {
    const float inv = 1.0f / (float)V.spp;
    const int64_t astride = (int64_t)V.crop_w * V.crop_h * 12;
    const float* dp = A.dout + px_off;
    float asens[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) asens[k] = 0.0f;
    for (int a = 0; a < V.n_analyzers; ++a) {
        float dl[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) dl[k] = gval(dp, (size_t)(a * astride + k)) * inv;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            float r4[4];
            analyzer_row(V.sensor, C2, S2, a, dl + 4 * c, r4);
#pragma unroll
            for (int k = 0; k < 4; ++k) asens[4 * c + k] += r4[k];
        }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const float a1 = asens[4 * c + 1], a2 = asens[4 * c + 2];
        av[4 * c] = asens[4 * c];
        av[4 * c + 1] = Cs * a1 - Ss * a2;
        av[4 * c + 2] = Ss * a1 + Cs * a2;
        av[4 * c + 3] = asens[4 * c + 3];
    }
}
// The same in rank-one form for a linear polarizer, whose analyzer row is q' = (1, C, S, 0): a_c = sc_c rho
// with one row rho shared by the channels.
DEV void sensor_row1(const WArgs& A, const DevView& V, int64_t px_off, float C2, float S2, float Cs, float Ss, float* rho,
                     float* sc) {
    const float inv = 1.0f / (float)V.spp;
    const float* dp = A.dout + px_off;
#pragma unroll
    for (int c = 0; c < 3; ++c)
        sc[c] = 0.5f * (gval(dp, 4 * c) * inv + C2 * (gval(dp, 4 * c + 1) * inv) + S2 * (gval(dp, 4 * c + 2) * inv));
    rho[0] = 1.0f;
    rho[1] = Cs * C2 - Ss * S2;
    rho[2] = Ss * C2 + Cs * S2;
    rho[3] = 0.0f;
}

// ============================================================================ shading
// The vertex where the ray of path `slot` hit a surface: sampling, weight, radiance or the backward's records,
// the continuing ray into the ray record (cont) and the next-event ray into its record (shadow).
template <int MODE, bool EXT>
DEV void shade_slot(const WArgs& A, const Call& K, int slot, Count& cnt, bool& cont, bool& shadow) {
    constexpr bool ADJ = MODE == 5 || MODE == 6;  // cached backward: adjoint rows carried forward
    const PathState& S = A.S;
    const int Q = A.Q;
    const float4* R = ray_rec(S, slot);
    const float4 r3 = R[3], r0 = R[0], r1 = R[1], r2 = R[2];  // one round trip
    const int info = __float_as_int(r3.x);
    int nb = info & 255, v = info >> 12;
    bool prev_delta = (info >> 8) & 1;
    int64_t g = A.g0 + slot;
    const uint32_t pix = __float_as_uint(r3.y), smp = __float_as_uint(r3.z);
    const DevWorld W = world_of(A, v);
    Hit h;
    h.prim = __float_as_int(r2.w);
    h.t = r2.x; h.u = r2.y; h.v = r2.z;
    v3 o = mk(r0.x, r0.y, r0.z), d = mk(r0.w, r1.x, r1.y);
    {  // every queued ray hit a surface
        int b = nb + 1;
        ++cnt.c[ST_VERTICES];
        if (MODE == 1 || MODE == 2 || MODE == 3 || ADJ) S.nv[slot] = (uint8_t)b;  // (the fold reads these)
        Vtx x;
        surface(W, h, o, d, x);
        v3 so, sd;
        float stmax = 0.0f;
        vertex_setup<EXT>(W, K, __float_as_uint(r3.w), A.seed, pix, smp, b, A.max_depth, A.flags, prev_delta, d, x,
                          so, sd, stmax);
        if (A.sig) {
            uint64_t sg = A.sig[g];
            sig_add(sg, (uint32_t)x.orig);
            // (a sampled direction's lobe word also carries the branch of the sampling frame,
            // the sign of ns.z in the Duff et al. basis, which rounding can flip for a normal
            // with z near 0)
            const bool framed = x.lobe == LOBE_DIFFUSE || x.lobe == LOBE_GLOSSY;
            sig_add(sg, (uint32_t)x.lobe | (framed && signbit(x.ns.z) ? 16u : 0u));
            if (x.nee != NEE_PENDING) sig_add(sg, (uint32_t)x.nee);
            A.sig[g] = sg;
        }
        WC w;
        w.kind = 0;
        float Ee[12], En[12];
        if (ADJ) eval_vertex<false, EXT, false, true>(W, K, x, w, nullptr, nullptr, nullptr, nullptr);
        else if (MODE != 2) eval_vertex<false, EXT>(W, K, x, w, Ee, En, nullptr, nullptr);
        cont = x.lobe != LOBE_NONE && x.lobe != LOBE_INVALID;
        shadow = x.nee == NEE_PENDING;
        // the vertex's info word carried by its shadow ray's record (vertex count and view;
        // the delta bit is the continuing ray's and is not read for a shadow ray)
        const int info_shd = info_make(b, false, v);
        if (MODE == 2) {
            // hybrid replay: the hit record, and at a block start the ray into this vertex
            const bool sphere = !x.tri;
            *hit_rec(S, A.Q, b - 1, slot) = f4(__int_as_float(h.prim | (x.nee << 26)), sphere ? h.t : h.u, h.v, 0.0f);
            if ((b - 1) % A.ckpt == 0) {
                float4* CK = ckpt_rec(S, A.Q, (b - 1) / A.ckpt, slot);
                CK[0] = f4(o.x, o.y, o.z, prev_delta ? 1.0f : 0.0f);
                CK[1] = f4(d.x, d.y, d.z, 0.0f);
            }
        } else if (MODE == 4) {
            // render with a linear-polarizer sensor: its analyzer is rank one, so the image
            // needs per channel only the scalar y_c = q^T R_s Lo_c (q: the analyzer's row, R_s:
            // the sensor rotation).  The path carries the row rho = q^T R_s beta (shared by
            // the channels, beside beta's RGB scales) instead of beta, and y instead of Lo:
            // one 64-byte record [rho | rgb | y | y before the next-event part], the shadow ray
            // in a dense record of its own
            float4* AC = r1_rec(S, slot);
            float rho[4], brgb[3], y[3];
            if (nb == 0) {
                const DevView V = gval(A.views, (size_t)v);
                const float th = K.p(V.theta_slot, V.theta_off);
                const float C2 = cosf(2.0f * th), S2 = sinf(2.0f * th);
                const float Cs = r1.z, Ss = r1.w;  // sensor rotation of the camera ray
                rho[0] = 0.5f;
                rho[1] = 0.5f * (C2 * Cs - S2 * Ss);
                rho[2] = 0.5f * (C2 * Ss + S2 * Cs);
                rho[3] = 0.0f;
#pragma unroll
                for (int c = 0; c < 3; ++c) { brgb[c] = 1.0f; y[c] = 0.0f; }
            } else {
                const float4 a0 = AC[0], a1 = AC[1], a4 = AC[2];
                rho[0] = a0.x; rho[1] = a0.y; rho[2] = a0.z; rho[3] = a0.w;
                brgb[0] = a1.x; brgb[1] = a1.y; brgb[2] = a1.z;
                y[0] = a4.x; y[1] = a4.y; y[2] = a4.z;
            }
            float pn[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                y[c] += brgb[c] * (rho[0] * Ee[4 * c] + rho[1] * Ee[4 * c + 1] + rho[2] * Ee[4 * c + 2] +
                                   rho[3] * Ee[4 * c + 3]);
                pn[c] = brgb[c] * (rho[0] * En[4 * c] + rho[1] * En[4 * c + 1] + rho[2] * En[4 * c + 2] +
                                   rho[3] * En[4 * c + 3]);
            }
            if (cont) {
                if (w.kind == 1) {
                    rho[1] = rho[2] = rho[3] = 0.0f;
                } else {
                    WC ws = w;
                    ws.rgb[0] = 1.0f;
                    float o4[4];
                    w_row(ws, 0, rho, o4);
                    rho[0] = o4[0]; rho[1] = o4[1]; rho[2] = o4[2]; rho[3] = o4[3];
                }
#pragma unroll
                for (int c = 0; c < 3; ++c) brgb[c] *= w.rgb[c];
            }
            // the whole record (partial records measured slower)
            AC[0] = f4(rho[0], rho[1], rho[2], rho[3]);
            AC[1] = f4(brgb[0], brgb[1], brgb[2], 0.0f);
            // y with the next-event part as if its light sample were visible (traversal then
            // writes nothing for a visible one, and restores y from word 3 for an occluded one)
            if (shadow)
                AC[2] = f4(y[0] + pn[0], y[1] + pn[1], y[2] + pn[2], 0.0f);
            else
                AC[2] = f4(y[0], y[1], y[2], 0.0f);
            AC[3] = f4(y[0], y[1], y[2], 0.0f);
            if (shadow) {  // the shadow ray in its dense 32-byte record
                float4* H4 = r1_shd(S, A.Q, slot);
                H4[0] = f4(so.x, so.y, so.z, stmax);
                H4[1] = f4(sd.x, sd.y, sd.z, __int_as_float(info_shd));
            }
        } else if (MODE == 0 || MODE == 3) {
            float4* AC = acc_rec(S, slot);
            float beta[16], brgb[3], Lo[12];
            if (nb == 0) {  // first vertex: beta = I, no radiance yet
#pragma unroll
                for (int k = 0; k < 16; ++k) beta[k] = (k % 5 == 0) ? 1.0f : 0.0f;
#pragma unroll
                for (int c = 0; c < 3; ++c) brgb[c] = 1.0f;
#pragma unroll
                for (int k = 0; k < 12; ++k) Lo[k] = 0.0f;
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    float4 t = AC[k];
                    beta[4 * k] = t.x; beta[4 * k + 1] = t.y; beta[4 * k + 2] = t.z; beta[4 * k + 3] = t.w;
                }
                float4 t = AC[4];
                brgb[0] = t.x; brgb[1] = t.y; brgb[2] = t.z;
                ld12(AC + 5, Lo);
            }
            // Lo_c += brgb_c beta Ee_c; the pending next-event part likewise
            float pn[12];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float se = beta[4 * r] * Ee[4 * c] + beta[4 * r + 1] * Ee[4 * c + 1] +
                               beta[4 * r + 2] * Ee[4 * c + 2] + beta[4 * r + 3] * Ee[4 * c + 3];
                    Lo[4 * c + r] += brgb[c] * se;
                    float sn = beta[4 * r] * En[4 * c] + beta[4 * r + 1] * En[4 * c + 1] +
                               beta[4 * r + 2] * En[4 * c + 2] + beta[4 * r + 3] * En[4 * c + 3];
                    pn[4 * c + r] = brgb[c] * sn;
                }
            }
            if (MODE == 3) {
                if (shadow) st12(shd_rec(S, slot) + 2, pn);
                st12(AC + 5, Lo);
                // the tape record of this vertex: weight, hit, emission (its next-event part is
                // added when the shadow ray is resolved), the prefix throughput before the
                // vertex, and the ray into it
                float4* T = tape_rec(S, A.Q, b - 1, slot);
                const bool sphere = !x.tri;
                T[0] = f4(w.rgb[0], w.rgb[1], w.rgb[2], w.A);
                T[1] = f4(w.B, w.C, w.D, w.ci);
                T[2] = f4(w.si, w.co, w.so, __int_as_float(h.prim | (x.nee << 26) | (w.kind << 29)));
                T[3] = f4(sphere ? h.t : h.u, h.v, 0.0f, 0.0f);
                st12(T + 4, Ee);
                T[7] = f4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
                for (int k = 0; k < 4; ++k) T[8 + k] = f4(beta[4 * k], beta[4 * k + 1], beta[4 * k + 2], beta[4 * k + 3]);
                T[12] = f4(brgb[0], brgb[1], brgb[2], prev_delta ? 1.0f : 0.0f);
                T[13] = f4(o.x, o.y, o.z, d.x);
                T[14] = f4(d.y, d.z, 0.0f, 0.0f);
            } else if (shadow) {
                // Lo with the next-event part as if its light sample were visible, the Lo that an occluded
                // one restores beside the shadow rays: traversal writes nothing for a visible one
                st12(rest_rec(S, Q, slot), Lo);
#pragma unroll
                for (int k = 0; k < 12; ++k) Lo[k] = add_rounded(Lo[k], pn[k]);
                st12(AC + 5, Lo);
            } else {
                st12(AC + 5, Lo);
            }
            if (cont) {
                if (w.kind == 1) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) { beta[4 * r + 1] = beta[4 * r + 2] = beta[4 * r + 3] = 0.0f; }
                } else {
                    WC ws = w;
                    ws.rgb[0] = 1.0f;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float row[4] = {beta[4 * r], beta[4 * r + 1], beta[4 * r + 2], beta[4 * r + 3]}, o4[4];
                        w_row(ws, 0, row, o4);
                        beta[4 * r] = o4[0]; beta[4 * r + 1] = o4[1]; beta[4 * r + 2] = o4[2]; beta[4 * r + 3] = o4[3];
                    }
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) AC[k] = f4(beta[4 * k], beta[4 * k + 1], beta[4 * k + 2], beta[4 * k + 3]);
                AC[4] = f4(brgb[0] * w.rgb[0], brgb[1] * w.rgb[1], brgb[2] * w.rgb[2], 0.0f);
            }
        } else if (ADJ) {
            // cached backward: what the reverse walk needs to evaluate the vertex again (32 bytes:
            // hit, incoming direction, visibility word), and the adjoint row of the next vertex,
            // a <- a W_b, started here from dL/dI (the first vertex's row is made again from it)
            float4* VR = vtx_rec(S, Q, b - 1, slot);
            VR[0] = f4(__int_as_float(h.prim | (prev_delta ? VTX_PREV_DELTA : 0)), x.tri ? h.u : x.p.x,
                       x.tri ? h.v : x.p.y, x.p.z);
            VR[1] = f4(d.x, d.y, d.z, 0.0f);
            if (cont) {
                float C2 = 1.0f, S2 = 0.0f;
                DevView V;
                if (nb == 0) {
                    V = gval(A.views, (size_t)v);
                    if (V.sensor == SENSOR_POLARIZER) {
                        const float th = K.p(V.theta_slot, V.theta_off);
                        C2 = cosf(2.0f * th);
                        S2 = sinf(2.0f * th);
                    }
                }
                if (MODE == 6) {
                    float rho[4], sc[3];
                    if (nb == 0) {
                        sensor_row1(A, V, pixel_offset(V, pix), C2, S2, r1.z, r1.w, rho, sc);
                    } else {
                        const float4* RR = row_rec<true>(S, Q, b - 1, slot);
                        const float4 a0 = RR[0], a1 = RR[1];
                        rho[0] = a0.x; rho[1] = a0.y; rho[2] = a0.z; rho[3] = a0.w;
                        sc[0] = a1.x; sc[1] = a1.y; sc[2] = a1.z;
                    }
                    if (w.kind == 1) {
                        rho[1] = rho[2] = rho[3] = 0.0f;
                    } else {
                        WC ws = w;
                        ws.rgb[0] = 1.0f;
                        float o4[4];
                        w_row(ws, 0, rho, o4);
                        rho[0] = o4[0]; rho[1] = o4[1]; rho[2] = o4[2]; rho[3] = o4[3];
                    }
                    float4* RW = row_rec<true>(S, Q, b, slot);
                    RW[0] = f4(rho[0], rho[1], rho[2], rho[3]);
                    RW[1] = f4(sc[0] * w.rgb[0], sc[1] * w.rgb[1], sc[2] * w.rgb[2], 0.0f);
                } else {
                    float av[12], an[12];
                    if (nb == 0) sensor_rows(A, V, pixel_offset(V, pix), C2, S2, r1.z, r1.w, av);
                    else ld12(row_rec<false>(S, Q, b - 1, slot), av);
#pragma unroll
                    for (int c = 0; c < 3; ++c) w_row(w, c, av + 4 * c, an + 4 * c);
                    st12(row_rec<false>(S, Q, b, slot), an);
                }
            }
            if (shadow) {  // the shadow ray in its dense 32-byte record
                float4* H1 = shd1_rec(S, slot);
                H1[0] = f4(so.x, so.y, so.z, stmax);
                H1[1] = f4(sd.x, sd.y, sd.z, __int_as_float(info_shd));
            }
        } else {  // MODE 1
            float4* C = cache_rec(S, A.Q, b - 1, slot);
            const bool sphere = !x.tri;
            C[0] = f4(w.rgb[0], w.rgb[1], w.rgb[2], w.A);
            C[1] = f4(w.B, w.C, w.D, w.ci);
            C[2] = f4(w.si, w.co, w.so, __int_as_float(h.prim | (x.nee << 26) | (w.kind << 29)));
            C[3] = f4(sphere ? h.t : h.u, h.v, 0.0f, 0.0f);
            // E_b with the next-event part as if its light sample were visible, so that traversal
            // writes nothing here for a visible one (an occluded one restores E_b from the
            // shadow record's words 5..7)
            if (shadow) {
                float EN[12];
#pragma unroll
                for (int k = 0; k < 12; ++k) EN[k] = Ee[k] + En[k];
                st12(C + 4, EN);
                // the shadow ray in its dense 32-byte record, and E_b where the vertex emits (an
                // occluded sample restores it; a non-emitting vertex's E_b is zero)
                float4* H1 = shd1_rec(S, slot);
                H1[0] = f4(so.x, so.y, so.z, stmax);
                H1[1] = f4(sd.x, sd.y, sd.z, __int_as_float(info_shd | (x.emit ? INFO_EMIT : 0)));
                if (x.emit) st12(rest_rec(S, A.Q, slot), Ee);
            } else {
                st12(C + 4, Ee);
            }
            // a whole 128-byte record is written; a pending light sample's visibility as if
            // visible (traversal rewrites it for an occluded one)
            C[7] = f4(__int_as_float(shadow ? NEE_VISIBLE : 0), 0.0f, 0.0f, 0.0f);
        }
        if ((MODE == 0 || MODE == 2 || MODE == 3) && shadow) {  // (the tape: a whole 128-byte record)
            float4* H = MODE == 3 ? shd_rec(S, slot) : shd1_rec(S, slot);
            H[0] = f4(so.x, so.y, so.z, stmax);
            H[1] = f4(sd.x, sd.y, sd.z, __int_as_float(info_shd));
            if (MODE == 3) st12(H + 5, En);  // (the tape's E_b takes the unweighted part)
        }
        float4* Rw = ray_rec(S, slot);
        if (cont) ray_set(Rw, spawn(x.p, x.ng, x.wi), x.wi, r1.z, r1.w);  // (keeps the sensor rotation)
        Rw[3].x = __int_as_float(info_make(b, is_delta(gval(W.mats, (size_t)x.mat).type), v));
    }
}

template <int MODE, bool EXT>
// (four waves per SIMD where the registers then fit without spills)
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(MODE == 1 && EXT ? 1 : 4, 8))) k_shade(WArgs A) {
    constexpr bool ADJ = MODE == 5 || MODE == 6;  // cached backward: adjoint rows carried forward
    PathState& S = A.S;
    Call K{A.table, nullptr};
    int* qout = A.qin ? S.queue0 : S.queue1;
    const int n = S.counts[CNT_HIT];
    if (ADJ && A.keep_deep && blockIdx.x == 0 && threadIdx.x == 0) S.counts[CNT_REPLAY] = n;
    __shared__ BlockQueue qn, qs;
    __shared__ CallTable tab;
    table_to_lds(&tab, A.table);
    K.tab = &tab;
    if (threadIdx.x == 0) { qn.n = 0; qs.n = 0; }
    __syncthreads();
    Count cnt;
    for (int bb = blockIdx.x * BLOCK; bb < n; bb += gridDim.x * BLOCK) {
        int i = bb + threadIdx.x;
        bool cont = false, shadow = false;
        int slot = 0;
        if (i < n) slot = S.hqueue[i];
        if (i < n) shade_slot<MODE, EXT>(A, K, slot, cnt, cont, shadow);  // (a queued ray is a live path's hit)
        bq_push(qn, cont, slot);
        bq_push(qs, shadow, slot);
        bq_flush(qn, &S.counts[CNT_RAY(1 - A.qin)], qout, false);
        bq_flush(qs, &S.counts[CNT_SHADOW], S.squeue, false);
    }
    bq_flush(qn, &S.counts[CNT_RAY(1 - A.qin)], qout, true);
    bq_flush(qs, &S.counts[CNT_SHADOW], S.squeue, true);
    flush_stats(A.stats, cnt);
}

#ifndef PPT_EXT_TU  // (in the main compilation unit only)
// ============================================================================ whole paths of a small call
// Every bounce of the paths of a small call in one launch: a wavefront takes per_wave consecutive paths
// (at most 32) in its lower lanes and traces and shades them from the camera to their end, through the same
// records as the launches per bounce.  The upper lanes trace the next-event rays beside the lower lanes'
// continuing rays.  A small call is bound by its launches (three per bounce, each some 5 us and as long
// as its slowest ray); here a path waits for the other paths of its wavefront only.
template <bool STATS>
DEV void trace(Trav& T, bool active, bool any, int* stack, Count& cnt) {
    bool todo = active;
    while (__any(todo)) {
        uint32_t nn = 0, np = 0;
        if (todo && trav_round<STATS>(T, any, nn, np, stack, false)) todo = false;
        if (STATS) {
            if (any) { cnt.c[ST_SHADOW_NODES] += nn; cnt.c[ST_SHADOW_PRIMS] += np; }
            else { cnt.c[ST_NODES] += nn; cnt.c[ST_PRIMS] += np; }
        }
    }
}
// what one lane wrote to global memory before is read by another lane of the wavefront after
DEV void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// MODE: the shading mode (0, 4 render; 5, 6 cached backward; 2 hybrid replay)
template <int MODE, bool STATS>
__global__ void __launch_bounds__(BLOCK) k_paths(WArgs A, int per_wave) {
    constexpr int SMODE = MODE == 6 ? 5 : MODE;
    extern __shared__ int lds_stack[];
    int* stack = lds_stack + threadIdx.x;
    trav_stack_init(stack);
    Call K{A.table, nullptr};
    __shared__ CallTable tab;
    table_to_lds(&tab, A.table);
    K.tab = &tab;
    __syncthreads();
    const PathState& S = A.S;
    const int wave = wave_number();
    const int lane = lane_id(), mate = lane & (WAVE / 2 - 1);  // (the lower lane of this lane's path)
    const bool lower = lane < WAVE / 2;
    const int slot = wave * per_wave + mate;
    const bool mine = mate < per_wave && slot < A.n_chunk;
    Count cnt;
    ViewRange range;
    Trav T;
    int info = 0;
    bool alive = false;
    view_find(A, range, lower && mine, A.g0 + slot);
    if (lower && mine) alive = camera_begin(A, range, slot, T, info, cnt);
    trace<STATS>(T, alive, false, stack, cnt);
    bool hit = false;
    if (alive) {
        camera_end(A, range, slot, T, info);
        hit = T.h.prim >= 0;
        if (!hit && A.sig) sig_add(A.sig[A.g0 + slot], 0xffffffffu);
    }
    for (int b = 1; b <= A.max_depth && __any(hit); ++b) {
        bool cont = false, shadow = false;
        if (hit) shade_slot<MODE, false>(A, K, slot, cnt, cont, shadow);
        hit = false;
        if (b == A.max_depth) break;  // (a vertex at the maximum depth starts no ray)
        wave_fence();
        const bool any = !lower & (__shfl((int)shadow, mate, WAVE) != 0);
        alive = any || (lower && cont);
        if (any) {
            shadow_begin<SMODE>(A, slot, T, info);
            ++cnt.c[ST_SHADOW_RAYS];
        } else if (alive) {
            const float4* R = ray_rec(S, slot);
            v3 o, d;
            ray_od(R, o, d);
            const int ri = A.one_world ? 0 : __float_as_int(R[3].x);
            trav_begin(T, world_of(A, ri >> 12), o, d, 3.0e38f);
            ++cnt.c[ST_RAYS];
        }
        trace<STATS>(T, alive, any, stack, cnt);
        if (any) shadow_end<SMODE>(A, slot, info, T.h.prim >= 0);
        wave_fence();  // (a path's next-event outcome before its next vertex or its end)
        if (alive && lower) {
            hit = T.h.prim >= 0;
            if (hit) ray_rec(S, slot)[2] = f4(T.tb, T.h.u, T.h.v, __int_as_float(T.h.prim));
            else if (A.sig) sig_add(A.sig[A.g0 + slot], 0xffffffffu);
        }
    }
    if (STATS) flush_stats(A.stats, cnt);
}

// ============================================================================ render: pixel reduction
// Every lane rotates its path's radiance into the sensor frame; the lanes of one pixel (adjacent,
// samples fastest) are summed by a segmented wavefront scan, and the last lane of each segment
// applies the analyzers and adds the mean to the image.  A pixel whose samples span two
// wavefronts or chunks receives several additions; one of up to STORE_SPP samples, all
// held by the wavefront, is stored to the cleared image instead: with many pixels a wavefront the additions, 9 to
// 48 atomics a pixel, bounded the kernel (1 sample, 0.9M paths: 266 -> 41 us; 16 samples, 33.6M paths: 0.75 -> 0.42 ms;
// but 32 samples, 67M paths: 0.84 -> 0.98 ms, since the next loads wait for the stores).
// The scan takes its segments from one ballot and as many steps as the longest one (67M paths of 32 samples:
// 1.17 -> 0.84 ms).
// R1: the rank-one render of a linear-polarizer sensor, whose paths carry y_c = q^T R_s Lo_c (rotation
// and analyzer row already applied): the scan sums three scalars and the output is (1, C, S, 0) y_c,
// C = cos 2 theta, S = sin 2 theta (the polarizer's Mueller matrix is q' q'^T / 2 with q' = (1, C, S, 0)).
constexpr int STORE_SPP = 16;
// Adds o to a pixel of the image; whole: nothing else is added to it (aligned: the image lies on 16 bytes).
DEV void pixel_add(float* out, const float* o, bool whole, bool aligned) {
    bool any = false;
#pragma unroll
    for (int k = 0; k < 12; ++k) any |= o[k] != 0.0f;
    if (!any) return;
    if (whole && aligned) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
            ((float4*)out)[k] = f4(o[4 * k] + 0.0f, o[4 * k + 1] + 0.0f, o[4 * k + 2] + 0.0f, o[4 * k + 3] + 0.0f);
    } else {
#pragma unroll
        for (int k = 0; k < 12; ++k)
            if (o[k] != 0.0f) atomicAdd(out + k, o[k]);
    }
}
template <bool R1>
__global__ void __launch_bounds__(BLOCK) k_accum(WArgs A) {
    if (!A.out) return;  // signature-only runs produce no image
    constexpr int NA = R1 ? 3 : 12;
    PathState& S = A.S;
    Call K{A.table, nullptr};
    ViewRange range;
    const int lane = lane_id();
    const bool aligned = ((uintptr_t)A.out & 15) == 0;
    for (int base = blockIdx.x * BLOCK + (threadIdx.x & ~(WAVE - 1)); base < A.n_chunk; base += gridDim.x * BLOCK) {
        int i = base + lane;
        bool valid = i < A.n_chunk;
        int64_t key = -1 - lane;  // distinct per invalid lane
        float acc[NA];
#pragma unroll
        for (int k = 0; k < NA; ++k) acc[k] = 0.0f;
        int v = 0;
        int64_t px_off = 0;  // the pixel's place in the image (first analyzer)
        // the keys from the path's index (the wavefront holds consecutive paths), and the radiance from the
        // path's record when the path has a vertex (one byte per path says so): no record of a path
        // without radiance is read
        for_views(A, range, valid, A.g0 + i, [&](int vw, const DevView& V) {
            const PathId id = path_keys(V, A.g0 + i);
            v = vw;
            key = ((int64_t)vw << 32) | (int64_t)id.pix;
            px_off = V.out_off + ((int64_t)id.ly * V.crop_w + id.lx) * 12;
        });
        if (valid && S.nv[i]) {
            if constexpr (R1) {
                const float4 y = r1_rec(S, i)[2];
                acc[0] = y.x; acc[1] = y.y; acc[2] = y.z;
            } else {
                const float4 r1 = ray_rec(S, i)[1];
                const float Cs = r1.z, Ss = r1.w;  // sensor rotation of the camera ray
                float Lo[12];
                ld12(acc_rec(S, i) + 5, Lo);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    float l1 = Lo[4 * c + 1], l2 = Lo[4 * c + 2];
                    acc[4 * c] = Lo[4 * c];
                    acc[4 * c + 1] = Cs * l1 + Ss * l2;
                    acc[4 * c + 2] = -Ss * l1 + Cs * l2;
                    acc[4 * c + 3] = Lo[4 * c + 3];
                }
            }
        }
        // inclusive segmented scan toward higher lanes, over as many steps as the longest segment needs; the
        // segments from one ballot of their first lanes
        const int64_t kprev = __shfl_up(key, 1, WAVE);
        const uint64_t first = __ballot(lane == 0 || kprev != key);
        const int start = 63 - __clzll((long long)(first & (~0ull >> (63 - lane))));
        for (int off = 1; off < WAVE; off <<= 1) {
            const bool take = lane - off >= start;
            if (!__any(take)) break;
#pragma unroll
            for (int k = 0; k < NA; ++k) {
                float t = __shfl_up(acc[k], off, WAVE);
                if (take) acc[k] += t;
            }
        }
        const bool tail = valid && (lane == WAVE - 1 || ((first >> (lane + 1)) & 1ull) != 0ull);
        if (tail) {
            const DevView V = gval(A.views, (size_t)v);
            float theta = V.sensor == SENSOR_POLARIZER ? K.p(V.theta_slot, V.theta_off) : 0.0f;
            float inv = 1.0f / (float)V.spp;
            const bool whole = lane - start + 1 == V.spp && V.spp <= STORE_SPP;
            if constexpr (R1) {
                const float C2 = cosf(2.0f * theta), S2 = sinf(2.0f * theta);
                float o[12];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    o[4 * c] = acc[c] * inv; o[4 * c + 1] = C2 * acc[c] * inv; o[4 * c + 2] = S2 * acc[c] * inv;
                    o[4 * c + 3] = 0.0f;
                }
                pixel_add(A.out + px_off, o, whole, aligned);
            } else {
                int64_t astride = (int64_t)V.crop_w * V.crop_h * 12;
                for (int a = 0; a < V.n_analyzers; ++a) {
                    float o[12];
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        analyzer_apply(V.sensor, theta, a, acc + 4 * c, o + 4 * c);
#pragma unroll
                        for (int k = 0; k < 4; ++k) o[4 * c + k] *= inv;
                    }
                    pixel_add(A.out + px_off + a * astride, o, whole, aligned);
                }
            }
        }
    }
}

#endif  // PPT_EXT_TU

// W_c applied to a Stokes vector without branches on the weight's kind (the loads of a record
// stay together ahead of the arithmetic): the Fresnel form is evaluated and then selected.
// Entries of kind-0 records are not read into the result.
DEV void w_apply_select(const WC& w, int c, const float* in, float* out) {
    float v1 = w.ci * in[1] + w.si * in[2], v2 = -w.si * in[1] + w.ci * in[2];
    float f0 = w.A * in[0] + w.B * v1, f1 = w.B * in[0] + w.A * v1;
    float f2 = w.C * v2 + w.D * in[3], f3 = -w.D * v2 + w.C * in[3];
    const float s = w.rgb[c];
    const bool fr = w.kind == 2, df = w.kind == 1;
    out[0] = fr ? s * f0 : (df ? s * in[0] : 0.0f);
    out[1] = fr ? s * (w.co * f1 + w.so * f2) : 0.0f;
    out[2] = fr ? s * (-w.so * f1 + w.co * f2) : 0.0f;
    out[3] = fr ? s * f3 : 0.0f;
}

// ============================================================================ hybrid replay blocks
// Hybrid cached replay (Sec. 4.4): the primal pass keeps a hit record per vertex and, every k
// vertices, the ray into the block's first vertex; suffix values are kept only at block ends.
// block_eval re-evaluates vertices [s, e) of the path in `slot` from the ray (o, d) into vertex s,
// with each vertex's recorded next-event visibility, into the scratch cache records rec0 ..
// rec0 + e-s-1 (W_b and E_b); block_fold then folds records rec0 .. rec0 + n-1 back from the
// suffix L beyond the last of them, leaving in L the suffix at the first one's vertex (with
// store_suffix, each record's E words receive the suffix beyond its vertex, which the replay reads).
template <bool EXT>
DEV void block_eval(const WArgs& A, const Call& K, const DevView& V, const DevWorld& W, int slot, uint32_t pix,
                    uint32_t smp, int s, int e, v3 o, v3 d, bool prev_delta, int rec0 = 0) {
    const PathState& S = A.S;
    const int Q = A.Q;
    for (int v = s; v < e; ++v) {
        const float4 hr = *hit_rec(S, Q, v, slot);
        const uint32_t hw = __float_as_uint(hr.x);
        Hit h;
        h.prim = (int)(hw & ((1u << 26) - 1));
        h.u = hr.y; h.t = hr.y; h.v = hr.z;
        Vtx x;
        surface(W, h, o, d, x);
        v3 so, sd;
        float stmax;
        vertex_setup<EXT>(W, K, V.view_id, A.seed, pix, smp, v + 1, A.max_depth, A.flags, prev_delta, d, x, so, sd, stmax);
        if (x.nee == NEE_PENDING) x.nee = (int)((hw >> 26) & 7);
        WC w;
        float Ee[12], En[12];
        eval_vertex<false, EXT>(W, K, x, w, Ee, En, nullptr, nullptr);
        float4* C = cache_rec(S, Q, rec0 + v - s, slot);
        C[0] = f4(w.rgb[0], w.rgb[1], w.rgb[2], w.A);
        C[1] = f4(w.B, w.C, w.D, w.ci);
        C[2] = f4(w.si, w.co, w.so, __int_as_float(w.kind << 29));
#pragma unroll
        for (int q = 0; q < 12; ++q) Ee[q] += En[q];
        st12(C + 4, Ee);
        prev_delta = is_delta(gval(W.mats, (size_t)x.mat).type);
        o = spawn(x.p, x.ng, x.wi);
        d = x.wi;
    }
}
DEV void block_fold(const PathState& S, int Q, int slot, int n, float* L, bool store_suffix, int rec0 = 0) {
    for (int u = rec0 + n - 1; u >= rec0; --u) {
        float4* C = cache_rec(S, Q, u, slot);
        const float4 c0 = C[0], c1 = C[1], c2 = C[2];
        float e[12];
        ld12(C + 4, e);
        if (store_suffix) st12(C + 4, L);
        WC w;
        w.rgb[0] = c0.x; w.rgb[1] = c0.y; w.rgb[2] = c0.z;
        w.A = c0.w; w.B = c1.x; w.C = c1.y; w.D = c1.z;
        w.ci = c1.w; w.si = c2.x; w.co = c2.y; w.so = c2.z;
        w.kind = (__float_as_int(c2.w) >> 29) & 3;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            float o4[4];
            w_apply_select(w, c, L + 4 * c, o4);
#pragma unroll
            for (int k = 0; k < 4; ++k) L[4 * c + k] = e[4 * c + k] + o4[k];
        }
    }
}

// ============================================================================ P-PRB comparator
// Regularisation noise of the noise-regularised polarized PRB (Sec. 4.2): one normal variate
// u ~ N(0, sigma) per path vertex (1-based index vtx) from two uniforms of the vertex's counter
// (call 2) by the Box-Muller transform; the fold and the replay draw the same value.
DEV float pprb_noise(const WArgs& A, uint32_t pix, uint32_t smp, uint32_t view_id, int vtx) {
    float u[4];
    uniforms(A.seed, pix, smp, view_id, (uint32_t)vtx, 2, u);
    return A.pprb_sigma * sqrtf(-2.0f * logf(1.0f - u[0])) * cosf(6.28318530717958648f * u[1]);
}
// W_c of a compact weight as a row-major 4x4 (column j = W_c e_j)
DEV void w_matrix(const WC& w, int c, float* m) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float e[4] = {j == 0 ? 1.0f : 0.0f, j == 1 ? 1.0f : 0.0f, j == 2 ? 1.0f : 0.0f, j == 3 ? 1.0f : 0.0f}, o[4];
        w_apply(w, c, e, o);
#pragma unroll
        for (int r = 0; r < 4; ++r) m[4 * r + j] = o[r];
    }
}

// Polarizer angles: one atomic per distinct view among the wavefront's running sums (gtheta of view
// tkey, -1 for none).  Every lane of the wavefront calls it.
DEV void flush_theta(const WArgs& A, const Call& K, int tkey, float gtheta) {
    bool pending = tkey >= 0;
    while (__ballot(pending)) {
        unsigned long long m = __ballot(pending);
        int leader = __ffsll((long long)m) - 1;
        int key = __shfl(tkey, leader, WAVE);
        bool mine = pending && tkey == key;
        float s = wave_sum(mine ? gtheta : 0.0f);
        if (lane_id() == leader) K.g(A.views[key].theta_slot, A.views[key].theta_off, s);
        pending = pending && !mine;
    }
}

// ============================================================================ backward: fold

// Per path with at least one vertex: folds the cache into the suffix radiance
// L[b] = E_b + W_b L[b+1] (L[b+1] written over E_b), adds the polarizer-angle term
// delta^T (dP/dtheta) R_s L[1],
// and sets up the replay: the adjoint rows a_c = (delta^T A / spp) R_s, the camera ray's direction,
// the path's keys and vertex count (all in the shadow record's words 0..4) and an entry of the replay queue (queue0, size counts[CNT_REPLAY]).  Each workgroup folds one
// contiguous range of slots, so its lanes mostly see a single view and keep the angle term in a
// register until the view changes.
// PPRB (the noise-regularised comparator of Sec. 4.2): the fold uses W_b + u_b I, keeps the records'
// E words (the replay inverts the weights instead of reading suffixes) and stores the path's
// regularised radiance L'[1] in the shadow record's words 5..7.
// TAPE (the conventional-AD baseline): no fold; the path's radiance comes from the forward
// accumulator, for the polarizer-angle term and the adjoint rows.
template <bool HYB, bool EXT, bool PPRB = false, bool TAPE = false>
// (six waves per SIMD for the cached fold: its registers then fit without spills, measured faster)
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(HYB ? 1 : 6, 8))) k_fold(WArgs A) {
    PathState& S = A.S;
    const int Q = A.Q;
    Call K{A.table, A.gacc};
    __shared__ BlockQueue rq;
    if (threadIdx.x == 0) rq.n = 0;
    __syncthreads();
    const int r0 = (int)((int64_t)A.n_chunk * blockIdx.x / gridDim.x);
    const int r1 = (int)((int64_t)A.n_chunk * (blockIdx.x + 1) / gridDim.x);
    ViewRange range;
    float gtheta = 0.0f;
    int tkey = -1;
    for (int base = r0; base < r1; base += BLOCK) {
        const int i = base + threadIdx.x;
        bool push = false;
        // the path's vertex count from the dense byte array and its keys from its index (no read of
        // its ray record, which would cost a 128-byte line for 16 bytes)
        const int B = i < r1 ? (int)S.nv[i] : 0;
        float gt = 0.0f;
        PathId id{};
        int v = 0;
        uint32_t view_id = 0;
        for_views(A, range, B > 0, A.g0 + i, [&](int vw, const DevView& V) {
            id = path_keys(V, A.g0 + i);
            v = vw;
            view_id = V.view_id;
        });
        if (B > 0) {
            push = true;
            // fold over records B-1 .. 0 (record r holds vertex r+1): the record's E words receive
            // the suffix beyond its vertex, L[r+2], so the replay of a vertex reads one record (the
            // last vertex's suffix is zero and is not stored)
            float L[12];
#pragma unroll
            for (int k = 0; k < 12; ++k) L[k] = 0.0f;
            if (HYB) {
                // blocks from the last to the first: re-evaluate from the block's checkpoint ray,
                // store the suffix beyond the block, fold back to the block's first vertex
                const DevView Vh = gval(A.views, (size_t)v);
                const DevWorld Wh = world_of(A, Vh);
                const int kc = A.ckpt;
                for (int j = (B + kc - 1) / kc - 1; j >= 0; --j) {
                    const int s0 = j * kc, e0 = min(B, s0 + kc);
                    float4* CK = ckpt_rec(S, Q, j, i);
                    const float4 k0 = CK[0], k1 = CK[1];
                    block_eval<EXT>(A, K, Vh, Wh, i, id.pix, id.smp, s0, e0, mk(k0.x, k0.y, k0.z), mk(k1.x, k1.y, k1.z),
                               k0.w != 0.0f);
                    st12(CK + 2, L);
                    block_fold(S, Q, i, e0 - s0, L, false);
                }
                // the suffix at the first vertex, the decision rule's remaining radiance of block 0
                if (A.hyb_rule) st12(shd_rec(S, i) + 5, L);
            }
            if (TAPE) ld12(acc_rec(S, i) + 5, L);
            for (int b = HYB || TAPE ? -1 : B - 1; b >= 0; --b) {
                float4* C = cache_rec(S, Q, b, i);
                const float4 c0 = C[0], c1 = C[1], c2 = C[2];
                float e[12];
                ld12(C + 4, e);
                if (!PPRB && b < B - 1) st12(C + 4, L);
                const float u = PPRB ? pprb_noise(A, id.pix, id.smp, view_id, b + 1) : 0.0f;
                WC w;
                w.rgb[0] = c0.x; w.rgb[1] = c0.y; w.rgb[2] = c0.z;
                w.A = c0.w; w.B = c1.x; w.C = c1.y; w.D = c1.z;
                w.ci = c1.w; w.si = c2.x; w.co = c2.y; w.so = c2.z;
                w.kind = (__float_as_int(c2.w) >> 29) & 3;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    float o4[4];
                    w_apply_select(w, c, L + 4 * c, o4);
#pragma unroll
                    for (int k = 0; k < 4; ++k) L[4 * c + k] = e[4 * c + k] + o4[k] + (PPRB ? u * L[4 * c + k] : 0.0f);
                }
            }
            if (PPRB) st12(shd_rec(S, i) + 5, L);
            const uint32_t pix = id.pix, smp = id.smp;
            const DevView V = gval(A.views, (size_t)v);
            const int py = (int)div_by(pix, V.inv_w), px = (int)(pix - (uint32_t)py * (uint32_t)V.width);
            const int lx = px - V.crop_x0, ly = py - V.crop_y0;
            v3 o, d;
            camera_ray(V, px, py, smp, A.seed, o, d);
            v3 kc = -d;
            float Cs, Ss;
            rot_cs(kc, canon_x(kc), normalize(ld3(V.r) - kc * dot(ld3(V.r), kc)), Cs, Ss);
            const bool pol = V.sensor == SENSOR_POLARIZER;
            const float theta = pol ? K.p(V.theta_slot, V.theta_off) : 0.0f;
            const float C2 = cosf(2.0f * theta), S2 = sinf(2.0f * theta);
            // adjoint of the pixel mean in the sensor frame: a_sens_c = sum_a delta_a,c^T A_a / spp;
            // the polarizer-angle term (one analyzer) is delta^T (dP/dtheta) R_s L[1]
            const float inv = 1.0f / (float)V.spp;
            const int64_t astride = (int64_t)V.crop_w * V.crop_h * 12;
            const float* dp = A.dout + V.out_off + ((int64_t)ly * V.crop_w + lx) * 12;
            float asens[12];
#pragma unroll
            for (int k = 0; k < 12; ++k) asens[k] = 0.0f;
            for (int a = 0; a < V.n_analyzers; ++a) {
                float dl[12];
#pragma unroll
                for (int k = 0; k < 12; ++k) dl[k] = dp[a * astride + k] * inv;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    float r4[4];
                    analyzer_row(V.sensor, C2, S2, a, dl + 4 * c, r4);
#pragma unroll
                    for (int k = 0; k < 4; ++k) asens[4 * c + k] += r4[k];
                    if (pol && a == 0) {
                        float l1 = L[4 * c + 1], l2 = L[4 * c + 2];
                        float ls[4] = {L[4 * c], Cs * l1 + Ss * l2, -Ss * l1 + Cs * l2, L[4 * c + 3]};
                        gt += polarizer_dtheta(C2, S2, dl + 4 * c, ls);
                    }
                }
            }
            float av[12];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                float a1 = asens[4 * c + 1], a2 = asens[4 * c + 2];
                av[4 * c] = asens[4 * c];
                av[4 * c + 1] = Cs * a1 - Ss * a2;
                av[4 * c + 2] = Ss * a1 + Cs * a2;
                av[4 * c + 3] = asens[4 * c + 3];
            }
            // the replay's start in one record: the camera ray's direction (its origin is the view's),
            // the info word (vertex count, view), the keys and the adjoint rows
            const int info_rs = info_make((int)S.nv[i], false, v);  // (B read again: fewer live registers)
            float4* Hs = shd_rec(S, i);
            Hs[0] = f4(d.x, d.y, d.z, __int_as_float(info_rs));
            Hs[1] = f4(__uint_as_float(pix), __uint_as_float(smp), 0.0f, 0.0f);
            st12(Hs + 2, av);
            // the rest of the 128-byte record where nothing else fills it (a line written in part
            // is the slower path)
            if (!PPRB && !(HYB && A.hyb_rule)) Hs[5] = Hs[6] = Hs[7] = f4(0.0f, 0.0f, 0.0f, 0.0f);
            if (pol) {
                if (tkey != v) {
                    if (tkey >= 0) K.g(A.views[tkey].theta_slot, A.views[tkey].theta_off, gtheta);
                    gtheta = 0.0f;
                    tkey = v;
                }
                gtheta += gt;
            }
        }
        bq_push(rq, push, i);
        bq_flush(rq, &S.counts[CNT_REPLAY], S.queue0, false);
    }
    bq_flush(rq, &S.counts[CNT_REPLAY], S.queue0, true);
    flush_theta(A, K, tkey, gtheta);
}

// ============================================================================ gradient accumulators
// Adds a workgroup's LDS gradient accumulators into the global FP64 accumulator (every thread calls
// it after a workgroup barrier).
DEV void flush_lds_grads(const WArgs& A, const Call& K) {
    __syncthreads();
    const CallTable* T = A.table;
    for (int s = 0; s < MAX_SLOTS; ++s) {
        int od = T->lds_d[s], of = T->lds_f[s];
        if (od < 0 && of < 0) continue;
        int64_t go = T->goff[s], nn = T->numel[s];
        for (int64_t q = threadIdx.x; q < nn; q += BLOCK) {
            double val = od >= 0 ? K.lds_d[od + q] : (double)K.lds_f[of + q];
            if (val != 0.0) unsafeAtomicAdd(A.gacc + go + q, val);
        }
    }
}

// The workgroup's LDS gradient accumulators cleared and the call table copied to LDS (every thread
// calls it; it ends with a workgroup barrier).
DEV void adjoint_begin(const WArgs& A, Call& K, CallTable* tab, double* lds_grad) {
    table_to_lds(tab, A.table);
    K.tab = tab;
    K.lds_d = lds_grad;
    K.lds_f = (float*)(lds_grad + A.lds_nd);
    K.stage = K.lds_f + A.lds_nf + (threadIdx.x / WAVE) * STAGE_WORDS;
    for (int k = threadIdx.x; k < A.lds_nd; k += BLOCK) K.lds_d[k] = 0.0;
    for (int k = threadIdx.x; k < A.lds_nf; k += BLOCK) K.lds_f[k] = 0.0f;
    __syncthreads();
}

// Vertex b of a path in the cached backward's reverse walk, from its record (c0, c1): adds the
// derivatives of E_b + W_b L[b+1] against the adjoint rows av, with L the suffix beyond the vertex (not
// read at the last vertex), and leaves L[b] = E_b + W_b L[b+1] in L.
DEV void adjoint_vertex(const WArgs& A, const Call& K, const DevWorld& W, uint32_t view_id, uint32_t pix, uint32_t smp,
                        int b, bool last, float4 c0, float4 c1, const float* av, float* L) {
    const int hw = __float_as_int(c0.x);
    const v3 d = mk(c1.x, c1.y, c1.z);
    Vtx x;
    surface_at(W, hw & (VTX_PREV_DELTA - 1), c0.y, c0.z, mk(c0.y, c0.z, c0.w), x);
    v3 so, sd;
    float stmax;
    vertex_setup<false>(W, K, view_id, A.seed, pix, smp, b, A.max_depth, A.flags, (hw & VTX_PREV_DELTA) != 0, d, x, so, sd,
                      stmax, last);
    if (x.nee == NEE_PENDING) x.nee = __float_as_int(c1.w) ? NEE_OCCLUDED : NEE_VISIBLE;
    WC w;
    float Ee[12], En[12];
    eval_vertex<true, false>(W, K, x, w, Ee, En, av, L);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        float o4[4];
        w_apply(w, c, L + 4 * c, o4);
#pragma unroll
        for (int k = 0; k < 4; ++k) L[4 * c + k] = (Ee[4 * c + k] + En[4 * c + k]) + o4[k];
    }
}

// ============================================================================ hybrid replay: decision rule
// 4x4 inverse by Laplace expansion along the first two rows: returns det m and writes its adjugate
// (row-major; inverse = adj / det).
DEV float adjugate4(const float* m, float* adj) {
    const float a0 = m[0], a1 = m[1], a2 = m[2], a3 = m[3], b0 = m[4], b1 = m[5], b2 = m[6], b3 = m[7];
    const float c0 = m[8], c1 = m[9], c2 = m[10], c3 = m[11], d0 = m[12], d1 = m[13], d2 = m[14], d3 = m[15];
    const float s0 = a0 * b1 - a1 * b0, s1 = a0 * b2 - a2 * b0, s2 = a0 * b3 - a3 * b0;
    const float s3 = a1 * b2 - a2 * b1, s4 = a1 * b3 - a3 * b1, s5 = a2 * b3 - a3 * b2;
    const float t0 = c0 * d1 - c1 * d0, t1 = c0 * d2 - c2 * d0, t2 = c0 * d3 - c3 * d0;
    const float t3 = c1 * d2 - c2 * d1, t4 = c1 * d3 - c3 * d1, t5 = c2 * d3 - c3 * d2;
    adj[0] = b1 * t5 - b2 * t4 + b3 * t3;   adj[1] = -a1 * t5 + a2 * t4 - a3 * t3;
    adj[2] = d1 * s5 - d2 * s4 + d3 * s3;   adj[3] = -c1 * s5 + c2 * s4 - c3 * s3;
    adj[4] = -b0 * t5 + b2 * t2 - b3 * t1;  adj[5] = a0 * t5 - a2 * t2 + a3 * t1;
    adj[6] = -d0 * s5 + d2 * s2 - d3 * s1;  adj[7] = c0 * s5 - c2 * s2 + c3 * s1;
    adj[8] = b0 * t4 - b1 * t2 + b3 * t0;   adj[9] = -a0 * t4 + a1 * t2 - a3 * t0;
    adj[10] = d0 * s4 - d1 * s2 + d3 * s0;  adj[11] = -c0 * s4 + c1 * s2 - c3 * s0;
    adj[12] = -b0 * t3 + b1 * t1 - b2 * t0; adj[13] = a0 * t3 - a1 * t1 + a2 * t0;
    adj[14] = -d0 * s3 + d1 * s1 - d2 * s0; adj[15] = c0 * s3 - c1 * s1 + c2 * s0;
    return s0 * t5 - s1 * t4 + s2 * t3 + s3 * t2 - s4 * t1 + s5 * t0;
}

// Eq. 3 at vertex v0 of the block [s0, e0) (v0 + 1 < e0): adds the vertex's detached weight and
// emission to the block throughput (Mb, bs) and the remaining radiance, then recovers the suffix
// L[v0+1] into Ln by the scalar PRB update, the inverse, or recomputation of vertices v0+1 .. e0-1
// into the scratch records (rec_from = v0 + 1 afterwards).  One decision serves the three channels:
// their throughputs differ by a scale, which neither test sees.
template <bool EXT>
DEV void suffix_by_rule(const WArgs& A, const Call& K, const DevView& V, const DevWorld& W, const Vtx& x, int slot,
                        uint32_t pix, uint32_t smp, int v0, int s0, int e0, float* Mb, float* bs, float* Lrem,
                        float* Ln, int& rec_from, uint32_t* n_br) {
    WC wf;
    float Ef[12], Enf[12];
    eval_vertex<false, EXT>(W, K, x, wf, Ef, Enf, nullptr, nullptr);
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float se = 0.0f;
#pragma unroll
            for (int j = 0; j < 4; ++j) se += Mb[4 * r + j] * (Ef[4 * c + j] + Enf[4 * c + j]);
            Lrem[4 * c + r] -= bs[c] * se;
        }
    if (wf.kind == 2) {
        WC ws = wf;
        ws.rgb[0] = 1.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float row[4] = {Mb[4 * r], Mb[4 * r + 1], Mb[4 * r + 2], Mb[4 * r + 3]}, o4[4];
            w_row(ws, 0, row, o4);
            Mb[4 * r] = o4[0]; Mb[4 * r + 1] = o4[1]; Mb[4 * r + 2] = o4[2]; Mb[4 * r + 3] = o4[3];
        }
    } else {  // diffuse: only the first column survives; no weight: nothing does
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (wf.kind == 0) Mb[4 * r] = 0.0f;
            Mb[4 * r + 1] = Mb[4 * r + 2] = Mb[4 * r + 3] = 0.0f;
        }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) bs[c] *= wf.kind == 0 ? 0.0f : wf.rgb[c];
    const float m00 = Mb[0];
    const bool live = m00 > 0.0f && bs[0] > 0.0f && bs[1] > 0.0f && bs[2] > 0.0f;
    int br = 2;
    float adj[16], det = 0.0f;
    if (live) {
        const float im = 1.0f / m00;
        float ss = 0.0f, Mn[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) { Mn[k] = Mb[k] * im; ss += Mn[k] * Mn[k]; }
        const float di = sqrtf(fmaxf(0.0f, ss - 1.0f)) * 0.57735026918962576f;  // (normalised: M00 = 1)
        if (di < A.hyb_gamma) {
            br = 0;
        } else {
            det = adjugate4(Mn, adj);
            if (fabsf(det) > A.hyb_eps) br = 1;
        }
    }
    n_br[0] += br == 0 ? 1u : 0u;  // (constant indices: the counters stay in registers)
    n_br[1] += br == 1 ? 1u : 0u;
    n_br[2] += br == 2 ? 1u : 0u;
    if (br == 0) {  // treated as depolarizing: the suffix's intensity only
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            Ln[4 * c] = Lrem[4 * c] / (m00 * bs[c]);
            Ln[4 * c + 1] = Ln[4 * c + 2] = Ln[4 * c + 3] = 0.0f;
        }
    } else if (br == 1) {  // beta^-1 Lrem = (Mn^-1 Lrem) / (m00 bs_c)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float f = 1.0f / (det * m00 * bs[c]);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                Ln[4 * c + r] = f * (adj[4 * r] * Lrem[4 * c] + adj[4 * r + 1] * Lrem[4 * c + 1] +
                                     adj[4 * r + 2] * Lrem[4 * c + 2] + adj[4 * r + 3] * Lrem[4 * c + 3]);
        }
    } else {  // recompute the rest of the block from the ray leaving this vertex
        const PathState& S = A.S;
        const int rec0 = v0 + 1 - s0;
        block_eval<EXT>(A, K, V, W, slot, pix, smp, v0 + 1, e0, spawn(x.p, x.ng, x.wi), x.wi,
                        is_delta(gval(W.mats, (size_t)x.mat).type), rec0);
        ld12(ckpt_rec(S, A.Q, s0 / A.ckpt, slot) + 2, Ln);
        block_fold(S, A.Q, slot, e0 - v0 - 1, Ln, true, rec0);
        rec_from = v0 + 1;
    }
}

// ============================================================================ backward: replay
// Persistent replay of the queued paths from their hit records (no second traversal): every lane
// replays one vertex per iteration and takes the next queued path as soon as its own ends, so
// short and long paths share a wavefront without idling.  At vertex b the lane differentiates
// E_b + W_b L[b+1] against its adjoint rows, then advances them, a <- a W_b.  Gradients go to
// workgroup LDS accumulators, flushed at the end.
//
// Hybrid replay (HYB): the suffix beyond a vertex comes from the scratch records of its block.
// Without RULE the whole block is recomputed from its checkpoint ray when the replay enters it.
// With RULE (Sec. 4.4, Eq. 3) the lane instead carries the detached block throughput beta (the
// product of the block's weights so far: a shared 4x4 and RGB scales) and the radiance of the
// block's checkpoint that its vertices have not yet emitted, Lrem = beta L[b+1], and recovers a
// suffix by the scalar PRB update (Lrem_0 / beta_00, unpolarized) when the depolarization index
// of beta is below gamma, by beta^-1 Lrem when |det beta| > eps beta_00^4, and otherwise by
// recomputing the rest of the block into the scratch records, which the block's later vertices
// then read.  The block's last suffix is the next checkpoint's.
//
// PPRB (the comparator of Sec. 4.2): no cached suffix; the lane carries the regularised radiance
// L'_b still to be explained and recovers the suffix as (W_b + u_b I)^-1 (L'_b - E_b) from the
// primal's weight and emission records, advancing its adjoint rows by W_b + u_b I.
template <bool HYB, bool EXT, bool RULE = false, bool PPRB = false>
// (three waves per SIMD for the hybrid replay: one register more had made it two, 7.2 ms against 5.1 ms for
// the 230,400 paths of depth 128)
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(HYB && !RULE && !EXT ? 3 : 1, 8))) k_replay(WArgs A) {
    extern __shared__ double lds_grad[];
    PathState& S = A.S;
    const int Q = A.Q;
    Call K{A.table, A.gacc};
    __shared__ CallTable tab;
    adjoint_begin(A, K, &tab, lds_grad);
    const int n = S.counts[CNT_REPLAY];
    WaveFetch F(n, 0, true);
    int slot = -1, b = 0, B = 0, v = 0;
    uint32_t pix = 0, smp = 0;
    bool prev_delta = false;
    float av[12];
    v3 o = mk(0.0f, 0.0f, 0.0f), d = o;
#pragma unroll
    for (int k = 0; k < 12; ++k) av[k] = 0.0f;
    // decision-rule state (RULE): block throughput (shared part and RGB scales), remaining radiance,
    // first vertex of the block whose suffix sits in the scratch records, and branch counts
    float Mb[RULE ? 16 : 1], bs[RULE ? 3 : 1], Lrem[RULE ? 12 : 1];
    float Lcur[PPRB ? 12 : 1];  // PPRB: the regularised suffix at the current vertex
    int rec_from = 0;
    uint32_t n_br[3] = {0u, 0u, 0u};
    while (true) {
        // hand queue entries to the lanes without a path
        const int idx = F.take(slot < 0, n, S, WORK_REPLAY);
        if (idx >= 0) {
            slot = S.queue0[idx];
            // the path's start as the fold left it in the shadow-record array (one record per path)
            const float4* H = shd_rec(S, slot);
            const float4 h0 = H[0], h1 = H[1];
            const int info = __float_as_int(h0.w);
            B = info & 255;
            v = info >> 12;
            b = 1;
            prev_delta = false;
            pix = __float_as_uint(h1.x);
            smp = __float_as_uint(h1.y);
            ld12(H + 2, av);
            if (PPRB) ld12(H + 5, Lcur);
            d = mk(h0.x, h0.y, h0.z);
            o = ld3(gval(A.views, (size_t)v).o);  // (a pinhole camera's rays leave the view's origin)
        }
        if (!__any(slot >= 0)) break;
        if (slot >= 0) {
            const DevView V = gval(A.views, (size_t)v);
            const DevWorld W = world_of(A, V);
            uint32_t hw;
            float hu, hv;
            const float4* C;  // the record whose E words hold the suffix beyond this vertex
            const int v0 = b - 1;
            const int s0 = HYB ? v0 - v0 % A.ckpt : 0, e0 = HYB ? min(B, s0 + A.ckpt) : 0;
            if (HYB) {
                if (!RULE && v0 == s0) {  // block start: recompute the block's suffix values
                    block_eval<EXT>(A, K, V, W, slot, pix, smp, v0, e0, o, d, prev_delta);
                    float Lb[12];
                    ld12(ckpt_rec(S, Q, v0 / A.ckpt, slot) + 2, Lb);
                    block_fold(S, Q, slot, e0 - v0, Lb, true);
                }
                if constexpr (RULE) {
                    if (v0 == s0) {  // block start: beta = I, Lrem = the suffix at the block's first vertex
#pragma unroll
                        for (int k = 0; k < 16; ++k) Mb[k] = (k % 5 == 0) ? 1.0f : 0.0f;
                        bs[0] = bs[1] = bs[2] = 1.0f;
                        ld12(s0 == 0 ? shd_rec(S, slot) + 5 : ckpt_rec(S, Q, s0 / A.ckpt - 1, slot) + 2, Lrem);
                        rec_from = 0x7fffffff;
                    }
                }
                const float4 hr = *hit_rec(S, Q, v0, slot);
                hw = __float_as_uint(hr.x); hu = hr.y; hv = hr.z;
                C = cache_rec(S, Q, v0 - s0, slot);
            } else {
                C = cache_rec(S, Q, b - 1, slot);
                const float4 c2 = C[2], c3 = C[3];
                hw = __float_as_uint(c2.w); hu = c3.x; hv = c3.y;
            }
            Hit h;
            h.prim = (int)(hw & ((1u << 26) - 1));
            // the next-event visibility: in the hit record's word (hybrid), in the cache record's
            // last vector (cached)
            const int rec_nee = HYB ? (int)((hw >> 26) & 7) : __float_as_int(C[7].x);
            h.u = hu; h.t = hu; h.v = hv;
            Vtx x;
            surface(W, h, o, d, x);
            v3 so, sd;
            float stmax;
            vertex_setup<EXT>(W, K, V.view_id, A.seed, pix, smp, b, A.max_depth, A.flags, prev_delta, d, x, so, sd, stmax);
            if (x.nee == NEE_PENDING) x.nee = rec_nee;
            float Ln[12];  // L[b+1], stored in this vertex's record by the fold (zero after the last)
            if (b >= B) {
#pragma unroll
                for (int q = 0; q < 12; ++q) Ln[q] = 0.0f;
            } else if (PPRB) {
                // (W_b + u I)^-1 (L'_b - E_b) per channel, from the primal's records
                const float4 c0 = C[0], c1 = C[1], c2 = C[2];
                WC wr;
                wr.rgb[0] = c0.x; wr.rgb[1] = c0.y; wr.rgb[2] = c0.z;
                wr.A = c0.w; wr.B = c1.x; wr.C = c1.y; wr.D = c1.z;
                wr.ci = c1.w; wr.si = c2.x; wr.co = c2.y; wr.so = c2.z;
                wr.kind = (__float_as_int(c2.w) >> 29) & 3;
                float e[12];
                ld12(C + 4, e);
                const float u = pprb_noise(A, pix, smp, V.view_id, b);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    float m[16], adj[16];
                    w_matrix(wr, c, m);
                    m[0] += u; m[5] += u; m[10] += u; m[15] += u;
                    const float idet = 1.0f / adjugate4(m, adj);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float t = 0.0f;
#pragma unroll
                        for (int j = 0; j < 4; ++j) t += adj[4 * r + j] * (Lcur[4 * c + j] - e[4 * c + j]);
                        Ln[4 * c + r] = t * idet;
                    }
                }
            } else if (!RULE) {
                ld12(C + 4, Ln);
            } else if (v0 + 1 == e0) {  // the block's last suffix: the next checkpoint's
                ld12(ckpt_rec(S, Q, s0 / A.ckpt, slot) + 2, Ln);
            } else if (v0 >= rec_from) {  // recomputed earlier in this block
                ld12(C + 4, Ln);
            } else {
                suffix_by_rule<EXT>(A, K, V, W, x, slot, pix, smp, v0, s0, e0, Mb, bs, Lrem, Ln, rec_from, n_br);
            }
            WC w;
            float Ee[12], En[12];
            K.coherent = b == 1;
            eval_vertex<true, EXT>(W, K, x, w, Ee, En, av, Ln);
            if (b >= B || x.lobe == LOBE_NONE || x.lobe == LOBE_INVALID) {
                slot = -1;
            } else {
                const float un = PPRB ? pprb_noise(A, pix, smp, V.view_id, b) : 0.0f;
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) {
                    float o4[4];
                    w_row(w, cc, av + 4 * cc, o4);
#pragma unroll
                    for (int q = 0; q < 4; ++q) av[4 * cc + q] = o4[q] + (PPRB ? un * av[4 * cc + q] : 0.0f);
                }
                if (PPRB)
#pragma unroll
                    for (int q = 0; q < 12; ++q) Lcur[q] = Ln[q];
                prev_delta = is_delta(gval(W.mats, (size_t)x.mat).type);
                o = spawn(x.p, x.ng, x.wi);
                d = x.wi;
                ++b;
            }
        }
    }
    // flush the workgroup accumulators into the global FP64 accumulator
    __syncthreads();
    if (RULE && A.hyb_stats) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const uint32_t t = wave_sum_u(n_br[k]);
            if (lane_id() == 0 && t) atomicAdd(&A.hyb_stats[k], (unsigned long long)t);
        }
    }
    flush_lds_grads(A, K);
}

#ifndef PPT_EXT_TU  // (in the main compilation unit only)
// ============================================================================ cached backward: reverse walk
// The gradient of the cached backward (Sec. 4.3, Fig. 2) without a separate fold: the forward pass of
// the backward carries each path's adjoint row a_b (known from the start, since dL/dI is an input)
// and keeps it per vertex, so one walk from the last vertex to the first can evaluate every vertex
// once, differentiate E_b + W_b L[b+1] against a_b, and advance the suffix L[b] = E_b + W_b L[b+1] in
// registers.  No Mueller matrix is inverted and no suffix goes through memory, except the one
// beyond the first vertex.  Against the fold (read 96 B, write 48 B of a 128-byte record per vertex)
// followed by a forward replay (read it again) this moves 32 B written and read per first vertex and
// 64 to 80 B per later one.
//
// the adjoint rows of a vertex from their rank-one form
DEV void row1_load(const float4* r, float* av) {
    const float4 a0 = r[0], a1 = r[1];
    const float sc[3] = {a1.x, a1.y, a1.z};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        av[4 * c] = sc[c] * a0.x; av[4 * c + 1] = sc[c] * a0.y;
        av[4 * c + 2] = sc[c] * a0.z; av[4 * c + 3] = sc[c] * a0.w;
    }
}
// the polarizer-angle term of a path whose radiance at its first vertex is L: dp is the pixel's dL/dI, inv = 1 / spp
DEV float theta_term(const float* dp, float inv, float C2, float S2, float Cs, float Ss, const float* L) {
    float gt = 0.0f;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const float l1 = L[4 * c + 1], l2 = L[4 * c + 2];
        const float ls[4] = {L[4 * c], Cs * l1 + Ss * l2, -Ss * l1 + Cs * l2, L[4 * c + 3]};
        const float dl[3] = {gval(dp, 4 * c) * inv, gval(dp, 4 * c + 1) * inv, gval(dp, 4 * c + 2) * inv};
        gt += polarizer_dtheta(C2, S2, dl, ls);
    }
    return gt;
}
// k_adjoint_deep walks the paths of two or more vertices (the hit queue of the second bounce) down to
// their second vertex: persistent, a lane takes the next path as soon as its own is walked, and
// leaves the suffix L[2] in the path's ray record, which nothing reads any more.
template <bool R1>
__global__ void __launch_bounds__(BLOCK) k_adjoint_deep(WArgs A) {
    extern __shared__ double lds_grad[];
    PathState& S = A.S;
    const int Q = A.Q;
    Call K{A.table, A.gacc};
    __shared__ CallTable tab;
    const int n = S.counts[CNT_REPLAY];
    if (!fetch_active(n) || n == 0) return;
    adjoint_begin(A, K, &tab, lds_grad);
    WaveFetch F(n);
    int slot = -1, b = 0, B = 0, v = 0;
    uint32_t pix = 0, smp = 0, view_id = 0;
    float L[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) L[k] = 0.0f;
    while (true) {
        const int idx = F.take(slot < 0, n, S, WORK_REPLAY);
        if (idx >= 0) {
            slot = S.dqueue[idx];
            const float4 r3 = ray_rec(S, slot)[3];
            const int info = __float_as_int(r3.x);
            B = b = info & 255;
            v = info >> 12;
            pix = __float_as_uint(r3.y);
            smp = __float_as_uint(r3.z);
            view_id = __float_as_uint(r3.w);
#pragma unroll
            for (int k = 0; k < 12; ++k) L[k] = 0.0f;
        }
        if (!__any(slot >= 0)) break;
        if (slot >= 0) {
            const float4* C = vtx_rec(S, Q, b - 1, slot);
            const float4 c0 = C[0], c1 = C[1];
            float av[12];
            if (R1) {
                row1_load(row_rec<true>(S, Q, b - 1, slot), av);
            } else {
                ld12(row_rec<false>(S, Q, b - 1, slot), av);
            }
            K.coherent = false;
            adjoint_vertex(A, K, world_of(A, v), view_id, pix, smp, b, b == B, c0, c1, av, L);
            if (--b == 1) {
                st12(ray_rec(S, slot), L);
                slot = -1;
            }
        }
    }
    flush_lds_grads(A, K);
}
// k_adjoint_first evaluates the first vertex of every path, a wavefront's lanes holding consecutive
// paths (the samples of one pixel or two: one material, one texel cell, no idle lanes beside the
// escaped camera rays), with the suffix beyond it from k_adjoint_deep, and adds the polarizer-angle
// term delta^T (dP/dtheta) R_s L[1].  A wavefront takes runs of ADJ_RUN paths from a counter (a fixed
// stride walks the same part of every view of a batch of equal views, and the wavefronts on its
// objects end last: 5.2 ms against 2.7 ms on the 128-view batch), long enough that its lanes seldom change
// view and keep the angle term in a register until they do.  TINY: a view's lanes are few, and each looks up its own.
constexpr int ADJ_RUN = 8 * WAVE;
template <bool TINY>
__global__ void __launch_bounds__(BLOCK) k_adjoint_first(WArgs A) {
    extern __shared__ double lds_grad[];
    PathState& S = A.S;
    const int Q = A.Q;
    Call K{A.table, A.gacc};
    const Call KG{A.table, A.gacc};  // (the angle terms: straight to the FP64 accumulator)
    __shared__ CallTable tab;
    adjoint_begin(A, K, &tab, lds_grad);
    K.coherent = true;
    const int n = A.n_chunk;
    const int waves = (int)gridDim.x * (BLOCK / WAVE);
    // (shorter where the paths are few: eight runs per wavefront even out their cost)
    const int run = min(ADJ_RUN, (n / (8 * waves) + WAVE) & ~(WAVE - 1));
    ViewRange range;
    float gtheta = 0.0f, C2 = 1.0f, S2 = 0.0f;
    int tkey = -1, angle_of = -1;
    while (true) {
        const int r0 = work_ticket(S, WORK_ADJOINT, wave_number(), waves) * run;
        if (r0 >= n) break;
        for (int base = r0; base < min(r0 + run, n); base += WAVE) {
            const int i = base + lane_id();
            const int B = i < n ? (int)S.nv[i] : 0;
            int v = -1;
            float gt = 0.0f;
            bool pol = false;
            auto first = [&](int vw, const DevView& V) {
                v = vw;
                const float4* C = vtx_rec(S, Q, 0, i);
                const float4 c0 = C[0], c1 = C[1];
                float L[12];
                if (B > 1) {
                    ld12(ray_rec(S, i), L);
                } else {
#pragma unroll
                    for (int k = 0; k < 12; ++k) L[k] = 0.0f;
                }
                const PathId id = path_keys(V, A.g0 + i);
                pol = V.sensor == SENSOR_POLARIZER;
                if (pol && angle_of != vw) {  // (the polarizer's angle again only where the view changes)
                    const float theta = K.p(V.theta_slot, V.theta_off);
                    C2 = cosf(2.0f * theta);
                    S2 = sinf(2.0f * theta);
                    angle_of = vw;
                }
                const int64_t px_off = V.out_off + ((int64_t)id.ly * V.crop_w + id.lx) * 12;
                const v3 kc = mk(-c1.x, -c1.y, -c1.z);
                float Cs, Ss;
                rot_cs(kc, canon_x(kc), normalize(ld3(V.r) - kc * dot(ld3(V.r), kc)), Cs, Ss);
                float av[12];
                sensor_rows(A, V, px_off, C2, S2, Cs, Ss, av);
                const DevWorld W = TINY || A.one_world ? world_of(A, V) : cval(A.worlds, V.world);
                adjoint_vertex(A, K, W, V.view_id, id.pix, id.smp, 1, B == 1, c0, c1, av, L);
                if (pol) gt = theta_term(A.dout + px_off, 1.0f / (float)V.spp, C2, S2, Cs, Ss, L);
            };
            if constexpr (TINY) {
                if (B > 0) {
                    const int vw = lane_view(A, A.g0 + i);
                    first(vw, gval(A.views, (size_t)vw));
                }
            } else {
                for_views<false>(A, range, B > 0, A.g0 + i, first);
            }
            if (__any(pol && tkey >= 0 && tkey != v)) {
                flush_theta(A, KG, tkey, gtheta);
                tkey = -1;
                gtheta = 0.0f;
            }
            if (pol) {
                tkey = v;
                gtheta += gt;
            }
        }
    }
    flush_theta(A, KG, tkey, gtheta);
    flush_lds_grads(A, K);
}

// The reverse walk of a small call in one launch, every vertex of a path from its last to its first: a
// wavefront takes per_wave consecutive paths, whose first vertices add to a texel cell together where that many
// can share one (196,608 paths of 12 samples, 256 x 256 maps of which six texels are in view, depth 6: 975 us against 1,785).
template <bool R1>
__global__ void __launch_bounds__(BLOCK) k_adjoint_paths(WArgs A, int per_wave) {
    extern __shared__ double lds_grad[];
    PathState& S = A.S;
    const int Q = A.Q;
    Call K{A.table, A.gacc};
    const Call KG{A.table, A.gacc};  // (the angle terms: straight to the FP64 accumulator)
    __shared__ CallTable tab;
    adjoint_begin(A, K, &tab, lds_grad);
    const int wave = wave_number();
    const int i = wave * per_wave + lane_id();
    const int B = lane_id() < per_wave && i < A.n_chunk ? (int)S.nv[i] : 0;
    int v = 0, tkey = -1;
    uint32_t pix = 0, smp = 0, view_id = 0;
    if (B > 0) {
        const float4 r3 = ray_rec(S, i)[3];
        v = __float_as_int(r3.x) >> 12;
        pix = __float_as_uint(r3.y);
        smp = __float_as_uint(r3.z);
        view_id = __float_as_uint(r3.w);
    }
    float L[12], gt = 0.0f;
#pragma unroll
    for (int k = 0; k < 12; ++k) L[k] = 0.0f;
    for (int b = B; b > 0; --b) {
        const float4* C = vtx_rec(S, Q, b - 1, i);
        const float4 c0 = C[0], c1 = C[1];
        float av[12], Cs = 1.0f, Ss = 0.0f, C2 = 1.0f, S2 = 0.0f, inv = 0.0f;
        const float* dp = nullptr;
        if (b == 1) {
            const DevView V = gval(A.views, (size_t)v);
            if (V.sensor == SENSOR_POLARIZER) {
                const float th = K.p(V.theta_slot, V.theta_off);
                C2 = cosf(2.0f * th);
                S2 = sinf(2.0f * th);
                tkey = v;
            }
            const v3 kc = mk(-c1.x, -c1.y, -c1.z);
            rot_cs(kc, canon_x(kc), normalize(ld3(V.r) - kc * dot(ld3(V.r), kc)), Cs, Ss);
            const int64_t px_off = pixel_offset(V, pix);
            sensor_rows(A, V, px_off, C2, S2, Cs, Ss, av);
            dp = A.dout + px_off;
            inv = 1.0f / (float)V.spp;
        } else if (R1) {
            row1_load(row_rec<true>(S, Q, b - 1, i), av);
        } else {
            ld12(row_rec<false>(S, Q, b - 1, i), av);
        }
        K.coherent = b == 1 && per_wave >= GROUP_MIN;
        adjoint_vertex(A, K, world_of(A, v), view_id, pix, smp, b, b == B, c0, c1, av, L);
        if (b == 1 && tkey >= 0) gt = theta_term(dp, inv, C2, S2, Cs, Ss, L);
    }
    flush_theta(A, KG, tkey, gt);
    flush_lds_grads(A, K);
}

// ============================================================================ P-RB comparator
// Polarized radiative backpropagation (the comparator of Sec. 5.1): the replay reads, for each vertex
// b1, an independent estimate of the suffix beyond it instead of the cached one.  Pass b1 traces,
// for every path with more than b1 vertices, a new path from the ray leaving vertex b1 (state S2,
// key prb_seed(seed, b1 + 1), vertex numbers continuing at b1 + 1) through the usual bounce kernels,
// and stores its radiance over the cached suffix in the vertex's record.
DEV uint64_t prb_seed(uint64_t seed, uint32_t v_first) { return seed + (uint64_t)v_first * 0x9E3779B97F4A7C15ull; }

// The ray leaving vertex b1 of each path: its prefix is replayed from the camera ray (its direction
// written by the fold) and the hit records, with the path's own key; the sub-path starts there with an identity
// throughput and no radiance.  Paths with b1 or fewer vertices start nothing.
__global__ void __launch_bounds__(BLOCK) k_prb_start(WArgs A, PathState S2, int b1) {
    const PathState& S = A.S;
    const int Q = A.Q;
    Call K{A.table, nullptr};
    for (int i = blockIdx.x * BLOCK + threadIdx.x; i < A.n_chunk; i += gridDim.x * BLOCK) {
        float4* R2 = ray_rec(S2, i);
        if ((int)S.nv[i] <= b1) {
            R2[3] = f4(__int_as_float(info_make(b1, false, 0) | INFO_DEAD), 0.0f, 0.0f, 0.0f);
            S2.hflag[i] = 2;
            continue;
        }
        const float4 r3 = ray_rec(S, i)[3];
        const int view = __float_as_int(r3.x) >> 12;
        const DevView V = gval(A.views, (size_t)view);
        const DevWorld W = world_of(A, V);
        const uint32_t pix = __float_as_uint(r3.y), smp = __float_as_uint(r3.z);
        // the camera ray: the view's origin and the direction the fold stored in the shadow record
        const float4 h0 = shd_rec(S, i)[0];
        v3 o = ld3(V.o), d = mk(h0.x, h0.y, h0.z);
        bool prev_delta = false;
        for (int b = 1; b <= b1; ++b) {
            const float4* C = cache_rec(S, Q, b - 1, i);
            const float4 c2 = C[2], c3 = C[3];
            const uint32_t hw = __float_as_uint(c2.w);
            Hit h;
            h.prim = (int)(hw & ((1u << 26) - 1));
            h.u = c3.x; h.t = c3.x; h.v = c3.y;
            Vtx x;
            surface(W, h, o, d, x);
            v3 so, sd;
            float stmax;
            vertex_setup<false>(W, K, V.view_id, A.seed, pix, smp, b, A.max_depth, A.flags, prev_delta, d, x, so, sd, stmax);
            prev_delta = is_delta(gval(W.mats, (size_t)x.mat).type);
            o = spawn(x.p, x.ng, x.wi);
            d = x.wi;
        }
        ray_set(R2, o, d);
        R2[2] = f4(0.0f, 0.0f, 0.0f, 0.0f);
        R2[3] = f4(__int_as_float(info_make(b1, prev_delta, view)), r3.y, r3.z, r3.w);
        float4* AC = acc_rec(S2, i);
        AC[0] = f4(1.0f, 0.0f, 0.0f, 0.0f); AC[1] = f4(0.0f, 1.0f, 0.0f, 0.0f);
        AC[2] = f4(0.0f, 0.0f, 1.0f, 0.0f); AC[3] = f4(0.0f, 0.0f, 0.0f, 1.0f);
        AC[4] = f4(1.0f, 1.0f, 1.0f, 0.0f);
        AC[5] = AC[6] = AC[7] = f4(0.0f, 0.0f, 0.0f, 0.0f);
        S2.hflag[i] = 0;
    }
}
// The sub-path radiance of pass b1 over the cached suffix beyond vertex b1.
__global__ void __launch_bounds__(BLOCK) k_prb_store(WArgs A, PathState S2, int b1) {
    const PathState& S = A.S;
    for (int i = blockIdx.x * BLOCK + threadIdx.x; i < A.n_chunk; i += gridDim.x * BLOCK) {
        if ((int)S.nv[i] <= b1) continue;
        float Lo[12];
        ld12(acc_rec(S2, i) + 5, Lo);
        st12(cache_rec(S, A.Q, b1 - 1, i) + 4, Lo);
    }
}

// ============================================================================ tape AD baseline: reverse sweep
// Conventional reverse-mode AD of the path loop (the "Conv. AD" the paper compares against, Sec. 5.1,
// 5.4): the forward pass stored every vertex's loop state on the tape (prefix throughput beta_b,
// weight W_b, emission E_b, hit and incoming ray); this kernel walks each path from its last vertex
// to its first, carrying the adjoint of the throughput as a full 4x4 matrix per channel, as a
// generic reverse sweep does (it does not know that the adjoint is an outer product):
//   Ebar_b = beta_b^T a0,   Wbar_b = beta_b^T betabar_{b+1},   betabar_b = a0 E_b^T + betabar_{b+1} W_b^T,
// with a0 the adjoint of the path's radiance at the sensor; each vertex's parameter derivatives
// come from its re-evaluated interaction with (Ebar_b, Wbar_b).  Scenes without the light-stage
// features only.
__global__ void __launch_bounds__(BLOCK) k_tape_reverse(WArgs A) {
    extern __shared__ double lds_grad[];
    PathState& S = A.S;
    const int Q = A.Q;
    Call K{A.table, A.gacc};
    __shared__ CallTable tab;
    adjoint_begin(A, K, &tab, lds_grad);
    const int n = S.counts[CNT_REPLAY];
    WaveFetch F(n, 0, true);
    int slot = -1, b = 0, v = 0;
    uint32_t pix = 0, smp = 0;
    float a0[12], bbar[48];  // adjoint at the sensor; adjoint of beta_{b+1} per channel (4x4, row-major)
#pragma unroll
    for (int k = 0; k < 12; ++k) a0[k] = 0.0f;
#pragma unroll
    for (int k = 0; k < 48; ++k) bbar[k] = 0.0f;
    while (true) {
        const int idx = F.take(slot < 0, n, S, WORK_REPLAY);
        if (idx >= 0) {
            slot = S.queue0[idx];
            const float4 r3 = ray_rec(S, slot)[3];
            const int info = __float_as_int(r3.x);
            b = info & 255;
            v = info >> 12;
            pix = __float_as_uint(r3.y);
            smp = __float_as_uint(r3.z);
            ld12(shd_rec(S, slot) + 2, a0);
#pragma unroll
            for (int k = 0; k < 48; ++k) bbar[k] = 0.0f;
        }
        if (!__any(slot >= 0)) break;
        if (slot >= 0) {
            const DevView V = gval(A.views, (size_t)v);
            const DevWorld W = world_of(A, V);
            const float4* T = tape_rec(S, Q, b - 1, slot);
            const float4 t0 = T[0], t1 = T[1], t2 = T[2], t3 = T[3], t12 = T[12], t13 = T[13], t14 = T[14];
            WC wt;
            wt.rgb[0] = t0.x; wt.rgb[1] = t0.y; wt.rgb[2] = t0.z;
            wt.A = t0.w; wt.B = t1.x; wt.C = t1.y; wt.D = t1.z;
            wt.ci = t1.w; wt.si = t2.x; wt.co = t2.y; wt.so = t2.z;
            const uint32_t hw = __float_as_uint(t2.w);
            wt.kind = (int)((hw >> 29) & 3);
            float E[12], M[16];
            ld12(T + 4, E);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 q = T[8 + k];
                M[4 * k] = q.x; M[4 * k + 1] = q.y; M[4 * k + 2] = q.z; M[4 * k + 3] = q.w;
            }
            const float brgb[3] = {t12.x, t12.y, t12.z};
            // Ebar_b = beta_b^T a0 and Wbar_b = beta_b^T betabar_{b+1}, per channel (beta_c = brgb_c M)
            float Eb[12], Wb[48];
#pragma unroll
            for (int c = 0; c < 3; ++c)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    float t = 0.0f;
#pragma unroll
                    for (int i = 0; i < 4; ++i) t += M[4 * i + j] * a0[4 * c + i];
                    Eb[4 * c + j] = brgb[c] * t;
#pragma unroll
                    for (int l = 0; l < 4; ++l) {
                        float u = 0.0f;
#pragma unroll
                        for (int i = 0; i < 4; ++i) u += M[4 * i + j] * bbar[16 * c + 4 * i + l];
                        Wb[16 * c + 4 * j + l] = brgb[c] * u;
                    }
                }
            // the interaction again, from the stored ray and hit
            Hit h;
            h.prim = (int)(hw & ((1u << 26) - 1));
            h.u = t3.x; h.t = t3.x; h.v = t3.y;
            const v3 o = mk(t13.x, t13.y, t13.z), d = mk(t13.w, t14.x, t14.y);
            Vtx x;
            surface(W, h, o, d, x);
            v3 so, sd;
            float stmax;
            vertex_setup<false>(W, K, V.view_id, A.seed, pix, smp, b, A.max_depth, A.flags, t12.w != 0.0f, d, x,
                                so, sd, stmax);
            if (x.nee == NEE_PENDING) x.nee = (int)((hw >> 26) & 7);
            WC w;
            float Ee[12], En[12];
            K.coherent = b == 1;
            eval_vertex<true, false, true>(W, K, x, w, Ee, En, Eb, Wb);
            // betabar_b = a0 E_b^T + betabar_{b+1} W_b^T (the stored weight)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                float Wm[16];
                w_matrix(wt, c, Wm);
                float nb_[16];
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        float t = a0[4 * c + i] * E[4 * c + j];
#pragma unroll
                        for (int k = 0; k < 4; ++k) t += bbar[16 * c + 4 * i + k] * Wm[4 * j + k];
                        nb_[4 * i + j] = t;
                    }
#pragma unroll
                for (int k = 0; k < 16; ++k) bbar[16 * c + k] = nb_[k];
            }
            if (--b == 0) slot = -1;
        }
    }
    flush_lds_grads(A, K);
}

// ============================================================================ small kernels
// Start of a call: the call table, the work counters, the queue counts of the first chunk, and the arrays that the
// call accumulates into (image, FP64 gradients) cleared, in one launch.
__global__ void k_setup(CallTable tab, CallTable* dst, Stats* stats, int reset_stats, int* counts, float* img,
                        int64_t n_img, double* gacc, int64_t n_gacc) {
    if (blockIdx.x == 0) {
        const int n = (int)(sizeof(CallTable) / sizeof(int));
        for (int k = threadIdx.x; k < n; k += BLOCK) ((int*)dst)[k] = ((const int*)&tab)[k];
        const int i = threadIdx.x;
        if (i < ST_COUNT && reset_stats) stats->c[i] = 0ull;
        if (i < 3 && reset_stats) stats->hyb[i] = 0ull;
        for (int k = i; k < COUNT_INTS; k += BLOCK) counts[k] = 0;
    }
    const int64_t i0 = (int64_t)blockIdx.x * BLOCK + threadIdx.x, step = (int64_t)gridDim.x * BLOCK;
    for (int64_t i = i0; i < n_img; i += step) img[i] = 0.0f;
    for (int64_t i = i0; i < n_gacc; i += step) gacc[i] = 0.0;
}
__global__ void k_finalize(const CallTable* tab, const double* gacc, int n_slots) {
    for (int s = 0; s < n_slots; ++s) {
        float* out = tab->gout[s];
        int64_t off = tab->goff[s], n = tab->numel[s];
        if (!out || off < 0) continue;
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
            out[i] = (float)gacc[off + i];
    }
}
__global__ void k_rng(uint64_t seed, const uint32_t* ctr, uint32_t* out, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t c0 = ctr[4 * i], c1 = ctr[4 * i + 1], c2 = ctr[4 * i + 2], c3 = ctr[4 * i + 3];
    philox(c0, c1, c2, c3, (uint32_t)seed, (uint32_t)(seed >> 32));
    out[4 * i] = c0; out[4 * i + 1] = c1; out[4 * i + 2] = c2; out[4 * i + 3] = c3;
}

// ============================================================================ fixed scratch
// Device memory of the allocation-free backward entry point: the per-path records of one chunk and
// the FP64 gradient accumulators live here instead of in a caller workspace.  Each GPU the library
// runs on holds its own copy until the process ends.  In host code `scratch` names a host-side
// stand-in, never the device array: its device address is looked up once per device
// (hipGetSymbolAddress with that device current) and only that address is used afterwards.
static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

hipError_t noalloc_scratch(void** ptr) {
    constexpr int MAX_DEVICES = 64;
    static std::mutex mu;
    static void* addr[MAX_DEVICES] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p || ((uintptr_t)p & 255) != 0) return hipErrorInvalidValue;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

// ============================================================================ launchers
static uint64_t prb_seed_host(uint64_t seed, uint32_t v_first) { return seed + (uint64_t)v_first * 0x9E3779B97F4A7C15ull; }
static int blocks_for(int64_t n, int cap) {
    int64_t b = (n + BLOCK - 1) / BLOCK;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (int)b;
}

hipError_t launch_setup(const CallTable& tab, CallTable* dst, Stats* stats, bool reset_stats, int* counts, float* img,
                        int64_t n_img, double* gacc, int64_t n_gacc, hipStream_t s) {
    const int64_t n = n_img > n_gacc ? n_img : n_gacc;
    hipLaunchKernelGGL(k_setup, dim3(blocks_for(n, 4096)), dim3(BLOCK), 0, s, tab, dst, stats, reset_stats ? 1 : 0, counts,
                       img, n_img, gacc, n_gacc);
    return hipGetLastError();
}
hipError_t launch_finalize(const CallTable* tab, const double* gacc, int n_slots, int64_t max_numel, hipStream_t s) {
    hipLaunchKernelGGL(k_finalize, dim3(blocks_for(max_numel, 2048)), dim3(BLOCK), 0, s, tab, gacc, n_slots);
    return hipGetLastError();
}
hipError_t launch_rng(uint64_t seed, const uint32_t* ctr, uint32_t* out, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_rng, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, seed, ctr, out, n);
    return hipGetLastError();
}

// Workgroups of a grid-filling launch of kernel fn: as many per compute unit as its registers and
// its LDS (static + lds bytes) allow, and no more than the items need.
static int resident_grid(const void* fn, size_t lds, int64_t n, const LaunchGrid& G) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, BLOCK, lds) != hipSuccess || per_cu < 1) per_cu = 1;
    return blocks_for(n, per_cu * G.cu);
}

// The variants for scenes with the light-stage features are compiled in their own unit
// (ppt_kernels_ext.hip) with FP32 division and square root correctly rounded: they differentiate
// the shading normal through the smooth dielectric's s/p rotators, which amplify rounding.
extern template __global__ void k_shade<0, true>(WArgs);
extern template __global__ void k_shade<1, true>(WArgs);
extern template __global__ void k_shade<2, true>(WArgs);
extern template __global__ void k_fold<true, true, false, false>(WArgs);
extern template __global__ void k_replay<false, true, false, false>(WArgs);
extern template __global__ void k_replay<true, true, false, false>(WArgs);
extern template __global__ void k_replay<true, true, true, false>(WArgs);
extern template __global__ void k_replay<false, true, false, true>(WArgs);

// LDS of a gradient kernel: the workgroup accumulators, and the staging memory of texture scatters
static size_t grad_lds(const WArgs& a) {
    return (size_t)a.lds_nd * sizeof(double) + (size_t)a.lds_nf * sizeof(float) +
           (a.lds_stage ? (size_t)(BLOCK / WAVE) * STAGE_WORDS * sizeof(float) : 0);
}

// Paths per wavefront of a small call, at least `least` and at most half a wavefront: spread over 4,096 wavefronts
// (four per SIMD, of which three are resident: all variants but the hybrid replay's without counters hold 130 to 155
// registers) where the tree is deep (a path's rays then differ, and wait for each other), over 2,048 where it is
// shallow and shading, the same for every wavefront, is the larger part.  16,384 paths, depth 6, render and backward, 4,096 and
// 2,048 wavefronts, by stack entries: 5 (three spheres) 112 and 88 us (the backward), 8 (40 triangles) 60 + 118 and
// 61 + 99, 9 (80 triangles) 98 + 168 and 90 + 131, 20 (20.5k triangles) 140 + 206 and 171 + 214.  In between 12 entries (200
// triangles) 149 + 235 and 145 + 208, 15 (1,000) 366 + 447 and 387 + 437, at 32,768 paths 453 + 539 and 392 + 446: the
// line lies where neither form loses below it.
constexpr int SMALL_LEAST = 2, SMALL_LEAST_ADJ = 4, SMALL_WAVES_DEEP = 4096, SMALL_WAVES_SHALLOW = 2048, SMALL_WAVES_WALK = 3072,
              SMALL_SCATTERS = 8192;
static int small_per_wave(const WArgs& a, int least) {
    const int waves = a.stack_cap > SHALLOW_STACK ? SMALL_WAVES_DEEP : SMALL_WAVES_SHALLOW;
    const int pw = (a.n_chunk + waves - 1) / waves;
    return pw < least ? least : pw > WAVE / 2 ? WAVE / 2 : pw;
}

// A traversal launch, with or without the work counters.
template <int SMODE>
static void launch_extend(const WArgs& a, int grid, size_t lds, hipStream_t s) {
    if (a.stats) hipLaunchKernelGGL((k_extend<SMODE, true>), dim3(grid), dim3(BLOCK), lds, s, a);
    else hipLaunchKernelGGL((k_extend<SMODE, false>), dim3(grid), dim3(BLOCK), lds, s, a);
}

// A small call: its paths in one launch, then the pixel reduction or the reverse walk.
template <int MODE>
static void launch_paths(const WArgs& a, int per_wave, size_t lds, hipStream_t s) {
    const int per_block = per_wave * (BLOCK / WAVE), grid = (a.n_chunk + per_block - 1) / per_block;
    if (a.stats) hipLaunchKernelGGL((k_paths<MODE, true>), dim3(grid), dim3(BLOCK), lds, s, a, per_wave);
    else hipLaunchKernelGGL((k_paths<MODE, false>), dim3(grid), dim3(BLOCK), lds, s, a, per_wave);
}
static void launch_small_paths(const WArgs& a, int mode, hipStream_t s) {
    const size_t lds = (size_t)a.stack_cap * BLOCK * sizeof(int);
    const int pw = small_per_wave(a, SMALL_LEAST);
    if (mode == 0 && a.r1) launch_paths<4>(a, pw, lds, s);
    else if (mode == 0) launch_paths<0>(a, pw, lds, s);
    else if (a.ckpt > 0) launch_paths<2>(a, pw, lds, s);
    else if (a.r1adj) launch_paths<6>(a, pw, lds, s);
    else launch_paths<5>(a, pw, lds, s);
}
static hipError_t launch_small(const WArgs& a, int mode, const LaunchGrid& G, hipStream_t s, const LaunchMarker& M) {
    M(KF_EXTEND, s);
    launch_small_paths(a, mode, s);
    if (mode == 0) {
        const int gb = blocks_for(a.n_chunk, G.other);
        if (a.out) M(KF_ACCUM, s);
        if (a.out && a.r1) hipLaunchKernelGGL(k_accum<true>, dim3(gb), dim3(BLOCK), 0, s, a);
        else if (a.out) hipLaunchKernelGGL(k_accum<false>, dim3(gb), dim3(BLOCK), 0, s, a);
        return hipGetLastError();
    }
    // (texture scatters: whole wavefronts once three per SIMD are filled.  Fewer, larger wavefronts issue fewer
    // atomics, and more of a pixel's samples meet: 196,608 paths, depth 6, 256 x 256 maps 400 -> 334 us, two texels of
    // them in view 2,230 -> 1,830; with fewer paths smaller wavefronts are the faster, 16,384 paths 161 us against 184,
    // unless the paths are short and little but scatters is left: depth 2, 94 -> 77 us, less than a texel in view 315 -> 122,
    // depth 3, 110 -> 107 and 404 -> 209, but depth 4, 125 -> 135, and 1,024 paths of depth 3, 106 -> 116)
    const bool scatters = a.lds_stage && a.max_depth <= 3 && a.n_chunk > SMALL_SCATTERS;
    const int full = a.lds_stage ? (a.n_chunk + SMALL_WAVES_WALK - 1) / SMALL_WAVES_WALK : 0;
    const int pw = small_per_wave(a, scatters ? WAVE / 2 : SMALL_LEAST_ADJ), aw = full <= pw ? pw : full < WAVE ? full : WAVE;
    const int per_block = aw * (BLOCK / WAVE);
    const int grid = (a.n_chunk + per_block - 1) / per_block;
    M(KF_REPLAY, s);
    if (a.r1adj) hipLaunchKernelGGL(k_adjoint_paths<true>, dim3(grid), dim3(BLOCK), grad_lds(a), s, a, aw);
    else hipLaunchKernelGGL(k_adjoint_paths<false>, dim3(grid), dim3(BLOCK), grad_lds(a), s, a, aw);
    return hipGetLastError();
}

// One chunk of paths through every bounce.  mode 0: render, 1: backward.  M is told the family
// of every kernel before its launch (event timing).
hipError_t launch_chunk(WArgs a, const PathState& S2, int mode, const LaunchGrid& G, hipStream_t s, const LaunchMarker& M) {
    // (with the light-stage features the fold and forward replay stay: the gradient of a normal-mapped smooth
    // dielectric runs through its s/p rotators, which amplify the rounding of the ray's direction, and
    // the reverse walk's differs from the replay's in the last bits: one texel moved by 5e-4)
    a.adj = mode == 1 && a.ckpt == 0 && !a.ext && !a.pprb && !a.tape && !a.prb ? 1 : 0;
    a.r1adj = a.adj && a.r1 ? 1 : 0;
    if (mode != 0) a.r1 = 0;  // (the rank-one record is the render's)
    size_t lds = (size_t)a.stack_cap * BLOCK * sizeof(int);
    if (a.small && (mode == 0 || a.adj)) return launch_small(a, mode, G, s, M);
    if (a.g0 > 0) {  // (the first chunk's counts were cleared with the call's other memory)
        M(KF_OTHER, s);
        hipLaunchKernelGGL(k_reset_counts, dim3(1), dim3(BLOCK), 0, s, a.S.counts);
    }
    const int gb = blocks_for(a.n_chunk, G.other), cg = blocks_for(a.n_chunk, 4 * G.cu);
    // (traversal's grid: enough workgroups for a queue of two rays a path, and for the most spread one)
    const int xg = blocks_for((int64_t)a.n_chunk * (a.stack_cap > SHALLOW_STACK ? WAVE / SPREAD_DEEP : 2),
                              a.stats ? G.extend_st : G.extend);
    a.qin = 0;
    a.first = 1;
    M(KF_EXTEND, s);
    if (a.small) {  // (the hybrid replay's forward pass)
        launch_small_paths(a, mode, s);
    } else {
        launch_extend<-2>(a, xg, lds, s);  // (camera rays generated in the launch)
    }
    for (int b = 1; b <= a.max_depth && !a.small; ++b) {
        a.qin = (b - 1) & 1;
        a.first = b == 1;
        // (cached backward: the second bounce's hits are the paths of two or more vertices, the
        // reverse walk's queue)
        a.keep_deep = a.adj && b == 2;
        int* const hqueue = a.S.hqueue;
        if (a.keep_deep) a.S.hqueue = a.S.dqueue;
        M(KF_COMPACT, s);
        hipLaunchKernelGGL(k_compact, dim3(cg), dim3(BLOCK), 0, s, a);
        M(KF_SHADE, s);
        // (a grid sized to each variant's own occupancy measured slower for the render variant)
        const int sg = blocks_for(a.n_chunk, G.shade);
        if (mode == 0 && a.r1) {
            hipLaunchKernelGGL((k_shade<4, false>), dim3(sg), dim3(BLOCK), 0, s, a);
        } else if (mode == 1 && a.tape) {
            hipLaunchKernelGGL((k_shade<3, false>), dim3(sg), dim3(BLOCK), 0, s, a);
        } else if (a.adj) {
            if (a.r1adj) hipLaunchKernelGGL((k_shade<6, false>), dim3(sg), dim3(BLOCK), 0, s, a);
            else hipLaunchKernelGGL((k_shade<5, false>), dim3(sg), dim3(BLOCK), 0, s, a);
        } else if (a.ext) {
            if (mode == 0) hipLaunchKernelGGL((k_shade<0, true>), dim3(sg), dim3(BLOCK), 0, s, a);
            else if (a.ckpt > 0) hipLaunchKernelGGL((k_shade<2, true>), dim3(sg), dim3(BLOCK), 0, s, a);
            else hipLaunchKernelGGL((k_shade<1, true>), dim3(sg), dim3(BLOCK), 0, s, a);
        } else {
            if (mode == 0) hipLaunchKernelGGL((k_shade<0, false>), dim3(sg), dim3(BLOCK), 0, s, a);
            else if (a.ckpt > 0) hipLaunchKernelGGL((k_shade<2, false>), dim3(sg), dim3(BLOCK), 0, s, a);
            else hipLaunchKernelGGL((k_shade<1, false>), dim3(sg), dim3(BLOCK), 0, s, a);
        }
        a.S.hqueue = hqueue;
        // the rays of bounce b + 1 and the shadow rays of bounce b in one traversal launch (a
        // vertex at the maximum depth starts neither, so nothing follows the last bounce)
        if (b < a.max_depth) {
            a.qin = b & 1;
            a.first = 0;
            M(KF_EXTEND, s);
            if (mode == 0 && a.r1) launch_extend<4>(a, xg, lds, s);
            else if (mode == 0) launch_extend<0>(a, xg, lds, s);
            else if (a.adj) launch_extend<5>(a, xg, lds, s);
            else if (a.tape) launch_extend<3>(a, xg, lds, s);
            else if (a.ckpt > 0) launch_extend<2>(a, xg, lds, s);
            else launch_extend<1>(a, xg, lds, s);
        }
    }
    if (mode == 0) {
        if (a.out) {
            M(KF_ACCUM, s);
            if (a.r1) hipLaunchKernelGGL(k_accum<true>, dim3(gb), dim3(BLOCK), 0, s, a);
            else hipLaunchKernelGGL(k_accum<false>, dim3(gb), dim3(BLOCK), 0, s, a);
        }
    } else {
        const size_t glds = grad_lds(a);
        if (a.adj) {
            // grids: as many workgroups per compute unit as this call's accumulator size and the
            // variant's registers allow
            if (a.max_depth > 1) {
                M(KF_FOLD, s);
                const void* fn = a.r1adj ? (const void*)k_adjoint_deep<true> : (const void*)k_adjoint_deep<false>;
                const int dg = resident_grid(fn, glds, a.n_chunk, G);
                if (a.r1adj) hipLaunchKernelGGL(k_adjoint_deep<true>, dim3(dg), dim3(BLOCK), glds, s, a);
                else hipLaunchKernelGGL(k_adjoint_deep<false>, dim3(dg), dim3(BLOCK), glds, s, a);
            }
            M(KF_REPLAY, s);
            const void* first = a.tiny_views ? (const void*)k_adjoint_first<true> : (const void*)k_adjoint_first<false>;
            const int fg = resident_grid(first, glds, a.n_chunk, G);
            if (a.tiny_views) hipLaunchKernelGGL(k_adjoint_first<true>, dim3(fg), dim3(BLOCK), glds, s, a);
            else hipLaunchKernelGGL(k_adjoint_first<false>, dim3(fg), dim3(BLOCK), glds, s, a);
            return hipGetLastError();
        }
        M(KF_FOLD, s);
        // each fold workgroup takes one contiguous slice of the chunk, so the grid is the resident
        // one (a second, partial round of workgroups would leave most of the GPU idle)
        const void* fold_fn = a.ckpt > 0 ? (a.ext ? (const void*)k_fold<true, true> : (const void*)k_fold<true, false>)
                              : a.tape ? (const void*)k_fold<false, false, false, true>
                              : a.pprb ? (const void*)k_fold<false, false, true> : (const void*)k_fold<false, false>;
        const int fg = resident_grid(fold_fn, 0, a.n_chunk, G);
        if (a.tape) hipLaunchKernelGGL((k_fold<false, false, false, true>), dim3(fg), dim3(BLOCK), 0, s, a);
        else if (a.ckpt > 0 && a.ext) hipLaunchKernelGGL((k_fold<true, true>), dim3(fg), dim3(BLOCK), 0, s, a);
        else if (a.ckpt > 0) hipLaunchKernelGGL((k_fold<true, false>), dim3(fg), dim3(BLOCK), 0, s, a);
        else if (a.pprb) hipLaunchKernelGGL((k_fold<false, false, true>), dim3(fg), dim3(BLOCK), 0, s, a);
        else hipLaunchKernelGGL((k_fold<false, false>), dim3(fg), dim3(BLOCK), 0, s, a);
        if (a.prb) {  // P-RB: independent suffix estimates, one sub-path pass per vertex index
            WArgs b2 = a;
            b2.S = S2;
            b2.stats = nullptr;
            b2.sig = nullptr;
            b2.mask = nullptr;
            b2.out = nullptr;
            for (int b1 = 1; b1 < a.max_depth; ++b1) {
                M(KF_OTHER, s);
                hipLaunchKernelGGL(k_reset_counts, dim3(1), dim3(BLOCK), 0, s, b2.S.counts);
                hipLaunchKernelGGL(k_prb_start, dim3(gb), dim3(BLOCK), 0, s, a, S2, b1);
                b2.seed = prb_seed_host(a.seed, (uint32_t)(b1 + 1));
                b2.qin = 0;
                b2.first = 1;
                M(KF_EXTEND, s);
                launch_extend<-1>(b2, xg, lds, s);
                for (int bb = b1 + 1; bb <= a.max_depth; ++bb) {
                    const int it = bb - b1;
                    b2.qin = (it - 1) & 1;
                    b2.first = it == 1;
                    M(KF_COMPACT, s);
                    hipLaunchKernelGGL(k_compact, dim3(cg), dim3(BLOCK), 0, s, b2);
                    M(KF_SHADE, s);
                    hipLaunchKernelGGL((k_shade<0, false>), dim3(blocks_for(a.n_chunk, G.shade)), dim3(BLOCK), 0, s, b2);
                    if (bb < a.max_depth) {
                        b2.qin = it & 1;
                        b2.first = 0;
                        M(KF_EXTEND, s);
                        launch_extend<0>(b2, xg, lds, s);
                    }
                }
                M(KF_OTHER, s);
                hipLaunchKernelGGL(k_prb_store, dim3(gb), dim3(BLOCK), 0, s, a, S2, b1);
            }
        }
        M(KF_REPLAY, s);
        // the persistent replay grid: as many workgroups per compute unit as this call's
        // accumulator size and the variant's registers allow
        if (a.tape) {  // the reverse sweep of the stored tape
            const int tg = resident_grid((const void*)k_tape_reverse, glds, a.n_chunk, G);
            hipLaunchKernelGGL(k_tape_reverse, dim3(tg), dim3(BLOCK), glds, s, a);
            return hipGetLastError();
        }
        const bool rule = a.ckpt > 0 && a.hyb_rule;
        const bool pprb = a.ckpt == 0 && a.pprb;
        const void* fn = a.ext ? (rule ? (const void*)k_replay<true, true, true>
                                       : pprb ? (const void*)k_replay<false, true, false, true>
                                       : a.ckpt > 0 ? (const void*)k_replay<true, true> : (const void*)k_replay<false, true>)
                               : (rule ? (const void*)k_replay<true, false, true>
                                       : pprb ? (const void*)k_replay<false, false, false, true>
                                       : a.ckpt > 0 ? (const void*)k_replay<true, false> : (const void*)k_replay<false, false>);
        const int rg = resident_grid(fn, glds, a.n_chunk, G);
        if (pprb) {
            if (a.ext) hipLaunchKernelGGL((k_replay<false, true, false, true>), dim3(rg), dim3(BLOCK), glds, s, a);
            else hipLaunchKernelGGL((k_replay<false, false, false, true>), dim3(rg), dim3(BLOCK), glds, s, a);
        } else if (a.ext) {
            if (rule) hipLaunchKernelGGL((k_replay<true, true, true>), dim3(rg), dim3(BLOCK), glds, s, a);
            else if (a.ckpt > 0) hipLaunchKernelGGL((k_replay<true, true>), dim3(rg), dim3(BLOCK), glds, s, a);
            else hipLaunchKernelGGL((k_replay<false, true>), dim3(rg), dim3(BLOCK), glds, s, a);
        } else {
            if (rule) hipLaunchKernelGGL((k_replay<true, false, true>), dim3(rg), dim3(BLOCK), glds, s, a);
            else if (a.ckpt > 0) hipLaunchKernelGGL((k_replay<true, false>), dim3(rg), dim3(BLOCK), glds, s, a);
            else hipLaunchKernelGGL((k_replay<false, false>), dim3(rg), dim3(BLOCK), glds, s, a);
        }
    }
    return hipGetLastError();
}

hipError_t occupancy_grid(int cu, int stack_cap, LaunchGrid* G) {
    int e = 0, sh = 0, ot = 0;
    size_t lds = (size_t)stack_cap * BLOCK * sizeof(int);
    hipError_t r;
    if ((r = hipOccupancyMaxActiveBlocksPerMultiprocessor(&e, k_extend<1, false>, BLOCK, lds)) != hipSuccess) return r;
    int es = 0;
    if ((r = hipOccupancyMaxActiveBlocksPerMultiprocessor(&es, k_extend<1, true>, BLOCK, lds)) != hipSuccess) return r;
    if ((r = hipOccupancyMaxActiveBlocksPerMultiprocessor(&sh, k_shade<1, false>, BLOCK, 0)) != hipSuccess) return r;
    if ((r = hipOccupancyMaxActiveBlocksPerMultiprocessor(&ot, k_accum<true>, BLOCK, 0)) != hipSuccess) return r;
    G->extend = (e > 0 ? e : 1) * cu;
    G->extend_st = (es > 0 ? es : 1) * cu;
    G->shade = (sh > 0 ? sh : 1) * cu;
    G->cu = cu;
    G->other = (ot > 0 ? ot : 1) * cu;
    return hipSuccess;
}

#endif  // PPT_EXT_TU
}  // namespace ppt
