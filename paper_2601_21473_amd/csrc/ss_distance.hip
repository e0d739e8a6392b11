// Distance kernels for gfx950: invocation distances of shared memory objects
// and the on-device distance estimators of Section 3.2.
//
// ss_object_distances (Appendix A, fine-grained distance assignment): an
// object referenced by several agents takes the smallest distance among them,
// and is needed now when any of them is active.  With v(a) = 0 for an active
// agent and D(a) otherwise, the object's distance is min over its referencing
// agents of v(a) and its activity is the OR of theirs, so one segmented
// min/or over the CSR map object -> agents computes both.
//
// The map is skewed (the root of a prefix tree is referenced by every agent,
// a leaf by one), so the work is split evenly over the merge of the two
// sorted lists "row ends" (obj_off[1..M]) and "reference indices" (0..R-1),
// the merge-path decomposition of Merrill and Garland (SC'16) for sparse
// products: every workgroup takes 2048 merge items, whatever the row lengths.
//   k_obj_prep  merge-path coordinates of every workgroup boundary (16 lanes
//               per boundary, 16 probes per round) and, in the same launch,
//               w[a] = 0 if a is active else D[a] + 1, one word per agent.
//   k_obj_min   per workgroup: coalesced staging of its row ends and of
//               w of its references into LDS (the gather of the agents'
//               words happens here, one load per reference; every thread
//               issues all its loads before using any), an 8-item walk
//               per thread, LDS atomics for rows split between threads,
//               coalesced stores of the rows that end in the block and one
//               carry record for the row that continues past it.
//   k_obj_fix   applies the carry records with global atomic min / stores,
//               after every k_obj_min block has written its rows.
// No dense contraction here; the kernel is bound by HBM bytes and by the rate
// of random gathers.
//
// ss_hop_distances (predefined activation paths): multi-source breadth-first
// hop counts over a CSR graph, level by level in one launch.
//   k_bfs       the workgroups own chunks of the vertices; a level sweeps each
//               chunk's hop counts for the vertices reached last, claims
//               their unvisited out-neighbours with compare-and-swap, and
//               counts its chunk done; nothing else passes between
//               workgroups, so no host round trip, queue or cache flush
//               separates levels.
//   k_queue     very large graphs: frontier queues, levels separated by a
//               grid barrier in a cooperative launch.
//
// ss_interaction_distances (interaction-involved simulations): D =
// min(D_action, floor(max(0, isqrt(d2) - radius) / velocity)) with d2 the
// squared distance to the nearest other agent on an integer tile grid.
//   k_pair      all pairs in one launch (few agents): per pair a packed 16-bit
//               subtract and a 16-bit dot product give dx^2 + dy^2 exactly.
//   k_near_*    many agents: sorted into cells, each looks only at the cells
//               about it (uniform on 2,048 x 2,048 tiles: 50,000 agents 205 us
//               by all pairs, 45 so; 200,000 3,280 and 54; gathered about 400
//               places on 8,192 x 8,192 tiles 200,000 take 81).
// Both are plain integer ALU work (no contraction), so no MFMA.
#include "scalesim.h"
#include "ss_internal.h"

#include <algorithm>
#include <mutex>

namespace ss {
namespace {

constexpr int kObjThreads = 256;
constexpr int kObjItems = 8;                          // merge items per thread
constexpr int kObjTile = kObjThreads * kObjItems;     // merge items per workgroup
constexpr unsigned kNone = 0xFFFFFFFFu;
constexpr unsigned kShared = kNone - 2;               // its agent word is also that of kNone - 1

struct ObjCarry {
    unsigned row;      // object, or kNone
    unsigned vmin;     // partial minimum of v over the block's references of row
    unsigned act;      // partial OR of activity
    unsigned pad;
};

struct ObjArgs {
    const unsigned* off;              // [M + 1]
    const unsigned* agents;           // [R]
    const unsigned* dist;             // [N]
    const unsigned char* active;      // [N]
    unsigned M, R, N;
    unsigned* out_dist;               // [M]
    unsigned char* out_act;           // [M]
    ObjCarry* carry;                  // [blocks]
    unsigned* coord;                  // [blocks + 1] rows consumed at each block boundary
    unsigned* w;                      // [N] 0 if active, else distance + 1; kNone for kNone
    unsigned* odd;                    // [odd_n] per workgroup that wrote w, a byte per wave: it met
    unsigned odd_n;                   // a distance of kNone - 1, whose w is that of kShared
};

// Merge-path coordinate (rows consumed) at diagonal d: the first p in
// [max(0, d - R), min(d, M)) whose row end comes after reference d - p - 1,
// i.e. off[p + 1] + p + 1 > d (strictly increasing in p), else the upper
// bound.  A group of 16 lanes searches one diagonal, 16 probes per round, so
// a wave serves four boundaries and a search takes a few dependent loads.
__device__ unsigned group_path_search(const unsigned* __restrict__ off, unsigned M, unsigned R,
                                      unsigned d, bool valid) {
    const unsigned lane = __lane_id(), g = lane >> 4, gl = lane & 15u;
    unsigned lo = d > R ? d - R : 0u;
    unsigned hi = d < M ? d : M;
    if (!valid) lo = hi = 0;
    for (;;) {
        const bool busy = lo < hi;
        if (__ballot(busy) == 0) break;
        const unsigned step = busy ? (hi - lo + 15u) / 16u : 1u;
        const unsigned p = lo + gl * step;
        bool after = false;
        if (busy && p < hi) after = (u64)min(off[p + 1], R) + p + 1 > d;
        const unsigned gm = (unsigned)(__ballot(after) >> (g * 16u)) & 0xFFFFu;
        if (busy) {
            if (gm == 0) {
                const unsigned n_probe = (hi - lo + step - 1) / step;   // lanes with p < hi
                lo = lo + (n_probe - 1) * step + 1;
            } else {
                const unsigned f = __ffs(gm) - 1;
                hi = lo + f * step;
                if (f > 0) lo = lo + (f - 1) * step + 1;
            }
        }
    }
    return lo;
}

// Two independent preparations in one launch.  Blocks [0, part_blocks): the
// merge-path coordinate of every workgroup boundary b * kObjTile,
// b = 0..blocks (16 per block).  The rest: w[a] = 0 if agent a is active,
// else D[a] + 1, so that k_obj_min gathers one 32-bit word per reference that
// carries both the distance and the activity.  That is a value too many: the
// two distances below 0xFFFFFFFF (which is common: never) share a word, and in
// the odd case that the larger one occurs, k_obj_min reads the distances of the
// agents with that word again.  (64-bit words need no such care, but
// the gathers miss the L1 more often and this kernel writes twice as much.  A
// call by those and so: 8 M agents and 56 M references 297 and 273 us, 2 M
// agents 63.9 and 60.6, 6,000 12.6 and 12.5, 300 10.5 and 10.5.)
__global__ void __launch_bounds__(256) k_obj_prep(ObjArgs A, unsigned n_bounds,
                                                  unsigned part_blocks) {
    if (blockIdx.x < part_blocks) {
        const unsigned b = (blockIdx.x * 256u + threadIdx.x) >> 4;
        const bool valid = b < n_bounds;
        const unsigned d = valid ? (unsigned)min((u64)b * kObjTile, (u64)A.M + A.R) : 0u;
        const unsigned x = group_path_search(A.off, A.M, A.R, d, valid);
        if (valid && (threadIdx.x & 15u) == 0) A.coord[b] = x;
        return;
    }
    // 2048 agents per block and round, eight per thread, loads before stores;
    // four at a time where the arrays allow it (this kernel on 6,000 agents: 3.5 us
    // with four only in whole rounds, 2.6 so)
    const unsigned blk = blockIdx.x - part_blocks;
    const u64 stride = (u64)(gridDim.x - part_blocks) * 2048u;
    bool odd = false;
    auto word = [&](unsigned d, bool act) {
        odd |= !act && d == kNone - 1;
        return act ? 0u : d == kNone ? kNone : min(d, kShared) + 1;
    };
    const bool wide = ((reinterpret_cast<uintptr_t>(A.dist) | reinterpret_cast<uintptr_t>(A.w)) & 15) == 0 &&
                      (reinterpret_cast<uintptr_t>(A.active) & 3) == 0;
    for (u64 base = (u64)blk * 2048u; base < A.N; base += stride) {      // workgroup-uniform
        if (wide) {
            const u64 n4 = A.N / 4;
            uint4 d[2];
            unsigned a[2];
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const u64 q = base / 4 + threadIdx.x + k * 256u;
                d[k] = make_uint4(0, 0, 0, 0);
                a[k] = 0;
                if (q < n4) {
                    d[k] = reinterpret_cast<const uint4*>(A.dist)[q];
                    a[k] = reinterpret_cast<const unsigned*>(A.active)[q];
                }
            }
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const u64 q = base / 4 + threadIdx.x + k * 256u;
                if (q < n4)
                    reinterpret_cast<uint4*>(A.w)[q] = make_uint4(
                        word(d[k].x, a[k] & 0xFFu), word(d[k].y, a[k] & 0xFF00u),
                        word(d[k].z, a[k] & 0xFF0000u), word(d[k].w, a[k] & 0xFF000000u));
            }
            const u64 rest = n4 * 4 + threadIdx.x;   // the last one to three agents
            if (base + 2048 > rest && rest < A.N) A.w[rest] = word(A.dist[rest], A.active[rest] != 0);
            continue;
        }
        unsigned dv[8];
        unsigned char ac[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const u64 a = base + threadIdx.x + k * 256u;
            dv[k] = 0;
            ac[k] = 0;
            if (a < A.N) {
                dv[k] = A.dist[a];
                ac[k] = A.active[a];
            }
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const u64 a = base + threadIdx.x + k * 256u;
            if (a < A.N) A.w[a] = word(dv[k], ac[k] != 0);
        }
    }
    const u64 any = __ballot(odd);                   // a byte per wave
    if (__lane_id() == 0)
        reinterpret_cast<unsigned char*>(A.odd + blk)[threadIdx.x >> 6] = any != 0;
}

// Persistent workgroups: the grid is a multiple of the eight XCDs, and
// workgroups are dispatched to the XCDs in turn (block b to XCD b % 8).  XCD x
// owns one contiguous range of tiles, which its workgroups walk side by side,
// so the objects of one subtree and the agent words they gather stay in that
// XCD's L2; a workgroup lives for many tiles, so the dispatcher is not the
// limit.
__global__ void __launch_bounds__(kObjThreads) k_obj_min(ObjArgs A, unsigned n_tiles) {
    // s_item[0, nrow) = row ends (absolute), s_item[nrow, nrow + nref) = v of
    // the block's references; nrow + nref = the block's merge items.  s_flag
    // has the same split: activity of the rows ending in the block (output),
    // then activity of the references.
    __shared__ unsigned s_item[kObjTile];
    __shared__ unsigned s_outd[kObjTile];     // rows ending in the block: min
    __shared__ unsigned char s_flag[kObjTile];
    __shared__ unsigned s_bmin, s_bact;
    __shared__ unsigned s_odd[kObjThreads / 64];
    static_assert(kObjThreads == 256, "four waves");

    constexpr unsigned kXcds = 8;
    const unsigned tid = threadIdx.x;
    const unsigned total = A.M + A.R;
    // any flag set: see k_obj_prep.  The workgroup's waves read a part each, used
    // only once the first tile is staged, so that the reads cost no round trip.
    unsigned flags = tid < A.odd_n ? A.odd[tid] : 0u;
    for (unsigned k = tid + kObjThreads; k < A.odd_n; k += kObjThreads) flags |= A.odd[k];
    const unsigned xcd = blockIdx.x % kXcds, per_xcd = gridDim.x / kXcds;
    const unsigned q = n_tiles / kXcds, rem = n_tiles % kXcds;
    const unsigned t_lo = xcd < rem ? xcd * (q + 1) : rem * (q + 1) + (xcd - rem) * q;
    const unsigned t_hi = t_lo + (xcd < rem ? q + 1 : q);
    for (unsigned tile = t_lo + blockIdx.x / kXcds; tile < t_hi; tile += per_xcd) {
        const unsigned d0 = tile * (unsigned)kObjTile;
        const unsigned d1 = min(d0 + (unsigned)kObjTile, total);
        const unsigned o0 = A.coord[tile], o1 = A.coord[tile + 1];
        const unsigned r0 = d0 - o0, r1 = d1 - o1;
        const unsigned nrow = o1 - o0, nref = r1 - r0;
        if (tid == 0) {
            s_bmin = kNone;
            s_bact = 0;
        }

        // Staging: every thread owns items i = tid + k * kObjThreads of the
        // block's merge range; all loads of a kind are issued before any is used.
        unsigned val[kObjItems];
    #pragma unroll
        for (int k = 0; k < kObjItems; ++k) {
            const unsigned i = tid + k * kObjThreads;
            val[k] = kNone;
            if (i < nrow) val[k] = min(A.off[o0 + 1 + i], A.R);
            else if (i < nrow + nref) val[k] = A.agents[r0 + (i - nrow)];
        }
        // one word per reference: e = 0 if the agent is active, else D + 1
        unsigned char act[kObjItems];
    #pragma unroll
        for (int k = 0; k < kObjItems; ++k) {
            const unsigned i = tid + k * kObjThreads;
            act[k] = 0;
            if (i >= nrow && i < nrow + nref) {
                const unsigned a = val[k];
                val[k] = kNone;
                if (a < A.N) {
                    const unsigned e = A.w[a];
                    act[k] = e == 0;
                    val[k] = e != kNone ? max(e, 1u) - 1 : kNone;
                }
            }
        }
    #pragma unroll
        for (int k = 0; k < kObjItems; ++k) {
            const unsigned i = tid + k * kObjThreads;
            if (i < nrow + nref) s_item[i] = val[k];
            if (i >= nrow && i < nrow + nref) s_flag[i] = act[k];
        }
        const u64 any = __ballot(flags != 0);
        if (__lane_id() == 0) s_odd[tid >> 6] = any != 0;
        __syncthreads();
        if (s_odd[0] | s_odd[1] | s_odd[2] | s_odd[3]) {          // workgroup-uniform
            // kShared may stand for kNone - 1: such agents' distances themselves
#pragma unroll 1
            for (unsigned i = tid; i < nrow + nref; i += kObjThreads) {
                if (i < nrow || s_item[i] != kShared) continue;
                const unsigned a = A.agents[r0 + (i - nrow)];
                if (a < A.N) s_item[i] = A.dist[a];
            }
            __syncthreads();
        }

        // this thread's start on the block's merge path (binary search in LDS)
        const unsigned k0 = tid * (unsigned)kObjItems;
        const unsigned n_items = d1 - d0;
        const unsigned* s_val = s_item + nrow;
        const unsigned char* s_act = s_flag + nrow;
        unsigned char* s_outa = s_flag;
        unsigned o = 0, r = 0, vmin = kNone, vact = 0;
        if (k0 < n_items) {
            unsigned lo = k0 > nref ? k0 - nref : 0u, hi = min(k0, nrow);
            while (lo < hi) {
                const unsigned mid = (lo + hi) >> 1;
                if (s_item[mid] + mid + 1 > r0 + k0) hi = mid;
                else lo = mid + 1;
            }
            o = lo;
            r = k0 - lo;
            const unsigned k1 = min(k0 + (unsigned)kObjItems, n_items);
            for (unsigned k = k0; k < k1; ++k) {
                if (o < nrow && (s_item[o] <= r0 + r || r >= nref)) {     // row o ends here
                    s_outd[o] = vmin;
                    s_outa[o] = (unsigned char)vact;
                    vmin = kNone;
                    vact = 0;
                    ++o;
                } else if (r < nref) {
                    vmin = min(vmin, s_val[r]);
                    vact |= s_act[r];
                    ++r;
                }
            }
        }
        __syncthreads();
        // references of a row that ends in a later thread (or block)
        if (k0 < n_items && (vmin != kNone || vact)) {
            if (o < nrow) {
                atomicMin(&s_outd[o], vmin);
                if (vact) s_outa[o] = 1;
            } else {
                atomicMin(&s_bmin, vmin);
                if (vact) s_bact = 1;
            }
        }
        __syncthreads();
        for (unsigned i = tid; i < nrow; i += kObjThreads) {
            A.out_dist[o0 + i] = s_outd[i];
            A.out_act[o0 + i] = s_outa[i];
        }
        if (tid == 0) {
            ObjCarry c{kNone, kNone, 0u, 0u};
            if (o1 < A.M && (s_bmin != kNone || s_bact)) c = ObjCarry{o1, s_bmin, s_bact, 0u};
            A.carry[tile] = c;
        }
        __syncthreads();          // LDS is refilled by the next tile
    }
}

__global__ void __launch_bounds__(256) k_obj_fix(const ObjCarry* __restrict__ carry,
                                                unsigned n, unsigned M, unsigned* out_dist,
                                                unsigned char* out_act) {
    const unsigned i = blockIdx.x * 256u + threadIdx.x;
    if (i >= n) return;
    const ObjCarry c = carry[i];
    if (c.row >= M) return;
    atomicMin(&out_dist[c.row], c.vmin);
    if (c.act) out_act[c.row] = 1;
}

// ---------------------------------------------------------------------------
// Hop counts
// ---------------------------------------------------------------------------

constexpr int kBfsThreads = 1024;
constexpr int kBfsEdges = 8;                 // edges claimed per vertex per round
constexpr int kBfsVerts = 2;                 // frontier vertices per lane per round
constexpr unsigned kBfsBatch = 8;            // vertices per lane that a sweep reads at once
// Bound of a wait of both searches, in polls of about a microsecond: what the
// longest level takes grows with the graph (one lane takes 0.45 us an edge of a
// vertex with very many), so the bound does too.
constexpr u64 kHopPolls = 1u << 24;
inline u64 hop_polls(u64 base, unsigned V, unsigned E) { return base + V + 2 * (u64)E; }

struct BfsArgs {
    const unsigned* row_off;                 // [V + 1]
    const unsigned* col;                     // [E]
    const unsigned* src;                     // [n_src]
    unsigned V, E, n_src, max_hops;
    unsigned* hops;                          // [V]
    unsigned* ctl;                           // [kCtlWords] see kCtl*
    u64* hint;                               // [V / 64 + 1] visited vertices, or null
    unsigned chunks;                         // chunks per level, of every chunks-th 64 vertices
    u64 polls;                               // bound of a wait
};
constexpr int kCtlTicket = 4;                // chunks given out
constexpr int kCtlError = 5;                 // 1 if a wait hit its bound
constexpr int kCtlDone = 8;                  // [kBfsSlots x 2 words] by level: chunks done (low
                                             // word), those that reached new vertices (high)
constexpr unsigned kBfsSlots = 8;
constexpr unsigned kCtlWords = kCtlDone + 2 * kBfsSlots;

// Every vertex unvisited, control words zero.
__global__ void __launch_bounds__(kBfsThreads) k_bfs_init(BfsArgs A) {
    const unsigned v = blockIdx.x * kBfsThreads + threadIdx.x;
    if (v < A.V) A.hops[v] = kNone;
    if (A.hint && v <= A.V / 64) A.hint[v] = 0;
    if (blockIdx.x == 0 && threadIdx.x < kCtlWords) A.ctl[threadIdx.x] = 0;
}

// Chunk c of the vertices at hop `level`: their unvisited out-neighbours get
// hop level + 1.  Returns whether this lane reached any.  A chunk is every
// chunks-th stretch of 64 vertices, a wave's width: callers number vertices so
// that neighbours are near each other, and a level that lies in one corner of
// the numbers is then every workgroup's work (by chunks of consecutive vertices
// and so: communities of 16,384 vertices of degree 16 among 4 M, 257 levels,
// 55.4 and 5.2 ms; of 1,024 among 50,000 0.66 and 0.62; a mesh of 2,048 x 2,048
// 62.7 and 56.1; one of 1,000 x 1,000, whose rows a chunk then shares with
// none of their neighbours, 20.3 and 22.5; random graphs the same).
__device__ __forceinline__ bool bfs_chunk(const BfsArgs& A, unsigned c, unsigned level,
                                          unsigned* list) {
    const unsigned lane = __lane_id(), w = threadIdx.x >> 6;
    constexpr unsigned kWaves = kBfsThreads / 64;
    bool found = false;
    const u64 stride = (u64)A.chunks * kWaves * 64;          // from a wave's stretch to its next
    for (u64 b = ((u64)w * A.chunks + c) * 64u; b < A.V; b += stride * kBfsBatch) {
        // a sweep of kBfsBatch x 64 vertices; those at this level go to the
        // wave's list
        unsigned h[kBfsBatch];
#pragma unroll
        for (unsigned k = 0; k < kBfsBatch; ++k) {
            const u64 v = b + k * stride + lane;
            h[k] = kNone;
            if (v < A.V)
                h[k] = __hip_atomic_load(&A.hops[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        unsigned n = 0;
#pragma unroll
        for (unsigned k = 0; k < kBfsBatch; ++k) {
            const u64 v0 = b + k * stride;
            const u64 m = __ballot(h[k] == level);
            if (A.hint && m && lane == 0)
                __hip_atomic_fetch_or(&A.hint[v0 / 64], m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (h[k] == level)
                list[n + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u))] =
                    (unsigned)v0 + lane;
            n += (unsigned)__popcll(m);
        }
        __builtin_amdgcn_wave_barrier();
        for (unsigned i0 = 0; i0 < n; i0 += 64 * kBfsVerts) {
            unsigned e[kBfsVerts], e1[kBfsVerts];
#pragma unroll
            for (int f = 0; f < kBfsVerts; ++f) {
                const unsigned i = i0 + f * 64u + lane;
                e[f] = e1[f] = 0;
                if (i < n) {
                    const unsigned v = list[i];
                    e[f] = min(A.row_off[v], A.E);
                    e1[f] = min(A.row_off[v + 1], A.E);
                }
            }
            bool more = false;
#pragma unroll
            for (int f = 0; f < kBfsVerts; ++f) more |= e[f] < e1[f];
            while (__ballot(more)) {
                unsigned v[kBfsVerts * kBfsEdges];
                bool claim[kBfsVerts * kBfsEdges];
#pragma unroll
                for (int f = 0; f < kBfsVerts; ++f)
#pragma unroll
                    for (int k = 0; k < kBfsEdges; ++k)
                        v[f * kBfsEdges + k] = e[f] + k < e1[f] ? A.col[e[f] + k] : kNone;
#pragma unroll
                for (int k = 0; k < kBfsVerts * kBfsEdges; ++k) claim[k] = v[k] < A.V;
                if (A.hint) {
                    u64 g[kBfsVerts * kBfsEdges];
#pragma unroll
                    for (int k = 0; k < kBfsVerts * kBfsEdges; ++k)
                        g[k] = claim[k] ? A.hint[v[k] / 64] : 0;
#pragma unroll
                    for (int k = 0; k < kBfsVerts * kBfsEdges; ++k)
                        claim[k] = claim[k] && !((g[k] >> (v[k] & 63)) & 1);
                }
#pragma unroll
                for (int k = 0; k < kBfsVerts * kBfsEdges; ++k)
                    if (claim[k]) found |= atomicCAS(&A.hops[v[k]], kNone, level + 1) == kNone;
                more = false;
#pragma unroll
                for (int f = 0; f < kBfsVerts; ++f) {
                    e[f] += kBfsEdges;
                    more |= e[f] < e1[f];
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    return found;
}

// The levels, in one launch.  Level 0 places the sources (hop 0); level k + 1
// expands the vertices at hop k.  The vertices are cut into chunks, each owned
// by the workgroup that drew its ticket; a level may run once all chunks of the
// level before it are done, which every workgroup reads off that level's
// counter itself.  Workgroups that wait long for the first level draw the
// tickets that are left, so the search ends whatever part of the grid is
// resident, and an ordinary launch does (a cooperative one costs about 20 us
// more).  What one workgroup learns of another are the hop counts, which are
// claimed and read by agent-scope atomics alone, and each claim is complete
// before its chunk counts as done, so no cache is written back or invalidated
// between levels.  (The hint may be out of date: a vertex that it misses fails
// its claim.)  A level is a chain of five round trips to memory: counter,
// hops, row, columns, claims.
constexpr unsigned kBfsMost = 512;                   // most chunks
constexpr unsigned kBfsPatience = 64;                // polls before another ticket is drawn

__global__ void __launch_bounds__(kBfsThreads) k_bfs(BfsArgs A) {
    __shared__ unsigned s_list[kBfsThreads / 64][64 * kBfsBatch];
    __shared__ unsigned s_own[kBfsMost], s_n, s_state;
    __shared__ int s_found[2];
    u64* done = reinterpret_cast<u64*>(A.ctl + kCtlDone);
    auto draw = [&]() {                              // thread 0: another chunk, if one is left
        const unsigned t = __hip_atomic_fetch_add(&A.ctl[kCtlTicket], 1u, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
        const bool mine = t < A.chunks && s_n < kBfsMost;
        if (mine) s_own[s_n++] = t;
        return mine;
    };
    if (threadIdx.x == 0) {
        s_n = 0;
        s_found[0] = s_found[1] = 0;
        draw();
    }
    __syncthreads();
    unsigned from = 0;                               // owned chunks done at this level
    for (unsigned level = 0; s_n;) {                 // workgroup-uniform
        bool found = false;
        const unsigned own = s_n;
        for (unsigned q = from; q < own; ++q) {
            const unsigned c = s_own[q];
            if (level == 0) {
                for (u64 i = (u64)c * kBfsThreads + threadIdx.x; i < A.n_src;
                     i += (u64)A.chunks * kBfsThreads) {
                    const unsigned v = A.src[i];
                    if (v >= A.V) continue;
                    __hip_atomic_exchange(&A.hops[v], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    found = true;
                }
            } else {
                found |= bfs_chunk(A, c, level - 1, s_list[threadIdx.x >> 6]);
            }
        }
        if (__ballot(found) && __lane_id() == 0) s_found[level & 1] = 1;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // every claim is complete
        __syncthreads();
        if (threadIdx.x == 0) {
            const bool any = s_found[level & 1];
            s_found[~level & 1] = 0;
            u64* slot = &done[level % kBfsSlots];
            unsigned state = 0;                      // 0: more chunks of this level, 1: next level,
                                                     // 2: the search is over
            u64 v;
            if (A.chunks == 1) {
                v = 1ull | ((u64)any << 32);
            } else {
                v = __hip_atomic_fetch_add(slot, (u64)(own - from) | ((u64)any << 32),
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) +
                    ((u64)(own - from) | ((u64)any << 32));
                // the slot of four levels on was last read four levels ago
                if (s_own[0] == 0 && from == 0)
                    __hip_atomic_store(&done[(level + kBfsSlots / 2) % kBfsSlots], 0ull,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                for (u64 spin = 0; (unsigned)v < A.chunks; ++spin) {
                    if (level == 0 && spin % kBfsPatience == kBfsPatience - 1 && draw()) break;
                    if (spin > A.polls) {
                        __hip_atomic_store(&A.ctl[kCtlError], 1u, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                        state = 2;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(4);             // fewer polls in the counter's way
                    v = __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            if ((unsigned)v >= A.chunks) state = (v >> 32) && level < A.max_hops ? 1 : 2;
            s_state = state;
            if (A.hint) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
        if (s_state == 2) return;
        if (s_state == 1) {
            ++level;
            from = 0;
        } else {
            from = own;
        }
    }
}

// Graphs of more than kBfsSweep vertices: frontier queues instead of sweeps over
// all vertices, whose cost per level grows with them.  By queues / by sweeps, a
// level that reaches one vertex: 4.2 M vertices 11.5 / 9.7 us, 6 M 12.1 / 14.8, 8 M
// 11.4 / 18.1, 16 M 15.3 / 31.0.  A shallow search gains by sweeps at any size
// (random graphs of degree 8, 5 to 11 levels: 4.2 M 1,226 / 778 us, 8 M 2,082 /
// 1,542, 16 M 3,833 / 3,105), but how deep a graph is shows only in the search,
// and a deep one loses the more the larger it is.
constexpr unsigned kBfsSweep = 1u << 22;
constexpr int kQueueThreads = 256;
constexpr int kQueueEdges = 8;               // edges claimed per vertex per round
constexpr int kQueueVerts = 2;               // frontier vertices per thread per round

struct QueueArgs {
    const unsigned* row_off;                 // [V + 1]
    const unsigned* col;                     // [E]
    const unsigned* src;                     // [n_src]
    unsigned V, E, n_src, max_hops;
    unsigned* hops;                          // [V]
    uint2* q0;                               // [V] frontier queues: edge ranges
    uint2* q1;
    unsigned* ctl;                           // [8] see kCtl*
    u64 polls;                               // bound of a wait
};
constexpr int kQueueCnt = 0;                   // [0..2] queue lengths, rotating
constexpr int kQueueBarCount = 3;              // grid barrier arrivals
constexpr int kQueueBarGen = 4;                // grid barrier generation
constexpr int kQueueError = 5;                 // 1 if a barrier wait hit its bound
constexpr int kQueueLevels = 6;                // levels expanded

// Grid-wide barrier for a cooperative launch (all workgroups resident).
// Thread 0 of each workgroup publishes the workgroup's writes with one
// agent-scope release fence and arrives on a counter; the last arrival bumps
// the generation word.  Waiters poll the generation with relaxed loads (an
// acquire per poll would invalidate the XCD's L2 each time) and take one
// acquire fence when it changes.  Returns false for every thread of a
// workgroup whose wait exceeded the bound; the caller then leaves the kernel,
// so every wave exits.
__device__ bool grid_barrier(unsigned* ctl, u64 polls) {
    __shared__ int s_ok;
    __syncthreads();
    if (threadIdx.x == 0) {
        int ok = 1;
        const unsigned gen = __hip_atomic_load(&ctl[kQueueBarGen], __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        const unsigned arrived = __hip_atomic_fetch_add(&ctl[kQueueBarCount], 1u, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT) + 1;
        if (arrived == gridDim.x) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
            __hip_atomic_store(&ctl[kQueueBarCount], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_fetch_add(&ctl[kQueueBarGen], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            u64 spin = 0;
            while (__hip_atomic_load(&ctl[kQueueBarGen], __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT) == gen) {
                if (++spin > polls) {
                    ok = 0;
                    __hip_atomic_store(&ctl[kQueueError], 1u, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
                __builtin_amdgcn_s_sleep(2);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        s_ok = ok;
    }
    __syncthreads();
    return s_ok != 0;
}

// Append the lanes' claimed vertices (claim[k] for k < n) to queue q as their
// edge ranges [row_off[v], row_off[v + 1]), with one counter atomic per wave;
// the range loads and the counter atomic are in flight together.  Entries at
// or beyond `cap` are dropped (a vertex is claimed once, so a queue never
// holds more than the vertex count).  Called by every lane of the wave.
template <int n>
__device__ __forceinline__ void wave_append(const bool (&claim)[n], const unsigned (&v)[n],
                                            const QueueArgs& A, uint2* q, unsigned* cnt) {
    u64 m[n];
    unsigned total = 0;
#pragma unroll
    for (int k = 0; k < n; ++k) {
        m[k] = __ballot(claim[k]);
        total += __popcll(m[k]);
    }
    if (total == 0) return;
    uint2 r[n];
#pragma unroll
    for (int k = 0; k < n; ++k) {
        r[k] = make_uint2(0u, 0u);
        if (claim[k]) r[k] = make_uint2(min(A.row_off[v[k]], A.E), min(A.row_off[v[k] + 1], A.E));
    }
    unsigned base = 0;
    if (__lane_id() == 0)
        base = __hip_atomic_fetch_add(cnt, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    base = __shfl(base, 0);
#pragma unroll
    for (int k = 0; k < n; ++k) {
        const unsigned below = __builtin_amdgcn_mbcnt_hi((unsigned)(m[k] >> 32),
                                                         __builtin_amdgcn_mbcnt_lo((unsigned)m[k], 0u));
        if (claim[k] && base + below < A.V) q[base + below] = r[k];
        base += __popcll(m[k]);
    }
}

// Every vertex unvisited, counters and barrier words zero.
__global__ void __launch_bounds__(kQueueThreads) k_queue_init(QueueArgs A) {
    const unsigned v = blockIdx.x * kQueueThreads + threadIdx.x;
    if (v < A.V) A.hops[v] = kNone;
    if (blockIdx.x == 0 && threadIdx.x < 8) A.ctl[threadIdx.x] = 0;
}

// Sources: hop 0, each vertex once, into the first queue.
__global__ void __launch_bounds__(kQueueThreads) k_queue_src(QueueArgs A) {
    const unsigned i = blockIdx.x * kQueueThreads + threadIdx.x;
    bool claim[1] = {false};
    unsigned v[1] = {kNone};
    if (i < A.n_src) {
        v[0] = A.src[i];
        if (v[0] < A.V) claim[0] = atomicCAS(&A.hops[v[0]], kNone, 0u) == kNone;
    }
    wave_append(claim, v, A, A.q0, &A.ctl[kQueueCnt + 0]);
}

// The levels, in one cooperative launch.
__global__ void __launch_bounds__(kQueueThreads) k_queue(QueueArgs A) {
    const unsigned lane = __lane_id();
    const unsigned gsz = gridDim.x * kQueueThreads;
    const unsigned wbase = blockIdx.x * kQueueThreads + (threadIdx.x & ~63u);   // wave's first thread
    for (unsigned level = 0;; ++level) {
        // ordered by the kernel start or the barrier's acquire fence; capped
        // at the queue length
        const unsigned n = min(__hip_atomic_load(&A.ctl[kQueueCnt + level % 3], __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT), A.V);
        if (n == 0 || level >= A.max_hops) break;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            __hip_atomic_store(&A.ctl[kQueueCnt + (level + 2) % 3], 0u, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&A.ctl[kQueueLevels], level + 1, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
        const uint2* cur = (level & 1) ? A.q1 : A.q0;
        uint2* nxt = (level & 1) ? A.q0 : A.q1;
        unsigned* cnt = &A.ctl[kQueueCnt + (level + 1) % 3];
        // Large frontiers first read a vertex's state and try to claim it only
        // while unvisited (fewer atomics); small ones go straight to the
        // compare-and-swap (one dependent access less per level).
        const bool precheck = n > 32768u;
        // each lane expands kQueueVerts frontier vertices per round, eight of
        // their edges at a time, so that many independent loads are in flight
        for (unsigned b0 = wbase * kQueueVerts; b0 < n; b0 += gsz * kQueueVerts) {
            unsigned e[kQueueVerts], e1[kQueueVerts];
#pragma unroll
            for (int f = 0; f < kQueueVerts; ++f) {
                const unsigned i = b0 + f * 64u + lane;
                const uint2 r = i < n ? cur[i] : make_uint2(0u, 0u);
                e[f] = r.x;
                e1[f] = min(r.y, A.E);
            }
            bool more = false;
#pragma unroll
            for (int f = 0; f < kQueueVerts; ++f) more |= e[f] < e1[f];
            while (__ballot(more)) {
                unsigned v[kQueueVerts * kQueueEdges];
                bool claim[kQueueVerts * kQueueEdges];
#pragma unroll
                for (int f = 0; f < kQueueVerts; ++f)
#pragma unroll
                    for (int k = 0; k < kQueueEdges; ++k)
                        v[f * kQueueEdges + k] = e[f] + k < e1[f] ? A.col[e[f] + k] : kNone;
#pragma unroll
                for (int k = 0; k < kQueueVerts * kQueueEdges; ++k)
                    claim[k] = v[k] < A.V && (!precheck || A.hops[v[k]] == kNone);
#pragma unroll
                for (int k = 0; k < kQueueVerts * kQueueEdges; ++k)
                    if (claim[k]) claim[k] = atomicCAS(&A.hops[v[k]], kNone, level + 1) == kNone;
                wave_append(claim, v, A, nxt, cnt);
                more = false;
#pragma unroll
                for (int f = 0; f < kQueueVerts; ++f) {
                    e[f] += kQueueEdges;
                    more |= e[f] < e1[f];
                }
            }
        }
        if (!grid_barrier(A.ctl, A.polls)) return;
    }
}

// ---------------------------------------------------------------------------
// Interaction distances
// ---------------------------------------------------------------------------

typedef short short2_t __attribute__((ext_vector_type(2)));

// Squared distance of two grid points held as packed 16-bit (x, y): one packed
// subtract and one 16-bit dot product (coordinates below 2^15, so neither the
// differences nor the sum of squares overflow).  The dot product is written
// in its three-operand form with a zero addend; the compiler's two-operand
// form would need a register cleared before every pair.
__device__ __forceinline__ unsigned dist2(unsigned a, unsigned b) {
    const short2_t d = __builtin_bit_cast(short2_t, a) - __builtin_bit_cast(short2_t, b);
    int r;
    asm("v_dot2_i32_i16 %0, %1, %1, 0" : "=v"(r) : "v"(d));
    return (unsigned)r;
}

// A position as packed 16-bit (x, y), each in [0, 2^15) whatever the caller
// passed (so that every index derived from it stays in its array).
__device__ __forceinline__ unsigned pack_pos(int x, int y) {
    return ((unsigned)x & 0x7FFFu) | (((unsigned)y & 0x7FFFu) << 16);
}

// Agent j's position, by one read; callers' arrays are only 4-byte aligned.
__device__ __forceinline__ int2 position(const int* __restrict__ pos, u64 j) {
    int q[2];
    __builtin_memcpy(q, pos + 2 * j, sizeof q);
    return make_int2(q[0], q[1]);
}

__device__ __forceinline__ unsigned isqrt_u32(unsigned x) {
    unsigned r = (unsigned)sqrt((double)x);
    while ((u64)r * r > x) --r;
    while ((u64)(r + 1) * (r + 1) <= x) ++r;
    return r;
}

// The result of an agent whose nearest other agent is at squared distance m
// (kNone: there is none) and whose current action ends in d steps.
__device__ __forceinline__ unsigned interaction_of(unsigned m, unsigned d, unsigned velocity,
                                                   unsigned radius) {
    if (m == kNone) return d;
    const unsigned dist = isqrt_u32(m);
    return min(d, (dist > radius ? dist - radius : 0u) / velocity);
}

// All pairs in one launch: a workgroup takes kOwn agents (one per lane, 64 /
// kOwn lanes for each of them), its kPairWaves waves take the others in turn,
// 64 at a time staged through the wave's own LDS as packed positions, of which
// an agent's lanes take equal parts, and the minima meet in LDS.  Bound by the
// vector ALU (2.5 instructions a pair), so by how evenly the workgroups cover
// the 256 CUs: see pair_launch.
constexpr int kPairWaves = 16;

struct PairArgs {
    const int* pos;                   // [n][2]
    const unsigned* d_action;         // [n] (may be `out`)
    unsigned* out;                    // [n]
    unsigned n, velocity, radius;
};

template <unsigned kOwn>
__global__ void __launch_bounds__(64 * kPairWaves) k_pair(PairArgs A) {
    constexpr unsigned kParts = 64 / kOwn, kPart = 64 / kParts;   // others per lane and group
    __shared__ uint4 s_pos[kPairWaves][2][16];
    __shared__ unsigned s_best[kPairWaves][64];
    const unsigned l = threadIdx.x & 63u, part = l / kOwn;
    const unsigned w = (unsigned)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const unsigned i = blockIdx.x * kOwn + l % kOwn;
    // past the end the last agent of all, whose repeats change no minimum
    auto load = [&](unsigned j) { return position(A.pos, min(j, A.n - 1)); };
    const int2 own = load(i);
    const unsigned pi = pack_pos(own.x, own.y), groups = (A.n + 63) / 64u;
    unsigned best = kNone;
    int2 q = load(w * 64u + l);
    for (unsigned g = w, buf = 0; g < groups; g += kPairWaves, buf ^= 1) {
        // the wave's LDS writes and reads are in order, and the other buffer
        // takes the next group, so no barrier is needed
        reinterpret_cast<unsigned*>(s_pos[w][buf])[l] = pack_pos(q.x, q.y);
        __builtin_amdgcn_wave_barrier();
        q = load((g + kPairWaves) * 64u + l);        // in flight meanwhile
        if (g == blockIdx.x * kOwn / 64u || g * 64u + 64u > A.n) {
            // its own agents (without the agent itself), or a partial group
            for (unsigned k = part * kPart; k < part * kPart + kPart; ++k)
                if (g * 64u + k != i && g * 64u + k < A.n)
                    best = min(best, dist2(pi, reinterpret_cast<unsigned*>(s_pos[w][buf])[k]));
            continue;
        }
        // four positions per 16-byte LDS read (an agent's lanes read the same
        // few addresses), so a read serves ten vector instructions
#pragma unroll
        for (unsigned k = 0; k < kPart / 4; ++k) {
            const uint4 v = s_pos[w][buf][part * (kPart / 4) + k];
            best = min(best, dist2(pi, v.x));
            best = min(best, dist2(pi, v.y));
            best = min(best, dist2(pi, v.z));
            best = min(best, dist2(pi, v.w));
        }
    }
    s_best[w][l] = best;
    __syncthreads();
    if (w == 0) {
#pragma unroll
        for (int k = 1; k < kPairWaves; ++k) best = min(best, s_best[k][l]);
#pragma unroll
        for (unsigned o = kOwn; o < 64; o <<= 1) best = min(best, (unsigned)__shfl_xor((int)best, o));
        if (l < kOwn && i < A.n)
            A.out[i] = interaction_of(best, A.d_action[i], A.velocity, A.radius);
    }
}

// Nearest neighbour by cells, in two levels so that neither a crowd in a
// corner of the grid nor empty land slows it: a fixed grid of 64 x 64 blocks of
// 512 x 512 tiles, and in each block a grid of its own of about as many cells
// as the block has agents, cells four times as tall as wide.  The agents are
// sorted block by block, row of cells by row of cells, so any stretch of a row
// is one contiguous run of sorted agents.
//   k_near_blocks  agents per block, one row of counts per workgroup; clears
//                  the cells' counts
//   k_near_cells   each block's agents, its cells and where they begin
//   k_near_count   cell of every agent, and its rank in it.  Agents that meet
//                  another of their workgroup on their very tile are done
//                  (distance 0), and one of them stands for all, so a crowd on
//                  one tile makes no long run.
//   k_near_sum     agents of every stretch of kNearScan cells (many agents)
//   k_near_scan    first sorted place of every cell
//   k_near_place   agents into their places
//   k_near_find    the search, one agent per lane in sorted order, and the
//                  result
// Whatever the workspace holds (two calls that share one, against the rules),
// every index stays inside its array.
constexpr unsigned kNearThreads = 256;
constexpr unsigned kNearSide = 64;                    // blocks per side
constexpr unsigned kNearBlocks = kNearSide * kNearSide;
constexpr unsigned kNearShift = 9;                    // tiles per block side, log2
constexpr unsigned kNearTiles = 1u << kNearShift;
constexpr unsigned kNearRows = 128;                   // most workgroups of k_near_blocks
constexpr unsigned kNearScan = 4096;                  // cells per workgroup of k_near_scan
constexpr unsigned kNearSums = 1u << 17;              // agents beyond which k_near_sum runs
constexpr unsigned kNearShared = 1u << 31;            // the agent shares its tile
constexpr unsigned kNearFew = 64;                     // agents that a lane simply looks at

struct NearArgs {
    const int* pos;                   // [n][2]
    const unsigned* d_action;         // [n] (may be `out`)
    unsigned* out;                    // [n]
    unsigned n, velocity, radius;
    unsigned cells;                   // n, up to a multiple of kNearScan
    unsigned rows;                    // workgroups of k_near_blocks
    u64* mask;                        // [kNearSide] block rows' non-empty blocks
    unsigned* alloc;                  // cells given out
    uint2* block;                     // [kNearBlocks] first cell; cell shifts (x, y << 4),
                                      // kNone: no agents
    unsigned* sum;                    // [cells / kNearScan] agents per stretch, or null
    unsigned* row;                    // [rows][kNearBlocks]
    unsigned* count;                  // [cells] agents per cell
    unsigned* first;                  // [cells + 1] agents before
    unsigned* cell;                   // [n] agent's cell, kNone: another one stands for it
    unsigned* rank;                   // [n] its rank in the cell; top bit: it shares its tile
    unsigned* spos;                   // [n] sorted packed positions
    unsigned* sid;                    // [n] and their agents; top bit as in rank
};

__device__ __forceinline__ unsigned near_block_of(unsigned p) {
    return ((p >> (16 + kNearShift)) & (kNearSide - 1)) * kNearSide +
           ((p & 0x7FFFu) >> kNearShift);
}

// Lanes of `mask` below this one.
__device__ __forceinline__ unsigned lanes_below(u64 mask) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

__global__ void __launch_bounds__(1024) k_near_blocks(NearArgs A) {
    __shared__ unsigned s_cnt[kNearBlocks];
    const unsigned t = threadIdx.x, step = gridDim.x * 1024u;
#pragma unroll
    for (unsigned k = 0; k < kNearBlocks; k += 1024) s_cnt[k + t] = 0;
    uint4* count = reinterpret_cast<uint4*>(A.count);
    for (unsigned c = blockIdx.x * 1024u + t; c < A.cells / 4; c += step)
        count[c] = make_uint4(0, 0, 0, 0);
    if (blockIdx.x == 0 && t == 0) *A.alloc = 0;
    __syncthreads();
    for (u64 i0 = blockIdx.x * 1024u; i0 < A.n; i0 += step) {      // workgroup-uniform
        const bool valid = i0 + t < A.n;
        unsigned b = 0;
        if (valid) {
            const int2 q = position(A.pos, i0 + t);
            b = near_block_of(pack_pos(q.x, q.y));
        }
        // the first lane's block by one addition of all its lanes (a town
        // may lie in one block), the others one by one
        const u64 rest = __ballot(valid);
        const unsigned b0 = (unsigned)__builtin_amdgcn_readfirstlane((int)b);
        const u64 m = __ballot(valid && b == b0);
        if (m && __lane_id() == (unsigned)__builtin_ctzll(m))
            atomicAdd(&s_cnt[b0], (unsigned)__popcll(m));
        if (((rest & ~m) >> __lane_id()) & 1) atomicAdd(&s_cnt[b], 1u);
    }
    __syncthreads();
#pragma unroll
    for (unsigned k = 0; k < kNearBlocks; k += 1024)
        A.row[(u64)blockIdx.x * kNearBlocks + k + t] = s_cnt[k + t];
}

// A row of blocks per workgroup: its waves add up the rows of counts, then its
// first wave gives every block 2^floor(log2 agents) cells, reserved for the
// whole row with one atomic (the order of the block rows does not matter).
__global__ void __launch_bounds__(1024) k_near_cells(NearArgs A) {
    __shared__ unsigned s_sum[16][64];
    const unsigned l = threadIdx.x & 63u, w = threadIdx.x >> 6;
    const unsigned b = blockIdx.x * 64u + l;
    unsigned m = 0;
#pragma unroll 4
    for (unsigned r = w; r < A.rows; r += 16) m += A.row[(u64)r * kNearBlocks + b];
    s_sum[w][l] = m;
    __syncthreads();
    if (w) return;
    m = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) m += s_sum[k][l];
    const u64 some = __ballot(m != 0);               // a workgroup is a block row
    if (l == 0) A.mask[blockIdx.x] = some;
    const unsigned lg = m ? 31u - (unsigned)__builtin_clz(m) : 0u;
    // 2^(2 kNearShift - area) cells of 2^sx x 2^sy tiles, sx + sy = area
    const unsigned area = 2 * kNearShift - min(lg, 2 * kNearShift);
    const unsigned sy = min(kNearShift, area - (area > 1 ? (area - 1) / 2 : 0u));
    const unsigned sx = area - sy;
    const unsigned cells = m ? 1u << (2 * kNearShift - area) : 0u;
    unsigned incl = cells;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned c = __shfl_up(incl, o);
        if (l >= (unsigned)o) incl += c;
    }
    unsigned base = 0;
    if (l == 63) base = atomicAdd(A.alloc, incl);
    A.block[b] = make_uint2(__shfl(base, 63) + incl - cells, m ? sx | (sy << 4) : kNone);
}

// The grid of one block: cell (cx, cy) is cell `base + (cy << sh) + cx` and
// covers 2^sx x 2^sy tiles.
struct NearGrid {
    unsigned base, sx, sy, sh;
    bool any;
    __device__ explicit NearGrid(uint2 v)
        : base(v.x), sx(min(v.y & 15u, kNearShift)), sy(min((v.y >> 4) & 15u, kNearShift)),
          sh(kNearShift - sx), any(v.y != kNone) {}
    __device__ unsigned cell(unsigned cx, unsigned cy) const { return base + (cy << sh) + cx; }
};

__global__ void __launch_bounds__(kNearThreads) k_near_count(NearArgs A) {
    constexpr unsigned kSlots = 2 * kNearThreads;
    static_assert(kSlots == 512, "9 hash bits");
    __shared__ unsigned s_key[kSlots], s_cnt[kSlots];    // tiles of the workgroup's agents
    const unsigned t = threadIdx.x;
#pragma unroll
    for (unsigned k = 0; k < kSlots; k += kNearThreads) {
        s_key[k + t] = kNone;
        s_cnt[k + t] = 0;
    }
    const u64 i = (u64)blockIdx.x * kNearThreads + t;
    const bool valid = i < A.n;
    unsigned c = 0, p = 0, slot = 0, r = 0;
    if (valid) {
        const int2 q = position(A.pos, i);
        p = pack_pos(q.x, q.y);
        const NearGrid g(A.block[near_block_of(p)]);
        c = min(g.cell((p & (kNearTiles - 1)) >> g.sx, ((p >> 16) & (kNearTiles - 1)) >> g.sy),
                A.cells - 1);
        slot = (p * 2654435761u) >> 23;              // multiplicative hash to 9 bits
    }
    __syncthreads();
    if (valid) {
        for (;;) {                                   // more slots than agents: ends
            unsigned key = s_key[slot];
            if (key == kNone) key = atomicCAS(&s_key[slot], kNone, p);
            if (key == kNone || key == p) break;
            slot = (slot + 1) & (kSlots - 1);
        }
        r = atomicAdd(&s_cnt[slot], 1u);
    }
    __syncthreads();
    if (!valid) return;
    const bool shared = s_cnt[slot] > 1;
    if (r == 0) r = atomicAdd(&A.count[c], 1u) | (shared ? kNearShared : 0u);
    else c = kNone;
    A.cell[i] = c;
    A.rank[i] = r;
    if (shared) A.out[i] = interaction_of(0, A.d_action[i], A.velocity, A.radius);
}

__global__ void __launch_bounds__(1024) k_near_sum(NearArgs A) {
    __shared__ unsigned s_sum;
    if (threadIdx.x == 0) s_sum = 0;
    __syncthreads();
    const uint4 v = reinterpret_cast<const uint4*>(A.count)[blockIdx.x * (kNearScan / 4) + threadIdx.x];
    unsigned all = v.x + v.y + v.z + v.w;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) all += __shfl_xor(all, o);
    if (__lane_id() == 0) atomicAdd(&s_sum, all);
    __syncthreads();
    if (threadIdx.x == 0) A.sum[blockIdx.x] = s_sum;
}

// Exclusive scan of the counts, kNearScan cells a workgroup, which adds up the
// cells before its own itself, so no workgroup waits for another: from the
// sums where there are many (n above kNearSums), else from the counts (at most
// 1 MiB, which costs less than the launch of k_near_sum).
__global__ void __launch_bounds__(1024) k_near_scan(NearArgs A) {
    __shared__ unsigned s_sum[17];
    const unsigned t = threadIdx.x, l = __lane_id(), w = t >> 6;
    const unsigned c = blockIdx.x * kNearScan + 4 * t;
    const uint4* cnt = reinterpret_cast<const uint4*>(A.count);
    unsigned before = 0;
    if (A.sum) {
        for (unsigned q = t; q < blockIdx.x; q += 1024) before += A.sum[q];
    } else {
#pragma unroll 4
        for (unsigned q = t; q < blockIdx.x * (kNearScan / 4); q += 1024) {
            const uint4 v = cnt[q];
            before += v.x + v.y + v.z + v.w;
        }
    }
    const uint4 v = cnt[c / 4];
    const unsigned own = v.x + v.y + v.z + v.w;
    unsigned incl = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned a = __shfl_up(incl, o);
        if (l >= (unsigned)o) incl += a;
        before += __shfl_xor(before, o);
    }
    if (t == 0) s_sum[16] = 0;
    if (l == 63) s_sum[w] = incl;
    __syncthreads();
    if (l == 0 && before) atomicAdd(&s_sum[16], before);
    unsigned ex = incl - own;
    for (unsigned k = 0; k < w; ++k) ex += s_sum[k];
    __syncthreads();
    ex += s_sum[16];
    *reinterpret_cast<uint4*>(A.first + c) =
        make_uint4(ex, ex + v.x, ex + v.x + v.y, ex + v.x + v.y + v.z);
    if (c + 4 == A.cells) A.first[A.cells] = ex + own;
}

__global__ void __launch_bounds__(kNearThreads) k_near_place(NearArgs A) {
    const u64 i = (u64)blockIdx.x * kNearThreads + threadIdx.x;
    if (i >= A.n) return;
    const unsigned c = A.cell[i], r = A.rank[i];
    if (c >= A.cells) return;
    const int2 q = position(A.pos, i);
    const unsigned at = A.first[c] + (r & ~kNearShared);
    if (at >= A.n) return;
    A.spos[at] = pack_pos(q.x, q.y);
    A.sid[at] = (unsigned)i | (r & kNearShared);
}

// Whole tiles that cover every point nearer than squared distance d2 >= 1:
// the root of d2 - 1, rounded down; the addend is more than the float's error
// (0.004 tiles at 2^31), so the result is never too small.
__device__ __forceinline__ unsigned near_reach(unsigned d2) {
    return (unsigned)(__builtin_sqrtf((float)(d2 - 1)) + 0.01f);
}

// Tiles between v and the stretch [lo, hi] (0 inside).
__device__ __forceinline__ unsigned near_gap(unsigned v, unsigned lo, unsigned hi) {
    return v < lo ? lo - v : v > hi ? v - hi : 0u;
}

// One lane's search for the agent nearest to agent k (sorted) at (x, y).
struct NearSearch {
    const NearArgs& A;
    const u64* mask;                  // LDS: block rows' non-empty blocks
    unsigned k, p, x, y, best;

    __device__ unsigned first(unsigned c) const { return min(A.first[min(c, A.cells)], A.n); }

    __device__ void one(unsigned j) {
        const unsigned d = dist2(p, A.spos[j]);
        if (j != k) best = min(best, d);
    }

    // the sorted agents [lo, hi), which do not hold agent k: sixteen at a time
    // by four reads, then the rest four at a time (the last one again where
    // there are fewer)
    __device__ void part(unsigned lo, unsigned hi) {
        const unsigned* s = A.spos + lo;
        unsigned left = hi - min(lo, hi);
        for (; left >= 16 && best; left -= 16, s += 16) {
            uint4 q[4];
            __builtin_memcpy(q, s, sizeof q);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                best = min(best, dist2(p, q[u].x));
                best = min(best, dist2(p, q[u].y));
                best = min(best, dist2(p, q[u].z));
                best = min(best, dist2(p, q[u].w));
            }
        }
        for (unsigned v = 0; v < left && best; v += 4) {
            unsigned q[4];
#pragma unroll
            for (unsigned u = 0; u < 4; ++u) q[u] = s[min(v + u, left - 1)];
#pragma unroll
            for (unsigned u = 0; u < 4; ++u) best = min(best, dist2(p, q[u]));
        }
    }
    // the sorted agents [lo, hi)
    __device__ void run(unsigned lo, unsigned hi) {
        if (k >= lo && k < hi) {
            part(lo, k);
            part(k + 1, hi);
        } else {
            part(lo, hi);
        }
    }

    // The run of row c of a block at bx, as wide as an agent `gap` tiles off
    // the row can be nearer than `best`: false if that leaves the block.
    __device__ bool row(const NearGrid& g, unsigned bx, unsigned c, unsigned gap, unsigned& lo,
                        unsigned& hi) const {
        const unsigned w = near_reach(best - gap * gap);
        if (x + w < bx || x > bx + kNearTiles - 1 + w) return false;
        const unsigned l = max(x > w ? x - w : 0u, bx) - bx;
        const unsigned r = min(x + w, bx + kNearTiles - 1) - bx;
        lo = first(g.cell(l >> g.sx, c));
        hi = first(g.cell(r >> g.sx, c) + 1);
        return lo < hi;
    }

    // Block (qx, qy): its rows from the one nearest outwards, 2 kAhead rows
    // looked up together, while they are nearer than the best so far.  In long
    // runs the agents about x come first, which mostly shortens them.
    __device__ void block(unsigned qx, unsigned qy) {
        constexpr int kAhead = 4;
        const NearGrid g(A.block[qy * kNearSide + qx]);
        if (!g.any) return;
        const unsigned bx = qx << kNearShift, by = qy << kNearShift;
        const unsigned rows = kNearTiles >> g.sy;
        const unsigned near = (min(max(y, by), by + kNearTiles - 1) - by) >> g.sy;
        const unsigned cx = (min(max(x, bx), bx + kNearTiles - 1) - bx) >> g.sx;
        // from above or below, the empty rows before the first agent are passed
        // over: the agents of whole rows are a difference of two cells' places
        unsigned start = 0;
        if (y < by || y > by + kNearTiles - 1) {
            const bool below = y > by + kNearTiles - 1;      // of the block
            const unsigned edge = first(g.cell(0, below ? rows : 0));
            unsigned over = rows - 1;                        // the row sought is in [start, over]
            while (start < over) {
                const unsigned mid = (start + over) / 2;
                if (first(g.cell(0, below ? rows - 1 - mid : mid + 1)) != edge) over = mid;
                else start = mid + 1;
            }
        }
        for (unsigned d0 = start; d0 < rows; d0 += kAhead) {
            unsigned lo[2 * kAhead], hi[2 * kAhead];
            auto place = [&](int s, unsigned& c, unsigned& gap) {
                const unsigned d = d0 + (s >> 1);
                c = s & 1 ? near + d : near - d;
                if (s & 1 ? d == 0 || c >= rows : d > near) return false;
                gap = near_gap(y, by + (c << g.sy), by + ((c + 1) << g.sy) - 1);
                return gap * gap < best;
            };
            bool any = false, wide = false;
#pragma unroll
            for (int s = 0; s < 2 * kAhead; ++s) {
                unsigned c, gap;
                lo[s] = hi[s] = 0;
                if (!place(s, c, gap)) continue;
                any = true;
                if (!row(g, bx, c, gap, lo[s], hi[s])) lo[s] = hi[s] = 0;
                wide |= hi[s] - lo[s] > 32;
            }
            if (!any) break;
            if (wide) {
                unsigned j[2 * kAhead];
#pragma unroll
                for (int s = 0; s < 2 * kAhead; ++s) {
                    unsigned c, gap;
                    j[s] = hi[s] > lo[s] && place(s, c, gap) ? first(g.cell(cx, c)) : 0u;
                }
#pragma unroll
                for (int s = 0; s < 2 * kAhead; ++s) {
                    if (j[s] >= lo[s] && j[s] < hi[s]) one(j[s]);
                    if (j[s] > lo[s] && j[s] <= hi[s]) one(j[s] - 1);
                }
#pragma unroll
                for (int s = 0; s < 2 * kAhead; ++s) {
                    unsigned c, gap;
                    if (hi[s] - lo[s] <= 32) continue;
                    if (!place(s, c, gap) || !row(g, bx, c, gap, lo[s], hi[s])) lo[s] = hi[s] = 0;
                }
            }
            // few agents: eight at a time whatever their row; else row by row
            unsigned end[2 * kAhead], total = 0;
#pragma unroll
            for (int s = 0; s < 2 * kAhead; ++s) end[s] = total += hi[s] - lo[s];
            if (total <= kNearFew) {
                for (unsigned v = 0; v < total && best; v += 8) {
                    unsigned q[8], at[8];
#pragma unroll
                    for (unsigned u = 0; u < 8; ++u) {
                        const unsigned w = min(v + u, total - 1);
                        at[u] = lo[0] + w;
#pragma unroll
                        for (int s = 1; s < 2 * kAhead; ++s)
                            at[u] = w >= end[s - 1] ? lo[s] + (w - end[s - 1]) : at[u];
                        q[u] = A.spos[at[u]];
                    }
#pragma unroll
                    for (unsigned u = 0; u < 8; ++u) {
                        const unsigned d = dist2(p, q[u]);
                        if (at[u] != k) best = min(best, d);
                    }
                }
                continue;
            }
            for (int s = 0; s < 2 * kAhead; ++s) {   // one copy of the run's code
                unsigned l = 0, h = 0;
#pragma unroll
                for (int q = 0; q < 2 * kAhead; ++q) {
                    l = q == s ? lo[q] : l;
                    h = q == s ? hi[q] : h;
                }
                if (l < h) run(l, h);
            }
        }
    }

    // `best` to one more than a distance within which some other agent must
    // be: the farthest corner of a non-empty block, from the nearest blocks of
    // each block row outwards.  `alone`: the agent is its block's only one.
    __device__ void bound(bool alone) {
        const unsigned qx = x >> kNearShift, qy = y >> kNearShift;
        auto take = [&](unsigned bx, unsigned by) {
            const unsigned x0 = bx << kNearShift, y0 = by << kNearShift;
            const unsigned dx = max(x > x0 ? x - x0 : x0 - x, near_far(x, x0));
            const unsigned dy = max(y > y0 ? y - y0 : y0 - y, near_far(y, y0));
            best = min(best, dx * dx + dy * dy + 1);
        };
        for (unsigned d = 0; d < kNearSide; ++d) {
            const unsigned gap = d ? min(y - ((qy - d + 1) << kNearShift) + 1,
                                         ((qy + d) << kNearShift) - y) : 0u;
            if (gap < 46341u && gap * gap >= best) break;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                if (s == 0 ? d > qy : d == 0 || qy + d >= kNearSide) continue;
                const unsigned r = s == 0 ? qy - d : qy + d;
                u64 m = mask[r];
                if (d == 0 && alone) m &= ~(1ull << qx);
                const u64 left = m & ((2ull << qx) - 1), right = m & ~((2ull << qx) - 1);
                if (left) take(63u - (unsigned)__builtin_clzll(left), r);
                if (right) take((unsigned)__builtin_ctzll(right), r);
            }
        }
    }
    __device__ static unsigned near_far(unsigned v, unsigned lo) {
        const unsigned hi = lo + kNearTiles - 1;
        return v > hi ? v - hi : hi - v;
    }

    // every block but its own that may hold a nearer agent
    __device__ void others() {
        const unsigned qx = x >> kNearShift, qy = y >> kNearShift;
        for (unsigned d = 0; d < kNearSide; ++d) {
            bool any = false;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                if (s == 0 ? d > qy : d == 0 || qy + d >= kNearSide) continue;
                const unsigned r = s == 0 ? qy - d : qy + d, by = r << kNearShift;
                const unsigned gy = near_gap(y, by, by + kNearTiles - 1);
                if (gy * gy >= best) continue;
                any = true;
                const unsigned w = near_reach(best);
                const unsigned b0 = (x > w ? x - w : 0u) >> kNearShift;
                const unsigned b1 = min(x + w, 0x7FFFu) >> kNearShift;
                u64 m = mask[r] & (~0ull << b0) & (~0ull >> (63 - b1));
                if (d == 0) m &= ~(1ull << qx);
                for (; m; m &= m - 1) {
                    const unsigned b = (unsigned)__builtin_ctzll(m), bx = b << kNearShift;
                    const unsigned gx = near_gap(x, bx, bx + kNearTiles - 1);
                    if (gx * gx + gy * gy < best) block(b, r);
                }
            }
            if (!any) break;
        }
    }
};

__global__ void __launch_bounds__(kNearThreads) k_near_find(NearArgs A) {
    __shared__ u64 s_mask[kNearSide];
    if (threadIdx.x < kNearSide) s_mask[threadIdx.x] = A.mask[threadIdx.x];
    __syncthreads();
    const u64 k64 = (u64)blockIdx.x * kNearThreads + threadIdx.x;
    const unsigned n = min(A.first[A.cells], A.n);   // sorted agents
    if (k64 >= n) return;
    const unsigned k = (unsigned)k64, id = A.sid[k], p = A.spos[k] & 0x7FFF7FFFu, x = p & 0xFFFFu, y = p >> 16;
    if (id & kNearShared) return;                    // done by k_near_count
    NearSearch S{A, s_mask, k, p, x, y, kNone};

    // Its cell, three cells either side and the rows above and below it, as
    // far as the block goes: their runs are looked up together, and in even
    // country that is the whole search.
    const unsigned qx = x >> kNearShift, qy = y >> kNearShift;
    const NearGrid g(A.block[qy * kNearSide + qx]);
    const unsigned bx = qx << kNearShift, by = qy << kNearShift;
    const unsigned cx = (x - bx) >> g.sx, cy = (y - by) >> g.sy;
    const unsigned l = cx > 3 ? cx - 3 : 0u, r = min(cx + 3, (kNearTiles >> g.sx) - 1);
    const unsigned u = cy ? cy - 1 : 0u, d = min(cy + 1, (kNearTiles >> g.sy) - 1);
    unsigned lo[3], hi[3];
    lo[0] = S.first(g.cell(l, cy));
    hi[0] = S.first(g.cell(r, cy) + 1);
    lo[1] = S.first(g.cell(l, u));
    hi[1] = u < cy ? S.first(g.cell(r, u) + 1) : 0u;
    lo[2] = S.first(g.cell(l, d));
    hi[2] = d > cy ? S.first(g.cell(r, d) + 1) : 0u;
    const unsigned s0 = S.first(g.cell(cx, cy)), e0 = S.first(g.cell(cx, cy) + 1);
    const unsigned n0 = hi[0] - min(lo[0], hi[0]), n1 = hi[1] - min(lo[1], hi[1]);
    const unsigned total = n0 + n1 + (hi[2] - min(lo[2], hi[2]));
    // squared distances below which any agent of the block, and any agent at
    // all, was looked at here
    unsigned here, all;
    if (total <= kNearFew) {
        for (unsigned v = 0; v < total; v += 8) {
            unsigned j[8], q[8];
#pragma unroll
            for (unsigned u8 = 0; u8 < 8; ++u8) {
                const unsigned w = min(v + u8, total - 1);
                j[u8] = w < n0 ? lo[0] + w : w - n0 < n1 ? lo[1] + (w - n0) : lo[2] + (w - n0 - n1);
                q[u8] = A.spos[j[u8]];
            }
#pragma unroll
            for (unsigned u8 = 0; u8 < 8; ++u8) {
                const unsigned d2 = dist2(p, q[u8]);
                if (j[u8] != k) S.best = min(S.best, d2);
            }
        }
        constexpr unsigned kOpen = 1u << 15;         // the block's own edge
        const unsigned ex = min(l ? x - bx - (l << g.sx) + 1 : kOpen,
                                r + 1 < kNearTiles >> g.sx ? bx + ((r + 1) << g.sx) - x : kOpen);
        const unsigned ey = min(u ? y - by - (u << g.sy) + 1 : kOpen,
                                d + 1 < kNearTiles >> g.sy ? by + ((d + 1) << g.sy) - y : kOpen);
        const unsigned e = min(ex, ey);
        const unsigned f = min(min(x - bx, bx + kNearTiles - 1 - x),
                               min(y - by, by + kNearTiles - 1 - y)) + 1;
        here = e * e;
        all = min(here, f * f);
    } else {
        S.run(s0, e0);
        here = all = 1;                              // its own tile at least
    }
    if (S.best > all) {
        if (S.best > here) {
            // the sorted neighbours are mostly near, however empty the cells
            if (k > 0) S.one(k - 1);
            if (k + 1 < n) S.one(k + 1);
            if (near_reach(S.best) > kNearTiles) S.bound(g.sx + g.sy == 2 * kNearShift);
            S.block(qx, qy);
        }
        S.others();
    }
    const unsigned i = id;
    if (i < A.n) A.out[i] = interaction_of(S.best, A.d_action[i], A.velocity, A.radius);
}

// The search by cells starts where it is at least as fast whatever the agents'
// places.  Agents uniform on 2048 x 2048 tiles: all pairs 49 us at 24,000, 78 at
// 28,000 and 221 at 50,000, the search 36, 36 and 40 us.  A dense town and a
// few agents very far from it, its slowest case seen: 92 us at 25,000 and 96 to
// 150 us at 50,000.
constexpr unsigned kNearAgents = 32768;

inline u64 near_cells(unsigned n) { return ((u64)n + kNearScan - 1) / kNearScan * kNearScan; }
inline unsigned near_rows(unsigned n) { return std::min<u64>(kNearRows, ((u64)n + 1023) / 1024); }

inline u64 near_bytes(unsigned n) {
    const u64 cells = near_cells(n);
    return 16 + 8 * (kNearSide + kNearBlocks) +
           4 * ((cells / kNearScan + 3) / 4 * 4 + (u64)near_rows(n) * kNearBlocks + 2 * cells + 4 +
                4 * (u64)n);
}

// Workgroups that write the agents' words: no more than there are agents.
inline unsigned obj_pack_blocks(unsigned N) {
    return (unsigned)std::min<u64>(((u64)N + 2047) / 2048, 1024);
}

inline unsigned obj_blocks(unsigned M, unsigned R) {
    return (unsigned)(((u64)M + R + kObjTile - 1) / kObjTile);
}

}  // namespace
}  // namespace ss

using namespace ss;

extern "C" {

uint64_t ss_object_distances_workspace(uint32_t n_objects, uint32_t n_refs, uint32_t n_agents) {
    const u64 blocks = obj_blocks(n_objects, n_refs);
    return blocks * sizeof(ObjCarry) + ((blocks + 1 + 3) & ~3ull) * 4 + (u64)n_agents * 8;
}

}  // extern "C"

namespace {

// Checks the arguments of ss_object_distances and fills the kernel arguments.
ss_status object_args(const uint32_t* obj_off, const uint32_t* obj_agents, uint32_t n_objects,
                      uint32_t n_refs, const uint32_t* distances, const uint8_t* active,
                      uint32_t n_agents, uint32_t* obj_distances, uint8_t* obj_active,
                      void* workspace, uint64_t workspace_bytes, ObjArgs* A) {
    if (n_objects >= (1u << 31) || n_refs >= (1u << 31))
        return set_err(SS_ERR_ARG, "n_objects and n_refs must be below 2^31");
    if (!obj_off || !obj_distances || !obj_active || !workspace ||
        (n_refs && !obj_agents) || (n_agents && (!distances || !active)))
        return set_err(SS_ERR_ARG, "NULL argument");
    const u64 need = ss_object_distances_workspace(n_objects, n_refs, n_agents);
    if (workspace_bytes < need)
        return set_err(SS_ERR_ARG, "workspace_bytes %llu < %llu", (unsigned long long)workspace_bytes,
                       (unsigned long long)need);
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return set_err(SS_ERR_ARG, "no current device");
    }
    if (!device_range_ok(obj_off, ((u64)n_objects + 1) * 4, dev) ||
        (n_refs && !device_range_ok(obj_agents, (u64)n_refs * 4, dev)) ||
        (n_agents && (!device_range_ok(distances, (u64)n_agents * 4, dev) ||
                      !device_range_ok(active, n_agents, dev))) ||
        !device_range_ok(obj_distances, (u64)n_objects * 4, dev) ||
        !device_range_ok(obj_active, n_objects, dev) ||
        !device_range_ok(workspace, need, dev))
        return set_err(SS_ERR_ARG, "every array must be device memory of the current device (%d)",
                       dev);
    A->off = obj_off;
    A->agents = obj_agents;
    A->dist = distances;
    A->active = active;
    A->M = n_objects;
    A->R = n_refs;
    A->N = n_agents;
    A->out_dist = obj_distances;
    A->out_act = obj_active;
    const u64 blocks = obj_blocks(n_objects, n_refs);
    A->carry = static_cast<ObjCarry*>(workspace);
    A->coord = reinterpret_cast<unsigned*>(A->carry + blocks);
    // eight bytes an agent: its word, and room for the workgroups' flags
    A->w = A->coord + ((blocks + 1 + 3) & ~3ull);
    A->odd = A->w + n_agents;
    A->odd_n = obj_pack_blocks(n_agents);
    return SS_OK;
}

hipError_t object_launch(const ObjArgs& A, hipStream_t st) {
    const unsigned blocks = obj_blocks(A.M, A.R);
    const unsigned part_blocks = (blocks + 1 + 15) / 16;
    const unsigned pack_blocks = A.odd_n;
    hipLaunchKernelGGL(k_obj_prep, dim3(part_blocks + pack_blocks), dim3(256), 0, st, A,
                       blocks + 1, part_blocks);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 256;
    // eight resident workgroups per CU (LDS and registers allow eight)
    const unsigned grid = (unsigned)std::min<u64>(((u64)blocks + 7) / 8 * 8,
                                                  (u64)std::max(cus, 8) / 8 * 8 * 8);
    hipLaunchKernelGGL(k_obj_min, dim3(grid), dim3(kObjThreads), 0, st, A, blocks);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_obj_fix, dim3((blocks + 255) / 256), dim3(256), 0, st, A.carry, blocks,
                       A.M, A.out_dist, A.out_act);
    return hipGetLastError();
}

}  // namespace

namespace {

// The search by frontier queues on `st`.
ss_status queue_launch(const QueueArgs& args, int dev, hipStream_t st) {
    QueueArgs A = args;
    int coop = 0, cus = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess ||
        !coop || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(k_queue),
                                                     kQueueThreads, 0) != hipSuccess || per_cu < 1) {
        (void)hipGetLastError();
        return set_err(SS_ERR_HIP, "cooperative launch is not available on device %d", dev);
    }
    // one workgroup per 512 vertices, at most one per CU: every workgroup
    // pays an L2 write-back and invalidate at each grid barrier, so fewer,
    // wider workgroups (two vertices per thread per round) are cheaper
    const u64 want = ((u64)A.V + kQueueThreads * kQueueVerts - 1) / (kQueueThreads * kQueueVerts);
    const unsigned grid = (unsigned)std::max<u64>(1, std::min<u64>(want, (u64)cus));
    hipLaunchKernelGGL(k_queue_init, dim3((A.V + kQueueThreads - 1) / kQueueThreads),
                       dim3(kQueueThreads), 0, st, A);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && A.n_src) {
        hipLaunchKernelGGL(k_queue_src, dim3((A.n_src + kQueueThreads - 1) / kQueueThreads),
                           dim3(kQueueThreads), 0, st, A);
        e = hipGetLastError();
    }
    if (e == hipSuccess) {
        void* a[] = {&A};
        e = hipLaunchCooperativeKernel(reinterpret_cast<const void*>(k_queue), dim3(grid),
                                       dim3(kQueueThreads), a, 0, st);
    }
    if (e != hipSuccess) return set_err(SS_ERR_HIP, "hop distance kernels: %s", hipGetErrorString(e));
    return SS_OK;
}

}  // namespace

extern "C" {

ss_status ss_object_distances(const uint32_t* obj_off, const uint32_t* obj_agents,
                              uint32_t n_objects, uint32_t n_refs, const uint32_t* distances,
                              const uint8_t* active, uint32_t n_agents, uint32_t* obj_distances,
                              uint8_t* obj_active, void* workspace, uint64_t workspace_bytes,
                              void* stream) {
    if (n_objects == 0 && n_refs < (1u << 31)) return SS_OK;
    ObjArgs A;
    ss_status st = object_args(obj_off, obj_agents, n_objects, n_refs, distances, active,
                               n_agents, obj_distances, obj_active, workspace, workspace_bytes, &A);
    if (st != SS_OK) return st;
    hipError_t e = object_launch(A, static_cast<hipStream_t>(stream));
    if (e != hipSuccess)
        return set_err(SS_ERR_HIP, "object distance kernels: %s", hipGetErrorString(e));
    return SS_OK;
}

ss_status ss_probe_object_distances(const uint32_t* obj_off, const uint32_t* obj_agents,
                                    uint32_t n_objects, uint32_t n_refs,
                                    const uint32_t* distances, const uint8_t* active,
                                    uint32_t n_agents, uint32_t* obj_distances,
                                    uint8_t* obj_active, void* workspace,
                                    uint64_t workspace_bytes, int iters, float* ms_per_iter) {
    if (iters < 1 || !ms_per_iter || n_objects == 0)
        return set_err(SS_ERR_ARG, "bad probe arguments");
    ObjArgs A;
    ss_status st = object_args(obj_off, obj_agents, n_objects, n_refs, distances, active,
                               n_agents, obj_distances, obj_active, workspace, workspace_bytes, &A);
    if (st != SS_OK) return st;
    hipEvent_t a = nullptr, b = nullptr;
    hipStream_t s = nullptr;
    hipError_t e = hipEventCreate(&a);
    if (e == hipSuccess) e = hipEventCreate(&b);
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
    if (e == hipSuccess) e = object_launch(A, s);                  // warm-up
    if (e == hipSuccess) e = hipEventRecord(a, s);
    for (int i = 0; i < iters && e == hipSuccess; ++i) e = object_launch(A, s);
    if (e == hipSuccess) e = hipEventRecord(b, s);
    if (e == hipSuccess) e = hipEventSynchronize(b);
    float t = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&t, a, b);
    if (s) (void)hipStreamDestroy(s);
    if (a) (void)hipEventDestroy(a);
    if (b) (void)hipEventDestroy(b);
    if (e != hipSuccess) return set_err(SS_ERR_HIP, "object distance probe: %s", hipGetErrorString(e));
    *ms_per_iter = t / iters;
    return SS_OK;
}

uint64_t ss_hop_distances_workspace(uint32_t n_vertices) {
    return 64 + 2 * (((uint64_t)n_vertices * 8 + 255) & ~255ull);
}

}  // extern "C"

namespace {

// ss_hop_distances with `base` polls of every wait's bound independent of the
// graph, and for up to kBfsSweep vertices at most `most` workgroups.
ss_status hop_call(const uint32_t* row_off, const uint32_t* col, uint32_t n_vertices,
                   uint32_t n_edges, const uint32_t* sources, uint32_t n_sources,
                   uint32_t max_hops, uint32_t* hops, void* workspace, uint64_t workspace_bytes,
                   unsigned most, u64 base, void* stream) {
    if (n_vertices >= (1u << 31) || n_edges >= (1u << 31))
        return set_err(SS_ERR_ARG, "n_vertices and n_edges must be below 2^31");
    if (n_vertices == 0) return SS_OK;
    if (!row_off || !hops || !workspace || (n_edges && !col) || (n_sources && !sources))
        return set_err(SS_ERR_ARG, "NULL argument");
    const u64 need = ss_hop_distances_workspace(n_vertices);
    if (workspace_bytes < need)
        return set_err(SS_ERR_ARG, "workspace_bytes %llu < %llu", (unsigned long long)workspace_bytes,
                       (unsigned long long)need);
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return set_err(SS_ERR_ARG, "no current device");
    }
    if (!device_range_ok(row_off, ((u64)n_vertices + 1) * 4, dev) ||
        (n_edges && !device_range_ok(col, (u64)n_edges * 4, dev)) ||
        (n_sources && !device_range_ok(sources, (u64)n_sources * 4, dev)) ||
        !device_range_ok(hops, (u64)n_vertices * 4, dev) || !device_range_ok(workspace, need, dev))
        return set_err(SS_ERR_ARG, "every array must be device memory of the current device (%d)",
                       dev);
    hipStream_t st = static_cast<hipStream_t>(stream);
    char* ws = static_cast<char*>(workspace);
    if (n_vertices > kBfsSweep) {
        const u64 qbytes = ((u64)n_vertices * 8 + 255) & ~255ull;
        return queue_launch({row_off, col, sources, n_vertices, n_edges, n_sources, max_hops, hops,
                             reinterpret_cast<uint2*>(ws + 64),
                             reinterpret_cast<uint2*>(ws + 64 + qbytes),
                             reinterpret_cast<unsigned*>(ws),
                             hop_polls(base, n_vertices, n_edges)}, dev, st);
    }
    int cus = 256;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        cus = 256;
    }
    BfsArgs A{};
    A.row_off = row_off;
    A.col = col;
    A.src = sources;
    A.V = n_vertices;
    A.E = n_edges;
    A.n_src = n_sources;
    A.max_hops = max_hops;
    A.hops = hops;
    A.ctl = reinterpret_cast<unsigned*>(ws);
    A.polls = hop_polls(base, n_vertices, n_edges);
    // claims that fail cost more than the hint's read once a level has many
    if (n_vertices >= 32768) A.hint = reinterpret_cast<u64*>(ws + 4 * kCtlWords);
    // chunks of 1,024 vertices, from 96 chunks on of up to 4,096, at most one
    // per CU: more workgroups expand faster, but all of them add to and poll one
    // counter per level (200,000 vertices: 196 chunks 97 us, 98 chunks 86 us;
    // 50,000: 25 chunks 79 us, 49 chunks 64 us; 1 M: 1,024 chunks of a quarter
    // of the threads 817 us, 256 chunks 212 us); fewer vertices where a chunk
    // would have more than 2^17 edges (20,000 of degree 500: 1,775 us by 20 chunks,
    // 961 us by 76)
    const u64 V = n_vertices;
    const u64 want = std::max({(V + 4095) / 4096, std::min<u64>((V + 1023) / 1024, 96),
                               std::min<u64>((V + 63) / 64, n_edges >> 17)});
    A.chunks = (unsigned)std::min<u64>(want, std::min<unsigned>(kBfsMost, std::max(cus, 1)));
    hipLaunchKernelGGL(k_bfs_init, dim3((n_vertices + kBfsThreads - 1) / kBfsThreads),
                       dim3(kBfsThreads), 0, st, A);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_bfs, dim3(std::min(A.chunks, most)), dim3(kBfsThreads), 0, st, A);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return set_err(SS_ERR_HIP, "hop distance kernels: %s", hipGetErrorString(e));
    return SS_OK;
}

}  // namespace

extern "C" {

ss_status ss_hop_distances(const uint32_t* row_off, const uint32_t* col, uint32_t n_vertices,
                           uint32_t n_edges, const uint32_t* sources, uint32_t n_sources,
                           uint32_t max_hops, uint32_t* hops, void* workspace,
                           uint64_t workspace_bytes, void* stream) {
    return hop_call(row_off, col, n_vertices, n_edges, sources, n_sources, max_hops, hops,
                    workspace, workspace_bytes, kBfsMost, kHopPolls, stream);
}

ss_status ss_probe_hop_distances(const uint32_t* row_off, const uint32_t* col, uint32_t n_vertices,
                                 uint32_t n_edges, const uint32_t* sources, uint32_t n_sources,
                                 uint32_t max_hops, uint32_t* hops, void* workspace,
                                 uint64_t workspace_bytes, uint32_t workgroups, uint32_t polls) {
    if (workgroups < 1) return set_err(SS_ERR_ARG, "workgroups must be >= 1");
    ss_status r = hop_call(row_off, col, n_vertices, n_edges, sources, n_sources, max_hops, hops,
                           workspace, workspace_bytes, workgroups, polls, nullptr);
    if (r != SS_OK || n_vertices == 0) return r;
    const hipError_t e = hipStreamSynchronize(nullptr);
    if (e != hipSuccess) return set_err(SS_ERR_HIP, "hop distance probe: %s", hipGetErrorString(e));
    return SS_OK;
}

uint64_t ss_interaction_distances_workspace(uint32_t n_agents) {
    return n_agents >= kNearAgents ? near_bytes(n_agents) : (uint64_t)n_agents * 4;
}

}  // extern "C"

// Workspace of ss_interaction_distances_static (4 MiB): one array per device, held from the library's load until the process ends, shared by
// every call on that device.  Host code never uses its name as an address:
// the device address is looked up once per device (scratch_addr) and kept.
static __device__ __align__(256) unsigned scratch[1u << 20];

namespace {

// Checks the arrays of an interaction-distance call (not its workspace) and
// returns the current device in *dev.
ss_status interaction_args(const int32_t* pos_xy, const uint32_t* d_action, uint32_t n_agents,
                           uint32_t velocity, const uint32_t* out, int* dev) {
    if (n_agents >= (1u << 31)) return set_err(SS_ERR_ARG, "n_agents must be below 2^31");
    if (velocity == 0) return set_err(SS_ERR_ARG, "velocity must be >= 1");
    if (n_agents == 0) return SS_OK;
    if (!pos_xy || !d_action || !out) return set_err(SS_ERR_ARG, "NULL argument");
    if (hipGetDevice(dev) != hipSuccess) {
        (void)hipGetLastError();
        return set_err(SS_ERR_ARG, "no current device");
    }
    if (!device_range_ok(pos_xy, (u64)n_agents * 8, *dev) ||
        !device_range_ok(d_action, (u64)n_agents * 4, *dev) ||
        !device_range_ok(out, (u64)n_agents * 4, *dev))
        return set_err(SS_ERR_ARG, "every array must be device memory of the current device (%d)",
                       *dev);
    return SS_OK;
}

// All pairs on `st`: no workspace.
template <unsigned kOwn>
void pair_blocks(const PairArgs& A, hipStream_t st) {
    hipLaunchKernelGGL(k_pair<kOwn>, dim3((A.n + kOwn - 1) / kOwn), dim3(64 * kPairWaves), 0, st, A);
}

// 16 agents a workgroup up to 12,288 agents, beyond that 32: the more, smaller
// workgroups leave fewer of the 256 CUs idle (4,000 agents 6.0 against 7.7 us),
// but each reads all positions again (24,000 agents 52.7 against 49.4 us; 64 a
// workgroup 73.5 us, as some CUs then get twice the work of others).
ss_status pair_launch(const PairArgs& A, hipStream_t st) {
    if (A.n <= 12288) pair_blocks<16>(A, st);
    else pair_blocks<32>(A, st);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return set_err(SS_ERR_HIP, "interaction distance kernel: %s", hipGetErrorString(e));
    return SS_OK;
}

// The search by cells on `st`, in a workspace of near_bytes(A.n) bytes.
ss_status near_launch(const PairArgs& P, void* workspace, hipStream_t st) {
    NearArgs A{};
    A.pos = P.pos;
    A.d_action = P.d_action;
    A.out = P.out;
    A.n = P.n;
    A.velocity = P.velocity;
    A.radius = P.radius;
    A.cells = (unsigned)near_cells(A.n);
    A.rows = near_rows(A.n);
    const unsigned chunks = A.cells / kNearScan;
    A.mask = static_cast<u64*>(workspace);
    A.alloc = reinterpret_cast<unsigned*>(A.mask + kNearSide);
    A.block = reinterpret_cast<uint2*>(A.alloc + 4);
    A.sum = reinterpret_cast<unsigned*>(A.block + kNearBlocks);
    A.row = A.sum + (chunks + 3) / 4 * 4;
    A.count = A.row + (u64)A.rows * kNearBlocks;
    A.first = A.count + A.cells;
    A.cell = A.first + A.cells + 4;
    A.rank = A.cell + A.n;
    A.spos = A.rank + A.n;
    A.sid = A.spos + A.n;
    const dim3 one(kNearThreads), all((A.n + kNearThreads - 1) / kNearThreads);
    hipLaunchKernelGGL(k_near_blocks, dim3(A.rows), dim3(1024), 0, st, A);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_near_cells, dim3(kNearBlocks / 64), dim3(1024), 0, st, A);
        e = hipGetLastError();
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_near_count, all, one, 0, st, A);
        e = hipGetLastError();
    }
    if (e == hipSuccess && A.n > kNearSums) {
        hipLaunchKernelGGL(k_near_sum, dim3(chunks), dim3(1024), 0, st, A);
        e = hipGetLastError();
    }
    if (A.n <= kNearSums) A.sum = nullptr;
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_near_scan, dim3(chunks), dim3(1024), 0, st, A);
        e = hipGetLastError();
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_near_place, all, one, 0, st, A);
        e = hipGetLastError();
    }
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_near_find, all, one, 0, st, A);
        e = hipGetLastError();
    }
    if (e != hipSuccess)
        return set_err(SS_ERR_HIP, "interaction distance kernels: %s", hipGetErrorString(e));
    return SS_OK;
}

constexpr uint32_t kStaticPairAgents = 1u << 20;
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
unsigned* g_scratch_addr[kMaxDevices] = {};

// Device address of `scratch` on device `dev` (current), looked up on the
// first call per device.
ss_status scratch_addr(int dev, unsigned** out) {
    if (dev < 0 || dev >= kMaxDevices) return set_err(SS_ERR_ARG, "device %d out of range", dev);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_addr[dev]) {
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return set_err(SS_ERR_HIP, "hipGetSymbolAddress(scratch) on device %d: %s", dev,
                           hipGetErrorString(e));
        g_scratch_addr[dev] = static_cast<unsigned*>(ptr);
    }
    *out = g_scratch_addr[dev];
    return SS_OK;
}

}  // namespace

extern "C" {

ss_status ss_interaction_distances(const int32_t* pos_xy, const uint32_t* d_action,
                                   uint32_t n_agents, uint32_t velocity, uint32_t radius,
                                   uint32_t* out, void* workspace, uint64_t workspace_bytes,
                                   void* stream) {
    int dev = -1;
    ss_status st = interaction_args(pos_xy, d_action, n_agents, velocity, out, &dev);
    if (st != SS_OK || n_agents == 0) return st;
    if (!workspace) return set_err(SS_ERR_ARG, "NULL argument");
    const u64 least = (u64)n_agents * 4, full = ss_interaction_distances_workspace(n_agents);
    if (workspace_bytes < least)
        return set_err(SS_ERR_ARG, "workspace_bytes %llu < %llu", (unsigned long long)workspace_bytes,
                       (unsigned long long)least);
    // a workspace of four bytes an agent takes all pairs
    const bool near = n_agents >= kNearAgents && workspace_bytes >= full &&
                      reinterpret_cast<uintptr_t>(workspace) % 16 == 0;
    if (!device_range_ok(workspace, near ? full : least, dev))
        return set_err(SS_ERR_ARG, "every array must be device memory of the current device (%d)",
                       dev);
    const PairArgs A{pos_xy, d_action, out, n_agents, velocity, radius};
    return near ? near_launch(A, workspace, static_cast<hipStream_t>(stream))
                : pair_launch(A, static_cast<hipStream_t>(stream));
}

ss_status ss_interaction_distances_static(const int32_t* pos_xy, const uint32_t* d_action,
                                          uint32_t n_agents, uint32_t velocity, uint32_t radius,
                                          uint32_t* out, void* stream) {
    if (n_agents > kStaticPairAgents)
        return set_err(SS_ERR_ARG, "n_agents %u exceeds the %u agents of the static scratch "
                                   "(use ss_interaction_distances with a workspace)",
                       n_agents, kStaticPairAgents);
    int dev = -1;
    ss_status st = interaction_args(pos_xy, d_action, n_agents, velocity, out, &dev);
    if (st != SS_OK || n_agents == 0) return st;
    const PairArgs A{pos_xy, d_action, out, n_agents, velocity, radius};
    // the search by cells as far as its workspace fits the scratch
    if (n_agents < kNearAgents || near_bytes(n_agents) > sizeof(scratch))
        return pair_launch(A, static_cast<hipStream_t>(stream));
    unsigned* ws = nullptr;
    st = scratch_addr(dev, &ws);
    if (st != SS_OK) return st;
    return near_launch(A, ws, static_cast<hipStream_t>(stream));
}

}  // extern "C"
