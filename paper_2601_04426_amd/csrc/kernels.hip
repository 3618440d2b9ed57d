// gfx950 (CDNA4, wave64) kernels of the token-mask cache path:
//   k_build        classes of (position, token) pairs by a rule-scoped Earley recogniser, one lane per
//                  token, item sets in LDS                              (XGrammar-2 section 3.4)
//   k_build_slow   the same recogniser with larger item sets (LDS, then device memory), for lanes that overflowed
//   k_copy_masked  short tokens of a plane taken from the plane of a state they cannot tell apart (section 3.6)
//   k_copy_first_byte  tokens of a plane taken from the plane of a state that moves alike on their first byte
//   k_upload       per-call plan and tables from pinned host memory
//   k_token_records  the vocabulary by token id, when it goes to the device
//   k_clear        a fill's counter words, where the fill of the call before did not clear them
//   k_stage        the same for a build, together with the clearing of fresh rows and the chunk records
//   k_plane_summary  per built plane: bit counts, and the short list of its uncertain tokens that the fill reads
//   k_finish_planes  the copy kernels and the summary in one pass, when no derived plane leans on another derived one
//   k_fill         union of cached planes over the scannable frontier and, beside it, the re-check of the uncertain
//                  tokens against the full Earley context              (section 3.4, runtime part)
//   k_recheck_slow the re-check with larger item sets, for the tokens that overflowed the short ones
//   k_apply_*      logits of disallowed tokens := -infinity, in place    (section 2.1)
// No MFMA: nothing here is a contraction.  All device writes are vector stores or LDS/L2 atomics.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <mutex>

#include <hip/hip_ext.h>

#include "device.hpp"
#include "earley_core.hpp"
#include "accept_core.hpp"

namespace xg2 {
namespace {

using namespace core;

// ---- per-lane item storage -------------------------------------------------------------------------
// LDS: word (slot, column) lives at slot * COLS + column (a lane's column is its place among the lanes at work), so a
// wave touching one slot per lane hits every bank once per 32 lanes whatever the slots are.
template <int K_, int WM_, int COLS_ = 64>
struct LdsStore {
    static constexpr int K = K_, WM = WM_, MAXLEN = 16, COLS = COLS_, SLOTS = 2 * K_ + 2 * WM_;
    uint32_t* cur; uint32_t* nxt; uint32_t* wait;  // this lane's column of the two item lists and the wait list (two words an entry)
    unsigned long long ws_lo = 0, ws_hi = 0;        // wait-list length at the start of each new set, 8 bits each
    __device__ void init(uint32_t* base) { cur = base; nxt = base + K * COLS; wait = base + 2 * K * COLS; }
    __device__ uint32_t get_cur(int k) const { return cur[k * COLS]; }
    __device__ void set_cur(int k, uint32_t v) { cur[k * COLS] = v; }
    __device__ uint32_t get_nxt(int k) const { return nxt[k * COLS]; }
    __device__ void set_nxt(int k, uint32_t v) { nxt[k * COLS] = v; }
    __device__ uint32_t wait_rule(int k) const { return wait[k * 2 * COLS]; }
    __device__ uint32_t wait_tgt(int k) const { return wait[k * 2 * COLS + COLS]; }
    __device__ void set_wait(int k, uint32_t rule, uint32_t tgt) { wait[k * 2 * COLS] = rule; wait[k * 2 * COLS + COLS] = tgt; }
    __device__ void swap() { uint32_t* t = cur; cur = nxt; nxt = t; }
    __device__ bool charge(int) { return true; }   // short lists: nothing to bound
    __device__ void reset() { ws_lo = 0; ws_hi = 0; }
    __device__ void set_wstart(int j, uint32_t v) {
        const int sh = 8 * (j & 7);
        unsigned long long& w = j < 8 ? ws_lo : ws_hi;
        w = (w & ~(0xFFull << sh)) | ((unsigned long long)v << sh);
    }
    __device__ uint32_t get_wstart(int j) const {
        return (uint32_t)((j < 8 ? ws_lo >> (8 * j) : ws_hi >> (8 * (j - 8))) & 0xFF);
    }
};

// The same layout with more room and the set starts in LDS too: the first resort of the large-capacity kernels
// (one wave per workgroup, 37 KB), before the lists in device memory.
template <int K_, int WM_, int MAXLEN_>
struct LdsStoreWide {
    static constexpr int K = K_, WM = WM_, MAXLEN = MAXLEN_, SLOTS = 2 * K_ + 2 * WM_ + MAXLEN_ + 1;
    uint32_t* cur; uint32_t* nxt; uint32_t* wait; uint32_t* ws;
    __device__ void init(uint32_t* base) { cur = base; nxt = base + K * 64; wait = base + 2 * K * 64; ws = base + (2 * K + 2 * WM) * 64; }
    __device__ uint32_t get_cur(int k) const { return cur[k * 64]; }
    __device__ void set_cur(int k, uint32_t v) { cur[k * 64] = v; }
    __device__ uint32_t get_nxt(int k) const { return nxt[k * 64]; }
    __device__ void set_nxt(int k, uint32_t v) { nxt[k * 64] = v; }
    __device__ uint32_t wait_rule(int k) const { return wait[k * 128]; }
    __device__ uint32_t wait_tgt(int k) const { return wait[k * 128 + 64]; }
    __device__ void set_wait(int k, uint32_t rule, uint32_t tgt) { wait[k * 128] = rule; wait[k * 128 + 64] = tgt; }
    __device__ void swap() { uint32_t* t = cur; cur = nxt; nxt = t; }
    __device__ bool charge(int) { return true; }
    __device__ void reset() {}
    __device__ void set_wstart(int j, uint32_t v) { ws[j * 64] = v; }
    __device__ uint32_t get_wstart(int j) const { return ws[j * 64]; }
};
using MidStore = LdsStoreWide<16, 32, 48>;

// Device memory: word (slot, lane) lives at slot * n_lanes + lane (coalesced across lanes).
struct GlobalStore {
    static constexpr int MAXLEN = kSlowMaxLen;
    int K = kSlowK, WM = kSlowWM;                   // capacities in use (the memory is laid out for kSlowK, kSlowWM)
    uint32_t* cur; uint32_t* nxt; uint32_t* wait; uint32_t* ws; size_t stride;
    uint32_t budget = kSlowSearchBudget;           // list entries one token may still compare against: a bound on its run time
    __device__ bool charge(int n) { if ((uint32_t)n > budget) { budget = 0; return false; } budget -= (uint32_t)n; return true; }
    __device__ void init(uint32_t* base, size_t n_lanes, uint32_t k_cap = kSlowK, uint32_t wm_cap = kSlowWM) {
        K = (int)min(k_cap, kSlowK); WM = (int)min(wm_cap, kSlowWM);
        stride = n_lanes; cur = base; nxt = base + (size_t)kSlowK * stride; wait = base + (size_t)2 * kSlowK * stride;
        ws = base + (size_t)(2 * kSlowK + 2 * kSlowWM) * stride;
    }
    __device__ uint32_t get_cur(int k) const { return cur[(size_t)k * stride]; }
    __device__ void set_cur(int k, uint32_t v) { cur[(size_t)k * stride] = v; }
    __device__ uint32_t get_nxt(int k) const { return nxt[(size_t)k * stride]; }
    __device__ void set_nxt(int k, uint32_t v) { nxt[(size_t)k * stride] = v; }
    __device__ uint32_t wait_rule(int k) const { return wait[(size_t)(2 * k) * stride]; }
    __device__ uint32_t wait_tgt(int k) const { return wait[(size_t)(2 * k + 1) * stride]; }
    __device__ void set_wait(int k, uint32_t rule, uint32_t tgt) { wait[(size_t)(2 * k) * stride] = rule; wait[(size_t)(2 * k + 1) * stride] = tgt; }
    __device__ void swap() { uint32_t* t = cur; cur = nxt; nxt = t; }
    __device__ void reset() { budget = kSlowSearchBudget; }
    __device__ void set_wstart(int j, uint32_t v) { ws[(size_t)j * stride] = v; }
    __device__ uint32_t get_wstart(int j) const { return ws[(size_t)j * stride]; }
};

#ifndef XG2_BUILD_ATTR
#define XG2_BUILD_ATTR
#endif
// Item-list capacities of the LDS path with all 64 lanes at work: the host picks one of two sizes per launch (see
// launch_build); the LDS of a workgroup is sized to match.
#ifndef XG2_BUILD_K_SMALL
#define XG2_BUILD_K_SMALL 3
#define XG2_BUILD_WM_SMALL 4
#endif
#ifndef XG2_BUILD_LEVELS
#define XG2_BUILD_LEVELS 3
#endif
constexpr int BUILD_LEVELS = XG2_BUILD_LEVELS;        // 64, 32, 16, ... lanes at work with 1, 2, 4, ... times the capacity
constexpr int BUILD_K_SMALL = XG2_BUILD_K_SMALL, BUILD_WM_SMALL = XG2_BUILD_WM_SMALL, BUILD_K_LARGE = 6, BUILD_WM_LARGE = 10;

// The build kernel's item lists: the LDS layout above with capacities chosen at run time.  The lists are kept short
// because their size bounds how many workgroups a compute unit holds, and the kernel lives on hiding the latency of
// dependent table loads behind other wavefronts.  A token that outgrows them is run again with only the lower 32 lanes
// at work, each with two lanes' worth of the same memory (word (slot, lane) at slot * 32 + lane): twice the capacity,
// no more LDS; one that outgrows those too, once more with 16 lanes and four times the capacity (BUILD_LEVELS).
struct BuildStore {
    static constexpr int MAXLEN = 16;
    int K, WM, sh;                                  // capacities; log2 of the distance between a lane's consecutive slots
    uint32_t* cur; uint32_t* nxt; uint32_t* wait;
    unsigned long long ws_lo = 0, ws_hi = 0;        // wait-list length at the start of each new set, 8 bits each
    // lds: the workgroup's (2 k + 2 wm) * 64 words for lists of k items and wm wait entries a lane; level l: lanes
    // 0 .. (64 >> l) - 1 only, 2^l times the capacity
    __device__ void init(uint32_t* lds, uint32_t lane, int k, int wm, int level) {
        K = k << level; WM = wm << level; sh = 6 - level;
        cur = lds + lane; nxt = lds + k * 64 + lane; wait = lds + 2 * k * 64 + lane;
    }
    __device__ uint32_t get_cur(int k) const { return cur[k << sh]; }
    __device__ void set_cur(int k, uint32_t v) { cur[k << sh] = v; }
    __device__ uint32_t get_nxt(int k) const { return nxt[k << sh]; }
    __device__ void set_nxt(int k, uint32_t v) { nxt[k << sh] = v; }
    __device__ uint32_t wait_rule(int k) const { return wait[(2 * k) << sh]; }
    __device__ uint32_t wait_tgt(int k) const { return wait[(2 * k + 1) << sh]; }
    __device__ void set_wait(int k, uint32_t rule, uint32_t tgt) { wait[(2 * k) << sh] = rule; wait[(2 * k + 1) << sh] = tgt; }
    __device__ void swap() { uint32_t* t = cur; cur = nxt; nxt = t; }
    __device__ bool charge(int) { return true; }
    __device__ void reset() { ws_lo = 0; ws_hi = 0; }
    __device__ void set_wstart(int j, uint32_t v) {
        const int s8 = 8 * (j & 7);
        unsigned long long& w = j < 8 ? ws_lo : ws_hi;
        w = (w & ~(0xFFull << s8)) | ((unsigned long long)v << s8);
    }
    __device__ uint32_t get_wstart(int j) const {
        return (uint32_t)((j < 8 ? ws_lo >> (8 * j) : ws_hi >> (8 * (j - 8))) & 0xFF);
    }
};

__device__ __forceinline__ void push_overflow(const SlowScratch& S, uint32_t a, uint32_t b) {
    uint32_t idx = atomicAdd(S.count, 1u);
    if (idx < S.list_cap) { S.list[2 * idx] = a; S.list[2 * idx + 1] = b; }
    else atomicOr(S.count + 1, 1u);
}

// The same for a fill: no room left is the caller's business.
__device__ __forceinline__ bool try_push(const SlowScratch& S, uint32_t b, uint32_t id) {
    if (*reinterpret_cast<volatile uint32_t*>(S.count) >= S.list_cap) return false;      // (the count does not run on and on)
    const uint32_t at = atomicAdd(S.count, 1u);
    if (at >= S.list_cap) return false;
    S.list[2 * at] = b; S.list[2 * at + 1] = id;
    return true;
}

__device__ __forceinline__ DevCtx position_ctx(const BuildPlan& P, uint32_t p) {
    const uint4 d = P.plane_ctx[p];
    DevCtx C;
    C.items = P.ctx_items + d.x;
    C.n_items = d.y;
    C.wait = P.ctx_wait;
    C.wait_off = P.ctx_wait_off + d.z;
    C.H = d.w;
    return C;
}

__device__ __forceinline__ void store_class(uint32_t* row, uint32_t W, uint32_t id, int res) {
    if (res & RES_ALIVE) atomicOr(row + (id >> 5), 1u << (id & 31));
    else if (res & RES_EARLY) atomicOr(row + W + (id >> 5), 1u << (id & 31));
}
__device__ __forceinline__ void store_class(const BuildPlan& P, uint32_t p, uint32_t W, uint32_t id, int res) {
    store_class(P.plane_ptr[p], W, id, res);
}
// The third row of a plane: the tokens that left the outermost rule early and then died, whatever the follow filter
// makes of them (with the filter off this is the uncertain row again).  It is what a plane of the same structure under
// another follow language is derived from (section 3.3: partial cache hit).
__device__ __forceinline__ void store_left_early(uint32_t* row, uint32_t W, uint32_t id) {
    atomicOr(row + 2 * W + (id >> 5), 1u << (id & 31));
}

// A persistent grid of single-wave workgroups: workgroup g handles chunks g, g + grid, g + 2 grid, ...
// (sorted ranks of one plane each; the host puts the long ones first), each in phases, so that the long
// divergent steps of the recogniser run on full waves instead of on the few lanes that need them.
// Phase 1 (when the plane's start set is a single item without rule edges, or one or two such items whose
// ends lead back into the outermost instance): every lane walks its token through the automaton, one table
// load per byte and thread.  A token that dies is rejected, one that reaches its end is accepted; one that
// reaches a state which predicts, or which completes a rule instance in a way the walk does not follow, goes
// on the deferred list.  One that dies after the outermost instance could have ended is what the plain run
// would call "left early": it goes straight to the follow-language run (or is stored as uncertain when that
// run is switched off).  Phase 2: the deferred tokens (for the other planes: all tokens of the chunk), 64 at
// a time, through the Earley recogniser.  Tokens that leave the outermost rule early and then die need the
// second, follow-language run; they are collected across chunks as (plane, rank) pairs and run 64 at a time too.
__device__ __forceinline__ void follow_batch(const DevTables& T, const DevVocab& Vd, const BuildPlan& P, const SlowScratch& S,
                                          const uint32_t* cls_words, uint32_t* lds, uint32_t* f_plane, uint32_t* f_rank,
                                          uint32_t first, uint32_t count, uint32_t lane) {
    // level 0: the batch, one token a lane; further levels: the tokens that outgrew the lists of the level before, half as
    // many at a time with twice the room (their entries have moved to the front of the batch's part of the queue, which
    // has been read)
    uint32_t cnt = count;
    for (int level = 0; level < BUILD_LEVELS && cnt; ++level) {
        const uint32_t lanes = 64u >> level;
        const bool last = level == BUILD_LEVELS - 1;
        uint32_t n_next = 0;
        for (uint32_t off = 0; off < cnt; off += lanes) {
            BuildStore st;
            st.init(lds, lane, (int)P.list_k, (int)P.list_wm, level);
            bool over = false;
            uint32_t p = 0, rank = 0;
            if (lane < lanes && off + lane < cnt) {
                p = f_plane[first + off + lane]; rank = f_rank[first + off + lane];
                const DevCtx C = position_ctx(P, p);
                const int n = (int)(Vd.off[rank + 1] - Vd.off[rank]);
                RegBytes tok;
                tok.v = Vd.tok16[rank];
                const int res = scan_token<BuildStore, true>(T, cls_words, C, tok, n, st);
                over = res & RES_OVERFLOW;
                if (over && last) push_overflow(S, p, rank);        // the large-capacity kernel takes it
                else if (res & RES_ALIVE) store_class(P, p, Vd.W, Vd.perm[rank], RES_EARLY);   // some context can take the rest: uncertain
            }
            if (!last) {
                const unsigned long long mo = __ballot(over);
                if (mo) {
                    __syncthreads();
                    if (over) {
                        const uint32_t at = first + n_next + (uint32_t)__popcll(mo & ((1ull << lane) - 1));
                        f_plane[at] = p; f_rank[at] = rank;
                    }
                    __syncthreads();
                    n_next += (uint32_t)__popcll(mo);
                }
            }
        }
        cnt = n_next;
    }
}

__global__ __launch_bounds__(64) XG2_BUILD_ATTR void k_build(DevTables T, DevVocab Vd, BuildPlan P, SlowScratch S) {
    extern __shared__ uint32_t lds[];                               // the item lists: (2 K + 2 WM) * 64 words, sized by the launch
    __shared__ uint32_t cls_words[64];                              // byte -> class, four a word
    const uint8_t* cls_bytes = reinterpret_cast<const uint8_t*>(cls_words);   // the same table, one byte an entry
    __shared__ uint8_t deferred[kBuildChunk];                       // tokens of the chunk for phase 2, as offsets from the chunk's first rank
    __shared__ uint32_t f_plane[128], f_rank[128];
    const uint32_t lane = threadIdx.x;
    cls_words[lane] = T.byte_class_words[lane];
    uint32_t n_follow = 0;                                          // same in every lane
    for (uint32_t chunk_idx = blockIdx.x; chunk_idx < P.n_chunks; chunk_idx += gridDim.x) {
        __syncthreads();                                            // one wave: orders the LDS traffic of the phases
        const uint4 chunk = P.chunk[2 * chunk_idx], chunk_b = P.chunk[2 * chunk_idx + 1];   // one 32-byte record: nothing else is loaded before the walk
        const uint32_t p = chunk.x;
        const uint32_t item0 = chunk_b.x;
        uint32_t* const row = reinterpret_cast<uint32_t*>(((uint64_t)chunk_b.w << 32) | chunk_b.z);
        // same for the whole chunk; that the start state itself can end its rule does not matter to a token (it has a byte)
        const bool walkable = chunk_b.y == 1 && (item0 & (F_BYTE | F_REF)) == F_BYTE;
        const bool root_instance = (item0 >> REF_BITS) == ROOT_ORIGIN;   // the start item is the plane's outermost rule instance
        const bool listed = chunk.w & kChunkListed;                 // ranks come from a list of long tokens
        const bool threaded = chunk.w & kChunkThreads;              // two thread descriptors follow the plane's items
        uint32_t n_work = chunk.z - chunk.y;
        // a token that left the outermost rule early and died: queued for the follow-language run, which starts
        // when 64 of them are there (`again` differs between lanes; everything else here is the same in all)
        auto queue_follow = [&](bool again, uint32_t rank) {
            const unsigned long long m = __ballot(again);
            if (!m) return;
            if (again) {
                const uint32_t at = n_follow + (uint32_t)__popcll(m & ((1ull << lane) - 1));
                f_plane[at] = p; f_rank[at] = rank;
            }
            n_follow += (uint32_t)__popcll(m);
            __syncthreads();
            if (n_follow >= 64) {
                n_follow -= 64;
                follow_batch(T, Vd, P, S, cls_words, lds, f_plane, f_rank, n_follow, 64, lane);
                __syncthreads();
            }
        };
        // what phase 1 does with such a token: the plain run would end dead with the early mark, so it is not made
        auto died_early = [&](bool yes, uint32_t rank) {
            if (yes) {
                const uint32_t id = Vd.perm[rank];
                store_left_early(row, Vd.W, id);
                if (!P.follow_filter) { store_class(row, Vd.W, id, RES_EARLY); yes = false; }
            }
            queue_follow(yes, rank);
        };
        if (chunk.w & kChunkDerive) {
            // partial cache hit: the plane's accepted row comes from a plane of the same structure built under another follow
            // language (copied by another kernel); of its tokens that left early and died -- mask words chunk.y .. chunk.z of
            // that plane's third row, one a lane -- those that this grammar's follow language can continue are uncertain here
            const uint32_t* base_left = reinterpret_cast<const uint32_t*>(((uint64_t)chunk_b.w << 32) | chunk_b.z);
            const uint32_t w = chunk.y + lane;
            uint32_t bits = w < chunk.z ? base_left[w] : 0u;
            while (__any(bits != 0)) {
                uint32_t rank = 0xFFFFFFFFu;
                if (bits) {
                    const uint32_t bit = (uint32_t)__ffs(bits) - 1;
                    bits &= bits - 1;
                    rank = Vd.rank[w * 32 + bit];
                }
                queue_follow(rank < Vd.n_sorted, rank);
            }
            continue;
        }
        if (walkable) {
            n_work = 0;
            for (uint32_t rank0 = chunk.y; rank0 < chunk.z; rank0 += 64) {
                uint32_t rank = rank0 + lane;
                int n = 0;
                uint4 tv = make_uint4(0, 0, 0, 0);
                if (rank < chunk.z) {
                    if (listed) rank = Vd.long_rank[rank];
                    n = (int)(Vd.off[rank + 1] - Vd.off[rank]); tv = Vd.tok16[rank];
                }
                bool defer = n > BuildStore::MAXLEN;                 // phase 2 hands it to the large-capacity kernel
                if (defer) n = 0;
                const WalkResult r = root_instance ? walk_tokens<true>(T.trans, T.n_classes, T.sink, cls_bytes, item0 & REF_MASK, tv, n)
                                                   : walk_tokens<false>(T.trans, T.n_classes, T.sink, cls_bytes, item0 & REF_MASK, tv, n);
                // a state that predicts, or that completes into a parent, is where the walk hands over to the recogniser
                defer |= n > 0 && (r.seen & (root_instance ? F_REF : (F_REF | F_FINAL))) != 0;
                const bool dead = r.state == T.sink;
                if (n > 0 && !dead && !defer) store_class(row, Vd.W, Vd.perm[rank], RES_ALIVE);      // reached its end alive
                // dead: rejected, unless the outermost rule could have ended on the way
                died_early(root_instance && n > 0 && dead && !defer && (r.seen_before_last & F_FINAL), rank);
                const unsigned long long m = __ballot(defer);
                if (defer) deferred[n_work + (uint32_t)__popcll(m & ((1ull << lane) - 1))] = (uint8_t)(rank0 + lane - chunk.y);
                n_work += (uint32_t)__popcll(m);
            }
            __syncthreads();
        } else if (threaded) {
            // Phase 1 for a start set of one or two scanning items that do not predict: each item is an automaton
            // thread; a thread of a waited-for instance that reaches a final state starts one thread of the outermost
            // instance at the state the host has looked up.  Three slots; anything else (a state that predicts, a
            // fourth thread) goes to phase 2.
            const uint4 pc = P.plane_ctx[p];
            const uint32_t* d = P.ctx_items + pc.x + pc.y;
            const uint32_t it_a = d[0], lead_a = d[1], it_b = d[2], lead_b = d[3];
            n_work = 0;
            for (uint32_t rank0 = chunk.y; rank0 < chunk.z; rank0 += 64) {
                uint32_t rank = rank0 + lane;
                bool defer = false;
                int n = 0;
                RegBytes tok;
                tok.v = make_uint4(0, 0, 0, 0);
                if (rank < chunk.z) {
                    if (listed) rank = Vd.long_rank[rank];
                    n = (int)(Vd.off[rank + 1] - Vd.off[rank]); tok.v = Vd.tok16[rank];
                }
                if (n > BuildStore::MAXLEN) { defer = true; n = 0; }
                uint32_t s0 = n > 0 ? it_a : kNoThread, s1 = n > 0 ? it_b : kNoThread, s2 = kNoThread;
                bool early = false;
                for (int i = 0; __any(i < n && !defer && (s0 & s1 & s2) != kNoThread); ++i) {
                    if (i < n && !defer && (s0 & s1 & s2) != kNoThread) {
                        const uint32_t cls = cls_bytes[tok.next()];
                        const bool more = i + 1 < n;
                        uint32_t start_a = kNoThread, start_b = kNoThread;
                        auto step = [&](uint32_t& s, uint32_t lead, uint32_t& start) {
                            if (s == kNoThread) return;
                            const uint32_t tgt = T.trans[(s & SID_MASK) * T.n_classes + cls];
                            if (tgt == T.sink) { s = kNoThread; return; }
                            if (tgt & F_REF) { defer = true; return; }
                            s = tgt | (s & ~REF_MASK);
                            if (tgt & F_FINAL) {
                                if ((s >> REF_BITS) == ROOT_ORIGIN) early |= more;
                                else start = lead;
                            }
                        };
                        uint32_t none = kNoThread;
                        step(s0, lead_a, start_a);
                        step(s1, lead_b, start_b);
                        step(s2, 0u, none);                          // only threads of the outermost instance get here
                        auto begin = [&](uint32_t item) {
                            if (item == kNoThread) return;
                            if (item & F_FINAL) early |= more;
                            if (item == s0 || item == s1 || item == s2) return;
                            if (s2 == kNoThread) s2 = item;
                            else if (s1 == kNoThread) s1 = item;
                            else if (s0 == kNoThread) s0 = item;
                            else defer = true;
                        };
                        begin(start_a);
                        begin(start_b);
                    }
                }
                bool dead_early = false;
                if (n > 0 && !defer) {
                    if ((s0 & s1 & s2) != kNoThread) store_class(row, Vd.W, Vd.perm[rank], RES_ALIVE);
                    else dead_early = early;
                }
                died_early(dead_early, rank);
                const unsigned long long m = __ballot(defer);
                if (defer) deferred[n_work + (uint32_t)__popcll(m & ((1ull << lane) - 1))] = (uint8_t)(rank0 + lane - chunk.y);
                n_work += (uint32_t)__popcll(m);
            }
            __syncthreads();
        }
        if (n_work == 0) continue;
        const DevCtx C = position_ctx(P, p);                        // only the recogniser needs the whole start set
        for (uint32_t base = 0; base < n_work; base += 64) {
            // level 0: 64 tokens of the list, one a lane; further levels: those of them that outgrew the item lists of the
            // level before, half as many at a time with twice the room (their offsets go through the part of the deferred
            // list that this batch has read)
            uint32_t cnt = min(64u, n_work - base);
            for (int level = 0; level < BUILD_LEVELS && cnt; ++level) {
                const uint32_t lanes = 64u >> level;
                const bool last = level == BUILD_LEVELS - 1;
                uint32_t n_next = 0;
                for (uint32_t off = 0; off < cnt; off += lanes) {
                    BuildStore st;
                    st.init(lds, lane, (int)P.list_k, (int)P.list_wm, level);
                    bool again = false, over = false;
                    uint32_t rank = 0, at = 0;                       // the token: sorted rank, and offset in the chunk
                    if (lane < lanes && off + lane < cnt) {
                        const uint32_t idx = base + off + lane;
                        at = (level > 0 || walkable || threaded) ? deferred[idx] : idx;
                        rank = listed ? Vd.long_rank[chunk.y + at] : chunk.y + at;
                        const int n = (int)(Vd.off[rank + 1] - Vd.off[rank]);
                        RegBytes tok;
                        tok.v = Vd.tok16[rank];
                        const int res = scan_token(T, cls_words, C, tok, n, st);
                        over = res & RES_OVERFLOW;
                        if (over && last) push_overflow(S, p, rank); // the large-capacity kernel takes it
                        else if (!over) {
                            // leaves the rule early and dies: it stays uncertain only if some context can take the rest of the token
                            const bool left_early = !(res & RES_ALIVE) && (res & RES_EARLY);
                            again = P.follow_filter && left_early;
                            if (left_early || !again) {
                                const uint32_t id = Vd.perm[rank];
                                if (left_early) store_left_early(row, Vd.W, id);
                                if (!again) store_class(row, Vd.W, id, res);
                            }
                        }
                    }
                    queue_follow(again, rank);
                    if (!last) {
                        const unsigned long long mo = __ballot(over);
                        if (mo) {
                            __syncthreads();
                            if (over) deferred[base + n_next + (uint32_t)__popcll(mo & ((1ull << lane) - 1))] = (uint8_t)at;
                            __syncthreads();
                            n_next += (uint32_t)__popcll(mo);
                        }
                    }
                }
                cnt = n_next;
            }
        }
    }
    __syncthreads();
    if (n_follow) follow_batch(T, Vd, P, S, cls_words, lds, f_plane, f_rank, 0, n_follow, lane);
}

// Both runs of one (plane, token) pair with the lists in `st`: the plain one and, if the token left the outermost
// rule early and died, the follow-language one.
template <class S>
__device__ int classify_slow(const DevTables& T, const DevVocab& Vd, const BuildPlan& P, const DevCtx& C, uint32_t off, int n, S& st) {
    st.reset();
    MemBytes tok{Vd.bytes + off};
    int res = scan_token<S, false, MemBytes>(T, T.byte_class_words, C, tok, n, st);
    if (!(res & (RES_ALIVE | RES_OVERFLOW)) && (res & RES_EARLY)) res |= RES_LEFT_EARLY;
    if (P.follow_filter && (res & RES_LEFT_EARLY)) {
        st.reset();
        int res2 = scan_token<S, true, MemBytes>(T, T.byte_class_words, C, tok, n, st);
        if (res2 & RES_OVERFLOW) res = RES_OVERFLOW;
        else if (!(res2 & RES_ALIVE)) res = RES_LEFT_EARLY;
    }
    return res;
}

__global__ __launch_bounds__(64) void k_build_slow(DevTables T, DevVocab Vd, BuildPlan P, SlowScratch S) {
    __shared__ uint32_t lds[MidStore::SLOTS * 64];
    const uint32_t gl = blockIdx.x * 64 + threadIdx.x;
    uint32_t count = S.count[0];
    if (count > S.list_cap) count = S.list_cap;
    MidStore mid;
    mid.init(lds + threadIdx.x);
    GlobalStore st;
    st.init(S.mem + gl, S.n_lanes, S.k_cap, S.wm_cap);
    for (uint32_t idx = gl; idx < count; idx += S.n_lanes) {
        if (*reinterpret_cast<volatile uint32_t*>(S.count + 1) & 2u) break;      // the build fails anyway: do not spend more on it
        const uint32_t p = S.list[2 * idx], rank = S.list[2 * idx + 1];
        const uint32_t off = Vd.off[rank];
        const int n = (int)(Vd.off[rank + 1] - off);
        DevCtx C = position_ctx(P, p);
        int res = S.k_cap >= (uint32_t)MidStore::K ? classify_slow(T, Vd, P, C, off, n, mid) : RES_OVERFLOW;   // (overflows at once if the token is too long for it)
        if (res & RES_OVERFLOW) res = classify_slow(T, Vd, P, C, off, n, st);
        if (res & RES_OVERFLOW) { atomicOr(S.count + 1, 2u); continue; }
        const uint32_t id = Vd.perm[rank];
        if (res & RES_LEFT_EARLY) store_left_early(P.plane_ptr[p], Vd.W, id);
        store_class(P, p, Vd.W, id, res);
    }
}

// Copies n 16-byte words from pinned host memory (read through its device address) to device memory: the per-call plan,
// tables and per-row records travel this way, without a trip through the copy engine.
__global__ __launch_bounds__(256) void k_upload(uint4* dst, const uint4* src, size_t n, uint64_t* stamp) {
    if (stamp && blockIdx.x == 0 && threadIdx.x == 0) *stamp = wall_clock64();
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) dst[i] = src[i];
}

// The vocabulary's records by token id, from its arrays by sorted rank.
__global__ __launch_bounds__(256) void k_token_records(DevVocab Vd, TokenRecord* rec) {
    const uint32_t id = blockIdx.x * 256 + threadIdx.x;
    if (id >= Vd.V) return;
    TokenRecord t{};
    const uint32_t rank = Vd.rank[id];
    if (rank < Vd.n_sorted) { t.head = Vd.tok16[rank]; t.off = Vd.off[rank]; t.n_bytes = Vd.off[rank + 1] - t.off; }
    rec[id] = t;
}

__global__ __launch_bounds__(64) void k_clear(uint32_t* words, uint32_t n) {
    if (threadIdx.x < n) words[threadIdx.x] = 0;
}

__device__ __forceinline__ void expand_range(const uint4* range_a, const uint4* range_b, const uint32_t* first, uint32_t r, uint4* chunk) {
    const uint4 a = range_a[r], b = range_b[r];
    const uint32_t step = a.w >> kChunkStepShift;
    uint4* out = chunk + 2 * (size_t)first[r];
    for (uint32_t lo = a.y; lo < a.z; lo += step, out += 2) {
        out[0] = make_uint4(a.x, lo, min(a.z, lo + step), a.w);
        out[1] = b;
    }
}

__global__ __launch_bounds__(256) void k_expand_chunks(const uint4* range_a, const uint4* range_b, const uint32_t* first, uint32_t n_ranges, uint4* chunk) {
    const uint32_t r = blockIdx.x * 256 + threadIdx.x;
    if (r < n_ranges) expand_range(range_a, range_b, first, r, chunk);
}

// Everything a build needs before its first kernel, in one launch of three independent parts: workgroups [0, nb_up) copy
// the plan (and tables) from pinned host memory, the next nb_zero clear the rows that the pool hands out for the first
// time, the rest write the chunk records, reading their ranges from the pinned host copy (not from the device copy that
// the first part is still writing).
__global__ __launch_bounds__(256) void k_stage(uint4* dst, const uint4* src, size_t n_up, uint32_t nb_up, StageZero Z, uint32_t nb_zero,
                                               const uint4* range_a, const uint4* range_b, const uint32_t* first, uint32_t n_ranges, uint4* chunk) {
    if (blockIdx.x < nb_up) {
        for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n_up; i += (size_t)nb_up * 256) dst[i] = src[i];
    } else if (blockIdx.x < nb_up + nb_zero) {
        const size_t t = (size_t)(blockIdx.x - nb_up) * 256 + threadIdx.x, stride = (size_t)nb_zero * 256;
        for (uint32_t k = 0; k < Z.n; ++k) {
            uint32_t* p = Z.p[k];
            const size_t words = Z.words[k];
            if ((reinterpret_cast<uintptr_t>(p) & 15) == 0) {
                uint4* p4 = reinterpret_cast<uint4*>(p);
                for (size_t i = t; i < words / 4; i += stride) p4[i] = make_uint4(0, 0, 0, 0);
                for (size_t i = (words & ~(size_t)3) + t; i < words; i += stride) p[i] = 0u;
            } else {
                for (size_t i = t; i < words; i += stride) p[i] = 0u;
            }
        }
    } else {
        const uint32_t r = (blockIdx.x - nb_up - nb_zero) * 256 + threadIdx.x;
        if (r < n_ranges) expand_range(range_a, range_b, first, r, chunk);
    }
}

__global__ __launch_bounds__(256) void k_copy_masked(const CopyJob* jobs, uint32_t W) {
    const CopyJob j = jobs[blockIdx.y];
    const uint32_t w = blockIdx.x * 256 + threadIdx.x;
    if (w >= W) return;
    const uint32_t m = j.mask[w];
    if (!m) return;
    j.dst[w] |= j.src[w] & m;
    j.dst[W + w] |= j.src[W + w] & m;
    j.dst[2 * W + w] |= j.src[2 * W + w] & m;
}

__global__ __launch_bounds__(256) void k_copy_first_byte(const FirstByteCopyJob* jobs, const uint8_t* first_byte, uint32_t W) {
    __shared__ uint32_t bytes[8];
    const FirstByteCopyJob* j = jobs + blockIdx.y;
    if (threadIdx.x < 8) bytes[threadIdx.x] = j->bytes[threadIdx.x];
    __syncthreads();
    const uint32_t w = blockIdx.x * 256 + threadIdx.x;
    if (w >= W) return;
    const uint32_t* src = j->src;
    uint32_t* dst = j->dst;
    const uint32_t a = src[w], u = src[W + w], e = src[2 * W + w];
    uint32_t todo = a | u | e, m = 0;                               // only the tokens the source has a bit for matter
    while (todo) {
        const uint32_t bit = __ffs(todo) - 1;
        todo &= todo - 1;
        const uint32_t b = first_byte[w * 32 + bit];
        m |= ((bytes[b >> 5] >> (b & 31)) & 1u) << bit;
    }
    if (a & m) dst[w] |= a & m;
    if (u & m) dst[W + w] |= u & m;
    if (e & m) dst[2 * W + w] |= e & m;
}

// Partial cache hit: the accepted row and the left-early row of a plane are those of the plane it is derived from.
__global__ __launch_bounds__(256) void k_copy_structure(const CopyJob* jobs, uint32_t W) {
    const CopyJob j = jobs[blockIdx.y];
    const uint32_t w = blockIdx.x * 256 + threadIdx.x;
    if (w >= W) return;
    j.dst[w] = j.src[w];
    j.dst[2 * W + w] = j.src[2 * W + w];
}

// Per plane: set bits of the accepted and of the uncertain row, and the plane's list of uncertain tokens behind its
// three rows: word 0 = how many (the list holds them if that is at most kUncListWords - 1), then their token ids in no
// particular order.
__global__ __launch_bounds__(256) void k_plane_summary(uint32_t* const* plane_ptr, uint32_t n_pos, uint32_t W, uint32_t* counts) {
    __shared__ uint32_t part[2][4];
    __shared__ uint32_t n_list;
    const uint32_t p = blockIdx.x;
    if (p >= n_pos) return;
    uint32_t* row = plane_ptr[p];
    uint32_t* list = row + 3 * (size_t)W;
    if (threadIdx.x == 0) n_list = 0;
    __syncthreads();
    uint32_t a = 0, u = 0;
    for (uint32_t w = threadIdx.x; w < W; w += blockDim.x) {
        const uint32_t aw = row[w], uw = row[W + w];
        a += __popc(aw); u += __popc(uw);
        uint32_t c = uw & ~aw;
        if (c) {
            uint32_t at = atomicAdd(&n_list, (uint32_t)__popc(c));
            for (; c; c &= c - 1, ++at)
                if (at < kUncListWords - 1) list[1 + at] = w * 32 + (uint32_t)__ffs(c) - 1;
        }
    }
    for (int s = 32; s > 0; s >>= 1) { a += __shfl_down(a, s); u += __shfl_down(u, s); }
    if ((threadIdx.x & 63) == 0) { part[0][threadIdx.x >> 6] = a; part[1][threadIdx.x >> 6] = u; }
    __syncthreads();
    if (threadIdx.x == 0) {
        counts[2 * p] = part[0][0] + part[0][1] + part[0][2] + part[0][3];
        counts[2 * p + 1] = part[1][0] + part[1][1] + part[1][2] + part[1][3];
        list[0] = n_list;
    }
}

// The copies of the derived planes and the summary in one pass: a plane's words are read once, completed from the
// planes it takes bits from, written back where they changed, and counted and listed from the registers.  A workgroup
// takes FINISH_WORDS words of one plane; the plane's counts and the length of its list are summed with one device atomic
// per workgroup each (they start at zero: the counts arrive as zeros with the plan, the list with the cleared row).
constexpr uint32_t FINISH_ITER = 4, FINISH_WORDS = 256 * FINISH_ITER;
__global__ __launch_bounds__(256) void k_finish_planes(uint32_t* const* plane_ptr, const FinishJob* jobs, uint32_t n_pos, const uint8_t* first_byte,
                                                       uint32_t W, uint32_t* counts) {
    __shared__ uint32_t part[2][4];
    __shared__ uint32_t n_list, list_base;
    __shared__ uint32_t bytes[8];
    const uint32_t p = blockIdx.y;
    uint32_t* row = plane_ptr[p];
    uint32_t* list = row + 3 * (size_t)W;
    const FinishJob* job = jobs + p;
    const uint32_t* m_src = job->m_src;
    const uint32_t* m_mask = job->m_mask;
    const uint32_t* f_src = job->f_src;
    if (threadIdx.x == 0) n_list = 0;
    if (threadIdx.x < 8) bytes[threadIdx.x] = job->f_bytes[threadIdx.x];
    __syncthreads();
    uint32_t na = 0, nu = 0, cand[FINISH_ITER], at[FINISH_ITER];
#pragma unroll
    for (uint32_t it = 0; it < FINISH_ITER; ++it) {
        const uint32_t w = blockIdx.x * FINISH_WORDS + it * 256 + threadIdx.x;
        cand[it] = 0; at[it] = 0;
        if (w >= W) continue;
        const uint32_t a0 = row[w], u0 = row[W + w];
        uint32_t a = a0, u = u0, e = 0;                             // e: bits to add to the third row (it is not read for a plane that takes none)
        if (m_src) {
            const uint32_t m = m_mask[w];
            if (m) { a |= m_src[w] & m; u |= m_src[W + w] & m; e |= m_src[2 * W + w] & m; }
        }
        if (f_src) {
            const uint32_t sa = f_src[w], su = f_src[W + w], se = f_src[2 * W + w];
            uint32_t todo = sa | su | se, m = 0;                    // only the tokens the source has a bit for matter
            while (todo) {
                const uint32_t bit = __ffs(todo) - 1;
                todo &= todo - 1;
                const uint32_t b = first_byte[w * 32 + bit];
                m |= ((bytes[b >> 5] >> (b & 31)) & 1u) << bit;
            }
            a |= sa & m; u |= su & m; e |= se & m;
        }
        if (a != a0) row[w] = a;
        if (u != u0) row[W + w] = u;
        if (e) { const uint32_t e0 = row[2 * W + w]; if (e & ~e0) row[2 * W + w] = e0 | e; }
        na += __popc(a); nu += __popc(u);
        cand[it] = u & ~a;
        if (cand[it]) at[it] = atomicAdd(&n_list, (uint32_t)__popc(cand[it]));
    }
    for (int s = 32; s > 0; s >>= 1) { na += __shfl_down(na, s); nu += __shfl_down(nu, s); }
    if ((threadIdx.x & 63) == 0) { part[0][threadIdx.x >> 6] = na; part[1][threadIdx.x >> 6] = nu; }
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t ta = part[0][0] + part[0][1] + part[0][2] + part[0][3], tu = part[1][0] + part[1][1] + part[1][2] + part[1][3];
        if (ta) atomicAdd(counts + 2 * p, ta);
        if (tu) atomicAdd(counts + 2 * p + 1, tu);
        list_base = n_list ? atomicAdd(list, n_list) : 0u;           // word 0 of the list: how many uncertain tokens the plane has
    }
    __syncthreads();
    if (n_list == 0) return;
#pragma unroll
    for (uint32_t it = 0; it < FINISH_ITER; ++it) {
        const uint32_t w = blockIdx.x * FINISH_WORDS + it * 256 + threadIdx.x;
        uint32_t k = list_base + at[it];
        for (uint32_t c = cand[it]; c; c &= c - 1, ++k)
            if (k < kUncListWords - 1) list[1 + k] = w * 32 + (uint32_t)__ffs(c) - 1;
    }
}

// ---- one token, one wavefront -----------------------------------------------------------------------
__device__ __forceinline__ uint32_t lane_value(uint32_t v, uint32_t k) { return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)k); }
// A value that is the same in all lanes, as the compiler cannot know where it came from memory.
__device__ __forceinline__ uint32_t same_in_all(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
// A load whose address is the same in all lanes, from memory that no kernel writes while this one runs: the scalar cache
// serves it, and the compiler knows that the value is uniform.  Word by word (the compiler joins them): a struct copied as such
// is fetched by vector loads, and every use of a pointer in it then pays for bringing it back to scalar registers.
template <class P>
__device__ __forceinline__ P uniform_load(const P* p) {
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(sizeof(P) % 4 == 0, "scalar loads are of words");
    const auto* q = (const __attribute__((address_space(4))) uint32_t*)p;
    uint32_t w[sizeof(P) / 4];
    _Pragma("unroll") for (unsigned k = 0; k < sizeof(P) / 4; ++k) w[k] = q[k];
    P v;
    __builtin_memcpy(&v, w, sizeof(P));
    return v;
#else
    return *p;
#endif
}
// Values that are wanted here: loads whose results are named are asked for before this point, all together, and not one after the
// other where the compiler would rather have them (behind the branch on an earlier one).
#if defined(__HIP_DEVICE_COMPILE__)
#define PIN(...) asm volatile("" : __VA_ARGS__)
#else
#define PIN(...) (void)0
#endif
// What a kernel was launched with, read anew from the launch's own memory (A: the struct that follows two pointers among its
// arguments): what only a way that is rarely taken needs must not take up registers on the way that nearly every row or token goes.
// The two pointers are those that a kernel's first loads need: the device has them in registers when it starts (build.py says how
// many words of arguments), where a load of them takes 560 - 700 cycles of the slowest row's chain.  (The
// decoding steps of 16 rows of tools, 64 of a JSON schema and 256 of tools 16.96 / 19.1 / 57.7 -> 16.7 / 18.8 / 57.1 us.)
template <class A>
__device__ __forceinline__ A args_again() {
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(alignof(A) == 8, "the struct lies right behind the two pointers");
    auto p = (const __attribute__((address_space(4))) A*)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() + 16);
    asm volatile("" : "+s"(p));
    return *p;
#else
    return A{};
#endif
}
// The lanes in which x holds: one compare.  (Of two conditions joined by && the compiler makes three vector instructions more than of
// two sets of lanes joined by &.)
__device__ __forceinline__ unsigned long long lanes_of(bool x) { return __builtin_amdgcn_ballot_w64(x); }
// Sets of lanes as 64 bits: whether this lane is one of them, how many of them are below it, and n < 64 lanes from `first` on.
__device__ __forceinline__ bool has_lane(unsigned long long m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
__device__ __forceinline__ uint32_t count_below(unsigned long long m) { return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0)); }
__device__ __forceinline__ unsigned long long lane_range(uint32_t first, uint32_t n) { return ((1ull << n) - 1) << first; }
__device__ __forceinline__ uint32_t next_bit(unsigned long long& m) { const uint32_t j = (uint32_t)__ffsll((long long)m) - 1; m &= m - 1; return j; }

// A word of a grammar's table, by its index; the byte offset is worked out in 32 bits, so that the load takes it as an offset to
// the uniform base address.  (The largest, transitions of 2^18 states to 256 classes, is 256 MiB.)  For arrays that can reach 4 GiB
// the base address has to be that of the part at hand.
template <class P>
__device__ __forceinline__ P tab_at(const P* base, uint32_t index) {
#if defined(__HIP_DEVICE_COMPILE__)
    return *(const __attribute__((address_space(1))) P*)((const __attribute__((address_space(1))) char*)base + index * (uint32_t)sizeof(P));
#else
    return base[index];
#endif
}

// The Earley steps of earley_core.hpp with one wavefront per token: lane k holds item k of the set at hand together with the
// state it goes to on the next byte (looked up when the item is entered: it is the lookahead and the next scanner step in
// one) and its rule.  Control flow is the same in all lanes; values picked out of a lane are wave-uniform.
// A step is bound by its chain of dependent loads (about 500 cycles each beside the logits that pass through the caches; a
// slot's wavefront waits three quarters of its time), so what can be asked for together is: a state that is entered has its
// record (rule, expansion) fetched beside its transition, and an item keeps its rule for the completer.
// Wait entries, REG: all in registers, the context's and the token's own: lane k < n_w holds entry k, lane s <= the set at
// hand where set s starts.  Not REG: in LDS, and in registers those of the set at hand.
template <bool REG>
struct WaveScan {
    static constexpr uint32_t N = 64;
    static constexpr uint32_t NO_ITEM = SID_MASK;  // what lanes without an item hold: no state has this number (it would be the sink's), no flags
    const DevTables T;
    const uint2* ctx_wait; const uint32_t* ctx_off; const uint32_t H;   // LDS: wait entries of the context's H sets, and where each set's start
    const uint2* own_wait; const uint32_t* own_off;                     // LDS: the same for the sets made during the token (numbered from H)
    const uint32_t lane;
    const uint32_t max_items;                     // at most N: more is an overflow
    uint32_t item, to, rule;                      // the set under construction: lane k < n holds item k, where it goes on the next byte, and its rule
    uint32_t n;                                   //   (not of an item that starts in the set: it completes nothing)
    uint32_t w_rule, w_tgt, w_beg, n_w;           // its wait entries so far: lane w_beg <= k < n_w holds entry k
    uint32_t set_off;                             // REG: lane s holds the first entry of set s
    uint32_t set_idx, la;                         // its number; class of the next byte, or NO_TARGET after the last one
    bool full, root_done;

    __device__ __forceinline__ bool add(uint32_t v, uint32_t v_to, uint32_t v_rule) {
        if (lanes_of(item == v)) return false;
        if (n == max_items) { full = true; return false; }
        if (lane == n) { item = v; to = v_to; rule = v_rule; }
        ++n;
        return true;
    }
    __device__ __forceinline__ void add_wait(uint32_t w, uint32_t tgt) {
        if (lanes_of(w_tgt == tgt) & lanes_of(w_rule == w) & lanes_of(lane < n_w) & (REG ? lanes_of(lane >= w_beg) : ~0ull)) return;
        if (n_w == N) { full = true; return; }
        if (lane == n_w) { w_rule = w; w_tgt = tgt; }
        ++n_w;
    }
    // where a state goes on the next byte (a gather over the lanes that ask)
    __device__ __forceinline__ uint32_t next_of(bool mine, uint32_t ref) const {
        uint32_t t = NO_TARGET;
        if (mine && (ref & F_BYTE) && la != NO_TARGET) t = tab_at(T.trans, (ref & SID_MASK) * T.n_classes + la);
        return t;
    }
    // byte edges only, not final, and none of them for the next byte: the item can do nothing
    __device__ __forceinline__ unsigned long long inert(uint32_t ref, uint32_t t) const { return lanes_of((ref & (F_BYTE | F_REF | F_FINAL)) == F_BYTE) & lanes_of(t == T.sink); }
    // what entering a state with record {of, at, n_items, n_waits} adds besides the item itself
    __device__ __forceinline__ void expand(uint32_t of, uint32_t at, uint32_t n_items, uint32_t n_waits, uint32_t origin) {
        const uint32_t* e = T.exp_list + at;
        const uint32_t* e2 = e + n_items;
        const uint32_t most = n_items > n_waits ? n_items : n_waits;
        for (uint32_t base = 0; base < most; base += N) {
            const bool has_item = base + lane < n_items, has_wait = base + lane < n_waits;
            uint32_t v = 0, w = 0, tgt = 0;
            if (has_item) v = tab_at(e, base + lane);
            if (has_wait) { w = tab_at(e2, 2 * (base + lane)); tgt = tab_at(e2, 2 * (base + lane) + 1); }
            const uint32_t t = next_of(has_item, v);
            // the wait entries while the transitions are on their way
            for (unsigned long long m = lanes_of(base + lane < n_waits); m;) {
                const uint32_t j = next_bit(m), x = lane_value(tgt, j);
                add_wait(lane_value(w, j), (x & REF_MASK) | (((x & EXP_CURRENT) ? set_idx : origin) << REF_BITS));
            }
            for (unsigned long long m = lanes_of(base + lane < n_items) & ~inert(entered(v), t); m;) {
                const uint32_t j = next_bit(m), x = lane_value(v, j);
                add((x & REF_MASK) | (((x & EXP_CURRENT) ? set_idx : origin) << REF_BITS), lane_value(t, j), of);   // (an advance stays in its rule)
            }
        }
    }
    // the lanes of m each enter the state `ref` with their origin
    __device__ __forceinline__ void enter(unsigned long long m, uint32_t ref, uint32_t origin) {
        const bool mine = has_lane(m);
        uint4 d = make_uint4(0, 0, 0, 0);
        if (mine && (ref & (F_REF | F_FINAL))) d = tab_at(T.state, ref & SID_MASK);
        const uint32_t t = next_of(mine, ref);
        m &= ~inert(ref, t);
        while (m) {
            const uint32_t j = next_bit(m), r = lane_value(ref, j), o = lane_value(origin, j), of = lane_value(d.x, j);
            if ((r & (F_BYTE | F_FINAL)) || !(r & F_REF)) { if (!add(r | (o << REF_BITS), lane_value(t, j), of)) continue; }
            if (r & F_REF) expand(of, lane_value(d.y, j), lane_value(d.z, j), lane_value(d.w, j), o);
        }
    }
    // One byte: scanner and completer over the set held in (cur_item, cur_to), NO_ITEM beyond its items.  False: nothing survives.
    __device__ __forceinline__ bool step(uint32_t cur_item, uint32_t cur_to) {
        n = 0; root_done = false;
        item = NO_ITEM;
        if (REG) { w_beg = n_w; if (lane == set_idx) set_off = n_w; }
        else n_w = 0;
        enter(lanes_of((cur_item & F_BYTE) != 0) & lanes_of(cur_to != T.sink), cur_to, cur_item >> REF_BITS);
        unsigned long long done = 0;
        for (;;) {
            unsigned long long m = lanes_of((item & F_FINAL) != 0) & lanes_of((item >> REF_BITS) != set_idx) & ~done;
            if (!m) break;
            done |= m;
            while (m) {                                              // (entering below only appends to the items)
                const uint32_t j = next_bit(m), o = lane_value(item, j) >> REF_BITS;
                if (o == ROOT_ORIGIN) { root_done = true; continue; }
                const uint32_t of = lane_value(rule, j);
                if (REG) {
                    const uint32_t lo = lane_value(set_off, o), hi = lane_value(set_off, o + 1);
                    const unsigned long long hit = lanes_of(w_rule == of) & lanes_of(lane >= lo) & lanes_of(lane < hi);
                    if (hit) enter(hit, w_tgt & REF_MASK, w_tgt >> REF_BITS);
                    continue;
                }
                const bool own = o >= H;
                const uint2* wait = own ? own_wait : ctx_wait;
                const uint32_t* off = own ? own_off + (o - H) : ctx_off + o;
                const uint32_t lo = same_in_all(off[0]), hi = same_in_all(off[1]);
                for (uint32_t base = lo; base < hi; base += N) {
                    uint2 w = make_uint2(0, 0);
                    if (base + lane < hi) w = wait[base + lane];
                    const unsigned long long hit = lanes_of(base + lane < hi) & lanes_of(w.x == of);
                    if (hit) enter(hit, w.y & REF_MASK, w.y >> REF_BITS);
                }
            }
        }
        return n != 0 || n_w != w_beg;
    }
};

// ---- fill ------------------------------------------------------------------------------------------
// k_fill: one workgroup per row, in two teams of wavefronts that work side by side.
//   The union team streams: per mask word the OR of the accepted rows of the row's frontier planes, plus the
//   end-of-sequence bit, stored with 16-byte accesses.
//   The re-check team takes the uncertain tokens of the frontier planes from the short list every plane carries behind
//   its three rows (written by k_plane_summary) and runs the Earley routine from the row's full context; what survives
//   is kept in LDS until the union is stored, and OR-ed in afterwards.
// The two teams need nothing from each other until that point, so the latency of the re-check (a chain of dependent
// table loads) hides behind the streaming and the other way round.  A token that another frontier plane accepts is in
// the mask anyway and is not parsed: its bit is looked up in the accepted rows, without waiting for the union.
// Most rows have no candidate and a few have a handful, but the launch lasts as long as its slowest row.  A row with few
// candidates (kFillWaveTokens) gives each a wavefront (WaveScan: a byte costs about one gather, where a lane of its own
// takes several dependent accesses), the union team joining in when it is done; a row with more gives each a lane.
// Wavefronts take as many at a time as the row has, lanes any number in one round.  Which is less depends on the grammar: six
// wavefronts / lanes from 19 on, two fills and a step, 37 rows of a JSON schema 27 / 32 us, 64 rows of records 72 / 67; 24 candidates
// deep in nested parentheses, 1 row, 49 / 39, and of 20 - 40 bytes 129 / 95.
// How many wavefronts a row's workgroup has (fill_row_waves).  A compute unit that has one row has room for sixteen: 64 rows of
// records with up to 47 candidates 23.8 / 17.1 / 15.8 us (six / twelve / sixteen wavefronts), 256 rows of tools 20.9 / 16.5 / 15.0.
// With more rows than compute units, six / twelve, us, grammars and vocabularies of the decoding cases:
//   25 - 48 candidates are a lane's each with six and a wavefront's each with twelve, of which the device holds two rows a compute
//   unit and not four.  300 / 512 / 1,024 / 2,048 rows of tools 18.9 / 20.8 / 24.9 / 33.9 against 16.4 / 16.7 / 21.6 / 34.9, of a
//   nested schema 20.3 / 20.6 / 24.8 / 31.6 against 18.1 / 18.4 / 24.7 / 34.5, of records 24.2 / 24.9 / 28.2 / 37.0 against 18.6 /
//   20.1 / 24.9 / 37.6: twelve up to four rows a compute unit.
//   Up to 24 are a wavefront's each with either.  300 / 512 / 600 / 1,024 / 2,048 rows of records (19) 13.5 / 14.6 / 14.5 / 18.3 / 28.1
//   against 13.6 / 14.5 / 16.6 / 21.1 / 33.2, of a nested schema (20) 14.2 / 16.4 / - / 17.4 / 22.3 against 12.6 / 13.5 / - / 17.5 /
//   23.9; none at all, 512 / 1,024 rows, 6.0 / 8.6 against 6.3 / 9.8: twelve up to two rows a compute unit, if there are any.
//   49 - 64 are a lane's each with either, in one round.  300 / 512 / 1,024 / 2,048 rows of repetitions (59) 26.4 / 29.0 / 32.5 / 47.9
//   against 28.1 / 32.0 / 37.2 / 58.9: six.
//   More take a second round with six and, up to 128, not with twelve.  Nested parentheses (80), 300 / 1,024 / 2,048 rows, 105.9 / 197.6 /
//   310.7 against 73.0 / 134.4 / 250.5: twelve.
//   Word by word, 64 / 300 / 600 tokens a plane, 512 rows 81 / 201 / 398 against 91 / 182 / 290, 1,024 rows 137 / 351 / 679 against 172 /
//   354 / 558, 2,048 rows 210 / 523 / 1,015 against 332 / 688 / 1,057: twelve up to two rows a compute unit.
// Everything that is asked for before the plan is known (the context, the tables, the first planes' lists, the first block of the
// union) used to wait for it: 0.5 - 1.5 us of every row.
// A row with a frontier plane whose uncertain tokens do not fit its list (or with more candidates than the LDS list
// holds) takes the sequential way: the union team also reads the uncertain rows and lists the words with candidates,
// the re-check team starts when the union is done, a lane each.
// A token that outgrows a lane's lists (or 16 bytes) goes to a wavefront, one that outgrows that too (or 64 bytes) to lists in device
// memory, in the row's own workgroup (own_lanes, up to six) or in the launch behind, which has 4,096 lanes over the device but costs
// every call 2 - 4 us.  Nested parentheses, us a call, without / with that launch: 63 tokens of 65 - 80 bytes, 1 / 64 / 192 rows
// 1,865 / 2,138 / 2,142 against 195 / 199 / 574; of 9 - 80 bytes 797 / 844 / 850 against 303 / 316 / 320; 18 of 3 - 14 bytes
// 15.9 / 18.4 / 20.0 against 18.3 / 20.5 / 22.3.  So where rows of a small batch may have more than kFillSpreadTokens tokens and the
// vocabulary has such long ones the host launches it.  What a wavefront can take is the wavefronts' in any case: 63 tokens of 20 - 40 bytes
// take 126 / 131 / 137 us that way and 104 / 110 / 315 in the launch behind, 24 of them 52 / 55 / 58 and 92 / 99 / 190; short tokens whose
// item sets outgrow a lane 64 and 128 (33 a row, 1 row, expansions of 25 items; six wavefronts a row).  The sequential way, which has no
// bound on its tokens, leaves all that a lane cannot take to that launch (100 of 20 - 40 bytes, 1 row: 112 us; one lane of the workgroup
// after another took 5,433).
// Four wavefronts stream, the others re-check: two with half of their lanes at work (measured: fewer lanes per wavefront or another
// split of the six gain nothing), more with a quarter.
constexpr int FILL_OR_WAVES = 4, FILL_OR_THREADS = 64 * FILL_OR_WAVES;
template <int WAVES> struct FillTeam {
    static constexpr int THREADS = 64 * WAVES;
    static constexpr int BLOCK = WAVES == 16 ? 5 : 4;                // vectors of the union a thread asks for together
    static constexpr int LANES = WAVES == 6 ? 32 : 16;               // lanes at work in a wavefront of the re-check team
    static constexpr int COLS = (WAVES - FILL_OR_WAVES) * LANES;     // tokens the team parses at a time
    using Store = LdsStore<kFillLaneItems, kFillLaneWaits, COLS>;
};
constexpr uint32_t FILL_LISTS = 2;                     // planes whose lists are asked for before their lengths are known
constexpr int FILL_K = kFillLaneItems, FILL_WM = kFillLaneWaits;
constexpr uint32_t FILL_SPARSE_CAP = kFillRowTokens;   // candidates of a row that the side-by-side way handles
// What became of a candidate: the token, or FILL_NONE if it was rejected; FILL_OVER: it did not fit the lists tried so far;
// FILL_LARGE: it did not fit a lane's, and a wavefront has decided it.
constexpr uint32_t FILL_OVER = 0x80000000u, FILL_LARGE = 0x40000000u, FILL_NONE = 0x3FFFFFFFu;
constexpr uint32_t FILL_CTX_WAITS = kFillContextWaits, FILL_CTX_SETS = kFillContextSets, FILL_OWN_WAITS = 128, FILL_WAVE_BYTES = kFillWaveBytes;   // what a wavefront's parse has room for

__device__ __forceinline__ DevCtx row_ctx(const FillBatch& F, const FillRow& r) {
    DevCtx C;
    C.items = F.ctx_items + r.item_off;
    C.n_items = r.item_n;
    C.wait = F.ctx_wait + r.wait_base;
    C.wait_off = F.ctx_wait_off + r.waitoff_off;
    C.H = r.H;
    return C;
}

// Candidate bits of one mask word of row b go to the scratch word; the word's index goes to the row's own
// work list (one LDS atomic per wave with candidates: no atomics on device memory).
__device__ __forceinline__ void list_candidates(const FillBatch& F, uint32_t* n_listed, uint32_t* n_cand, uint32_t cand, size_t row_base, uint32_t w) {
    const unsigned long long has = __ballot(cand != 0);
    if (has) {
        const uint32_t lane = threadIdx.x & 63;
        const uint32_t leader = (uint32_t)__ffsll((long long)has) - 1;
        uint32_t base = 0;
        if (lane == leader) base = atomicAdd(n_listed, (uint32_t)__popcll(has));
        base = __shfl(base, (int)leader);
        if (cand) {
            atomicAdd(n_cand, (uint32_t)__popc(cand));
            F.cand_words[row_base + w] = cand;
            F.work_list[row_base + base + (uint32_t)__popcll(has & ((1ull << lane) - 1))] = w;
        }
    }
}

constexpr int RECHECK_NO = 0, RECHECK_YES = 1, RECHECK_OVER = 2;
// One candidate token, one lane, against the row's full context.
template <class Store>
__device__ __forceinline__ int recheck_lane(const DevVocab& Vd, const DevTables& T, const uint32_t* cls_words, const DevCtx& C, uint32_t id, Store& st) {
    const TokenRecord rec = tab(Vd.rec + id);
    if (rec.n_bytes == 0) return RECHECK_NO;
    RegBytes tok;
    tok.v = rec.head;
    st.reset();
    const int res = scan_token(T, cls_words, C, tok, (int)rec.n_bytes, st);
    return (res & RES_OVERFLOW) ? RECHECK_OVER : (res & RES_ALIVE) ? RECHECK_YES : RECHECK_NO;
}

// A row's context in LDS for the wavefronts that parse from it, and each wavefront's room for what its token adds.
struct FillCtx { uint2 wait[FILL_CTX_WAITS]; uint32_t off[FILL_CTX_SETS + 1]; uint32_t cls_words[64]; };
struct WaveToken { uint32_t words[4], id, off, n_bytes; };           // a token that a wavefront parses: its first 16 bytes, ...
struct FillOwn { uint2 wait[FILL_OWN_WAITS]; uint32_t off[FILL_WAVE_BYTES + 1]; };
__device__ __forceinline__ void wave_sync() {                       // orders a wavefront's LDS traffic (which completes in order) for the compiler
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
// One candidate token (the same in all lanes), one wavefront.  *large: it would not have fitted the short lists of a lane,
// whatever became of it (so that the count does not depend on the way a row takes).
__device__ __forceinline__ int recheck_wave(const DevVocab& Vd, const SlowScratch& S, const DevTables& T, const FillCtx& X, FillOwn& own, uint32_t H, uint32_t item_n, uint32_t my_item,
                                            uint32_t tok_word, uint32_t at, uint32_t n_bytes, uint32_t lane, bool* large) {
    if (n_bytes == 0) return RECHECK_NO;
    if (n_bytes > FILL_WAVE_BYTES) return RECHECK_OVER;
    *large |= n_bytes > 16 || item_n > (uint32_t)FILL_K;
    uint32_t byte = ((uint32_t)__shfl((int)tok_word, (int)(lane >> 2) & 3) >> (8 * (lane & 3))) & 0xFF;
    if (n_bytes > 16) byte = lane < n_bytes ? tab(Vd.bytes + at + lane) : 0u;
    const uint32_t cls_of = reinterpret_cast<const uint8_t*>(X.cls_words)[byte];
    const uint32_t max_items = S.k_cap < WaveScan<false>::N ? S.k_cap : WaveScan<false>::N, max_waits = S.wm_cap < FILL_OWN_WAITS ? S.wm_cap : FILL_OWN_WAITS;
    WaveScan<false> A{T, X.wait, X.off, H, own.wait, own.off, lane, max_items, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, false, false};
    if (item_n > max_items) return RECHECK_OVER;
    A.la = lane_value(cls_of, 0);
    uint32_t cur = lane < item_n ? my_item : A.NO_ITEM, cur_to = A.next_of(true, cur), n_own = 0;
    if (lane == 0) own.off[0] = 0;
    for (uint32_t i = 0; i < n_bytes; ++i) {
        A.set_idx = H + i;
        A.la = i + 1 < n_bytes ? lane_value(cls_of, i + 1) : NO_TARGET;
        wave_sync();
        const bool alive = A.step(cur, cur_to);
        if (A.full) return RECHECK_OVER;
        if (!alive) return RECHECK_NO;
        *large |= A.n > (uint32_t)FILL_K || n_own + A.n_w > (uint32_t)FILL_WM;
        if (n_own + A.n_w > max_waits) return RECHECK_OVER;
        wave_sync();
        if (lane < A.n_w) own.wait[n_own + lane] = make_uint2(A.w_rule, A.w_tgt);
        n_own += A.n_w;
        if (lane == 0) own.off[i + 1] = n_own;
        cur = A.item; cur_to = A.to;
    }
    return RECHECK_YES;
}

// A pair that nobody decides keeps its bit 0, and the call must not pass for complete: the pair goes to the host's list (it can
// decide it with its own parser), a slot on the device is marked unusable.
__device__ __forceinline__ void leave_undecided(const SlowScratch& S, uint32_t b, uint32_t id) {
    atomicOr(S.count + 1, 2u);
    if (S.mark_rows) S.mark_rows[b].pad[1] = 2u;
    if (S.unresolved) {                                              // plain stores only: the list is host memory
        const uint32_t at = atomicAdd(S.count + 2, 1u);
        S.unresolved[0] = 1u;
        if (at < S.unresolved_cap) { S.unresolved[2 + 2 * at] = b; S.unresolved[3 + 2 * at] = id; }
        else S.unresolved[1] = 1u;
    }
}
// One (row, token) pair that outgrew every shorter list: one lane, item lists in device memory (lane gl of the scratch).
__device__ __forceinline__ bool recheck_large(const FillBatch& F, const DevVocab& Vd, const SlowScratch& S, const FillRow& r, uint32_t b, uint32_t id, uint32_t gl) {
    const TokenRecord rec = tab(Vd.rec + id);
    const int n = (int)rec.n_bytes;
    if (n == 0) return false;
    const DevTables T = F.tables[r.tables_idx];
    MemBytes tok{Vd.bytes + rec.off};
    GlobalStore st;
    st.init(S.mem + gl, S.n_lanes, S.k_cap, S.wm_cap);
    st.reset();
    const int res = scan_token<GlobalStore, false, MemBytes>(T, T.byte_class_words, row_ctx(F, r), tok, n, st);
    if (!(res & RES_OVERFLOW)) return (res & RES_ALIVE) != 0;
    leave_undecided(S, b, id);
    return false;
}

// Entry with the smallest index whose inclusive prefix sum exceeds t (every lane of the wave calls this; incl is the
// lanes' non-decreasing prefix, lane 63 holds the total).
__device__ __forceinline__ uint32_t prefix_owner(uint32_t incl, uint32_t t) {
    uint32_t lo = 0, hi = 63;
#pragma unroll
    for (int it = 0; it < 6; ++it) {
        const uint32_t mid = (lo + hi) >> 1;
        const uint32_t v = (uint32_t)__shfl((int)incl, (int)mid);
        if (v > t) hi = mid; else lo = mid + 1;
    }
    return lo;
}

// Four consecutive mask words from a word boundary (a row of any W, at any word address); words at or beyond W read as 0 and
// are not written.
typedef uint32_t Words4 __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ void load4(const uint32_t* row, uint32_t w, uint32_t W, uint32_t (&v)[4]) {
    if (w + 4 <= W) {
        const Words4 x = *(const __attribute__((address_space(1))) Words4*)(row + w);
        v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
    } else {
        _Pragma("unroll") for (uint32_t c = 0; c < 4; ++c) v[c] = w + c < W ? tab(row + w + c) : 0u;
    }
}
__device__ __forceinline__ void store4(uint32_t* row, uint32_t w, uint32_t W, const uint32_t (&v)[4]) {
    if (w + 4 <= W) {
        Words4 x; x.x = v[0]; x.y = v[1]; x.z = v[2]; x.w = v[3];
        *(__attribute__((address_space(1))) Words4*)(row + w) = x;
    } else {
        _Pragma("unroll") for (uint32_t c = 0; c < 4; ++c) if (w + c < W) row[w + c] = v[c];
    }
}

// One block of a row's union: BLOCK vectors of four words a thread, FILL_OR_THREADS apart, from v0 (of thread 0) on.  What lies
// beyond the row holds other bits of the plane: nobody may look at it.  (Asked for whether the row reaches that far or not: with a way
// round the loads of a short row the compiler waited for the first before it sent the second.)
template <int BLOCK>
__device__ __forceinline__ void union_load(const uint32_t* row, uint32_t n_vec, uint32_t v0, uint32_t (&x)[BLOCK][4]) {
#pragma unroll
    for (int s = 0; s < BLOCK; ++s) {
        const uint32_t v = min(v0 + s * FILL_OR_THREADS + threadIdx.x, n_vec - 1);
        const Words4 y = *(const __attribute__((address_space(1))) Words4*)((const __attribute__((address_space(1))) char*)row + 16 * v);
        x[s][0] = y.x; x[s][1] = y.y; x[s][2] = y.z; x[s][3] = y.w;
    }
}
template <int BLOCK>
__device__ __forceinline__ void union_add(uint32_t (&acc)[BLOCK][4], const uint32_t (&x)[BLOCK][4]) {
    _Pragma("unroll") for (int s = 0; s < BLOCK; ++s)
        _Pragma("unroll") for (int c = 0; c < 4; ++c) acc[s][c] |= x[s][c];
}
__device__ __forceinline__ uint64_t lane_address(uint64_t a, uint32_t k) { return ((uint64_t)lane_value((uint32_t)(a >> 32), k) << 32) | lane_value((uint32_t)a, k); }
__device__ __forceinline__ const uint32_t* plane_row(uint64_t a) { return reinterpret_cast<const uint32_t*>(a & ~(uint64_t)1); }
// Whole blocks: all loads of a block and a plane are issued before the first is used.  Lane k holds the address of frontier plane k.
// The first block of the first plane has been asked for already (acc), as soon as its address was known, so that it is on its way
// while the rest of the row's plan is worked out.
template <int BLOCK>
__device__ __forceinline__ void fill_union(const FillBatch& F, uint32_t W, uint64_t addr, uint32_t front_n, bool eos, uint32_t* out, uint32_t (&acc)[BLOCK][4]) {
    const uint32_t eos_word = F.eos_id >> 5, eos_bit = 1u << (F.eos_id & 31), n_vec = (W + 3) / 4;
    uint32_t k = 1;
    for (uint32_t v0 = 0; v0 < n_vec; v0 += BLOCK * FILL_OR_THREADS) {
        for (; k < front_n; ++k) {
            uint32_t x[BLOCK][4] = {};
            union_load(plane_row(lane_address(addr, k)), n_vec, v0, x);
            union_add(acc, x);
        }
        k = 0;
#pragma unroll
        for (int s = 0; s < BLOCK; ++s) {
            const uint32_t v = v0 + s * FILL_OR_THREADS + threadIdx.x;
            if (eos && eos_word / 4 == v) {
                _Pragma("unroll") for (int c = 0; c < 4; ++c) if (eos_word % 4 == (uint32_t)c) acc[s][c] |= eos_bit;
            }
            if (v < n_vec) store4(out, 4 * v, W, acc[s]);
            _Pragma("unroll") for (int c = 0; c < 4; ++c) acc[s][c] = 0;
        }
    }
}
// The same for a frontier of any length, with the uncertain rows: the tokens of theirs that no plane accepts are listed.
template <int BLOCK>
__device__ __forceinline__ void fill_union_listing(const FillBatch& F, uint32_t W, uint32_t b, uint32_t front_off, uint32_t front_n, bool eos, uint32_t* out, uint32_t* n_listed, uint32_t* n_cand) {
    const uint32_t eos_word = F.eos_id >> 5, eos_bit = 1u << (F.eos_id & 31), n_vec = (W + 3) / 4;
    for (uint32_t v0 = threadIdx.x; v0 - threadIdx.x < n_vec; v0 += BLOCK * FILL_OR_THREADS) {       // same rounds for every thread: the ballots see whole waves
        uint32_t acc[BLOCK][4] = {}, unc[BLOCK][4] = {};
        for (uint32_t k = 0; k < front_n; ++k) {
            const uint64_t pa = uniform_load(F.front_planes + front_off + k);
#pragma unroll
            for (int s = 0; s < BLOCK; ++s) {
                const uint32_t v = v0 + s * FILL_OR_THREADS;
                if (v >= n_vec) continue;
                uint32_t x[4];
                load4(plane_row(pa), 4 * v, W, x);
                _Pragma("unroll") for (int c = 0; c < 4; ++c) acc[s][c] |= x[c];
                if (pa & 1) continue;
                load4(plane_row(pa) + W, 4 * v, W, x);
                _Pragma("unroll") for (int c = 0; c < 4; ++c) unc[s][c] |= x[c];
            }
        }
#pragma unroll
        for (int s = 0; s < BLOCK; ++s) {
            const uint32_t v = v0 + s * FILL_OR_THREADS;
            uint32_t cand[4], any = 0;
            _Pragma("unroll") for (int c = 0; c < 4; ++c) { cand[c] = v < n_vec ? (unc[s][c] & ~acc[s][c]) : 0u; any |= cand[c]; }
            if (__any(any != 0))                                    // candidates are few: most wavefronts have none
                _Pragma("unroll") for (int c = 0; c < 4; ++c) list_candidates(F, n_listed, n_cand, cand[c], (size_t)b * W, v * 4 + c);
            if (eos && eos_word / 4 == v) {
                _Pragma("unroll") for (int c = 0; c < 4; ++c) if (eos_word % 4 == (uint32_t)c) acc[s][c] |= eos_bit;
            }
            if (v < n_vec) store4(out, 4 * v, W, acc[s]);
        }
    }
}

// Six wavefronts a SIMD at least: a compute unit then holds four rows of six wavefronts, i.e. the device 1,024 at once.
struct FillArgs { FillBatch F; DevVocab Vd; int32_t* bitmask; long long row_stride; SlowScratch S; };
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(WAVES == 16 ? 4 : 6))) void k_fill(const FillRow* rows, const uint64_t* front_planes, FillArgs A) {
    const FillBatch& F = A.F;
    const DevVocab& Vd = A.Vd;
    using Team = FillTeam<WAVES>;
    constexpr uint32_t THREADS = Team::THREADS, LANES = Team::LANES, COLS = Team::COLS;
    constexpr uint32_t FILL_WAVE_TOKENS = kFillWaveTokens * WAVES;
    static_assert(FILL_WAVE_TOKENS <= 64, "a row's candidates lie across the lanes");
    static_assert(WAVES >= kFillOwnLanes, "each of a row's own lanes of the large-capacity scratch is a wavefront's");
    __shared__ uint32_t lds_store[Team::Store::SLOTS * COLS];
    __shared__ uint32_t sh_surv[FILL_SPARSE_CAP];
    __shared__ FillCtx ctx;
    __shared__ FillOwn sh_own[WAVES];
    __shared__ uint32_t n_listed, n_cand, n_over, next_token, n_to_parse;
    __shared__ WaveToken sh_tok[FILL_WAVE_TOKENS];
    const uint32_t b = blockIdx.x, lane = threadIdx.x & 63, wave = same_in_all(threadIdx.x >> 6);
    FillRow r = uniform_load(rows + b);
    uint64_t started = wall_clock64();
    // (all that the first loads of planes and context go by, waited for once)
    const DevTables* tables = F.tables;
    const uint32_t* ctx_items = F.ctx_items;
    uint64_t* stamps = F.stamps;
    uint32_t W = Vd.W;
    PIN("+s"(stamps), "+s"(r.front_off), "+s"(r.flags), "+s"(r.planes[0]), "+s"(r.planes[1]), "+s"(r.n_wait), "+s"(started), "+s"(tables), "+s"(ctx_items), "+s"(W));
    auto stamp_end = [&]() { if (stamps && lane == 0) stamps[kStampsRows + (WAVES + 1) * b + 1 + wave] = wall_clock64(); };
    const uint32_t front_off = r.front_off, front_n = r.front_n, flags = r.flags;
    const bool live = !(flags & 2u);
    // the plan, worked out by every wavefront for itself: lane k looks at frontier plane k.  (The first two planes' addresses come with the
    // row: to find them behind it took a load of 300 - 900 cycles more before anything of a plane could be asked for.)
    uint64_t addr = 1;
    uint32_t n_unc = 0;
    if (live && front_n <= 64) {
        static_assert(kRowPlanes == 2, "lanes 0 and 1 below");
        if (lane < front_n) addr = lane == 0 ? r.planes[0] : r.planes[1];
        if (front_n > kRowPlanes && lane >= kRowPlanes && lane < front_n) addr = front_planes[front_off + lane];
    }
    // What a parse starts from does not hang on the frontier, and is asked for together with it: the grammar's tables, the context.
    static_assert(kFillContextItems <= WaveScan<false>::N, "a context's items lie across the lanes");
    DevTables T = uniform_load(tables + r.tables_idx);
    const uint32_t n_wait = live ? r.n_wait : 0u;
    const bool ctx_fits = live && r.item_n <= kFillContextItems && r.H <= FILL_CTX_SETS && n_wait <= FILL_CTX_WAITS;
    uint32_t my_item = 0, x0[Team::BLOCK][4] = {}, list[FILL_LISTS] = {};
    if (lane < front_n && !(addr & 1)) n_unc = tab(plane_row(addr) + 3 * (size_t)W);
    if (ctx_fits && lane < r.item_n) my_item = tab(ctx_items + r.item_off + lane);
    if (wave < FILL_OR_WAVES) {
        if (live && front_n != 0 && front_n <= 64) union_load(plane_row(lane_address(addr, 0)), (W + 3) / 4, 0, x0);
    } else {
        if (wave == FILL_OR_WAVES) {
            // the first planes' lists, whose lengths are on their way (a plane has room for a whole list, whatever it holds)
            if (live && front_n != 0 && front_n <= 64)
                _Pragma("unroll") for (uint32_t k = 0; k < FILL_LISTS; ++k)
                    if (k < front_n) { const uint64_t a = lane_address(addr, k); if (!(a & 1)) list[k] = tab(plane_row(a) + 3 * (size_t)W + lane); }
            ctx.cls_words[lane] = tab(T.byte_class_words + lane);
        }
        if (ctx_fits) {
            for (uint32_t t = threadIdx.x - FILL_OR_THREADS; t < n_wait; t += THREADS - FILL_OR_THREADS) ctx.wait[t] = tab(F.ctx_wait + r.wait_base + t);
            for (uint32_t t = threadIdx.x - FILL_OR_THREADS; t <= r.H; t += THREADS - FILL_OR_THREADS) ctx.off[t] = tab(F.ctx_wait_off + r.waitoff_off + t);
        }
    }
    PIN("+s"(T.trans));                                              // (asked for above, and not where the compiler needs it first)
    if (threadIdx.x == 0) {
        n_listed = 0; n_cand = 0; n_over = 0; next_token = 0;
        if (stamps) stamps[kStampsRows + (WAVES + 1) * b] = started;
    }
    if (F.zero_words && b == 0 && threadIdx.x < 4) F.zero_words[threadIdx.x] = 0;      // the words the next call counts in
    const bool no_list = n_unc > kUncListWords - 1;                   // more uncertain tokens than the plane's list holds
    uint32_t incl = no_list ? 0u : n_unc, total = 0;
    const bool some_list = __any(incl != 0);
    if (some_list) {
        for (int d = 1; d < 64; d <<= 1) { const uint32_t up = (uint32_t)__shfl_up((int)incl, d); if ((int)lane >= d) incl += up; }
        total = lane_value(incl, 63);
    }
    const bool listed_way = live && front_n != 0 && (front_n > 64 || __any(no_list) || total > FILL_SPARSE_CAP);
    const bool wave_way = ctx_fits && !listed_way && total <= FILL_WAVE_TOKENS;
    if (wave_way && total != 0 && wave == FILL_OR_WAVES) {
        // every candidate at once, one a lane: its token, its bytes, whether a frontier plane accepts it (then it is in the mask already)
        const uint32_t k = prefix_owner(incl, lane);
        const uint32_t end_k = (uint32_t)__shfl((int)incl, (int)k), n_k = (uint32_t)__shfl((int)n_unc, (int)k), at = 1 + (lane - (end_k - n_k));
        uint32_t id = 0, accepted = 1;
        _Pragma("unroll") for (uint32_t p = 0; p < FILL_LISTS; ++p) {
            const uint32_t x = (uint32_t)__shfl((int)list[p], (int)at);
            if (k == p) id = x;
        }
        if (front_n > FILL_LISTS) {
            const uint32_t a_lo = (uint32_t)__shfl((int)(uint32_t)addr, (int)k), a_hi = (uint32_t)__shfl((int)(uint32_t)(addr >> 32), (int)k);
            if (lane < total && k >= FILL_LISTS) id = tab(plane_row(((uint64_t)a_hi << 32) | a_lo) + 3 * (size_t)Vd.W + at);
        }
        TokenRecord rec{};
        if (lane < total) {
            rec = tab(Vd.rec + id);
            accepted = 0;
            // four planes at a time: their words are asked for together (256 rows of tools, the step 56.5 -> 55.9 us)
            for (uint32_t k2 = 0; k2 < front_n; k2 += 4) {
                uint32_t w[4];
                _Pragma("unroll") for (uint32_t c = 0; c < 4; ++c) w[c] = tab(plane_row(lane_address(addr, min(k2 + c, front_n - 1))) + (id >> 5));
                accepted |= (w[0] | w[1] | w[2] | w[3]) >> (id & 31);
            }
            accepted |= rec.n_bytes == 0;
        }
        const unsigned long long parse = lanes_of(!(accepted & 1u));
        if (has_lane(parse)) {
            WaveToken& x = sh_tok[count_below(parse)];
            x.words[0] = rec.head.x; x.words[1] = rec.head.y; x.words[2] = rec.head.z; x.words[3] = rec.head.w;
            x.id = id; x.off = rec.off; x.n_bytes = rec.n_bytes;
        }
        if (lane == 0) n_to_parse = (uint32_t)__popcll(parse);
    }
    uint32_t* out = reinterpret_cast<uint32_t*>(A.bitmask) + (long long)b * A.row_stride;
    typename Team::Store st;
    const uint32_t col = (wave - FILL_OR_WAVES) * LANES + lane;      // re-check team: this lane's place among the lanes at work
    const bool at_work = wave >= FILL_OR_WAVES && lane < LANES;
    if (at_work) st.init(lds_store + col);
    __syncthreads();

    if (wave < FILL_OR_WAVES) {
        if (listed_way) fill_union_listing<2>(F, Vd.W, b, front_off, front_n, (flags & 3u) != 0, out, &n_listed, &n_cand);
        else fill_union(F, Vd.W, addr, live ? front_n : 0u, (flags & 3u) != 0, out, x0);
    } else if (!listed_way && total != 0 && !wave_way) {
        // side by side with the union, a lane per candidate: candidate t is entry t - (tokens of the planes before) of its plane's list
        const FillArgs Z = args_again<FillArgs>();
        const DevCtx C = row_ctx(Z.F, uniform_load(Z.F.rows + b));
        for (uint32_t t0 = 0; t0 < total; t0 += COLS) {
            const uint32_t t = t0 + col;
            const bool mine = at_work && t < total;
            const uint32_t k = prefix_owner(incl, t);
            const uint32_t end_k = (uint32_t)__shfl((int)incl, (int)k), n_k = (uint32_t)__shfl((int)n_unc, (int)k);
            const uint32_t a_lo = (uint32_t)__shfl((int)(uint32_t)addr, (int)k), a_hi = (uint32_t)__shfl((int)(uint32_t)(addr >> 32), (int)k);
            uint32_t id = 0;
            if (mine) id = tab(reinterpret_cast<const uint32_t*>(((uint64_t)a_hi << 32) | a_lo) + 3 * (size_t)Vd.W + 1 + (t - (end_k - n_k)));
            // a token that a frontier plane accepts is in the mask already: no need to parse it
            uint32_t accepted = 0;
            for (uint32_t k2 = 0; k2 < front_n; k2 += 4) {
                uint32_t w[4];
                _Pragma("unroll") for (uint32_t c = 0; c < 4; ++c) w[c] = tab(plane_row(lane_address(addr, min(k2 + c, front_n - 1))) + (id >> 5));
                accepted |= (w[0] | w[1] | w[2] | w[3]) >> (id & 31);
            }
            if (mine) {
                const int res = (accepted & 1u) ? RECHECK_NO : recheck_lane(Vd, T, ctx.cls_words, C, id, st);
                sh_surv[t] = res == RECHECK_YES ? id : res == RECHECK_OVER ? (id | FILL_OVER) : FILL_NONE;
                if (res == RECHECK_OVER) atomicAdd(&n_over, 1u);
            }
        }
    }
    // (the wavefronts' way: of the tokens that no plane accepts; below, sh_surv is theirs)
    const uint32_t n_tokens = wave_way && total != 0 ? same_in_all(n_to_parse) : total;
    bool waves_parse = wave_way && total != 0;
    if (!listed_way && total != 0 && !wave_way) {                   // (the same for the whole row)
        __syncthreads();
        waves_parse = ctx_fits && n_over != 0;
    }
    if (waves_parse) {
        // a wavefront per candidate, the union team joining in when its row is stored; or per token that did not fit a lane's lists
        for (;;) {
            // The wavefront stays together from token to token: with nothing between "lane 0 stores a result" below and "lane 0
            // takes the next token" here the compiler may send the other lanes round the loop without lane 0.
            wave_sync();
            uint32_t t = 0;
            if (lane == 0) t = atomicAdd(&next_token, 1u);
            wave_sync();
            t = same_in_all(t);
            if (t >= n_tokens) break;
            uint32_t id, at, n_bytes;
            uint32_t tok_word;                                       // lane k: bytes 4 k .. 4 k + 3 (of the first 16)
            if (wave_way) {
                id = same_in_all(sh_tok[t].id); at = same_in_all(sh_tok[t].off); n_bytes = same_in_all(sh_tok[t].n_bytes);
                tok_word = sh_tok[t].words[lane & 3];
            } else {
                const uint32_t v = same_in_all(sh_surv[t]);
                if (!(v & FILL_OVER)) continue;
                id = v & ~FILL_OVER;
                at = uniform_load(&Vd.rec[id].off); n_bytes = uniform_load(&Vd.rec[id].n_bytes);
                tok_word = tab(reinterpret_cast<const uint32_t*>(Vd.rec + id) + (lane & 3));
            }
            bool large = !wave_way;
            const int res = recheck_wave(Vd, A.S, T, ctx, sh_own[wave], r.H, r.item_n, my_item, tok_word, at, n_bytes, lane, &large);
            if (lane == 0) {
                sh_surv[t] = (res == RECHECK_NO ? FILL_NONE : id) | (res == RECHECK_OVER ? FILL_OVER : large ? FILL_LARGE : 0u);
                if (wave_way && res == RECHECK_OVER) atomicAdd(&n_over, 1u);
            }
        }
    }
    __syncthreads();

    if (!listed_way) {
        uint32_t n_large = 0;
        for (uint32_t t0 = wave * 64; t0 < n_tokens; t0 += THREADS) {
            const uint32_t t = t0 + lane, v = t < n_tokens ? sh_surv[t] : FILL_NONE, id = v & FILL_NONE;
            n_large += (uint32_t)__popcll(__ballot((v & (FILL_OVER | FILL_LARGE)) != 0));
            if (v & FILL_OVER) {
                const FillArgs Z = args_again<FillArgs>();
                if (Z.F.follows && try_push(Z.S, b, id)) sh_surv[t] = FILL_NONE;
                else if (!Z.F.own_lanes) leave_undecided(Z.S, b, id);
            } else if (id != FILL_NONE) atomicOr(out + (id >> 5), 1u << (id & 31));
        }
        if (n_large != 0 && lane == 0) atomicAdd(args_again<FillArgs>().S.count + 3, n_large);
        if (threadIdx.x == 0) F.row_count[b] = total;               // every row writes its count: nothing to clear beforehand
        // what fits nowhere else: one lane of every wavefront that has a lane of the large-capacity scratch
        if (n_over != 0 && args_again<FillArgs>().F.own_lanes != 0) {
            const FillArgs Z = args_again<FillArgs>();
            const FillRow q = uniform_load(Z.F.rows + b);
            if (Z.F.follows) __syncthreads();
            if (lane == 0 && wave < Z.F.own_lanes)
                for (uint32_t t = wave; t < n_tokens; t += Z.F.own_lanes) {
                    const uint32_t v = sh_surv[t], id = v & FILL_NONE;
                    if ((v & FILL_OVER) && recheck_large(Z.F, Z.Vd, Z.S, q, b, id, b * Z.F.own_lanes + wave)) atomicOr(out + (id >> 5), 1u << (id & 31));
                }
        }
        stamp_end();
        return;
    }
    if (threadIdx.x == 0) F.row_count[b] = n_cand;
    if (wave < FILL_OR_WAVES) { stamp_end(); return; }                // (a barrier below is for the wavefronts that have not ended)
    // the sequential way: each wave of the re-check team takes its share of the listed words, at a time at most as many as it has lanes
    // at work, and spreads their set bits densely over those lanes.  (As many words as lanes, however few there are, leave all of them
    // to the first waves: 64 / 100 / 300 / 600 neighbouring tokens of up to 14 bytes, 1 row, 120 / 186 / 541 / 880 us against 73 / 68 /
    // 94 / 170; 512 rows, twelve wavefronts, 142 / 236 / 661 / 1,127 against 91 / 88 / 182 / 290.
    // The streaming wavefronts end before: were they kept for the barrier, 800 / 1,024 / 2,048 rows of six wavefronts with 64 tokens took
    // 144 / 156 / 275 us instead of 94 / 137 / 210.)
    const FillArgs Z = args_again<FillArgs>();
    const FillRow q = uniform_load(Z.F.rows + b);
    const uint32_t count = n_listed;
    const uint32_t* wlist = Z.F.work_list + (size_t)b * Z.Vd.W;
    uint32_t* cands = Z.F.cand_words + (size_t)b * Z.Vd.W;
    const DevTables T2 = uniform_load(Z.F.tables + q.tables_idx);
    const DevCtx C = row_ctx(Z.F, q);
    uint32_t large = 0, n_left = 0;
    constexpr uint32_t TEAM = WAVES - FILL_OR_WAVES;
    const uint32_t n_words = min(LANES, (count + TEAM - 1) / TEAM);
    for (uint32_t base = (wave - FILL_OR_WAVES) * n_words; base < count; base += TEAM * n_words) {
        uint32_t idx = 0, cand = 0, left = 0;                      // left: the tokens of this lane's word that are for the end
        const bool has_word = lane < n_words && base + lane < count;
        if (has_word) { idx = wlist[base + lane]; cand = cands[idx]; }
        uint32_t pre = (uint32_t)__popc(cand);
        for (int d = 1; d < 64; d <<= 1) { const uint32_t up = (uint32_t)__shfl_up((int)pre, d); if ((int)lane >= d) pre += up; }
        const uint32_t n_tok = lane_value(pre, 63);
        for (uint32_t t0 = 0; t0 < n_tok; t0 += LANES) {
            const uint32_t my = t0 + lane;
            const uint32_t j = prefix_owner(pre, my);
            uint32_t c = (uint32_t)__shfl((int)cand, (int)j);
            const uint32_t end_j = (uint32_t)__shfl((int)pre, (int)j), w = (uint32_t)__shfl((int)idx, (int)j);
            bool over = false;
            uint32_t id = 0;
            if (lane < LANES && my < n_tok) {
                uint32_t skip = my - (end_j - (uint32_t)__popc(c));
                while (skip--) c &= c - 1;                         // drop the lowest set bits that other lanes take
                id = w * 32 + (uint32_t)__ffs(c) - 1;
                const int res = recheck_lane(Z.Vd, T2, ctx.cls_words, C, id, st);
                if (res == RECHECK_YES) atomicOr(out + w, 1u << (id & 31));
                over = res == RECHECK_OVER;
            }
            unsigned long long m = __ballot(over);
            if (!m) continue;
            large += (uint32_t)__popcll(m);
            if (Z.F.follows) {                                     // to k_recheck_slow, if its list has room
                uint32_t at = 0;
                if (lane == 0) at = atomicAdd(Z.S.count, (uint32_t)__popcll(m));
                at = lane_value(at, 0) + (uint32_t)__popcll(m & ((1ull << lane) - 1));
                const bool fits = over && at < Z.S.list_cap;
                if (fits) { Z.S.list[2 * at] = b; Z.S.list[2 * at + 1] = id; }
                m = __ballot(over && !fits);
            }
            n_left += (uint32_t)__popcll(m);
            while (m) {
                const uint32_t k = next_bit(m), id2 = lane_value(id, k);
                if (Z.F.own_lanes) left |= lane == lane_value(j, k) ? 1u << (id2 & 31) : 0u;
                else if (lane == 0) leave_undecided(Z.S, b, id2);
            }
        }
        if (Z.F.own_lanes && has_word) cands[idx] = left;
    }
    if (lane == 0 && large) atomicAdd(Z.S.count + 3, large);
    if (lane == 0 && n_left) atomicAdd(&n_over, n_left);
    if (Z.F.own_lanes) {
        // what is left: one lane of every wavefront that has a lane of the large-capacity scratch.  (A wavefront without one must
        // not parse with its lists in device memory: there are more of them than lanes, and the next lane is the next row's.)
        __syncthreads();
        const uint32_t n_own = min(Z.F.own_lanes, TEAM), me = wave - FILL_OR_WAVES;
        if (n_over != 0 && lane == 0 && me < n_own)
            for (uint32_t k = me; k < count; k += n_own) {
                const uint32_t w = wlist[k];
                for (uint32_t m = cands[w]; m; m &= m - 1) {
                    const uint32_t bit = (uint32_t)__ffs(m) - 1;
                    if (recheck_large(Z.F, Z.Vd, Z.S, q, b, w * 32 + bit, b * Z.F.own_lanes + me)) atomicOr(out + w, 1u << bit);
                }
            }
    }
    stamp_end();
}

__global__ __launch_bounds__(64) void k_recheck_slow(FillBatch F, DevVocab Vd, int32_t* bitmask, long long row_stride, SlowScratch S) {
    __shared__ uint32_t lds[MidStore::SLOTS * 64];
    const uint32_t gl = blockIdx.x * 64 + threadIdx.x;
    uint32_t count = S.count[0];
    if (count > S.list_cap) count = S.list_cap;
    MidStore mid;
    mid.init(lds + threadIdx.x);
    for (uint32_t idx = gl; idx < count; idx += S.n_lanes) {
        const uint32_t b = S.list[2 * idx], id = S.list[2 * idx + 1];
        const FillRow r = F.rows[b];
        const TokenRecord rec = tab(Vd.rec + id);
        const int n = (int)rec.n_bytes;
        if (n == 0) continue;
        bool alive;
        int res = RES_OVERFLOW;
        if (S.k_cap >= (uint32_t)MidStore::K) {
            const DevTables T = F.tables[r.tables_idx];
            MemBytes tok{Vd.bytes + rec.off};
            mid.reset();
            res = scan_token<MidStore, false, MemBytes>(T, T.byte_class_words, row_ctx(F, r), tok, n, mid);
        }
        if (res & RES_OVERFLOW) alive = recheck_large(F, Vd, S, r, b, id, gl);
        else alive = (res & RES_ALIVE) != 0;
        if (alive) atomicOr(reinterpret_cast<uint32_t*>(bitmask) + (long long)b * row_stride + (id >> 5), 1u << (id & 31));
    }
    if (F.stamps && threadIdx.x == 0) F.stamps[kStampsRows + (F.row_waves + 1) * F.B + blockIdx.x] = wall_clock64();
}

// ---- matchers on the device ------------------------------------------------------------------------
// k_accept: one wavefront per matcher slot.  The kernel lasts as long as its slowest slot, and a slot is one chain of
// dependent steps, so the wavefront works on one slot as a whole (WaveScan above): items, wait entries and expansions lie
// across the lanes, a set's look-ups in the transition table are one gather, a prediction is one load, and what remains in
// order are list insertions in registers.  (With lane 0 doing everything on lists in LDS the same steps took 16 us at 16 - 64
// slots and 24 us at 1,024; one lane per slot 458 us.)  Bound by the latency of a dozen dependent loads (300 - 850 cycles each;
// the wavefront waits three quarters of its time), so everything that can be asked for at once is: a token comes as one record by
// its id, the slot's context straight into registers, pointers by scalar loads.  Against vector loads of the structs, contexts in
// LDS and three loads in a row to find a token's bytes, us at 1 / 64 / 1,024 slots (JSON schemas, records): 6.0 / 9.4 / 12.1 -> 5.0 / 7.6 / 9.6.
// A token or context that does not fit across 64 lanes takes the
// recogniser of accept_core.hpp on lane 0, with its lists, the renumbering table and the frontier staging in LDS, and one
// too large for that the same with everything in device memory.  A slot whose capacity is exceeded gets a sticky error and
// answers XG2_EOVERFLOW until it is reset.
constexpr int ACCEPT_K = 64, ACCEPT_WM = 256, ACCEPT_MAXLEN = 48;  // lane 0's item lists
struct OneLaneStore {
    static constexpr int K = ACCEPT_K, WM = ACCEPT_WM, MAXLEN = ACCEPT_MAXLEN, WORDS = 2 * ACCEPT_K + 2 * ACCEPT_WM + ACCEPT_MAXLEN + 1;
    uint32_t* cur; uint32_t* nxt; uint32_t* wait; uint32_t* ws;
    __device__ void init(uint32_t* base) { cur = base; nxt = base + K; wait = base + 2 * K; ws = base + 2 * K + 2 * WM; }
    __device__ uint32_t get_cur(int k) const { return cur[k]; }
    __device__ void set_cur(int k, uint32_t v) { cur[k] = v; }
    __device__ uint32_t get_nxt(int k) const { return nxt[k]; }
    __device__ void set_nxt(int k, uint32_t v) { nxt[k] = v; }
    __device__ uint32_t wait_rule(int k) const { return wait[2 * k]; }
    __device__ uint32_t wait_tgt(int k) const { return wait[2 * k + 1]; }
    __device__ void set_wait(int k, uint32_t rule, uint32_t tgt) { wait[2 * k] = rule; wait[2 * k + 1] = tgt; }
    __device__ void swap() { uint32_t* t = cur; cur = nxt; nxt = t; }
    __device__ bool charge(int) { return true; }
    __device__ void reset() {}
    __device__ void set_wstart(int j, uint32_t v) { ws[j] = v; }
    __device__ uint32_t get_wstart(int j) const { return ws[j]; }
};
template <int N_MAP, int N_FRONT>
struct OneLaneScratchX {
    uint8_t* map; uint64_t* front;
    __device__ uint32_t map_cap() const { return N_MAP; }
    __device__ uint32_t front_cap() const { return N_FRONT; }
    __device__ uint32_t map_get(uint32_t i) const { return map[i]; }
    __device__ void map_set(uint32_t i, uint32_t v) { map[i] = (uint8_t)v; }
    __device__ uint64_t front_get(uint32_t k) const { return front[k]; }
    __device__ void front_set(uint32_t k, uint64_t v) { front[k] = v; }
};
struct GlobalScratchX {
    uint8_t* map; uint64_t* front; size_t stride; uint32_t n_map, n_front;
    __device__ uint32_t map_cap() const { return n_map; }
    __device__ uint32_t front_cap() const { return n_front; }
    __device__ uint32_t map_get(uint32_t i) const { return map[(size_t)i * stride]; }
    __device__ void map_set(uint32_t i, uint32_t v) { map[(size_t)i * stride] = (uint8_t)v; }
    __device__ uint64_t front_get(uint32_t k) const { return front[(size_t)k * stride]; }
    __device__ void front_set(uint32_t k, uint64_t v) { front[(size_t)k * stride] = v; }
};

__device__ __forceinline__ void start_sequence(const BatchDev& D, uint32_t b, uint32_t cache_idx, uint32_t lane, uint32_t n_lanes) {
    const CacheDev& Cd = D.caches[cache_idx];
    FillRow r{};
    r.front_off = b * D.KF; r.front_n = Cd.start_n_front;
    r.item_off = b * D.KI; r.item_n = Cd.start_n_items;
    r.wait_base = b * D.KW; r.waitoff_off = b * (D.KH + 1); r.H = Cd.start_H;
    r.tables_idx = cache_idx; r.flags = Cd.start_flags;
    r.n_wait = Cd.start_wait_off[Cd.start_H];
    _Pragma("unroll") for (uint32_t k = 0; k < kRowPlanes; ++k) if (k < Cd.start_n_front) r.planes[k] = Cd.start_front[k];
    for (uint32_t k = lane; k < Cd.start_n_front; k += n_lanes) D.front[r.front_off + k] = Cd.start_front[k];
    for (uint32_t k = lane; k < Cd.start_n_items; k += n_lanes) D.items[r.item_off + k] = Cd.start_items[k];
    for (uint32_t k = lane; k <= Cd.start_H; k += n_lanes) D.wait_off[r.waitoff_off + k] = Cd.start_wait_off[k];
    for (uint32_t k = lane; k < r.n_wait; k += n_lanes) D.wait[r.wait_base + k] = Cd.start_wait[k];
    if (lane == 0) D.rows[b] = r;
}

__global__ __launch_bounds__(256) void k_batch_assign(BatchDev D, const int32_t* rows, uint32_t n, uint32_t cache_idx) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const uint32_t b = rows ? (uint32_t)rows[i] : i;
    if (b < D.B) start_sequence(D, b, cache_idx, 0, 1);
}

constexpr uint32_t ACC_KI = kSlotItems, ACC_KH = kSlotSets, ACC_KW = kSlotWaits, ACC_KF = kSlotPlanes;     // the slot capacities the LDS staging is laid out for

// What the kernel is launched with besides rows and tokens (read anew where a way is rarely taken).
struct AcceptArgs { BatchDev D; DevVocab Vd; uint32_t eos_id; const int32_t* token_ids; int32_t* status; };

// What accepting a token needs of a cache.
struct CacheView {
    DevTables T;
    const uint64_t* plain_row; const uint32_t* pair_off; const uint64_t* pair_row; const uint32_t* site_of_off; const uint2* site_of;
    uint32_t context_depth;
};
__device__ __forceinline__ CacheView cache_view(const CacheDev* p) {
    CacheView c;
    c.T = uniform_load(&p->T);
    c.plain_row = uniform_load(&p->plain_row); c.pair_off = uniform_load(&p->pair_off); c.pair_row = uniform_load(&p->pair_row);
    c.site_of_off = uniform_load(&p->site_of_off); c.site_of = uniform_load(&p->site_of);
    c.context_depth = uniform_load(&p->context_depth);
    return c;
}

// The slot's next state from token `tok16` (1 .. 16 bytes), written to the slot's other buffer `slot`; results in out_n (items,
// sets, planes, root can end, wait entries) and, if all went well, out_planes (the first of the planes).  Lane k has the context's item k, wait entry k and start of set k (what lies beyond the counts is
// not looked at), and the classes of bytes 4 k .. 4 k + 3.  ACC_RETRY: something does not fit across the lanes, nothing has been
// written that counts.
__device__ __forceinline__ int accept_wave(const BatchDev& D, const CacheView& C, uint32_t b, size_t slot, uint4 tok16, uint32_t n_bytes, uint32_t H, uint32_t item_n,
                                           uint32_t in_item, uint2 in_wait, uint32_t in_off, uint32_t cls_word, uint32_t lane, uint32_t out_n[5], uint64_t out_planes[kRowPlanes]) {
    const DevTables& T = C.T;
    const bool depth1 = C.context_depth == 1;
    const uint32_t n_sets = H + n_bytes;
    const uint32_t n_wait_in = lane_value(in_off, H < 64 ? H : 0);
    if (n_sets > 64 || H > 63 || item_n > 64 || n_wait_in > 64) return ACC_RETRY;
    // classes of the token's bytes, one a lane
    const uint32_t words[4] = {tok16.x, tok16.y, tok16.z, tok16.w};
    const uint32_t byte = (words[(lane >> 2) & 3] >> (8 * (lane & 3))) & 0xFF;
    const uint32_t cls_of = ((uint32_t)__shfl((int)cls_word, (int)(byte >> 2)) >> (8 * (byte & 3))) & 0xFF;
    WaveScan<true> A{T, nullptr, nullptr, H, nullptr, nullptr, lane, 64, 0, 0, 0, 0, in_wait.x, in_wait.y, 0, n_wait_in, in_off, 0, 0, false, false};
    uint32_t cur = lane < item_n ? in_item : A.NO_ITEM;
    A.la = lane_value(cls_of, 0);
    uint32_t cur_to = A.next_of(true, cur);
    for (uint32_t i = 0; i < n_bytes; ++i) {
        A.set_idx = H + i;
        A.la = i + 1 < n_bytes ? lane_value(cls_of, i + 1) : NO_TARGET;
        const bool alive = A.step(cur, cur_to);
        if (A.full) return ACC_RETRY;
        if (!alive) return ACC_REJECTED;
        cur = A.item; cur_to = A.to;
    }
    const uint32_t n_wait = A.n_w;
    const uint2 my_wait = make_uint2(A.w_rule, A.w_tgt);
    const uint32_t my_off = lane < n_sets ? A.set_off : n_wait, w_origin = my_wait.y >> REF_BITS, c_origin = cur >> REF_BITS;
    const unsigned long long scanning = lanes_of((cur & F_BYTE) != 0);   // final-only items have done their work in the closure
    const unsigned long long alone = depth1 ? scanning : lanes_of(c_origin == ROOT_ORIGIN) & scanning;   // items whose plane has no context
    // The planes of the frontier hang on three loads, one after the other; the first of them is under way while the sets are
    // renumbered: of every item its rule and its state's row of planes (or its plane), of every wait entry the row of sites of
    // the state it continues in.
    uint32_t rule_of = 0, planes_at = 0, planes_end = 0, sites_at = 0, sites_end = 0;
    uint64_t row = 0;
    if (has_lane(alone)) row = tab_at(C.plain_row, cur & SID_MASK);
    if (has_lane(scanning & ~alone)) {
        rule_of = tab_at(T.state, cur & SID_MASK).x;
        planes_at = tab_at(C.pair_off, cur & SID_MASK); planes_end = tab_at(C.pair_off, (cur & SID_MASK) + 1);
    }
    if (lane < n_wait && !depth1) {
        sites_at = tab_at(C.site_of_off, my_wait.y & SID_MASK); sites_end = tab_at(C.site_of_off, (my_wait.y & SID_MASK) + 1);
    }
    // Which sets are still reachable: the current one, the origins of its items, and on from there through the wait entries (an
    // entry's origin is never above its own set, so each set is looked at once, the highest first); `kept`: their wait entries.
    unsigned long long reach = 0, kept = 0, next = 1ull << (n_sets - 1);
    const unsigned long long w_inner = ~lanes_of(w_origin == ROOT_ORIGIN);
    for (unsigned long long m = scanning & ~lanes_of(c_origin == ROOT_ORIGIN); m;) next |= 1ull << lane_value(c_origin, next_bit(m));
    while (next) {
        const uint32_t s = 63u - (uint32_t)__clzll((long long)next), begin = lane_value(my_off, s), end = s < 63 ? lane_value(my_off, s + 1) : n_wait;
        reach |= 1ull << s;
        if (begin < end) {
            const unsigned long long range = end - begin < 64 ? lane_range(begin, end - begin) : ~0ull;
            kept |= range;
            for (unsigned long long m = range & w_inner; m;) next |= 1ull << lane_value(w_origin, next_bit(m));
        }
        next &= ~reach;
    }
    // The place of every wait entry among its rule's sites: under way while the rest is worked out.
    const uint32_t n_sites = sites_end - sites_at;
    uint2 site = make_uint2(kNoRule, 0u);
    if (lane < n_wait && n_sites != 0) site = tab_at(C.site_of, sites_at + site_home(my_wait.x, n_sites));
    // Sets are renumbered in their old order, all at once: a set's number is how many of the sets that are kept lie below it, and its
    // start how many of the wait entries that are kept.  (Set by set, every set looked at, the site looked up for each plane and the
    // stores before it: the decoding steps of 16 rows of tools, 64 and 37 of JSON schemas, 256 of tools 16.67 / 18.83 / 18.52 / 57.0 us,
    // now 16.20 / 18.16 / 17.93 / 56.5; it was 4,400 - 7,500 of a slot's 8,500 - 23,000 cycles.)
    auto below = [](unsigned long long set, uint32_t k) { return (uint32_t)__popcll(k < 64 ? set & ((1ull << k) - 1) : set); };
    const uint32_t newH = (uint32_t)__popcll(reach), n_kept = (uint32_t)__popcll(kept);
    const uint32_t w_new = has_lane(w_inner) ? below(reach, w_origin) : ROOT_ORIGIN, c_new = c_origin != ROOT_ORIGIN ? below(reach, c_origin) : ROOT_ORIGIN, new_off = below(kept, my_off);
    uint32_t place = site.x == my_wait.x ? site.y : kNoRule;
    if (lanes_of(site.x != my_wait.x) & lanes_of(site.x != kNoRule)) {                     // (another rule lies where this one's place begins: seldom)
        if (site.x != my_wait.x && site.x != kNoRule) place = find_in_row(C.site_of, sites_at, n_sites, my_wait.x);
    }
    // The frontier's planes: of every item alone (root instance, or context depth 1), then under every entry of the item's origin
    // that waits for its rule, an entry a lane.  (An entry that two items wait at is looked up in two rounds.)  Each plane once;
    // where it is listed with and without its uncertain tokens, they count.
    uint32_t nf = 0, f_lo = 0, f_hi = 0;
    // the root instance: leaving the rule leaves the grammar, so its uncertain tokens are never allowed
    if (c_origin == ROOT_ORIGIN && row != 0) row |= 1u;
    unsigned long long todo = scanning & ~alone, found = alone;
    for (;;) {
        if (lanes_of(row == 0) & found) return ACC_NO_PLANE;
        while (found) {
            const uint32_t j = (uint32_t)__ffsll((long long)found) - 1, lo = lane_value((uint32_t)row, j), hi = lane_value((uint32_t)(row >> 32), j);
            const unsigned long long same = lanes_of((((uint32_t)row ^ lo) & ~1u) == 0) & lanes_of((uint32_t)(row >> 32) == hi) & found;
            const uint32_t counts = (lanes_of(((uint32_t)row & 1u) == 0) & same) ? ~1u : ~0u;
            const unsigned long long listed = lanes_of(lane < nf) & lanes_of(((f_lo ^ lo) & ~1u) == 0) & lanes_of(f_hi == hi);
            if (listed) { if (has_lane(listed)) f_lo &= counts; }
            else {
                if (nf >= ACC_KF) return ACC_OVERFLOW;
                if (lane == nf) { f_lo = lo & counts; f_hi = hi; }
                ++nf;
            }
            found &= ~same;
        }
        if (!todo) break;
        uint32_t at = 0, end = 0;
        do {
            const uint32_t j = (uint32_t)__ffsll((long long)todo) - 1, o = lane_value(c_origin, j), of = lane_value(rule_of, j);
            const uint32_t first = lane_value(my_off, o), n = (o + 1 < 64 ? lane_value(my_off, o + 1) : n_wait) - first;
            const unsigned long long hit = lanes_of(my_wait.x == of) & (n < 64 ? lane_range(first, n) : ~0ull);
            if (!hit) return ACC_NO_PLANE;
            if (hit & found) break;
            found |= hit;
            if (has_lane(hit)) { at = lane_value(planes_at, j); end = lane_value(planes_end, j); }
            todo &= todo - 1;
        } while (todo);
        row = 0;
        if (has_lane(found) && place < end - at) row = tab_at(C.pair_row, at + place);
    }
    // (stores last: a load behind them would be waited for together with them)
    uint2* const wait_out = D.wait + slot * ACC_KW;
    uint32_t* const off_out = D.wait_off + slot * (ACC_KH + 1);
    uint32_t* const items_out = D.items + slot * ACC_KI;
    if (has_lane(kept)) wait_out[count_below(kept)] = make_uint2(my_wait.x, (my_wait.y & REF_MASK) | (w_new << REF_BITS));
    if (has_lane(reach)) off_out[count_below(reach)] = new_off;
    if (lane == 0) off_out[newH] = n_kept;
    if (has_lane(scanning)) items_out[count_below(scanning)] = (cur & REF_MASK) | (c_new << REF_BITS);
    if (lane < nf) D.front[(size_t)b * ACC_KF + lane] = ((uint64_t)f_hi << 32) | f_lo;
    out_n[0] = (uint32_t)__popcll(scanning); out_n[1] = newH; out_n[2] = nf; out_n[3] = A.root_done ? 1u : 0u; out_n[4] = n_kept;
    _Pragma("unroll") for (uint32_t k = 0; k < kRowPlanes; ++k) out_planes[k] = ((uint64_t)lane_value(f_hi, k) << 32) | lane_value(f_lo, k);
    return ACC_OK;
}

__global__ __launch_bounds__(64) void k_accept(const FillRow* rows, const int32_t* token_ids, AcceptArgs A) {
    __shared__ uint32_t in_items[ACC_KI], in_wait_off[ACC_KH + 1], out_items[ACC_KI], out_wait_off[ACC_KH + 1];
    __shared__ uint2 in_wait[ACC_KW], out_wait[ACC_KW];
    __shared__ uint64_t out_front[ACC_KF], x_front[ACC_KF];
    __shared__ uint32_t lists[OneLaneStore::WORDS];
    __shared__ uint8_t x_map[ACC_KH + ACCEPT_MAXLEN + 4];
    __shared__ int sh_acc;
    __shared__ uint32_t sh_out[5];                                 // n_items, H, n_front, root_done, wait entries
    __shared__ uint64_t sh_planes[kRowPlanes];
    const uint32_t lane = threadIdx.x, b = blockIdx.x;              // one wavefront per slot: everything below is the same in all lanes
    int32_t* status = A.status;
    const TokenRecord* records = A.Vd.rec;
    uint32_t V = A.Vd.V, eos_id = A.eos_id, B = A.D.B;
    int32_t tok = uniform_load(token_ids + b);
    FillRow r = uniform_load(rows + b);                             // (no other workgroup writes this row)
    PIN("+s"(tok), "+s"(r.pad[1]), "+s"(r.flags), "+s"(r.tables_idx), "+s"(status), "+s"(records), "+s"(V), "+s"(eos_id), "+s"(B));
    int32_t code = kAccOk;
    if (tok == kTokenReset) start_sequence(A.D, b, r.tables_idx, lane, 64);
    else if (tok < 0) code = kAccOk;                                 // nothing for this slot
    else if (r.pad[1]) code = kAccOverflow;                          // unusable until reset
    else if ((r.flags & 2u) || (uint32_t)tok >= V) code = kAccInvalid;
    else if ((uint32_t)tok == eos_id) {
        if (!(r.flags & 1u)) code = kAccRejected;
        else if (lane == 0) A.D.rows[b].flags = r.flags | 2u;        // the sequence ends here
    } else {
        // everything the parse starts from, asked for at once: the token, the grammar, and the first 64 of everything in the
        // slot's context, without waiting for the counts (a slot has room for that many and more)
        const CacheDev* const Cp = A.D.caches + r.tables_idx;
        TokenRecord rec = uniform_load(records + tok);
        CacheView C = cache_view(Cp);
        uint32_t cls_word = tab(Cp->cls_words + lane);
        // (a whole batch's wait entries can reach 8 GiB)
        uint32_t my_item = tab_at(A.D.items + r.item_off, lane), my_off = tab_at(A.D.wait_off + r.waitoff_off, lane);
        uint2 my_wait = tab_at(A.D.wait + r.wait_base, lane);
        PIN("+s"(rec.head.x), "+s"(rec.n_bytes), "+s"(C.T.trans), "+s"(C.T.state), "+s"(C.T.exp_list), "+s"(C.T.n_classes), "+s"(C.T.sink), "+s"(C.plain_row), "+s"(C.pair_off), "+s"(C.pair_row), "+s"(C.site_of_off), "+s"(C.site_of), "+s"(C.context_depth), "+v"(cls_word), "+v"(my_item), "+v"(my_off),
            "+v"(my_wait.x), "+v"(my_wait.y));
        const uint32_t nb = r.pad[0] ^ 1u;
        const size_t slot = (size_t)nb * B + b;
        if (rec.n_bytes == 0) code = kAccRejected;                   // special and empty tokens are never allowed
        else {
            uint32_t got[5] = {0, 0, 0, 0, 0};
            uint64_t planes[kRowPlanes] = {0, 0};
            int acc = ACC_RETRY;
            if (rec.n_bytes <= 16)
                acc = accept_wave(A.D, C, b, slot, rec.head, rec.n_bytes, r.H, r.item_n, my_item, my_wait, my_off, cls_word, lane, got, planes);
            if (acc == ACC_RETRY) {
                // lane 0, with the slot's whole context in LDS
                const AcceptArgs Z = args_again<AcceptArgs>();
                const BatchDev& D = Z.D;
                const FillRow q = uniform_load(D.rows + b);
                const TokenRecord t = uniform_load(Z.Vd.rec + uniform_load(Z.token_ids + b));
                const int n = (int)t.n_bytes;
                const CacheDev* const C0 = D.caches + q.tables_idx;
                __syncthreads();
                for (uint32_t k = lane; k < q.item_n; k += 64) in_items[k] = D.items[q.item_off + k];
                for (uint32_t k = lane; k <= q.H; k += 64) in_wait_off[k] = D.wait_off[q.waitoff_off + k];
                const uint32_t n_wait_in = D.wait_off[q.waitoff_off + q.H];
                for (uint32_t k = lane; k < n_wait_in; k += 64) in_wait[k] = D.wait[q.wait_base + k];
                __syncthreads();
                if (lane == 0) {
                    const CacheDev& Cd = *C0;
                    MatcherIn in{in_items, q.item_n, in_wait, in_wait_off, q.H};
                    MatcherOut out{out_items, out_wait, out_wait_off, out_front, ACC_KI, ACC_KH, ACC_KW, ACC_KF, 0, 0, 0, 0};
                    OneLaneStore st;
                    st.init(lists);
                    OneLaneScratchX<ACC_KH + ACCEPT_MAXLEN, ACC_KF> x{x_map, x_front};
                    int a = accept_token(Cd, Cd.cls_words, in, Z.Vd.bytes + t.off, n, st, x, out);
                    if (a == ACC_RETRY) {
                        // lists in device memory, results straight to the slot's other buffer
                        MatcherIn gin{D.items + q.item_off, q.item_n, D.wait + q.wait_base, D.wait_off + q.waitoff_off, q.H};
                        MatcherOut gout{D.items + slot * D.KI, D.wait + slot * D.KW, D.wait_off + slot * (D.KH + 1), D.front + (size_t)b * D.KF,
                                        D.KI, D.KH, D.KW, D.KF, 0, 0, 0, 0};
                        GlobalStore gs;
                        gs.init(D.slow_mem + b, D.B);
                        GlobalScratchX gx{D.slow_map + b, D.slow_front + b, D.B, D.KH + kSlowMaxLen + 1, D.KF};
                        a = accept_token(Cd, Cd.cls_words, gin, Z.Vd.bytes + t.off, n, gs, gx, gout);
                        out.n_items = gout.n_items; out.H = gout.H; out.n_front = gout.n_front; out.root_done = gout.root_done;
                        if (a == ACC_OK) a = -1;                     // done, nothing to copy out
                    }
                    sh_acc = a;
                    sh_out[0] = out.n_items; sh_out[1] = out.H; sh_out[2] = out.n_front; sh_out[3] = out.root_done;
                    if (a == ACC_OK || a == -1) {
                        sh_out[4] = a == ACC_OK ? out_wait_off[out.H] : D.wait_off[slot * (D.KH + 1) + out.H];
                        for (uint32_t k = 0; k < kRowPlanes && k < out.n_front; ++k) sh_planes[k] = a == ACC_OK ? out_front[k] : D.front[(size_t)b * D.KF + k];
                    }
                }
                __syncthreads();
                acc = sh_acc;
                _Pragma("unroll") for (int k = 0; k < 5; ++k) got[k] = sh_out[k];
                _Pragma("unroll") for (uint32_t k = 0; k < kRowPlanes; ++k) planes[k] = sh_planes[k];
                if (acc == ACC_OK) {
                    for (uint32_t k = lane; k < got[0]; k += 64) D.items[slot * D.KI + k] = out_items[k];
                    for (uint32_t k = lane; k <= got[1]; k += 64) D.wait_off[slot * (D.KH + 1) + k] = out_wait_off[k];
                    const uint32_t n_wait = out_wait_off[got[1]];
                    for (uint32_t k = lane; k < n_wait; k += 64) D.wait[slot * D.KW + k] = out_wait[k];
                    for (uint32_t k = lane; k < got[2]; k += 64) D.front[(size_t)b * D.KF + k] = out_front[k];
                } else if (acc == -1) acc = ACC_OK;
            }
            if (acc == ACC_OK) {
                if (lane == 0) {
                    FillRow w{};
                    w.front_off = b * ACC_KF; w.front_n = got[2];
                    w.item_off = (uint32_t)(slot * ACC_KI); w.item_n = got[0];
                    w.wait_base = (uint32_t)(slot * ACC_KW); w.waitoff_off = (uint32_t)(slot * (ACC_KH + 1)); w.H = got[1];
                    w.tables_idx = r.tables_idx; w.flags = got[3]; w.pad[0] = nb; w.n_wait = got[4];
                    _Pragma("unroll") for (uint32_t k = 0; k < kRowPlanes; ++k) w.planes[k] = planes[k];
                    A.D.rows[b] = w;
                }
            } else if (acc == ACC_REJECTED) code = kAccRejected;
            else { if (lane == 0) A.D.rows[b].pad[1] = 1u; code = kAccOverflow; }   // a capacity of the slot (or of the device-memory lists) was exceeded
        }
    }
    if (status && lane == 0) status[b] = code;
}

// ---- apply -----------------------------------------------------------------------------------------
// One wavefront per 2,048 tokens of a row (APPLY_WAVE), counted from the 128-byte boundary of memory at or before the row's
// begin, so that rows of any length and base are accessed in whole aligned cache lines.  Each lane takes one mask word: a
// piece that is allowed as a whole (most of free text) ends there, after one coalesced load.  Otherwise a piece goes one of three ways.
// Vector by vector, where neither of the two below is the better one: 16-byte vectors (4 fp32 or
// 8 bf16), 64 a step, their bits from the lane that holds the word: a vector whose tokens are all allowed is left alone (no
// read, no write); one whose tokens are all disallowed is overwritten without a read; only mixed vectors are read, merged and
// written back, all reads before the first store.  Vectors that the row shares with its neighbours are done by the element.
// Bound by memory (a large copy moves 5.4 TB/s on this card, a large fill 6.9), and where nothing is masked by instructions
// issued, which is why a mask word is loaded once and not once per vector.  With a mask look-up per vector, and rows off a
// 16-byte boundary done by the element, against now, us at 1,024 rows of V = 151,936 / 151,937, bf16: nothing masked 9.8 / 130
// -> 6.2 / 7.3; nearly everything 80 / 204 -> 52 / 53.
// One by one, where the mixed vectors of a piece hold few masked tokens: nothing is read, a store need not wait for a
// load, and a piece nearly all of which is allowed writes what it masks and no more; vectors masked as a whole are still stored as such.
// Each lane goes through its own word, so the most in one word counts (APPLY_FEW_WORD), and every token is a store of its own, so their sum
// counts too (of logits beyond 64 MB with the vectors masked as a whole: memory pays for lines that arrive in parts).
// All, where many words of a piece of logits beyond the last-level cache are mixed and few are allowed as a whole: all that is not
// masked as a whole is read, and all is written.  A line that a store leaves with holes is merged in memory, which costs more than reading
// and writing what was allowed; a line that is written whole need not stay in the second-level cache from load to store.
// Where the lines lie.  us, V = 151,936, medians of one process with the kernels in turn, in two settings: the same logits again / with the
// copy that writes the logits and the maximum that reads them around the call, as an engine has it.
// One by one, 64 words of a piece with k masked tokens each, by vectors -> one by one: bf16, 58 MB, k = 3, 4, 6: 21.8 -> 18.3 / 71.6 -> 68.1,
// 22.0 -> 22.5 / 71.8 -> 72.2, 21.2 -> 30.8 / 71.1 -> 80.5; 32 words, k = 4, 6: 15.4 -> 12.9 / 65.5 -> 62.5, 15.2 -> 17.4 / 65.1 -> 66.9; so 40 tokens
// and three a word.  fp32, 58 MB, 64 words, k = 4, 6, 8: 19.3 -> 15.9 / 66.2 -> 62.7, 19.8 -> 18.4 / 66.9 -> 65.2, 19.8 -> 22.1 / 67.0 -> 69.1;
// 32 words, k = 4, 6, 8: 10.4 -> 9.2 / 58.7 -> 56.0, 10.3 -> 11.4 / 58.8 -> 58.1, 10.3 -> 13.7 / 58.6 -> 60.4: 80 and three.  148 MB, 64 words, k = 2, 3:
// 43.6 -> 28.5 / 129.9 -> 128.2, 47.1 -> 34.0 / 131.6 -> 123.4, but over three sets of logits in turn 71.8 -> 68.8, 75.0 -> 78.6: 96 and one.
// Beyond 256 MB: bf16, 297 MB, 16 words, k = 4, 6: 46.7 -> 27.2 / 241 -> 243, 46.3 -> 37.7 / 241 -> 250; 32 words, k = 3, 4: 72.6 -> 40.2 / 271 -> 274,
// 73.2 -> 50.1 / 271 -> 277: 32 tokens and two a word.  fp32, 32 words, k = 3, 4: 52.1 -> 31.2 / 241 -> 237, 53.9 -> 32.9 / 240 -> 238, over three sets
// 75 -> 80; 64 words, k = 1, 2: 82 -> 35 / 298 -> 276, 92 -> 53 / 296 -> 305 (all: 91 / 276): 96.
// Up to 8 MB no sum is needed (fp32, 64 rows of 32,000, 64 words with 8: 5.5 -> 5.7 / 22.2 -> 20.9; counting cost the smallest steps 0.2 - 0.3).
// All, by vectors -> all; words that are not named are allowed as a whole: bf16, 297 MB, 36 and 40 half masked words (others masked): not
// taken 88.8 / 282, 90.5 -> 85.9 / 287 -> 271; 40 and 48 half masked (24 and 16 allowed): 76.9 -> 97.3 / 284 -> 273, 86.5 -> 91.8 / 297 -> 280.
// 408 MB, 40 half masked (24 allowed): 146 -> 135 / 427 -> 397.  fp32, 297 MB, 48, 52 and 60 half masked (16, 12, 4 allowed): 78.1 -> 99.5 / 261 -> 271,
// 83.7 -> 100.1 / even, 93.9 -> 89.6 / 294 -> 275 at 408 MB 393 -> 373: 8.  Half masked throughout, bf16, 297, 408 and 594 MB: 300 -> 278, 443 -> 395, 629 -> 553 (the second setting).
// Half of a piece's loads go through the caches up to 384 MB, and none beyond: what the program wrote before the call is partly still in the
// last-level cache.  By vectors / half through / none, masks of a list of records, second setting, bf16: 297 MB 257 / 258 / 266, 371 MB
// 352 / 346 / 350, 445 MB 417 / 406 / 411, 594 MB 558 / 540 / 534; fp32: 254 / 256 / 266, 322 / 321 / 330, 396 / 389 / 392, 546 / 532 / 520; the same records
// beside rows with a third masked at random, 445 MB, bf16 458 / 430 / 426, fp32 427 / 412 / 405.  (Masks of tools, few pieces of which are
// mixed, gain nothing: 237 / 238 at 297 MB, and with the same logits again 38 / 42.)  Within the last-level cache, 256 rows, fp32, by vectors
// and all: 48 and 50, over three sets 60 and 52, second setting 97 and 100: left as it was.
constexpr int APPLY_WAVE = 64 * 32, APPLY_WAVES = 4;
// Where the logits of a call end up: tiny and small ones stay in the caches, large ones fit the last-level cache (256 MB) but share it
// with what else the program touches between two steps, what is beyond it is streamed past it, and of a huge one hardly anything is
// left in it when it is asked for again.
enum ApplySize { APPLY_TINY, APPLY_SMALL, APPLY_LARGE, APPLY_STREAM, APPLY_HUGE };
constexpr uint32_t APPLY_FEW_WORD = 8;
constexpr int APPLY_DENSE_MIXED = 40;
template <class E> struct ApplyE;
template <> struct ApplyE<uint32_t> { static constexpr uint32_t NINF = 0xFF800000u, NINF_WORD = 0xFF800000u; };
template <> struct ApplyE<uint16_t> { static constexpr uint16_t NINF = 0xFF80; static constexpr uint32_t NINF_WORD = 0xFF80FF80u; };
typedef uint32_t Vec4 __attribute__((ext_vector_type(4)));

template <class E, ApplySize SIZE>
__global__ __launch_bounds__(64 * APPLY_WAVES) void k_apply_vec(E* logits, long long row_stride, int V, const uint32_t* bitmask, long long bm_stride) {
    constexpr bool STREAM = SIZE >= APPLY_STREAM, HALVES = sizeof(E) == 2;
    constexpr int EPV = 16 / sizeof(E), STEPS = 32 / EPV;
    constexpr uint32_t ALL = (1u << EPV) - 1, NI = ApplyE<E>::NINF_WORD;
    const long long b = blockIdx.y;
    E* const row = logits + b * row_stride;
    const uint32_t* const bm = bitmask + b * bm_stride;
    const int lane = threadIdx.x & 63, wave = (int)same_in_all(threadIdx.x >> 6);
    const int before = (int)(reinterpret_cast<uintptr_t>(row) & 127) / (int)sizeof(E);       // elements between the boundary and the row
    const long long e0 = ((long long)blockIdx.x * (blockDim.x >> 6) + wave) * APPLY_WAVE - before;   // the wavefront's first element
    if (e0 >= V) return;
    // this lane's 32 tokens from e0 + 32 * lane on; what lies outside the row counts as allowed
    const int first = (int)e0 + 32 * lane, shift = (int)(e0 & 31), at = first >> 5, last = (V - 1) >> 5;    // (an arithmetic shift: rounds down)
    uint32_t word = at >= 0 && at <= last ? bm[at] : ~0u;
    if (shift != 0) {                                                // (the same in all lanes)
        const uint32_t next = at + 1 >= 0 && at + 1 <= last ? bm[at + 1] : ~0u;
        word = (word >> shift) | (next << (32 - shift));
    }
    if (first < 0) word |= first <= -32 ? ~0u : (1u << -first) - 1;
    if (first + 32 > V) word |= first >= V ? ~0u : ~0u << (V - first);
    if (__ballot(word != ~0u) == 0) return;
    E* const piece = row + e0;
    // the word's masked tokens: those of vectors that are masked as a whole, and the others
    const uint32_t masked = ~word;
    uint32_t whole = masked & (masked >> 1);
    whole &= whole >> 2;
    if (EPV == 8) whole &= whole >> 4;
    whole = (whole & (EPV == 8 ? 0x01010101u : 0x11111111u)) * ALL;
    uint32_t part = masked & ~whole;
    const Vec4 none{NI, NI, NI, NI};
    const uint32_t count = (uint32_t)__popc(SIZE <= APPLY_SMALL ? part : masked);
    bool singly = __ballot(count > APPLY_FEW_WORD) == 0;
    if (SIZE != APPLY_TINY && singly) {
        const uint32_t words = (uint32_t)__popcll(__ballot(count != 0));
        const uint32_t most = HALVES ? (!STREAM ? 40 + 3 * words : words < APPLY_DENSE_MIXED ? 32 + 2 * words : 48) : STREAM ? 96 : SIZE == APPLY_LARGE ? 96 + words : 80 + 3 * words;
        if (APPLY_FEW_WORD * words > most) {                         // (else there is no need to count)
            static_assert(APPLY_FEW_WORD < 16, "a count is four bits");
            uint32_t total = 0;
            _Pragma("unroll") for (int k = 0; k < 4; ++k) total += (uint32_t)__popcll(__ballot((count >> k) & 1u)) << k;
            singly = total <= most;
        }
    }
    if (singly) {
#pragma unroll
        for (int j = 0; j < STEPS; ++j) {
            const int v = j * 64 + lane;
            if (((uint32_t)__shfl((int)whole, v / STEPS) >> (v % STEPS * EPV)) & 1u) {
                Vec4* const to = reinterpret_cast<Vec4*>(piece) + v;
                if (STREAM) __builtin_nontemporal_store(none, to);
                else *to = none;
            }
        }
        E* const mine = piece + 32 * lane;
        while (__ballot(part != 0) != 0) {
            if (part != 0) { mine[__ffs(part) - 1] = ApplyE<E>::NINF; part &= part - 1; }
        }
        return;
    }
    auto merge = [](Vec4& v, uint32_t b) {
        if (sizeof(E) == 4) {
            _Pragma("unroll") for (int c = 0; c < 4; ++c) if (!((b >> c) & 1)) v[c] = NI;
        } else {
            _Pragma("unroll") for (int c = 0; c < 4; ++c) {
                if (!((b >> (2 * c)) & 1)) v[c] = (v[c] & 0xFFFF0000u) | 0xFF80u;
                if (!((b >> (2 * c)) & 2)) v[c] = (v[c] & 0x0000FFFFu) | 0xFF800000u;
            }
        }
    };
    if (STREAM && e0 >= 0 && e0 + APPLY_WAVE <= V) {
        if (__popcll(__ballot(part != 0)) >= APPLY_DENSE_MIXED && __popcll(__ballot(word == ~0u)) <= (!HALVES ? 8 : SIZE == APPLY_HUGE ? 24 : 16)) {
            Vec4 x[STEPS];
            uint32_t bits[STEPS];
            const Vec4* const from = reinterpret_cast<const Vec4*>(piece) + lane;
#pragma unroll
            for (int j = 0; j < STEPS; ++j) {
                bits[j] = ((uint32_t)__shfl((int)word, (j * 64 + lane) / STEPS) >> (lane % STEPS * EPV)) & ALL;
                x[j] = none;
            }
            // (two loops: a load that the compiler makes of one through the caches and one past them goes through them)
            constexpr int PAST = SIZE == APPLY_HUGE ? STEPS : STEPS / 2;
            _Pragma("unroll") for (int j = 0; j < PAST; ++j) if (bits[j] != 0) x[j] = __builtin_nontemporal_load(from + j * 64);
            _Pragma("unroll") for (int j = PAST; j < STEPS; ++j) if (bits[j] != 0) x[j] = from[j * 64];
#pragma unroll
            for (int j = 0; j < STEPS; ++j) {
                merge(x[j], bits[j]);
                __builtin_nontemporal_store(x[j], reinterpret_cast<Vec4*>(piece) + j * 64 + lane);
            }
            return;
        }
    }
    Vec4 x[STEPS];
    uint32_t bits[STEPS];
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
        const int v = j * 64 + lane;
        bits[j] = ((uint32_t)__shfl((int)word, v / STEPS) >> (v % STEPS * EPV)) & ALL;
        x[j] = none;
        const int e = (int)e0 + v * EPV;
        if (bits[j] != 0 && bits[j] != ALL && e >= 0 && e + EPV <= V) x[j] = reinterpret_cast<const Vec4*>(piece)[v];
    }
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
        if (bits[j] == ALL) continue;
        const int v = j * 64 + lane, e = (int)e0 + v * EPV;
        if (e < 0 || e + EPV > V) {                                  // shared with a neighbour
            for (int c = 0; c < EPV; ++c) if (!((bits[j] >> c) & 1)) row[e + c] = ApplyE<E>::NINF;
            continue;
        }
        merge(x[j], bits[j]);
        Vec4* const to = reinterpret_cast<Vec4*>(piece) + v;
        if (STREAM) __builtin_nontemporal_store(x[j], to);
        else *to = x[j];
    }
}

// Logits that do not lie at a multiple of their own size (or rows too long to count in 32 bits above).
template <class E>
__global__ __launch_bounds__(256) void k_apply_scalar(E* logits, long long row_stride, int V, const uint32_t* bitmask, long long bm_stride) {
    const long long b = blockIdx.y;
    const int v = blockIdx.x * 256 + threadIdx.x;
    if (v >= V) return;
    if (!((bitmask[b * bm_stride + (v >> 5)] >> (v & 31)) & 1u)) logits[b * row_stride + v] = ApplyE<E>::NINF;
}

}  // namespace

// ---- scratch of the entry point that allocates nothing ---------------------------------------------
// One array per GPU the library runs on, held until the process ends.  In host code the array's name is only
// a stand-in: the device address comes from hipGetSymbolAddress, once per device, and only that address is
// handed to kernels and copies.
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

hipError_t noalloc_scratch(void** ptr_out) {
    constexpr int kMaxDevices = 64;
    static void* ptr_of[kMaxDevices] = {};
    static std::mutex mu;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!ptr_of[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        ptr_of[dev] = p;
    }
    *ptr_out = ptr_of[dev];
    return hipSuccess;
}

void launch_expand_chunks(const uint4* range_a_dev, const uint4* range_b_dev, const uint32_t* first_dev, uint32_t n_ranges,
                          uint4* chunk_dev, hipStream_t stream) {
    if (!n_ranges) return;
    hipLaunchKernelGGL(k_expand_chunks, dim3((n_ranges + 255) / 256), dim3(256), 0, stream, range_a_dev, range_b_dev, first_dev, n_ranges, chunk_dev);
}

void launch_stage(void* dst_dev, const void* src_host_mapped, size_t bytes, const StageZero& Z, const uint4* range_a_host_mapped,
                  const uint4* range_b_host_mapped, const uint32_t* first_host_mapped, uint32_t n_ranges, uint4* chunk_dev, hipStream_t stream) {
    const size_t n = bytes / sizeof(uint4);
    const uint32_t nb_up = (uint32_t)std::min<size_t>((n + 255) / 256, 2048);
    size_t zero_words = 0;
    for (uint32_t k = 0; k < Z.n; ++k) zero_words += Z.words[k];
    const uint32_t nb_zero = (uint32_t)std::min<size_t>((zero_words / 4 + 255) / 256, 2048);
    const uint32_t nb_exp = (n_ranges + 255) / 256;
    if (nb_up + nb_zero + nb_exp == 0) return;
    hipLaunchKernelGGL(k_stage, dim3(nb_up + nb_zero + nb_exp), dim3(256), 0, stream, static_cast<uint4*>(dst_dev), static_cast<const uint4*>(src_host_mapped), n,
                       nb_up, Z, nb_zero, range_a_host_mapped, range_b_host_mapped, first_host_mapped, n_ranges, chunk_dev);
}

uint32_t wave_slots() {
    static const uint32_t n = [] {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
            cus = 256;
        return (uint32_t)cus * 32u;                                 // 4 SIMDs of 8 wave slots each
    }();
    return n;
}

void launch_build(const DevTables& T, const DevVocab& Vd, BuildPlan P, const SlowScratch& S, hipStream_t stream) {
    if (P.n_chunks == 0) return;
    // Short item lists let a compute unit hold more workgroups, which is what hides the latency of the automaton
    // walks' dependent table loads when there is far more work than the device holds at once; long ones spare the
    // tokens that need them a second run at half width, which is what counts when the launch is a few chunks per
    // wave slot and lasts as long as its slowest workgroup.
    P.large_lists = P.n_chunks <= 4 * wave_slots() ? 1u : 0u;
#ifdef XG2_BUILD_FORCE_LISTS
    P.large_lists = XG2_BUILD_FORCE_LISTS;
#endif
    P.list_k = P.large_lists ? BUILD_K_LARGE : BUILD_K_SMALL;
    P.list_wm = P.large_lists ? BUILD_WM_LARGE : BUILD_WM_SMALL;
    const uint32_t lds_bytes = (2 * P.list_k + 2 * P.list_wm) * 64 * sizeof(uint32_t);
    // Workgroup g takes chunks g, g + grid, ...  At least one workgroup per wave slot of the device; a large launch is cut
    // into shares of about a dozen chunks, small enough for the hardware to even out the load as workgroups end and
    // large enough for a workgroup's tokens for the follow-language run to fill whole batches (measured: 8,192 for the
    // 10,063 chunks of the repetition workload, 65,536 for the 856,956 of the dispatch workload).
    uint32_t grid = std::min(P.n_chunks, std::max(wave_slots(), std::min(P.n_chunks / 12, 8 * wave_slots())));
#ifdef XG2_TUNE
    if (const char* e = getenv("XG2_BUILD_GRID")) grid = std::min<uint32_t>(P.n_chunks, (uint32_t)atoi(e));
    if (getenv("XG2_DEBUG_PLAN")) fprintf(stderr, "launch: chunks %u grid %u lds %u\n", P.n_chunks, grid, lds_bytes);
#endif
    hipLaunchKernelGGL(k_build, dim3(grid), dim3(64), lds_bytes, stream, T, Vd, P, S);
}

void launch_build_slow(const DevTables& T, const DevVocab& Vd, const BuildPlan& P, const SlowScratch& S, hipStream_t stream) {
    hipLaunchKernelGGL(k_build_slow, dim3(S.n_lanes / 64), dim3(64), 0, stream, T, Vd, P, S);
}

void launch_accept(const BatchDev& D, const DevVocab& Vd, uint32_t eos_id, const int32_t* token_ids_dev, int32_t* status_dev, hipStream_t stream) {
    if (!D.B || D.KI != ACC_KI || D.KH != ACC_KH || D.KW != ACC_KW || D.KF != ACC_KF) return;
    hipLaunchKernelGGL(k_accept, dim3(D.B), dim3(64), 0, stream, D.rows, token_ids_dev, AcceptArgs{D, Vd, eos_id, token_ids_dev, status_dev});
}

void launch_token_records(const DevVocab& Vd, TokenRecord* rec_dev, hipStream_t stream) {
    if (Vd.V) hipLaunchKernelGGL(k_token_records, dim3((Vd.V + 255) / 256), dim3(256), 0, stream, Vd, rec_dev);
}

void launch_batch_assign(const BatchDev& D, const int32_t* rows_dev, uint32_t n, uint32_t cache_idx, hipStream_t stream) {
    if (!n) return;
    hipLaunchKernelGGL(k_batch_assign, dim3((n + 255) / 256), dim3(256), 0, stream, D, rows_dev, n, cache_idx);
}

void launch_upload(void* dst_dev, const void* src_host_mapped, size_t bytes, hipStream_t stream, uint64_t* stamp, hipEvent_t done) {
    const size_t n = bytes / sizeof(uint4);
    if (!n) return;
    const uint32_t grid = (uint32_t)std::min<size_t>((n + 255) / 256, 2048);
    uint4* dst = static_cast<uint4*>(dst_dev);
    const uint4* src = static_cast<const uint4*>(src_host_mapped);
    if (done) hipExtLaunchKernelGGL(k_upload, dim3(grid), dim3(256), 0, stream, nullptr, done, 0, dst, src, n, stamp);
    else hipLaunchKernelGGL(k_upload, dim3(grid), dim3(256), 0, stream, dst, src, n, stamp);
}

void launch_clear(uint32_t* words_dev, uint32_t n, hipStream_t stream) {
    hipLaunchKernelGGL(k_clear, dim3(1), dim3(64), 0, stream, words_dev, n);
}

void launch_copy_masked(const CopyJob* jobs_dev, uint32_t n_jobs, uint32_t W, hipStream_t stream) {
    if (!n_jobs) return;
    for (uint32_t first = 0; first < n_jobs; first += 65535) {      // grid.y limit
        const uint32_t n = std::min<uint32_t>(65535, n_jobs - first);
        hipLaunchKernelGGL(k_copy_masked, dim3((W + 255) / 256, n), dim3(256), 0, stream, jobs_dev + first, W);
    }
}

void launch_copy_structure(const CopyJob* jobs_dev, uint32_t n_jobs, uint32_t W, hipStream_t stream) {
    for (uint32_t first = 0; first < n_jobs; first += 65535) {      // grid.y limit
        const uint32_t n = std::min<uint32_t>(65535, n_jobs - first);
        hipLaunchKernelGGL(k_copy_structure, dim3((W + 255) / 256, n), dim3(256), 0, stream, jobs_dev + first, W);
    }
}

void launch_copy_first_byte(const FirstByteCopyJob* jobs_dev, uint32_t n_jobs, const uint8_t* first_byte_dev, uint32_t W, hipStream_t stream) {
    for (uint32_t first = 0; first < n_jobs; first += 65535) {      // grid.y limit
        const uint32_t n = std::min<uint32_t>(65535, n_jobs - first);
        hipLaunchKernelGGL(k_copy_first_byte, dim3((W + 255) / 256, n), dim3(256), 0, stream, jobs_dev + first, first_byte_dev, W);
    }
}

void launch_plane_summary(uint32_t* const* plane_ptr_dev, uint32_t n_pos, uint32_t W, uint32_t* counts_dev, hipStream_t stream) {
    if (n_pos == 0) return;
    hipLaunchKernelGGL(k_plane_summary, dim3(n_pos), dim3(256), 0, stream, plane_ptr_dev, n_pos, W, counts_dev);
}

void launch_finish_planes(uint32_t* const* plane_ptr_dev, const FinishJob* jobs_dev, uint32_t n_pos, const uint8_t* first_byte_dev, uint32_t W,
                          uint32_t* counts_dev, hipStream_t stream) {
    for (uint32_t first = 0; first < n_pos; first += 65535) {       // grid.y limit
        const uint32_t n = std::min<uint32_t>(65535, n_pos - first);
        hipLaunchKernelGGL(k_finish_planes, dim3((W + FINISH_WORDS - 1) / FINISH_WORDS, n), dim3(256), 0, stream, plane_ptr_dev + first, jobs_dev + first, n,
                           first_byte_dev, W, counts_dev + 2 * (size_t)first);
    }
}

void launch_fill(const FillBatch& F, const DevVocab& Vd, int32_t* bitmask_dev, int64_t row_stride_words,
                 const SlowScratch& S, hipStream_t stream, hipEvent_t done) {
    if (F.B == 0) return;
    auto* const kernel = F.row_waves == 16 ? k_fill<16> : F.row_waves == 12 ? k_fill<12> : k_fill<6>;
    const dim3 block(64 * F.row_waves);
    const FillArgs A{F, Vd, bitmask_dev, (long long)row_stride_words, S};
    if (done) hipExtLaunchKernelGGL(kernel, dim3(F.B), block, 0, stream, nullptr, done, 0, F.rows, F.front_planes, A);
    else hipLaunchKernelGGL(kernel, dim3(F.B), block, 0, stream, F.rows, F.front_planes, A);
}

void launch_recheck_slow(const FillBatch& F, const DevVocab& Vd, int32_t* bitmask_dev, int64_t row_stride_words,
                         const SlowScratch& S, hipStream_t stream) {
    hipLaunchKernelGGL(k_recheck_slow, dim3(S.n_lanes / 64), dim3(64), 0, stream, F, Vd, bitmask_dev, (long long)row_stride_words, S);
}

// Ordinary stores leave the logits in the last-level cache (256 MB), where the next pass over them finds them; logits that do
// not fit there push each other out, and streaming stores take them straight to memory.  Ordinary / streaming, us, nearly
// everything masked: 205 MB 33 / 39, 233 MB 39 / 40, 266 MB (below the line) 46 / 51, 273 MB (above) 57 / 46, 311 MB 70 / 52.
constexpr long long APPLY_STREAM_BYTES = 256ll << 20, APPLY_HUGE_BYTES = 384ll << 20, APPLY_LARGE_BYTES = 64ll << 20, APPLY_TINY_BYTES = 8ll << 20;

template <class E>
static void launch_apply_as(E* logits, int32_t B, int32_t V, int64_t row_stride_elems, const uint32_t* bm, int64_t bm_row_stride_words, hipStream_t stream) {
    if (reinterpret_cast<uintptr_t>(logits) % sizeof(E) != 0 || V > 1 << 30) {
        hipLaunchKernelGGL(k_apply_scalar<E>, dim3(V / 256 + (V % 256 != 0), B), dim3(256), 0, stream, logits, (long long)row_stride_elems, V, bm, (long long)bm_row_stride_words);
        return;
    }
    // a row that begins `before` elements behind a 128-byte boundary has that much more to cover
    const uint32_t pieces = ((uint32_t)V + 128 / sizeof(E) - 1 + APPLY_WAVE - 1) / APPLY_WAVE;
    // few pieces: a workgroup each, to reach as many compute units (one row, V = 32,000, fp32: 3.7 us against 4.0); many: four share one
    // (1,024 rows, V = 151,936, bf16, nothing masked: 6.2 us against 17.5, which is how long it takes to start the workgroups)
    const uint32_t waves = (uint64_t)pieces * (uint32_t)B <= 512 ? 1 : APPLY_WAVES;
    const long long bytes = (long long)B * V * (int)sizeof(E);
    auto* const kernel = bytes > APPLY_HUGE_BYTES ? k_apply_vec<E, APPLY_HUGE> : bytes > APPLY_STREAM_BYTES ? k_apply_vec<E, APPLY_STREAM>
                         : bytes > APPLY_LARGE_BYTES ? k_apply_vec<E, APPLY_LARGE> : bytes > APPLY_TINY_BYTES ? k_apply_vec<E, APPLY_SMALL> : k_apply_vec<E, APPLY_TINY>;
    hipLaunchKernelGGL(kernel, dim3((pieces + waves - 1) / waves, B), dim3(64 * waves), 0, stream, logits, (long long)row_stride_elems, V, bm,
                       (long long)bm_row_stride_words);
}

void launch_apply(void* logits_dev, int32_t dtype, int32_t B, int32_t V, int64_t row_stride_elems,
                  const int32_t* bitmask_dev, int64_t bm_row_stride_words, hipStream_t stream) {
    if (B == 0 || V == 0) return;
    const uint32_t* bm = reinterpret_cast<const uint32_t*>(bitmask_dev);
    if (dtype == 0) launch_apply_as((uint32_t*)logits_dev, B, V, row_stride_elems, bm, bm_row_stride_words, stream);
    else launch_apply_as((uint16_t*)logits_dev, B, V, row_stride_elems, bm, bm_row_stride_words, stream);
}

}  // namespace xg2
