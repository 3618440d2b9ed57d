// Launchers of the gfx950 kernels.  Plain pointers and sizes only; every pointer named *_dev is
// device memory.  All launches go to `stream`; none of them synchronises.
#pragma once
#include <cstdint>
#include <hip/hip_runtime.h>

namespace xg2 {

struct DevTables {                       // packed grammar tables (see tables.hpp for the word layout)
    const uint4* state;                  // {rule, expansion offset, n_items, n_triples}: loaded only for states with
                                         // rule edges (what entering them adds) and for completing items (their rule)
    const uint32_t* exp_list;            // expansions: item words, then {rule, target} pairs
    const uint32_t* trans;               // [(n_states + 1) * n_classes] state reference of the byte target, or `sink`
    const uint32_t* byte_class_words;    // [64] byte -> class, four per word
    uint32_t n_classes;
    uint32_t sink;                       // the state (without flags) that missing edges lead to; its own row leads back to it
    const uint32_t* site_off;            // per rule: states in which referencing rules continue (CSR)
    const uint32_t* site_tgt;
};

// A token by its id: what a parse of it starts from, in one load.
struct alignas(16) TokenRecord {
    uint4 head;                          // its first 16 bytes, zero padded
    uint32_t off, n_bytes;               // its place in DevVocab::bytes; 0 bytes: never checked (special or empty)
    uint32_t pad[2];
};
struct DevVocab {                        // byte-sorted vocabulary in HBM
    const uint8_t* bytes;                // concatenated token bytes in sorted order
    const uint32_t* off;                 // [n_sorted + 1]
    const uint4* tok16;                  // [n_sorted] first 16 bytes of each token, zero padded: one coalesced load
                                         // instead of sixteen byte loads for the tokens the LDS path handles
    const uint32_t* perm;                // sorted rank -> token id
    const uint32_t* rank;                // token id -> sorted rank, 0xFFFFFFFF for tokens never checked
    const uint32_t* long_rank;           // per length bound d, ascending: the sorted ranks of the tokens longer than d bytes
    const TokenRecord* rec;              // [V] by token id
    uint32_t n_sorted;                   // checkable tokens (non-special, non-empty)
    uint32_t V, W;
};

// Work plan of one cache build.  A chunk is a record of two uint4: the first {plane, first rank, end rank, flags}, the
// second what the automaton walk needs of the plane without a further load {first item of the start set, number of
// its items, row address low, row address high}.  Below, chunk[c] stands for the first half of record c.
// Chunk c covers sorted ranks [chunk[c].y, chunk[c].z) of plane chunk[c].x
// (at most build_chunk() tokens, all with a first byte the plane's start set can read); with bit 0 of chunk[c].w
// set, y and z index DevVocab::long_rank instead and the ranks are read from there (a plane that needs only
// its long tokens checked).  The workgroups of a persistent grid take chunks round-robin.  plane_ctx[k] = {first item, number of items, first wait offset, H} describes the closed start
// set of plane k as a scan context (H = 1: the position alone; H = 2: the position inside one level of
// referencing rule).  ctx_wait holds, set after set, what the waiting items wait for as pairs
// {rule, state reference of the target | origin << 21}; ctx_wait_off counts pairs.  With bit 2 of chunk[c].w set,
// four more words follow the plane's items in ctx_items: {item a, lead a, item b or kNoThread, lead b}, the start
// set's one or two scanning items and, for an item of a waited-for instance, the item of the outermost instance
// that its end leads to (the only wait entry of its rule; neither predicts) — the kernel walks these as threads.
#ifndef XG2_BUILD_CHUNK
#define XG2_BUILD_CHUNK 128
#endif
constexpr uint32_t kBuildChunk = XG2_BUILD_CHUNK;
// Ranks of a chunk, for a launch that has n_full chunks of kBuildChunk.  In a small launch workgroups take one or two chunks and it
// lasts as long as its slowest, and a chunk of half the size goes through each phase once (64 tokens, a wavefront's lanes) and not
// twice.  In a large one a chunk's fixed costs and part-filled batches count.  The line is the number of wavefront slots of the
// device (wave_slots), where the measured times change sides.  k_build, us, 128 / 64
// ranks: 16 - 740 chunks of a just-in-time build 29.7 / 21.7 on average, 1,901 chunks 53.5 / 44.3, 3,509 67.7 / 48.6, 6,248 64.9 / 49.4,
// 6,506 64.3 / 52.6, but 9,892 82.7 / 86.6, 9,963 66.0 / 79.1, 13,000 123.7 / 133.8 (17,000 - 30,000: 6 - 14 % less again).  32 ranks: no
// gain just in time (22.0), 77.6 at 6,506.
uint32_t wave_slots();                                       // wavefronts that the device has slots for: 32 a compute unit
constexpr uint32_t build_chunk(size_t n_full, uint32_t slots) { return n_full <= slots ? 64 : kBuildChunk; }
static_assert(kBuildChunk >= 64, "build_chunk makes chunks smaller, not larger");
static_assert(kBuildChunk <= 256, "the deferred list is sized for kBuildChunk and holds one-byte offsets");
struct BuildPlan {
    const uint4* chunk; uint32_t n_chunks;                      // 2 * n_chunks uint4
    const uint4* plane_ctx;                                     // [n_planes]
    const uint32_t* ctx_items; const uint2* ctx_wait; const uint32_t* ctx_wait_off;
    uint32_t* const* plane_ptr;                                 // [n_planes] accepted row; uncertain row at + W words, left-early row at + 2 W
    uint32_t follow_filter;                                     // drop uncertain tokens that no reference site can continue
    uint32_t large_lists, list_k, list_wm;                      // set by launch_build: long or short item lists; item and wait-entry capacity a lane
};

struct FillRow;
struct SlowScratch {                     // large-capacity per-lane Earley scratch in device memory
    uint32_t* mem; uint32_t n_lanes;     // mem holds n_lanes * kSlowSlots words
    uint32_t* list; uint32_t list_cap;   // overflow work list: pairs (a, b)
    uint32_t* count;                     // [0] = entries in list, [1] = sticky error flag; fill only: [2] = undecided pairs, [3] = pairs
                                         // that did not fit a lane's lists, whoever took them
    uint32_t k_cap, wm_cap;              // item and wait-entry capacity in use (at most kSlowK, kSlowWM; smaller only in tests
                                         // of the overflow handling); below the LDS lists' 16 / 32 those are skipped
    // fill only: where the (row, token) pairs that even these lists could not decide are reported: a counter and a list in
    // pinned host memory (device-side address; null: not reported), and, for matchers on the device, the slots' rows
    uint32_t* unresolved; uint32_t unresolved_cap;       // [0] = 1 if any, [1] = 1 if more than fit; pairs from word 2 on (the host presets them to ~0)
    FillRow* mark_rows;                                  // not null: rows[b].pad[1] gets the sticky error
};
constexpr uint32_t kSlowK = 256, kSlowWM = 1024, kSlowMaxLen = 1024;
constexpr uint32_t kSlowSearchBudget = 1u << 20;     // list entries one token may compare against in the device-memory lists
constexpr uint32_t kSlowLanes = 64 * 64;                      // lanes of the large-capacity scratch (the fixed array's has fewer)
constexpr uint32_t kSlowSlots = 2 * kSlowK + 2 * kSlowWM + kSlowMaxLen + 1;

constexpr uint32_t kChunkListed = 1u, kChunkHeavy = 2u, kChunkThreads = 4u, kChunkDerive = 8u;   // bits of chunk[c].w,
constexpr uint32_t kChunkStepShift = 8;                      //   and from this one on the ranks (words) that the chunks of its range have
constexpr uint32_t kDeriveChunk = 64;                        // mask words of a derive chunk: y and z are word indices there, and the second
                                                             // half of the record holds the address of the base plane's third row
constexpr uint32_t kNoThread = 0xFFFFFFFFu;                  // an empty slot of the thread walk (what the transition table holds for "no edge")

// dst gets, for the tokens in mask (token ids, W words), the bits src holds: all three rows of a plane at once
// (accepted at [0, W), uncertain at [W, 2 W), left early at [2 W, 3 W)).  The mask bits of dst must be clear before.
struct CopyJob { uint32_t* dst; const uint32_t* src; const uint32_t* mask; uint64_t pad; };
void launch_copy_masked(const CopyJob* jobs_dev, uint32_t n_jobs, uint32_t W, hipStream_t stream);
// dst gets src's accepted row and left-early row whole (mask unused): what a plane derived from another one shares with it.
void launch_copy_structure(const CopyJob* jobs_dev, uint32_t n_jobs, uint32_t W, hipStream_t stream);
// The same with the mask given by first bytes: dst gets the bits src holds for the tokens whose first byte is in the
// set `bytes` (256 bits).  first_byte_dev: first byte of every token id, padded to W * 32 entries.
struct FirstByteCopyJob { uint32_t* dst; const uint32_t* src; uint32_t bytes[8]; };
void launch_copy_first_byte(const FirstByteCopyJob* jobs_dev, uint32_t n_jobs, const uint8_t* first_byte_dev, uint32_t W, hipStream_t stream);

// Writes the chunk records of a build: thread r cuts range_a[r] = {plane, first rank, end rank, flags} into chunks of
// range_a[r].w >> kChunkStepShift ranks, records first[r], first[r] + 1, ..., each followed by range_b[r].
void launch_expand_chunks(const uint4* range_a_dev, const uint4* range_b_dev, const uint32_t* first_dev, uint32_t n_ranges,
                          uint4* chunk_dev, hipStream_t stream);
// One launch for what a build needs first: the copy of `bytes` (a multiple of 16) from pinned host memory (given by its
// device address) to dst_dev, the clearing of up to kStageZeroRanges ranges of words, and the chunk records (as
// launch_expand_chunks, but reading the ranges through the device addresses of their pinned host copies).
constexpr uint32_t kStageZeroRanges = 8;
struct StageZero { uint32_t* p[kStageZeroRanges]; uint64_t words[kStageZeroRanges]; uint32_t n; };
void launch_stage(void* dst_dev, const void* src_host_mapped, size_t bytes, const StageZero& Z, const uint4* range_a_host_mapped,
                  const uint4* range_b_host_mapped, const uint32_t* first_host_mapped, uint32_t n_ranges, uint4* chunk_dev, hipStream_t stream);
void launch_build(const DevTables& T, const DevVocab& Vd, BuildPlan P, const SlowScratch& S, hipStream_t stream);
void launch_build_slow(const DevTables& T, const DevVocab& Vd, const BuildPlan& P, const SlowScratch& S, hipStream_t stream);
// What a freshly classed plane still lacks: the bits it takes from other planes (either kind, or none: null sources).
// m_src under the token mask m_mask (all three rows, as launch_copy_masked); f_src for the tokens whose first byte is in
// f_bytes (as launch_copy_first_byte).  The sources must not themselves be planes that take bits in the same launch.
struct FinishJob { const uint32_t* m_src; const uint32_t* m_mask; const uint32_t* f_src; uint32_t f_bytes[8]; uint32_t pad[2]; };
// One pass over every built plane: the copies above, then what launch_plane_summary does, on the words in registers.
void launch_finish_planes(uint32_t* const* plane_ptr_dev, const FinishJob* jobs_dev, uint32_t n_pos, const uint8_t* first_byte_dev, uint32_t W,
                          uint32_t* counts_dev, hipStream_t stream);
// A plane in device memory: three rows of W words (accepted, uncertain, left early) and behind them the list of its
// uncertain tokens: word 0 = how many (the list holds them if that is at most kUncListWords - 1), then their token ids.
constexpr uint32_t kUncListWords = 64;
constexpr size_t plane_words(uint32_t W) { return (3 * (size_t)W + kUncListWords + 3) & ~(size_t)3; }   // rows start 16-byte aligned
// counts_dev[2p], counts_dev[2p + 1] = set bits of the accepted and of the uncertain row of plane p; also writes the
// plane's list of uncertain tokens
void launch_plane_summary(uint32_t* const* plane_ptr_dev, uint32_t n_pos, uint32_t W, uint32_t* counts_dev, hipStream_t stream);

// One row of a fill batch.
constexpr uint32_t kRowPlanes = 2;       // planes of the frontier that a row's record names itself
struct alignas(16) FillRow {
    uint32_t front_off, front_n;         // into front_planes
    uint32_t item_off, item_n;           // into ctx_items
    uint32_t wait_base;                  // into ctx_wait (pairs)
    uint32_t waitoff_off, H;             // into ctx_wait_off ([H + 1] entries, relative to wait_base)
    uint32_t tables_idx;                 // into tables
    uint32_t flags;                      // bit 0: root can end, bit 1: terminated
    uint32_t pad[2];
    uint32_t n_wait;                     // wait entries of the context: ctx_wait_off[waitoff_off + H]
    uint64_t planes[kRowPlanes];         // front_planes[front_off], ... again (as many as there are), so that their loads need wait for nothing
                                         // but the record
};
struct FillBatch {
    const FillRow* rows; uint32_t B;
    const uint64_t* front_planes;        // device addresses of accepted rows (uncertain at + W words, list of uncertain tokens at + 3 W);
                                         // bit 0 set: only the accepted row counts (root instance)
    const uint32_t* ctx_items; const uint2* ctx_wait; const uint32_t* ctx_wait_off;
    const DevTables* tables;
    uint32_t eos_id;
    // re-check scratch: candidate bits of every mask word; per row, the indices of the non-zero ones and their count
    uint32_t* cand_words;                // [B * W]
    uint32_t* work_list;                 // [B * W], row b's list starts at b * W
    uint32_t* row_count;                 // [B], written by the fill kernel: candidate tokens of the row
    uint32_t* zero_words;                // if not null: four words the fill kernel clears for the next call (the overflow list's length
                                         // and flag, where no upload brings them in as zeros: two sets take turns)
    uint32_t own_lanes;                  // lanes of the large-capacity scratch that are a row's own while k_fill runs (at most kFillOwnLanes: a
                                         // wavefront of it uses lane own_lanes * row + its number, and only if that is below own_lanes), or 0:
                                         // there are too few
    uint32_t follows;                    // k_recheck_slow is launched behind it and takes what the rows leave on the overflow list (always
                                         // if own_lanes is 0)
    uint32_t row_waves;                  // wavefronts of a row's workgroup: fill_row_waves()
    uint64_t* stamps;                    // if not null: when the call's work started and ended, on the device's constant-rate clock:
                                         // [0] the upload kernel's start; row_waves + 1 words for each row (start, end of each of
                                         // its wavefronts); the end of each workgroup of k_recheck_slow
};
// What k_fill handles how (the host decides by the same numbers whether k_recheck_slow follows).
constexpr uint32_t kFillLaneItems = 8, kFillLaneWaits = 12;  // lists of a lane that parses a token (of up to 16 bytes) by itself
constexpr uint32_t kFillWaveTokens = 4;                      // up to that many candidates for each wavefront of the workgroup get a wavefront each
constexpr uint32_t kFillWaveBytes = 64;                      // bytes of a token that a wavefront parses
constexpr uint32_t kFillPlaneTokens = kUncListWords - 1;     // with more uncertain tokens in a frontier plane (than its list holds), or in a
constexpr uint32_t kFillRowTokens = 2048;                    //   frontier (than any slot's can have otherwise), a row is worked through word by word
// Wavefronts of a row's workgroup, in a batch of `rows` rows on a device of `units` compute units: some frontier plane has `tokens`
// uncertain tokens, and rows have up to about `candidates` in all (k_fill has the figures).
constexpr uint32_t kFillMostWaves = 16, kFillOwnLanes = 6;
constexpr uint32_t fill_row_waves(uint32_t rows, uint32_t units, uint32_t tokens, uint32_t candidates) {
    if (rows <= units) return 16;
    if (tokens > kFillPlaneTokens) return rows <= 2 * units ? 12 : 6;
    if (candidates > 64) return 12;
    if (rows > 4 * units || candidates > 12 * kFillWaveTokens) return 6;
    return tokens > (rows <= 2 * units ? 2 : 6 * kFillWaveTokens) ? 12 : 6;
}
constexpr uint32_t kFillSpreadRows = 192, kFillSpreadTokens = 18;    // up to that many rows with more tokens than that, which may be longer than a wavefront takes
constexpr uint32_t kFillContextItems = 64, kFillContextSets = 240, kFillContextWaits = 512;   // contexts that wavefronts parse from (every slot's)
constexpr uint32_t kStampsRows = 1;
void launch_fill(const FillBatch& F, const DevVocab& Vd, int32_t* bitmask_dev, int64_t row_stride_words,
                 const SlowScratch& S, hipStream_t stream, hipEvent_t done = nullptr);
void launch_recheck_slow(const FillBatch& F, const DevVocab& Vd, int32_t* bitmask_dev, int64_t row_stride_words,
                         const SlowScratch& S, hipStream_t stream);

// ---- matchers that live on the device ------------------------------------------------------------------------
// What a matcher needs of its mask cache besides the tables: the plane of every (state) and (state, state the
// referencing rule continues in), as device addresses of accepted rows with bit 0 = "only the accepted row counts"
// (an all-zero uncertain row), and the matcher state a new sequence starts from.
struct CacheDev {
    DevTables T;
    const uint64_t* plain_row;           // [n_states] plane of a position without context (root rule, or context depth 1), 0 = none
    const uint32_t* pair_off;            // [n_states + 1] CSR over states: the planes of the state under its referencing sites
    const uint32_t* pair_key;            //   state id the referencing rule continues in (its class: site_rep), ascending within a state
    const uint64_t* pair_row;
    const uint32_t* site_rep;            // [n_states] the state that stands for each state's class as a site; null: every state for itself
    const uint32_t* site_of_off;         // [n_states + 1] site table (tables.hpp) over states x: for a rule after which a referencing rule
    const uint2* site_of;                //   continues in x, which of the rule's sites x is: plane of (state, x) = pair_row[pair_off[state] + that]
    uint32_t context_depth;
    uint32_t start_n_items, start_H, start_n_front, start_flags;
    uint32_t cls_words[64];              // T's byte classes: here, too, so that accepting a token need not wait for T to find them
    const uint32_t* start_items; const uint2* start_wait; const uint32_t* start_wait_off; const uint64_t* start_front;
};
// B matcher slots of fixed capacity.  Slot b's state is what FillRow b points at: its frontier planes at front[b * KF ..],
// and its parser context (items of the current closed set that can scan; per reachable older set what its waiting items
// wait for) in one of two buffers, c = rows[b].pad[0]: items[(c * B + b) * KI ..], wait[(c * B + b) * KW ..],
// wait_off[(c * B + b) * (KH + 1) ..].  Accepting a token writes the other buffer and switches.  rows[b].pad[1] holds a
// sticky error (a capacity was exceeded: the slot is unusable until it is reset), rows[b].tables_idx the slot's cache.
constexpr uint32_t kSlotItems = 64, kSlotSets = 240, kSlotWaits = 512, kSlotPlanes = 32;   // capacities of a matcher slot
constexpr uint32_t kMostSlots = 1u << 20;                    // slots of a batch
static_assert(2ull * kMostSlots * kSlotWaits <= 0xFFFFFFFFull, "places of items, sets and wait entries in a batch's arrays are 32-bit numbers of entries");
static_assert(kSlotItems <= kFillContextItems && kSlotSets <= kFillContextSets && kSlotWaits <= kFillContextWaits, "wavefronts can parse from every slot's context");
static_assert(kSlotPlanes * kFillPlaneTokens <= kFillRowTokens, "a slot's row goes word by word only for a plane without a list");
struct BatchDev {
    uint32_t B, KI, KH, KW, KF;                          // KI .. KF: the four capacities above
    FillRow* rows;
    uint64_t* front; uint32_t* items; uint2* wait; uint32_t* wait_off;
    const CacheDev* caches; const DevTables* tables;     // [number of caches in use] (tables: the same DevTables, as fill wants them)
    uint32_t* slow_mem;                                   // item lists in device memory for tokens the LDS lists cannot take: B * kSlowSlots words
    uint8_t* slow_map;                                    // and the set renumbering table: B * (KH + kSlowMaxLen + 1) bytes
    uint64_t* slow_front;                                 // B * KF staging words
};
constexpr int32_t kTokenReset = -2;      // xg2_batch_accept_tokens: "start a new sequence in this slot"
// status codes written per slot (the XG2_* values of the C ABI)
constexpr int32_t kAccOk = 0, kAccInvalid = -1, kAccRejected = -3, kAccOverflow = -4;
// rec_dev[id] for every token, from the other arrays of Vd.
void launch_token_records(const DevVocab& Vd, TokenRecord* rec_dev, hipStream_t stream);
void launch_accept(const BatchDev& D, const DevVocab& Vd, uint32_t eos_id, const int32_t* token_ids_dev, int32_t* status_dev, hipStream_t stream);
// rows_dev (n of them; nullptr = slots 0 .. n - 1) start a new sequence of cache `cache_idx`
void launch_batch_assign(const BatchDev& D, const int32_t* rows_dev, uint32_t n, uint32_t cache_idx, hipStream_t stream);

// Copies `bytes` (a multiple of 16) from pinned host memory, given by its device-side address, to device memory with
// a kernel, or the other way: for the small per-call transfers this has less latency than the copy engine.
void launch_upload(void* dst_dev, const void* src_host_mapped, size_t bytes, hipStream_t stream, uint64_t* stamp = nullptr, hipEvent_t done = nullptr);

// Up to 64 words := 0.
void launch_clear(uint32_t* words_dev, uint32_t n, hipStream_t stream);

// The entry point that allocates nothing works in a fixed device array of the library (one per GPU, kept until the
// process ends) instead of buffers that grow with the batch: staging of the per-row records, candidate words and
// work lists, row counts, the overflow list and the large-capacity item lists.  noalloc_scratch gives the array's
// device address on the current device (looked up once per device).
constexpr size_t kNoAllocStagingLimit = (size_t)1 << 20;            // per-row records (without the planes they repeat), frontier planes, context slices
constexpr size_t kNoAllocMaskWords = (size_t)1 << 20;               // rows x ceil(V/32) of one call
constexpr size_t kNoAllocMaxRows = 4096;
constexpr size_t kNoAllocStagingBytes = kNoAllocStagingLimit + kNoAllocMaxRows * sizeof(uint64_t) * kRowPlanes + 256;
constexpr uint32_t kNoAllocSlowLanes = 256, kNoAllocListCap = 1u << 16;
constexpr size_t kNoAllocScratchBytes = kNoAllocStagingBytes + 2 * kNoAllocMaskWords * 4 + kNoAllocMaxRows * 4
                                        + (size_t)kNoAllocListCap * 8 + (size_t)kNoAllocSlowLanes * kSlowSlots * 4;
hipError_t noalloc_scratch(void** ptr_out);

void launch_apply(void* logits_dev, int32_t dtype, int32_t B, int32_t V, int64_t row_stride_elems,
                  const int32_t* bitmask_dev, int64_t bm_row_stride_words, hipStream_t stream);

}  // namespace xg2
