// Internal definitions shared by the planner (host C++) and the decode launcher (HIP).
#pragma once

#include <cstdint>
#include <map>
#include <mutex>
#include <vector>

#include "deft.h"

namespace deft {

// A stage-1 task is a (chunk, range of up to eight 16-row tiles) pair; with the KV head taken from the
// workgroup id it is the job of one workgroup.  Its descriptor is kItemInts int32, read with scalar
// loads, and carries everything the workgroup needs to start streaming a single-segment chunk
// without touching any other table.
constexpr int kItemInts = 16;
constexpr int kMaxTilesPerTask = 8;
// Stage 2 reads one record per plan query: {number of partials n, caller's query index, where its list starts in
// q_part_slot, the first slot ids}.  A record has kQueryHeadInts int32, or up to kQueryHeadMost where that holds the
// longest list of the plan and the records stay within kQueryHeadBytes: a slot id in the record saves a round trip (one
// query of 77 partials, whole call 12.2 us with the list, 11.7 with the record), but every query's record has the length
// of the longest, and the image is sent for every new plan.  Queries with more partials than fit go on to the list, which
// is left out where none has.
constexpr int kQueryHeadInts = 32;
constexpr int kQueryHeadMost = 128;
constexpr int kQueryHeadFixed = 3;
constexpr size_t kQueryHeadBytes = 16 * 1024;
enum ItemField {
    kItChunk = 0,     // chunk id
    kItTile0 = 1,     // first 16-row tile of the chunk's group handled by this task
    kItNTiles = 2,    // number of tiles, 1..kMaxTilesPerTask
    kItSeg0 = 3,      // first segment of the chunk
    kItNSeg = 4,      // number of segments
    kItQlo = 5,       // chunk_qlo
    kItWidth = 6,     // chunk_qhi - chunk_qlo
    kItSlotBase = 7,  // chunk_slot_base
    kItLen = 8,       // tokens in the chunk
    kItBegin0 = 9,    // first segment: physical row of its first token,
    kItSegQlo0 = 10,  //                its query interval
    kItSegQhi0 = 11,
    kItPrecise = 12,  // 1: the softmax weights enter the products as two bf16 terms (short paths, or on request)
    kItPieces = 14,   // segments to tell apart: 1 where they continue one another and have the same queries, else kItNSeg
    kItFresh = 15,    // blocks (a power of two) after which a stream of one piece starts a new reference; 0: it keeps one
    kItChunks = 13,   // chunks worked on as one: the result goes to the slots of the first, those of the others stay empty
};
// A group one of whose queries has fewer tokens than this on its whole path gets two-term weights.
constexpr int kPreciseBelowTokens = 1024;

// Row tiles to a task, from coarse to fine.  The schedule takes the finest cut whose workgroups are all on the chip at
// once: a row tile more in a task costs more than reading its chunk a second time from L2 (20 queries x 4 heads over 8
// KV heads, 288 -> 416 workgroups: stage 1 16.0 -> 12.2 us; 64 queries x 4 heads, d = 64: 13.5 -> 9.2 us), but a second
// round of workgroups costs more than either (432 workgroups cut to 680: 12.6 -> 16.2 us).
constexpr int kTaskTiles[] = {kMaxTilesPerTask, 4, 3, 2};
constexpr int kResidentGroups = 512;  // workgroups of stage 1 that an MI355X holds: two on each of 256 compute units

// Tasks of chunks longer than kLongChunk stream their tokens through LDS in steps that take as long for three row tiles
// as for four, and half as many steps for two (with d = 64 chunks of up to twice that can still be held in registers; the
// schedule serves both).  The wide ones among them (more than two tiles) have a cut of their own, to 4 or 2 tiles, as long
// as they stay at one to a compute unit: always where all workgroups then still fit the chip at once, and otherwise only if
// the longest task costs kLongestShare times the work of the launch per place on the chip (a task of several pieces, whose
// rows are looked up token by token, counts a third more).  More tasks read the chunk more often and form its weights in
// smaller batches, which a launch of several rounds pays for.  Whole call, us, uncut -> cut, by that ratio: 0.9 45.0 ->
// 49.2, 1.7 58.2 -> 66.8, 2.3 60.5 -> 71.6, 2.5 33.6 -> 38.2, 3.3 34.7 -> 38.5, 3.4 81.5 -> 90.8; with several pieces 4.5
// 37.8 -> 31.1, 4.5 54.3 -> 45.2, 6.0 37.7 -> 30.7; one piece 4.7 22.7 -> 17.1, 5.9 38.9 -> 25.6, 9.3 31.8 -> 22.5.
constexpr int kLongChunk = 256;
constexpr int kResidentTiles = 3;  // of a task of one piece that is held in registers, see is_resident in deft_decode.hip
constexpr int kLongGroups = kResidentGroups / 2;
constexpr int kLongestShare = 4;
constexpr int kRecutOthers = kLongGroups / 4;  // see recut_runs
constexpr int kJoinTokens = kLongChunk;  // chunks are joined up to the longest run that is not long

// Stage 1's tasks and the records with which stage 2 finds their partial results.
struct TaskSet {
    size_t off_items = 0;        // task descriptors
    size_t off_q_head = 0;       // per-query records for stage 2
    size_t off_q_part_slot = 0;  // per-query slot lists, where some query's does not fit its record
    int32_t n_items = 0;
    int32_t n_items_precise = 0;         // tasks among them that want two-term weights
    int32_t head_ints = kQueryHeadInts;  // int32 per record
    int32_t max_parts = 0;               // partials of the query that has most
};

// Launch schedule + image layout for one Hq/Hkv ratio.  The row cut and the joining of chunks suit the number of KV heads
// that an image was first uploaded for; the schedule is right for any.
struct Schedule {
    int32_t group = 0;        // G = Hq / Hkv, rows per query within one KV head
    int32_t Hkv = 0;          // KV heads that it suits
    size_t bytes = 0;         // total image size
    // byte offsets of the canonical arrays inside the image
    size_t off_seg_tok_begin = 0, off_seg_len = 0, off_seg_qlo = 0, off_seg_qhi = 0, off_seg_off = 0;
    size_t off_q_order = 0;
    TaskSet by_chunk;         // one partial result per (chunk, query of its group): what the two stages called apart use
    TaskSet fused;            // the same work on joined chunks: what a whole call uses; the same as by_chunk if none are
    TaskSet recut;            // wide chunks cut anew (recut_runs): for whole calls with d = 128 and Hkv KV heads, if there are any
    int32_t table_len = 32;   // longest chunk made of several pieces, rounded up to whole blocks: LDS table size
    std::vector<uint8_t> host_image;  // packed image, kept for repeated uploads
};

}  // namespace deft

struct deft_plan_s {
    int32_t chunk_size = 0, n_nodes = 0, nq = 0, ntok = 0, n_flat = 0;
    uint32_t mode = 0;  // DEFT_SPLIT_* / DEFT_GROUP_QUERY
    bool precise_all = false;  // DEFT_PRECISE_WEIGHTS was given
    std::vector<int32_t> q_path_len;  // tokens on the whole path of plan position p (saturating)

    // What the plan was built from and where its chunks start, kept so that deft_plan_update can tell what a new
    // tree has in common with this one and take over the chunks in front of the first change.
    uint32_t flags = 0;
    std::vector<int32_t> in_parent, in_query_node, in_tok_len, in_ext_ptr, in_ext_begin, in_ext_len;
    std::vector<int32_t> pre;              // depth-first order of the nodes
    std::vector<int32_t> chunk_first_i;    // position in `pre` of the node of a chunk's first piece,
    std::vector<int32_t> chunk_first_done; // tokens of that node that lie in earlier chunks,
    std::vector<int32_t> chunk_last_i;     // position in `pre` of the node of its last piece,
    std::vector<int64_t> chunk_flat_begin; // flattened position of its first token
    std::vector<int32_t> q_order, node_q_lo, node_q_hi;
    std::vector<int32_t> chunk_seg_ptr, seg_tok_begin, seg_len, seg_qlo, seg_qhi, seg_node;
    std::vector<int32_t> chunk_qlo, chunk_qhi, chunk_slot_base;
    std::vector<int32_t> seg_mask_ptr;
    std::vector<uint64_t> seg_mask;
    std::vector<int32_t> q_part_ptr, q_part_chunk, q_part_slot;

    int32_t n_chunks() const { return (int32_t)chunk_qlo.size(); }
    int32_t n_segs() const { return (int32_t)seg_len.size(); }
    int32_t n_slots() const { return chunk_slot_base.empty() ? 0 : chunk_slot_base.back(); }

    // schedules by G, built on demand (the canonical arrays above never change)
    mutable std::mutex mu;
    mutable std::map<int32_t, deft::Schedule> schedules;
};

namespace deft {
// Size of an image for G = Hq/Hkv that holds the schedule for any number of KV heads.
size_t image_bytes(const deft_plan_t *plan, int32_t group);
// The partial results of a plan, and the workspace that holds them and the marks a whole call in one launch needs.
size_t partials_bytes(const deft_plan_t *plan, int32_t Hq, int32_t d);
size_t workspace_bytes(const deft_plan_t *plan, int32_t Hq, int32_t d);
// Builds (or returns the cached) schedule for G = Hq/Hkv.  Thread-safe.
const Schedule *get_schedule(const deft_plan_t *plan, int32_t group, int32_t Hkv);
const Schedule *find_schedule(const deft_plan_t *plan, int32_t group);
}  // namespace deft

// deft_tree_attn_decode with another limit to the wait inside a call of one launch, 1 .. the library's: the result does not
// depend on it.  Not part of the interface; the tests see with it that a wait which is given up costs no result.
extern "C" int deft_decode_polls(const deft_plan_t *plan, const void *dev_image, const void *q, const void *k, const void *v, void *o,
                                 int32_t Hq, int32_t Hkv, int32_t d, float scale, uint32_t flags, void *workspace,
                                 size_t workspace_bytes, void *stream, int32_t polls);
