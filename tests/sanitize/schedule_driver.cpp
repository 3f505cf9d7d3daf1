// Host-only check of the launch schedules (deft_plan.cpp), built with -fsanitize=address,undefined by
// tests/test_schedule.py: for random forests, every split, head counts and ratios, the image of a plan holds each chunk's
// row tiles exactly once in either task set, whole calls join only consecutive chunks with the same queries, and only in
// the two flattened splits, every query's list in the whole call's set is its list in the plan less the slots of chunks
// that are not the first of their run, and the size that deft_plan_device_bytes states is enough.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <vector>

#include "deft.h"
#include "deft_internal.h"

static uint64_t state = 0x2545f4914f6cdd1dull;
static uint32_t rnd() {
    state = state * 6364136223846793005ull + 1442695040888963407ull;
    return (uint32_t)(state >> 33);
}
static int32_t below(int32_t n) { return (int32_t)(rnd() % (uint32_t)n); }

#define CHECK(x) do { if (!(x)) { printf("plan %d mode %u G %d Hkv %d: %s (line %d)\n", it, mode, G, Hkv, #x, __LINE__); return 1; } } while (0)

int main() {
    using namespace deft;
    long joined = 0, lists = 0;
    for (int it = 0; it < 1200; ++it) {
        const bool big = it % 4 == 0;
        const int32_t n = 1 + below(big ? 120 : 12), nq = below(big ? 300 : 20), root = below(3) ? 0 : below(6000);
        std::vector<int32_t> begin(n), len(n), parent(n), qn(nq);
        int32_t cur = 0;
        for (int32_t u = 0; u < n; ++u) {
            parent[u] = u == 0 || below(9) == 0 ? -1 : (below(3) ? 0 : below(u));
            len[u] = u == 0 ? root : (below(6) == 0 ? 0 : below(300));
            begin[u] = cur;
            cur += len[u];
        }
        for (int32_t &q : qn) q = below(n);
        const uint32_t mode = (uint32_t)below(5);
        const int32_t G = 1 << below(5), Hkv = 1 << below(7), chunk = 32 << below(6);
        deft_plan_t *P = nullptr;
        CHECK(deft_plan(begin.data(), len.data(), parent.data(), n, nq ? qn.data() : nullptr, nq, cur, chunk,
                        mode | DEFT_ROWS_PER_QUERY(G), &P) == DEFT_OK);
        CHECK(deft_plan_device_bytes(P, G, 1) == deft_plan_device_bytes(P, G * Hkv, Hkv));
        CHECK(find_schedule(P, G) == nullptr);
        const Schedule *S = get_schedule(P, G, Hkv);
        CHECK(S->bytes == S->host_image.size() && S->bytes <= deft_plan_device_bytes(P, G * Hkv, Hkv));
        auto at = [&](size_t off) { return reinterpret_cast<const int32_t *>(S->host_image.data() + off); };
        for (const TaskSet *T : {&S->by_chunk, &S->fused}) {
            std::map<int32_t, int32_t> run_chunks, run_tiles;  // by first chunk
            int32_t precise = 0;
            for (int32_t i = 0; i < T->n_items; ++i) {
                const int32_t *d = at(T->off_items) + (size_t)i * kItemInts, c0 = d[kItChunk], k = d[kItChunks];
                int32_t tokens = 0, short_path = 0;
                CHECK(k >= 1 && c0 >= 0 && c0 + k <= P->n_chunks() && d[kItNTiles] >= 1 && d[kItNTiles] <= kMaxTilesPerTask);
                for (int32_t c = c0; c < c0 + k; ++c) {
                    CHECK(P->chunk_qlo[c] == d[kItQlo] && P->chunk_qhi[c] == d[kItQlo] + d[kItWidth]);
                    CHECK(P->chunk_slot_base[c] == d[kItSlotBase] + (c - c0) * d[kItWidth]);
                    for (int32_t s = P->chunk_seg_ptr[c]; s < P->chunk_seg_ptr[c + 1]; ++s) tokens += P->seg_len[s];
                }
                for (int32_t p = d[kItQlo]; p < d[kItQlo] + d[kItWidth]; ++p) short_path |= P->q_path_len[p] < kPreciseBelowTokens;
                CHECK(tokens == d[kItLen] && d[kItPrecise] == short_path && (k == 1 || tokens <= kJoinTokens));
                CHECK(d[kItSeg0] == P->chunk_seg_ptr[c0] && d[kItNSeg] == P->chunk_seg_ptr[c0 + k] - d[kItSeg0]);
                CHECK(run_tiles[c0] == d[kItTile0]);  // the tasks of a run come in the order of its rows
                run_tiles[c0] += d[kItNTiles];
                CHECK(run_chunks.emplace(c0, k).first->second == k);
                precise += d[kItPrecise];
                joined += k > 1;
                CHECK(k == 1 || (T == &S->fused && (mode == DEFT_SPLIT_FLATTEN || mode == DEFT_SPLIT_BALANCED)));
            }
            CHECK(precise == T->n_items_precise);
            std::vector<char> first((size_t)P->n_chunks(), 0);
            int32_t next = 0;  // runs cover the chunks, in order and without a gap
            for (const auto &r : run_chunks) {
                CHECK(r.first == next);
                next += r.second;
                first[r.first] = 1;
                const int64_t rows = (int64_t)(P->chunk_qhi[r.first] - P->chunk_qlo[r.first]) * G;
                CHECK(run_tiles[r.first] == (rows + 15) / 16);
            }
            CHECK(next == P->n_chunks());
            int32_t most = 0;
            for (int32_t p = 0; p < nq; ++p) {
                std::vector<int32_t> want;
                for (int32_t i = P->q_part_ptr[p]; i < P->q_part_ptr[p + 1]; ++i)
                    if (first[P->q_part_chunk[i]]) want.push_back(P->q_part_slot[i]);
                const int32_t *h = at(T->off_q_head) + (size_t)p * T->head_ints, room = T->head_ints - kQueryHeadFixed;
                CHECK(h[0] == (int32_t)want.size() && h[1] == P->q_order[p]);
                for (int32_t i = 0; i < h[0]; ++i) {
                    CHECK(i >= room || h[kQueryHeadFixed + i] == want[i]);
                    if (h[0] > room) CHECK(at(T->off_q_part_slot)[h[2] + i] == want[i]);
                }
                lists += h[0] > room;
                most = std::max(most, h[0]);
            }
            CHECK(most == T->max_parts);
        }
        deft_plan_destroy(P);
    }
    printf("schedules checked, %ld joined tasks, %ld lists past a record\n", joined, lists);
    return joined > 500 && lists > 500 ? 0 : 2;
}
