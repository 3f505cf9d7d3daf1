// Host-only check of the tasks of wide chunks cut anew (deft_plan.cpp, recut_runs), built with -fsanitize=address,undefined
// by tests/test_recut.py: for random trees with wide nodes (a root under leaves, two of them, a chain of them; with gaps between
// nodes, and paged), the tasks of the set hold every row tile of every token exactly once under the queries that see it, a task
// of one piece has no query that does not, every slot of the plan is written or marked empty exactly once, and a query's list
// names the slots that its tasks write.  Long tasks are at most one to a compute unit, and all are on the chip at once.
#include <cstdint>
#include <cstdio>
#include <map>
#include <set>
#include <utility>
#include <vector>

#include "deft.h"
#include "deft_internal.h"

static uint64_t state = 0x9e3779b97f4a7c15ull;
static int32_t below(int32_t n) {
    state = state * 6364136223846793005ull + 1442695040888963407ull;
    return (int32_t)((uint32_t)(state >> 33) % (uint32_t)n);
}

#define CHECK(x) do { if (!(x)) { printf("plan %d G %d Hkv %d: %s (line %d)\n", it, G, Hkv, #x, __LINE__); return 1; } } while (0)

int main() {
    using namespace deft;
    long sets = 0, rests = 0, whole = 0, several = 0;
    for (int it = 0; it < 1500; ++it) {
        const int32_t G = 1 + below(it & 1 ? 8 : 16), Hkv = 1 + below(32), leaves = 2 + (64 + below(300)) / G;
        const int32_t kind = below(3), shape = below(4);
        const int32_t page = below(4) ? 0 : 16, gap = below(3) ? 0 : 64 * below(2), inner = shape == 0 ? 2 : shape == 1 ? 3 : 1;
        const int32_t nodes = leaves + inner;
        std::vector<int32_t> begin(nodes), len(nodes), parent(nodes, 0), qn(leaves);
        for (int32_t u = 0, at = 0; u < nodes; at += len[u++] + gap) {
            const int32_t root = 32 * (20 + below(2500) / Hkv) + below(3) * below(32);
            len[u] = u < inner ? root : kind == 0 ? 1 : kind == 1 ? below(12) : (u == inner ? 300 : 1 + below(4));
            // shape 0: two trees of half the leaves each; 1: a chain of three wide nodes; else one root
            parent[u] = u < inner ? (shape == 1 ? u - 1 : -1) : shape == 0 ? (u - inner) * 2 / leaves : inner - 1;
            begin[u] = at;
            if (u >= inner) qn[u - inner] = u;
        }
        int32_t total = 0;
        for (int32_t n : len) total += n + gap;
        const uint32_t mode = below(2) ? DEFT_SPLIT_FLATTEN : DEFT_SPLIT_BALANCED;
        const int32_t chunk = 32 * (1 + below(16));
        deft_plan_t *P = nullptr;
        if (page) {  // every other page in its place, the others swapped: roots of several pieces
            std::vector<int32_t> ptr(1, 0), ids;
            for (int32_t u = 0; u < nodes; ++u) {
                for (int32_t i = 0; i < (len[u] + page - 1) / page; ++i) ids.push_back((int32_t)ids.size());
                ptr.push_back((int32_t)ids.size());
            }
            if (it & 1) for (size_t i = 0; i + 2 < ids.size(); i += 4) std::swap(ids[i], ids[i + 2]);
            CHECK(deft_plan_paged(ptr.data(), ids.data(), page, (int32_t)ids.size(), len.data(), parent.data(), nodes, qn.data(),
                                  leaves, chunk, mode | DEFT_ROWS_PER_QUERY(G), &P) == DEFT_OK);
        } else {
            CHECK(deft_plan(begin.data(), len.data(), parent.data(), nodes, qn.data(), leaves, total, chunk,
                            mode | DEFT_ROWS_PER_QUERY(G), &P) == DEFT_OK);
        }
        const Schedule *S = get_schedule(P, G, Hkv);
        CHECK(S->bytes == S->host_image.size() && S->bytes <= deft_plan_device_bytes(P, G * Hkv, Hkv));
        const TaskSet &T = S->recut;
        auto at = [&](size_t off) { return reinterpret_cast<const int32_t *>(S->host_image.data() + off); };
        std::map<int32_t, int32_t> tiles;                     // of a run, by its first slot
        std::set<int32_t> slots_done;                         // written or marked empty
        std::vector<std::set<int32_t>> written(leaves);       // by query
        const std::pair<int32_t, int32_t> nobody(-1, -1);
        std::vector<std::pair<int32_t, int32_t>> sees((size_t)P->ntok, nobody);  // queries that see a row of the cache; taken out
        for (int32_t s = 0; s < P->n_segs(); ++s)                                // when a task has it
            for (int32_t x = 0; x < P->seg_len[s]; ++x) sees[P->seg_tok_begin[s] + x] = {P->seg_qlo[s], P->seg_qhi[s]};
        for (int32_t i = 0; i < T.n_items; ++i) {
            const int32_t *d = at(T.off_items) + (size_t)i * kItemInts, lo = d[kItQlo], hi = lo + d[kItWidth];
            CHECK(d[kItNTiles] >= 1 && d[kItNTiles] <= kMaxTilesPerTask && d[kItChunks] >= 1 && d[kItLen] >= 1);
            CHECK(d[kItPieces] == 1 || d[kItPieces] == d[kItNSeg]);
            CHECK(tiles[d[kItSlotBase]] == d[kItTile0]);
            tiles[d[kItSlotBase]] += d[kItNTiles];
            if (d[kItTile0]) continue;
            whole += d[kItPieces] > 1 && d[kItChunk] > 0 && d[kItSeg0] == P->chunk_seg_ptr[d[kItChunk]] &&
                     P->seg_qlo[d[kItSeg0]] == lo && P->seg_qhi[d[kItSeg0]] == hi && P->chunk_qlo[d[kItChunk] - 1] == lo &&
                     P->chunk_qhi[d[kItChunk] - 1] == hi;
            for (int32_t k = 0; k < d[kItChunks] * d[kItWidth]; ++k) CHECK(slots_done.insert(d[kItSlotBase] + k).second);
            for (int32_t p = lo; p < hi; ++p) written[p].insert(d[kItSlotBase] + p - lo);
            std::vector<int32_t> rows;
            if (d[kItPieces] == 1) {
                for (int32_t x = 0; x < d[kItLen]; ++x) rows.push_back(d[kItBegin0] + x);
                CHECK(d[kItSegQlo0] == lo && d[kItSegQhi0] == hi);
            } else {
                rests += d[kItSeg0] > 0 && d[kItSeg0] > P->chunk_seg_ptr[d[kItChunk]];
                CHECK(d[kItBegin0] == P->seg_tok_begin[d[kItSeg0]]);
                for (int32_t s = d[kItSeg0]; s < d[kItSeg0] + d[kItNSeg]; ++s)
                    for (int32_t x = 0; x < P->seg_len[s]; ++x) rows.push_back(P->seg_tok_begin[s] + x);
            }
            CHECK((int32_t)rows.size() == d[kItLen]);
            for (int32_t r : rows) {
                CHECK(r >= 0 && r < P->ntok && sees[r] != nobody && sees[r].first >= lo && sees[r].second <= hi);
                if (d[kItPieces] == 1) CHECK(sees[r].first == lo && sees[r].second == hi);
                sees[r] = nobody;
            }
        }
        if (T.n_items) {
            ++sets;
            several += shape < 2;
            for (int32_t i = 0; i < T.n_items; ++i) {
                const int32_t *d = at(T.off_items) + (size_t)i * kItemInts;
                CHECK(tiles[d[kItSlotBase]] == (d[kItWidth] * G + 15) / 16);
                const int32_t fresh = d[kItFresh];
                CHECK(fresh >= 0 && (fresh & (fresh - 1)) == 0 && (fresh == 0 || d[kItPieces] == 1));
            }
            for (const auto &x : sees) CHECK(x == nobody);
            CHECK((int32_t)slots_done.size() == P->n_slots());
            int64_t groups = (int64_t)T.n_items * Hkv, of_long = 0;
            for (int32_t i = 0; i < T.n_items; ++i) of_long += at(T.off_items)[(size_t)i * kItemInts + kItLen] > kLongChunk ? Hkv : 0;
            CHECK(groups <= kResidentGroups && of_long <= kLongGroups && 4 * groups > 3 * kLongGroups);
            int32_t most = 0;
            for (int32_t p = 0; p < leaves; ++p) {
                const int32_t *h = at(T.off_q_head) + (size_t)p * T.head_ints, room = T.head_ints - kQueryHeadFixed;
                CHECK(h[0] == (int32_t)written[p].size() && h[1] == P->q_order[p]);
                std::set<int32_t> list;
                for (int32_t i = 0; i < h[0]; ++i) list.insert(h[0] > room ? at(T.off_q_part_slot)[h[2] + i] : h[kQueryHeadFixed + i]);
                CHECK(list == written[p]);
                most = std::max(most, h[0]);
            }
            CHECK(most == T.max_parts);
        }
        deft_plan_destroy(P);
    }
    // sets; with a rest of a last chunk, with a last chunk that stays whole, of trees with several wide nodes
    printf("recut sets checked: %ld, %ld with a rest, %ld whole chunks, %ld of several wide nodes\n", sets, rests, whole, several);
    return sets > 40 && rests > 10 && whole > 5 && several > 10 ? 0 : 2;
}
