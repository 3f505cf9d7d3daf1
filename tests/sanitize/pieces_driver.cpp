// Host-only check of the piece counts in task descriptors (deft_plan.cpp), built with -fsanitize=address,undefined by
// tests/test_pieces.py: a task is written as one piece if and only if the rows of its tokens are consecutive and all of its
// segments have the same queries; the per-token table is long enough for every other task.
#include <cstdint>
#include <cstdio>
#include <numeric>
#include <utility>
#include <vector>

#include "deft.h"
#include "deft_internal.h"

static uint64_t state = 0x9e3779b97f4a7c15ull;
static int32_t below(int32_t n) {
    state = state * 6364136223846793005ull + 1442695040888963407ull;
    return (int32_t)((uint32_t)(state >> 33) % (uint32_t)n);
}

#define CHECK(x) do { if (!(x)) { printf("plan %d: %s (line %d)\n", it, #x, __LINE__); return 1; } } while (0)

int main() {
    using namespace deft;
    long merged = 0, apart = 0;
    for (int it = 0; it < 600; ++it) {
        const int32_t n = 1 + below(30), nq = 1 + below(60), P = 1 << below(6);
        const bool paged = it % 2;
        std::vector<int32_t> begin(n), len(n), parent(n), qn(nq), pptr{0}, pages;
        int32_t cur = 0;
        for (int32_t u = 0; u < n; ++u) {
            parent[u] = u == 0 ? -1 : below(3) ? 0 : below(u);
            len[u] = u == 0 ? below(4000) : below(300);
            begin[u] = cur;
            cur += len[u] + (below(3) ? 0 : below(9));  // gaps now and then
            for (int32_t i = 0; i < (len[u] + P - 1) / P; ++i) pages.push_back((int32_t)pages.size());
            pptr.push_back((int32_t)pages.size());
        }
        if (it % 4 == 1)  // pages in order, or some of them out of it
            for (int k = 0; k < 5 && pages.size() > 1; ++k) std::swap(pages[below((int32_t)pages.size())], pages[below((int32_t)pages.size())]);
        for (int32_t &q : qn) q = below(n);
        const uint32_t mode = it % 3 == 0 ? DEFT_SPLIT_BALANCED | DEFT_ROWS_PER_QUERY(4) : (uint32_t)below(4);
        const int32_t chunk = 32 << below(4);
        deft_plan_t *plan = nullptr;
        const int rc = paged ? deft_plan_paged(pptr.data(), pages.empty() ? pptr.data() : pages.data(), P, (int32_t)pages.size() + 1, len.data(), parent.data(), n,
                                               qn.data(), nq, chunk, mode, &plan)
                             : deft_plan(begin.data(), len.data(), parent.data(), n, qn.data(), nq, cur + 9, chunk, mode, &plan);
        if (rc == DEFT_EINVAL && (mode & 0xff) == DEFT_SPLIT_NODE) continue;  // a scattered node longer than a chunk may be
        CHECK(rc == DEFT_OK);
        const Schedule *S = get_schedule(plan, 4, 8);
        for (const TaskSet *T : {&S->by_chunk, &S->fused})
            for (int32_t i = 0; i < T->n_items; ++i) {
                const int32_t *d = reinterpret_cast<const int32_t *>(S->host_image.data() + T->off_items) + (size_t)i * kItemInts;
                const int32_t s0 = d[kItSeg0], s1 = s0 + d[kItNSeg];
                std::vector<int32_t> rows;
                bool same = true;
                for (int32_t s = s0; s < s1; ++s) {
                    for (int32_t x = 0; x < plan->seg_len[s]; ++x) rows.push_back(plan->seg_tok_begin[s] + x);
                    same = same && plan->seg_qlo[s] == d[kItQlo] && plan->seg_qhi[s] == d[kItQlo] + d[kItWidth];
                }
                CHECK((int32_t)rows.size() == d[kItLen] && rows[0] == d[kItBegin0]);
                for (size_t x = 1; x < rows.size(); ++x) same = same && rows[x] == rows[0] + (int32_t)x;
                CHECK(d[kItPieces] == (same ? 1 : d[kItNSeg]) && (!same || d[kItSegQlo0] == d[kItQlo]));
                CHECK(same || S->table_len >= d[kItLen]);
                merged += same && d[kItNSeg] > 1;
                apart += !same;
            }
        deft_plan_destroy(plan);
    }
    printf("pieces checked, %ld tasks of several segments as one, %ld not\n", merged, apart);
    return merged > 200 && apart > 200 ? 0 : 2;
}
