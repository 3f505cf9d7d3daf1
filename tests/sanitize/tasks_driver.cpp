// The tasks of a whole call on one tree, a root and equal branches under the equal-token split (deft_plan.cpp), built with
// -fsanitize=address,undefined by tests/test_schedule.py: prints the workgroups of stage 1, and how many tasks are resident
// (at most resident_tokens long) although they have more row tiles than a task of one piece may have there.
//   tasks_driver root leaves length Hq Hkv chunk resident_tokens tiles_of_one_piece
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "deft.h"
#include "deft_internal.h"

int main(int argc, char **argv) {
    using namespace deft;
    if (argc != 9) return 2;
    const int32_t leaves = atoi(argv[2]), Hq = atoi(argv[4]), Hkv = atoi(argv[5]), tokens = atoi(argv[7]), tiles = atoi(argv[8]);
    std::vector<int32_t> len{atoi(argv[1])}, parent{-1}, begin{0}, query;
    for (int32_t i = 1; i <= leaves; ++i) {
        begin.push_back(begin.back() + len.back());
        len.push_back(atoi(argv[3]));
        parent.push_back(0);
        query.push_back(i);
    }
    deft_plan_t *P = nullptr;
    if (deft_plan(begin.data(), len.data(), parent.data(), leaves + 1, query.data(), leaves, begin.back() + len.back(), atoi(argv[6]), 0, &P)) return 1;
    const Schedule *S = get_schedule(P, Hq / Hkv, Hkv);
    const int32_t *it = reinterpret_cast<const int32_t *>(S->host_image.data() + S->fused.off_items);
    int wide = 0;
    for (int32_t i = 0; i < S->fused.n_items; ++i, it += kItemInts)
        wide += it[kItPieces] > 1 && it[kItNTiles] > tiles && it[kItLen] <= tokens;
    printf("%d %d\n", S->fused.n_items * Hkv, wide);
    deft_plan_destroy(P);
}
