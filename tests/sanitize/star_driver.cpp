// The tasks of a whole call at d = 128 on a star, a root under leaves of given lengths with one query each (deft_plan.cpp), built
// with -fsanitize=address,undefined by the tests: prints whether the chunks are cut anew (recut_runs), then one line per kind of
// task, "workgroups tokens tiles pieces".
//   star_driver Hq Hkv chunk flags root leaf...
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <vector>

#include "deft.h"
#include "deft_internal.h"

int main(int argc, char **argv) {
    using namespace deft;
    if (argc < 7) return 2;
    const int32_t Hq = atoi(argv[1]), Hkv = atoi(argv[2]), leaves = argc - 6;
    std::vector<int32_t> begin, len, parent, query;
    int32_t total = 0;
    for (int32_t u = 0; u <= leaves; ++u) {
        begin.push_back(total);
        len.push_back(atoi(argv[5 + u]));
        parent.push_back(u ? 0 : -1);
        if (u) query.push_back(u);
        total += len.back();
    }
    deft_plan_t *P = nullptr;
    if (deft_plan(begin.data(), len.data(), parent.data(), leaves + 1, query.data(), leaves, total, atoi(argv[3]),
                  (uint32_t)strtoul(argv[4], nullptr, 0), &P))
        return 1;
    const Schedule *S = get_schedule(P, Hq / Hkv, Hkv);
    const TaskSet &T = S->recut.n_items ? S->recut : S->fused;
    const int32_t *d = reinterpret_cast<const int32_t *>(S->host_image.data() + T.off_items);
    std::map<std::vector<int32_t>, int32_t> kinds;
    for (int32_t i = 0; i < T.n_items; ++i, d += kItemInts) kinds[{d[kItLen], d[kItNTiles], d[kItPieces]}] += Hkv;
    printf("%s\n", S->recut.n_items ? "cut anew" : "as planned");
    for (const auto &k : kinds) printf("%d %d %d %d\n", k.second, k.first[0], k.first[1], k.first[2]);
    deft_plan_destroy(P);
}
