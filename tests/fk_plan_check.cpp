// CPU check of the forward-kinematics plan (build_fk_plan): for many trees the
// steps are walked as the kernel walks them; each joint must come once, after
// its parent and from its parent's frame, carry its own EEs, and the slots stay
// within PK_FK_MAX_SLOTS, for breadth-first orders too.
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>

#include "tree_layout.hpp"

using namespace pk;

static int failures = 0;

static int check(const std::vector<int> &parent, const std::vector<int> &ee, const char *what)
{
    RobotC *R = new RobotC;
    memset(R, 0, sizeof *R);
    const int n = R->n = (int)parent.size(), m = R->m = (int)ee.size();
    for (int j = 0; j < n; ++j) R->j[j].parent = parent[j];
    for (int k = 0; k < m; ++k) R->e[k].joint = ee[k];
    build_fk_plan(*R);
    const int slots = R->fk_slots;
    bool ok = slots >= 0 && slots <= PK_FK_MAX_SLOTS;
    int run = -2, held[PK_FK_MAX_SLOTS];
    for (int &h : held) h = -2;
    std::vector<int> seen(n, 0);
    for (int i = 0; i < n && ok; ++i) {
        const uint32_t w = R->fk_step[i], from = w >> 8 & 0xff, save = w >> 16 & 0xff;
        const int j = (int)(w & 0xff);
        ok = j < n && !seen[j]++ && (from >= PK_FK_RUN || (int)from < slots) &&
             (save == PK_FK_NONE || (int)save < slots);
        if (!ok) break;
        const int frame = from == PK_FK_BASE ? -1 : from == PK_FK_RUN ? run : held[from];
        uint32_t on = 0;
        for (int k = 0; k < m; ++k) on |= ee[k] == j ? 1u << k : 0;
        ok = frame == parent[j] && w >> 24 == on;
        run = j;
        if (save != PK_FK_NONE) held[save] = j;
    }
    if (!ok) {
        ++failures;
        printf("FAIL %s: n=%d slots=%d\n", what, n, slots);
    }
    delete R;
    return slots;
}

int main()
{
    std::mt19937 rng(1);
    auto pick = [&](int n) { return (int)(rng() % (unsigned)n); };
    for (int it = 0; it < 20000; ++it) {
        const int n = 1 + pick(PK_MAX_JOINTS), kind = it % 3, reach = 1 + pick(6);
        std::vector<int> parent(n), ee(1 + pick(PK_MAX_EES));
        for (int j = 0; j < n; ++j)
            parent[j] = kind == 0 ? pick(j + 1) - 1 : kind == 1 ? j - 1 - pick(j < reach ? j + 1 : reach) : (j + reach) / (reach + 1) - 1;
        for (int &e : ee) e = pick(n);
        check(parent, ee, "random");
    }
    std::vector<int> chain(64), star(64), binary(63);
    for (int j = 0; j < 64; ++j) {
        chain[j] = j - 1;
        star[j] = j < 32 ? -1 : j - 32;
    }
    for (int j = 0; j < 63; ++j) binary[j] = (j + 1) / 2 - 1;
    if (check(chain, {63}, "chain") != 0 || check(star, {40}, "star") != 0 || check(binary, {62}, "binary") != 5) {
        ++failures;
        printf("FAIL slots of the known trees\n");
    }
    printf("%d failures\n", failures);
    return failures ? 1 : 0;
}
