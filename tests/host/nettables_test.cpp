// CPU test of the packed network tables (zb_nettables.h) against the reactions themselves: every
// field at its limits (64 species, 4096 reactions, stoichiometry -2 to 2), row order, padding, the
// room past the rows, and no consumed-reaction rows where none are asked for.
#include <stdio.h>

#include <random>

#include "zb_nettables.h"

static int fails = 0;
#define CHECK(c)                                               \
    do {                                                       \
        if (!(c) && ++fails < 10)                              \
            printf("check failed line %d: %s\n", __LINE__, #c); \
    } while (0)

static void one(std::mt19937 &g, int ns, int nr, int hub)
{
    std::vector<int> ra(2 * nr), pa(2 * nr);
    std::vector<double> q(nr);
    for (int r = 0; r < nr; ++r) {
        for (int k = 0; k < 2; ++k) {
            ra[2 * r + k] = (int)(g() % ns);
            pa[2 * r + k] = (int)(g() % ns);
        }
        if (g() % 4 == 0) ra[2 * r + 1] = -1;
        if (g() % 4 == 0) pa[2 * r + 1] = -1;
        if (g() % 4 == 0) ra[2 * r + 1] = ra[2 * r];
        if (g() % 4 == 0) pa[2 * r] = ra[2 * r];
        if (hub && g() % 3) ra[2 * r] = ns - 1;
        q[r] = 1.0 + r;
    }
    const zbh::NetTables t = zbh::pack_network(ns, nr, ra.data(), pa.data(), q.data(), true);
    CHECK(t.inv_len % 4 == 0 && t.inv_len >= 4 && t.con_len % 4 == 0 && t.con_len >= 4);
    CHECK((int)t.inv.size() == ns * t.inv_len + 12);
    CHECK((int)t.con.size() == ns * t.con_len && t.con.size() == t.conq.size());
    CHECK((int)t.rct.size() == (nr ? nr : 1));
    for (int r = 0; r < nr; ++r) {
        CHECK((int)(t.rct[r] & 0xffffu) == 8 * ra[2 * r]);
        const int ob = (int)t.rct[r] >> 16;
        CHECK(ra[2 * r + 1] >= 0 ? ob == 8 * ra[2 * r + 1] : ob < 0);
    }
    int longest = 0, longest_con = 0;
    for (int i = 0; i < ns; ++i) {
        const unsigned *row = t.inv.data() + (size_t)i * t.inv_len;
        int n = 0;
        for (int r = 0; r < nr; ++r) {
            const int a = ra[2 * r], b = ra[2 * r + 1];
            const int nu = (pa[2 * r] == i) + (pa[2 * r + 1] == i) - (a == i) - (b == i);
            if (nu == 0) continue;
            CHECK(n < t.inv_len);
            const int e = (int)row[n++];
            CHECK((e & 0xffff) == 8 * r && ((e >> 16) & 63) == a && ((e >> 22) & 63) == (b >= 0 ? b : a) &&
                  (e >> 29) == nu);
        }
        longest = std::max(longest, n);
        for (; n < t.inv_len; ++n) CHECK(row[n] == (unsigned)(8 * nr));
        // the reactant places of the species, 64 reactions at a time, first places first
        const unsigned *con = t.con.data() + (size_t)i * t.con_len;
        const double *cq = t.conq.data() + (size_t)i * t.con_len;
        n = 0;
        for (int r0 = 0; r0 < nr; r0 += 64)
            for (int side = 0; side < 2; ++side)
                for (int r = r0; r < nr && r < r0 + 64; ++r)
                    if (ra[2 * r + side] == i) {
                        CHECK(n < t.con_len);
                        CHECK(con[n] == (unsigned)(8 * ((side + 1) * (nr + 1) + r)) && cq[n] == q[r]);
                        ++n;
                    }
        longest_con = std::max(longest_con, n);
        for (; n < t.con_len; ++n) CHECK(con[n] == (unsigned)(8 * nr) && cq[n] == 0.0);
    }
    CHECK(t.inv_len < longest + 4 || t.inv_len == 4);
    CHECK(t.con_len < longest_con + 4 || t.con_len == 4);
    const zbh::NetTables u = zbh::pack_network(ns, nr, ra.data(), pa.data(), q.data(), false);
    CHECK(u.con_len == 0 && u.con.empty() && u.conq.empty());
    CHECK(u.inv_len == t.inv_len && u.inv == t.inv && u.rct == t.rct);
}

int main()
{
    std::mt19937 g(17);
    for (int hub = 0; hub < 2; ++hub) {
        for (int it = 0; it < 200; ++it) one(g, 1 + (int)(g() % 64), (int)(g() % 200), hub);
        one(g, 64, 4096, hub);
        one(g, 1, 4096, hub);
        one(g, 64, 0, hub);
    }
    printf(fails ? "%d failures\n" : "net tables ok\n", fails);
    return fails ? 1 : 0;
}
