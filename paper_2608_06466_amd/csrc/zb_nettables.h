// The packed tables of a network as the kernels read them (DevNet), made on the host.  Free of
// HIP, so that a CPU test covers them under the sanitizers.
#pragma once

#include <stddef.h>

#include <algorithm>
#include <vector>

namespace zbh {

struct NetTables {
    int inv_len = 0, con_len = 0;
    std::vector<unsigned> rct, inv, con;
    std::vector<double> conq;
};

// Reactions as reactant[2 r], product[2 r] pairs (-1: absent), valid for ns <= 64 species, and
// their q.  consumed: also the con and conq rows (only kernels that hold the Jacobian rows in
// FP32 read them, and only with temperature); without it those are empty.
inline NetTables pack_network(int ns, int nr, const int *reactant, const int *product, const double *q,
                              bool consumed)
{
    NetTables t;
    t.rct.assign(std::max(nr, 1), 0u);
    // the species whose net stoichiometry in a reaction is not 0, each once
    auto involved = [&](int r, auto &&f) {
        const int x[4] = {reactant[2 * r], reactant[2 * r + 1], product[2 * r], product[2 * r + 1]};
        for (int k = 0; k < 4; ++k) {
            if (x[k] < 0 || std::find(x, x + k, x[k]) != x + k) continue;
            int nu = 0;
            for (int m = 0; m < 4; ++m)
                if (x[m] == x[k]) nu += m < 2 ? -1 : 1;
            if (nu != 0) f(x[k], nu);
        }
    };
    std::vector<int> n(ns, 0);
    for (int r = 0; r < nr; ++r) {
        t.rct[r] = (unsigned)(8 * reactant[2 * r]) | ((unsigned)(8 * reactant[2 * r + 1]) << 16);
        involved(r, [&](int i, int) { ++n[i]; });
    }
    // rows in whole loads of four entries
    auto row_len = [&] { return (std::max(4, ns ? *std::max_element(n.begin(), n.end()) : 0) + 3) & ~3; };
    t.inv_len = row_len();
    // padding: the 0 slot; room for the three loads the 14-row kernels make of every row
    t.inv.assign((size_t)ns * t.inv_len + 12, (unsigned)(8 * nr));
    std::fill(n.begin(), n.end(), 0);
    for (int r = 0; r < nr; ++r) {
        const int a = reactant[2 * r], b = reactant[2 * r + 1];
        const unsigned w = (unsigned)(8 * r) | (unsigned)a << 16 | (unsigned)(b >= 0 ? b : a) << 22;
        involved(r, [&](int i, int nu) { t.inv[(size_t)i * t.inv_len + n[i]++] = w | ((unsigned)nu << 29); });
    }
    if (!consumed) return t;
    std::fill(n.begin(), n.end(), 0);
    for (int k = 0; k < 2 * nr; ++k)
        if (reactant[k] >= 0) ++n[reactant[k]];
    t.con_len = row_len();
    t.con.assign((size_t)ns * t.con_len, (unsigned)(8 * nr));
    t.conq.assign((size_t)ns * t.con_len, 0.0);
    std::fill(n.begin(), n.end(), 0);
    for (int r0 = 0; r0 < nr; r0 += 64)
        for (int side = 0; side < 2; ++side)
            for (int r = r0; r < std::min(nr, r0 + 64); ++r) {
                const int i = reactant[2 * r + side];
                if (i < 0) continue;
                const size_t e = (size_t)i * t.con_len + n[i]++;
                t.con[e] = (unsigned)(8 * ((side + 1) * (nr + 1) + r));
                t.conq[e] = q[r];
            }
    return t;
}

}  // namespace zbh
