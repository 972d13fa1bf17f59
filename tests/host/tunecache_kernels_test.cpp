// CPU test of the kernels' id in the autotuner's JSON file (zb_tunecache.h): it reads back, a file
// without one or with another one does not apply, and one that is no string is refused.
#include <stdio.h>

#include <string>
#include <vector>

#include "zb_tunecache.h"

using zbh::TuneEntry;

static int fails = 0;
#define CHECK(c)                                               \
    do {                                                       \
        if (!(c)) {                                            \
            printf("check failed line %d: %s\n", __LINE__, #c); \
            ++fails;                                           \
        }                                                      \
    } while (0)

int main()
{
    const std::string arch = "gfx950:sramecc+:xnack-", id = "0123456789abcdef";
    const std::vector<TuneEntry> es = {{48, 150, 1, 64, 64, 1}};
    auto parse = [&](const std::string &t, std::string &kernels) {
        std::vector<TuneEntry> back;
        std::string a, err;
        int rt = 0;
        kernels = "unset";
        return zbh::tune_parse(t, 64, 4096, a, rt, back, err, &kernels) && a == arch && rt == 7 && back.size() == 1;
    };
    std::string k;
    const std::string with = zbh::tune_json(arch, 7, es, id);
    CHECK(parse(with, k) && k == id);
    CHECK(zbh::tune_applies(arch, 7, k, arch, 7, id));
    CHECK(!zbh::tune_applies(arch, 7, k, arch, 7, "0123456789abcdee"));
    CHECK(!zbh::tune_applies(arch, 8, k, arch, 7, id));
    CHECK(!zbh::tune_applies("gfx942", 7, k, arch, 7, id));
    // written by a library whose files name no kernels
    CHECK(parse(zbh::tune_json(arch, 7, es), k) && k.empty());
    CHECK(!zbh::tune_applies(arch, 7, k, arch, 7, id));
    CHECK(!zbh::tune_applies(arch, 7, "", arch, 7, ""));
    // not a string
    std::string bad = with;
    bad.replace(bad.find("\"" + id + "\""), id.size() + 2, "17");
    CHECK(!parse(bad, k));
    printf(fails ? "%d failures\n" : "tunecache kernels ok\n", fails);
    return fails ? 1 : 0;
}
