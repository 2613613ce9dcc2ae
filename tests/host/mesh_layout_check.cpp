// Host check of csrc/ram_mesh_layout.h: every table's place is aligned, holds what
// the kernels write and read there, ends before the next one, and nothing is reserved
// beyond what the tables and their alignment take.
#include <cstdio>
#include <cstdlib>

#include "ram_mesh_layout.h"

int main()
{
    for (int64_t n = 2; n < 40000; n += n < 600 ? 1 : 37) {
        const ram::MeshLayout m = ram::mesh_layout(n);
        const size_t c = (size_t)n, pad = c + 16;
        const struct { const char *name; size_t at, need; } t[] = {
            {"dx", m.dx, 8 * c},           {"dxinv", m.dxinv, 8 * c},
            {"hinv", m.hinv, 8 * c},       {"dxf", m.dxf, 4 * pad},
            {"dxinvf", m.dxinvf, 4 * pad}, {"hinvf", m.hinvf, 4 * c},
            {"bucket", m.bucket, 16 * c},  {"bnext", m.bnext, 64 * c},
            {"scal", m.scal, 24},          {"crf", m.crf, 64 * c},
            {"crd", m.crd, 112 * c},       {"rrf", m.rrf, 8 * pad},
            {"rrd", m.rrd, 16 * c},        {"stp", m.stp, 36 * c},
            {"stpd", m.stpd, 96 * c},      {"stdv", m.stdv, 36 * c},
            {"ppmd", m.ppmd, 40 * c},      {"ppmf", m.ppmf, 20 * c},
            {"nonu", m.nonu, 4 * (c + 1)}, {"nonu_min", m.nonu_min, 4 * (c + 1)},
            {"runs_size", m.runs_size, n > 16384 ? 16 * 513u : 0u},
            {"runs_cnt", m.runs_cnt, n > 16384 ? 8 * 512 * 8u : 0u},
        };
        const int k = (int)(sizeof(t) / sizeof(t[0]));
        size_t sum = 0;
        for (int i = 0; i < k; ++i) {
            const size_t end = i + 1 < k ? t[i + 1].at : m.bytes;
            if (t[i].at % 256 != 0 || t[i].at + t[i].need > end) {
                printf("n %lld: %s at %zu needs %zu, next at %zu\n", (long long)n, t[i].name, t[i].at,
                       t[i].need, end);
                return 1;
            }
            sum += t[i].need;
        }
        if (m.bytes > sum + 256 * (size_t)k) {
            printf("n %lld: %zu reserved for %zu\n", (long long)n, m.bytes, sum);
            return 1;
        }
    }
    printf("all checks passed\n");
    return 0;
}
