// Host-only check of the momentum pass's chunks (no device call): every plane
// of every tile of a plan is in one chunk of one workgroup, the workgroups
// are no more than the partial-result slots a flow allocates, the chunk is
// the cheapest for a device that holds 768 of the kernel's workgroups, and
// the grids whose times the rule was taken from.  Prints "ok" or the first
// failure and exits non-zero.
#include <cstdio>
#include <vector>

#include "flow_tile.hpp"

using namespace pcx::flow;

static BoxList list_of(int nx, int ny, int nz, int per, TilePlan &p)
{
    FGrid G{};
    G.n[0] = nx; G.n[1] = ny; G.n[2] = nz;
    for (int d = 0; d < 3; ++d) G.per[d] = per >> d & 1;
    p = tile_plan(G);
    return momentum_list(p);
}

int main()
{
    for (int nx : {4, 64, 70, 130, 200})
        for (int ny : {3, 6, 18, 54})
            for (int nz : {2, 3, 5, 17, 50, 64, 200})
                for (int per = 0; per < 8; ++per) {
                    TilePlan p;
                    const BoxList L = list_of(nx, ny, nz, per, p), all = box_list(p, true, true);
                    std::vector<int> seen((size_t)nz * ((nx + FTI - 1) / FTI) * ((ny + FTJ - 1) / FTJ), 0);
                    const int ti = (nx + FTI - 1) / FTI, tj = (ny + FTJ - 1) / FTJ;
                    int first = 0;
                    bool ok = L.n == p.n && L.grid <= p.nslots;
                    for (int q = 0; ok && q < L.n; ++q) {
                        const TileBox &b = L.box[q];
                        ok = L.first[q] == first && L.kend[q] == p.box[q].k0 + p.box[q].nk;
                        first += box_grid(b);
                        for (int c = 0; c < b.nk; ++c)
                            for (int k = b.k0 + c * L.ck; k < b.k0 + (c + 1) * L.ck && k < L.kend[q]; ++k)
                                for (int j = 0; j < b.njt; ++j)
                                    for (int i = 0; i < b.nit; ++i) ++seen[((size_t)k * tj + b.jt0 + j) * ti + b.it0 + i];
                    }
                    for (int v : seen) ok = ok && v == 1;
                    for (int c : {1, 2, 3, 4, 6, 8, 16, 32})
                        ok = ok && (L.grid + 767) / 768 * (L.ck + 3) <= (box_chunks(all, c).grid + 767) / 768 * (c + 3);
                    if (!ok) {
                        std::printf("FAIL %d x %d x %d periodic %d: chunks of %d planes\n", nx, ny, nz, per, L.ck);
                        return 1;
                    }
                }
    const struct { int nx, ny, nz, per, want; } at[] = {{512, 512, 512, 3, 32}, {256, 256, 256, 3, 16}, {256, 256, 256, 0, 16},
                                                        {128, 128, 128, 3, 6},  {512, 512, 64, 3, 16},  {144, 54, 50, 0, 3},
                                                        {64, 64, 64, 3, 2}};
    for (const auto &q : at) {
        TilePlan p;
        const int c = list_of(q.nx, q.ny, q.nz, q.per, p).ck;
        if (c != q.want) {
            std::printf("FAIL %d x %d x %d periodic %d: chunks of %d planes, not %d\n", q.nx, q.ny, q.nz, q.per, c, q.want);
            return 1;
        }
    }
    std::printf("ok\n");
    return 0;
}
