// pcx_plan.hpp -- host-side plan objects shared by the single-domain and
// batched forms.
#pragma once

#include <string>
#include <vector>

#include "pcx.h"
#include "pcx_dev.hpp"

namespace pcx {

struct Shapes {
    int tj = 8, tk = 8, zg = 64, smax = 8;
    int yth = 256, mth = 512, mthc = 1024, xth = 512;
    bool batch = false;
    int xfix = 0, yfix = 0; // lines per tile of the fixed-plan passes (0: general passes)
    // planes per chunk of the marching passes ([0] RHS and residual, [1]
    // correction); 0: chosen for a domain that has the device to itself
    int ckc[2] = {0, 0};
};

// Optional overrides picked by the autotuner (0 / empty = default).
struct TuneParams {
    int tj = 0, tk = 0, zg = 0;
};
struct RadixChoice {
    std::vector<int> x, y;
};

struct DomTables {
    void *dev = nullptr;
    size_t bytes = 0;
};

// Host image of a domain's device tables and the byte offset of each table
// in it (each 256-byte aligned).
struct HostTables {
    std::vector<char> bytes;
    size_t o_dzf = 0, o_idzf = 0, o_idzc = 0, o_rzlo = 0, o_rzhi = 0, o_za = 0, o_zb = 0, o_zc = 0, o_dzfs = 0,
           o_lx = 0, o_ly = 0, o_twr = 0, o_twx = 0, o_twy = 0, o_dcx = 0, o_dcy = 0;
};

// Byte offsets of a single-domain step's workspace pieces inside one region
// (each 256-byte aligned; r and ppart are used by the refined form only).
struct WsLayout {
    size_t s1 = 0, s2 = 0, f = 0, r = 0, stats = 0, psum = 0, xpart = 0, ppart = 0, spart = 0, total = 0;
};

extern thread_local std::string g_err;
pcx_status fail(pcx_status s, const std::string &msg);
FastDiv mkdiv(uint32_t d);
std::vector<int> default_radices(int n);
void fill_fft(FftDesc &fd, int n, const std::vector<int> &rad);
pcx_status validate_grid(const pcx_grid *g);
// Planes per chunk of a marching launch of txy tiles per plane that has the
// device (256 CUs, occ workgroups each) to itself: a workgroup takes about
// one memory latency per plane and three to start, so the launch takes
// rounds x (planes + 3).  At 32^3 the correction takes 12 us in 1-plane
// chunks against 46 in 16-plane ones, at 108 x 162 x 75 31 (7) against 49
// (16), at 256^3 229 (64) against 239 (16); at 512^3 1.62-1.65 ms in one
// chunk of 512 against 1.69 (128) and 1.83-1.85 (16).
// Chunks of more than `most` planes are whole columns only, of up to 128
// planes or in four rounds or more.  For the RHS and the residual `most` is
// 64: the columns of a launch drift apart, read halos their neighbours' cache
// lines no longer hold, and with few rounds nothing follows that would fill
// the CUs that are done early.  RHS at 512^3 (512 tiles a plane, one round of
// whole columns) 1.25-1.29 ms, in chunks of 128 1.22-1.29, of 64 1.21-1.23, of
// 16 1.26-1.28; 768 x 512 x 384 1.53 (192) and 1.49-1.50 (64); whole columns at
// 512 x 512 x 100 0.249 against 0.26 in two halves, at 1024 x 1024 x 512 (four
// rounds) 5.1-5.2 against 5.1-5.5 (64).  The correction has no such loss.
inline int march_chunk(int nz, long txy, int occ, int most)
{
    int best = nz;
    long cost = -1;
    for (int n = 1; n <= nz; ++n) {
        const int ckc = (nz + n - 1) / n;
        const long wgs = txy * ((nz + ckc - 1) / ckc), rounds = (wgs + 256L * occ - 1) / (256L * occ);
        const long c = rounds * (ckc + 3);
        if (ckc > most && (ckc < nz || (nz > 128 && rounds < 4))) continue;
        if (cost < 0 || c < cost) { cost = c; best = ckc; }
    }
    return best;
}
// lone: of a domain that has the device to itself
void choose_shapes(const pcx_grid &g, int prec, const TuneParams *tp, Shapes &sh, bool batch, bool lone = false);
void make_domain(const pcx_grid &g, int prec, const Shapes &sh, const RadixChoice *rc, HostTables &ht, Dom &d);
void bind_tables(Dom &d, const HostTables &ht, char *base);
pcx_status build_domain(const pcx_grid &g, int prec, const Shapes &sh, const RadixChoice *rc, DomTables &tb, Dom &d);
size_t lds_x(const Dom &d, int prec);
size_t lds_y(const Dom &d, int prec);
size_t lds_z(const Dom &d, int prec);
// grouped (batched) launches: the kernel variant, tile count and LDS bytes
// of pass `kind` for domain d
struct GVariant;
GVariant variant_of(const Dom &d, int kind);
long group_tiles(const Dom &d, int kind);
size_t group_lds(const Dom &d, int kind, int prec);

} // namespace pcx

struct pcx_plan_s;

namespace pcx {
// Pieces of plan creation shared by pcx_plan_create and the allocation-free
// step: option defaults, the host part of a plan (grid copy, shapes, domain
// descriptor and table image; no device call unless autotuning), the
// workspace layout of a prepared plan, and the binding of a plan to its
// tables and workspace in device memory.
pcx_status plan_options(const pcx_options *opts, pcx_options &o);
pcx_status plan_prepare(pcx_plan_s *P, const pcx_grid *grid, const pcx_options &o, HostTables &ht);
WsLayout plan_layout(const pcx_plan_s *P);
// The layout with columns and z-lines rounded up to whole 128-byte lines, or
// without the rounding where it alone would take the plan beyond `most` bytes.
WsLayout plan_layout_within(pcx_plan_s *P, size_t most);
// pcx_plan_create; words: with the plan's words of host memory.
pcx_status plan_create(const pcx_grid *grid, const pcx_options *opts, pcx_plan *out, bool words);
// The plan's words of host memory by their device address (host: hrep),
// allocated by the first call; NULL where no such memory can be had: the
// caller copies from the device instead.  The allocation takes 15-25 us, as
// much as the rest of a small plan's creation, and a call in the middle of a
// step waits for kernels on their way: a plan of a caller's and a flow's take
// it at creation, since a report or a substep follows, a projection's with
// its first iteration, of milliseconds.
unsigned long long *plan_host_words(pcx_plan_s *P);
void plan_bind(pcx_plan_s *P, const HostTables &ht, char *tables, char *ws, const WsLayout &L);
} // namespace pcx

struct pcx_plan_s {
    int device = 0;
    pcx_grid grid;
    std::vector<double> zf;
    pcx_options opt;
    int prec = 0;
    pcx::Shapes sh;
    pcx::DomTables tables;
    pcx::Dom dom;
    void *ws = nullptr;             // owned workspace region (pcx_plan_create); NULL when borrowed
    void *s1 = nullptr, *s2 = nullptr;
    double *f = nullptr;
    double *r = nullptr;
    double *psum = nullptr;
    // statistics and plane sums of a report in host memory, host and device
    // address, and one word more for the flow or the projection that owns the
    // plan (plan_host_words)
    unsigned long long *hrep = nullptr, *drep = nullptr;
    bool hrep_tried = false;
    size_t owner_word() const { return pcx::NSTAT + (size_t)grid.nz; }
    double *ppart = nullptr;
    double *xpart = nullptr;
    double *spart = nullptr;
    bool fuse_rhs = false;          // RHS evaluated inside the forward x pass
    bool fuse_resid = false;        // residual evaluated inside the forward x pass
    unsigned long long *stats = nullptr;
    size_t ws_bytes = 0;
    size_t lx = 0, ly = 0, lzs = 0;
    int timing = 0; // 0 off, 1 every pass, 2 the velocity correction only
    std::vector<hipEvent_t> ev;
    std::vector<std::string> names, pass_names;
    int nev = 0, npass = 0;
};
