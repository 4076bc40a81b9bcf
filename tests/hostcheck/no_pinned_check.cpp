// Host-only check that nothing is refused where no pinned host memory can be
// had (no device call: the HIP memory functions below take the runtime's
// place in this program): a plan, a flow and a projection are created and
// given back, with every allocation freed once; a plan and a flow ask for one
// buffer of it, a projection for none before its first call.  Prints "ok" or the first failure and
// exits non-zero.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <vector>

#include "pcx.h"
#include "pcx_flow.h"
#include "pcx_varcoef.h"

static bool pinned_ok = false;
static int pinned_asked = 0, bad_free = 0;
static std::map<void *, int> dev, host;

extern "C" {
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n)
{
    *p = std::malloc(n);
    dev[*p] = 1;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    bad_free += p && !dev.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    ++pinned_asked;
    if (!pinned_ok) return hipErrorOutOfMemory;
    *p = std::malloc(n);
    host[*p] = 1;
    return hipSuccess;
}
hipError_t hipHostFree(void *p)
{
    bad_free += p && !host.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return hipSuccess; }
}

static int expect(const char *what, pcx_status st)
{
    if (st == PCX_OK) return 0;
    std::printf("FAIL %s: status %d (%s)\n", what, (int)st, pcx_last_error());
    return 1;
}

int main()
{
    std::vector<double> zf(25);
    for (int k = 0; k <= 24; ++k) zf[k] = k / 24.0;
    pcx_grid g{};
    g.nx = 64; g.ny = 48; g.nz = 24;
    g.lx = g.ly = 1.0;
    g.zf = zf.data();
    g.bc_z = PCX_BC_WALL;
    pcx_options o{};
    o.precision = PCX_FP64;
    o.rtol = 1e-10;
    o.max_iters = 8;
    pcx_flow_params q{};
    q.rho1 = q.rho2 = q.gamma = q.eps = 1.0;
    for (bool ok : {false, true}) {
        pinned_ok = ok;
        for (int what = 0; what < 3; ++what) {
            pinned_asked = 0;
            if (what == 0) {
                pcx_plan h = nullptr;
                if (expect("pcx_plan_create", pcx_plan_create(&g, &o, &h))) return 1;
                pcx_plan_destroy(h);
            } else if (what == 1) {
                pcx_flow h = nullptr;
                if (expect("pcx_flow_create", pcx_flow_create(&g, &q, &o, &h))) return 1;
                pcx_flow_destroy(h);
            } else {
                pcx_varcoef h = nullptr;
                if (expect("pcx_varcoef_create", pcx_varcoef_create(&g, &o, &h))) return 1;
                pcx_varcoef_destroy(h);
            }
            if (pinned_asked != (what < 2) || bad_free || !dev.empty() || !host.empty()) {
                std::printf("FAIL handle %d, pinned memory %d: %d pinned buffers, %d bad frees, %zu and %zu left\n", what, (int)ok,
                            pinned_asked, bad_free, dev.size(), host.size());
                return 1;
            }
        }
    }
    std::printf("ok\n");
    return 0;
}
