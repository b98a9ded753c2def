// The launches of a time step, recorded instead of run: hipLaunchKernel is
// defined here, so that the library's launchers hand over their grids and
// workgroups on any machine.  Exit status 0 when every expectation holds.
#include "ugks_internal.h"

#include <dlfcn.h>

#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

namespace {

struct Launch {
    std::string name;  // mangled name of the kernel's host stub
    dim3 grid, block;
    size_t lds;
};
std::vector<Launch> g_launches;
int g_checks = 0, g_fail = 0;

void expect(bool ok, const std::string &what)
{
    ++g_checks;
    if (!ok) {
        ++g_fail;
        std::fprintf(stderr, "FAILED: %s\n", what.c_str());
    }
}

// Parameters of a case as the launchers read them; no pointer is followed.
ugx::Params params(int dim, int fstore, int nc, int nv, int ntab, int chunk)
{
    ugx::Params p;
    std::memset(&p, 0, sizeof(p));
    p.dim = dim;
    p.fstore = fstore;
    p.nc = nc;
    p.nf = dim * nc;
    p.nv = nv;
    p.ntab = ntab;
    p.chunk = chunk;
    p.nchunk = chunk ? (nv + chunk - 1) / chunk : 0;
    return p;
}

// Every launch within HIP's limit of 2^32 - 1 work-items along a dimension;
// `per_cell` names kernels of one workgroup a cell, which must cover nc.
void expect_launchable(const std::string &what, int nc, const std::vector<std::string> &per_cell)
{
    for (const Launch &l : g_launches) {
        const unsigned long long x = (unsigned long long)l.grid.x * l.block.x, y = (unsigned long long)l.grid.y * l.block.y;
        expect(x < (1ull << 32) && y < (1ull << 32),
               what + ": " + l.name + " takes " + std::to_string(x) + " x " + std::to_string(y) + " work-items");
        for (const std::string &n : per_cell)
            if (l.name.find(n) != std::string::npos)
                expect((unsigned long long)l.grid.x * l.grid.y >= (unsigned long long)nc,
                       what + ": " + l.name + " does not reach every cell");
    }
    expect(!g_launches.empty(), what + ": no launch");
    g_launches.clear();
}

// The largest meshes: every kernel of a step can be launched.
void largest_meshes()
{
    for (int dim : {2, 3})
        for (int fs : {0, 1, 2})
            for (int ntab : {0, 60})
                for (int nc : {400, 4194304, 8388608, 16000000})
                    for (int nv : {1536, 1537, 5120, 5121, 16384}) {
                        const ugx::Params p = params(dim, fs, nc, nv, ntab, 1024);
                        const std::string what = std::to_string(dim) + "D, storage " + std::to_string(fs) + ", " +
                                                 std::to_string(nc) + " cells x " + std::to_string(nv);
                        const int all[2] = {0, nc};
                        for (bool bricks : {false, true}) {
                            if (bricks && fs != 0) continue;
                            (void)ugx::launch_push_step(p, nullptr, nullptr, true, nullptr, all, 1, bricks, nullptr, 0, nullptr);
                            expect_launchable(what + ", push", nc, {"k_push_final", "k_push_base"});
                        }
                        (void)ugx::launch_push_inplace(p, nullptr, nullptr, all, 1, nullptr, 0, nullptr);
                        expect_launchable(what + ", push in place", nc, {"k_push_final_inplace", "k_push_chunk_turn"});
                        (void)ugx::launch_sweep(p, nullptr, nullptr, nullptr);
                        expect_launchable(what + ", gather", nc, {"k_sweep"});
                        (void)ugx::launch_sweep_inplace(p, nullptr, true, nullptr);
                        expect_launchable(what + ", gather in place", nc, {"k_sweep", "k_wall_density"});
                        (void)ugx::launch_init(p, nullptr, nullptr, nullptr);
                        (void)ugx::launch_moments(p, nullptr, nullptr);
                        (void)ugx::launch_cfl(p, nullptr, nullptr);
                        expect_launchable(what + ", start", nc, {"k_init", "k_moments", "k_cfl"});
                        (void)ugx::launch_prologue(p, nullptr);
                        expect_launchable(what + ", prologue", nc, {});
                    }
}

}  // namespace

// A launch is pushed with its shape, popped by the kernel's host stub, and
// handed on with the stub's address; without a device the runtime's own
// functions refuse the first.
namespace {
Launch g_pushed;
}
extern "C" hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t)
{
    g_pushed = Launch{"", grid, block, lds};
    return hipSuccess;
}
extern "C" hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *stream)
{
    *grid = g_pushed.grid;
    *block = g_pushed.block;
    *lds = g_pushed.lds;
    *stream = nullptr;
    return hipSuccess;
}
extern "C" hipError_t hipLaunchKernel(const void *kernel, dim3 grid, dim3 block, void **, size_t lds, hipStream_t)
{
    Dl_info at;
    g_launches.push_back({dladdr(kernel, &at) && at.dli_sname ? at.dli_sname : "?", grid, block, lds});
    return hipSuccess;
}
extern "C" hipError_t hipGetLastError() { return hipSuccess; }

int main()
{
    largest_meshes();
    std::printf("%d checks, %d failed\n", g_checks, g_fail);
    return g_fail ? 1 : 0;
}
