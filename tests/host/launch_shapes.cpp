// The launches of a time step, recorded instead of run: hipLaunchKernel is
// defined here, so that the library's launchers hand over their grids and
// workgroups on any machine; copies are made between host arrays.  The host file is included for the push sweep's
// orders and colours.  Exit status 0 when every expectation holds.
#include "../../paper_2412_06546_amd/csrc/ugks_api.cpp"

#include <dlfcn.h>

#include <map>

namespace {

struct Launch {
    std::string name;  // mangled name of the kernel's host stub
    dim3 grid, block;
    size_t lds;
};
std::vector<Launch> g_launches;
size_t g_copied = 0;  // bytes of the copies since it was cleared
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
                        for (int bricks : {0, 512, 768}) {
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

// The final kernel: FP64 sums in a form that holds the slab with few pairs left
// empty, FP32 sums in workgroups of few wavefronts, more of them on a small mesh
// or with long tables.
void final_forms()
{
    for (int dim : {2, 3})
        for (int fs : {0, 1, 2})
            for (int nv = 1; nv <= 16384; ++nv) {
                const ugx::Params p = params(dim, fs, 20000, nv, 0, 0);
                g_launches.clear();
                (void)ugx::launch_push_step(p, nullptr, nullptr, false, nullptr, nullptr, 0, 0, nullptr, 0, nullptr);
                if (g_launches.size() != 1) {
                    expect(false, "one launch of a step without colours");
                    return;
                }
                const std::string &n = g_launches[0].name;
                const int bs = (int)g_launches[0].block.x;
                if (fs) {
                    expect(bs == (nv <= 2560 ? 64 : nv <= 5120 ? 128 : 256) && n.find("ELi" + std::to_string(bs) + "ELi0EEEv") != std::string::npos,
                           std::to_string(nv) + " velocities, FP32 sums: " + n);
                    continue;
                }
                int pairs = 0;
                for (int np : {3, 5, 8})
                    if (n.find("ELi" + std::to_string(bs) + "ELi" + std::to_string(np) + "EEEv") != std::string::npos) pairs = np;
                expect(2 * bs * pairs >= nv, std::to_string(nv) + " velocities do not fit " + n);
                if (nv > 3072) expect(2 * bs * (pairs - 3) < nv, std::to_string(nv) + " velocities leave pairs empty in " + n);
            }
    g_launches.clear();
    auto width = [&](int nc, int nv, int ntab) {
        g_launches.clear();
        (void)ugx::launch_push_step(params(2, 1, nc, nv, ntab, 0), nullptr, nullptr, true, nullptr, nullptr, 0, 0, nullptr, 0,
                                    nullptr);
        expect(g_launches.size() == 2 && g_launches[0].block.x == g_launches[1].block.x, "base and final kernel alike");
        return (int)g_launches[1].block.x;
    };
    expect(width(20000, 400, 800) == 256, "long tables");
    expect(width(512, 2145, 60) == 512 && width(512, 200, 60) == 128 && width(1331, 400, 60) == 128, "small mesh");
    g_launches.clear();
}

// A small class of cells is split down to one iteration a share, unless the
// tables that every share fills are long.
void cell_shares()
{
    auto shares = [](int dim, int cells, int nv, int ntab) {
        const int all[2] = {0, cells};
        g_launches.clear();
        (void)ugx::launch_push_step(params(dim, 1, cells, nv, ntab, 0), nullptr, nullptr, false, nullptr, all, 1, 0, nullptr, 0,
                                    nullptr);
        expect(g_launches.size() == 2, "a class and the final kernel");
        return (int)g_launches[0].grid.y;
    };
    expect(shares(3, 157, 1331, 33) == 6 && shares(3, 273, 2145, 0) == 9 && shares(2, 100, 3600, 120) == 15,
           "a class of few cells is not split");
    expect(shares(2, 1350, 400, 800) == 1 && shares(3, 500, 290, 870) == 1 && shares(2, 128, 4096, 800) == 8,
           "shares shorter than their tables");
    expect(shares(3, 40, 285, 855) == 2, "a class of very few cells is split all the same");
    g_launches.clear();
}

// Bricks only where the velocities fill the lanes, and a launch of few bricks
// on as many workgroups as their velocity iterations give.
void brick_launches()
{
    for (int dim : {2, 3})
        for (bool unordered : {false, true})
            for (int ntab : {0, 40, 75})
                for (int nv = 1; nv <= 16384; nv += nv < 2600 ? 1 : 97) {
                    const int w = ugx::brick_threads(dim, unordered, 1 << 20, nv, ntab);
                    const std::string what = std::to_string(dim) + "D, " + std::to_string(nv) + " velocities, " +
                                             std::to_string(ntab) + " table entries" + (unordered ? "" : ", colours");
                    expect(w == 0 || w == 512 || (w == 768 && ntab), what + ": width " + std::to_string(w));
                    if (!w) continue;
                    const int iters = (nv + w - 1) / w;
                    expect(nv >= (dim == 2 ? 0.65 : 0.775) * w * iters, what + ": lanes stand idle");
                    const int slots = 24 / (w / 64) * 256;
                    for (int bricks : {1, 3, 44, 137, 700, 5000}) {
                        const int all[2] = {0, 4 * bricks};
                        const ugx::Params p = params(dim, 0, 4 * bricks, nv, ntab, 0);
                        g_launches.clear();
                        (void)ugx::launch_push_step(p, nullptr, nullptr, false, nullptr, all, 1, w, nullptr, 0, nullptr);
                        expect(g_launches.size() == 2 && g_launches[0].name.find("k_push_brick") != std::string::npos,
                               what + ": not a brick launch");
                        const Launch &l = g_launches[0];
                        expect((int)l.block.x == w && (int)l.grid.x >= bricks && (int)l.grid.y <= iters, what + ": shape");
                        expect((int)l.grid.y * bricks >= std::min(iters * bricks, slots) / 2,
                               what + ": " + std::to_string(bricks) + " bricks leave the chip idle");
                        expect(l.lds + sizeof(double) * 4 * (dim == 2 ? 2 : 1) * w <= 80 * 1024, what + ": LDS");
                    }
                }
    // 5,600 velocities fill 512 threads better, but with 154 table entries in
    // 2D only the tables and sums of 768 leave room for all their workgroups
    expect(ugx::brick_threads(2, true, 12800, 5600, 154) == 768 && ugx::brick_threads(2, true, 12800, 5600, 120) == 512,
           "width by LDS");
    // small meshes, and velocity counts that leave most lanes idle
    for (int dim : {2, 3})
        for (int nv : {1, 37, 100, 216, 1025}) {
            expect(ugx::brick_threads(dim, true, 8191, 4548, 40) == 0 && ugx::brick_threads(dim, false, 32767, 4548, 40) == 0,
                   "small mesh");
            if (dim == 3 || nv < 300)
                expect(ugx::brick_threads(dim, true, 1 << 20, nv, 40) == 0, std::to_string(nv) + " velocities by bricks");
        }
}

// A lattice of n^3 cells with a share of them missing: cells and neighbours
// only, which is all that orders and colours read.
std::vector<ugx::CellGeo<3>> holed_lattice(int n, unsigned seed, int of_16)
{
    std::vector<int> id((size_t)n * n * n, -1);
    int nc = 0;
    unsigned r = seed;
    for (int &c : id) {
        r = r * 1664525u + 1013904223u;
        if ((int)(r >> 28) >= of_16) c = nc++;
    }
    std::vector<ugx::CellGeo<3>> g((size_t)nc);
    for (int z = 0, t = 0; z < n; ++z)
        for (int y = 0; y < n; ++y)
            for (int x = 0; x < n; ++x, ++t) {
                if (id[t] < 0) continue;
                ugx::CellGeo<3> &c = g[id[t]];
                std::memset(&c, 0, sizeof(c));
                const int d[6][3] = {{1, 0, 0}, {-1, 0, 0}, {0, 1, 0}, {0, -1, 0}, {0, 0, 1}, {0, 0, -1}};
                c.nf = 6;
                for (int j = 0; j < 6; ++j) {  // periodic in x
                    const int a = (x + d[j][0] + n) % n, b = y + d[j][1], e = z + d[j][2];
                    c.nb[j] = b < 0 || b >= n || e < 0 || e >= n ? -1 : id[((size_t)e * n + b) * n + a];
                }
            }
    return g;
}

// No stored cell may be written by two workgroups of a colour's launch: the
// order of the adds into it would be open.  A workgroup takes kBrickCells
// entries of the class, or one by cells, and writes them and their neighbours.
void colours_write_apart()
{
    for (int of_16 : {0, 3, 5, 9})
        for (int per : {1, ugx::kBrickCells}) {
            const auto g = holed_lattice(17, 7u + of_16, of_16);
            const int nc = (int)g.size();
            std::vector<int> order(nc), group(nc), cells, off;
            int n_groups = nc;
            for (int c = 0; c < nc; ++c) order[c] = group[c] = c;
            if (per > 1) order = brick_order<3>(g, per, group, n_groups);
            push_colours<3>(g, order, group, n_groups, cells, off);
            const std::string what = std::to_string(of_16) + "/16 holes, " + std::to_string(per) + " cells a workgroup";
            std::vector<int> seen(nc, 0);
            for (int c : cells) ++seen[c];
            expect(std::count(seen.begin(), seen.end(), 1) == nc, what + ": every cell once");
            std::map<int, int> sizes;
            for (int x : group) ++sizes[x];
            int alone = 0;
            for (auto &s : sizes) alone += s.second == 1;
            if (per > 1 && of_16) expect(alone > nc / 100, what + ": cells without a brick are missing from the test");
            for (size_t k = 0; k + 1 < off.size(); ++k) {
                std::vector<int> writer(nc, -1);
                for (int a = off[k]; a < off[k + 1]; ++a) {
                    const int wg = (a - off[k]) / per, c = cells[a];
                    auto write = [&](int x) {
                        if (x < 0) return;
                        expect(writer[x] < 0 || writer[x] == wg, what + ": cell " + std::to_string(x) + " has two writers");
                        writer[x] = wg;
                    };
                    write(c);
                    for (int j = 0; j < g[c].nf; ++j) write(g[c].nb[j]);
                }
            }
        }
}

// The read-out copies what it is asked for, and puts it in the caller's order.
void read_out()
{
    for (int dim : {2, 3})
        for (bool pinned : {false, true}) {
            const int nc = 70, NW = dim + 2;
            ugks h;
            h.dim = dim;
            h.nc = nc;
            std::vector<double> state((size_t)nc * (NW + dim)), staging(state.size());
            for (size_t i = 0; i < state.size(); ++i) state[i] = 1.0 + (double)i;
            for (int i = 0; i < nc; ++i) h.cell_of.push_back((i * 33) % nc);
            h.W = state.data();
            h.q = h.W + (size_t)nc * NW;
            h.h_macro = pinned ? staging.data() : nullptr;
            for (int ask = 0; ask < 4; ++ask) {
                std::vector<double> W((size_t)nc * NW, -1.0), q((size_t)nc * dim, -1.0);
                g_copied = 0;
                expect(ugks_macros(&h, ask & 1 ? W.data() : nullptr, ask & 2 ? q.data() : nullptr) == UGKS_OK, "macros");
                const std::string what = std::to_string(dim) + "D read-out " + std::to_string(ask);
                expect(g_copied == sizeof(double) * nc * ((ask & 1 ? NW : 0) + (ask & 2 ? dim : 0)),
                       what + " copies " + std::to_string(g_copied) + " bytes");
                for (int i = 0; i < nc; ++i) {
                    const int c = h.cell_of[i];
                    for (int m = 0; m < NW; ++m)
                        expect(W[(size_t)c * NW + m] == (ask & 1 ? h.W[(size_t)i * NW + m] : -1.0), what + ": W");
                    for (int d = 0; d < dim; ++d)
                        expect(q[(size_t)c * dim + d] == (ask & 2 ? h.q[(size_t)i * dim + d] : -1.0), what + ": q");
                }
            }
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
extern "C" hipError_t hipMemcpyAsync(void *to, const void *from, size_t bytes, hipMemcpyKind, hipStream_t)
{
    g_copied += bytes;
    std::memcpy(to, from, bytes);
    return hipSuccess;
}
extern "C" hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }

int main()
{
    largest_meshes();
    final_forms();
    cell_shares();
    brick_launches();
    colours_write_apart();
    read_out();
    std::printf("%d checks, %d failed\n", g_checks, g_fail);
    return g_fail ? 1 : 0;
}
