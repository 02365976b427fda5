// Prints which passes of a step run on staged transforms for a grid, on the CPU:
//   dispatch nx ny nz medium [lds=BYTES] [hint|set:AXIS:R,R,..:TILE] ...
// medium: maps, water or lossless.  The plan arguments are given to
// kw_suggest_plan (hint) or kw_set_plan (set) in turn; their status is printed.
// engine.cpp is part of this program (its launch configuration is not public);
// hip_host_stub.cpp stands in for the HIP runtime and the kernel launchers.
#include "engine.cpp"

#include <cstdio>
#include <cstdlib>
#include <cstring>

int main(int argc, char **argv) {
    if (argc < 5) return 2;
    kw_grid g{};
    g.nx = std::atoi(argv[1]);
    g.ny = std::atoi(argv[2]);
    g.nz = std::atoi(argv[3]);
    g.dx = g.dy = g.dz = 1e-4;
    g.cfl = 0.3;
    const size_t n = (size_t)g.nx * g.ny * g.nz;
    const bool maps = !std::strcmp(argv[4], "maps"), lossless = !std::strcmp(argv[4], "lossless");
    kw_medium m{};
    m.alpha_power = 1.5;
    m.c0_scalar = 1500.0;
    m.rho0_scalar = 1000.0;
    m.alpha0_scalar = 0.75;
    m.bona_scalar = 5.0;
    m.flags = lossless ? 0 : KW_NONLINEAR | KW_ABSORBING;
    std::vector<float> c0, rho0;
    if (maps) {
        c0.assign(n, 1500.0f);
        rho0.assign(n, 1000.0f);
        for (size_t i = 0; i < n; i += 3) c0[i] = 1600.0f, rho0[i] = 1050.0f;
        m.c0 = c0.data();
        m.rho0 = rho0.data();
    }
    const size_t need = kw_workspace_size(&g, &m, nullptr, nullptr);
    void *ws = need ? std::aligned_alloc(256, (need + 255) / 256 * 256) : nullptr;
    kw_sim *s = nullptr;
    if (!ws || kw_create(&g, &m, nullptr, nullptr, ws, need, nullptr, &s) != KW_OK) {
        std::printf("error=%s\n", kw_last_error());
        return 1;
    }
    for (int i = 5; i < argc; ++i) {
        if (!std::strncmp(argv[i], "lds=", 4)) {
            s->max_lds = std::strtoul(argv[i] + 4, nullptr, 10);
            std::printf("status=%d ", pick_tiles(s, 0, 0));
            continue;
        }
        const bool hint = !std::strncmp(argv[i], "hint:", 5);
        char *p = argv[i] + (hint ? 5 : 4);
        const int axis = (int)std::strtol(p, &p, 10);
        std::vector<int32_t> rad;
        for (++p; *p && *p != ':'; p += *p == ',') rad.push_back((int32_t)std::strtol(p, &p, 10));
        const int tile = *p ? std::atoi(p + 1) : 0;
        const int32_t *r = rad.empty() ? nullptr : rad.data();
        std::printf("status=%d ", hint ? kw_suggest_plan(s, axis, r, (int32_t)rad.size(), tile)
                                       : kw_set_plan(s, axis, r, (int32_t)rad.size(), tile));
    }
    const LaunchCfg &c = s->cfg;
    const int nz = g.nz;
    std::printf("zs=%d zs_skip=%u ys=%d xs=%d xs_passes=%u planes=%u xs_adj=%u eng_x=%d eng_y=%d eng_z=%d "
                "routes=%u tb_x=%d tb_y=%d tb_z=%d lds_grad=%zu lds_div=%zu lds_absm=%zu\n",
                c.zs, c.zs_skip, c.ys, c.xs, c.xs_passes, c.planes, c.xs_adj, c.eng_x, c.eng_y, c.eng_z, kw_routes(s),
                c.tb_x, c.tb_y, c.tb_z, 8 * ((size_t)2 * nz + (size_t)(c.zs_grad3 ? 3 : 1) * nz * c.zs_tb_grad),
                8 * ((size_t)2 * nz + (size_t)nz * c.zs_tb), 8 * ((size_t)2 * nz + (size_t)2 * nz * c.zs_tb_absm));
    kw_destroy(s);
    std::free(ws);
    return 0;
}
