// Host-side context behind the opaque dirac_ctx handle.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

// What a batch run of some steps by choice q launches: the item count and, for the
// register tile, its passes, shape and ring.
struct BatchRun {
    int q = 0;
    int64_t nitems = 0, passes = 0;
    int shape = 0, ring = 0;
};

struct dirac_ctx {
    // lattice
    int ndim = 3;
    int64_t nx = 1, ny = 1, nz = 1;
    int dtype = 2;
    double dt = 0.0, rx = 0.0, ry = 0.0, rz = 0.0;
    unsigned flags = 0;
    int zh = 0;               // z-slab mode: halo planes per side (arrays hold nz + 2 zh planes)
    bool zbc = false;         // zero values outside the lattice instead of periodic wrap
    std::string err;

    // state: two caller-owned buffer sets; cur says which holds the state
    void *buf[2][8] = {};
    bool bound = false;
    int cur = 0;

    // caller-owned scratch (reductions, coefficient tables, gradient partials)
    void *scratch = nullptr;
    size_t scratch_bytes = 0;

    // mass and V(z) profile, or per-site theta
    double m = 0.0;
    std::vector<double> v_int, v_half;
    std::vector<double> w_int, w_half;    // Im V(z) (absorbing layers), empty if none
    bool tab_dirty = true;
    std::vector<double> tab_host64;
    void *theta[8] = {};
    bool site_mode = false;

    // gauge links (vector potential), caller-owned; links_on when bound
    void *links[24] = {};
    bool links_on = false;

    // kernel choice
    int kernel = 0, tile_y = 0, zchunk = 0;

    // batched lattices
    bool is_batch = false;
    int64_t count = 0;
    std::vector<int64_t> bnx, bny;
    std::vector<double> bdt;      // per-lattice time step (r_x = r_y = dt, unit spacing)
    std::vector<void *> bstate, bpartner, btheta;
    size_t batch_scratch_need = 0;
    int tune_choice = -1;
    hipGraph_t graph[2] = {};             // by the buffer set that holds the state before the run
    hipGraphExec_t graph_exec[2] = {};
    int64_t graph_n = -1;                 // what they were captured for: steps, mode, the tuner's choice
    int graph_mode = -1, graph_tune = -1;
    BatchRun graph_run;
    int64_t graph_flips = 0;              // ping-pong launches in a captured graph
    hipStream_t graph_stream = nullptr;
};

// The launches of dirac_batch_run's mode 1 over n steps, as dirac_route writes them.
std::string batch_route_text(const dirac_ctx *c, int64_t n);
