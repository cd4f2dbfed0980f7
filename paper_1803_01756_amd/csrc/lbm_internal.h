// Internal interface between the C-ABI runtime (lbm_runtime.cpp) and the
// HIP kernels (lbm_kernels.hip).  Not installed, not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace lbmk {

// Owned columns per wave-strip: 64 lanes minus a 5-column halo on each side
// (psi needs rho one column out, u needs psi one further, and each of the four
// RK4 stages widens the temperature stencil by one more column).
constexpr int kLanes = 64;
constexpr int kHalo = 5;
constexpr int kOwned = kLanes - 2 * kHalo;

// Tiles of the step: a workgroup of `waves` waves with `rows` rows each holds
// up to own() rows of a strip and their halo; per_simd is the number of waves
// per SIMD its register budget is held to.  The waves of a workgroup are a
// multiple of four, one share for each SIMD: with 9 or 10 a second workgroup
// does not fit beside the first (8192 x 512: 118 and 112 us for 96 with 8).
// FP32: Mid keeps three workgroups on a CU, Tall two; taller waves of five
// rows (5 x 8) leave four waves per SIMD and measured 87.3 against Tall's 84.3.
// Mass-exact storage keeps one FP64 density per row more: in Tall's 80
// registers it spills three and writes 31 MB of them per step (8192 x 512: 104
// us), so its tall tile is the 5 x 8 one (97.5; 4 x 8: 100.8).  Its Mid tile spills
// three as well.
// FP64: the halo exchange in LDS leaves one workgroup per CU.
struct TileShape {
    int rows, waves, per_simd;
    constexpr int own() const { return rows * waves - 2 * kHalo; }
};
enum { kTileFlat, kTileMid, kTileTall, kTileTallMX, kTileFlat64, kTileMid64, kTileTall64, kTileCount };
constexpr TileShape kTiles[kTileCount] = {{1, 16, 4}, {3, 8, 6},  {3, 12, 6}, {5, 8, 4},  // FP32
                                          {1, 16, 4}, {2, 16, 4}, {3, 12, 3}};  // FP64

// Constants that enter arithmetic done in the storage precision R, given in
// R on the host so that the kernels never convert them per use.
template <class R>
struct PhysR {
    // the collision's combinations of the Eq. 3 rates (collide())
    R se4, se12, se36;  // (1 - s_e)/4, s_e/12, s_e/36
    R q_u, q_F, q_th;   // the factors of rho u^2, u.F and |F_m|^2 / psi^2 in Q
    R xc, xd;           // s_q/12, (3 - 2 s_q)/12
    R b, rkA, rkB1, rkB2, inv_Cv, lam6;  // lam6 = lambda / 6
    R T_ref, dT_wall, rho_ref, rho_v, g_x, g_y;
    R rho_g, inv_drho, tau_g, dtau;
};

// Uniform physical constants, resolved on the host in FP64.  The kernels
// read them from the kernel-argument segment (scalar registers).
struct Phys {
    double rho_ref, T_ref, dT_wall;     // storage references; T_w - T_ref
    double a, b, R, kappa, inv_Tc;      // Eq. 11
    double two_inv_G, negG12;           // Eq. 10 (2/G) and Eq. 9 (-G/12)
    double psi_wall_eff;                // psi_w G_w / G: solid-row potential
    double Gw_psiw;                     // G_w psi_w (Eq. 14 on the wall rows)
    double tau_g, dtau, rho_g, inv_drho;// Eq. 5 (inv_drho = 0: constant tau)
    double inv_Cv, lambda;              // Eq. 16
    double g_osc, period, inv_period;   // drive g_osc sin(2 pi n / period) along +x
    double g_x, g_y, rho_v;             // Eq. 15
    double rho_frame;                   // reservoir density of a frame
    // open ends: inlet pressure p0 (1 + p_amp sin(...)); its EOS at the inlet
    // temperature T in e = in_e rho (b rho, CS: b rho / 4): in_A = R T / b (CS:
    // 4 R T / b), in_B = a phi(T) / b^2 (CS: 16 a / b^2), in_rho = 1 / in_e; and
    // the vapour spinodal density there (bracket)
    double p0, p_amp, p_period, inv_p_period;
    double in_e, in_rho, in_A, in_B, rho_sp;
    double dT_in;                       // inlet temperature - T_ref
    double dT_out;                      // held outlet temperature - T_ref (hold_out)
    int hold_out;                       // the outlet column holds its temperature
    double alpha_max;                   // > 0: cap of lambda / (rho C_v) in the conduction term
    double dT_w_end;                    // plate temperature at x = Nx-1 - T_ref
    int wall_ramp;                      // plate temperature linear in x
    double lam_l, cv_l;                 // liquid conductivity and heat capacity
    double dT_w_bot;                    // bottom plate temperature - T_ref (TOP_MIXED)
    int cold_x0, cold_x1;               // cold columns of the top plate (TOP_MIXED)
    double rkA, rkB1, rkB2;             // R, a k (1+k)/sqrt(Tc), a k^2 / Tc
    uint32_t flags;                     // LBM_FREEZE_T | LBM_SINGLE_PHASE | LBM_PERIODIC_Y
    uint32_t pad_;
    PhysR<float> rf;                    // the same constants in FP32 and FP64
    PhysR<double> rd;
};

struct Grid {
    int Nx, Ny;        // nodes incl. plate rows
    int pitch;         // elements per stored row (multiple of 64)
    int rows;          // stored (fluid) rows
    int y_first;       // y of stored row 0 (1 with plates, 0 periodic)
    int periodic_y;
    int frame_t;       // T held at T_w on the frame: outermost columns (and rows if periodic_y)
    int frame_rho;     // the frame is a reservoir at rest with density rho_frame
    int open_x;        // Zou-He pressure inlet at x = 0, outlet at x = Nx-1
    int tile;              // tile shape (kTile...)
    int seg_rows;          // rows of a tile
    int n_strips, n_segs;  // tiles across and up
    int strips_per_xcd;    // > 0: strips of an XCD's chunk (tile_of_block)
    int n_blocks;          // workgroups of a step, a multiple of 8
    unsigned plane;    // rows * pitch
};

// The tile of block `j` of a grid's g.n_blocks on XCD `xcd`.  Blocks are dealt
// round-robin over the eight XCDs, each with its own L2.  A wide grid gives every
// XCD a chunk of neighbouring strips and walks its rows chunk-width tiles at a
// time, so that the tiles in flight on an XCD are a compact patch whose halos
// meet in its L2, and all XCDs are on the same rows (HBM reads per step on
// 8192 x 512: 176 MB against 235 for one row band per XCD, 88.9 us against
// 93.9; fill_grid has the line).  A narrow grid gives every XCD a run of tiles in
// row order, for the same shared halos (against tiles dealt one by one: 100 x 300
// 7.4 us for 8.0, 1111 x 77 mass-exact 9.5 for 10.5, the pool of 20 76.2 for
// 79.5).  down: the rows from the last to the first.  A channel's steps alternate:
// the rows that a step wrote last are then read first, while the memory-side
// cache still has them (84.8 against 88.4 us).
__host__ __device__ inline bool tile_of_block(const Grid& g, int j, int xcd, bool down, int& strip,
                                              int& seg) {
    if (g.strips_per_xcd) {
        const int i = j >> 3;
        seg = i / g.strips_per_xcd;
        strip = xcd * g.strips_per_xcd + (i - seg * g.strips_per_xcd);
    } else {
        const int i = xcd * (g.n_blocks >> 3) + (j >> 3);
        seg = i / g.n_strips;
        strip = i - seg * g.n_strips;
    }
    if (down) seg = g.n_segs - 1 - seg;
    return strip < g.n_strips && seg >= 0 && seg < g.n_segs;
}

// Every buffer a step touches lies in one device allocation; the kernel
// reaches them all through one buffer resource on `base`, by byte offsets.
template <class S>
struct Bufs {
    const char* base;         // the allocation
    unsigned span;            // bytes from base to the end of the last buffer
    unsigned fin, fout;       // population buffers: 9 planes of S
    unsigned lo_in, lo_out;   // mass-exact low parts of the rest population (float)
    unsigned Tin, Tout;       // temperature planes (Tout unused when T is frozen)
    // health counters, added to by every step: [0] owned nodes whose state
    // at the step's time level holds a non-finite rho or T, [1] owned nodes
    // whose Eq. 10 argument was clamped (psi = 0)
    unsigned long long* stat;
};

// One fused time step n -> n+1 (pull-stream + bounce-back, psi, forces, u,
// MRT collision, RK4 temperature) over all units of the grid.
hipError_t launch_step_f32(const Grid& g, const Phys& k, const Bufs<float>& b, bool mass_exact,
                           int64_t n, hipStream_t s);
hipError_t launch_step_f64(const Grid& g, const Phys& k, const Bufs<double>& b, int64_t n,
                           hipStream_t s);

// One channel of a batch (FP32 deviation storage).  The table of slots is
// constant during a chunk of steps; step i of the chunk reads buffer
// (cur + i) & 1 and writes the other, at time level n0 + i, and a slot takes
// part only while i < steps_left.
struct Slot {
    Grid g;
    Phys k;
    const char* mem;          // the slot's allocation
    unsigned span;            // bytes of it the step touches
    unsigned off_f[2];        // byte offsets of the population buffers
    unsigned off_T[2];        // and of the temperature planes
    int64_t n0;
    int cur_f, cur_T;
    int steps_left;
    int block_begin;  // first workgroup of this slot in the batch
    unsigned long long* stat;  // the slot's health counters (see Bufs::stat)
};

// The block of the batch that workgroup `wg` of `n` takes at step `step_i` of a
// chunk: odd steps take the batch from its end, for the same reason as a
// channel's rows (tile_of_block), each slot's tiles from its end with them.  Its
// XCD stays that of the workgroup, so that a tile meets the same L2 on every step.
// (A pool of 20 channels 72.4 us per step and 64 channels 243.4 us; with the rows
// of a slot turned round once more, so that only the slots' order alternated, 72.8
// and 246.5; with neither 84.0 for the 20.)
__host__ __device__ inline int batch_block(int wg, int n, int step_i) {
    return (step_i & 1) ? n - 1 - wg : wg;
}

// Step i of a chunk over every slot of the table (slots sorted by
// block_begin, total_blocks = sum of their workgroups), all with one tile shape.
// ext: some slot uses an optional feature (frames, Carnahan-Starling EOS,
// open ends, plate temperature ramp, phase-dependent properties, Sec. 3.2
// plates), so the batch runs the kernel build that has them
hipError_t launch_step_batched(const Slot* slots, int n_slots, int total_blocks, int tile,
                               int step_i, bool ext, hipStream_t s);

// rho, u (half force) and T at the current time level into arrays of Nx*Ny
// doubles in memory that the device can write (any may be null).
struct Moments {
    double *rho, *ux, *uy, *T;
};
// Pinned host memory that a read-out fills: the channel's kStepWords health
// counters, and for each of its readout_blocks workgroups the number of fluid
// nodes whose rho or T is not finite.
constexpr int kStepWords = 2;
struct Readout {
    unsigned long long* words;
    unsigned* bad;
};
int readout_blocks(int Nx, int Ny);
hipError_t launch_moments_f32(const Grid& g, const Phys& k, const float* f, const float* f0lo,
                              const float* T, const Moments& out, int64_t n,
                              const unsigned long long* stat, const Readout& ro, hipStream_t s);
hipError_t launch_moments_f64(const Grid& g, const Phys& k, const double* f, const double* T,
                              const Moments& out, int64_t n, const unsigned long long* stat,
                              const Readout& ro, hipStream_t s);

// Rest-equilibrium start from a device density field rho0 (Nx*Ny doubles).
hipError_t launch_init_f32(const Grid& g, const Phys& k, const double* rho0, float* f,
                           float* f0lo, float* T, hipStream_t s);
hipError_t launch_init_f64(const Grid& g, const Phys& k, const double* rho0, double* f,
                           double* T, hipStream_t s);

// Deterministic FP64 reduction of the moment arrays: out[5] = {sum rho,
// sum rho ux, sum rho uy, sum rho Cv T, non-finite count}.  partials holds
// kReduceBlocks*5 doubles.
constexpr int kReduceBlocks = 256;
hipError_t launch_reduce(const double* rho, const double* ux, const double* uy,
                         const double* T, int n, double Cv, double* partials, double* out,
                         hipStream_t s);

// The totals of launch_reduce (out_dev[5], device memory) computed in one
// pass from the stored state at time level n_t, with the block partials in
// the library's file-scope scratch array (kStaticReduceBlocks blocks at
// most; no allocation, no clearing): the allocation-free reduction.  Calls
// that overlap on one device share that scratch and race.
constexpr int kStaticReduceBlocks = 1024;
hipError_t launch_reduce_state_f32(const Grid& g, const Phys& k, const float* f,
                                   const float* f0lo, const float* T, double Cv, int64_t n_t,
                                   double* out_dev, hipStream_t s);
hipError_t launch_reduce_state_f64(const Grid& g, const Phys& k, const double* f, const double* T,
                                   double Cv, int64_t n_t, double* out_dev, hipStream_t s);

// Plain device copy of bytes (a multiple of 16) for the bandwidth probe.
hipError_t launch_copy(const void* src, void* dst, size_t bytes, hipStream_t s);

}  // namespace lbmk
