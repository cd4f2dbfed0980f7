// Host helpers shared by the single-channel runtime and the slot pool.
// Internal; not part of the C-ABI.
#pragma once

#include <cstddef>

#include "lbm.h"
#include "lbm_internal.h"

namespace lbmhost {

constexpr int kAlign = 256;
inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// Elements added to the population plane stride beyond pitch x rows (a
// multiple of 64, so rows keep their 256-byte alignment).  When pitch x rows
// is a multiple of a large power of two (8192 x 510 FP32 values are
// 255 x 64 KiB) the nine planes of one row start at addresses that agree in
// all their low bits and their loads and stores pile onto the same HBM
// channels; skewing each plane by 3.25 KiB (FP32) spreads them.
constexpr size_t kPlaneSkew = 832;

// Device memory layout of one channel: two population buffers
// [9][rows][pitch] with a plane stride of pitch x rows + kPlaneSkew,
// optional mass-exact low planes, two temperature planes, then the moment
// arrays and reduction scratch.
struct Layout {
    int pitch, rows;
    size_t plane, esz;
    size_t off_f[2], off_lo[2], off_T[2], off_mom, off_part, off_out, off_stat, total;
};

// Health counters of a channel (unsigned 64-bit, device memory) that the step
// kernels add to: non-finite readings, psi clamps.
enum { kStatNonfinite = 0, kStatClamps = 1, kStatWords = lbmk::kStepWords };

// Pinned host memory for a read-out of Nx x Ny nodes (grown, never shrunk;
// null members while none is held).
struct ReadoutMem {
    lbmk::Readout ro = {nullptr, nullptr};
    int cap = 0;  // workgroups it holds
    // blocks it has grown out of, together no larger than the present one
    // (each is at least twice the last, so 31 at most)
    void* outgrown[31];
    int n_outgrown = 0;
};
hipError_t reserve_readout(ReadoutMem& m, int Nx, int Ny);
void free_readout(ReadoutMem& m);
// Fluid nodes found not finite by the last read-out of Nx x Ny nodes.
unsigned long long readout_bad(const ReadoutMem& m, int Nx, int Ny);

// Where a read-out writes its fields: an array of the caller's that lies in
// pinned host memory as a whole is written by the kernel itself if the arrays
// named are no larger than `direct` bytes together; any other is copied from
// the device array that stands for it.  The kernel's stores to the host hold up
// whatever else the GPU runs until the link has taken them (a smaller grid of
// workgroups does not help), a copy does not.  Alone the kernel is the faster of
// the two up to some 16 MiB (us, kernel / one copy of four adjoining arrays / four
// copies: 128 x 32 23 / 33 / 57, 200 x 200 45 / 55 / 79, 1024 x 128 96 / 110 / 135,
// 2048 x 256 331 / 337 / 363, 4096 x 512 1282 / 1247 / 1273, 8192 x 512 2545 / 2455 /
// 2485); beside steps on another stream a read-out costs them 20 us for 2 (200 x
// 200), 73 for 4 (1024 x 128: 4 MiB), 308 for 16 (2048 x 256) and 1294 for 40 (4096 x
// 512).  A channel does not know what else the GPU runs: its line is 4 MiB, up to
// where the caller gains what others lose against two passes and five copies (96
// and 73 us for 160 and 7).  A pool knows its own batch: 16 MiB while no chunk is
// left running beside the slot's own, else nothing.
constexpr size_t kDirectChannel = (size_t)4 << 20, kDirectPool = (size_t)16 << 20;
struct ReadoutPlan {
    lbmk::Moments direct;  // what the kernel writes
    double* copy_to[4];    // host arrays to copy to afterwards (null: none)
    double* copy_from[4];
};
ReadoutPlan plan_readout(double* const host[4], double* const dev[4], size_t cells, size_t direct);
hipError_t enqueue_copies(const ReadoutPlan& r, size_t cells, hipStream_t s);

lbm_status fail(lbm_status st, const char* fmt, ...);
bool make_layout(const lbm_params& p, Layout* L);
lbm_status validate(const lbm_params& p);
// Initial density field (host, Nx*Ny, NULL: uniform rho_v) against the EOS:
// every fluid node needs 0 < b rho below the packing limit and a positive
// Eq. 10 argument 2 (P_EOS - rho/3) / G at its initial temperature.
lbm_status check_initial(const lbm_params& p, const double* rho0);
// Tall tiles from which on they are the default (default_tile).
constexpr long long kTallTiles = 2048;
// The tile shape of a channel stepped alone by default, and the smallest one
// that holds seg_rows rows (the tallest if none does).
int default_tile(const lbm_params& p, int rows);
// Rows of a segment of a channel stepped alone by default, in that tile.
int default_rows(const lbm_params& p, int rows, int tile);
int tile_for(const lbm_params& p, int seg_rows);
// Grid of a launch with segments of seg_rows rows in tiles of shape `tile`:
// segments taller than a tile are split evenly.
void fill_grid(const lbm_params& p, const Layout& L, int seg_rows, int tile, lbmk::Grid& g,
               bool in_batch = false);
// Segments of about `target` rows, balanced over the channel's rows.
int balanced_rows(int rows, int target);
void fill_phys(const lbm_params& p, lbmk::Phys& k);

}  // namespace lbmhost
