// Host/device view of the fused scan path: bit tables of the clash test and
// the launchers (one set per precision and FFT edge, N <= 128).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "scan_types.hpp"

namespace fftdg {

__host__ __device__ constexpr int ilog2c(int n) { return n <= 1 ? 0 : 1 + ilog2c(n / 2); }

// Longest run piece of the clash test (its two windows lie within one word
// of each other); runs of 2^k <= len < 2^(k+1) points read level k.
constexpr int RUN_MAX = 63;

// OR-dilated receptor occupancy rows of one snapshot, u32 words
// [k][Z][Y][q]: level k (window 2^k, k = 0 .. log2(RUN_MAX + 1) - 1, the
// levels runs of at most RUN_MAX points read); slice Z = z + M and row
// Y = y + M for true coordinates z, y in [-M, N + M) (row (y, z) holds
// receptor row (y mod N, z mod N): the periodic domain of the FFT with M
// rows continued past each end, so a row index z + t_z or y + t_y of a
// ligand point within M of the box needs no reducing); bit x + M of the
// row's RW words is point x mod N, x in [-M, 32 RW - M), so a run starting
// at x >= -M reads its words without wrapping.  A row's words lie together:
// one 12- or 16-byte load brings all that a run needs of it, and 64
// consecutive rows are 1280 contiguous bytes at N = 128 (a layout with the
// rows fastest took one load and three cache lines per word).  The whole
// table is 2.5 MB at N = 128, inside one XCD's 4 MB L2.  PADW words follow
// it: a run's load may pass the end of the last row (bits that belong to no
// box-valid translation).
template <int N>
struct Dil {
    static constexpr int NW = N / 32;
    static constexpr int M = 8;
    static constexpr int E = N + 2 * M;
    static constexpr int RW = (E + 31) / 32;
    static constexpr int K = ilog2c(RUN_MAX + 1);
    static constexpr int PADW = 8;
    static_assert((1 << (K - 1)) <= N, "a level's window must fit in a row");
    __host__ __device__ static constexpr int64_t words() { return (int64_t)K * E * E * RW + PADW; }
    __host__ __device__ static constexpr int64_t index(int k, int Z, int q, int Y) {
        return (((int64_t)k * E + Z) * E + Y) * RW + q;
    }
};

// LDS budget of the per-block factor table of the fused z kernel.
constexpr size_t FUSED_TABLE_BYTES = 16384;

// Strides between the snapshots of one launch (blockIdx.y) of the clash
// test and the direct energies.
struct SnapStride {
    int64_t dil;    // words of a receptor bit table
    int64_t fb;     // words of free bits
    int64_t live;   // bytes of live flags
    int64_t surv;   // slots of the undecided-segment lists
    int64_t counts; // ints of the counts (scnt, fcnt, out)
    int64_t zlist;  // ints of the list of configurations that take the transforms
    int64_t grid;   // elements of the receptor grids
    int64_t pp;     // plane partials
};

struct FusedSet {
    int n_fft;
    int64_t dil_words;  // words of one snapshot's dilation table
    int margin;         // Dil<N>::M: occupancy may reach this many points past the box
    // occ [n_rec^3] bytes -> dil (Dil<N> layout)
    hipError_t (*rec_dilate)(hipStream_t, const uint8_t *occ, int n_rec, uint32_t *dil);
    // ligand occupancy runs of the scanned configurations zcfg[0..nz) of a
    // chunk: two words per run from runs[2 run_off], run_count[local index]
    hipError_t (*lig_runs)(hipStream_t, const CfgDev *cfgs, const int32_t *zcfg, int nz, const int32_t *ulat,
                           const double *thr, uint32_t *runs, int32_t *run_count);
    // clears n ints
    hipError_t (*zero)(hipStream_t, int32_t *p, int64_t n);
    // free bits and live flags: item_off[0..n_cfg] running counts of the
    // phase-1 items (tz, 64-row group), item2_off those of the phase-2
    // blocks (each takes every n-th 64 of a configuration's undecided segments); surv holds the
    // lists (at surv_off), scnt their lengths, fcnt the free translations per
    // configuration (n_cfg ints each, zero on entry); ns snapshots a launch
    hipError_t (*clash)(hipStream_t, int ns, const SnapStride &st, const int32_t *item_off, const int32_t *item2_off,
                        int n_cfg, int n_items, int n_items2, const CfgDev *cfgs, const uint32_t *runs,
                        const int32_t *run_count, const uint32_t *dil, uint32_t *fb, uint8_t *live, uint32_t *surv,
                        int32_t *scnt, int32_t *fcnt);
    // direct energies (direct and what belongs to it are nullptr where every
    // configuration takes the transforms, see offers_direct): per scanned configuration its atoms' corner offsets
    // and weights (nz x max_atoms records of corner_bytes); which
    // configurations go through the transforms (zlist, need, out[2] as
    // k_modes writes them; done: one int per configuration, zero at the
    // chunk's start); Eq. 2 plane partials of the others from the receptor
    // grids (grid_points).  ns snapshots a launch; need and out[1] are for all
    // of them together
    size_t corner_bytes;
    hipError_t (*corner_atoms)(hipStream_t, const CfgDev *cfgs, const int32_t *zcfg, int nz, int max_atoms,
                               const int32_t *ulat, const void *gam, int n_rec, void *atoms);
    hipError_t (*modes)(hipStream_t, int ns, const SnapStride &st, const CfgDev *cfgs, const int32_t *zcfg, int nz,
                        const int32_t *fcnt, int32_t *done, int32_t *zlist, uint8_t *need, int32_t *out);
    hipError_t (*direct)(hipStream_t, int ns, const SnapStride &st, const int32_t *inv_off, int n_cfg, int n_items,
                         const CfgDev *cfgs, const void *atoms, int max_atoms, const void *grids, int n_rec,
                         double beta, const uint32_t *fb, const uint8_t *live, const int32_t *fcnt, void *pp);
    // a snapshot's receptor grids [3][n_rec^3] in the layout direct reads, [n_rec^3][3]
    hipError_t (*grid_points)(hipStream_t, const void *grids, int n_rec, void *out);
    // per scanned configuration of a chunk: its atoms sorted by plane with
    // their x/y placement and channel weights, and the plane starts
    // (zat: nz x max_atoms records, zbt: nz x (N + 2) ints)
    hipError_t (*zprep)(hipStream_t, const CfgDev *cfgs, const int32_t *zcfg, int nz, int max_atoms,
                        const int32_t *ulat, const void *gam, void *zat, int32_t *zbt);
    size_t zat_bytes;  // bytes of one atom record
    // z pass of one snapshot (spectra rspec, 3 energy channels); with clash,
    // only the z-translations whose live flag is set, and with a zlist only
    // the configurations zlist[0 .. nfft[0]) (indices into zcfg)
    hipError_t (*zpass)(hipStream_t, bool zhalf, bool clash, const CfgDev *cfgs, const int32_t *zcfg, int nz,
                        int max_atoms, const void *zat, const int32_t *zbt, const void *rspec, const void *tw,
                        void *wsi, const uint8_t *live, const int32_t *zlist, const int32_t *nfft);
    // z pass of one snapshot from energy planes in ws (direct forward pass)
    hipError_t (*zplanes)(hipStream_t, bool zhalf, bool clash, const CfgDev *cfgs, const int32_t *zcfg, int nz,
                          const void *ws, const void *rspec, const void *tw, void *wsi, const uint8_t *live,
                          const int32_t *zlist, const int32_t *nfft);
    // inverse xy + Eq. 2 plane partials; e_count (nullable) counts planes read;
    // fcnt (nullable): only the configurations that go through the transforms
    hipError_t (*inv)(hipStream_t, bool clash, const int32_t *inv_off, int n_cfg, int n_items, const CfgDev *cfgs,
                      const void *wsi, double beta, const void *tw, const uint32_t *fb, const uint8_t *live,
                      void *pp, void *psi_out, uint8_t *clash_out, unsigned int *e_count, const int32_t *fcnt,
                      const int32_t *nfft);
    // dynamic LDS bytes of the z kernel for ligands of up to max_atoms atoms
    size_t (*z_lds)(int max_atoms);
};

// nullptr where the fused path is not built (N = 256)
const FusedSet *fused_set(int precision, int n_fft);

}  // namespace fftdg
