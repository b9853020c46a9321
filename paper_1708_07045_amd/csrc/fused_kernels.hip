// Fused scan path for gfx950 (wave64): clashes by an exact bitwise test, then
// energies summed at the clash-free translations where these are few (k_direct),
// else the energy channels alone through the FFT.
//
// Clash test (occupancy mode, Eq. 10).  The overlap count of Eq. 10 is
// positive exactly when some occupied ligand grid point n lands on an
// occupied receptor point n + t (indices mod n_fft over the zero-padded
// receptor grid, the convention the FFT correlation has).  Instead of a
// fourth FFT channel thresholded at 1/2, the test is made on bits:
//   - the ligand's occupied points (union of its atoms' balls, the integer
//     membership test of the occupancy grid) are written as runs along x,
//     one per maximal segment of a (y, z) row (k_lig_runs);
//   - each receptor occupancy row is kept OR-dilated over windows of 2^k
//     points, D_k(x) = OR_{0 <= j < 2^k} O_R(x + j) (k_rec_dilate);
//   - a run of length L starting at x = a meets receptor occupancy at
//     translation t iff D_k(a + t_x) | D_k(a + L - 2^k + t_x) on row
//     (y + t_y, z + t_z), 2^k <= L < 2^(k+1); one 32-bit word answers 32
//     x-translations at once (k_clash1, k_clash2).
// The result is the clash mask the FFT threshold reproduces, without its
// rounding: every decision is an integer one.  (Known defect: configurations of
// 33 to 96 runs can keep clashing translations, see k_clash1's stride.)
//
// Energy channels (Eqs. 4-9).  The x/y DFT of a trilinearly spread atom
// factorises,
//   sum_{dx,dy} w_dx w_dy w^(kx (ax+dx) + ky (ay+dy))
//     = w^(kx ax) ((1-fx) + fx w^kx) * w^(ky ay) ((1-fy) + fy w^ky),
// (w = exp(-2 pi i / N)) and the atom reaches only the planes floor(uz)
// (weight 1-fz) and floor(uz)+1 (weight fz).  The z kernel (k_zfused) forms
// each z-pencil's input from these factors (a table per block over its
// pencils and the configuration's atoms, atoms sorted by plane), runs the
// forward z FFT, the product with the receptor spectra summed over the three
// channels (Eq. 9) and the inverse z FFT, and stores only the z-translations
// that have a clash-free translation (all box-valid ones in cap mode or when
// energies are exported).  k_inv_fused finishes the inverse along y and x on
// those planes, skips row pairs without a clash-free translation, and folds
// the clash-free energies into the Eq. 2 partials.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "../../include/fftdg.h"
#include "fft_device.hpp"
#include "fused.hpp"
#include "scan_common.hpp"
#include "scan_types.hpp"

namespace fftdg {

// ------------------------------------------------------------ receptor rows
// One thread per stored row (Z, Y) of the table.  Level 0 holds the
// occupancy bits of receptor row ((Y - M) mod N, (Z - M) mod N) (zero
// outside the n_rec^3 receptor grid); level k ORs level k-1 with itself
// advanced by 2^(k-1) points (mod N).
template <int N>
__global__ __launch_bounds__(NT) void k_rec_dilate(const uint8_t *__restrict__ occ, int n_rec,
                                                    uint32_t *__restrict__ dil) {
    using D = Dil<N>;
    constexpr int NW = D::NW;
    const int r = (int)blockIdx.x * NT + (int)threadIdx.x;
    if (r >= D::E * D::E) return;
    const int Z = r / D::E, Y = r - (r / D::E) * D::E;
    const int z = (Z - D::M + N) & (N - 1), y = (Y - D::M + N) & (N - 1);
    uint32_t v[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) v[w] = 0u;
    if (z < n_rec && y < n_rec) {
        const uint8_t *row = occ + ((int64_t)z * n_rec + y) * n_rec;
        for (int x = 0; x < n_rec; ++x)
            if (row[x]) v[x >> 5] |= 1u << (x & 31);
    }
#pragma unroll
    for (int k = 0; k < D::K; ++k) {
        if (k > 0) {
            const int s = 1 << (k - 1);  // bit x of the advanced row is bit (x + s) mod N
            uint32_t t[NW];
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const int p = (32 * w + s) & (N - 1);
                const int q = p >> 5, sh = p & 31;
                const uint32_t lo = v[q], hi = v[(q + 1) % NW];
                t[w] = sh ? ((lo >> sh) | (hi << (32 - sh))) : lo;
            }
#pragma unroll
            for (int w = 0; w < NW; ++w) v[w] |= t[w];
        }
        // word q holds points 32 q - M + j, j = 0 .. 31, mod N
#pragma unroll
        for (int q = 0; q < D::RW; ++q) {
            const uint32_t lo = v[(q + NW - 1) % NW], hi = v[q % NW];
            dil[D::index(k, Z, q, Y)] = (lo >> (32 - D::M)) | (hi << D::M);
        }
    }
    if (r == 0)
        for (int i = 0; i < D::PADW; ++i) dil[D::words() - D::PADW + i] = 0u;
}

// ------------------------------------------------------------ ligand runs
// Exclusive prefix sum over a block of NTH threads (fixed order), `total` =
// block sum; sh holds one int per wavefront.
template <int NTH = NT>
__device__ __forceinline__ int block_excl_scan(int v, int &total, int *sh) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    if (lane == 63) sh[w] = x;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NTH / 64; ++i) {
        base += i < w ? sh[i] : 0;
        tot += sh[i];
    }
    __syncthreads();
    total = tot;
    return base + x - v;
}

// The ball of atom `a` on row (y, z): [xlo, xhi] in true grid x, or false.
// Point x belongs to it iff (2^16 x - Ux)^2 < rem, with rem what the row
// leaves of the squared radius: an estimate of the ends from a FP32 root
// (good to a fraction of a lattice step of 2^-16), moved by that integer test.
struct RunAtom {
    int Ux, Uy, Uz;
    long long T;
};
__device__ __forceinline__ bool ball_row(const RunAtom &A, int y, int z, int &xlo, int &xhi) {
    const int dz = z * 65536 - A.Uz;
    const long long rz = A.T - (long long)dz * dz;
    if (rz <= 0) return false;
    const int dy = y * 65536 - A.Uy;
    const long long rem = rz - (long long)dy * dy;
    if (rem <= 0) return false;
    auto in = [&](int x) {
        const int d = x * 65536 - A.Ux;
        return (long long)d * d < rem;
    };
    const int s = (int)__builtin_sqrtf((float)rem);
    xlo = (A.Ux - s + 65535) >> 16;
    xhi = (A.Ux + s) >> 16;
    if (in(xlo - 1)) --xlo;
    else if (!in(xlo)) ++xlo;
    if (in(xhi + 1)) ++xhi;
    else if (!in(xhi)) --xhi;
    return xlo <= xhi;
}

// A run of the clash test as two words: the byte offset of its first table
// word for a translation of zero, o = 4 Dil<N>::index(k, z + M, b / 32,
// y + M) with b = a + M (the lane adds 4 RW (t_z E + t_y)), and the two
// window shifts, b mod 32 | ((b + len - 2^k) mod 32) << 8 | (second window
// one word on) << 16 | (len - 2^k) << 24, with 2^k <= len < 2^(k+1).  The planner keeps z, y,
// a >= -M and the rows and words a translated run reads inside the table.
template <int N>
__device__ __forceinline__ uint2 pack_run(int z, int y, int a, int len) {
    using D = Dil<N>;
    const int ax = a + D::M;
    const int k = 31 - __builtin_clz((unsigned)len);
    const int p2 = ax + len - (1 << k);
    const uint32_t off = (uint32_t)(4 * D::index(k, z + D::M, ax >> 5, y + D::M));
    const uint32_t meta = (uint32_t)(ax & 31) | ((uint32_t)(p2 & 31) << 8) | ((uint32_t)((p2 >> 5) > (ax >> 5)) << 16) |
                          (uint32_t)(len - (1 << k)) << 24;
    return make_uint2(off, meta);
}
__device__ __forceinline__ int run_pieces(int len) { return (len + RUN_MAX - 1) / RUN_MAX; }
// Write a run as pieces of at most RUN_MAX points from slot pos (slots at
// or past cap are not written); returns the number of pieces.
template <int N>
__device__ __forceinline__ int emit_run(uint2 *out, int pos, int cap, int z, int y, int a, int len) {
    int k = 0;
    for (int o = 0; o < len; o += RUN_MAX, ++k) {
        const int l = len - o < RUN_MAX ? len - o : RUN_MAX;
        if (pos + k < cap) out[pos + k] = pack_run<N>(z, y, a + o, l);
    }
    return k;
}

// The set bits of a row, N <= 128 of them in 64-bit words.
template <int N>
struct RowBits {
    static constexpr int NQ = N > 64 ? 2 : 1;
    unsigned long long q[NQ];
    __device__ void clear() {
#pragma unroll
        for (int i = 0; i < NQ; ++i) q[i] = 0ull;
    }
    __device__ bool any() const { return NQ == 2 ? (q[0] | q[1]) != 0ull : q[0] != 0ull; }
    // points l .. h (0 <= l <= h < N)
    __device__ void set(int l, int h) {
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int lo = max(l - 64 * i, 0), n = min(h - 64 * i, 63) - lo + 1;
            if (n > 0) q[i] |= (~0ull >> (64 - n)) << lo;
        }
    }
    // lowest maximal segment [s, e), removed
    __device__ void take(int &s, int &e) {
        if (NQ == 1 || q[0]) {
            s = __builtin_ctzll(q[0]);
            const unsigned long long r = ~(q[0] >> s);
            const int len = r ? __builtin_ctzll(r) : 64;
            e = min(s + len, 64);
            q[0] &= s + len >= 64 ? 0ull : ~0ull << e;
            if (NQ == 2 && e == 64) {
                const unsigned long long u = ~q[NQ - 1];
                const int more = u ? __builtin_ctzll(u) : 64;
                e += more;
                q[NQ - 1] &= more >= 64 ? 0ull : ~0ull << more;
            }
        } else {
            s = 64 + __builtin_ctzll(q[NQ - 1]);
            const unsigned long long r = ~(q[NQ - 1] >> (s - 64));
            const int len = r ? __builtin_ctzll(r) : 64;
            e = min(s + len, 128);
            q[NQ - 1] &= e >= 128 ? 0ull : ~0ull << (e - 64);
        }
    }
};

// One block per scanned configuration.  Runs are written in a fixed order:
// first each atom's chord through the row nearest its centre (its widest
// segment; a subset of the union, so harmless to the OR, and the most likely
// to meet receptor occupancy, which lets the clash test stop early), then
// the maximal segments of the union of the balls on every row of the
// occupancy window, z-major.  Bound: latency, a chunk of 256 configurations
// being one block a compute unit; 16 wavefronts take a site ligand's 2000
// rows in two rounds (4 took eight), and a ball's row costs a FP32 root and
// four integer tests (it was an FP64 root moved by 64-bit squares and four
// 64-bit divisions).  256 site configurations: 118 -> 31 us.
constexpr int RUN_NT = 1024;
template <int N>
__global__ __launch_bounds__(RUN_NT) void k_lig_runs(const CfgDev *__restrict__ cfgs, const int32_t *__restrict__ zcfg,
                                                  const int32_t *__restrict__ ulat, const double *__restrict__ thr,
                                                  uint32_t *__restrict__ runs, int32_t *__restrict__ run_count) {
    __shared__ RunAtom at[MAXA];
    __shared__ int sh[RUN_NT / 64];
    const int lc = zcfg[blockIdx.x];
    const CfgDev &c = cfgs[lc];
    const int n = c.n_atoms;
    static_assert(RUN_NT >= MAXA, "a thread per atom");
    if ((int)threadIdx.x < n) {
        const int a = threadIdx.x;
        const int32_t *U = ulat + 3 * (c.u_base + a);
        at[a] = RunAtom{U[0], U[1], U[2], (long long)thr[c.atom_base + a]};
    }
    __syncthreads();
    uint2 *out = reinterpret_cast<uint2 *>(runs) + c.run_off;
    const int cap = c.run_cap;
    int base = 0, total;
    {  // chords through the centre rows
        const int a = threadIdx.x;
        int xlo = 0, xhi = -1, yc = 0, zc = 0;
        bool has = false;
        if (a < n) {
            yc = (at[a].Uy + 32768) >> 16;
            zc = (at[a].Uz + 32768) >> 16;
            has = ball_row(at[a], yc, zc, xlo, xhi);
        }
        const int len = has ? xhi - xlo + 1 : 0;
        const int pos = base + block_excl_scan<RUN_NT>(has ? run_pieces(len) : 0, total, sh);
        if (has) emit_run<N>(out, pos, cap, zc, yc, xlo, len);
        base += total;
    }
    // every row of the occupancy window: union of the balls as a bit row
    // relative to xo0 (the window's x extent is at most N), then its runs
    const int Lyo = c.Lyo, nrows = c.Lo * Lyo, zo0 = c.zo0, yo0 = c.yo0, xo0 = c.xo0;
    for (int r0 = 0; r0 < nrows; r0 += RUN_NT) {
        const int r = r0 + (int)threadIdx.x;
        RowBits<N> m;
        m.clear();
        int z = 0, y = 0;
        if (r < nrows) {
            z = zo0 + r / Lyo;
            y = yo0 + r - (r / Lyo) * Lyo;
            for (int a = 0; a < n; ++a) {
                int xlo, xhi;
                if (ball_row(at[a], y, z, xlo, xhi)) m.set(xlo - xo0, xhi - xo0);
            }
        }
        // maximal segments of the row, in pieces of at most RUN_MAX points:
        // counted, then written
        int cnt = 0, s, e;
        for (RowBits<N> t = m; t.any();) {
            t.take(s, e);
            cnt += run_pieces(e - s);
        }
        int pos = base + block_excl_scan<RUN_NT>(cnt, total, sh);
        while (m.any()) {
            m.take(s, e);
            pos += emit_run<N>(out, pos, cap, z, y, xo0 + s, e - s);
        }
        base += total;
    }
    if (threadIdx.x == 0) run_count[lc] = base < cap ? base : cap;
}

// ------------------------------------------------------------ clash test
// The test runs in two phases.  Phase 1: one wavefront per (configuration,
// z-translation tz, group of 64 y-translations), lane = ty, tests the atom
// chords and an evenly spread sample of the runs.  Rows whose
// translations all clash are done (no free bit); the bits left of the others
// are appended to the configuration's list of undecided segments, 32
// translations of one row each.  Phase 2: blocks over each configuration's
// list, lane = one segment, test every run.  Only the configurations that
// still have undecided rows (those near clash-free translations) pay for the
// full run list, and of a row only the words that its undecided bits need.
constexpr int CLASH_R1 = 96;      // most runs of phase 1
constexpr int CLASH_CHORDS = 32;  // of these the first so many in order, the others spread

// K consecutive words of a table row, one or two loads
template <int K>
__device__ __forceinline__ void load_words(__amdgpu_buffer_rsrc_t rsrc, int vo, int so, uint32_t *v) {
    static_assert(K >= 3 && K <= 6, "words of a run");
    if constexpr (K == 3) {
        const u32x3 t = __builtin_amdgcn_raw_buffer_load_b96(rsrc, vo, so, 0);
        v[0] = t.x, v[1] = t.y, v[2] = t.z;
    } else {
        const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(rsrc, vo, so, 0);
        v[0] = t.x, v[1] = t.y, v[2] = t.z, v[3] = t.w;
        if constexpr (K == 5) v[4] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, vo + 16, so, 0);
        if constexpr (K == 6) {
            const u32x2 u = __builtin_amdgcn_raw_buffer_load_b64(rsrc, vo + 16, so, 0);
            v[4] = u.x, v[5] = u.y;
        }
    }
}

// The first k1 runs of the phase-1 sample of one wavefront: the first NCH
// runs, the atom chords, then stride S over the rest.  Lane row (tzl, ty);
// W output words per lane; UR runs in flight (their table words
// all requested before use).  Runs are at most 63 points long, so a run's
// second window starts at most one word after its first: the words q1 ..
// q1 + W + 1 of its row serve both.  rl, k and the run entries are
// wave-uniform and must be so for the compiler (derived from blockIdx or
// readfirstlane): the entries then come by scalar loads and their offset
// travels in an SGPR.  With an offset the compiler takes for a lane value
// every table load became a loop over the distinct offsets, 2700 cycles per
// four runs.  Bound: the loads' way through L1 (20 bytes a lane and run at
// 70 translations a row).  8000 site configurations (25 atoms, 96^3 in
// 128^3): 4.1 -> 2.0 ms.
template <int N, int W>
__device__ __forceinline__ void clash_runs(const uint2 *__restrict__ rl, int nr, int k1, int NCH, int S, int tzl,
                                           int ty, bool act, uint32_t lm, __amdgpu_buffer_rsrc_t rsrc,
                                           uint32_t *acc) {
    using D = Dil<N>;
    constexpr int UR = W <= 2 ? 8 : 4;
    int m = 0;  // position of the strided walk over the runs after the chords
    const int R = nr - NCH;
    auto run_index = [&](int k) {
        if (k < NCH) return k;
        const int i = NCH + m;
        m += S;
        if (m >= R) m -= R;
        return i;
    };
    const int vo = (tzl * D::E + ty) * (D::RW * 4);  // the lane's part of every table offset
    auto test = [&](auto urc, int k) {
        constexpr int U = decltype(urc)::value;
        uint32_t v[U][W + 2];
        uint32_t meta[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint2 e = rl[run_index(k + u)];
            meta[u] = e.y;
            load_words<W + 2>(rsrc, vo, (int)e.x, v[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned sh1 = meta[u] & 31u, sh2 = (meta[u] >> 8) & 31u;
            const bool hi2 = (meta[u] & 0x10000u) != 0u;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const uint32_t o1 = __builtin_amdgcn_alignbit(v[u][w + 1], v[u][w], sh1);
                const uint32_t lo = hi2 ? v[u][w + 1] : v[u][w], hi = hi2 ? v[u][w + 2] : v[u][w + 1];
                acc[w] |= o1 | __builtin_amdgcn_alignbit(hi, lo, sh2);
            }
        }
    };
    auto all_full = [&]() {
        bool full = true;
#pragma unroll
        for (int w = 0; w < W; ++w) full = full && ((w == W - 1) ? ((acc[w] & lm) == lm) : (acc[w] == ~0u));
        return __all(!act || full) != 0;
    };
    int k = 0;
    for (; k + UR <= k1; k += UR) {
        test(std::integral_constant<int, UR>{}, k);
        if (all_full()) return;
    }
    for (; k < k1; ++k) test(std::integral_constant<int, 1>{}, k);
}

template <int N>
__device__ __forceinline__ void clash_dispatch(int W, const uint2 *rl, int nr, int k1, int NCH, int S, int tzl, int ty,
                                               bool act, uint32_t lm, __amdgpu_buffer_rsrc_t rsrc, uint32_t *acc) {
    constexpr int NW = N / 32;
#define FFTDG_RUNS(WW) clash_runs<N, WW>(rl, nr, k1, NCH, S, tzl, ty, act, lm, rsrc, acc)
    switch (W) {  // wave-uniform
    case 1: FFTDG_RUNS(1); break;
    case 2: if constexpr (NW >= 2) FFTDG_RUNS(2); break;
    case 3: if constexpr (NW >= 3) FFTDG_RUNS(3); break;
    case 4: if constexpr (NW >= 4) FFTDG_RUNS(4); break;
    default: break;
    }
#undef FFTDG_RUNS
}

// Adds the lanes' counts to *total.
__device__ __forceinline__ void wave_count(int n, int lane, int32_t *total) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) n += __shfl_xor(n, off);
    if (lane == 0 && n) atomicAdd(total, n);
}

// Phase 1.  Bits (box-valid and not found to clash) of row (tz, ty) go to
// fb[free_off + (tz Vy + ty) W + w], W = ceil(Vx / 32), bit tx & 31 of word
// tx >> 5: final where every run was tested.  Otherwise the row's bits are
// cut, from the lowest on, into segments of 32 translations, and each is
// appended to the list at surv_off as (tz << 16 | ty << 8 | first tx),
// scnt[local config] counting.  live[item_base + tz ny + g] = 1 iff the group
// has a free bit once decided (0 until phase 2 decides its segments).
// fcnt[local config] counts the free translations of both phases (scnt and
// fcnt start at zero).
template <int N>
__global__ __launch_bounds__(NT) void k_clash1(const int32_t *__restrict__ item_off, int n_cfg, int n_items,
                                                const CfgDev *__restrict__ cfgs, const uint32_t *__restrict__ runs,
                                                const int32_t *__restrict__ run_count,
                                                const uint32_t *__restrict__ dil, uint32_t *__restrict__ fb,
                                                uint8_t *__restrict__ live, uint32_t *__restrict__ surv,
                                                int32_t *__restrict__ scnt, int32_t *__restrict__ fcnt, SnapStride st) {
    using D = Dil<N>;
    constexpr int NW = D::NW;
    dil += blockIdx.y * st.dil, fb += blockIdx.y * st.fb, live += blockIdx.y * st.live;
    surv += blockIdx.y * st.surv, scnt += blockIdx.y * st.counts, fcnt += blockIdx.y * st.counts;
    const int item = (int)blockIdx.x * (NT / 64) + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (item >= n_items) return;
    const int lane = threadIdx.x & 63;
    const int ic = find_cfg(item_off, n_cfg, item);
    const CfgDev c = cfgs[ic];
    const int Vx = c.V[0], Vy = c.V[1];
    const int ny = (Vy + 63) >> 6;
    const int loc = item - item_off[ic];
    const int tz = loc / ny, g = loc - (loc / ny) * ny;
    const int ty = 64 * g + lane;
    const bool act = ty < Vy;
    const int W = (Vx + 31) >> 5;
    const uint32_t lm = (Vx & 31) ? ((1u << (Vx & 31)) - 1u) : ~0u;
    uint32_t acc[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) acc[w] = 0u;
    const int nr = run_count[ic];
    // a twelfth of the runs, the chords at least: a longer sample costs every
    // row, a shorter one leaves phase 2 more segments.  Phase 1 and 2 of 8000
    // site configurations (1550 runs) 6.40 ms with 96, 6.43 with 64; of a
    // coarse batch at 64^3 (some 350 runs) 3.26 ms with 96, 2.88 with 64,
    // 2.62 by this rule; up to 96 runs all are tested here
    const int k1 = nr <= CLASH_R1 ? nr : min(CLASH_R1, max(CLASH_CHORDS, nr / 12));
    const int NCH = min(nr, CLASH_CHORDS);
    // stride of the spread sample: near 0.618 of the runs after the chords.
    // Known defect: where it shares a factor with their number R the walk visits
    // R / gcd of them, and with nr <= CLASH_R1 the row counts as decided all the
    // same: 24 of the 64 counts nr = 33 .. 96 (ligands of a few atoms on a coarse
    // grid) keep clashing translations.  A stride of 1 where nr <= CLASH_R1 mends
    // it and changes those ligands' results
    const int S = max(1, (nr - NCH) * 618 / 1000) % max(1, nr - NCH);
    const auto rsrc = make_rsrc(dil, (int)(D::words() * 4));
    clash_dispatch<N>(W, reinterpret_cast<const uint2 *>(runs) + c.run_off, nr, k1, NCH, S, tz, ty, act, lm, rsrc, acc);
    const bool final = k1 == nr;  // every run tested: the row is decided either way
    uint32_t f[NW];
    bool any = false;
    int nfree = 0;
    uint32_t *o = fb + c.free_off + ((int64_t)tz * Vy + ty) * W;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        f[w] = act && w < W ? ~acc[w] & (w == W - 1 ? lm : ~0u) : 0u;
        if (act && w < W) o[w] = f[w];
        any = any || f[w] != 0u;
        nfree += __popc(f[w]);
    }
    if (!final && __any(any))
        for (int r = 0; r < NW; ++r) {  // segment r of every row that has one
            int p = -1;
#pragma unroll
            for (int w = NW - 1; w >= 0; --w)
                if (f[w]) p = 32 * w + __builtin_ctz(f[w]);
            const unsigned long long um = __ballot(p >= 0);
            if (!um) break;
            int base = 0;
            if (lane == 0) base = atomicAdd(&scnt[ic], __popcll(um));
            base = __shfl(base, 0);
            if (p < 0) continue;
            surv[c.surv_off + base + __popcll(um & ((1ull << lane) - 1ull))] =
                ((uint32_t)tz << 16) | ((uint32_t)ty << 8) | (uint32_t)p;
#pragma unroll
            for (int w = 0; w < NW; ++w) {  // bits below p + 32 are done
                const int d = p + 32 - 32 * w;
                f[w] = d >= 32 ? 0u : (d > 0 ? f[w] & (~0u << d) : f[w]);
            }
        }
    const unsigned long long bal = __ballot(final && any);
    if (lane == 0) live[c.item_base + loc] = bal != 0ull ? 1 : 0;
    if (bal) wave_count(nfree, lane, fcnt + ic);
}

// Phase 2: a configuration's blocks go over its list of undecided segments,
// 64 at a time, one per lane; a block's wavefronts test a quarter of the runs
// each and exchange what they found through LDS.  A segment with a free
// translation has to meet every run (about 1550 at the site), and one
// wavefront walking them alone was a chain of some 350 us even on an idle
// chip; a chunk of 256 configurations has about 3000 such wavefronts for the
// 8192 places the chip has, so the quarters also fill it.  A lane reads
// three words per run, at the word of its own first translation, and takes
// both windows from them.  Bound: the loads' way through L1 (12 bytes a lane
// and run).  8000 site configurations (25 atoms, 96^3 in 128^3): 32.0 ->
// 4.5 ms (5.95 with a lane to a whole row and its five words).
template <int N>
__global__ __launch_bounds__(NT) void k_clash2(const int32_t *__restrict__ item2_off, int n_cfg, int n_items,
                                                const CfgDev *__restrict__ cfgs, const uint32_t *__restrict__ runs,
                                                const int32_t *__restrict__ run_count,
                                                const uint32_t *__restrict__ dil, uint32_t *__restrict__ fb,
                                                uint8_t *__restrict__ live, const uint32_t *__restrict__ surv,
                                                const int32_t *__restrict__ scnt, int32_t *__restrict__ fcnt,
                                                SnapStride st) {
    using D = Dil<N>;
    dil += blockIdx.y * st.dil, fb += blockIdx.y * st.fb, live += blockIdx.y * st.live;
    surv += blockIdx.y * st.surv, scnt += blockIdx.y * st.counts, fcnt += blockIdx.y * st.counts;
    constexpr int NWV = NT / 64, UR = 8;
    __shared__ uint32_t sacc[64];
    const int ic = find_cfg(item2_off, n_cfg, (int)blockIdx.x);
    const int nblk = item2_off[ic + 1] - item2_off[ic];
    const int cnt = scnt[ic];
    const int lane = threadIdx.x & 63, part = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const CfgDev &c = cfgs[ic];
    const int Vx = c.V[0], Vy = c.V[1];
    const int ny = (Vy + 63) >> 6;
    const int W = (Vx + 31) >> 5;
    const int nr = run_count[ic];
    const auto rsrc = make_rsrc(dil, (int)(D::words() * 4));
    const uint2 *__restrict__ rl = reinterpret_cast<const uint2 *>(runs) + c.run_off;
    // this wavefront's quarter of the runs after the chords, which phase 1 tested
    const int n0 = min(nr, CLASH_CHORDS), nq = nr - n0;
    const int k0 = n0 + nq * part / NWV, k1 = n0 + nq * (part + 1) / NWV;
    int nfree = 0;
    for (int wv = (int)blockIdx.x - item2_off[ic]; 64 * wv < cnt; wv += nblk) {  // block-uniform
        const int idx = 64 * wv + lane;
        const bool act = idx < cnt;
        const uint32_t ent = act ? surv[c.surv_off + idx] : 0u;
        const int tz = (int)(ent >> 16), ty = (int)(ent >> 8) & 255, first = (int)(ent & 255u);
        // the window's words must lie in the row: the last one starts at word
        // W - 1, its bits before `first` belong to other segments
        const int p = min(first, 32 * (W - 1)), w0 = p >> 5, sh = p & 31;
        uint32_t *o = fb + c.free_off + ((int64_t)tz * Vy + ty) * W + w0;
        uint32_t cand = 0u;
        if (part == 0) {
            if (act) cand = ((sh ? o[1] << (32 - sh) : 0u) | o[0] >> sh) & (~0u << (first - p));
            sacc[lane] = ~cand;
        }
        __syncthreads();
        uint32_t acc = sacc[lane];
        // clash bits only ever get set, so wavefronts may exchange them unordered
        auto share = [&]() { acc |= atomicOr(&sacc[lane], acc); };
        const int vo = (tz * D::E + ty) * (D::RW * 4);
        auto test = [&](auto urc, int k) {
            constexpr int U = decltype(urc)::value;
            uint32_t v[U][3], meta[U];
            int s[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint2 e = rl[k + u];
                meta[u] = e.y;
                s[u] = p + (int)(e.y & 31u);
                load_words<3>(rsrc, vo + (s[u] >> 5) * 4, (int)e.x, v[u]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t lo = __builtin_amdgcn_alignbit(v[u][1], v[u][0], s[u]);
                const uint32_t hi = __builtin_amdgcn_alignbit(v[u][2], v[u][1], s[u]);
                acc |= lo | __builtin_amdgcn_alignbit(hi, lo, meta[u] >> 24);
            }
        };
        if (k1 - k0 >= UR) {
            // the last group starts early enough to be whole: a run tested twice is harmless
            for (int k = k0, g = 0; k < k1; k += UR, ++g) {
                test(std::integral_constant<int, UR>{}, min(k, k1 - UR));
                if ((g & 3) == 3) share();
                if (__all(acc == ~0u)) break;
            }
        } else {
            for (int k = k0; k < k1; ++k) test(std::integral_constant<int, 1>{}, k);
        }
        share();
        __syncthreads();
        if (part == 0 && act) {
            const uint32_t clash = cand & sacc[lane], f = cand & ~sacc[lane];
            // segments of a row can meet in a word: cleared by atomics
            if (clash << sh) atomicAnd(o, ~(clash << sh));
            if (sh && clash >> (32 - sh)) atomicAnd(o + 1, ~(clash >> (32 - sh)));
            if (f) live[c.item_base + tz * ny + (ty >> 6)] = 1;  // same value from every writer
            nfree += __popc(f);
        }
    }
    if (part == 0) wave_count(nfree, lane, fcnt + ic);
}

__global__ void k_zero32(int32_t *__restrict__ p, int n) {
    const int i = (int)blockIdx.x * NT + (int)threadIdx.x;
    if (i < n) p[i] = 0;
}

// ------------------------------------------------------------ direct energies
// Eq. 8 with the trilinear weights written out: at translation t,
//   Psi(t) = sum_a sum_(8 corners) w sum_ch gamma_ch G_ch(floor(u_a) + t + corner),
// the sum the transforms evaluate at every translation.  Where few
// translations are clash-free it is evaluated at those alone (k_direct; N = 64
// and 128): no forward planes, no z pass, no inverse.  What decides is the number of
// (free translation, atom) pairs of a configuration and snapshot, known on
// the device once the clash test is done; a configuration with more than
// direct_pairs goes through the transforms, listed by k_modes.  The lines lie
// a little below where the two cost the same (one stream, us per
// configuration): N = 128, FP32: 0.2 + 2.7 per million pairs against 6.7-7.4
// of transforms (8.1 at 347 k pairs and above), equal at 2.5 million; N = 64:
// 0.12 + 3.6 against 1.0-1.15 in FP32, at 270 k, and 0.16 + 7.4 against 2.4 in
// FP64, at 300 k.  8000 site configurations (25 atoms, 3 % of the
// translations free, 160 k pairs each): 46.0 ms of forward planes, z pass and
// inverse -> 3.4 ms.
template <typename T, int N>
__host__ __device__ constexpr long long direct_pairs() {
    return N == 128 ? 2000000 : (sizeof(T) == 8 ? 250000 : 200000);
}
// Whether a grid offers the choice.  It goes by the grid alone: a
// configuration's record is then the same, to the last bit, whatever others
// its call scans.  At N = 32 a transform is so short that the choice's launches,
// some 20 us of a scan's chain, cost as much as it saves: one scan and reduce
// with it against without, us: FP64, 1 configuration 169 : 122, 31 190 : 148,
// 1000 706-765 : 672-787; FP32, 1 188 : 151, 1000 760 : 610-700, 4000
// 1590-1770 : 1420-1730 (300 receptor atoms).  At N = 64 it costs a scan of one
// configuration less than 20 us and pays from a few on: FP32, 1 173 : 158, 24
// 203 : 208, 47 220-228 : 227; FP64, 1 156 : 129, 4 170-176 : 173, 7 168-176 : 179.
template <int N>
constexpr bool offers_direct() {
    return N >= 64;
}
template <typename T, int N>
__device__ __forceinline__ bool by_transforms(int n_free, int n_atoms) {
    return (long long)n_free * n_atoms > direct_pairs<T, N>();
}

// A placed atom of a scanned configuration as k_direct reads it (by scalar
// loads): byte offset of its first corner's point, and the weight of corner
// (dz, dy, dx) for channel ch at [(2 dz + dy) 6 + 3 dx + ch].
template <typename T>
struct alignas(16) CornerAtom {
    int32_t off;
    int32_t pad[3];
    T w[24];
};

template <typename T>
__global__ __launch_bounds__(NT) void k_corner_atoms(const CfgDev *__restrict__ cfgs, const int32_t *__restrict__ zcfg,
                                                     int nz, int ma, const int32_t *__restrict__ ulat,
                                                     const T *__restrict__ gam, int n_rec,
                                                     CornerAtom<T> *__restrict__ out) {
    const int e = (int)blockIdx.x * NT + (int)threadIdx.x;
    const int zi = e / ma, a = e - (e / ma) * ma;
    if (zi >= nz) return;
    const CfgDev c = cfgs[zcfg[zi]];
    if (a >= c.n_atoms) return;
    const int32_t *U = ulat + 3 * (c.u_base + a);
    double f[3][2];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        f[d][1] = (double)(U[d] & 0xffff) * (1.0 / 65536.0);
        f[d][0] = 1.0 - f[d][1];
    }
    CornerAtom<T> r;
    r.off = (((U[2] >> 16) * n_rec + (U[1] >> 16)) * n_rec + (U[0] >> 16)) * 3 * (int)sizeof(T);
    r.pad[0] = r.pad[1] = r.pad[2] = 0;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        const double g = (double)gam[3 * (c.atom_base + a) + ch];
#pragma unroll
        for (int k = 0; k < 8; ++k)  // k = 4 dz + 2 dy + dx; rounded once
            r.w[(k >> 1) * 6 + 3 * (k & 1) + ch] = (T)(f[2][k >> 2] * f[1][(k >> 1) & 1] * f[0][k & 1] * g);
    }
    out[(int64_t)zi * ma + a] = r;
}

// The configurations of a chunk that go through the transforms, per snapshot
// (the launch's ns of them, strides st): zlist[0 .. out[0]) their indices
// among the scanned ones, in order; need[local] = 1 for those whose forward
// planes are not there yet (out[1] of the first snapshot of them), noted in
// done.  One block.
template <typename T, int N>
__global__ __launch_bounds__(NT) void k_modes(const CfgDev *__restrict__ cfgs, const int32_t *__restrict__ zcfg, int nz,
                                              const int32_t *__restrict__ fcnt, int32_t *__restrict__ done,
                                              int32_t *__restrict__ zlist, uint8_t *__restrict__ need,
                                              int32_t *__restrict__ out, int ns, SnapStride st) {
    __shared__ int sh[NT / 64];
    int nneed = 0, total;
    for (int s = 0; s < ns; ++s) {
        int base = 0;
        for (int z0 = 0; z0 < nz; z0 += NT) {
            const int zi = z0 + (int)threadIdx.x;
            bool fft = false, nd = false;
            if (zi < nz) {
                const int l = zcfg[zi];
                fft = by_transforms<T, N>(fcnt[s * st.counts + l], cfgs[l].n_atoms);
                nd = fft && done[l] == 0;  // each configuration by one thread throughout
                if (nd) done[l] = 1;
                if (s == 0 || nd) need[l] = nd ? 1 : 0;
            }
            const int pos = base + block_excl_scan(fft ? 1 : 0, total, sh);
            if (fft) zlist[s * st.zlist + pos] = zi;
            base += total;
            nneed += __syncthreads_count(nd);
        }
        if (threadIdx.x == 0) out[s * st.counts] = base;
    }
    if (threadIdx.x == 0) out[1] = nneed;
}

// Receptor grids [3][n^3] as k_direct reads them, a point's three channels
// side by side.
template <typename T>
__global__ __launch_bounds__(NT) void k_grid_points(const T *__restrict__ grids, int64_t n3, T *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x;
    if (i >= n3) return;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) out[3 * i + ch] = grids[ch * n3 + i];
}

// A grid point's three channels
__device__ __forceinline__ void load_point(__amdgpu_buffer_rsrc_t r, int vo, int so, float *v) {
    const u32x3 a = __builtin_amdgcn_raw_buffer_load_b96(r, vo, so, 0);
    const uint32_t x = a.x, y = a.y, z = a.z;
    v[0] = __builtin_bit_cast(float, x), v[1] = __builtin_bit_cast(float, y), v[2] = __builtin_bit_cast(float, z);
}
__device__ __forceinline__ void load_point(__amdgpu_buffer_rsrc_t r, int vo, int so, double *v) {
    const double2 a = buf_load(r, vo, so, (double2 *)nullptr);
    v[0] = a.x, v[1] = a.y;
    v[2] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, vo + 16, so, 0));
}

// One block per (configuration, box-valid z-translation).  A lane has a point
// of the plane that is a free translation or the point after one, in order of
// the linear index.  A wavefront walks the configuration's atoms; a lane
// reads the four grid points (two along y, two along z) at its own point plus
// an offset in an SGPR, three channels each, and sums them with the atom's
// weights for the near corners and with those for the far ones (scalar
// operands).  The far sum belongs to the translation before, which is the
// lane before: one shuffle after the last atom.  The last lane of a wavefront
// only supplies that; its point is the first of the next group.
// Bound: the loads' way through L1, 48 bytes a lane and atom.  8000 site
// configurations (25 atoms, 96^3 in 128^3): 6.9 ms with both points of a pair
// read by every lane and a grid per channel (lines twice as many), 5.2 with
// the channels side by side, 3.4 with a point a lane.
template <int N>
__host__ __device__ constexpr int direct_threads() {
    return N == 128 ? 256 : 64;
}
template <typename T, int N>
__global__ __launch_bounds__(direct_threads<N>()) void k_direct(
    const int32_t *__restrict__ inv_off, int n_cfg, const CfgDev *__restrict__ cfgs,
    const CornerAtom<T> *__restrict__ atoms, int ma, const T *__restrict__ grids, int n_rec, T beta,
    const uint32_t *__restrict__ fb, const uint8_t *__restrict__ live, const int32_t *__restrict__ fcnt,
    PlanePartial<T> *__restrict__ pp, SnapStride st) {
    grids += blockIdx.y * st.grid, fb += blockIdx.y * st.fb, live += blockIdx.y * st.live;
    fcnt += blockIdx.y * st.counts, pp += blockIdx.y * st.pp;
    constexpr int ND = direct_threads<N>(), NW = N / 32;
    constexpr int MAXW = N * NW;                   // words of a plane's free bits
    constexpr int PER = (MAXW + ND - 1) / ND;
    __shared__ int pre[PER * ND + 1];              // points read before each word
    __shared__ int sh[ND / 64];
    __shared__ LseAcc<T> red[ND / 64];
    const int ic = find_cfg(inv_off, n_cfg, (int)blockIdx.x);
    const CfgDev &c = cfgs[ic];
    const int n_atoms = c.n_atoms;
    if (by_transforms<T, N>(fcnt[ic], n_atoms)) return;
    const int Vx = c.V[0], Vy = c.V[1], tz = (int)blockIdx.x - inv_off[ic];
    LseAcc<T> acc;
    acc.init();
    const int ny = (Vy + 63) >> 6;
    bool l = false;
    for (int g = 0; g < ny; ++g) l = l || live[c.item_base + tz * ny + g] != 0;
    if (!l) {  // block-uniform: every translation of the plane clashes
        if (threadIdx.x == 0) {
            PlanePartial<T> o;
            o.m = -(T)INFINITY;
            o.s = (T)0;
            o.psi_min = (T)INFINITY;
            o.n_finite = 0;
            o.argmin = -1;
            pp[c.pp_base + tz] = o;
        }
        return;
    }
    const int W = (Vx + 31) >> 5, WS = (Vx >> 5) + 1, nw = Vy * WS;  // free words, slot words of a row
    const uint32_t *fp = fb + c.free_off + (int64_t)tz * Vy * W;
    // free bits of slot word w, and the points read: those and the ones after
    auto free_word = [&](int w) {
        const int r = w / WS, q = w - r * WS;
        return q < W ? fp[r * W + q] : 0u;
    };
    auto slot_word = [&](int w) {
        const int r = w / WS, q = w - r * WS;
        const uint32_t f = q < W ? fp[r * W + q] : 0u;
        return f | f << 1 | (q > 0 ? fp[r * W + q - 1] >> 31 : 0u);
    };
    // running counts over the plane's words: thread t owns words PER t ..
    int cnt[PER], mine = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int w = PER * (int)threadIdx.x + k;
        cnt[k] = w < nw ? __popc(slot_word(w)) : 0;
        mine += cnt[k];
    }
    int x = mine;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    if (lane == 63) sh[wv] = x;
    __syncthreads();
    int base = x - mine, S = 0;
#pragma unroll
    for (int i = 0; i < ND / 64; ++i) {
        base += i < wv ? sh[i] : 0;
        S += sh[i];
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        pre[PER * threadIdx.x + k] = base;
        base += cnt[k];
    }
    __syncthreads();
    const int row = n_rec * 3 * (int)sizeof(T), plane = n_rec * row;
    const auto rs = make_rsrc(grids, n_rec * plane);
    const CornerAtom<T> *__restrict__ A = atoms + (int64_t)c.zrow * ma;
    for (int j0 = 63 * wv; j0 < S - 1; j0 += 63 * (ND / 64)) {  // the plane's last point is no translation
        const int j = j0 + lane;
        double near = 0.0, far = 0.0;  // over atoms in FP64: four instructions beside an atom's 24
        int lin = -1;                  // of a free translation
        if (j < S) {
            // word holding slot j, then its (j - pre)-th set bit
            int lo = 0, hi = nw;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (pre[mid] <= j) lo = mid; else hi = mid;
            }
            uint32_t b = slot_word(lo);
            for (int k = j - pre[lo]; k > 0; --k) b &= b - 1u;
            const int bit = __builtin_ctz(b);
            const int ty = lo / WS, tx = 32 * (lo - (lo / WS) * WS) + bit;
            if (lane < 63 && (free_word(lo) >> bit & 1u)) lin = (tz * Vy + ty) * Vx + tx;
            const int vo = ((tz * n_rec + ty) * n_rec + tx) * 3 * (int)sizeof(T);
#pragma unroll 2
            for (int a = 0; a < n_atoms; ++a) {
                const int off = A[a].off;
                T e[2] = {(T)0, (T)0};
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    T v[3];
                    load_point(rs, vo, off + (p >> 1) * plane + (p & 1) * row, v);
#pragma unroll
                    for (int k = 0; k < 6; ++k) e[k / 3] += A[a].w[6 * p + k] * v[k % 3];
                }
                near += (double)e[0];
                far += (double)e[1];
            }
        }
        const double next = __shfl_down(far, 1);
        if (lin >= 0) {
            const T psi = (T)(near + next);
            acc.add(-beta * psi, psi, lin);
        }
    }
    block_partial_store<T, ND>(acc, red, pp + c.pp_base + tz);
}

// ------------------------------------------------------------ z pass
// A placed atom as the energy inputs use it: x/y lattice position and
// fraction, and its channel weights on its two planes, gamma_ch (1 - fz)
// (plane floor(uz)) and gamma_ch fz (plane floor(uz) + 1).
template <typename T>
struct ZAtom {
    T fx, fy;
    int32_t ax, ay;
    T w[6];
};

// One wavefront per scanned configuration of a chunk: its atoms sorted by
// plane (ties in atom order) into zat[zi][.], and zbt[zi][j] = number of
// atoms on planes below ze0 + j - 1 (j = 0 .. Le + 1): plane j of the energy
// window receives the sorted atoms [zbt[j], zbt[j + 2]), those before
// zbt[j + 1] with weight gamma fz, the rest with gamma (1 - fz).
template <typename T, int N>
__global__ __launch_bounds__(NT) void k_zprep(const CfgDev *__restrict__ cfgs, const int32_t *__restrict__ zcfg,
                                               int nz, int ma, const int32_t *__restrict__ ulat,
                                               const T *__restrict__ gam, ZAtom<T> *__restrict__ zat,
                                               int32_t *__restrict__ zbt) {
    __shared__ int saz[NT / 64][MAXA];
    const int wv = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
    const int zi = (int)blockIdx.x * (NT / 64) + wv;
    if (zi >= nz) return;  // per-wavefront work only, no block barrier below
    const CfgDev c = cfgs[zcfg[zi]];
    const int n = c.n_atoms;
    int *az = saz[wv];
    for (int a = lane; a < n; a += 64) az[a] = ulat[3 * (c.u_base + a) + 2] >> 16;
    wave_sync();
    for (int a = lane; a < n; a += 64) {
        const int z = az[a];
        int rk = 0;
        for (int o = 0; o < n; ++o) rk += (az[o] < z || (az[o] == z && o < a)) ? 1 : 0;
        const int32_t *U = ulat + 3 * (c.u_base + a);
        const T fz = (T)(U[2] & 0xffff) * (T)(1.0 / 65536.0);
        ZAtom<T> r;
        r.fx = (T)(U[0] & 0xffff) * (T)(1.0 / 65536.0);
        r.fy = (T)(U[1] & 0xffff) * (T)(1.0 / 65536.0);
        r.ax = U[0] >> 16;
        r.ay = U[1] >> 16;
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            const T g = gam[3 * (c.atom_base + a) + ch];
            r.w[ch] = g * ((T)1 - fz);
            r.w[3 + ch] = g * fz;
        }
        zat[(int64_t)zi * ma + rk] = r;
    }
    for (int j = lane; j <= c.Le + 1; j += 64) {
        const int zt = c.ze0 + j - 1;
        int k = 0;
        for (int o = 0; o < n; ++o) k += az[o] < zt ? 1 : 0;
        zbt[(int64_t)zi * (N + 2) + j] = k;
    }
}

// Block -> (tile of P z-pencils, configuration), with the XCD-aware order
// of the plane path's z kernel: block b of a launch of nb takes logical index
// (b mod 8) (nb / 8) + b / 8.  LIST and a zlist: the configurations are those
// of zlist, nfft[0] of them, a count the host does not know; a grid of fixed
// size then strides over the same order (a launch that finds no configuration
// ends after one load a block).
template <bool LIST>
struct ZWork {
    int nz, total, nb, b;
    const int32_t *zlist;
    __device__ ZWork(int n, int n_tiles, const int32_t *list, const int32_t *nfft) {
        nz = LIST && list ? nfft[0] : n;
        total = n_tiles * nz;
        nb = LIST ? (total + 7) & ~7 : (int)gridDim.x;
        b = (int)blockIdx.x;
        zlist = list;
    }
    __device__ bool more() const { return b < nb; }
    __device__ void next() { b = LIST ? b + (int)gridDim.x : nb; }
    __device__ bool at(int &tile, int &zi) const {
        const int L = (nb % 8 == 0) ? (b % 8) * (nb / 8) + b / 8 : b;
        if (L >= total) return false;
        tile = L / nz;
        zi = L - tile * nz;
        if (LIST && zlist) zi = zlist[zi];
        return true;
    }
};

// ZHI: the configuration's energy window
// (L_e planes, loaded from plane 0; the correlation of the shifted grid is
// the wanted one shifted by ze0, undone at the store) fits in the lower half
// of the pencil, so the first radix-2 stage is pruned.  CLASH: store only
// the z-translations whose live flag is set; a configuration with none is
// skipped whole.
// (The 128-point FP32 instantiations are held to 3 waves per SIMD.)
template <typename T, int N, bool ZHI, bool CLASH>
__global__ __launch_bounds__(NT)
__attribute__((amdgpu_waves_per_eu((N == 128 && sizeof(T) == 4) ? 3 : 1))) void k_zfused(const CfgDev *__restrict__ cfgs, const int32_t *__restrict__ zcfg,
                                                int nz, int n_tiles, int ma, int ac,
                                                const ZAtom<T> *__restrict__ zat, const int32_t *__restrict__ zbt,
                                                const typename Cx<T>::t *__restrict__ rspec,
                                                const typename Cx<T>::t *__restrict__ twg,
                                                typename Cx<T>::t *__restrict__ wsi, const uint8_t *__restrict__ live,
                                                const int32_t *__restrict__ zlist, const int32_t *__restrict__ nfft) {
    using C2 = typename Cx<T>::t;
    using G = Geo<T, N>;
    constexpr int R1 = G::R1, R2 = G::R2, P = G::U, NP = G::NP, H = G::H, PW = G::PW, PAD = G::PAD;
    constexpr int FP = P + 1;  // table row stride (complex): lanes of different planes on distinct banks
    static_assert(R2 <= 16 && NT % P == 0, "store masks and table columns");
    __shared__ C2 buf[4 * G::WREG];
    __shared__ C2 tw[N];
    __shared__ uint32_t lv[N / 32];
    __shared__ int4 pd[N];        // plane j: atoms [x, z) of plane j - 1 (to y) and of plane j
    __shared__ uint32_t smask[R1];  // bit i: FFT lane n1 stores its output slot i
    extern __shared__ __align__(16) unsigned char dyn[];
    ZWork<CLASH> work(nz, n_tiles, zlist, nfft);
    if (!CLASH || work.more()) load_tw<T, N>(tw, twg);
    for (; work.more(); work.next()) {
    int tile, zi;
    if (!work.at(tile, zi)) continue;
    const int tid = CLASH ? opaque(threadIdx.x) : (int)threadIdx.x;  // nothing held across items
    const CfgDev c = cfgs[zcfg[zi]];
    const int Vz = c.V[2];
    if (tid < N / 32) lv[tid] = 0u;
    __syncthreads();
    if (CLASH) {
        const int ny = (c.V[1] + 63) >> 6;
        for (int tz = tid; tz < Vz; tz += NT) {
            bool l = false;
            for (int g = 0; g < ny; ++g) l = l || live[c.item_base + tz * ny + g] != 0;
            if (l) atomicOr(&lv[tz >> 5], 1u << (tz & 31));
        }
    } else {
        for (int tz = tid; tz < Vz; tz += NT) atomicOr(&lv[tz >> 5], 1u << (tz & 31));
    }
    __syncthreads();
    {
        uint32_t any = 0u;
#pragma unroll
        for (int w = 0; w < N / 32; ++w) any |= lv[w];
        if (any == 0u) continue;  // block-uniform: no translation of this configuration is clash-free
    }
    // dynamic LDS (ma = most atoms of a ligand in the launch): per sorted
    // atom its x/y placement, its channel weights [ch][corner][atom], then
    // the factor table F[ac][FP]
    const int n = c.n_atoms;
    int2 *sxy = (int2 *)dyn;                                                  // [ma] ax, ay
    T *sfr = (T *)(((uintptr_t)(sxy + ma) + 15) & ~(uintptr_t)15);           // [ma][2] fx, fy
    T *swt = sfr + 2 * ma;                                                    // [6][ma]
    C2 *F = (C2 *)(((uintptr_t)(swt + 6 * ma) + 15) & ~(uintptr_t)15);       // [ac][FP]
    for (int a = tid; a < n; a += NT) {
        const ZAtom<T> A = zat[(int64_t)zi * ma + a];
        sxy[a] = make_int2(A.ax, A.ay);
        sfr[2 * a] = A.fx;
        sfr[2 * a + 1] = A.fy;
#pragma unroll
        for (int k = 0; k < 6; ++k) swt[k * ma + a] = A.w[k];  // k = corner * 3 + ch: (1 - fz) for 0..2, fz for 3..5
    }
    for (int j = tid; j < c.Le; j += NT) {
        const int32_t *zr = zbt + (int64_t)zi * (N + 2) + j;
        pd[j] = make_int4(zr[0], zr[1], zr[2], 0);
    }
    if (tid < R1) {
        // FFT lane n1 holds output z = n1 + R1 i, translation (z - ze0) mod N
        uint32_t m = 0u;
#pragma unroll
        for (int i = 0; i < R2; ++i) {
            const int tt = (tid + R1 * i - c.ze0) & (N - 1);
            m |= (uint32_t)(tt < Vz && ((lv[tt >> 5] >> (tt & 31)) & 1u)) << i;
        }
        smask[tid] = m;
    }
    __syncthreads();
    const ZLane<N> zl(tid);
    const int n1 = zl.n1, p = zl.p;
    C2 *ex = buf + zl.w * G::WREG + zl.pl;
    const int nchunk = (n + ac - 1) / ac;
    const int pen = tile * P + p;
    const bool ok = pen < NP;
    const int rlane = rs_lane<T, N>(n1, ok ? pen : 0);
    auto build_table = [&](int e0) {
        const int na = min(ac, n - e0);
        const int q = tid % P;
        const int pq = tile * P + q;
        const bool okq = pq < NP;
        const int kyq = okq ? pq / H : 0, kxq = okq ? pq - (pq / H) * H : 0;
        const C2 wx = tw[kxq & (N - 1)], wy = tw[kyq & (N - 1)];
        for (int e = tid / P; e < na; e += NT / P) {
            const int2 axy = sxy[e0 + e];
            const T fx = sfr[2 * (e0 + e)], fy = sfr[2 * (e0 + e) + 1];
            const C2 ex_ = tw[(kxq * axy.x) & (N - 1)], ey = tw[(kyq * axy.y) & (N - 1)];
            const T sxr = (T)1 - fx + fx * wx.x, sxi = fx * wx.y;
            const T syr = (T)1 - fy + fy * wy.x, syi = fy * wy.y;
            const T xr = ex_.x * sxr - ex_.y * sxi, xi = ex_.x * sxi + ex_.y * sxr;
            const T yr = ey.x * syr - ey.y * syi, yi = ey.x * syi + ey.y * syr;
            F[e * FP + q] = okq ? C2{xr * yr - xi * yi, xr * yi + xi * yr} : C2{(T)0, (T)0};
        }
    };
    T er[R2], ei[R2];
#pragma unroll
    for (int i = 0; i < R2; ++i) er[i] = ei[i] = (T)0;
    // Inputs of channel ch: the wavefront computes the values (plane j,
    // pencil pl) of its PW pencils, j-major, into its own exchange region
    // (free until the transform), element j of pencil pl at
    // j PW + (j / R2) PAD + pl; each lane then reads its slots.
    C2 *wbuf = buf + zl.w * G::WREG;
    const int lane = tid & 63;
    const int fcol = zl.w * PW;  // first table column of this wavefront's pencils
    constexpr int NIN = ZHI ? R2 / 2 : R2;
#pragma unroll 1
    for (int ch = 0; ch < 3; ++ch) {
        T re[R2], im[R2];
#pragma unroll
        for (int i = 0; i < R2; ++i) re[i] = im[i] = (T)0;
        const T *w1 = swt + (3 + ch) * ma, *w0 = swt + ch * ma;  // weights gamma fz, gamma (1 - fz)
        for (int ck = 0; ck < nchunk; ++ck) {
            const int e0 = ck * ac, e1 = min(n, e0 + ac);
            if (ch == 0 || nchunk > 1) {
                __syncthreads();
                build_table(e0);
                __syncthreads();
            }
            wave_sync();  // the region may still be read by the previous transform
            for (int idx = lane; idx < PW * c.Le; idx += 64) {
                const int j = idx / PW, pl = idx - (idx / PW) * PW;
                const int4 r = pd[j];
                const C2 *fp = F + (fcol + pl) - e0 * FP;
                T ar = (T)0, ai = (T)0;
                for (int e = max(r.x, e0); e < min(r.y, e1); ++e) {  // atoms of plane j - 1: weight gamma fz
                    const C2 f = fp[e * FP];
                    ar += w1[e] * f.x;
                    ai += w1[e] * f.y;
                }
                for (int e = max(r.y, e0); e < min(r.z, e1); ++e) {  // atoms of plane j: weight gamma (1 - fz)
                    const C2 f = fp[e * FP];
                    ar += w0[e] * f.x;
                    ai += w0[e] * f.y;
                }
                C2 &slot = wbuf[j * PW + (j / R2) * PAD + pl];
                if (ck == 0) slot = C2{ar, ai};
                else slot = C2{slot.x + ar, slot.y + ai};
            }
        }
        wave_sync();
#pragma unroll
        for (int i = 0; i < NIN; ++i) {
            const int j = n1 + R1 * i;
            if (j < c.Le) {
                const C2 v = ex[j * PW + (j / R2) * PAD];
                re[i] = v.x;
                im[i] = v.y;
            }
        }
        fft_unit<T, N, false, ZHI>(re, im, n1, ex, PW, tw, true, PAD);
        rprod<T, N, true>(make_rsrc(rspec + (int64_t)ch * N * NP, N * NP * (int)sizeof(C2)), rlane, re, im, er, ei);
    }
    fft_unit_rev<T, N, true>(er, ei, n1, ex, PW, tw, true, PAD);
    // element z = n1 + R1 i of the output is translation t = z - ze0 (mod N);
    // the live ones (t < Vz) are stored, the others fall outside the
    // descriptor
    const auto rd = make_rsrc(wsi + c.off_inv, Vz * NP * (int)sizeof(C2));
    const int oor = Vz * NP * (int)sizeof(C2);
    const uint32_t sm = ok ? smask[n1] : 0u;
#pragma unroll
    for (int i = 0; i < R2; ++i) {
        const int tt = (n1 + R1 * i - c.ze0) & (N - 1);
        buf_store(rd, ((sm >> i) & 1u) ? (tt * NP + pen) * (int)sizeof(C2) : oor, C2{er[i], ei[i]});
    }
    if (CLASH) __syncthreads();  // the next item reuses the block's tables
    }
}

// z pass from energy planes in device memory (the direct per-atom x/y DFT of
// the forward pass writes plane p of channel ch at off_fwd + (ch L_e + p)
// NP): the same transforms, product and stores as k_zfused, with the next
// channel's planes loaded while the current one is transformed.  Planes at
// or past L_e lie beyond the load descriptor and read as zero.
template <typename T, int N, bool ZHI, bool CLASH>
__global__ __launch_bounds__(NT) void k_zplanes(const CfgDev *__restrict__ cfgs, const int32_t *__restrict__ zcfg,
                                                 int nz, int n_tiles, const typename Cx<T>::t *__restrict__ ws,
                                                 const typename Cx<T>::t *__restrict__ rspec,
                                                 const typename Cx<T>::t *__restrict__ twg,
                                                 typename Cx<T>::t *__restrict__ wsi, const uint8_t *__restrict__ live,
                                                 const int32_t *__restrict__ zlist, const int32_t *__restrict__ nfft) {
    using C2 = typename Cx<T>::t;
    using G = Geo<T, N>;
    constexpr int R1 = G::R1, R2 = G::R2, P = G::U, NP = G::NP, PW = G::PW, PAD = G::PAD;
    static_assert(R2 <= 16, "store masks");
    __shared__ C2 buf[4 * G::WREG];
    __shared__ C2 tw[N];
    __shared__ uint32_t lv[N / 32];
    __shared__ uint32_t smask[R1];  // bit i: FFT lane n1 stores its output slot i
    ZWork<CLASH> work(nz, n_tiles, zlist, nfft);
    if (!CLASH || work.more()) load_tw<T, N>(tw, twg);
    for (; work.more(); work.next()) {
    int tile, zi;
    if (!work.at(tile, zi)) continue;
    const int tid = CLASH ? opaque(threadIdx.x) : (int)threadIdx.x;  // nothing held across items
    const CfgDev c = cfgs[zcfg[zi]];
    const int Vz = c.V[2];
    if (tid < N / 32) lv[tid] = 0u;
    __syncthreads();
    if (CLASH) {
        const int ny = (c.V[1] + 63) >> 6;
        for (int tz = tid; tz < Vz; tz += NT) {
            bool l = false;
            for (int g = 0; g < ny; ++g) l = l || live[c.item_base + tz * ny + g] != 0;
            if (l) atomicOr(&lv[tz >> 5], 1u << (tz & 31));
        }
    } else {
        for (int tz = tid; tz < Vz; tz += NT) atomicOr(&lv[tz >> 5], 1u << (tz & 31));
    }
    __syncthreads();
    {
        uint32_t any = 0u;
#pragma unroll
        for (int w = 0; w < N / 32; ++w) any |= lv[w];
        if (any == 0u) continue;  // block-uniform: no translation of this configuration is clash-free
    }
    if (tid < R1) {
        uint32_t m = 0u;
#pragma unroll
        for (int i = 0; i < R2; ++i) {
            const int tt = (tid + R1 * i - c.ze0) & (N - 1);
            m |= (uint32_t)(tt < Vz && ((lv[tt >> 5] >> (tt & 31)) & 1u)) << i;
        }
        smask[tid] = m;
    }
    __syncthreads();
    const ZLane<N> zl(tid);
    const int n1 = zl.n1, p = zl.p;
    C2 *ex = buf + zl.w * G::WREG + zl.pl;
    const int pen = tile * P + p;
    const bool ok = pen < NP;
    const int rlane = rs_lane<T, N>(n1, ok ? pen : 0);
    const int po = ok ? pen : NP * N;  // out of every descriptor's range
    constexpr int NIN = ZHI ? R2 / 2 : R2;
    C2 pf[NIN];
    auto fetch = [&](int ch) {
        const auto rs = make_rsrc(ws + c.off_fwd + (int64_t)ch * c.Le * NP, c.Le * NP * (int)sizeof(C2));
#pragma unroll
        for (int i = 0; i < NIN; ++i) pf[i] = buf_load(rs, ((n1 + R1 * i) * NP + po) * (int)sizeof(C2), (C2 *)nullptr);
    };
    T er[R2], ei[R2];
#pragma unroll
    for (int i = 0; i < R2; ++i) er[i] = ei[i] = (T)0;
    fetch(0);
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        T re[R2], im[R2];
#pragma unroll
        for (int i = 0; i < R2; ++i) {
            re[i] = i < NIN ? pf[i].x : (T)0;
            im[i] = i < NIN ? pf[i].y : (T)0;
        }
        if (ch < 2) fetch(ch + 1);
        fft_unit<T, N, false, ZHI>(re, im, n1, ex, PW, tw, true, PAD);
        rprod<T, N, true>(make_rsrc(rspec + (int64_t)ch * N * NP, N * NP * (int)sizeof(C2)), rlane, re, im, er, ei);
    }
    fft_unit_rev<T, N, true>(er, ei, n1, ex, PW, tw, true, PAD);
    const auto rd = make_rsrc(wsi + c.off_inv, Vz * NP * (int)sizeof(C2));
    const int oor = Vz * NP * (int)sizeof(C2);
    const uint32_t sm = ok ? smask[n1] : 0u;
#pragma unroll
    for (int i = 0; i < R2; ++i) {
        const int tt = (n1 + R1 * i - c.ze0) & (N - 1);
        buf_store(rd, ((sm >> i) & 1u) ? (tt * NP + pen) * (int)sizeof(C2) : oor, C2{er[i], ei[i]});
    }
    if (CLASH) __syncthreads();  // the next item reuses the block's tables
    }
}

// ------------------------------------------------------------ inverse xy
// One block per (configuration, box-valid z-translation): inverse y on the
// packed columns, C2R along x on row pairs, Eq. 2 partial over the
// clash-free translations.  CLASH: free bits from k_clash; a plane without
// any is not read (its partial is empty) unless energies are exported.
// LIST: only the configurations that go through the transforms (nfft[0] of
// them; k_direct has the others), by a grid that strides over the items.
// WT threads per plane (N = 128: 512, 64 units with one packed column and
// one row pair each, two planes per CU at 4 wavefronts per SIMD).
template <int N>
__host__ __device__ constexpr int inv_fused_threads() {
    return N == 128 ? 512 : NT;
}
template <typename T, int N, bool CLASH, bool LIST, int WT = inv_fused_threads<N>()>
__global__ __launch_bounds__(WT, WT == 512 ? 4 : 1) void k_inv_fused(const int32_t *__restrict__ inv_off, int n_cfg,
                                                   const CfgDev *__restrict__ cfgs,
                                                   const typename Cx<T>::t *__restrict__ wsi, T beta, T inv_n3,
                                                   const typename Cx<T>::t *__restrict__ twg,
                                                   const uint32_t *__restrict__ fb, const uint8_t *__restrict__ live,
                                                   PlanePartial<T> *__restrict__ pp, T *__restrict__ psi_out,
                                                   uint8_t *__restrict__ clash_out,
                                                   unsigned int *__restrict__ e_count, int n_items,
                                                   const int32_t *__restrict__ fcnt,
                                                   const int32_t *__restrict__ nfft) {
    using C2 = typename Cx<T>::t;
    using G = Geo<T, N>;
    constexpr int R1 = G::R1, R2 = G::R2, M = G::M, S = G::S, U = WT / R1, NP = G::NP;
    constexpr int NW = N / 32;
    static_assert(N + (R1 - 1) * G::RPAD <= 2 * S, "row-pair exchange must fit in two rows");
    __shared__ C2 Pl[N * S];
    __shared__ C2 tw[N];
    __shared__ LseAcc<T> red[WT / 64];
    if (LIST && nfft[0] == 0) return;
    load_tw<T, N>(tw, twg);
    for (int item = (int)blockIdx.x; item < n_items; item = LIST ? item + (int)gridDim.x : n_items) {
    const int ic = find_cfg(inv_off, n_cfg, item);
    const CfgDev c = cfgs[ic];
    if (LIST && !by_transforms<T, N>(fcnt[ic], c.n_atoms)) continue;
    const int tid = LIST ? opaque(threadIdx.x) : (int)threadIdx.x;  // nothing held across items
    const int Vx = c.V[0], Vy = c.V[1], tz = item - inv_off[ic];
    const bool exporting = psi_out != nullptr || clash_out != nullptr;
    LseAcc<T> acc;
    acc.init();
    if (CLASH && !exporting) {
        const int ny = (Vy + 63) >> 6;
        bool l = false;
        for (int g = 0; g < ny; ++g) l = l || live[c.item_base + tz * ny + g] != 0;
        if (!l) {  // block-uniform: every translation of the plane clashes
            if (tid == 0) {
                PlanePartial<T> o;
                o.m = -(T)INFINITY;
                o.s = (T)0;
                o.psi_min = (T)INFINITY;
                o.n_finite = 0;
                o.argmin = -1;
                pp[c.pp_base + tz] = o;
            }
            continue;
        }
    }
    if (tid == 0 && e_count) atomicAdd(e_count, 1u);
    const int unit = tid / R1, n1 = tid % R1;
    const C2 *src = wsi + c.off_inv + (int64_t)tz * NP;
    plane_copy<T, N, true, WT>(Pl, const_cast<C2 *>(src), tid);
    __syncthreads();
    T re[R2], im[R2];
    // inverse y on columns (kx = 0 and N/2 packed into column 0), keep y < Vy
    constexpr int rounds_b = (N / 2 + U - 1) / U;
    for (int rd = 0; rd < rounds_b; ++rd) {
        const int col = unit + U * rd;
        const bool lv = col < N / 2;
        const bool c0 = col == 0;
#pragma unroll
        for (int i = 0; i < R2; ++i) {
            const int ky = n1 + R1 * i;
            re[i] = im[i] = (T)0;
            if (lv) {
                const C2 v = Pl[ky * S + col];
                const C2 bq = c0 ? Pl[ky * S + N / 2] : C2{(T)0, (T)0};
                re[i] = v.x - bq.y;
                im[i] = v.y + bq.x;
            }
        }
        C2 *cp = Pl + (lv ? col : 0);
        fft_unit<T, N, true, false, true>(re, im, n1, cp, S, tw, lv);
        wave_sync();  // column col (and N/2 for col = 0) is private to this unit
        if (lv) {
#pragma unroll
            for (int i = 0; i < M; ++i)
#pragma unroll
                for (int k1 = 0; k1 < R1; ++k1) {
                    const int y = spec_index<N>(n1, i, k1);
                    if (y < Vy) {
                        if (c0) {
                            Pl[y * S] = C2{re[i * R1 + k1], (T)0};
                            Pl[y * S + N / 2] = C2{im[i * R1 + k1], (T)0};
                        } else {
                            Pl[y * S + col] = C2{re[i * R1 + k1], im[i * R1 + k1]};
                        }
                    }
                }
        }
    }
    __syncthreads();
    const int W = (Vx + 31) >> 5;
    const uint32_t *fp = fb + c.free_off + (int64_t)tz * Vy * W;
    // inverse x (C2R) of row pairs (y, y+1), y < Vy
    const int npairs = (Vy + 1) / 2;
    const int rounds_a = (npairs + U - 1) / U;
    const int m1 = LIST ? opaque(n1) & (R1 - 1) : n1;
    for (int rd = 0; rd < rounds_a; ++rd) {
        const int y = 2 * (unit + U * rd);
        const bool lv = y < Vy;
        uint32_t f0[NW], f1[NW];
        bool anyf = false;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            f0[w] = f1[w] = 0u;
            if (CLASH && lv && w < W) {
                f0[w] = fp[(int64_t)y * W + w];
                if (y + 1 < Vy) f1[w] = fp[(int64_t)(y + 1) * W + w];
            }
            anyf = anyf || (f0[w] | f1[w]) != 0u;
        }
        // a wavefront whose row pairs hold no clash-free translation has
        // nothing to add
        if (CLASH && !exporting && !__any(lv && anyf)) continue;
        C2 *row = Pl + (lv ? y * S : 0);
#pragma unroll
        for (int i = 0; i < R2; ++i) {
            const int k = m1 + R1 * i;
            re[i] = im[i] = (T)0;
            if (lv) {
                // row values at k (k <= N/2) or conj at N - k; kx = 0, N/2 are real
                const int kk = k <= N / 2 ? k : N - k;
                C2 a = row[kk], bq = row[S + kk];
                const T sg = (k == 0 || k == N / 2) ? (T)0 : (k < N / 2 ? (T)1 : (T)-1);
                a.y *= sg;
                bq.y *= sg;
                re[i] = a.x - bq.y;
                im[i] = a.y + bq.x;
            }
        }
        fft_unit<T, N, true>(re, im, m1, row, 1, tw, lv, G::RPAD);
        if (lv) {
            // clash flags in the epilogue's slot layout: bit 2 sl + h is
            // (x, y + h) with x = spec_index(m1, sl / R1, sl % R1)
            uint32_t cb = 0u;
            if (CLASH) {
#pragma unroll
                for (int sl = 0; sl < R2; ++sl) {
                    const int k1 = sl % R1;
                    const int x = spec_index<N>(m1, sl / R1, k1);
                    const int wi = (R2 * k1) >> 5;  // x >> 5 (compile-time)
                    cb |= (uint32_t)(((f0[wi] >> (x & 31)) & 1u) == 0u) << (2 * sl);
                    cb |= (uint32_t)(((f1[wi] >> (x & 31)) & 1u) == 0u) << (2 * sl + 1);
                }
            }
            uint32_t vb;
            (void)row_pair_epilogue<T, N, CLASH>(re, im, m1, y, Vx, Vy, tz, false, cb, inv_n3, beta, psi_out,
                                                clash_out, acc, vb);
        }
    }
    block_partial_store<T, WT>(acc, red, pp + c.pp_base + tz, tid);
    }
}

// ------------------------------------------------------------ launchers
template <typename T, int N>
struct LaunchFused {
    // blocks of a launch over a list made on the device: a few times what the
    // chip holds of them (z pass three, inverse two a compute unit), so that the
    // last round is short and an empty list costs about 5 us
    static constexpr int LIST_BLOCKS_Z = 3072, LIST_BLOCKS = 1024;
    using C2 = typename Cx<T>::t;
    using G = Geo<T, N>;
    static hipError_t rec_dilate(hipStream_t st, const uint8_t *occ, int n_rec, uint32_t *dil) {
        constexpr int rows = Dil<N>::E * Dil<N>::E;
        hipLaunchKernelGGL((k_rec_dilate<N>), dim3((rows + NT - 1) / NT), dim3(NT), 0, st, occ, n_rec, dil);
        return hipGetLastError();
    }
    static hipError_t lig_runs(hipStream_t st, const CfgDev *cfgs, const int32_t *zcfg, int nz, const int32_t *ulat,
                               const double *thr, uint32_t *runs, int32_t *run_count) {
        if (nz <= 0) return hipSuccess;
        hipLaunchKernelGGL((k_lig_runs<N>), dim3(nz), dim3(RUN_NT), 0, st, cfgs, zcfg, ulat, thr, runs, run_count);
        return hipGetLastError();
    }
    static hipError_t zero(hipStream_t st, int32_t *p, int64_t n) {
        constexpr int64_t most = 1 << 30;  // of a launch, whose threads must number fewer than 2^32
        for (; n > 0; p += most, n -= most) {
            const int k = (int)(n < most ? n : most);
            hipLaunchKernelGGL(k_zero32, dim3((unsigned)((k + NT - 1) / NT)), dim3(NT), 0, st, p, k);
        }
        return hipGetLastError();
    }
    static hipError_t clash(hipStream_t st, int ns, const SnapStride &ss, const int32_t *item_off,
                            const int32_t *item2_off, int n_cfg, int n_items, int n_items2, const CfgDev *cfgs,
                            const uint32_t *runs, const int32_t *run_count, const uint32_t *dil, uint32_t *fb,
                            uint8_t *live, uint32_t *surv, int32_t *scnt, int32_t *fcnt) {
        if (n_items <= 0) return hipSuccess;
        hipLaunchKernelGGL((k_clash1<N>), dim3((n_items + NT / 64 - 1) / (NT / 64), ns), dim3(NT), 0, st, item_off,
                           n_cfg, n_items, cfgs, runs, run_count, dil, fb, live, surv, scnt, fcnt, ss);
        if (n_items2 > 0)
            hipLaunchKernelGGL((k_clash2<N>), dim3(n_items2, ns), dim3(NT), 0, st, item2_off, n_cfg, n_items2, cfgs,
                               runs, run_count, dil, fb, live, surv, scnt, fcnt, ss);
        return hipGetLastError();
    }
    static hipError_t corner_atoms(hipStream_t st, const CfgDev *cfgs, const int32_t *zcfg, int nz, int max_atoms,
                                   const int32_t *ulat, const void *gam, int n_rec, void *atoms) {
        if (nz <= 0) return hipSuccess;
        hipLaunchKernelGGL((k_corner_atoms<T>), dim3((unsigned)(((int64_t)nz * max_atoms + NT - 1) / NT)), dim3(NT), 0,
                           st, cfgs, zcfg, nz, max_atoms, ulat, (const T *)gam, n_rec, (CornerAtom<T> *)atoms);
        return hipGetLastError();
    }
    static hipError_t modes(hipStream_t st, int ns, const SnapStride &ss, const CfgDev *cfgs, const int32_t *zcfg,
                            int nz, const int32_t *fcnt, int32_t *done, int32_t *zlist, uint8_t *need, int32_t *out) {
        hipLaunchKernelGGL((k_modes<T, N>), dim3(1), dim3(NT), 0, st, cfgs, zcfg, nz, fcnt, done, zlist, need, out,
                           ns, ss);
        return hipGetLastError();
    }
    static hipError_t direct(hipStream_t st, int ns, const SnapStride &ss, const int32_t *inv_off, int n_cfg,
                             int n_items, const CfgDev *cfgs, const void *atoms, int max_atoms, const void *grids, int n_rec, double beta,
                             const uint32_t *fb, const uint8_t *live, const int32_t *fcnt, void *pp) {
        if (n_items <= 0) return hipSuccess;
        hipLaunchKernelGGL((k_direct<T, N>), dim3(n_items, ns), dim3(direct_threads<N>()), 0, st, inv_off, n_cfg, cfgs,
                           (const CornerAtom<T> *)atoms, max_atoms, (const T *)grids, n_rec, (T)beta, fb, live, fcnt,
                           (PlanePartial<T> *)pp, ss);
        return hipGetLastError();
    }
    static hipError_t grid_points(hipStream_t st, const void *grids, int n_rec, void *out) {
        const int64_t n3 = (int64_t)n_rec * n_rec * n_rec;
        hipLaunchKernelGGL((k_grid_points<T>), dim3((unsigned)((n3 + NT - 1) / NT)), dim3(NT), 0, st, (const T *)grids,
                           n3, (T *)out);
        return hipGetLastError();
    }
    static int atoms_per_table() {
        constexpr int FP = G::U + 1;
        int a = (int)(FUSED_TABLE_BYTES / (FP * sizeof(C2)));
        return a < 1 ? 1 : a;
    }
    static size_t dyn_bytes(int max_atoms) {
        const int ac = max_atoms < atoms_per_table() ? max_atoms : atoms_per_table();
        size_t o = (size_t)max_atoms * 2 * sizeof(int);
        o = (o + 15) & ~(size_t)15;
        o += (size_t)max_atoms * 8 * sizeof(T);
        o = (o + 15) & ~(size_t)15;
        return o + (size_t)ac * (G::U + 1) * sizeof(C2) + 16;
    }
    static hipError_t zprep(hipStream_t st, const CfgDev *cfgs, const int32_t *zcfg, int nz, int max_atoms,
                            const int32_t *ulat, const void *gam, void *zat, int32_t *zbt) {
        if (nz <= 0) return hipSuccess;
        hipLaunchKernelGGL((k_zprep<T, N>), dim3((nz + NT / 64 - 1) / (NT / 64)), dim3(NT), 0, st, cfgs, zcfg, nz,
                           max_atoms, ulat, (const T *)gam, (ZAtom<T> *)zat, zbt);
        return hipGetLastError();
    }
    // blocks of a z pass: one per (tile, configuration), or, over a list whose
    // length only the device knows, as many as keep the chip full
    static long long z_blocks(int n_tiles, int nz, bool list) {
        const long long nb = ((long long)n_tiles * nz + 7) / 8 * 8;
        return list && nb > LIST_BLOCKS_Z ? LIST_BLOCKS_Z : nb;
    }
    static hipError_t zpass(hipStream_t st, bool zhalf, bool clash, const CfgDev *cfgs, const int32_t *zcfg, int nz,
                            int max_atoms, const void *zat, const int32_t *zbt, const void *rspec, const void *tw,
                            void *wsi, const uint8_t *live, const int32_t *zlist, const int32_t *nfft) {
        if (nz <= 0) return hipSuccess;
        const int n_tiles = (G::NP + G::U - 1) / G::U;
        const long long nb = z_blocks(n_tiles, nz, zlist != nullptr);
        const int ac = max_atoms < atoms_per_table() ? max_atoms : atoms_per_table();
        const size_t dyn = dyn_bytes(max_atoms);
#define FFTDG_ZF(Z, C)                                                                                            \
    hipLaunchKernelGGL((k_zfused<T, N, Z, C>), dim3((unsigned)nb), dim3(NT), dyn, st, cfgs, zcfg, nz, n_tiles,      \
                       max_atoms, ac, (const ZAtom<T> *)zat, zbt, (const C2 *)rspec, (const C2 *)tw, (C2 *)wsi, live, zlist, \
                       nfft)
        if (zhalf && clash) FFTDG_ZF(true, true);
        else if (zhalf) FFTDG_ZF(true, false);
        else if (clash) FFTDG_ZF(false, true);
        else FFTDG_ZF(false, false);
#undef FFTDG_ZF
        return hipGetLastError();
    }
    static hipError_t zplanes(hipStream_t st, bool zhalf, bool clash, const CfgDev *cfgs, const int32_t *zcfg,
                              int nz, const void *ws, const void *rspec, const void *tw, void *wsi,
                              const uint8_t *live, const int32_t *zlist, const int32_t *nfft) {
        if (nz <= 0) return hipSuccess;
        const int n_tiles = (G::NP + G::U - 1) / G::U;
        const long long nb = z_blocks(n_tiles, nz, zlist != nullptr);
#define FFTDG_ZP(Z, C)                                                                                     \
    hipLaunchKernelGGL((k_zplanes<T, N, Z, C>), dim3((unsigned)nb), dim3(NT), 0, st, cfgs, zcfg, nz, n_tiles, \
                       (const C2 *)ws, (const C2 *)rspec, (const C2 *)tw, (C2 *)wsi, live, zlist, nfft)
        if (zhalf && clash) FFTDG_ZP(true, true);
        else if (zhalf) FFTDG_ZP(true, false);
        else if (clash) FFTDG_ZP(false, true);
        else FFTDG_ZP(false, false);
#undef FFTDG_ZP
        return hipGetLastError();
    }
    static hipError_t inv(hipStream_t st, bool clash, const int32_t *inv_off, int n_cfg, int n_items,
                          const CfgDev *cfgs, const void *wsi, double beta, const void *tw, const uint32_t *fb,
                          const uint8_t *live, void *pp, void *psi_out, uint8_t *clash_out, unsigned int *e_count,
                          const int32_t *fcnt, const int32_t *nfft) {
        if (n_items <= 0) return hipSuccess;
        const T b = (T)beta, s = (T)(1.0 / ((double)N * N * N));
        const int nb = fcnt && n_items > LIST_BLOCKS ? LIST_BLOCKS : n_items;
#define FFTDG_INV(C, L)                                                                                            \
    hipLaunchKernelGGL((k_inv_fused<T, N, C, L>), dim3(nb), dim3(inv_fused_threads<N>()), 0, st, inv_off, n_cfg, cfgs, \
                       (const C2 *)wsi, b, s, (const C2 *)tw, fb, live, (PlanePartial<T> *)pp, (T *)psi_out,        \
                       clash_out, e_count, n_items, fcnt, nfft)
        if constexpr (offers_direct<N>())
            if (clash && fcnt) {
                FFTDG_INV(true, true);
                return hipGetLastError();
            }
        if (clash) FFTDG_INV(true, false);
        else FFTDG_INV(false, false);
#undef FFTDG_INV
        return hipGetLastError();
    }
};

template <typename T, int N>
static FusedSet fused_launchers() {
    using L = LaunchFused<T, N>;
    FusedSet s{};
    s.n_fft = N;
    s.dil_words = Dil<N>::words();
    s.margin = Dil<N>::M;
    s.rec_dilate = L::rec_dilate;
    s.lig_runs = L::lig_runs;
    s.zero = L::zero;
    s.clash = L::clash;
    if constexpr (offers_direct<N>()) {
        s.corner_bytes = sizeof(CornerAtom<T>);
        s.corner_atoms = L::corner_atoms;
        s.modes = L::modes;
        s.direct = L::direct;
        s.grid_points = L::grid_points;
    }
    s.zprep = L::zprep;
    s.zat_bytes = sizeof(ZAtom<T>);
    s.zpass = L::zpass;
    s.zplanes = L::zplanes;
    s.inv = L::inv;
    s.z_lds = L::dyn_bytes;
    return s;
}
template <typename T, int N>
static const FusedSet *make_fused() {
    static const FusedSet s = fused_launchers<T, N>();
    return &s;
}

const FusedSet *fused_set(int precision, int n_fft) {
    if (precision == FFTDG_F32) {
        if (n_fft == 32) return make_fused<float, 32>();
        if (n_fft == 64) return make_fused<float, 64>();
        if (n_fft == 128) return make_fused<float, 128>();
    } else if (precision == FFTDG_F64) {
        if (n_fft == 32) return make_fused<double, 32>();
        if (n_fft == 64) return make_fused<double, 64>();
    }
    return nullptr;
}

}  // namespace fftdg
