// psm_internal.h -- structures and device helpers shared by the engine's
// kernels and host code (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace psm {

constexpr int NQ = 19;
constexpr int WG = 256;          // threads per workgroup of the step kernel
constexpr int NWAVE = WG / 64;   // 64-wide wavefronts per workgroup
constexpr int MAXC = 64;         // sphere candidates per tile staged in LDS
constexpr int TZ_MAX = 32;   // largest cells per thread along z of a tile
constexpr int NXCD = 8;          // MI355X: 8 accelerator complex dies, 32 CUs each
#ifndef PSM_BLK
#define PSM_BLK 64
#endif
constexpr int BLK = PSM_BLK;     // cells per PDF storage block (one wavefront)

// D3Q19 velocity set in the canonical order of the ABI (psm.h). Directions
// come in inverse pairs (2k-1, 2k) for k = 1..9.
constexpr int CX[NQ] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
constexpr int CY[NQ] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1};
constexpr int CZ[NQ] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1};
constexpr double W0 = 1.0 / 3.0, W1 = 1.0 / 18.0, W2 = 1.0 / 36.0;
__host__ __device__ constexpr double wq(int q) { return q == 0 ? W0 : (q <= 6 ? W1 : W2); }

// Per-box constants, stored in device memory and read with scalar loads.
struct BoxDev {
    int nx, ny, nz, N;
    int ntx, nty, ntz, tile_base;   // tiles per axis, first global tile
    unsigned div_ntx[2], div_nty[2];   // udiv_magic of ntx and nty
    int part_base, np, mapping, nsub;
    // force partials of a sphere: slots pbase + (local id) * pstride + k for
    // the k-th tile of its bounding box (pstride bounds the tiles a sphere of
    // this box can touch at the current tile shape), each one partial per
    // workgroup that shares the tile
    int pstride, pbase;
    // PDF storage: each z-plane holds pblk blocks of 64 cells (pitch*ny
    // rounded up); a block stores its 19 directions one after another, 64
    // values each. Cell (x, y) of a plane is in-plane cell x + pitch*y.
    int pitch;                      // row pitch in cells, see row_pitch() and row_pitches()
    int pblk;                       // blocks per z-plane
    long long plane_elems;          // values per z-plane, pblk * 19 * 64
    void* grid[2];                  // ping-pong PDF grids, nz * plane_elems values
    double omega, pref;             // 1/tau, 1 - 1/(2 tau)
    double g[3];                    // body-force density
    // Forcing constants of eq. (8) with the Guo prefactor, precomputed on the
    // host so that the kernel reads them from scalar registers:
    //   F_q = fa[k] + fs[k] (c_q.U) - pw[class] 3 (U.g) for the pair k = (q, q+1),
    //   F_qbar = -fa[k] + fs[k] (c_q.U) - pw[class] 3 (U.g).
    double fa[9], fs[9];            // 3 pref w (c.g), 9 pref w (c.g)
    double fa_scaled[9];            // fa times the FP16 storage scale
    double pw[3];                   // pref w for the rest, axis and diagonal weights
    // Collision constants per weight class c (rest, axis, diagonal) with the
    // FP16 storage scale s folded in (s = 1 otherwise):
    //   k15 = 1.5/s, k45 = 4.5/s, wk[c] = W_c k45, owk[c] = omega W_c k45, ow3[c] = 3 omega W_c
    double om1, k15, k45, wk[3], owk[3], ow3[3];
    // FP32 copies of the collision constants for the deviation forms
    float omega_f, g_f[3], fa_f[9], fs_f[9], fa_scaled_f[9], pw_f[3];
    float om1_f, k15_f, k45_f, wk_f[3], owk_f[3], ow3_f[3];
    // rounding margin (cells) of the step kernel's FP32 reach test
    double margin32;
    // Geometry constants for the minimum image and the sub-sample test.
    double L[3], halfL[3];          // box lengths and their halves
    double sub_off[16];             // (k + 1/2)/nsub - 1/2, k < nsub
    double reach;                   // sqrt(3) (1/2 - 1/(2 nsub)) + 1e-9
    // Sphere dynamics of the box: density ratio to the fluid and external
    // acceleration (gravity minus buoyancy) used by the integrator.
    double rho_p;
    double accel[3];
    // Faces at z = 0 and z = nz instead of periodicity (walls != 0). On a
    // velocity face w a population q entering a boundary cell is the one the
    // cell sent against the face (direction inv_dir(q)) plus bw[w][q] =
    // 6 w_q (c_q . u_w) (half-way bounce-back); on a pressure face it is
    // minus that population plus 2 w_q (face_rho[w] + 4.5 (c_q.u)^2 - 1.5 u.u)
    // with u the cell's post-collision velocity (anti-bounce-back).
    int walls;
    int walls_xy;                   // bit 0: resting walls at x = 0, nx; bit 1: at y = 0, ny
    int face_type[2];               // FACE_VELOCITY or FACE_PRESSURE
    double face_rho[2];
    double bw[2][NQ];
};
enum { FACE_VELOCITY = 0, FACE_PRESSURE = 1 };

// Multiplier and shift of a division by d: with l = ceil(log2 d) and mul =
// ceil(2^(31+l) / d) < 2^32, n / d = mulhi(mul, n) >> (l - 1) for n < 2^31 (the
// excess mul n / 2^(31+l) - n / d is below n / 2^(31+l) < 2^-l <= 1 / d).
// d = 1: mul = 0, which stands for n itself.
inline void udiv_magic(unsigned d, unsigned out[2]) {
    unsigned l = 0;
    while ((1ull << l) < d) ++l;
    out[0] = l ? (unsigned)(((1ull << (31 + l)) + d - 1) / d) : 0;
    out[1] = l ? l - 1 : 0;
}

// Opposite direction: the pairs (1,2), (3,4), ..., (17,18) are opposite.
__host__ __device__ constexpr int inv_dir(int q) { return q == 0 ? 0 : ((q & 1) ? q + 1 : q - 1); }

// Global particle table, SoA, indexed by global particle id.
struct Particles {
    double *x, *y, *z, *r, *fr, *ux, *uy, *uz, *ox, *oy, *oz;
    double* acc;     // [P][6]: F (3), T (3) of the last step
    double* fprev;   // [P][6]: total force and torque of the previous integration (velocity Verlet)
    int* prev_ok;    // [P]: 1 once fprev holds a value
};

struct TileShape {
    int tx, ty, tz;
    int persistent;   // 1: occupancy-sized grid walking the tiles; 0: a workgroup per part of a tile
    int filter;       // 1: per-wave candidate filter before the per-cell mapping
    int ref_z;        // depth of the z-blocks whose centres the FP32 geometry refers to (a multiple of tz)
    int zshift;       // 1 << zshift workgroups share a tile's cells along z
};

// ---------------------------------------------------------------------------
// Tiles of one axis touched by a particle's bounding box.
// The box along the axis covers cells [lo, hi] (unwrapped, hi - lo + 1 <= L).
// Wrapped into [0, L) it is one or two cell segments; their tiles form at most
// two contiguous tile ranges [a0,a1] and [b0,b1] (b empty if b1 < b0), with no
// tile listed twice. Every caller walks them in the same order.
struct AxisTiles {
    int a0, a1, b0, b1;
    __host__ __device__ int count() const { return (a1 - a0 + 1) + (b1 >= b0 ? b1 - b0 + 1 : 0); }
    __host__ __device__ int at(int k) const {
        int na = a1 - a0 + 1;
        return k < na ? a0 + k : b0 + (k - na);
    }
};

__host__ __device__ inline int floordiv(int a, int b) { return a >= 0 ? a / b : -((-a + b - 1) / b); }

__host__ __device__ inline AxisTiles axis_tiles(int lo, int hi, int L, int T, int nt) {
    AxisTiles r;
    if (lo >= 0 && hi < L) {
        r.a0 = lo / T; r.a1 = hi / T; r.b0 = 0; r.b1 = -1;
        return r;
    }
    int s0, s1, u0, u1;   // segment [s0, L-1] and [0, u1]
    if (lo < 0) { s0 = lo + L; u1 = hi; }
    else { s0 = lo; u1 = hi - L; }
    (void)u0; (void)s1;
    int ta0 = s0 / T, tb1 = u1 / T;
    if (tb1 >= ta0) { r.a0 = 0; r.a1 = nt - 1; r.b0 = 0; r.b1 = -1; }
    else { r.a0 = ta0; r.a1 = nt - 1; r.b0 = 0; r.b1 = tb1; }
    return r;
}

// Cell range of the bounding box [x - (r+1), x + (r+1)] along one axis.
__host__ __device__ inline void aabb_cells(double x, double r, int& lo, int& hi) {
    lo = (int)floor(x - (r + 1.0));
    hi = (int)floor(x + (r + 1.0));
}

// Row pitch of the PDF layout: a row that does not fill whole 64-cell
// blocks is padded to the next block boundary when that costs at most 1/8 of
// the row, so that every row of a tile starts on a block and a wave's loads
// and stores of one direction stay in one block (or two, for a shift in x).
// Narrower rows are packed back to back, unless the host's choice for large
// grids lets each start at a line.
__host__ __device__ inline int row_pitch(int nx) {
    int up = (nx + BLK - 1) / BLK * BLK;
    return 8LL * up <= 9LL * nx ? up : nx;
}

// Element index of direction q of cell (x, y, z) in a box's PDF grid.
__host__ __device__ inline long long pdf_index(const BoxDev& b, int q, int x, int y, int z) {
    int s = x + b.pitch * y;
    return (long long)z * b.plane_elems + (long long)(s / BLK) * (NQ * BLK) + q * BLK + (s % BLK);
}

// ---------------------------------------------------------------------------
// Minimum image of one displacement component into [-L/2, L/2)
// (hL = L/2, exact).
__host__ __device__ inline double min_image(double d, double L, double hL) {
    // two selects (no branch): the conditions exclude each other
    double r = d >= hL ? d - L : d;
    return d < -hL ? d + L : r;
}

// Overlap fraction of a sphere (radius r, f(r) = fr) with the cell whose
// centre lies at displacement (dx, dy, dz) from the sphere centre.
// Linear approximation (Sec. 2.3.2, eq. 26): eps = f(r) - (|d| - r), overlap
// iff eps > 0, capped at 1. No fused multiply-add, so that the fraction is
// reproducible bit for bit.
__device__ inline double overlap_linear(double dx, double dy, double dz, double r, double fr) {
#pragma clang fp contract(off)
    double d2 = dx * dx + dy * dy + dz * dz;
    double lim = r + fr + 1e-9;
    if (d2 > lim * lim) return 0.0;
    double eps = fr - (sqrt(d2) - r);
    if (eps <= 0.0) return 0.0;
    return eps < 1.0 ? eps : 1.0;
}

// Sub-division sampling: fraction of the nsub^3 points at offsets off[k] =
// (k+1/2)/nsub - 1/2 that lie inside the sphere (|s| <= r). Cells farther
// than r + reach from the centre hold no sample inside, cells nearer than
// r - reach hold only inside samples. The test is discontinuous: no fused
// multiply-add, evaluation order ((sx sx + sy sy) + sz sz).
template <class OffPtr>
__device__ inline double overlap_subsample(double dx, double dy, double dz, double r, int nsub, OffPtr off,
                                           double reach) {
#pragma clang fp contract(off)
    double d2 = dx * dx + dy * dy + dz * dz;
    double hi = r + reach;
    if (d2 > hi * hi) return 0.0;
    double lo = r - reach;
    if (lo > 0.0 && d2 < lo * lo) return 1.0;
    const double r2 = r * r;
    int inside = 0;
    // The squares of one chunk of four offsets per axis stay in registers: with
    // off[] read inside the three loops each of the nsub^3 tests waited for a
    // scalar load (4^3 points: FP64 32^3 19.4 -> 13.5 us a step, 128^3 154 ->
    // 134; FP16 128^3 113 -> 82). An offset past nsub gives an infinite square,
    // which is never inside.
    for (int cx = 0; cx < nsub; cx += 4) {
        double sx2[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double sx = dx + off[cx + k];   // off has 16 entries
            sx2[k] = cx + k < nsub ? sx * sx : __builtin_inf();
        }
        for (int cy = 0; cy < nsub; cy += 4) {
            double sy2[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double sy = dy + off[cy + k];
                sy2[k] = cy + k < nsub ? sy * sy : __builtin_inf();
            }
            for (int cz = 0; cz < nsub; cz += 4) {
                double sz2[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const double sz = dz + off[cz + k];
                    sz2[k] = cz + k < nsub ? sz * sz : __builtin_inf();
                }
#pragma unroll
                for (int kx = 0; kx < 4; ++kx)
#pragma unroll
                    for (int ky = 0; ky < 4; ++ky) {
                        const double xy = sx2[kx] + sy2[ky];
#pragma unroll
                        for (int kz = 0; kz < 4; ++kz) inside += (xy + sz2[kz] <= r2) ? 1 : 0;
                    }
            }
        }
    }
    return (double)inside / ((double)nsub * nsub * nsub);
}

// Two-slot list of one cell (Sec. 3.1.1 stores at most two fractions per
// cell). A candidate is stronger with a larger fraction, ties broken by the
// smaller particle id; a third overlap drops the weakest and is counted.
struct Slots {
    int c0, c1;      // candidate index (or particle id), -1 if empty
    int p0, p1;      // particle id used for ordering
    double B0, B1;
    int dropped;
};

__device__ inline bool stronger(double Ba, int pa, double Bb, int pb) {
    return Ba > Bb || (Ba == Bb && pa < pb);
}

__device__ inline void slots_init(Slots& s) {
    s.c0 = s.c1 = -1; s.p0 = s.p1 = 0x7fffffff; s.B0 = s.B1 = 0.0; s.dropped = 0;
}

__device__ inline void slots_insert(Slots& s, int c, int p, double B) {
    if (s.c0 < 0) { s.c0 = c; s.p0 = p; s.B0 = B; return; }
    if (s.c1 < 0) { s.c1 = c; s.p1 = p; s.B1 = B; return; }
    s.dropped++;
    // the weaker of the two kept slots
    bool w1 = stronger(s.B0, s.p0, s.B1, s.p1);
    if (w1) {
        if (stronger(B, p, s.B1, s.p1)) { s.c1 = c; s.p1 = p; s.B1 = B; }
    } else {
        if (stronger(B, p, s.B0, s.p0)) { s.c0 = c; s.p0 = p; s.B0 = B; }
    }
}

// Ascending particle id, then the B > 1 renormalisation of Sec. 2.3.
__device__ inline void slots_finish(Slots& s) {
    if (s.c1 >= 0 && s.p0 > s.p1) {
        int tc = s.c0; s.c0 = s.c1; s.c1 = tc;
        int tp = s.p0; s.p0 = s.p1; s.p1 = tp;
        double tb = s.B0; s.B0 = s.B1; s.B1 = tb;
    }
    if (s.c1 >= 0) {
        double sum = s.B0 + s.B1;
        if (sum > 1.0) { s.B0 = s.B0 / sum; s.B1 = s.B1 / sum; }
    }
}

// ---------------------------------------------------------------------------
// Launch parameters (passed by value) and launchers of psm_kernels.hip.

struct StepParams {
    const BoxDev* boxes;
    const int* box_tile_base;   // [nbox+1]
    int nbox;
    Particles P;
    const int* tile_cnt;        // [T] spheres of each tile's list (uncapped); compact lists: then [T] their first entries
    const int2* tile_ent;       // global particle id and force-partial slot
    int list_cap;               // entries per list; compact lists: minus the most that one holds
    double* partial;            // [slots << zshift][6]
    // force reduction of the step before (its partials; null: none) by the
    // workgroups from `grid` on, 4 spheres each
    const double* partial_prev;
    const int* part_box;        // [P] box of each global particle slot
    int P_total;
    int grid;                   // workgroups that walk tiles
    int T_total;                // parts of tiles: tiles << zshift
    int tx, ty, tz;
    int depth, zshift;          // cells per thread: tz >> zshift, TileShape::zshift
    int ref_z;                  // TileShape::ref_z
    int parity;
    float h_scale, h_inv;       // FP16 storage scale and its inverse (1 otherwise)
    int* flags;                 // device error word: |= FLAG_SLOT_OVERFLOW when a cell meets a third sphere,
                                // FLAG_LIST_CUT when a tile's list was cut
    int run;                    // parts taken from the queue at once: 1 << run
    int* queue;                 // [NXCD] tile counters of the persistent grid (zeroed before the launch), or null
};

// Work per sphere (one wave each): any of the force reduction, the sphere
// update and the tile lists.
enum { SCHEME_NONE = -1, SCHEME_EULER = 0, SCHEME_VERLET = 1 };
struct SphereParams {
    const BoxDev* boxes;
    const int* part_box;        // [P] box of each global particle slot
    Particles P;
    // force partials [slots << zshift][6] of the last step, and those the next step
    // writes: both zeroed for an entry a full list drops
    double *partial, *partial_next;
    int P_total;
    TileShape ts;
    double dt;                  // sphere update
    // tile lists: the counts filled here are zero on entry; those of the
    // lists they replace are zeroed for the next build
    int *cnt, *cnt_old;         // [T]
    const int* off;             // [T] first entry of each list (compact lists; null: list_cap entries each)
    int count_only;             // count the lists' spheres only (compact lists, before their offsets)
    int2* ent;
    int list_cap;
    int T_total;                // counts to zero (compact lists: none)
    int *over, *over_old;       // largest uncapped count where it exceeds MAXC, else 0
    // force read-back: pinned host copy of P.acc and the error words behind
    // it (null: none)
    double* host_acc;
    const int* err;
};

// Sphere-table columns uploaded from pinned host staging: `ncols` columns from
// column `first` on (x y z r f(r) U Omega), n values each, m apart in the
// staging and `pitch` apart on the device.
struct UploadParams {
    const double* src;
    double* table;              // column 0 of the box's spheres
    long long pitch;
    int first, ncols, n, m;
    int* prev_ok;               // [m] cleared when velocities are uploaded (null: not)
    int* np;                    // the box's sphere count, set to n (null: not)
    int part_base;              // first global sphere slot of the box
};
// Sphere data written to pinned host memory, with the error words after it.
struct DownloadParams {
    const double* src[2];
    long long pitch[2];         // doubles between the columns of a range
    int ncols[2];
    long long n;                // values per column
    double* dst;                // the columns one after another
    const int* err;
    int* err_dst;
};

// Instance of the step kernel.
enum CacheForm {
    MIXED,     // nontemporal stores
    KEEP,      // ordinary loads and stores
    STREAM,    // nontemporal stores, and loads of the lines that one wave alone reads
};
struct StepForm {
    bool map;       // a box samples its fractions
    bool filter;    // per-wave candidate filter
    bool walls;     // a box has walls or faces
    int cache;      // CacheForm (MIXED with the filter)
};
hipError_t launch_step(int storage, const StepForm& form, const StepParams& kp, hipStream_t st);
hipError_t launch_pattern_copy(int storage, bool shifted, const StepParams& kp, hipStream_t st);
int step_blocks_per_cu(int storage, const StepForm& form);
hipError_t launch_spheres(bool reduce, int scheme, bool bin, const SphereParams& sp, hipStream_t st);
hipError_t launch_list_offsets(int* cnt, int* off, int T, int list_cap, hipStream_t st);
hipError_t launch_upload_bin(const SphereParams& sp, const UploadParams& up, hipStream_t st);
hipError_t launch_upload(const UploadParams& up, hipStream_t st);
hipError_t launch_download(const DownloadParams& dp, hipStream_t st);
hipError_t launch_set_pdfs(int storage, const BoxDev& bx, int parity, const double* f, float scale, hipStream_t st);
hipError_t launch_set_equilibrium(int storage, const BoxDev& bx, int parity, const double* rho, const double* u,
                                  float scale, hipStream_t st);
hipError_t launch_get_pdfs(int storage, const BoxDev& bx, int parity, double* f, float inv, hipStream_t st);
hipError_t launch_get_pdfs_at(int storage, const BoxDev& bx, int parity, const int* cells, int ncells, double* out,
                              float inv, int* flags, hipStream_t st);
hipError_t launch_macroscopic(int storage, const BoxDev& bx, int parity, double* rho, double* u, float inv,
                              hipStream_t st);
hipError_t launch_map_dense(const BoxDev& bx, const Particles& P, const int* tile_cnt, const int* tile_off,
                            const int2* tile_ent, int list_cap, TileShape ts, double* B, int* pid,
                            unsigned long long* dropped, hipStream_t st);
int stats_blocks();
hipError_t launch_stats(int storage, const BoxDev& bx, int parity, float inv, double* part, double* out,
                        hipStream_t st);
hipError_t launch_stream_copy(const void* src, void* dst, size_t bytes, hipStream_t st);
// Bits of the device error word of a context, set by kernels and read and
// cleared by the host at its next synchronising call.
enum {
    FLAG_LIST_CUT = 2,        // a step ran on a tile list that holds fewer spheres than reach the tile
    FLAG_SLOT_OVERFLOW = 4,   // a step met a cell overlapped by more than two spheres
    FLAG_BAD_CELL = 8         // psm_get_pdfs_at was given a cell index outside the box
};
// Two words follow the error word, one per list parity: the largest uncapped
// count of the lists of that parity where a tile lists more than MAXC spheres
// (lists that no step has used may still be replaced without harm).
constexpr int ERR_WORDS = 3;
hipError_t launch_fill_int(int* a, long long n, int v, hipStream_t st);
// FP64 mass and momentum of a canonical field [19][N] into out[4] (device),
// with the partial sums in the library's static per-GPU array
long long noalloc_max_cells();
hipError_t launch_field_stats_noalloc(const double* f, long long N, double* out, hipStream_t st);

}  // namespace psm
