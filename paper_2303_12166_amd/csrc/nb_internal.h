// nb_internal.h -- device-side data structures shared by the HIP kernels and the C++ runtime of
// libnbody. Not part of the public ABI (include/nbody.h is).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace nbk {

// Waves per SIMD asked of the compiler (its vector-register cap) for the force kernels: the most
// at which the pair loops do not spill (eqs. (4)-(6) at two rows and four waves: 13.9 ms at
// 262,144 elements against 12.8 at three; the contact law at two rows 10.1-10.2 ms at four waves,
// 10.25-10.34 at three).
constexpr int PLAIN_WAVES = 4;
constexpr int rows_waves(bool fp64, int law, int r)
{
    return fp64 ? (law == 0 ? 3 : 2) : (law == 0 ? (r == 1 ? 5 : 4) : (r == 1 ? 4 : 3));
}

constexpr int CU_COUNT = 256;    // compute units of the card
constexpr int BT = 256;          // threads per block, every kernel
constexpr int TJ = 256;          // j elements staged in LDS per tile (one per thread)
constexpr int MAX_BAND = 4;      // tallest band of the FP32 symmetric kernel (tile rows per lane)
constexpr int RED_STRIDE = 16;   // doubles per O(N)-unit partial record of the read-backs
constexpr int REC_STRIDE = 8;    // doubles per record of a step (position sums, non-finite count)
constexpr int COM_FUSE_UNITS = 256;  // largest system (in units of 256 elements) whose records
                                     // every workgroup of k_advance sums for itself
// Most i elements per workgroup of the one-sided force kernel. Under eqs. (4)-(6) eight would need 144
// registers (velocities are held too): three workgroups on a CU instead of four.
constexpr int os_ib(bool fp64, int law) { return fp64 ? 4 : (law == 0 ? 8 : 7); }
constexpr int KERNEL_CLASSES = 4;    // force kernels of a launch: one-sided, bands of 1, 2, 4 rows
constexpr int ADV_INIT = 2;      // k_advance: record the sides at creation
constexpr int RED_DIAG = 0;      // record slots [0, 10): diagnostics sums
constexpr int RED_RET = 10;      // record slots [10, 15): retention sums
constexpr int SORT_TILE = 2048;  // elements per workgroup of a pass of the order's sort
constexpr int SORT_BOUNDS = 64;  // most workgroups that find the stars' bounding boxes
constexpr size_t sort_work_bytes(int64_t n)
{
    return 12 * SORT_BOUNDS * sizeof(double) +
           256 * sizeof(uint32_t) * (1 + (size_t)((n + SORT_TILE - 1) / SORT_TILE));
}
constexpr int L1_LOG_CAP = 4096; // rows of the per-step L1 log
// Position of padding slots in the sorted layout. A padding element at 1e18 (FP32) or 1e150
// (FP64) gives w^3 below the type's smallest subnormal, so its contribution is exactly 0.
constexpr float SENTINEL_F32 = 1.0e18f;
constexpr double SENTINEL_F64 = 1.0e150;
constexpr float FAR_MARGIN = 2.0e-5f;  // relative margin on D^2 for the far-tile test

// Squared gap in FP32 from which two boxes are far for the diameter D. Positions and diameters may be
// in any unit: where D^2 leaves the range in which FP32 squares keep that margin, no gap is far.
__host__ __device__ inline float far_limit(double D)
{
    const double d2 = D * D * (1.0 + (double)FAR_MARGIN);
    return d2 > 1.0e-30 && d2 < 1.0e38 ? (float)d2 : INFINITY;
}

// Pair classes: 0 = star 1 with star 1, 1 = across the stars, 2 = star 2 with star 2.

// What the donor growth changes: the donor's element diameter and the force constants that follow.
struct LawState {
    double D2;               // FP64 master
    double c1d[3], c2d[3];   // 11 / D^3 and 10 / D^2 per pair class
    float c1f[3], c2f[3];    // FP32 copies used by the FP32 kernels
    float far2f[3];          // far_limit(D) per pair class
    float lD_f[3];           // D per pair class
    int32_t growth_stopped, pad;
};

// Per-system state that lives in device memory (first bytes of the system's workspace).
struct alignas(16) DevState {
    // FP64 masters
    double D1, D2_0, R2_0, rL_a, growth_rate;
    double G, m, dt, xi_l1;
    double gm_d, h_d;        // G m and dt / 2
    // L1 plane of the current step
    double com1[3], com2[3], e[3], xi_cut;
    float gm_f, h_f, dt_f, pad_f;
    LawState cur;            // after the last completed call
    LawState slot[2];        // within a call, one-sided systems: before odd and before even steps
    int64_t step;
    int64_t step_done;       // within a call, one-sided systems: `step` after the step in progress
    int32_t growth_on, nonfinite;
    int32_t n_past, fwd, bwd;
    int32_t plane_ok, law, pad_s;
    // element law of eqs. (4)-(6), with the overlap volume written as (pi / 12) (D - r)^2
    // (r + 2D), D = 2R the pair's element diameter: gc = gamma pi / (12 G m^2) and
    // gcb = beta gc scale it for converging and separating pairs; eps softens the attraction
    double gamma, beta, leps_d, lgc_d, lgcb_d;
    float leps_f, lgc_f, lgcb_f, pad_l;
    // accretor-side retention (nb_retention): star 1's mean velocity and the two counts
    double v1[3];
    int32_t ret_past, ret_bound;
};

struct DiagOut {
    double v[16];  // com[3], P[3], L[3], KE, PE
};

// One entry of a launch's segment table.
//
// The force kernels work on a sorted copy of the positions: each star's elements in Morton
// order of their initial positions, star 1 in slots [0, n1), star 2 from slot p1 =
// roundup(n1, TJ), both padded with sentinels to a multiple of TJ (npad slots in all, nalloc
// allocated). Every j tile then lies inside one star, and each tile's bounding box lets the
// kernel skip the contact test for tiles that are provably farther than D.
struct SysDesc {
    void *x, *y, *z, *vx, *vy, *vz, *ax, *ay, *az;
    int8_t *side;
    DevState *st;
    void *xs, *ys, *zs;   // sorted positions, nalloc slots
    int32_t *perm;        // nalloc: element index of each sorted slot, -1 for padding
    float *tbox;          // ntiles * 8: min xyz, pad, max xyz, pad of each j tile
    void *part;         // chunk partial sums, nsplit * 3 * nalloc values (symmetric kernels only)
    double *red;        // n_ounits * RED_STRIDE doubles
    double *rec;        // records of a step, rec_len * REC_STRIDE doubles (one-sided: twice, the
                        // second for odd steps of a call)
    void *alt;          // one-sided systems: positions and half-step velocities of three steps of a
                        // call, 3 * 6 * nalloc values
    double *pe_part;    // potential-energy partials, n_peunits doubles
    int32_t *l1_log;    // L1_LOG_CAP * 4 int32
    DiagOut *diag;
    int32_t n, n1;
    int32_t nsplit, jchunk;     // j chunks per i-block and chunk length (multiple of TJ)
    int32_t iblock, n_iblocks;  // i elements per block (BT * ki) and block count
    int32_t n_units, n_ounits;  // force units (n_iblocks * nsplit) and O(N) units (ceil(n / BT))
    int32_t n_rec, one_sided;   // records of a step; 1 for the one-sided force kernel, whose units
                                // are its workgroups
    int32_t rec_len, ib;        // at least n_rec and n_ounits (at creation there are n_ounits records)
    int32_t unit_begin, ounit_begin;  // prefix offsets in the launch's segment table
    int32_t n_peunits, pe_ch;         // potential energy: units (tile row, chunk), tiles per chunk
    int32_t npad, p1, nalloc, ntiles;  // sorted layout (see above)
    int32_t tunit_begin, pad2;         // prefix offset of this system's tiles in the launch
    // symmetric kernels (FP32 Kahan and FP64 modes): work units (band g, chunk c) and reaction
    // partials, per band g the tiles after its first row: 3 * TJ * sum_g (T - rows g - 1)
    int32_t *units;       // n_units pairs (g, c)
    float *react;         // (double * in the FP64 mode)
    int32_t ch, sym;      // tiles per chunk; 1 when the symmetric kernel is used
    void *vxs, *vys, *vzs;  // sorted velocities (eqs. 4-6 and the symmetric kernels' steps)
    void *as;               // sorted accelerations between a call's steps, 3 * nalloc (sym only; the
                            // contact law: chunk 0 of `part`)
    int32_t law, rows;    // element law; tile rows per band (1 in the FP64 mode)
};

// Kernel argument describing one launch over a segment table.
struct Launch {
    const SysDesc *sys;
    int32_t n_sys;
    int32_t unit_base;     // first force unit of this launch (a force launch may cover a range)
    int32_t total_units;   // force units: (i-block, j chunk) pairs; the launch ends before this
    int32_t total_ounits;  // O(N) units: 256 elements in element order
    int32_t total_tunits;  // tiles: 256 slots in sorted order
    int32_t law;           // element law of every system in the launch (NB_LAW_*)
    int32_t ounit_base;    // first O(N) unit of the systems outside the first class below
    int32_t any_big;       // a system has more than COM_FUSE_UNITS units
    int32_t any_empty;     // a system has no elements
    // the table is ordered by force kernel: one-sided (and empty) systems, then bands of 1, 2 and 4 rows (the
    // plain and FP64 kernels count as 1); they own the force units up to band_end[0] .. band_end[3]
    int32_t band_end[KERNEL_CLASSES];
};

// Segment-table entries written on the device from the systems' own one-entry tables (each
// system's SysDesc in its workspace), with this launch's prefix offsets: up to TABLE_CHUNK
// systems per kernel launch, passed by value as a kernel argument.
constexpr int TABLE_CHUNK = 64;
struct TableChunk {
    const SysDesc *src[TABLE_CHUNK];
    int32_t unit_begin[TABLE_CHUNK], ounit_begin[TABLE_CHUNK], tunit_begin[TABLE_CHUNK];
    int32_t first, count;  // entries [first, first + count) of the destination table
};

// Host-side launchers (nb_kernels.hip). All return the HIP status of the launch.
hipError_t launch_init_state(DevState *st, const DevState &init, hipStream_t s);
hipError_t launch_reset_sorted(const SysDesc &d, int mode, hipStream_t s);
hipError_t launch_zero_velocities(const SysDesc &d, int mode, hipStream_t s);
hipError_t launch_sort(const SysDesc &d, int mode, void *work, hipStream_t s);
hipError_t launch_gather(const Launch &L, int mode, hipStream_t s);
hipError_t launch_forces(const Launch &L, int mode, int step, int last, int max_blocks,
                         hipStream_t s);
hipError_t launch_combine(const Launch &L, int mode, int kick, int last, hipStream_t s);
hipError_t launch_kick_stats(const Launch &L, int mode, int do_kick, hipStream_t s);
hipError_t launch_finalize_step(const Launch &L, int in_step, hipStream_t s);
hipError_t launch_advance(const Launch &L, int mode, int finish, int kick, int n_steps,
                          hipStream_t s);
hipError_t launch_diag(const Launch &L, int mode, int with_pe, int n_peunits, hipStream_t s);
hipError_t launch_retention(const Launch &L, int mode, hipStream_t s);
hipError_t launch_valu_probe(int op, float *sink, int blocks, int iters, hipStream_t s);
hipError_t launch_copy_table(SysDesc *dst, const TableChunk &c, hipStream_t s);

}  // namespace nbk
