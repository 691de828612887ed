// Internal definitions shared by the host runtime and the gfx950 kernels of
// libvpmc.  Nothing here is part of the public C ABI (include/vpmc.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace vpmc {

// ---------------------------------------------------------------- tables
// Per-material tables X(E) (Methods A): NE nodes log-spaced on [1, 256] MeV.
constexpr int NE = 256;
constexpr int NMAT = 5;
constexpr double E_LO = 1.0;
constexpr double E_HI = 256.0;
enum Material { MAT_WATER = 0, MAT_AIR = 1, MAT_PMMA = 2, MAT_BRASS = 3, MAT_BONE = 4 };

// FP32 device blob, high parts first.  Shared: segment energy widths
// E_i+1 - E_i, energy nodes, reciprocal widths.  Per material: R, reciprocal
// slopes, slopes dE/dR, R_i+1 - R_i, omega^2, T, Sigma_nuc; NE floats each, all
// per unit of density x path length in mm (10 x g/cm^2).  Tables per segment
// use NE - 1 entries; the last one is a sentinel for the table behind it, read
// at index -1 by the walks down the segments: -inf before the energy nodes, 0
// before the slopes, +inf before the range widths.  The reciprocals are
// computed on the device (derive_tables_kernel), by the instructions the step
// would use.  Then the low parts that make the node, width, slope and
// range-width tables (high, low) FP32 pairs of the FP64 values, for the
// double-float bookkeeping of the deterministic mode.  The materials of the
// patient come first, those of the beam line last: each kernel stages in LDS
// the shared tables and the materials it meets.
enum { TAB_DWH = 0, TAB_E = NE, TAB_RDW = 2 * NE, TAB_SHARED = 3 * NE, TAB_PER_MAT = 7 * NE };
enum { T_R = 0, T_RS = 1, T_SH = 2, T_DH = 3, T_W2 = 4, T_T = 5, T_SN = 6 };
enum { TABL_E = 0, TABL_DW = NE, TABL_SHARED = 2 * NE, TAB_PER_LMAT = 2 * NE };
enum { L_SL = 0, L_DL = 1 };
enum { DM_WATER = 0, DM_AIR = 1, DM_BONE = 2, DM_PMMA = 3, DM_BRASS = 4 };   // order of the materials in the blob
constexpr int kTabSlot[NMAT] = {DM_WATER, DM_AIR, DM_PMMA, DM_BRASS, DM_BONE};
constexpr int tab_hi_floats(int nm) { return TAB_SHARED + nm * TAB_PER_MAT; }
constexpr int tab_lo_floats(int nm) { return TABL_SHARED + nm * TAB_PER_LMAT; }
constexpr int TAB_HI_FLOATS = tab_hi_floats(NMAT);
constexpr int TAB_FLOATS = TAB_HI_FLOATS + tab_lo_floats(NMAT);

struct MaterialDef {
    double z_over_a, mean_exc_ev, rad_len_gcm2, nuc_coeff, density;
};
extern const MaterialDef kMaterials[NMAT];

// FP64 host tables (generated once per process)
struct HostTables {
    double E[NE];
    double R[NMAT][NE], W2[NMAT][NE], T[NMAT][NE], SN[NMAT][NE];
};
const HostTables &host_tables();
void pack_device_tables(float *blob /* TAB_FLOATS */);
double range_host(int m, double E);           // piecewise-linear CSDA range (g/cm^2)
double rs_thickness_mm(double wet_mm);        // PMMA slab thickness for a given WET

// model constants (readings of the paper's unstated physics)
constexpr float STEP_FRACTION = 0.25f;     // step <= 1/4 residual range
constexpr float NUC_F_LOCAL = 0.10f;       // nuclear event: share deposited locally
constexpr float NUC_F_ESCAPE = 0.30f;      // share carried off by neutral secondaries
constexpr float NUC_SIGMA_RAD = 0.15f;     // deflection of the leading secondary
constexpr float EDGE_PUSH_MM = 1e-4f;      // push across an aperture edge in the BEV plane (FP32)
constexpr int MAX_STEPS = 1000000;         // safety bound on steps per VP
constexpr int MAX_BLOCK_ITER = 10000;      // bound on crossing-number tests per block traversal
constexpr double kSdfMargin = 8.0;         // mm of aperture distance raster beyond the polygon's box
constexpr double kListRadius = 1.9;        // mm: edges listed per raster cell around its reference point
constexpr double MEV_TO_J = 1.602176634e-13;

enum { L_GRID = 0, L_RS = 1, L_BLOCK = 2, L_ESCAPED = 3, L_NUC = 4, NLEDGER = 6 };
enum { PH_STRAGGLE = 1, PH_MCS = 2, PH_NUCLEAR = 4 };

// ------------------------------------------------------- kernel arguments
struct GeomDev {
    int kind, nx, ny, nz;
    float sp[3], lo[3];
    const int16_t *hu;
    // density per voxel (CT geometry), the value the calibration gives in
    // physics mode; nx * ny entries before the first and behind the last voxel
    // are readable, so the next voxel's density is fetched before it is known
    // to be inside the grid
    const float *rho;
};

// Linear index of the voxel behind a face, stride (1, nx or nx * ny) from vox
// up or down.  Behind the grid's own faces it runs from -nx * ny to
// voxels + nx * ny - 1, for grids near the limit of 2^31 - 1 voxels more than 32
// signed bits hold.
__host__ __device__ inline int64_t voxel_behind(uint32_t vox, int stride, bool up) {
    return (int64_t)vox + (up ? stride : -stride);
}

struct FieldDev {
    float iso[3], ex[3], ey[3], ez[3];
    int has_block, nv;
    const float2 *poly;
    // signed distance raster of the polygon (+ inside the opening), cell size
    // 1/sdf_ih, for conservative bounds that skip the exact edge loops
    const float *sdf;
    float sdf_x0, sdf_y0, sdf_ih, sdf_r, sdf_far;
    int sdf_nx, sdf_ny;
    // per raster cell near the boundary: edge lists around a reference point
    // whose side is known, for exact tests on a handful of edges; valid for
    // BEV paths up to list_reach from the point.  cell: x the first entry in
    // cell_edge (bits 0-29), bit 30 a reference point exists, bit 31 it is
    // inside; y one past the last entry
    const uint2 *cell;
    const uint16_t *cell_edge;
    const float2 *cell_ref;
    float list_reach;
    float blk_zu, blk_zd, blk_rho, blk_t, blk_tl;
    int has_rs;
    float rs_zu, rs_zd, rs_r2, rs_rho, rs_rhol, rs_t, rs_tl;   // *_l: low parts of the FP64 values
    // virtual source vsad upstream of the origin plane (0: parallel beam);
    // divergent block (div): the opening at block depth pz is the polygon
    // scaled by pz * fs + fc0 (walls through the focus)
    float vsad;
    int div;
    float fs, fc0;
};

// Distance raster and edge lists of an aperture polygon while they are made.
struct Raster {
    double x0, y0, h;
    int nx, ny;
    const float2 *poly;
    int nv;
    double radius;                // edges listed around a cell's reference point
    float *d;                     // [nx * ny] signed distance of the cell centres
    uint2 *cell;                  // [nx * ny]
    float2 *ref;                  // [nx * ny]
    uint16_t *edge;
    unsigned long long *count;    // [0] listed edges in all, [1] those placed so far
};
hipError_t launch_raster(const Raster &r, hipStream_t s);         // distances, reference points, counts
hipError_t launch_raster_lists(const Raster &r, hipStream_t s);   // the lists

struct SpotDev {
    float x, y, e0, sigma, esig, emax, scale;   // scale = w/N * 2^k
    uint32_t nh;
};

// VP deferred at the block entry for the surrogate: its whole state on the
// block's upstream face (E + Elo is the compensated energy, pzlo the low part
// of the depth), so the plain transport can resume it unchanged
struct DeferRec {
    uint32_t spot, hist, nblk, tag;   // tag: the row within the epoch (influence-matrix runs)
    float x, y, u, v, w, E, Elo, pzlo, d_edge, thick, pad[2];
};
static_assert(sizeof(DeferRec) == 64, "DeferRec is 64 bytes");

struct SurDev {
    int enabled;
    float d_fallback;                 // VPs nearer the opening's edge stay on the plain transport
    unsigned long long *count;        // records written (may exceed capacity: the rest ran plain)
    unsigned long long capacity;
    DeferRec *rec;
};

struct LaunchDev {
    const SpotDev *spots;
    const unsigned long long *item_off;   // [n_spots + 1] prefix of items per spot
    int n_spots;
    unsigned long long n_items;
    int batch, n_batches;
    uint32_t key0, key1;
    unsigned physics;
    float shift[3];
    float range_scale;
    unsigned long long *tally;            // int64 fixed point, two's complement
    unsigned long long *let_tally;        // dose-averaged LET numerator (same layout) or null
    unsigned long long *ledger;           // [NLEDGER]
    unsigned long long *stats;            // [2]: steps, histories
    const float *tables;                  // TAB_FLOATS
    SurDev sur;
};

constexpr int POLY_LDS = 1024;  // == VPMC_MAX_VERTICES
constexpr int kLetShift = 8;    // LET numerator scale 2^(k - 8): LET <= 256 keV/um keeps it within the dose bound

// ------------------------------------------- influence-matrix (CSR) mode
// One row = (scenario, field, spot).  Rows are processed in epochs of at
// most kMaxSlots rows; row (row_begin + i) of an epoch owns slot i: a dense
// int64 grid plus one byte per block of 32 voxels that is set when the block
// receives a deposit.  Compaction counts and emits per chunk of 256 blocks.
constexpr int kMaxSlots = 1024;

struct RowDev {
    int field;            // index into the field table of the launch
    uint32_t field_id;    // caller's field id (part of the Philox key)
    uint32_t spot;        // spot index within its field (Philox counter)
    uint32_t spot_global; // index into the flattened spot table
    int scen;
    uint32_t n_hist;
    // dense runs: a row is a range of a batch's items in one scenario
    uint32_t batch, dest;           // batch, and the tally its deposits go to
    unsigned long long item0;       // first item of the batch's items
    int tlo[3], tn[3];    // LDS tile box of the row in voxel indices (tn = 0: none; tile_box_kernel)
};

struct ScenDev {
    float shift[3];
    float range_scale;
};

// Per row of the run: particles staged by the beam line and records drawn by
// the patient loop (a row's part of one round, at most kMaxStage records).
struct RowCtl {
    unsigned int staged, next;
};

// An epoch's histories are transported in rounds: as many groups of 64
// histories (of one row each) as the staging buffer holds, normally all.
struct QueueDev {
    const RowDev *rows;
    const unsigned long long *grp_off;    // [rows of the run + 1] prefix of the rows' groups
    unsigned long long g_begin, g_end;    // groups of this round
    int row_begin, n_rows;                // rows of this round (of the epoch in the compaction passes)
    uint32_t slot0;                       // slot of the round's first row (grid and mark start there)
    unsigned long long *head;             // fresh-row counter of this round
    RowCtl *ctl;                          // [rows of the run]
    int tile_cap;                         // 32-bit entries of the workgroup's LDS tile (< 2^16)
    int hist_per_lane;                    // one draw = 64 * hist_per_lane staged records
    int beam_groups;                      // consecutive groups a wave of the beam line takes at a time
    int refill_min;                       // idle lanes that trigger a refill in the patient loop
    float *stage;                         // [64 * (g_end - g_begin)] staged VPs (64 B)
    // dense runs: items of batch b = histories of all spots in spot_order, spot
    // spot_order[s] from item_off[b * (n_spots + 1) + s] on
    int dense, n_spots, n_batches;
    const unsigned long long *item_off;
    const uint32_t *spot_order;
    int let;                              // dense grids hold (dose, LET numerator) pairs
    const FieldDev *fields;
    const int *poly_off;                  // per field: offset into polys
    const float2 *polys;
    int n_poly_total;
    const SpotDev *spots;
    const ScenDev *scen;
    uint32_t key0, seed_hi;
    unsigned physics;
    int div;                              // some field is divergent (virtual source or divergent block)
    unsigned long long *grid;             // [slots][gstride] int64 tallies
    uint8_t *mark;                        // [slots][mstride] touched-block bytes (32 voxels each)
    size_t nvox, nblk, nchunk;            // blocks = ceil(nvox/32), chunks = ceil(blocks/256)
    size_t gstride, mstride;              // gstride = 32 * nblk voxels, mstride >= nblk bytes
    unsigned long long *ledger;           // [n_scen][NLEDGER]
    unsigned long long *stats;            // [2]
    const float *tables;
    SurDev sur;                           // surrogate queue (enabled = 0: off)
    unsigned long long iter_cap;          // quarters of work-queue iterations a wavefront may make
    uint32_t draw_cost;                   // those of a draw (4, or 1 of the default size)
    unsigned int *flags;                  // bit 2 (value 4) set when a wavefront reached iter_cap
};
constexpr unsigned long long kDefaultQueueCap = 1ull << 40;   // far above any run's chunk count
constexpr unsigned int kFlagAborted = 4u;

// staging records of a round: all histories of an epoch up to kMaxStage
// (2 GiB of 64 B records: a head epoch of 1000 rows x 2e4 histories fits); with
// a cap on device memory what queue_stage_min gives, one refill of every wave
constexpr size_t kStageFields = 16;
constexpr int kStageHpl = 32;
constexpr unsigned long long kMaxStage = 1ull << 25;
constexpr int kBeamGroups = 16;  // consecutive groups a wave of the beam line takes at a time, at most
constexpr uint32_t kLeaveIdle = 32;   // idle lanes at which a wave of an exhausted row leaves the tile
constexpr int kRefillMin = 8;    // idle lanes that trigger a refill of the patient loop
inline unsigned long long queue_stage_min(int blocks, int threads, int hist_per_lane) {
    const int hps = hist_per_lane < kStageHpl ? hist_per_lane : kStageHpl;
    return (unsigned long long)blocks * (unsigned long long)((threads + 63) / 64) * 64ull * (unsigned long long)hps;
}
hipError_t launch_derive_tables(float *blob, hipStream_t s);
hipError_t launch_density(const int16_t *hu, float *rho, size_t margin, size_t n, hipStream_t s);
hipError_t launch_tile_box(const GeomDev &g, const QueueDev &Q, RowDev *rows, hipStream_t s);
hipError_t launch_beam(const GeomDev &g, QueueDev Q, int cus, hipStream_t s);
hipError_t launch_queue(const GeomDev &g, const QueueDev &Q, int blocks, int threads, hipStream_t s);
size_t queue_static_lds(unsigned physics);
// workgroup size the queue kernel runs with for a requested size, and the
// LDS tile entries that leave the CU its full wave occupancy
int queue_threads(unsigned physics, int threads);
int queue_tile_cap(unsigned physics, int threads);

// ------------------------------------------------------- aperture surrogate
// MLP 8 -> 256 -> 256 -> 256 -> 256 -> 29, parameters layer by layer as
// W[out][in] then b[out] (FP32 master, BF16 copy in the same layout).
constexpr int MLP_LAYERS = 5;
constexpr int MLP_IN = 8;
constexpr int MLP_OUT = 29;
constexpr int MLP_HIDDEN = 256;
constexpr int kMlpSplit = 16;    // K split of the weight-gradient products
constexpr int MLP_MAX_BATCH = 16384;
constexpr unsigned long long kSurMaxRecords = 1ull << 22;   // surrogate queue (64 B each)

// One training (or gradient) step's operands; *f are MFMA fragments.
struct MlpStep {
    const float *x, *y, *t;   // samples: [][8] inputs, [][3] targets, [] outcome
    const int *idx;           // which of them (NULL: 0 .. n-1)
    int n, np;                // samples, parameters
    float inv_n;
    float *w, *m, *v;         // FP32 master parameters, Adam moments
    __bf16 *wb, *fwd, *bwd;   // BF16 parameters, as fragments of both directions
    __bf16 *xf, *hf[4];       // inputs and hidden activations
    __bf16 *dof, *df[4];      // d loss / d outputs and pre-activations
    float *dout;              // [29][n] d loss / d outputs (batch mean)
    float *bpart[4];          // [(n + 31) / 32][256] 32-sample sums of d loss / d pre-activations
    float *part;              // [kMlpSplit][np] partial weight gradients
    float *loss;              // [n] per-sample loss
    double *loss_acc;         // += the batch-mean loss
    float *grad;              // the gradient instead of an update (or NULL)
};

hipError_t launch_sur_resume(const GeomDev &g, const FieldDev &f, const LaunchDev &L, const DeferRec *rec,
                             const float *out, unsigned long long n, float p_lo, float p_hi, hipStream_t s);
hipError_t launch_sur_resume_csr(const GeomDev &g, const QueueDev &Q, const DeferRec *rec, const float *out,
                                 unsigned long long n, float p_lo, float p_hi, hipStream_t s);
hipError_t launch_surrogate_sample(const FieldDev &f, const float *entries, int n, uint32_t key0, uint32_t key1,
                                   unsigned physics, const float *tables, float *x, float *y, float *t, hipStream_t s);
int mlp_param_count();
size_t mlp_frag_bytes();   // both directions' weight fragments, the forward ones' share first
constexpr int MLP_FWD_ELEMS = (8 + 3 * 128 + 16) * 512;
// fused inference of n samples: inputs x [n][8] FP32, or (rec != NULL) the
// features of deferred-VP records; outputs out [n][29] FP32
hipError_t mlp_infer(const float *x, const DeferRec *rec, int n, const __bf16 *wb, const float *wf, float *out,
                     hipStream_t s);
// S.fwd, S.bwd from S.wb; forward, loss, backward and update (or gradient) of
// S.n samples
hipError_t mlp_pack(const MlpStep &S, hipStream_t s);
hipError_t mlp_step(const MlpStep &S, float lr, int step, hipStream_t s);
hipError_t mlp_to_bf16(const float *x, __bf16 *y, size_t n, hipStream_t s);
hipError_t launch_csr_count(const QueueDev &Q, unsigned int *cnt, hipStream_t s);
hipError_t launch_csr_chunk_scan(const unsigned int *cnt, unsigned int *coff, unsigned int *rowcnt, int n_rows,
                                 size_t nchunk, hipStream_t s);
hipError_t launch_csr_offsets(const unsigned int *nnz, int n_rows, int row_begin, unsigned long long *row_off,
                              unsigned long long *row_nnz, unsigned long long *used, unsigned long long capacity,
                              unsigned int *flags, hipStream_t s);
hipError_t launch_csr_emit(const QueueDev &Q, const unsigned int *cnt, const unsigned int *coff,
                           const unsigned long long *row_off, const unsigned long long *row_nnz, int32_t *col,
                           long long *qv, unsigned long long capacity, unsigned int *flags, hipStream_t s);
hipError_t launch_fill_u64(unsigned long long *p, size_t n, unsigned long long v, hipStream_t s);
hipError_t launch_atomic_rate(unsigned long long *grid, int nx, int ny, int nz, unsigned long long n_tracks, int len,
                              float sigma, uint32_t seed, hipStream_t s);
hipError_t launch_csr_scatter(const int32_t *col, const long long *qv, unsigned long long begin,
                              unsigned long long end, unsigned long long *dense, hipStream_t s);
hipError_t launch_csr_export(const int32_t *col, const long long *qv, size_t n, const GeomDev &g, double mev_scale,
                             int32_t *ocol, float *val, long long *oq, hipStream_t s);
// dynamic voxel spacing: merge influence-matrix rows into cells (runs of
// consecutive voxels of a non-decreasing voxel -> cell map), a wavefront per
// piece of at most kCellPiece entries of one row
constexpr int kCellPiece = 4096;
struct CellPiece {
    long long begin;   // first entry (CSR index)
    int len;
    int row;
};
hipError_t launch_cell_map(const int32_t *cmap, int nvox, int n_cells, int32_t *cstart, unsigned *st, hipStream_t s);
hipError_t launch_cell_mass(const GeomDev &g, const int32_t *cstart, int n_cells, double *mass, hipStream_t s);
hipError_t launch_cell_count(const long long *rp, const CellPiece *pcs, long long n_pieces, const int32_t *col,
                             const int32_t *cmap, int nvox, unsigned long long *cnt, unsigned *err, hipStream_t s);
hipError_t launch_cell_rows(const long long *first_piece, const long long *pout, size_t n, long long *rp_out,
                            hipStream_t s);
hipError_t launch_cell_emit(const long long *rp, const CellPiece *pcs, long long n_pieces, const int32_t *col,
                            const long long *q, const int32_t *cmap, const long long *pout, const double *mass,
                            double mev_scale, int32_t *ocell, long long *oq, float *oval, hipStream_t s);

// ------------------------------------------------- spot-weight optimiser
// Voxels per forward workgroup (int64 LDS sums): 2^bits.  Over the structure
// voxels of the iterations the largest of 2^5 .. 2^11 that leaves kOptLists
// lists (three workgroups a CU) of at most kOptListLen entries on average: more
// lists sum too few entries each (2^9 voxels of the whole grid per list: 12 500
// lists of 590 entries, 46 us a sweep; 2^11 structure voxels: 1000 of 7300, 19
// us), fewer leave CUs idle, and long ones want several a CU to even out
// (1040 lists of 95 600: 203 us, 2080 of 47 800: 169).  The sweep of whole rows
// for the dose output takes kOptChunkBits.
constexpr int kOptChunkBits = 9, kOptMinBits = 5, kOptMaxBits = 11;
constexpr long long kOptLists = 768, kOptListLen = 65536;
enum { kOptPowerInit, kOptPower, kOptPowerNorm, kOptFistaInit, kOptFista, kOptFinalPrep, kOptFinal };
enum { kOptLam = 0, kOptL = 1 };   // device scalars

// Entries per gradient wavefront: the largest of 256 .. 1024 that leaves
// kOptWaves wavefronts.  Long pieces are chains of loads (4096 entries: 29 us for
// 7.3 M, 1024: 20, 512: 18; 38 000 entries: 5.6 us at 1024, 4.2 at 256), short
// ones more partials for the update to add.
constexpr int kOptMinPiece = 256, kOptMaxPiece = 1024;
constexpr long long kOptWaves = 8192;
constexpr int kRoiParts = 8;       // wavefronts of a row in the passes that restrict the rows
constexpr int kOptParts = 512;     // workgroups of the update at most

// 64 voxels: which have a structure bit, and the structure voxels before them
struct OptMask {
    unsigned long long bits;
    uint32_t before, pad;
};

// consecutive entries of one row
struct OptPiece {
    long long begin;   // first entry (CSR index)
    int len;
    int row;           // compact row s * n_spots + j
};

// a list of the forward sweep: scenario * chunks + chunk, its entries
struct OptWork {
    long long begin, len;
    uint32_t list;
};

struct OptDev {
    const long long *row_ptr;       // CSR row pointer, row of (s, j) = s*row_stride + row_offset + j
    const int32_t *col;             // voxel indices per row
    const float *val;               // Gy per unit spot weight
    const uint8_t *roi;             // [nvox] bit 0 target, bit 1 organ at risk
    int n_scen, n_spots, row_stride, row_offset;
    int nvox, nchunks, bits;        // voxels (of the iterations: structure voxels), chunks of 2^bits
    double d_presc, w_target, d_max, w_oar;
    // chunk-bucketed copy of the entries by list (s, chunk): key = spot << bits | voxel - chunk base
    const uint32_t *bkey;
    const float *bval;
    const OptWork *work;            // [n_work] lists to sweep, in decreasing entry count
    long long n_work;
    const OptPiece *piece;          // gradient pieces, row-major
    long long n_pieces;
    const long long *piece_off;     // [n_scen * n_spots + 1] first piece of each compact row
    float *amax;                    // [n_scen * n_spots] largest |a| of each row
    const OptPiece *units;          // row pieces of the index passes (NULL: whole rows)
    long long n_units;
    float *rstruct;                 // [n_scen][nvox] residual of the last forward sweep (or NULL)
    double *fpart;                  // [n_work] objective partials
    double *gpart;                  // [n_pieces] piece products with the residual
    double *x, *y, *z, *gvec;       // [n_spots]
    int n_part;                     // workgroups of the update (without the objective's)
    double *bpart;                  // [n_scen][n_part] their parts of the next sweep's bounds
    double *sq;                     // [2][n_part] and of |g|^2, |z|^2
    double *scal;                   // device scalars (kOptLam, kOptL)
};

hipError_t opt_build_count(const OptDev &O, unsigned long long *cnt, unsigned *err, hipStream_t st);
hipError_t opt_structures(const uint8_t *roi, int nvox, OptMask *mask, unsigned long long *cnt,
                          unsigned long long *off, uint8_t *keep, uint8_t *sroi, hipStream_t st);
hipError_t opt_roi_same(const uint8_t *a, const uint8_t *b, int nvox, unsigned *err, hipStream_t st);
hipError_t opt_roi_count(const OptDev &O, const OptMask *mask, unsigned *rcnt, unsigned *err, hipStream_t st);
hipError_t opt_roi_copy(const OptDev &O, const OptMask *mask, const unsigned *rcnt, const long long *rptr,
                        int32_t *ccol, float *cval, hipStream_t st);
hipError_t opt_build_scan(unsigned long long *cnt, unsigned long long *off, size_t n, hipStream_t st);
hipError_t opt_build_emit(const OptDev &O, const unsigned long long *off, unsigned long long *cur, uint32_t *bkey,
                          float *bval, hipStream_t st);
hipError_t opt_forward(const OptDev &O, const double *w, int mode, float *dose_out, hipStream_t st);
hipError_t opt_gradient(const OptDev &O, hipStream_t st);
hipError_t opt_update(const OptDev &O, int mode, double beta, int it, double *hist, hipStream_t st);

// launchers (vpmc_kernels.hip)
hipError_t launch_transport(const GeomDev &g, const FieldDev &f, const LaunchDev &L, int blocks,
                            int threads, hipStream_t s);
hipError_t launch_fold_batch(unsigned long long *q_batch, int nb, long long *q_total, double *s2, long long *let, size_t n,
                             hipStream_t s);
hipError_t launch_fold_dose(unsigned long long *q_batch, int n_batches, long long *q_total, long long *let, const GeomDev &g,
                            double mev_scale, float *dose, float *sigma, size_t n, hipStream_t s);
hipError_t launch_dose(const long long *q, const double *s2, int n_batches, const GeomDev &g,
                       double mev_scale, float *dose, float *sigma, size_t n, hipStream_t s);

// Static device scratch of the allocation-free dense run
// (vpmc_run_spots_noalloc): a file-scope __device__ array in
// vpmc_kernels.hip, one copy per GPU, held until the process ends.
constexpr size_t kScratchBytes = (size_t)32 << 20;
constexpr int kMaxScratchDevices = 64;
// Device address of the scratch on `device`, which must be the current
// device: looked up once per device with hipGetSymbolAddress and kept.
hipError_t scratch_device_ptr(int device, void **out);

}  // namespace vpmc
