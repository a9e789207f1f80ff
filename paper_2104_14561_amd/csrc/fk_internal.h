// fk_internal.h -- device-side plan records and kernel launchers shared by the
// host runtime (fk_host.cpp) and the gfx950 kernels (fk_device.h, instantiated
// by fk_launch.hip and fk_node_inst.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

namespace fk {

constexpr int kMaxDim = 3;
constexpr int kTimeFactors = 4;   // per (step, instance) time table entries
constexpr int kThetaSlots = 8;    // gradient entries per instance (FK_MAX_THETA)
constexpr int kBoxClasses = 5;    // separable-form footprint classes

constexpr int kTileClasses = 3;   // classes of the per-point transposed step's tiles
constexpr int kAdjLdsMax = 159 * 1024;   // dynamic LDS of a transposed step, of a CU's 160 KB
constexpr int kTileLdsMax = 60 * 1024;   // of a per-point transposed step's tile

// The one-launch step of small 2D plans: lanes per node, and the patch of 256 /
// lanes nodes that a workgroup takes (rows x columns, at most kSmallPatch each).
constexpr int small_lanes(int qs) { return qs <= 2 ? 2 : (qs <= 4 ? 4 : 8); }
constexpr int kSmallPatch = 16;
inline void small_patch(int qs, int *rows, int *cols)
{
    const int n = 256 / small_lanes(qs);   // 32, 64 or 128 nodes
    *rows = n == 32 ? 4 : 8;
    *cols = n == 128 ? 16 : 8;
}
constexpr int kSmallCells = 1024;   // records of a patch and its reach at most

// Longest footprint (nodes per axis) of a class of the separable form, and the
// threads of a workgroup that takes its 256-node work items.  Forward: 128 for
// the wide classes in FP64 (3D: from 9 nodes on in FP32 too), so that their LDS
// columns leave room for more than one workgroup per CU.  Transposed: 256 share
// a tile, except in 3D in FP64 from 9 nodes on, whose columns would not fit
// beside it.
inline int box_len(int d, int c)
{
    constexpr int l2[kBoxClasses] = {6, 9, 12, 15, 0}, l3[kBoxClasses] = {3, 4, 6, 9, 12};
    return d == 2 ? l2[c] : l3[c];
}
// Nodes that the separable kernels of class length L read along axis a from a
// footprint's first node: the instance's own footprint on the axes they loop
// over, the unrolled length on the others (in 2D axis 1, read in threes up to 6;
// in 3D axis 2, and every axis up to 4).  The columns past the footprint carry no
// weight, but their records must exist.
inline int sep_reads(int d, int L, int a, const int *sep_l)
{
    const int own = sep_l[a] < L ? sep_l[a] : L;
    if (d == 2) return a == 0 ? own : (L > 6 || own > 3 ? L : 3);
    return L <= 4 || a == 2 ? L : own;
}
constexpr int adj_threads(int d, int L, bool f32)
{
    return d == 3 && L > 6 && !f32 ? 128 : 256;
}
constexpr int box_threads(int d, int L, bool f32)
{
    return d == 2 ? (L > 6 && !f32 ? 128 : 256) : (L > 6 || (L > 4 && !f32) ? 128 : 256);
}

// Per-instance record read by every kernel (one per instance of a plan).
struct DevInst {
    int d;
    int n[kMaxDim];
    int periodic[kMaxDim];
    int uniform[kMaxDim];          // nearly equal spacing: guess the cell arithmetically
    int affine[kMaxDim];           // x_k == k * step + lo exactly (k < n-1), x_{n-1} == hi
    int coef_kind;
    int region_kind;
    int n_act;
    int pad0;
    long long stride[kMaxDim];     // node strides inside the instance
    long long node_off;            // offset of the instance in a packed field
    long long coord_off[kMaxDim];  // offsets of the axes in the coordinate array
    long long act_off;             // offset in the packed active list
    double lo[kMaxDim], hi[kMaxDim], inv_h[kMaxDim], period[kMaxDim], step[kMaxDim];
    double coef[16];
    double D;
    double center[kMaxDim];
    double r2;
    double S;       // sqrt(2 D) * sqrt(2 dt)
    double dSdD;    // S / (2 D)  (adjoint)
    // assembled (ELL) form: this instance's row box, width (box nodes x
    // (d + 1) fields), box nodes per field padded to whole 16-byte blocks,
    // and storage offset
    int ell_box[kMaxDim];
    int ell_w;
    int ell_nbp;
    long long ell_off;
    // offset of the instance in the caller's fields: node_off, except in the
    // FP64 sub-plan of an FP32 plan, whose inputs and outputs use the
    // parent's layout
    long long out_off;
    int face[kMaxDim][2];          // FK_FACE_* per axis and side
    int sdiff;                     // diffusion depends on the node (runaway model)
    int blo[kMaxDim];              // reachable box (the nodes a step's gathers can touch, with
    int blen[kMaxDim];             // or without weight): first node and length per axis (0
                                   // without active nodes)
    int sep_l[kMaxDim];            // footprint nodes per axis of one node's landing cells
    // axes that are not uniform: cell lookup by buckets of the smallest spacing,
    // lut_n entries of the coordinate array from lut_off (0 entries: bisection)
    long long lut_off[kMaxDim];
    double lut_inv[kMaxDim];
    int lut_n[kMaxDim];
    int pad1;
};

// A contiguous chunk of one instance's nodes (slope pass) or active nodes
// (step pass) handled by one workgroup.  kind 0: nodes first .. first+count-1;
// kind 1 + a: entries of the trig table of axis a.
constexpr int kEllClasses = 8;   // ELL assembly width classes

struct WorkItem {
    int inst;
    int first;
    int count;
    int kind;
};

// LDS tile of an adjoint work item: node box lo[a] .. lo[a] + ext[a] - 1.
struct TileBox {
    int lo[kMaxDim];
    int ext[kMaxDim];
    int use_lds;
    int pad;
    int soff;   // first entry of the tile's staging slot, or -1 (flush with atomics)
};

// The adjoint's work lists: active nodes handled per landing point (fw) and
// separable nodes by footprint class (box), each work item with its LDS tile.
struct AdjLists {
    const int *fw_nodes;
    const WorkItem *fw_work;
    const TileBox *fw_tiles;
    // by class of tile bytes, each launch's dynamic LDS its largest tile
    int fw_work_off[kTileClasses];
    int n_fw_work[kTileClasses];
    int fw_grid[kTileClasses];
    int fw_lds[kTileClasses];
    // tile staging: each tile's entries (fields interleaved) at its soff; per
    // node the staging entries (field 0) of the tiles that cover it
    void *stage;                // T, or null when the tiles flush with atomics
    int fresh;                  // every tile is staged: the gather stores mu, which need not be cleared
    int n_cov;                  // nodes covered by a staged tile
    const int *cov_node;        // [n_cov] packed node index
    const int *cov_ptr;         // [n_cov + 1] into cov_base
    const int *cov_base;        // staging index of field 0, per (node, covering tile)
    // separable nodes by footprint class (box_len), each launch's dynamic LDS
    // the largest of its work items'
    const int *box_nodes;
    const WorkItem *box_work;
    const TileBox *box_tiles;
    int box_work_off[kBoxClasses];
    int n_box_work[kBoxClasses];
    int box_grid[kBoxClasses];
    int box_lds[kBoxClasses];
};

// Pointers into the workspace that every launch needs.
struct PlanDev {
    const DevInst *inst;
    const double *coords;       // packed node coordinates of all axes
    const int *active;          // node index inside its instance, per active node
    const unsigned char *chi;   // terminal values (0/1) per packed node
    const double *gh_a;         // 1D GH nodes (Q*)
    const double *gh_w;         // tensor weights (Q), double
    const float *gh_wf;         // tensor weights (Q), float
    const double *gh_w1;        // 1D weights (Q*), double
    const float *gh_w1f;        // 1D weights (Q*), float
    const double *tfac;         // [n_steps][n_inst][kTimeFactors]
    double2 *trig;              // per-axis (sin, cos) of the drift arguments at t_n
    const WorkItem *slope_work; // trig table items, then pieces of the reachable boxes
    const WorkItem *node_work;  // all nodes (adjoint passes)
    const WorkItem *act_work;   // step pass work list (block / G active nodes each)
    const WorkItem *row_work;   // row-per-thread work list (block active nodes each)
    int *flags;                 // bit 0: non-finite value produced
    int n_inst;
    int n_slope_work;
    int n_table_work;
    int n_node_work;
    int n_act_work;
    int n_row_work;
    int d;
    int qs;                     // Q*
    int n_quad;                 // Q
    int n_steps;
    int block;                  // threads per workgroup
    int group;                  // lanes per active node in the step passes
    int step_kind;              // 0: thread per node, 1: lane group, 2: split node
    // one-launch step of small 2D plans (n_small_work > 0), a tile of records
    // per work item (its pad and soff hold the patch's first row and column)
    const WorkItem *small_work;
    const TileBox *small_tiles;
    const int *small_nodes;
    int n_small_work;
    int small_lds;              // bytes of the largest tile
    int all_affine;             // every axis of every instance is affine
    int pt_groups;              // 2D landing points by lane groups, a thread per node if not
    int rel_ok;                 // all_affine, and no landing point more than one period away
    int hermite2;               // R2 interpolant: 2D twist field in the records' fourth entry,
                                // 3D twist fields in a second record per node (packed2)
    void *packed2;              // 3D R2: (t01, t02, t12, t012) per node, or null
    int faces;                  // face kinds other than exit-1, or node-dependent diffusion
    double *retab;              // runaway model: kReTab values per coordinate, or null
    int retab_step;             // its time factors depend on the step
    // 3D plans with faces or axes of any kind (box region): nodes in entry form
    const int *ent_nodes;
    const WorkItem *ent_work;
    int n_ent_work;
    int ent_grid;
    // forward step work: nodes handled per landing point (fw) and separable
    // nodes handled in box form, by box class
    const int *fw_nodes;
    const WorkItem *fw_work;
    int n_fw_work;
    int fw_grid;
    const WorkItem *fw_split_work;
    int n_fw_split_work;
    int fw_split_grid;
    const int *box_nodes;
    const WorkItem *box_work;
    int box_work_off[kBoxClasses];
    int n_box_work[kBoxClasses];
    int box_grid[kBoxClasses];
    AdjLists adj;               // adjoint step work
    const WorkItem *split_work; // chunks of block / pow2(Q*) active nodes
    int n_split_work;
    int split_grid;
    int slope_grid;             // workgroups of the slope pass
    int node_grid;              // workgroups of all-node passes
    int act_grid;               // workgroups of the step pass
    int row_grid;               // workgroups of row-per-thread passes
    double dt;
    double t0;
    long long n_nodes;
    long long n_active;
    // ELL form
    int ell_width;
    int ell_box[kMaxDim];
    int ell_grid;
    // assembly work by row-width class: the LDS row boxes of a launch are
    // sized by its class's widest row, not by the widest row of the plan
    const WorkItem *ell_work;
    const WorkItem *ell_sep_work;   // separable rows, assembled as outer products,
    int n_ell_sep_cls;              // by class of the longest box axis
    int ell_sep_off[kEllClasses];
    int ell_sep_n[kEllClasses];
    int ell_sep_l[kEllClasses];     // longest box axis in the class (LDS vectors)
    int ell_sep_tb[kEllClasses];    // bytes of the class's largest block table
    int ell_sep_grid[kEllClasses];
    int n_ell_cls;
    int ell_cls_off[kEllClasses];
    int ell_cls_n[kEllClasses];
    int ell_cls_w[kEllClasses];
    int ell_cls_grid[kEllClasses];
};

// Kernel launchers (fk_launch.hip).  T is double or float; all return the
// HIP error of the launch.
hipError_t launch_init_field(const PlanDev &P, bool f32, void *u, hipStream_t s);
hipError_t launch_slopes(const PlanDev &P, bool f32, int n, const void *u, void *packed,
                         hipStream_t s);
// the slope pass of nc columns (fields ustride, records pstride elements apart),
// the tables of step n in place
hipError_t launch_slopes_mc(const PlanDev &P, bool f32, int n, const void *u, long long ustride,
                            void *packed, long long pstride, int nc, hipStream_t s);
hipError_t launch_tables(const PlanDev &P, int n, hipStream_t s);
// room of the static scratch beside FK_STATIC_SCRATCH_BYTES (lists of small and
// 3D entry-form plans: at most 64 bytes per node of up to 131 thousand)
constexpr size_t kScratchExtra = 8u << 20;
constexpr int kReTab = 8;   // runaway model: tabulated values per coordinate
// the runaway model's per-coordinate tables at step n (P.retab)
hipError_t launch_runaway_tables(const PlanDev &P, int n, hipStream_t s);
hipError_t launch_step_fused(const PlanDev &P, bool f32, int n, const void *packed,
                             void *u_out, hipStream_t s);
// The step of 3D plans in entry form (P.n_ent_work > 0).
hipError_t launch_step_ent3(const PlanDev &P, bool f32, int n, const void *packed, void *u_out,
                            hipStream_t s);
// The whole step u_in -> u_out of a small 2D plan (P.n_small_work > 0).
hipError_t launch_step_small2(const PlanDev &P, bool f32, int n, const void *u_in, void *u_out,
                              hipStream_t s);
bool step_node_compiled(int d, int qs);
// LDS bytes of a separable-assembly launch: the axis vectors of 64 rows
// (d x 2 x lm columns) and a zero column, then the class's block table
inline size_t ell_sep_lds(int d, int lm, int tb, bool f32)
{
    return (size_t)(d * 2 * lm + 1) * 64 * (f32 ? 4 : 8) + (size_t)tb;
}
// Workgroups of an assembly kernel resident per CU at an LDS size, at most 8
// (the persistent grids of the assembly are sized so that every workgroup is
// resident at once): sep = the separable kernel (256 threads), else the
// LDS-box kernel with lane groups of G.  *out = 8 when the query fails.
hipError_t ell_per_cu(int d, int G, bool f32, bool sep, size_t lds, int *out);
// the separable-box form: d >= 2, affine axes, a compiled Q*
bool box_compiled(int d, int qs);

// Thread-per-node and separable-box launchers, one per (precision, dimension)
// (fk_node_inst.hip).  Each returns false when the plan's Q* (or its mix of
// box work and axis kinds) has no compiled specialisation.
#define FK_NODE_ENTRY(name) \
    bool name(const PlanDev &P, int n, const void *packed, void *u_out, hipStream_t s);
#define FK_ADJ_ENTRY(name)                                                                  \
    bool name(const PlanDev &P, int n, const void *packed, const void *lam, void *mu,       \
              double *grad, hipStream_t s);
FK_NODE_ENTRY(step_node_f32_d1) FK_NODE_ENTRY(step_node_f32_d2) FK_NODE_ENTRY(step_node_f32_d3)
FK_NODE_ENTRY(step_node_f64_d1) FK_NODE_ENTRY(step_node_f64_d2) FK_NODE_ENTRY(step_node_f64_d3)
FK_ADJ_ENTRY(adjoint_node_f32_d1) FK_ADJ_ENTRY(adjoint_node_f32_d2) FK_ADJ_ENTRY(adjoint_node_f32_d3)
FK_ADJ_ENTRY(adjoint_node_f64_d1) FK_ADJ_ENTRY(adjoint_node_f64_d2) FK_ADJ_ENTRY(adjoint_node_f64_d3)
#undef FK_NODE_ENTRY
#undef FK_ADJ_ENTRY
hipError_t launch_assemble_ell(const PlanDev &P, bool f32, int n, int *org, void *vals,
                               void *exit_mass, hipStream_t s);
hipError_t launch_ell_apply(const PlanDev &P, bool f32, const int *org, const void *vals,
                            const void *exit_mass, const void *packed, void *u_out,
                            hipStream_t s);
// The assembled operator applied to nc <= 4 columns (records of column c at
// packed + c * plane elements, its field at u_out + c * fstride elements).
hipError_t launch_ell_apply_mc(const PlanDev &P, bool f32, const int *org, const void *vals,
                               const void *exit_mass, const void *packed, long long plane,
                               void *u_out, long long fstride, int nc, hipStream_t s);
hipError_t launch_export_ell(const PlanDev &P, bool f32, const int *org_in, const void *vals_in,
                             int *cols_out, void *vals_out, hipStream_t s);
hipError_t launch_export_cells(const PlanDev &P, int inst, int n, int *cells,
                               unsigned char *exit_flags, hipStream_t s);
hipError_t launch_clear_flags(const PlanDev &P, hipStream_t s);

// Adjoint launchers.
// part 0: the whole transposed step; 1: the per-point work list only (or the
// lane-group form); 2: the separable-box lists only
hipError_t launch_adjoint_step(const PlanDev &P, bool f32, int n, const void *packed,
                               const void *lam, void *mu, double *grad, hipStream_t s,
                               int part = 0);
hipError_t launch_adjoint_slopes_T(const PlanDev &P, bool f32, const void *u, void *mu,
                                   void *lam_next, hipStream_t s);
hipError_t launch_adjoint_init(const PlanDev &P, bool f32, const void *lam0, void *lam,
                               hipStream_t s, bool lam0_parent_f32 = false);
// FP64 sub-plan <-> the parent FP32 plan's fields: out[out_off + j] =
// (float) u[node_off + j] and back, over every node of every instance.
hipError_t launch_convert_out(const PlanDev &P, const double *u, float *out, hipStream_t s);
hipError_t launch_convert_in(const PlanDev &P, const float *in, double *u, hipStream_t s);
// out[inst] = max over the instance's nodes of |a - b| (out cleared by the caller)
hipError_t launch_inst_maxdiff(const PlanDev &P, const double *a, const float *b, double *out,
                               hipStream_t s);
hipError_t launch_zero(void *p, size_t bytes, hipStream_t s);
// LDS atomic throughput probe (measurement): blocks x 256 lanes, iters
// conflict-free ds_add per lane, out[blocks] written.
hipError_t launch_lds_atomic_probe(bool f32, int blocks, int iters, double *out, hipStream_t s);

// 1D plans, steps n_hi - 1 .. n_lo in one launch (fk_line.hip): from u_in;
// u^{n_lo} to u_out and u^m to store + (m / every - shift) fields for every m
// divisible by `every` (each may be null).  Affine axes of at most nmax nodes,
// no landing point more than one period away, exit-1 faces, a compiled Q*.
hipError_t launch_line_steps(const PlanDev &P, bool f32, int nmax, int n_hi, int n_lo, const void *u_in,
                             void *u_out, void *store, int every, int shift, hipStream_t s);
constexpr int kLineNodes = 4096;   // its longest axis: two record buffers and the masks in LDS
constexpr size_t line_lds(int nmax, bool f32) { return (size_t)nmax * (2 * 2 * (f32 ? 4 : 8) + 5); }

// Device address of the static scratch array on the current device (taken
// with hipGetSymbolAddress on the first call per device).
hipError_t static_scratch(void **out);

// Step-operator hooks: (d + 1) fields <-> node records; a - b on active nodes
// and 0 elsewhere (b may be null).
hipError_t launch_pack_fields(const PlanDev &P, bool f32, const void *x, void *packed,
                              hipStream_t s);
hipError_t launch_unpack_fields(const PlanDev &P, bool f32, const void *packed, void *x,
                                hipStream_t s);
hipError_t launch_masked_diff(const PlanDev &P, bool f32, const void *a, const void *b, void *out,
                              hipStream_t s);

}  // namespace fk
