// kernels.h -- argument blocks and host launchers of the libgsr kernels.
#pragma once
#include "gsr_device.h"

namespace gsr {

struct ProjectArgs {
    int64_t n;
    const float *mean, *quat, *log_scale, *opacity_logit, *colour;
    const float* poses;        // [V][12]
    const ViewTable* views;    // device copy
    DevCfg cfg;
    float4 *geom, *conic_o, *rgb_d;
    float* qthr;
    void* stage;               // StageRec or (mixed) StageRecM per slot
    double* grad2d;            // [slots][9], zeroed for live slots
    unsigned long long* acc;   // [slots][GSR_FIX_LIMBS][9] (deterministic mode) or null, zeroed for live slots
    Counters* counters;
    unsigned long long* stamps;  // [V + 1]: [V] = device wall clock when the projection starts
    uint64_t* live_mask;       // [mask_words][views]: bit k of word [w][v] set when slot (v, 64 w + k) is live
    int64_t mask_words;        // ceil(n / 64)
};

struct BinArgs {
    int64_t n;                 // Gaussians per view
    int32_t n_views;
    const ViewTable* views;
    DevCfg cfg;
    const float4* geom;
    const float4* conic_o;
    const float* qthr;
    const float4* rgb_d;
    int32_t chunks;            // most chunks of GSR_BIN_CHUNK * chunk_mult live slots a view can have
    int32_t chunk_mult;
    const uint64_t* live_mask; // [mask_words][views]: the projection's liveness ballots
    int64_t mask_words;
    uint32_t* live;            // [views][n]: per view, the live Gaussians (built by the binning)
    uint32_t* live_count;      // their number, view v's at [GSR_LIVE_STRIDE v]
    int32_t total_tiles;
    uint32_t* cnt;             // per view: [chunks][tiles of the view] pair counts, then offsets
    Counters* counters;
    uint2* ranges;             // [total_tiles]: [first, last + 1) of each tile's pairs
    unsigned long long* seg;   // [capacity]: (depth bits << 32 | Gaussian index), grouped by tile
    unsigned long long* tile_blocks;  // [ceil(total_tiles / GSR_COL_TILES)]: pairs of each run of that many tiles
    uint32_t* order;           // [tiles]: tiles by pair count, descending (few tiles)
    uint32_t* buckets;         // [64]: tiles per log2 bucket, then cursors
};

struct SegArgs {
    const Counters* counters;
    const ViewTable* views;
    const uint2* ranges;
    const uint32_t* order;     // tiles by pair count, descending
    unsigned long long* seg;   // [capacity]: emitted keys, sorted in place per tile (scratch)
    unsigned long long* keys;  // [capacity]: sorted (tile << 32 | depth bits)
    uint32_t* vals;            // [capacity]: sorted slots (links of waiting lists before)
    int64_t n;
};

struct RangeArgs {
    const Counters* counters;
    const uint2* ranges;
    int32_t total_tiles;
    uint32_t* order;           // [tiles]: tiles by pair count, descending
    uint32_t* buckets;         // [64]: per log2-bucket counts, then cursors
};

struct RasterArgs {
    const ViewTable* views;
    DevCfg cfg;
    Counters* counters;         // overflow flag (read), accumulator flag (written)
    const uint2* ranges;
    const uint32_t* order;     // processing order of the tiles
    const uint32_t* vals;
    const float4* geom;        // liveness of a slot (rx >= 0)
    const void* stage;         // per-slot staging records (StageRec, or StageRecM when cfg.mixed)
    void* rgb;                 // [sum 3 H W], float (or binary16 when cfg.mixed)
    float* T_final;            // [sum H W]
    int32_t* n_contrib;        // [sum H W]
    int32_t* n_blend;          // nullable
    uint32_t* fwd_queue;       // [1]: next (long tile, part) item of the split forward
    // backward only
    const float* T_final_in;   // forward outputs, read by the backward
    const int32_t* n_contrib_in;
    const float* dL_drgb;
    const float* dL_dT;        // nullable
    double* grad2d;            // [slots][9]
    unsigned long long* acc;   // [slots][GSR_FIX_LIMBS][9] in deterministic mode, else null
    int64_t slots;
    unsigned long long* tiles_done;  // [V]: backward tiles of each view completed, over all calls
    unsigned long long* stamps;  // [V + 1]: wall clock when a view's last backward tile ends
};

struct ProjectBwdArgs {
    int64_t n;
    const float *mean, *quat, *log_scale, *opacity_logit, *colour;
    const float* poses;
    const ViewTable* views;
    DevCfg cfg;
    const uint64_t* live_mask;      // [mask_words][views]: the projection's liveness ballots
    const double* grad2d;
    unsigned long long pose_only;   // bit v set: view v updates the pose only
    float *d_mean, *d_quat, *d_log_scale, *d_opacity_logit, *d_colour;
    double* xi_partial;             // [V][blocks][6]
    double* xi_partial_sh;          // [V][blocks][6], the SH chain's (degree >= 1)
    int32_t blocks;
};

struct LossArgs {
    const void* rgb;           // float, or binary16 (half_image)
    int32_t half_image;
    const float* target;
    float* dL_drgb;
    int64_t count;      // 3 * total pixels
    float scale;        // 1 / count
};

struct TrackArgs {
    const ViewTable* views;
    const float* rgb;          // render [3][H][W] per view, concatenated
    const float* T_final;      // [H][W] per view
    const float* target;       // observation, like rgb
    double tau_alpha, tau_grad;
    double* part;              // [views][GSR_TRACK_BLOCKS][GSR_TRACK_SLOTS] partial sums
    double* loss;              // [views]
    double* exposure;          // [views][2]: g, b
    float* dL_drgb;            // like rgb
    float* dL_dT;              // like T_final, nullable
};

struct MapLossArgs {
    const ViewTable* views;
    const float* rgb;          // render [3][H][W] per view, concatenated
    const float* target;       // like rgb
    float w[11];               // window weights of offsets -5..5
    float c1, c2;              // SSIM stabilisers
    float scale_ssim;          // -lambda / (3 P), P = pixels of all views
    float scale_l1;            // (1 - lambda) / (3 P)
    double lambda, inv_n;      // lambda, 1 / (3 P)
    int32_t max_tiles;         // most 32 x 32 tiles of one view
    double* part;              // [views][max_tiles][2]: sum SSIM, sum |x - y| per block
    double* loss;              // [1]
    float* dL_drgb;            // like rgb
};

#define GSR_ADAM_BLOCKS 1024         // blocks of the gradient-norm pass

// Gaussians per block of the pruning scan: 512, or 2048 past 2^20 of them,
// where the one block that scans the blocks' counts would take longer than the
// others gain (30k: a pass 7 us with 2048, 4 with 512; 30M: the three 344 and
// 453).
#define GSR_PRUNE_SMALL (1 << 20)
static inline int32_t prune_chunk(int64_t n) { return n <= GSR_PRUNE_SMALL ? 512 : 2048; }

struct AdamArgs {
    float* p[5];               // planes: mean, quat, log_scale, opacity_logit, colour
    const float* g[5];
    float* m[5];
    float* v[5];
    int64_t len[5];            // floats per plane
    float step_size[5];        // lr / (1 - beta1^t) per plane
    float inv_sqrt_bc2;        // 1 / sqrt(1 - beta2^t)
    float beta1, beta2, omb1, omb2;  // beta and 1 - beta, each rounded once from double
    float eps, max_norm, ema;
    float* anchor;             // [3][n] or null
    double* part;              // [GSR_ADAM_BLOCKS + 1]: norm partials, then the clip factor
    double* norm;              // [1] or null
};

struct CovisArgs {
    int64_t pixels;
    int32_t frames;
    float tau;
    const float* T_key;        // [pixels]
    const float* T_frames;     // [frames][pixels]
    unsigned long long* counts;  // [frames][2]: intersection, union
    double* iou;               // [frames]
};

struct PruneArgs {
    int64_t n;
    int32_t chunk;             // prune_chunk(n) Gaussians per block, a multiple of 256
    int32_t blocks;            // ceil(n / chunk)
    const int32_t* m_obs;
    const float* v_vis;
    const float* log_scale;    // [3][n]
    const float* opacity_logit;
    const int32_t* mask;       // null: the pruning rule; else keep where mask != 0
    int32_t m_min;
    double v_min, sigma_max2, alpha_min;
    uint32_t* block_count;     // [blocks]: kept per block, then offsets
    int32_t* keep_index;       // [n]: kept indices in order
    long long* kept;           // [1]
};

struct MergeArgs {
    int64_t n;
    int32_t colour_rows;
    const float* in[5];        // planes: mean, quat, log_scale, opacity_logit, colour
    float* out[5];             // the same layout
    const float* v_vis;        // [n] merge weights
    const int32_t* nn;         // [n] nearest other Gaussian (-1: none)
    double radius, colour_tol;
    int32_t* keep;             // [n] 1 kept, 0 merged into its partner
};

struct CompactArgs {
    int64_t n;
    int32_t rows;
    const float* src;          // [rows][n]
    const int32_t* keep_index;
    const long long* kept;
    float* dst;                // [rows][n], columns < kept written
};

#define GSR_SEED_MAX_NEIGHBOURS 8
#define GSR_KNN_BLOCKS 256          // blocks of the points' bounding-box pass
#define GSR_KNN_BOX 9               // floats of one block: box (lo, hi), a point
#define GSR_KNN_SMALL 16384         // up to this many points are searched without a tree

struct SeedView {
    double P[12];              // 3x4 projection matrix K [R | t], row-major
    double centre[3];          // camera centre, world
    int32_t width, height;
    const float* image;        // [3][H][W]
    double gain, bias;         // exposure: observed = gain * radiance + bias
};

struct SeedArgs {
    SeedView views[GSR_SEED_MAX_NEIGHBOURS + 1];  // reference, then neighbours
    int64_t n;
    int32_t K;
    double max_reproj, min_parallax, alpha_lo, alpha_hi;
    const float* x_ref;        // [2][n]
    const float* x_nb;         // [K][2][n]
    const float* kappa;        // [K][n]
    float* mean;               // [3][n]
    float* colour;             // [3][n]
    float* opacity_logit;      // [n]
    int32_t* valid;            // [n]
    int32_t* best;             // [n]
    float* err;                // [n]
    float* angle;              // [n]
    float* kappa_bar;          // [n]
};

// the cells along whose Hilbert curve the points are sorted (knn_cell), and how
// many leaves of 64 points they make
struct KnnTree {
    double centre[3];
    double inv_half;           // 1 / half the side of the cube about the bulk of the points
    double knee;               // scaled offset above which its logarithm is taken
    double least[3];           // least warped offset of a finite valid point, per axis
    double cells;              // cells per unit of it
    int32_t leaves;
};

struct KnnArgs {
    int64_t n;
    const float* mean;         // [3][n]
    const int32_t* valid;      // [n]
    float floor_scale;
    int32_t buckets;           // buckets of the sample sort: 256, 1024 or 4096
    int32_t per_block;         // points per block of the counting passes
    int64_t max_leaves;
    float* box;                // [GSR_KNN_BLOCKS][GSR_KNN_BOX]
    KnnTree* tree;
    uint64_t* split;           // [buckets] least code of each bucket
    uint32_t* total;           // [buckets] points
    uint32_t* bucket_leaf;     // [buckets + 1] first leaf
    uint32_t* row;             // [blocks][buckets] a block's offset inside each bucket
    uint16_t* bucket_of;       // [n] (0xffff: invalid)
    float4 *super_lo, *super_hi;    // [ceil(max_leaves / 64)] boxes of 64 consecutive leaves
    float4 *leaf_lo, *leaf_hi;      // [max_leaves] boxes
    float* groups;             // [max_leaves][8][6]: lo, hi of a leaf's groups of 8 points
    float4* placed;            // [max_leaves * 64]: (x, y, z, index bits) by bucket
    float4* pts;               // [max_leaves * 64]: the same, sorted
    double* mom;               // [10][leaves * 64] neighbour moments
    float* log_scale;          // [3][n] or null
    int32_t* nn_index;         // [n] or null: each point's nearest other (-1: none)
};

// anisotropic initialisation of the seeds
struct FrameArgs {
    double P[12];              // reference projection, row-major 3 x 4
    double centre[3];          // reference camera centre
    double radius;             // plane-fit neighbourhood
    double c_par;              // calibration of the axial scale
    double floor_scale;
    const float* err;          // [n] reprojection error of the kept hypothesis (px)
    const float* angle;        // [n] its baseline angle (rad)
    float* quat;               // [4][n] out
    float* log_scale;          // [3][n] out
};

#define GSR_TRACK_BLOCKS 256        // blocks per view of the tracking-loss kernels
#define GSR_TRACK_SLOTS 8           // partial sums per block (4 exposure sums, 3 loss/sign sums)
#define GSR_BIN_CHUNK 256           // Gaussians staged in LDS at a time by the binning blocks (x256)
#define GSR_BIN_LDS_TILES 16384     // views with more tiles count and place with global atomics
#define GSR_ONE_TILES 4096          // most tiles whose ranges and order one block forms
#define GSR_COL_TILES 32            // tiles per block of the count matrix's column scan
#ifndef GSR_BIN_LEAST
#define GSR_BIN_LEAST 64            // least live slots of a chunk
#endif
#ifndef GSR_BIN_BLOCKS
#define GSR_BIN_BLOCKS 512          // chunks below which they are made smaller
#endif
#define GSR_BIN_MATRIX (64 << 20)   // bytes of the count matrix past which chunks of fewer than 256 add no rows to it
#ifndef GSR_BIN_CHUNK_MULT
#define GSR_BIN_CHUNK_MULT 2        // live slots per binning chunk, in units of GSR_BIN_CHUNK
#endif
#define GSR_LIVE_STRIDE 64          // uint32 between two views' live counters (one 256-byte line each)
#define GSR_XCDS 8                  // accelerator dies; workgroups are dealt to them in turn
#ifndef GSR_SEG_THREADS
#define GSR_SEG_THREADS 256         // threads of a sorting block
#endif
#define GSR_SEG_WAVES 5             // resident waves per SIMD (the LDS of five blocks of 256 threads)
#define GSR_SEG_PER_THREAD 8        // keys per thread: a block sorts 8 x threads keys at once
#define GSR_SEG_COARSE 1024         // linear depth bins that measure a list's depth distribution
// Mean bin-mates of a key above which the digits are sorted instead.  128 lists
// of 2000 keys, whole binning: with 32 mates 50 us placed and 65 by digits, with
// 64 58 and 66, with 128 68 and 65, with 250 91 and 66.
#define GSR_SEG_CROWDED 64
#define GSR_FWD_LONG 4096           // least list length of a tile composited in parts (power of 2)
#define GSR_FWD_WAVES 5120          // resident compositing waves (256 CUs x 4 SIMDs x 5)
#ifndef GSR_FWD_SPLIT
#define GSR_FWD_SPLIT 2             // parts of a long tile (at most the pixels per lane)
#endif
#ifndef GSR_FWD_FEW_WAVES
#define GSR_FWD_FEW_WAVES 8192      // most waves for which every tile is composited in parts
#endif
#ifndef GSR_BWD_FEW_TILES
#define GSR_BWD_FEW_TILES 1536      // most tiles whose backward deals a tile to several waves
#endif
#define GSR_BWD_GROUP 8             // entries between its barriers
#define GSR_FWD_LONG_WAVES 2048     // persistent waves of the long tiles' parts (two per SIMD)

hipError_t launch_project(const ProjectArgs& a, int sh_degree, hipStream_t s);
// pair counting, offsets, emission into per-tile segments; max_tiles_view is
// the largest tile count of one view
hipError_t launch_bin(const BinArgs& a, int max_tiles_view, hipStream_t s);
hipError_t launch_order(const RangeArgs& a, hipStream_t s);
hipError_t launch_seg_sort(const SegArgs& a, int total_tiles, hipStream_t s);
hipError_t launch_raster_fwd(const RasterArgs& a, int total_tiles, int tile_px, int batch, hipStream_t s,
                             hipStream_t side, hipEvent_t fork, hipEvent_t join);
hipError_t launch_clear_grad2d(const RasterArgs& a, hipStream_t s);
hipError_t launch_raster_bwd(const RasterArgs& a, int total_tiles, int tile_px, int batch, hipStream_t s);
hipError_t launch_project_bwd(const ProjectBwdArgs& a, int sh_degree, float* d_xi, int n_views,
                              hipStream_t s);
hipError_t launch_loss_l1(const LossArgs& a, hipStream_t s);
hipError_t launch_loss_track(const TrackArgs& a, int n_views, hipStream_t s);
hipError_t launch_loss_mapping(const MapLossArgs& a, int n_views, hipStream_t s);
hipError_t launch_adam(const AdamArgs& a, bool vec, hipStream_t s);
hipError_t launch_covis(const CovisArgs& a, hipStream_t s);
hipError_t launch_prune(const PruneArgs& a, hipStream_t s);
hipError_t launch_compact(const CompactArgs& a, hipStream_t s);
hipError_t launch_merge(const MergeArgs& a, hipStream_t s);
hipError_t launch_seed_triangulate(const SeedArgs& a, hipStream_t s);
hipError_t launch_seed_scale(const KnnArgs& a, hipStream_t s);
hipError_t launch_seed_frame(const KnnArgs& a, const FrameArgs& f, hipStream_t s);

}  // namespace gsr
