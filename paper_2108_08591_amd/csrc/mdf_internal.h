// mdf_internal.h -- declarations shared by the host API (mdf_api.cpp) and the
// HIP kernels (mdf_kernels.h and the lat_*.hip units).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

#include "mdf.h"

namespace mdf {

// Number of FP64 reduction slots per check:
//   0: sum |u - u_snap|^2   1: sum |u|^2   2..5: sum ubar_a (a = 0..d)
//   6: sum_{a>=1} J_aa      7: count of nodes with a non-finite moment
constexpr int kNRed = 8;

// Per-case parameters as the kernels see them (passed by value).
struct KCase {
    int nx, ny, nz;
    int pitch;              // row stride of the population planes, elements
    long long dstride;      // elements from one (set, direction) plane to the next: nz*ny*pitch and a gap
    double s0, s1, s2;
    double rho0;
    double R;
    double fbar[4];         // Fbar_a, a = 0..d  (Fbar_0 = R, Fbar_a = F_a)
    double wallu[6][3];
    int bc[6];
    float scale, inv_scale; // 16-bit deviation storage: f = rest + scale * stored
    // the same parameters rounded to FP32 once on the host (the FP32 and
    // 16-bit kernels compute in FP32), and the rest populations w_i rho0 of
    // the set a = 0 (index 0: i = 0, index 1: i > 0)
    float s1f, s2f, rho0f, Rf;
    // cs^2 R / s1, the mass-source part of P (eq. 3-15), formed once on the
    // host in the operation order the kernels used to form it per node:
    // (cs^2 R) / s1, in FP64 and in FP32
    double rps;
    float rpsf;
    float fbarf[4];
    float walluf[6][3];
    double restd[3];        // w * rho0 by weight class: rest, axis, diagonal
    float restf[3];
    // optional per-node force, d x nodes values component-major in the
    // compute dtype (caller-owned device memory), added to fbar[1..d]
    const void *ffield;
    // forcing scheme: 0 = eq. 3-21, 1 = Scheme II (eq. 2-3c, 2-7a); fmove is
    // the factor of w_i Fbar on the moving populations (1, or 1 - s2/2)
    int forcing;
    double fmove;
    float fmovef;
    // 1: the step kernels write populations with a non-temporal hint (the
    // context's population buffers exceed the Infinity Cache)
    int ntstore;
};

// Device pointers of one case inside the workspace.
struct CaseBufs {
    void *pop[2];           // ping-pong population buffers (storage dtype)
    uint8_t *links;         // bit 7: solid node; bit i: upstream of direction i is solid
    void *snap;             // d * nodes velocity snapshot (compute dtype)
    double *partial;        // per-block reduction slots (kNRed each)
    double *result;         // kNRed reduced values
    int max_blocks;         // capacity of `partial`, in blocks
};

struct LaunchShape {
    int bx, by;             // threads per block along x and y (bx * by <= 256)
    int groups;             // > 1: hand out tiles in `groups` contiguous bands, one per XCD
    int vx;                 // > 1: step kernels give each thread the storage's vector width of x-nodes
    int fuse;               // 1: advance several steps per launch where possible (axis-link lattices)
};

// Tile grid of one launch: gx * gy * gz tiles of bx * by threads, launched
// as a 1D grid of nb = gx * gy * gz blocks.  zc: z-planes per tile of the
// three-dimensional two-step kernel (which walks a chunk of planes), else 1.
struct Tiling {
    int gx, gy, nb, groups;
    int zc = 1;
};

// How launches of several steps cover a grid: strips of columns walked row
// by row, or tiles of one of two sizes.
enum Cover { kCoverStrips = 0, kCoverSmall = 1, kCoverLarge = 2 };

// Units of one case in launches of several steps: strips (of 64 columns,
// `halo` of them on either side not written, `step` written) by chunks of
// `rows` rows, or nx by ny tiles.
struct MarchGrid {
    int nx, ny;
    int rows, step, halo;
};

enum ReadMode { kReadFields = 0, kReadPops = 1, kReadCheck = 2, kReadSums = 3 };

// One case of a batched context, as the batched kernel reads it from device
// memory (the host keeps a mirror and uploads it before batched launches).
struct BatchEntry {
    KCase p;
    void *pop[2];
    const uint8_t *links;
    void *snap;
    double *partial;
    double *result;
    void *out;              // emitted fields of the current call, or null
    int gx, gy, ntiles;     // tile grid of the case for the batch launch shape
    int gx2, gy2, ntiles2;  // tile grid of two-step launches (2D axis-link lattices), else 0
    MarchGrid march;        // units of launches of several steps (2D axis-link lattices), else zero
    int cur;                // buffer holding f*(t) when the table was uploaded
};

// Arguments of one batched launch.
struct BatchLaunch {
    const BatchEntry *tab;  // device table (all cases)
    const int *meta;        // device: {active cases, total tiles}
    const int *tile_start;  // device: prefix offsets of the active cases' tiles
    const int *tile_start2; // device: the same for the units of launches of several steps
    const int *tile_start3; // device: the same for two-step tiles (follows tile_start2)
    const int *active;      // device: case ids of the active cases
    int parity;             // launches since the table upload, mod 2
    uint32_t fields;        // emitted fields (0: none)
    int grid;               // blocks of the persistent launch (one and two steps), march_grid() units (more)
    int steps;              // steps of the launch
    Cover cover;            // units of several steps
    bool gen;               // any case has a force field or runs Scheme II
    bool mask;              // any case has obstacles
    bool ntstore;           // non-temporal stores and 32-bit node offsets
    LaunchShape shape;
};

// Entry points of one lattice for every storage.  Each lattice's kernels are
// instantiated in a translation unit of their own (lat_*.hip).
struct LatOps {
    hipError_t (*step)(int storage, const KCase &p, const CaseBufs &b, int src, bool check, uint32_t fields,
                       void *out, LaunchShape s, hipStream_t stream);
    hipError_t (*step2)(int storage, const KCase &p, const CaseBufs &b, int src, uint32_t fields, void *out,
                        LaunchShape s, hipStream_t stream);
    hipError_t (*march)(int storage, const KCase &p, const CaseBufs &b, int src, int steps, Cover cover, uint32_t fields,
                        void *out, LaunchShape s, hipStream_t stream);
    hipError_t (*read)(int storage, const KCase &p, const CaseBufs &b, int src, bool pull, int mode,
                       uint32_t fields, void *out, LaunchShape s, hipStream_t stream);
    hipError_t (*init)(int storage, const KCase &p, const CaseBufs &b, int cur, int kind, const void *data,
                       hipStream_t stream);
    hipError_t (*batch)(int storage, const BatchLaunch &bl, bool check, bool emit, hipStream_t stream);
    hipError_t (*batch2)(int storage, const BatchLaunch &bl, bool emit, hipStream_t stream);
    hipError_t (*march_batch)(int storage, const BatchLaunch &bl, bool emit, hipStream_t stream);
    hipError_t (*batch_cap)(int storage, LaunchShape shape, bool mask, int *blocks_per_cu);
    hipError_t (*batch2_cap)(int storage, bool mask, int *blocks_per_cu);
    hipError_t (*links)(const KCase &p, const uint8_t *solid, uint8_t *links, hipStream_t stream);
    double cs2;             // the lattice's c_s^2 (of the velocity sets, on a lattice per set)
};
const LatOps &lat_ops_d2q5();
const LatOps &lat_ops_d3q7();
const LatOps &lat_ops_d2q5v();
const LatOps &lat_ops_d3q7v();
const LatOps &lat_ops_d2q4();
const LatOps &lat_ops_d3q6();
const LatOps &lat_ops_d2q4v();
const LatOps &lat_ops_d3q6v();
const LatOps &lat_ops_d2q9();
const LatOps &lat_ops_d3q15();
const LatOps &lat_ops_d2q9v();
const LatOps &lat_ops_d3q15v();
const LatOps &lat_ops_d2q9q5();
const LatOps &lat_ops_d3q15q7();

// Launchers (implemented in mdf_launch.hip).  All enqueue on `stream` and
// return the hipError_t of the launch.
hipError_t launch_links(int lattice, const KCase &p, const uint8_t *solid, uint8_t *links,
                        hipStream_t stream);
hipError_t launch_init(int lattice, int storage, const KCase &p, const CaseBufs &b, int cur,
                       int kind, const void *data, hipStream_t stream);
// Two steps in one launch (the lattices with axis links): f*(t) in pop[src] -> f*(t+2) in
// pop[src ^ 1]; fields (if any) emitted at both steps.
hipError_t launch_step2(int lattice, int storage, const KCase &p, const CaseBufs &b, int src, uint32_t fields,
                        void *out, LaunchShape shape, hipStream_t stream);
// Several steps in one launch (3 .. march_max; the 2D lattices with axis links): f*(t) in
// pop[src] -> f*(t + steps) in pop[src ^ 1]; fields (if any) emitted at the
// last step, or accumulated at every step.
hipError_t launch_march(int lattice, int storage, const KCase &p, const CaseBufs &b, int src, int steps, Cover cover,
                        uint32_t fields, void *out, LaunchShape shape, hipStream_t stream);
hipError_t launch_step(int lattice, int storage, const KCase &p, const CaseBufs &b, int src,
                       bool check, uint32_t fields, void *out, LaunchShape shape,
                       int *nblocks_out, hipStream_t stream);
hipError_t launch_read(int lattice, int storage, const KCase &p, const CaseBufs &b, int src,
                       bool pull, int mode, uint32_t fields, void *out, LaunchShape shape,
                       int *nblocks_out, hipStream_t stream);
hipError_t launch_finalize(const CaseBufs &b, int nblocks, hipStream_t stream);
hipError_t launch_step_batch(int lattice, int storage, const BatchLaunch &bl, bool check, hipStream_t stream);
hipError_t batch_blocks_per_cu(int lattice, int storage, LaunchShape shape, bool mask, int *blocks_per_cu);
// Batched two steps per launch (the 2D lattices with axis links) over the
// two-step tile list.
hipError_t launch_step2_batch(int lattice, int storage, const BatchLaunch &bl, hipStream_t stream);
hipError_t batch2_blocks_per_cu(int lattice, int storage, bool mask, int *blocks_per_cu);
// Two-step tile grid of a 2D case: tiles of 64 x rows nodes.
int step2_rows(int storage);
// Batched launch of bl.steps steps over the list of units (the 2D lattices with axis links).
hipError_t launch_march_batch(int lattice, int storage, const BatchLaunch &bl, hipStream_t stream);
// Units of one case in launches of several steps.
MarchGrid march_plan(const KCase &p, int storage, Cover cover);
hipError_t launch_finalize_batch(const BatchEntry *tab, const int *meta, const int *active, int nactive,
                                 hipStream_t stream);

// Nodes per thread along x of the step kernels for a storage and shape.
int step_vx(int storage, LaunchShape shape);
// c_s^2 of a lattice's (velocity) sets, from its kernels' traits; 0 for an unknown id
double lattice_cs2(int lattice);
// Blocks of one step launch / one read launch.
int grid_blocks(const KCase &p, int storage, LaunchShape shape);
int read_blocks(const KCase &p, LaunchShape shape);

// Units of launches of several steps of cases with `nodes` nodes in all:
// strips for FP32 and the 16-bit formats beyond the Infinity Cache, where
// the traffic per step counts (4096^2: FP32 116 us per step in strips and 166
// in tiles, FP16 99 and 125); tiles inside it (1024^2: FP32 9.8 and 7.5 us,
// FP16 13.9 and 9.4) and for FP64 (4096^2 320 and 247 us, 1024^2 21.5 and
// 13.4), small ones up to 73728 nodes, 65536 in the 16-bit formats (101 steps, us
// in small and in large ones: 256^2 FP64 226 and 258, FP32 162 and 183, FP16 199 and
// 197; 264^2 237 and 262, 175 and 185, 227 and 204; 288^2 265 and 266, 191 and 184,
// 246 and 197; 320^2 293 and 282, 208 and 194, 273 and 200; batches as their nodes:
// 4 x 128^2 257 and 292, 194 and 207, 233 and 231; 6 x 128^2 329 and 312, 234 and 223,
// 291 and 244).
inline Cover march_cover(long long nodes, int storage, bool beyond_cache)
{
    if (nodes <= (storage == MDF_F64 || storage == MDF_F32 ? 73728 : 65536)) return kCoverSmall;
    return storage != MDF_F64 && beyond_cache ? kCoverStrips : kCoverLarge;
}

// Units of such launches that emit: a strip that accumulates fields reads and
// writes them at every step of every row and waits each time, a tile takes all
// its nodes' at once.  21 steps, in strips, tiles and (before) launches of one
// and two steps: 4096^2 FP16 6.33, 4.51 and 5.57 ms, BF16 6.87, 4.93 and 5.94,
// 8192^2 FP32 27.6, 24.5 and 30.5.
inline Cover march_emit_cover(Cover cover, uint32_t fields)
{
    return cover == kCoverStrips && (fields & MDF_FIELD_ACCUMULATE) ? kCoverLarge : cover;
}

// Blocks (or wavefronts, in strips) of a batched launch of several steps whose
// running cases have `active` units, of `all` in the batch: the next power of
// two, so that a captured launch serves many sets of running cases.  100 steps
// of one running case of 512 x 128^2: FP16 1.53 ms and FP32 0.82 ms with the
// units and the grid of the whole batch, 0.17 and 0.16 ms with its own.
inline int march_grid(long long active, long long all)
{
    long long g = 1;
    while (g < active) g *= 2;
    return int(g < all ? g : all);
}

// Most steps of a launch of several steps: four, and five in FP32 strips
// without obstacles, force field and Scheme II (21 steps, five and four at a
// time, and with five the registers that do not fit: 8192^2 plain 9.52 and
// 11.42 ms, with emitted fields 12.15 and 13.64 ms, 8 registers).  With
// obstacles 38 registers do not fit (20.9 and 11.4 ms; and emitted fields, 80,
// 32.9 and 13.4 ms), with a force field or Scheme II 84 (39.3 and 16.0 ms, 31.9
// and 11.6 ms).  Five steps of the 16-bit formats do not fit either.
inline int march_max(Cover cover, int storage, bool mask, bool gen)
{
    return cover == kCoverStrips && storage == MDF_F32 && !mask && !gen ? 5 : 4;
}

// What a launch of several steps of one case works on: the stored sets and
// populations of a node, the nodes, and the fields emitted.
struct MarchWork {
    int sets, pops;
    long long nodes;
    bool mask, gen, walls;
    uint32_t fields;
};

// Channels of the fields of a 2D case.
inline int channels_2d(uint32_t fields)
{
    return (fields & MDF_FIELD_MOMENTS ? 4 : 0) + (fields & MDF_FIELD_GRAD ? 4 : 0) + (fields & MDF_FIELD_DIV ? 1 : 0) +
           (fields & MDF_FIELD_STRAIN ? 3 : 0) + (fields & MDF_FIELD_STRESS ? 3 : 0) + (fields & MDF_FIELD_VORT ? 1 : 0);
}

// Whether two steps per launch (k_step2) take less time than march_max in
// tiles, one case at a time (batches do better in tiles: 4 x 1000^2 FP16 754 and
// 898 us): for the 16-bit formats with all three sets on periodic grids of more
// than 3.5 million nodes, still inside the Infinity Cache, where k_step2's rows of
// 64 nodes read and write whole lines and no halo of 4 is computed again (21
// steps, us in tiles and in launches of two: BF16 D2Q4 1800^2 550 and 558, 1900^2
// 619 and 602, 2100^2 757 and 714; FP16 D2Q5 1800^2 535 and 552, 2048^2 691 and
// 665, between walls 645 and 665; with two sets 2100^2 509 and 532); and for
// FP64 that accumulates many channels, most of what a step then moves, of which
// tiles of 24 columns share the lines of their edges: more than one and a half
// per population (21 steps, 16 channels, ms: D2Q4 two sets 512^2 0.289 and 0.251,
// 1500^2 3.14 and 3.09, 4096^2 24.5 and 21.3, D2Q5 1500^2 3.28 and 3.41, 4096^2 25.9
// and 23.8; three sets D2Q4 1500^2 3.45 and 3.78, 4096^2 27.1 and 26.8; 4 channels
// D2Q4 two sets 4096^2 7.29 and 7.82), and ten and more on grids of few tiles per
// CU, which leave it waiting (us, D2Q5 three sets 16 channels 350^2 252
// and 217, 420^2 288 and 252, 512^2 317 and 383; 8 channels 350^2 135 and 154).
inline bool march_two(Cover cover, int storage, const MarchWork &w)
{
    if (cover != kCoverLarge || w.gen) return false;
    if (storage == MDF_F64) {
        const int ch = channels_2d(w.fields);
        const bool small = w.nodes > 100000 && w.nodes * w.pops <= 3200000;
        return (w.fields & MDF_FIELD_ACCUMULATE) && (2 * ch > 3 * w.pops || (small && ch >= 10));
    }
    return storage != MDF_F32 && w.sets == 3 && w.nodes > 3500000 && !w.mask && !w.walls && !w.fields;
}

// Steps of the next launch of a call that has `left` steps to go: 2 .. most, as
// even as they come, but for the last step, which is a launch of its own, so
// that the other buffer holds f*(t - 1) for the read kernels (and because the
// check rides on a one-step launch).  A call of three steps, two and one: 8192^2
// FP32 2.97 ms, 4.27 in launches of one step, FP64 1024^2 78 and 110 us.
inline int march_next(int64_t left, int most)
{
    const int64_t m = left - 1;
    if (m < 2) return 1;
    const int64_t launches = (m + most - 1) / most;
    return int((m + launches - 1) / launches);
}

// The 3D two-step launch: tiles of TX x TY nodes of a plane that walk chunks
// of zc planes, and its fill, nodes advanced over node slots of its duration.
constexpr int step2z_tx(int storage) { return storage == MDF_F32 || storage == MDF_F64 ? 32 : 64; }
constexpr int step2z_ty(int storage) { return storage == MDF_F64 ? 4 : 8; }
struct Step2zPlan {
    int zc;
    double fill;
};

// At most 32 planes per block (the two chunk-end planes then cost 2/32 of a
// read).  Blocks stay resident for their whole chunk, so a launch takes as
// long as its rounds of resident blocks times the zc + 2 planes that each
// walks: the length with the least product is taken, the longest of several.
// Resident are 256 CUs x as many copies of the LDS planes as 160 KB hold, two
// for four sets of seven directions and three for three; of the 16-bit
// formats, whose blocks are twice as large, two at their register budget.
// Against lengths of 32, halved until 512 blocks were reached (per step):
// 200 x 200 x 40 FP64 227 to 131 us, 138 x 148 x 60 123 to 100, FP32 cavity
// 237 x 199 x 49 127 to 95; three sets 123 x 254 x 35 FP64 99 to 53, 192^3 FP32
// 210 to 158; unchanged where the old length already filled its rounds (256^3
// FP32 525).
inline Step2zPlan step2z_plan(int storage, int sets, int q, int nx, int ny, int nz)
{
    const int tx = step2z_tx(storage), ty = step2z_ty(storage), ni = tx * ty;
    const int bytes = storage == MDF_F64 ? 8 : storage == MDF_F32 ? 4 : 2;
    const int lds = bytes * sets * (2 * ((q - 2) * ni + 2 * (tx + ty)) + 3 * 2 * ni);
    const long long resident = 256ll * (bytes == 2 ? 2 : 163840 / lds);
    const long long tiles = (long long)((nx + tx - 1) / tx) * ((ny + ty - 1) / ty);
    int zc = 0;
    long long least = 0;
    for (int most = nz < 32 ? nz : 32; most >= 1 && (zc == 0 || most >= 4); --most) {
        const int chunks = (nz + most - 1) / most, len = (nz + chunks - 1) / chunks;
        const long long cost = (tiles * chunks + resident - 1) / resident * (len + 2);
        if (zc == 0 || cost < least) {
            zc = len;
            least = cost;
        }
    }
    return {zc, double(nx) * ny * nz / (double(least) * resident * ni)};
}

// Two steps per launch pay in 3D where the launch is well filled: small grids,
// and tiles with much padding, leave the chip idle while blocks walk their
// planes, and walls cost the second step more than the one-step kernel.  Over 52
// grids of 24^3 to 256^3 nodes, FP64 and FP32, three and four sets, periodic and
// between walls, one step per launch is faster below these lines and two above,
// but for a few grids close to them and the cube of 64 (us per step of two and
// one; FP64 periodic, four sets: 40 x 40 x 250, filled 0.51, 35.6 and 27.4; 72 x 88 x
// 120, 0.58, 75.8 and 79.2; 64^3, 0.67, 19.6 and 17.2; three sets: 138 x 148 x 60,
// 0.73, 60.4 and 88.1; walls, four sets: 130 x 97 x 75, 0.69, 103 and 90; 150 x 65 x
// 150, 0.83, 143 and 168; FP32 periodic, three sets: 80^3, 0.43, 16.3 and 15.2; 39 x
// 223 x 123, 0.45, 42.2 and 52.8; walls: 138 x 148 x 60, 0.62, 31.2 and 36.2; four
// sets: 130 x 97 x 75, 0.56, 44.0 and 40.0; 138 x 148 x 60, 0.67, 59.7 and 60.8).
inline bool step2z_pays(int storage, int sets, int q, bool walls, int nx, int ny, int nz)
{
    double line = walls ? 0.64 : 0.5;
    if (storage == MDF_F64 && sets == 4) line = walls ? 0.72 : 0.53;
    if (storage == MDF_F32 && sets == 3) line = 0.44;
    return step2z_plan(storage, sets, q, nx, ny, nz).fill >= line;
}

}  // namespace mdf
