// Internal declarations shared by the host API and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "sop.h"

namespace sop {

// Device-side error bits (sticky until new coordinates are loaded).
enum : unsigned {
    ERR_FENE = 1u << 0,
    ERR_OVERFLOW = 1u << 1,
    ERR_NONFINITE = 1u << 2,
    ERR_TIP = 1u << 3,
    ERR_CELL = 1u << 4,  // a rebuild cell holds more than CELL_CAP residues
    ERR_STAGE = 1u << 5, // a tile interacts with more residues than its LDS staging holds
};

// Per-residue energy record written on energy steps:
// FENE, native, repulsive, external, virial, external-force report.
constexpr int RES_E = 6;

struct PullDev {
    double anchor0[3];
    double v[3];
    double vhat[3];
    double kappa;
    int32_t residue;
    int32_t has_dir;
};

struct TipDev {
    double c0[3];
    double v[3];
    double vhat[3];
    double radius;
    double eps;
    double sigma;
    int32_t on;
    int32_t has_dir;
};

// Cell grid used to rebuild the list: wrapped (periodic-index) grid of
// gx*gy*gz cells of edge `cell`, so any position maps to a valid cell.
struct GridDev {
    float inv_cell;
    int gx, gy, gz;
    int n_cells;
};

// Residues per cell of the list-rebuild grid (fixed capacity; more is the
// list-overflow error).  A cell's edge is the search radius, 24 A by
// default: at protein density (about 120 A^3 per residue) a cell holds some
// 115 residues on average.
constexpr int CELL_CAP = 256;
// Bonded plus native partners per residue (larger is rejected at load).
constexpr int TOPO_CAP = 64;
// Largest staging set of a tile of the plain schedule (the kernels hold some
// 1,800 to 3,000 of its slots in LDS at once), of any tile size.  The rows
// hold four times the slot in 16 bits.
constexpr int STAGE_MAX = 4096;
static_assert(4 * STAGE_MAX <= 0xffff, "16-bit entries");

// Fixed-point copies of the positions: whole numbers of units of 2^-k, modulo
// 2^32 units.  `direct`: 2^50 units.  `reach` is a quarter of the period, in
// the caller's units: a bonded or native pair within it on every axis at a
// rebuild is taken from the copies until the next one, others (and every
// such pair when `bond_far`, every list pair when `list_far`) from the
// compensated positions; the batched schedule, which has the copies alone,
// keeps the periods below them beside them and takes such pairs (and, when
// `list_far`, all) over both.  That holds while no residue has moved too far
// since the rebuild: more than `jump` in one step, or, unless `by_step`, more
// than `move` units (batched and `list_far`: of 2^-22 periods) from its place
// then; and, batched, while a trajectory's residues are within `spread` of its
// first at the rebuild.
struct FixDev {
    double scale, period, inv_period;  // 2^k, 2^(32-k), 2^(k-32)
    float unit, s2, reach, direct;     // 2^-k, 2^2k, 2^(30-k), 2^(50-k)
    float narrow;                      // plain: largest half-width of a tile taken around one origin
    int list_far, bond_far;
    unsigned move;
    float jump, spread;
    int by_step;
};

// Plain schedule: what a workgroup's steps need to know of it, written at
// each rebuild; one scalar load.
struct WgRec {
    int ox, oy, oz;    // origin (fixed-point)
    int flags;         // WG_*
    int first, count;  // the tile's residues
    int slots;         // its staging set
    int base;          // lowest id of its slots
    int waves[4];      // per wave: list chunks | rounds of bonded entries << 16 | all rounds << 24
    int pad[4];
};

// Device buffers carved out of the caller's workspace.
struct DevBufs {
    // positions, two time layers; residue i is pos[l][2i] = {hi.xyz, tag},
    // pos[l][2i+1] = {lo.xyz, trajectory}; tag = index inside the
    // trajectory | fixed << 31.  x = hi + lo.
    float4 *pos[2];
    int4 *fix[2];     // plain: fixed-point copies of the positions, per layer
    int2 *trow;       // per residue: {first entry, n_bond | n_native << 12}
    float2 *tent;     // {partner id bits, r0}: bonds first, then natives
    int *list_cnt;    // partners per residue (plain: of the skin rows)
    unsigned short *list16;  // plain: skin rows (pairs within r_list + skin at the last skin build),
                             // lane order; batched: the list, rows by residue (cap entries) of 16
                             // times the local slot of its pack
    unsigned short *skin_len;  // plain: skin entries of each lane (workgroup * 256 + lane)
    unsigned short *flist16; // plain: the list rows (the skin rows filtered at r_list), lane order;
                             // during a skin search its rows by residue (cap entries)
    unsigned short *llen;    // plain: list entries of each lane (workgroup * 256 + lane)
    unsigned char *grho;     // plain: residue in the tile of each lane group (workgroup * groups + group)
    WgRec *wg_rec;           // plain: per workgroup, what its steps need of it
    int4 *tile_top;          // plain: per tile, rounds of bonded and of native entries in `ltop`,
                             // lowest id of its slots, whether stage16 holds them
    uint2 *ltop;             // plain: bonded and native entries in lane order (top_index): {partner, r0 bits}
    float4 *hi_skin;         // plain: high parts of the positions at the last skin build
    unsigned *skin_flag;     // plain: nonzero when the next rebuild must rebuild the skin
    unsigned *place;         // per residue, its copy at the last rebuild to 10 bits an axis (unless FixDev::by_step)
    unsigned *pack_moved;    // batched: per pack, whether a residue has moved too far since the rebuild
    int *pack_done;          // batched: per pack, steps of the last launch before that
    unsigned long long *list_stats;  // plain: {rebuilds, skin builds} since binding
    unsigned short *skin_ord;  // plain: per tile (tile * T + rank), 1 + its residues by decreasing
                               // skin row length (0 before the first skin search: identity)
    float4 *vel;             // plain, underdamped: per-residue velocity before its last half kick
    double *re_kbt;          // batched, replica exchange: the temperature ladder (kB T)
    int *re_tidx;            // batched, replica exchange: temperature index of each trajectory
    float *re_tscale;        // batched, replica exchange: sqrt(kB T / kB T of the parameters)
    unsigned long long *re_stats;  // batched, replica exchange: {accepted, attempted} per ladder pair
    float4 *facc;            // plain, pair-based forces: per-residue force accumulator
    double4 *eacc;           // plain, pair-based forces: per-residue energies of the pairs in its row
    int *stage;       // plain: per tile, global ids of its slots (STAGE_MAX per tile)
    int *stage_raw;   // the same in the search's order
    unsigned short *stage16;  // plain: the same less the tile's lowest id (tile_top), where all
                              // differences fit 16 bits: half the bytes of every step's ids
    int *stage_cnt;   // plain: slots per tile
    int *pack_off;    // batched form: first slot of each pack (n_packs + 1)
    int *slot_res;    // batched form: residue of each slot (a permutation of the residues)
    float4 *pos_save; // one saved layer (autotuning restores the state it found)
    int *cell_count;  // residues per cell
    float4 *cells;    // CELL_CAP slots per cell: {hi.xyz, residue id bits}
    int *cell_of;     // per residue: its cell at the last rebuild
    int *tile_first[3];  // plain: first residue of each tile (+ n) for tiles of 64, 128, 256
    int n_tiles[3];
    int max_bonds, max_natives;  // most bonded and native entries of a residue
    int4 *traj_cell;  // per trajectory: cell-index offset that keeps trajectories apart
    int *traj_lo;     // per residue: first residue of its trajectory
    int *traj_hi;     // per residue: one past the last residue of its trajectory
    int *pull_slot;   // per residue: cantilever index or -1
    PullDev *pulls;
    unsigned *stream_ids;    // per trajectory
    uint2 *noise_key;        // per residue: {tag, stream id}, the static words of its Philox counter
    long long *res_offsets;  // n_traj + 1
    double *res_energy;      // n_res * RES_E
    int *chunk_lo;           // energy reduction: first residue of each chunk (+ n_res)
    int *chunk_first;        // energy reduction: first chunk of each trajectory (+ n_chunks)
    double *chunk_sum;       // energy reduction: RES_E partial sums per chunk
    int n_chunks;
    double *energy;          // n_traj * SOP_NTERMS, last record
    double *f_ext;           // n_traj, last record
    float4 *fout;            // forces (compute_forces), noise samples
    uint4 *words;            // Philox words (noise samples)
    long long *step_base;    // graph replays: step of the period's first step
    long long *step_next;
    unsigned *err;           // ERR_*; plain: MOVED words from it, per layer, nonzero where a residue has moved too
                             // far since the rebuild, which end where wg_rec begins (to be loaded with it)
};
constexpr int MOVED = 2;

struct StepConsts {
    float k_fene, R0sq, inv_R0sq, eps_h, eps_l, sigma2;
    float c_drift, c_noise;
    float ud_c1, ud_c2;  // underdamped: exp(-zeta h/m), sqrt((1 - c1^2) kB T/m)
    unsigned key0, key1;
    double h;
};

// ---- kernel launchers (sop_kernels.hip) ----------------------------------
// Plain schedule, tiles of `tile` residues (64, 128 or 256).
// The skin search (the per-tile rows within sqrt(rs2) from the cell grid,
// renumbered by residue id) runs only when the device skin flag is set; the
// filter to rc2 runs unless `filter` is false (then the next step kernel
// filters).  `binned`: the cells already hold the current
// positions (binned by the last step kernel of the period); otherwise they
// are cleared and filled first.
void launch_rebuild(const DevBufs &b, int cur, int n_res, int cap, int tile, const GridDev &g,
                    const FixDev &fix, float rc2, float rs2, int multi, hipStream_t s, bool advance_step_base,
                    int list_every, bool binned, bool filter = true);
// Sets the skin flag so that the next rebuild rebuilds the skin.
void launch_force_skin(const DevBufs &b, hipStream_t s);
// As if a residue had moved too far: until the next rebuild the steps take the
// compensated positions.
void launch_distrust_copies(const DevBufs &b, int cur, hipStream_t s);
// Clears the cells, bins every residue at its current position and writes
// the fixed-point copies of the layer.
void launch_bin_all(const DevBufs &b, int cur, int n_res, const GridDev &g, const FixDev &fix, hipStream_t s);
// mode: 0 = step, 1 = forces only.  check_thr2 > 0: after the update, a
// residue that moved more than sqrt(check_thr2) from its position at the
// last skin build sets the skin flag.
// force_mode 0: particle-based (each residue sums its own rows); 1:
// pair-based (each pair once, atomic accumulation, then the update kernel).
// filter_rc2 > 0 (particle-based stepping only): the first step after a
// rebuild launched without its filter (launch_rebuild, filter = false),
// which filters the skin rows at filter_rc2 itself, then clears the
// n_cells cell counts and the skin flag.
void launch_step(const DevBufs &b, int cur, int n_res, int cap, int tile, const StepConsts &c,
                 const FixDev &fix, const TipDev &tip, int has_pull, bool energy, int mode,
                 const long long *step_base, long long step_off, float check_thr2, hipStream_t s,
                 int force_mode = 0, float ud_kick = 0.0f, const GridDev *bin_grid = nullptr,
                 float filter_rc2 = 0.0f, int n_cells = 0);
// Residues per chunk of the energy reduction (chunks never span trajectories).
constexpr int ECHUNK = 1024;
void launch_reduce_energy(const DevBufs &b, int n_traj, hipStream_t s);
// Batched ensemble: n_steps steps of every pack in one launch.  mode 0:
// steps without energy records; 2: steps that record at multiples of
// energy_every; 1: one force evaluation with records, no update.
void launch_batch(const DevBufs &b, int cur, int n_packs, int wg, int cap, const StepConsts &c,
                  const FixDev &fix, const TipDev &tip, int has_pull, float rc2, int list_every, long long energy_every,
                  int n_steps, int stale, int mode, const long long *step_base, long long step_off,
                  hipStream_t s, const float *tscale = nullptr);
// Replica exchange: the swaps of one round from the energies recorded in
// b.energy (see k_exchange).
void launch_exchange(const DevBufs &b, int n_rep, int n_groups, double kbt_ref, long long round,
                     unsigned key0, unsigned key1, hipStream_t s);
void launch_add_step(long long *base, long long k, hipStream_t s);
void launch_set_step(long long *dst, long long value, hipStream_t s);
void launch_noise(const DevBufs &b, int cur, int n, const StepConsts &c, long long step, uint4 *words,
                  float4 *g, hipStream_t s);

// Plain schedule, lane order.  A workgroup of 256 lanes serves 256 / nl
// residues, nl adjacent lanes each; a tile of T residues takes W = T nl / 256
// workgroups, and the residue of rank r in skin_ord belongs to group r / W of
// workgroup tile W + r % W.  A residue's partners are dealt to its lanes by
// their id modulo nl, in ascending order, so which lane sums a partner, and in
// which order, depends on the list alone; a list row that would give one lane
// more than its share of the capacity and 16 is dealt in turn instead.  A lane's
// entries (4 * slot, 16 bits) lie four to a chunk of 8 bytes, chunk k of a
// workgroup's 256 lanes side by side: a wave reads its chunks as one
// contiguous piece at an address that needs no row length, and a lane filters
// its own entries without its neighbours.  Bonded and native entries lie the
// same way, one {partner, r0} a round.
#define SOP_HD __host__ __device__ __forceinline__
// Lanes per residue.  A 64-residue tile in one workgroup (4 lanes) keeps the
// redundant staging lowest and is best once the tiles fill the 256 compute
// units about three times over; below that a step is as long as one wave's
// chain of instructions, and 8 or 16 lanes shorten it.  us a step, 4 / 8 / 16
// lanes: 16 tiles (1,000 residues) 10.7 / 8.5 / 7.4; 76 (4,800 at protein
// density) 19.0 / 14.1 / 12.1; 160 10.0 / 8.3 / 7.8; 320 10.9 / 9.1 / 10.6;
// 640 13.6 / 13.3 / 16.9; 1,200 18.9 / 21.8 / 27.7.
inline int lanes_for(int tile, int n_tiles)
{
    if (tile == 64)
        return n_tiles <= 200 ? 16 : (n_tiles <= 640 ? 8 : 4);
    return 256 / tile;
}
// Chunks of a lane's entries (even: the skin rows are read two at a time).
SOP_HD int lane_chunks(int cap, int nl) { return ((cap + nl - 1) / nl + 16 + 7) / 8 * 2; }
SOP_HD size_t chunk_index(int wg, int k, int lane, int chunks) { return ((size_t)wg * chunks + k) * 256 + lane; }
// Rounds of bonded, then of native entries: for the most of each that a
// residue of the topology has.  TOP_MIN of them, and STAGE_MIN slots of a
// staging set, are there for any tile (if only as the residue itself and the
// lowest id): the steps load them untested.
constexpr int TOP_MIN = 4, STAGE_MIN = 1024;
inline int top_rounds(int max_bonds, int max_natives, int nl)
{
    const int r = (max_bonds + nl - 1) / nl + (max_natives + nl - 1) / nl;
    return r > TOP_MIN ? r : TOP_MIN;
}
SOP_HD size_t top_index(int wg, int round, int lane, int rounds) { return ((size_t)wg * rounds + round) * 256 + lane; }

inline int tile_index(int tile) { return tile == 64 ? 0 : (tile == 128 ? 1 : 2); }

}  // namespace sop
