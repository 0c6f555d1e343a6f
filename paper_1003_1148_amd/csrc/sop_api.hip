// Host side of the C ABI: topology -> per-residue CSR (Algorithm 2's P_p and
// PairsMap, bonds and natives in both directions), workspace layout, the
// step driver with HIP-graph replays of whole list periods, and the
// asynchronous device error word.
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <initializer_list>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "sop_internal.hpp"

using namespace sop;

struct sop_ctx {
    sop_params p{};
    hipStream_t stream = nullptr;

    // topology (host copies)
    int n_traj = 0;
    long long n_res = 0;
    std::vector<long long> res_offsets;
    std::vector<unsigned> stream_ids;
    std::vector<int2> trow;
    std::vector<float2> tent;
    std::vector<int> traj_lo, traj_hi, traj_of, local;
    std::vector<unsigned char> fixed;
    std::vector<PullDev> pulls;
    std::vector<int> pull_slot;
    std::vector<int4> traj_cell;
    std::vector<int> tiles[3];  // plain: first residue of each tile (+ n) for tiles of 64, 128, 256
    std::vector<int> chunk_lo, chunk_first;  // energy reduction chunks
    TipDev tip{};

    // schedule: plain (kernel per step) or batched (persistent packs)
    int schedule = SOP_SCHEDULE_PLAIN;
    int tile_req = 0, tile = 128, cap = 256, cap_req = 0;
    // plain: the Verlet skin.  Rows of pairs within r_list + skin are built
    // on the cell grid only when some residue has moved more than skin/2
    // since the last such build; every rebuild filters them to r_list.
    double skin = 4.0;
    int force_mode = SOP_FORCES_PARTICLE;  // plain: particle- or pair-based force evaluation
    int integrator = SOP_INTEGRATOR_OVERDAMPED;
    double mass = 1.0;               // underdamped: mass of a residue
    // batched: replica exchange over groups of re_rep consecutive trajectories
    int re_rep = 0;
    std::vector<double> re_kbt;
    long long re_every = 0, re_last = -1;
    bool ud_half = true;             // underdamped: the stored velocities are at the current step
    long long skin_checked = -1;     // step at which the skin was last known valid
    long long binned_at = -1;        // step whose positions the cells hold (consumed by a rebuild)
    std::vector<double> xyz_set;     // the coordinates the grid was laid out for
    int graph_steps = 1;
    long long energy_every = 0;
    int batch_wg_req = 0, batch_wg = 1024, batch_steps = 100;
    long long max_len = 0;           // longest trajectory
    int max_bonds = 0, max_natives = 0;  // of a residue
    double min_r0 = 0.0;             // shortest bonded or native reference length (huge if none)
    std::vector<int> pack_off;       // batched: first slot of each pack
    std::vector<int> slot_res;       // batched: residue of each slot
    hipGraphExec_t bgraphs[2][2] = {};  // batched launch graphs by layer parity, records

    // device state
    bool topo = false, bound = false, coords = false, list_valid = false;
    void *ws = nullptr;
    size_t ws_bytes = 0;
    DevBufs b{};
    GridDev grid{};
    int n_cells_cap = 0;
    int cur = 0;
    long long step = 0;
    long long energy_step = -1;
    unsigned sticky = 0;
    std::string last_error;

    // graphs over whole list periods, keyed by [layer parity][energy at first step]
    hipStream_t cap_stream = nullptr;
    hipGraphExec_t graphs[2][2] = {{nullptr, nullptr}, {nullptr, nullptr}};
    hipGraphExec_t long_graphs[2][2] = {{nullptr, nullptr}, {nullptr, nullptr}};  // several of them in one
    int graph_runs = 0;  // replays of `graphs`, up to LONG_AFTER

    // two halves of host memory that results and coordinates pass through
    char *pin = nullptr;
    size_t pin_half = 0;
    bool pin_paged = false;  // not page-locked (none was to be had)
};

namespace {

sop_status fail(sop_ctx *c, sop_status s, const std::string &msg)
{
    if (c)
        c->last_error = msg;
    return s;
}

sop_status hip_fail(sop_ctx *c, hipError_t e, const char *what)
{
    return fail(c, SOP_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

#define HIP_TRY(ctx, expr)                                 \
    do {                                                   \
        hipError_t e_ = (expr);                            \
        if (e_ != hipSuccess)                              \
            return hip_fail((ctx), e_, #expr);             \
    } while (0)

// A list that overflowed leaves the forces undefined, so it is reported first.
sop_status status_from_bits(unsigned bits)
{
    if (bits & (ERR_OVERFLOW | ERR_CELL | ERR_STAGE))
        return SOP_E_LIST_OVERFLOW;
    if (bits & ERR_FENE)
        return SOP_E_FENE;
    if (bits & ERR_TIP)
        return SOP_E_TIP;
    if (bits & ERR_NONFINITE)
        return SOP_E_NONFINITE;
    return SOP_OK;
}

const char *bits_message(unsigned bits)
{
    if (bits & ERR_OVERFLOW)
        return "a residue has more list partners than the list capacity";
    if (bits & ERR_CELL)
        return "more than 256 residues fell into one cell of the list-rebuild grid";
    if (bits & ERR_STAGE)
        return "a tile of the plain schedule interacts with more residues than its LDS staging holds, or its cell neighbourhood exceeds the rebuild's LDS table";
    if (bits & ERR_FENE)
        return "a FENE bond reached |r - r0| >= R0";
    if (bits & ERR_TIP)
        return "a residue reached the tip surface";
    if (bits & ERR_NONFINITE)
        return "a force or position became non-finite";
    return "";
}

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Row capacity: the requested one, else 1024 entries for the plain schedule
// (its skin rows hold the partners within r_list + skin: at protein density,
// about 120 A^3 per residue, some 480 within 24 A) and 256 for the batched
// one; a multiple of 16.
int list_cap(const sop_ctx *c)
{
    const int cap = c->cap_req ? c->cap_req : (c->schedule == SOP_SCHEDULE_PLAIN ? 1024 : 256);
    return ((cap + 15) / 16) * 16;
}

// Workspace layout: returns total bytes; fills pointers when base != null.
size_t layout(const sop_ctx *c, char *base, DevBufs *b)
{
    const size_t n = (size_t)c->n_res;
    const size_t T = (size_t)c->n_traj;
    const bool plain = c->schedule == SOP_SCHEDULE_PLAIN;
    // per-tile blocks, for the largest need over the tile sizes
    size_t n_tiles_max = 0, stage_elems = 0, tf_elems[3] = {1, 1, 1};
    size_t chunk_elems = 0, ltop_elems = 0, wg_elems = 0;
    if (plain)
        for (int k = 0; k < 3; ++k) {
            const size_t T = (size_t)64 << k, nt = c->tiles[k].size() - 1;
            const int nl = lanes_for((int)T, (int)nt);
            const size_t wgs = nt * (T * nl / 256);
            chunk_elems = std::max(chunk_elems, wgs * 1024 * (size_t)lane_chunks(c->cap, nl));
            ltop_elems = std::max(ltop_elems, wgs * 256 * (size_t)top_rounds(c->max_bonds, c->max_natives, nl));
            wg_elems = std::max(wg_elems, wgs);
            stage_elems = std::max(stage_elems, nt * (size_t)STAGE_MAX);
            n_tiles_max = std::max(n_tiles_max, nt);
            tf_elems[k] = nt + 1;
        }
    const size_t ncell = plain ? (size_t)c->n_cells_cap : 0;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *p = base ? base + off : nullptr;
        off = align256(off + std::max<size_t>(bytes, 1));
        return p;
    };
    DevBufs d{};
    d.max_bonds = c->max_bonds;
    d.max_natives = c->max_natives;
    d.pos[0] = (float4 *)take(2 * n * sizeof(float4));
    d.pos[1] = (float4 *)take(2 * n * sizeof(float4));
    d.trow = (int2 *)take(n * sizeof(int2));
    d.tent = (float2 *)take(c->tent.size() * sizeof(float2));
    d.list_cnt = (int *)take(n * sizeof(int));
    d.list16 = (unsigned short *)take((plain ? chunk_elems : n * (size_t)c->cap) * sizeof(unsigned short));
    d.flist16 = (unsigned short *)take(chunk_elems * sizeof(unsigned short));
    d.skin_len = (unsigned short *)take(wg_elems * 256 * sizeof(unsigned short));
    d.llen = (unsigned short *)take(wg_elems * 256 * sizeof(unsigned short));
    d.grho = (unsigned char *)take(wg_elems * 256);
    if (char *rec = take((wg_elems + 1) * sizeof(WgRec))) {
        d.wg_rec = (WgRec *)rec + 1;
        d.err = (unsigned *)d.wg_rec - MOVED - 2;
    }
    d.tile_top = (int4 *)take(n_tiles_max * sizeof(int4));
    d.ltop = (uint2 *)take(ltop_elems * sizeof(uint2));
    for (auto &f : d.fix)
        f = (int4 *)take((plain ? n : 0) * sizeof(int4));
    d.hi_skin = (float4 *)take((plain ? n : 0) * sizeof(float4));
    d.skin_flag = (unsigned *)take(sizeof(unsigned));
    d.place = (unsigned *)take(n * sizeof(unsigned));
    d.pack_moved = (unsigned *)take((plain ? 0 : T) * sizeof(unsigned));
    d.pack_done = (int *)take((plain ? 0 : T) * sizeof(int));
    d.list_stats = (unsigned long long *)take(2 * sizeof(unsigned long long));
    d.skin_ord = (unsigned short *)take((plain ? n_tiles_max * 256 : 0) * sizeof(unsigned short));
    d.vel = (float4 *)take((plain ? n : 0) * sizeof(float4));
    d.facc = (float4 *)take((plain ? n : 0) * sizeof(float4));
    d.re_kbt = (double *)take((plain ? 0 : T) * sizeof(double));
    d.re_tidx = (int *)take((plain ? 0 : T) * sizeof(int));
    d.re_tscale = (float *)take((plain ? 0 : T) * sizeof(float));
    d.re_stats = (unsigned long long *)take((plain ? 0 : 2 * T) * sizeof(unsigned long long));
    d.eacc = (double4 *)take((plain ? n : 0) * sizeof(double4));
    d.stage = (int *)take(stage_elems * sizeof(int));
    d.stage_raw = (int *)take(stage_elems * sizeof(int));
    d.stage16 = (unsigned short *)take(stage_elems * sizeof(unsigned short));
    d.stage_cnt = (int *)take(n_tiles_max * sizeof(int));
    d.pack_off = (int *)take((T + 1) * sizeof(int));
    d.slot_res = (int *)take(n * sizeof(int));
    d.pos_save = (float4 *)take(2 * n * sizeof(float4));
    d.cell_count = (int *)take(ncell * sizeof(int));
    d.cells = (float4 *)take(ncell * CELL_CAP * sizeof(float4));
    d.cell_of = (int *)take((plain ? n : 0) * sizeof(int));
    for (int k = 0; k < 3; ++k) {
        d.tile_first[k] = (int *)take(tf_elems[k] * sizeof(int));
        d.n_tiles[k] = plain ? (int)(tf_elems[k] - 1) : 0;
    }
    d.traj_cell = (int4 *)take(T * sizeof(int4));
    d.traj_lo = (int *)take(n * sizeof(int));
    d.traj_hi = (int *)take(n * sizeof(int));
    d.pull_slot = (int *)take(n * sizeof(int));
    d.pulls = (PullDev *)take(std::max<size_t>(c->pulls.size(), 1) * sizeof(PullDev));
    d.stream_ids = (unsigned *)take(T * sizeof(unsigned));
    d.noise_key = (uint2 *)take(n * sizeof(uint2));
    d.res_offsets = (long long *)take((T + 1) * sizeof(long long));
    d.res_energy = (double *)take(n * RES_E * sizeof(double));
    d.n_chunks = (int)c->chunk_lo.size() - 1;
    d.chunk_lo = (int *)take(c->chunk_lo.size() * sizeof(int));
    d.chunk_first = (int *)take(c->chunk_first.size() * sizeof(int));
    d.chunk_sum = (double *)take((size_t)std::max(d.n_chunks, 1) * RES_E * sizeof(double));
    d.energy = (double *)take(T * SOP_NTERMS * sizeof(double));
    d.f_ext = (double *)take(T * sizeof(double));
    d.fout = (float4 *)take(n * sizeof(float4));
    d.words = (uint4 *)take(n * sizeof(uint4));
    d.step_base = (long long *)take(sizeof(long long));
    d.step_next = (long long *)take(sizeof(long long));
    if (b)
        *b = d;
    return off;
}

// Residues per workgroup of the plain schedule: enough tiles to cover the
// 256 compute units a few times over.
// 64-residue tiles: four lanes per residue in the step kernel, four waves
// sharing each tile's rebuild (sop_autotune measures the others).
int default_tile(long long) { return 64; }

void destroy_graphs(sop_ctx *c)
{
    for (auto *set : {&c->graphs, &c->long_graphs})
        for (auto &row : *set)
            for (auto &g : row)
                if (g) {
                    (void)hipGraphExecDestroy(g);
                    g = nullptr;
                }
    c->graph_runs = 0;
    for (auto &gp : c->bgraphs)
        for (auto &g : gp)
            if (g) {
                (void)hipGraphExecDestroy(g);
                g = nullptr;
            }
}

// Packs of whole trajectories for the batched schedule: first-fit
// decreasing by length (ties by index) into workgroups of `wg` residues, so
// packs start with the longest trajectories and all but one are more than
// half full. Inside a pack the trajectories keep their index order, residues
// consecutive. The results do not depend on the packing.
void make_packs(sop_ctx *c)
{
    const int T = c->n_traj, wg = c->batch_wg;
    std::vector<int> order(T);
    for (int t = 0; t < T; ++t)
        order[t] = t;
    auto len = [&](int t) { return c->res_offsets[t + 1] - c->res_offsets[t]; };
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return len(x) > len(y); });
    // first fit: the leftmost pack with room, from a max-tree over the rooms
    // of T packs (the ones not opened yet are empty, so the leftmost fit is
    // an open pack or the next new one)
    int leaves = 1;
    while (leaves < std::max(T, 1))
        leaves <<= 1;
    std::vector<long long> tree(2 * (size_t)leaves, 0);
    for (int k = 0; k < T; ++k)
        tree[leaves + k] = wg;
    for (int v = leaves - 1; v >= 1; --v)
        tree[v] = std::max(tree[2 * v], tree[2 * v + 1]);
    std::vector<std::vector<int>> members;
    for (int t : order) {
        int v = 1;
        while (v < leaves)
            v = tree[2 * v] >= len(t) ? 2 * v : 2 * v + 1;
        const int k = v - leaves;  // exists: every trajectory fits an empty pack
        if (k >= (int)members.size())
            members.resize(k + 1);
        members[k].push_back(t);
        tree[v] -= len(t);
        for (v >>= 1; v >= 1; v >>= 1)
            tree[v] = std::max(tree[2 * v], tree[2 * v + 1]);
    }
    c->pack_off.assign(1, 0);
    c->slot_res.clear();
    c->slot_res.reserve((size_t)c->n_res);
    for (auto &m : members) {
        std::sort(m.begin(), m.end());
        for (int t : m)
            for (long long r = c->res_offsets[t]; r < c->res_offsets[t + 1]; ++r)
                c->slot_res.push_back((int)r);
        c->pack_off.push_back((int)c->slot_res.size());
    }
}

sop_status upload_packs(sop_ctx *c)
{
    HIP_TRY(c, hipMemcpyAsync(c->b.pack_off, c->pack_off.data(), c->pack_off.size() * sizeof(int),
                              hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipMemcpyAsync(c->b.slot_res, c->slot_res.data(), c->slot_res.size() * sizeof(int),
                              hipMemcpyHostToDevice, c->stream));
    return SOP_OK;
}

int pick_batch_wg(const sop_ctx *c)
{
    if (c->batch_wg_req)
        return c->batch_wg_req;
    return c->max_len <= 256 ? 256 : (c->max_len <= 512 ? 512 : 1024);
}

int n_packs(const sop_ctx *c) { return (int)c->pack_off.size() - 1; }

StepConsts step_consts(const sop_ctx *c)
{
    StepConsts k{};
    k.k_fene = (float)c->p.k_fene;
    k.R0sq = (float)(c->p.R0 * c->p.R0);
    k.inv_R0sq = (float)(1.0 / (c->p.R0 * c->p.R0));
    k.eps_h = (float)c->p.eps_h;
    k.eps_l = (float)c->p.eps_l;
    k.sigma2 = (float)(c->p.sigma * c->p.sigma);
    k.c_drift = (float)(c->p.h / c->p.zeta);
    k.c_noise = (float)std::sqrt(2.0 * c->p.kBT * c->p.h / c->p.zeta);
    const double c1 = std::exp(-c->p.zeta / c->mass * c->p.h);
    k.ud_c1 = (float)c1;
    k.ud_c2 = (float)std::sqrt((1.0 - c1 * c1) * c->p.kBT / c->mass);
    k.key0 = (unsigned)(c->p.seed & 0xffffffffu);
    k.key1 = (unsigned)(c->p.seed >> 32);
    k.h = c->p.h;
    return k;
}

// Scale of the fixed-point copies: the coarsest power of two that keeps 2.5
// times the distance a listed pair can have (r_list, and 16 standard deviations
// of the thermal drift of a list period, eight for each partner) inside half
// the period of 2^32 units, H.  At r_list = 20 A: k = 25, H 64 A, unit 3e-8 A.
// Bonded and native terms, which are steep where the forces cancel, use the
// copies only while a unit is at most 2^-26 of the shortest reference length, a
// quarter of what rounding that length to single precision leaves: L2 force
// error 5.84e-7 against 5.94e-7 of compensated positions for 1,500 residues at
// 3.8 A; at twice the unit, as r_list = 24 to 45 A would have, 5.99e-7, at four
// times 6.46e-7.  Beyond it the plain schedule takes the compensated positions
// for them (20,000 residues at 30 A 10.4 -> 10.95 us a step, the movement check
// in the second), the batched one a finer unit, and the list over the periods
// from r_list = 0.75 H (48 A) on (200 chains 13.7 -> 18.1 us a step at the same
// list).  The list uses the copies only while a unit is below 2e-6 sigma.
// `narrow`: copies relative to a tile's origin wrap at H, and a list partner
// lies up to r_list further out than the tile's residues, plus what it moves
// until the next rebuild, for which a margin is left.  At 300 K and the time
// step of the reference workloads: 40 A from r_list = 10.6 A (H = 64 A) to
// 20 A, 37 A at 23 A, 18 A at 10 A (H = 32 A).
// The margin is also what a residue may move until the next rebuild, H / 4 at
// most (pairs are H / 2 apart at most at the rebuild): 4 A at r_list = 20 A.
// Thermal motion never exceeds it; whatever does (a clash that throws a
// residue off, a fast anchor) makes the steps until the next rebuild take the
// compensated positions.  `by_step`: no step may take more than its share of
// the margin, which must be 8.5 standard deviations of a step's noise: one
// comparison a step, for list periods up to some 100 steps (H / 8).  Longer ones
// compare every residue with its place at the rebuild, to 10 bits an axis
// (`move`, from below; a step of at most `jump`, four times it, cannot go
// round).  us a step kernel without a check, by step, by place: 56 residues 4.0,
// 4.1, 4.2; 4,801 8.4, 8.8, 8.9; 75,000 13.5, 13.6, 13.9; 250,000 35.2, 35.7,
// 36.3.  Batched: H / 8, as a launch within a list period takes the reach of
// bonded and native pairs anew; 128 periods where differences are taken over
// the periods, of which the copies hold 1,024, and a trajectory may span 256.
// 500 steps of 200 chains 6.04 -> 6.27 ms with the check and the launches
// behind (k_batch_exact), of 4,096 31.6 -> 31.9.
constexpr double NARROW_MAX = 40.0;

FixDev fix_consts(const sop_ctx *c)
{
    const double steps = c->p.list_every;
    double noise = std::sqrt(2.0 * c->p.kBT * c->p.h / c->p.zeta), drift = 16.0 * noise * std::sqrt(steps);
    if (c->integrator == SOP_INTEGRATOR_UNDERDAMPED) {
        // no further than at the thermal velocity (low friction)
        const double flight = std::sqrt(c->p.kBT / c->mass) * c->p.h;
        noise = std::min(noise, flight);
        drift = std::min(drift, 16.0 * flight * steps);
    }
    const double half = 2.5 * (c->p.r_list + drift);
    int k = 31 - (int)std::ceil(std::log2(std::min(std::max(half, 1e-9), 1e30)));
    // batched: bonded and native terms have the copies alone, so the unit
    // follows the shortest reference length where that asks for a finer one
    if (c->schedule == SOP_SCHEDULE_BATCHED)
        k = std::max(k, std::min(k + 8, 26 - (int)std::floor(std::log2(std::min(std::max(c->min_r0, 1e-9), 1e30)))));
    k = std::max(-60, std::min(60, k));
    const double H = std::ldexp(1.0, 31 - k);
    FixDev f{};
    f.scale = std::ldexp(1.0, k);
    f.period = std::ldexp(1.0, 32 - k);
    f.inv_period = std::ldexp(1.0, k - 32);
    f.unit = (float)std::ldexp(1.0, -k);
    f.s2 = (float)std::ldexp(1.0, 2 * k);
    f.reach = (float)std::ldexp(1.0, 30 - k);
    f.direct = (float)std::ldexp(1.0, 50 - k);
    // batched: pairs of r_list, and an eighth of H of movement for either partner
    const bool wraps = c->schedule == SOP_SCHEDULE_BATCHED ? c->p.r_list > 0.75 * H : half > H;
    f.list_far = (wraps || f.unit > 2e-6 * c->p.sigma) ? 1 : 0;
    f.bond_far = f.unit > std::ldexp(c->min_r0, -26) ? 1 : 0;
    const double share = 8.5 * noise * steps, periods = 256 * H;  // 128 of them
    double move, grain = 1.0;
    if (c->schedule == SOP_SCHEDULE_BATCHED) {
        move = f.list_far ? periods : H / 8;
        grain = f.list_far ? std::ldexp(1.0, -10) : 1.0;
        f.by_step = share <= move ? 1 : 0;
    } else {
        f.by_step = share <= H / 8 ? 1 : 0;
        f.narrow = (float)std::min(NARROW_MAX, H - c->p.r_list - std::max({drift, H / 16, f.by_step ? share : 0.0}));
        // less the low parts, which neither the tile's box nor the list has
        // (up to |x| = 2^14 H, some 1e6 A)
        move = f.list_far ? H / 4 : std::min(H / 4, H - f.narrow - c->p.r_list - H / 512);
    }
    f.move = (unsigned)(move * f.scale * grain) - (1u << 22);
    f.jump = (float)(f.by_step ? move / steps : 4 * move);
    f.spread = (float)periods;
    return f;
}

// Underdamped integrator: the kick of the next step (h/2m right after the
// velocities were set, else h/m); 0 selects the overdamped update.
float ud_kick(const sop_ctx *c)
{
    if (c->integrator != SOP_INTEGRATOR_UNDERDAMPED)
        return 0.0f;
    return (float)((c->ud_half ? 0.5 : 1.0) * c->p.h / c->mass);
}

float list_rc2(const sop_ctx *c) { return (float)(c->p.r_list * c->p.r_list); }

// The plain schedule's skin build radius r_list + skin (the batched schedule
// builds its list directly).
double skin_radius(const sop_ctx *c)
{
    return c->p.r_list + (c->schedule == SOP_SCHEDULE_PLAIN ? c->skin : 0.0);
}
float skin_rs2(const sop_ctx *c) { return (float)(skin_radius(c) * skin_radius(c)); }

// Largest displacement since the skin build that keeps the skin valid
// (squared; 0 = rebuild the skin at every rebuild): skin/2 less a margin
// far above the rounding of the single-precision distances.
float skin_check_thr2(const sop_ctx *c)
{
    const double thr = 0.5 * c->skin - 0.01;
    return (c->schedule == SOP_SCHEDULE_PLAIN && thr > 0.0) ? (float)(thr * thr) : 0.0f;
}

// Cell edge slightly above the skin radius so that any pair passing the
// single-precision predicate lies in adjacent cells despite rounding of the
// cell index.
float cell_edge(const sop_ctx *c) { return (float)(skin_radius(c) * 1.002 + 0.05); }

// Grid for the list rebuild.  Each trajectory's cells are shifted to its own
// block of a lattice of trajectory boxes so that independent trajectories
// that overlap in space do not share cells; the grid wraps, so positions
// outside the initial boxes still map to valid (shared) cells.
void set_grid(sop_ctx *c, const double *xyz)
{
    const double e = cell_edge(c);
    const int T = c->n_traj;
    std::vector<long long> lo(3 * (size_t)T), ext(3 * (size_t)T);
    long long span[3] = {1, 1, 1};
    for (int t = 0; t < T; ++t) {
        double mn[3] = {1e300, 1e300, 1e300}, mx[3] = {-1e300, -1e300, -1e300};
        for (long long i = c->res_offsets[t]; i < c->res_offsets[t + 1]; ++i)
            for (int a = 0; a < 3; ++a) {
                mn[a] = std::min(mn[a], xyz[3 * i + a]);
                mx[a] = std::max(mx[a], xyz[3 * i + a]);
            }
        for (int a = 0; a < 3; ++a) {
            if (c->res_offsets[t + 1] == c->res_offsets[t]) {
                mn[a] = mx[a] = 0.0;
            }
            lo[3 * t + a] = (long long)std::floor(mn[a] / e);
            ext[3 * t + a] = (long long)std::floor(mx[a] / e) - lo[3 * t + a] + 1;
            span[a] = std::max(span[a], ext[3 * t + a] + 1);  // one empty cell between boxes
        }
    }
    // lattice of trajectory boxes, about as many along each axis
    long long A = 1;
    while (A * A * A < T)
        ++A;
    c->traj_cell.assign(T, int4{0, 0, 0, 0});
    long long g[3] = {3, 3, 3};
    for (int t = 0; t < T; ++t) {
        const long long ix = t % A, iy = (t / A) % A, iz = t / (A * A);
        const long long org[3] = {ix * span[0], iy * span[1], iz * span[2]};
        long long off[3];
        for (int a = 0; a < 3; ++a) {
            off[a] = org[a] - lo[3 * t + a];
            g[a] = std::max(g[a], org[a] + ext[3 * t + a] + 1);
        }
        c->traj_cell[t] = int4{(int)off[0], (int)off[1], (int)off[2], 0};
    }
    while (g[0] * g[1] * g[2] > c->n_cells_cap) {
        int m = 0;
        for (int a = 1; a < 3; ++a)
            if (g[a] > g[m])
                m = a;
        g[m] = std::max<long long>(3, (g[m] * 3) / 4);
        if (g[0] == 3 && g[1] == 3 && g[2] == 3)
            break;
    }
    c->grid.inv_cell = 1.0f / (float)e;
    c->grid.gx = (int)g[0];
    c->grid.gy = (int)g[1];
    c->grid.gz = (int)g[2];
    c->grid.n_cells = (int)(g[0] * g[1] * g[2]);
}

// Host memory for the copies between the device and the caller: page-locked
// (a copy to or from it is asynchronous and takes no staging of the
// runtime's), at most 2 MiB a half, belongs to the context.
constexpr size_t PIN_MAX = (size_t)2 << 20, PIN_ALIGN = 256;

void free_pin(sop_ctx *c)
{
    if (c->pin_paged)
        std::free(c->pin);
    else if (c->pin)
        (void)hipHostFree(c->pin);
    c->pin = nullptr;
    c->pin_half = 0;
}

sop_status make_pin(sop_ctx *c)
{
    const size_t want = std::min(PIN_MAX, (size_t)c->n_res * 32 / 4096 * 4096 + 65536);
    if (c->pin && c->pin_half >= want)
        return SOP_OK;
    free_pin(c);
    void *p = nullptr;
    c->pin_paged = hipHostMalloc(&p, 2 * want, hipHostMallocPortable) != hipSuccess;
    if (c->pin_paged) {
        (void)hipGetLastError();
        p = std::malloc(2 * want);
        if (!p)
            return fail(c, SOP_E_HIP, "no host memory");
    }
    c->pin = static_cast<char *>(p);
    c->pin_half = want;
    return SOP_OK;
}

// Device ranges brought to the host: use(k, offset, bytes, data) for every
// piece of range k in order, while the next piece is on its way.  One wait for
// all of them where they fit half of the host memory: scoring 10,000 residues
// (which copied four ranges with a wait for each) 299 -> 245 us, 500 steps of
// 4,096 chains with their 1.1e6 coordinates (which passed through a pageable
// copy of all of them) 38.7 -> 35.1 ms.
struct DeviceRange {
    const void *dev;
    size_t bytes;
};

template <class F>
sop_status fetch(sop_ctx *c, std::initializer_list<DeviceRange> list, F use)
{
    struct Part {
        int k;
        size_t off, bytes, at;
    };
    std::vector<Part> parts[2];
    const DeviceRange *r = list.begin();
    const int n = (int)list.size();
    int k = 0;
    size_t off = 0;
    auto issue = [&](int h) -> hipError_t {
        parts[h].clear();
        size_t at = 0;  // a multiple of PIN_ALIGN, as the halves are
        while (k < n && at < c->pin_half) {
            const size_t b = std::min(r[k].bytes - off, c->pin_half - at);
            if (b > 0) {
                const hipError_t e = hipMemcpyAsync(c->pin + h * c->pin_half + at,
                                                    static_cast<const char *>(r[k].dev) + off, b,
                                                    hipMemcpyDeviceToHost, c->stream);
                if (e != hipSuccess)
                    return e;
                parts[h].push_back({k, off, b, h * c->pin_half + at});
            }
            off += b;
            at += (b + PIN_ALIGN - 1) / PIN_ALIGN * PIN_ALIGN;
            if (off == r[k].bytes) {
                ++k;
                off = 0;
            }
        }
        return hipSuccess;
    };
    HIP_TRY(c, issue(0));
    for (int h = 0; !parts[h].empty(); h ^= 1) {
        HIP_TRY(c, hipStreamSynchronize(c->stream));
        HIP_TRY(c, issue(h ^ 1));
        for (const Part &p : parts[h])
            use(p.k, p.off, p.bytes, c->pin + p.at);
    }
    return SOP_OK;
}

// The error word as a range of a fetch, and what it says.
DeviceRange error_range(const sop_ctx *c) { return {c->b.err, sizeof(unsigned)}; }

void take_errors(sop_ctx *c, const char *data)
{
    unsigned bits;
    std::memcpy(&bits, data, sizeof(bits));
    c->sticky |= bits;
}

sop_status error_status(sop_ctx *c)
{
    return c->sticky ? fail(c, status_from_bits(c->sticky), bits_message(c->sticky)) : SOP_OK;
}

sop_status check_device_errors(sop_ctx *c)
{
    if (!c->bound)
        return SOP_OK;
    const sop_status st = fetch(c, {error_range(c)}, [&](int, size_t, size_t, const char *p) { take_errors(c, p); });
    return st != SOP_OK ? st : error_status(c);
}

sop_status need_ready(sop_ctx *c)
{
    if (!c)
        return SOP_E_ARG;
    if (!c->topo)
        return fail(c, SOP_E_STATE, "no topology loaded");
    if (!c->bound)
        return fail(c, SOP_E_STATE, "no workspace bound");
    if (!c->coords)
        return fail(c, SOP_E_STATE, "no coordinates set");
    return SOP_OK;
}

// Plain-schedule list rebuild at step c->step.  The skin is rebuilt first
// when there is no skin, or unless the displacement check of the step before
// left it valid (graph replays capture rebuilds that rely on that check:
// `captured`).
// `filter` false: the step kernel that follows filters the skin rows.
void rebuild(sop_ctx *c, hipStream_t s, bool advance, bool captured = false, bool filter = true)
{
    // in cadence: the step before was a period's last step, which binned its
    // positions and checked their displacements (a rebuild consumes the bins)
    const bool checked = captured || c->skin_checked == c->step;
    const bool binned = captured || c->binned_at == c->step;
    if (skin_check_thr2(c) <= 0.0f || !checked)
        launch_force_skin(c->b, s);
    launch_rebuild(c->b, c->cur, (int)c->n_res, c->cap, c->tile, c->grid, fix_consts(c), list_rc2(c), skin_rs2(c),
                   c->n_traj > 1 ? 1 : 0, s, advance, c->p.list_every, binned, filter);
    if (!captured)
        c->binned_at = -1;
}

// Whether step `step` is the last of a list period: its kernel checks the
// displacements against the skin.
bool checks_skin(const sop_ctx *c, long long step) { return (step + 1) % c->p.list_every == 0; }

// Whether the first step after a rebuild filters the skin rows itself: the
// particle-based step kernel does, unless that step is also the period's
// last (it would clear the cell counts it bins into).
bool fuses_filter(const sop_ctx *c, bool check) { return c->force_mode == SOP_FORCES_PARTICLE && !check; }

// `check`: the last step of a list period, which bins its new positions for
// the next skin search and checks their displacements.
// `first`: the first step after a rebuild launched without its filter,
// which filters the skin rows itself.
void one_step(sop_ctx *c, hipStream_t s, const long long *base, long long off, bool energy, bool check,
              bool first = false)
{
    launch_step(c->b, c->cur, (int)c->n_res, c->cap, c->tile, step_consts(c), fix_consts(c), c->tip,
                c->pulls.empty() ? 0 : 1, energy, 0, base, off, check ? skin_check_thr2(c) : 0.0f, s,
                c->force_mode, ud_kick(c), check ? &c->grid : nullptr, first ? list_rc2(c) : 0.0f,
                c->grid.n_cells);
    if (energy)
        launch_reduce_energy(c->b, c->n_traj, s);
}

// mode 1: one force evaluation; otherwise n_steps steps, recording energies
// only when `records` (a launch whose steps hold a multiple of the energy
// interval).
void batch_launch(sop_ctx *c, hipStream_t s, int n_steps, int stale, int mode, const long long *base,
                  long long off, bool records = false)
{
    launch_batch(c->b, c->cur, n_packs(c), c->batch_wg, c->cap, step_consts(c), fix_consts(c), c->tip,
                 c->pulls.empty() ? 0 : 1, list_rc2(c), c->p.list_every, c->energy_every, n_steps,
                 stale, mode == 1 ? 1 : (records ? 2 : 0), base, off, s,
                 c->re_rep > 0 ? c->b.re_tscale : nullptr);
}

// Last step in [first, first + n) whose energies are recorded, or -1.
long long last_record(const sop_ctx *c, long long first, long long n)
{
    const long long E = c->energy_every;
    if (E <= 0 || n <= 0)
        return -1;
    const long long last = first + n - 1;
    const long long r = last - last % E;
    return r >= first ? r : -1;
}

// Batched schedule: steps one launch may take from `step` on.  A record step
// is a launch of its own where the interval is at least REC_SPLIT: the kernel
// compiled for both kinds of steps takes 20% longer over the others than the
// one without records, a launch more costs about two steps (4,096 chains, us a
// step with launches of both kinds and split: 75.8 and 88.4 at an interval of
// 8, 73.6 and 73.7 at 16, 71.7 and 61.2 at 100; 200 chains 14.8 and 16.5, 14.3
// and 13.9, 14.2 and 11.8).
constexpr long long REC_SPLIT = 16;

long long record_span(const sop_ctx *c, long long step)
{
    const long long E = c->energy_every;
    if (E < REC_SPLIT)
        return INT_MAX;
    return step % E == 0 ? 1 : E - step % E;
}

// Batched schedule: a graph of one persistent launch of batch_steps steps plus
// the device step-counter advance, for layer parity `par`, with or without
// energy records.
sop_status capture_batch_graph(sop_ctx *c, int par, int records)
{
    if (!c->cap_stream)
        HIP_TRY(c, hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking));
    const int saved = c->cur;
    c->cur = par;
    hipGraph_t g = nullptr;
    HIP_TRY(c, hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeRelaxed));
    batch_launch(c, c->cap_stream, c->batch_steps, 0, 0, c->b.step_base, 0, records != 0);
    launch_add_step(c->b.step_base, c->batch_steps, c->cap_stream);
    hipError_t e = hipStreamEndCapture(c->cap_stream, &g);
    c->cur = saved;
    if (e != hipSuccess)
        return hip_fail(c, e, "hipStreamEndCapture");
    hipGraphExec_t ex = nullptr;
    e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess)
        return hip_fail(c, e, "hipGraphInstantiate");
    c->bgraphs[par][records] = ex;
    return SOP_OK;
}

// Plain schedule: from one graph launch to the next the GPU idles about 8 us
// (within a graph not at all), so a context that has replayed its graphs of
// graph_steps list periods LONG_AFTER times makes one of LONG_PERIODS and
// replays that wherever a call has the steps for it: 56 residues 5.85 -> 5.14
// us a step, 4,801 at protein density 11.15 -> 10.17, 75,000 17.4 -> 16.75;
// 25 periods give no more.  Making it (about 120 nodes) costs a context once
// what the first 50 replays of it save, so a context that only runs a few
// hundred steps does not.  Nor does one whose list periods are long: a graph of
// ten periods of 1,000 steps takes 21 ms to make and saves 72 us a replay, and
// an idle 8 us a hundred steps is 2% of the shortest steps.
constexpr int LONG_PERIODS = 10, LONG_AFTER = 64, LONG_STEPS = 128;

// Graphs of graph_steps list periods in one long graph.
int long_factor(const sop_ctx *c)
{
    if (c->graph_steps <= 0)
        return 1;
    const long long span = (long long)c->graph_steps * c->p.list_every;
    return (int)std::max(1LL, std::min<long long>((LONG_PERIODS + c->graph_steps - 1) / c->graph_steps, LONG_STEPS / span));
}

// Capture `periods` list periods (rebuild + list_every steps each) starting at
// layer parity `par`; energies are recorded at the first step when `energy`.
sop_status capture_graph(sop_ctx *c, int par, int energy, int periods, hipGraphExec_t *out)
{
    if (!c->cap_stream)
        HIP_TRY(c, hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking));
    const int saved = c->cur;
    c->cur = par;
    hipGraph_t g = nullptr;
    HIP_TRY(c, hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeRelaxed));
    const bool half_saved = c->ud_half;
    c->ud_half = false;  // graphs start only after the first (half-kick) step
    for (int q = 0; q < periods; ++q) {
        const bool fuse = fuses_filter(c, c->p.list_every == 1);
        rebuild(c, c->cap_stream, true, true, !fuse);
        for (int k = 0; k < c->p.list_every; ++k) {
            one_step(c, c->cap_stream, c->b.step_base, k, energy && q == 0 && k == 0,
                     k == c->p.list_every - 1, fuse && k == 0);
            c->cur ^= 1;
        }
    }
    hipError_t e = hipStreamEndCapture(c->cap_stream, &g);
    c->cur = saved;
    c->ud_half = half_saved;
    if (e != hipSuccess)
        return hip_fail(c, e, "hipStreamEndCapture");
    hipGraphExec_t ex = nullptr;
    e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (e != hipSuccess)
        return hip_fail(c, e, "hipGraphInstantiate");
    *out = ex;
    return SOP_OK;
}

bool valid_pair(const sop_ctx *c, long long i, long long j)
{
    if (i < 0 || j < 0 || i >= c->n_res || j >= c->n_res || i == j)
        return false;
    return c->traj_of[i] == c->traj_of[j];
}

}  // namespace

extern "C" {

const char *sop_status_string(sop_status s)
{
    switch (s) {
    case SOP_OK: return "ok";
    case SOP_E_ARG: return "invalid argument";
    case SOP_E_STATE: return "call out of order";
    case SOP_E_WORKSPACE: return "workspace missing or too small";
    case SOP_E_HIP: return "HIP runtime error";
    case SOP_E_FENE: return "FENE bond broken";
    case SOP_E_LIST_OVERFLOW: return "pair list overflow";
    case SOP_E_NONFINITE: return "non-finite force or position";
    case SOP_E_TIP: return "residue reached the tip surface";
    }
    return "unknown status";
}

const char *sop_last_error(const sop_ctx *c) { return c ? c->last_error.c_str() : "null context"; }

sop_status sop_create(const sop_params *params, void *hip_stream, sop_ctx **out)
{
    if (!params || !out)
        return SOP_E_ARG;
    const sop_params &p = *params;
    const bool ok = p.k_fene > 0 && p.R0 > 0 && p.eps_h >= 0 && p.eps_l >= 0 && p.sigma > 0 &&
                    p.r_list > 0 && p.kBT >= 0 && p.zeta > 0 && p.h > 0 && p.list_every > 0 &&
                    p.list_capacity >= 0 && p.list_capacity <= 1024 && std::isfinite(p.r_list) && std::isfinite(p.h);
    if (!ok)
        return SOP_E_ARG;
    sop_ctx *c = new (std::nothrow) sop_ctx();
    if (!c)
        return SOP_E_ARG;
    c->p = p;
    c->stream = (hipStream_t)hip_stream;
    c->cap_req = p.list_capacity;
    c->cap = list_cap(c);
    *out = c;
    return SOP_OK;
}

sop_status sop_destroy(sop_ctx *c)
{
    if (!c)
        return SOP_E_ARG;
    destroy_graphs(c);
    free_pin(c);
    if (c->cap_stream)
        (void)hipStreamDestroy(c->cap_stream);
    delete c;
    return SOP_OK;
}

sop_status sop_load_topology(sop_ctx *c, int32_t n_traj, const int64_t *res_offsets,
                             const uint32_t *stream_ids, int64_t n_bonds, const int32_t *bonds,
                             const double *bond_r0, int64_t n_native, const int32_t *natives,
                             const double *native_r0, const uint8_t *fixed)
{
    if (!c)
        return SOP_E_ARG;
    if (n_traj <= 0 || !res_offsets || n_bonds < 0 || n_native < 0 ||
        (n_bonds > 0 && (!bonds || !bond_r0)) || (n_native > 0 && (!natives || !native_r0)))
        return fail(c, SOP_E_ARG, "bad topology arguments");
    if (res_offsets[0] != 0)
        return fail(c, SOP_E_ARG, "res_offsets[0] must be 0");
    for (int t = 0; t < n_traj; ++t)
        if (res_offsets[t + 1] < res_offsets[t])
            return fail(c, SOP_E_ARG, "res_offsets must be non-decreasing");
    const long long n = res_offsets[n_traj];
    if (n <= 0 || n >= (1LL << 31) - 64)
        return fail(c, SOP_E_ARG, "residue count out of range");

    c->topo = false;
    c->bound = false;
    c->coords = false;
    destroy_graphs(c);
    c->n_traj = n_traj;
    c->n_res = n;
    c->res_offsets.assign(res_offsets, res_offsets + n_traj + 1);
    c->stream_ids.resize(n_traj);
    for (int t = 0; t < n_traj; ++t)
        c->stream_ids[t] = stream_ids ? stream_ids[t] : (unsigned)t;
    c->traj_of.assign(n, 0);
    c->traj_lo.assign(n, 0);
    c->traj_hi.assign(n, 0);
    c->local.assign(n, 0);
    for (int t = 0; t < n_traj; ++t)
        for (long long i = res_offsets[t]; i < res_offsets[t + 1]; ++i) {
            c->traj_of[i] = t;
            c->traj_lo[i] = (int)res_offsets[t];
            c->traj_hi[i] = (int)res_offsets[t + 1];
            c->local[i] = (int)(i - res_offsets[t]);
        }
    c->fixed.assign(n, 0);
    if (fixed)
        for (long long i = 0; i < n; ++i)
            c->fixed[i] = fixed[i] ? 1 : 0;

    // validate pairs: range, same trajectory, no self/duplicate, r0 > 0
    std::vector<std::pair<long long, int>> keys;  // (i*n + j, kind)
    keys.reserve((size_t)(n_bonds + n_native));
    for (int kind = 0; kind < 2; ++kind) {
        const long long m = kind ? n_native : n_bonds;
        const int32_t *pr = kind ? natives : bonds;
        const double *r0 = kind ? native_r0 : bond_r0;
        for (long long k = 0; k < m; ++k) {
            long long i = pr[2 * k], j = pr[2 * k + 1];
            if (!valid_pair(c, i, j))
                return fail(c, SOP_E_ARG, (kind ? "native " : "bond ") + std::to_string(k) +
                                              ": index out of range, self pair, or pair across trajectories");
            if (!(r0[k] > 0.0) || !std::isfinite(r0[k]))
                return fail(c, SOP_E_ARG, (kind ? "native " : "bond ") + std::to_string(k) + ": r0 <= 0");
            if (i > j)
                std::swap(i, j);
            keys.push_back({i * n + j, kind});
        }
    }
    std::sort(keys.begin(), keys.end());
    for (size_t k = 1; k < keys.size(); ++k)
        if (keys[k].first == keys[k - 1].first)
            return fail(c, SOP_E_ARG, keys[k].second != keys[k - 1].second
                                          ? "a pair is both bonded and native"
                                          : "duplicate pair");

    // per-residue rows: bonds then natives, partners ascending
    std::vector<std::vector<std::pair<int, float>>> rb(n), rn(n);
    for (long long k = 0; k < n_bonds; ++k) {
        int i = bonds[2 * k], j = bonds[2 * k + 1];
        rb[i].push_back({j, (float)bond_r0[k]});
        rb[j].push_back({i, (float)bond_r0[k]});
    }
    for (long long k = 0; k < n_native; ++k) {
        int i = natives[2 * k], j = natives[2 * k + 1];
        rn[i].push_back({j, (float)native_r0[k]});
        rn[j].push_back({i, (float)native_r0[k]});
    }
    c->trow.assign(n, int2{0, 0});
    c->max_bonds = c->max_natives = 0;
    c->tent.clear();
    c->tent.reserve((size_t)(2 * (n_bonds + n_native)));
    for (long long i = 0; i < n; ++i) {
        std::sort(rb[i].begin(), rb[i].end());
        std::sort(rn[i].begin(), rn[i].end());
        c->max_bonds = std::max(c->max_bonds, (int)rb[i].size());
        c->max_natives = std::max(c->max_natives, (int)rn[i].size());
        if (rb[i].size() + rn[i].size() > (size_t)TOPO_CAP)
            return fail(c, SOP_E_ARG, "more than " + std::to_string(TOPO_CAP) +
                                          " bonded and native partners on residue " + std::to_string(i));
        c->trow[i] = int2{(int)c->tent.size(), (int)(rb[i].size() | (rn[i].size() << 12))};
        for (auto &e : rb[i]) {
            int bits = e.first;
            float f;
            std::memcpy(&f, &bits, 4);
            c->tent.push_back(float2{f, e.second});
        }
        for (auto &e : rn[i]) {
            int bits = e.first;
            float f;
            std::memcpy(&f, &bits, 4);
            c->tent.push_back(float2{f, e.second});
        }
    }
    // plain-schedule tiles: consecutive residues, a new tile at a chain start
    // (first residue of a trajectory or not bonded to its predecessor) once
    // the current one is half full, so that tiles stay compact in space
    std::vector<char> chain_start(n, 0);
    for (long long i = 0; i < n; ++i) {
        bool bonded = false;
        for (auto &e : rb[i])
            bonded |= e.first == i - 1;
        chain_start[i] = (i == c->traj_lo[i] || !bonded) ? 1 : 0;
    }
    for (int k = 0; k < 3; ++k) {
        const int T = 64 << k;
        auto &tl = c->tiles[k];
        tl.clear();
        int cnt = 0;
        for (long long i = 0; i < n; ++i) {
            if (cnt == 0 || cnt == T || (chain_start[i] && 2 * cnt >= T)) {
                tl.push_back((int)i);
                cnt = 0;
            }
            ++cnt;
        }
        tl.push_back((int)n);
    }
    // energy-reduction chunks: ECHUNK residues, never across trajectories
    c->chunk_lo.clear();
    c->chunk_first.clear();
    for (int t = 0; t < n_traj; ++t) {
        c->chunk_first.push_back((int)c->chunk_lo.size());
        const long long a0 = res_offsets[t], b0 = res_offsets[t + 1];
        for (long long r = a0; r < b0 || r == a0; r += ECHUNK) {
            c->chunk_lo.push_back((int)r);
            if (b0 == a0)
                break;
        }
    }
    c->chunk_first.push_back((int)c->chunk_lo.size());
    c->chunk_lo.push_back((int)n);
    c->pulls.clear();
    c->pull_slot.assign(n, -1);
    c->tip = TipDev{};
    c->tile = c->tile_req ? c->tile_req : default_tile(n);
    c->min_r0 = 1e300;
    for (long long k = 0; k < n_bonds; ++k)
        c->min_r0 = std::min(c->min_r0, bond_r0[k]);
    for (long long k = 0; k < n_native; ++k)
        c->min_r0 = std::min(c->min_r0, native_r0[k]);
    c->max_len = 0;
    for (int t = 0; t < n_traj; ++t)
        c->max_len = std::max<long long>(c->max_len, res_offsets[t + 1] - res_offsets[t]);
    c->n_cells_cap = (int)std::min<long long>(std::max<long long>(n / 2, 4096), 1LL << 21);
    c->topo = true;
    return SOP_OK;
}

sop_status sop_set_pulling(sop_ctx *c, int32_t traj, int64_t residue, double kappa,
                           const double anchor0[3], const double v[3])
{
    if (!c)
        return SOP_E_ARG;
    if (!c->topo)
        return fail(c, SOP_E_STATE, "load a topology first");
    if (c->bound)
        return fail(c, SOP_E_STATE, "set protocols before binding the workspace");
    if (traj < 0 || traj >= c->n_traj || residue < c->res_offsets[traj] ||
        residue >= c->res_offsets[traj + 1] || !anchor0 || !v || !(kappa >= 0))
        return fail(c, SOP_E_ARG, "bad cantilever arguments");
    if (c->pull_slot[residue] >= 0)
        return fail(c, SOP_E_ARG, "residue already has a cantilever");
    PullDev pd{};
    double vv = 0;
    for (int a = 0; a < 3; ++a) {
        pd.anchor0[a] = anchor0[a];
        pd.v[a] = v[a];
        vv += v[a] * v[a];
    }
    pd.has_dir = vv > 0 ? 1 : 0;
    for (int a = 0; a < 3; ++a)
        pd.vhat[a] = vv > 0 ? v[a] / std::sqrt(vv) : 0.0;
    pd.kappa = kappa;
    pd.residue = (int)residue;
    c->pull_slot[residue] = (int)c->pulls.size();
    c->pulls.push_back(pd);
    return SOP_OK;
}

sop_status sop_set_tip(sop_ctx *c, double radius, double eps, double sigma, const double c0[3],
                       const double v[3])
{
    if (!c)
        return SOP_E_ARG;
    if (!c->topo)
        return fail(c, SOP_E_STATE, "load a topology first");
    if (c->bound)
        return fail(c, SOP_E_STATE, "set protocols before binding the workspace");
    if (radius < 0) {
        c->tip = TipDev{};
        return SOP_OK;
    }
    if (!c0 || !v || !(sigma > 0) || !(eps >= 0))
        return fail(c, SOP_E_ARG, "bad tip arguments");
    TipDev t{};
    double vv = 0;
    for (int a = 0; a < 3; ++a) {
        t.c0[a] = c0[a];
        t.v[a] = v[a];
        vv += v[a] * v[a];
    }
    t.has_dir = vv > 0 ? 1 : 0;
    for (int a = 0; a < 3; ++a)
        t.vhat[a] = vv > 0 ? v[a] / std::sqrt(vv) : 0.0;
    t.radius = radius;
    t.eps = eps;
    t.sigma = sigma;
    t.on = 1;
    c->tip = t;
    return SOP_OK;
}

sop_status sop_set_tile(sop_ctx *c, int32_t tile)
{
    if (!c)
        return SOP_E_ARG;
    if (!(tile == 0 || tile == 64 || tile == 128 || tile == 256))
        return fail(c, SOP_E_ARG, "tile must be 0, 64, 128 or 256 residues");
    c->tile_req = tile;
    if (c->topo) {
        const int nt = tile ? tile : default_tile(c->n_res);
        if (nt != c->tile) {
            c->tile = nt;
            c->list_valid = false;  // the list layout follows the tile size
            c->skin_checked = c->binned_at = -1;
            destroy_graphs(c);
        }
    }
    return SOP_OK;
}

sop_status sop_get_tile(const sop_ctx *c, int32_t *tile)
{
    if (!c || !tile)
        return SOP_E_ARG;
    if (!c->topo)
        return SOP_E_STATE;
    *tile = c->tile;
    return SOP_OK;
}

sop_status sop_set_schedule(sop_ctx *c, int32_t schedule)
{
    if (!c)
        return SOP_E_ARG;
    if (schedule != SOP_SCHEDULE_PLAIN && schedule != SOP_SCHEDULE_BATCHED)
        return fail(c, SOP_E_ARG, "unknown schedule");
    if (c->bound)
        return fail(c, SOP_E_STATE, "set the schedule before binding the workspace");
    c->schedule = schedule;
    c->cap = list_cap(c);
    return SOP_OK;
}

sop_status sop_set_batch(sop_ctx *c, int32_t wg, int32_t steps)
{
    if (!c)
        return SOP_E_ARG;
    if (!(wg == 0 || wg == 256 || wg == 512 || wg == 1024) || steps < 1)
        return fail(c, SOP_E_ARG, "workgroup residues must be 0, 256, 512 or 1024 and steps >= 1");
    if (c->topo && wg && wg < c->max_len)
        return fail(c, SOP_E_ARG, "workgroup smaller than the longest trajectory");
    c->batch_wg_req = wg;
    c->batch_steps = steps;
    for (auto &gp : c->bgraphs)
        for (auto &g : gp)
            if (g) {
                (void)hipGraphExecDestroy(g);
                g = nullptr;
            }
    if (c->bound && c->schedule == SOP_SCHEDULE_BATCHED) {
        c->batch_wg = pick_batch_wg(c);
        make_packs(c);
        const sop_status st = upload_packs(c);
        if (st != SOP_OK)
            return st;
        c->list_valid = false;  // the list layout follows the packs
    }
    return SOP_OK;
}

sop_status sop_get_batch(const sop_ctx *c, int32_t *wg, int32_t *steps, int32_t *np)
{
    if (!c)
        return SOP_E_ARG;
    if (wg)
        *wg = c->bound ? c->batch_wg : pick_batch_wg(c);
    if (steps)
        *steps = c->batch_steps;
    if (np)
        *np = c->bound ? n_packs(c) : 0;
    return SOP_OK;
}

sop_status sop_set_force_mode(sop_ctx *c, int32_t mode)
{
    if (!c || (mode != SOP_FORCES_PARTICLE && mode != SOP_FORCES_PAIR))
        return SOP_E_ARG;
    if (mode != c->force_mode) {
        c->force_mode = mode;
        destroy_graphs(c);  // the graphs hold the kernels of the old mode
    }
    return SOP_OK;
}

sop_status sop_get_force_mode(const sop_ctx *c, int32_t *mode)
{
    if (!c || !mode)
        return SOP_E_ARG;
    *mode = c->force_mode;
    return SOP_OK;
}

sop_status sop_set_integrator(sop_ctx *c, int32_t kind, double mass)
{
    if (!c || (kind != SOP_INTEGRATOR_OVERDAMPED && kind != SOP_INTEGRATOR_UNDERDAMPED))
        return SOP_E_ARG;
    if (kind == SOP_INTEGRATOR_UNDERDAMPED && !(mass > 0.0 && std::isfinite(mass)))
        return fail(c, SOP_E_ARG, "the mass must be positive and finite");
    if (kind == SOP_INTEGRATOR_UNDERDAMPED && c->schedule != SOP_SCHEDULE_PLAIN)
        return fail(c, SOP_E_STATE, "the underdamped integrator runs on the plain schedule");
    const double scale = fix_consts(c).scale;
    c->integrator = kind;
    if (kind == SOP_INTEGRATOR_UNDERDAMPED)
        c->mass = mass;
    c->ud_half = true;
    if (c->bound && c->coords && c->schedule == SOP_SCHEDULE_PLAIN && fix_consts(c).scale != scale) {
        // the copies are in another unit: binned (and copied) anew before the
        // next rebuild, and not read until then
        c->binned_at = -1;
        launch_distrust_copies(c->b, c->cur, c->stream);
        HIP_TRY(c, hipGetLastError());
    }
    destroy_graphs(c);  // the integrator's constants are kernel arguments
    return SOP_OK;
}

sop_status sop_set_velocities(sop_ctx *c, const double *v)
{
    sop_status st = need_ready(c);
    if (st != SOP_OK)
        return st;
    if (!v)
        return fail(c, SOP_E_ARG, "null velocities");
    if (c->schedule != SOP_SCHEDULE_PLAIN)
        return fail(c, SOP_E_STATE, "velocities belong to the plain schedule");
    const long long n = c->n_res;
    std::vector<float4> vv(n);
    for (long long i = 0; i < n; ++i) {
        for (int a = 0; a < 3; ++a)
            if (!std::isfinite(v[3 * i + a]))
                return fail(c, SOP_E_ARG, "non-finite velocity");
        vv[i] = c->fixed[i] ? float4{0.f, 0.f, 0.f, 0.f}
                            : float4{(float)v[3 * i], (float)v[3 * i + 1], (float)v[3 * i + 2], 0.f};
    }
    HIP_TRY(c, hipMemcpyAsync(c->b.vel, vv.data(), n * sizeof(float4), hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    c->ud_half = true;
    return SOP_OK;
}

sop_status sop_get_velocities(sop_ctx *c, double *v)
{
    sop_status st = need_ready(c);
    if (st != SOP_OK)
        return st;
    if (!v)
        return fail(c, SOP_E_ARG, "null output");
    if (c->schedule != SOP_SCHEDULE_PLAIN)
        return fail(c, SOP_E_STATE, "velocities belong to the plain schedule");
    const size_t n = (size_t)c->n_res;
    const bool add_kick = c->integrator == SOP_INTEGRATOR_UNDERDAMPED && !c->ud_half;
    if (add_kick) {
        // the stored velocities lack the last half kick, whose force is this step's
        if (!c->list_valid || c->step % c->p.list_every == 0)
            rebuild(c, c->stream, false);
        c->list_valid = true;
        launch_step(c->b, c->cur, (int)c->n_res, c->cap, c->tile, step_consts(c), fix_consts(c), c->tip,
                    c->pulls.empty() ? 0 : 1, false, 1, nullptr, c->step, 0.0f, c->stream, c->force_mode);
        HIP_TRY(c, hipGetLastError());
    }
    const double hk = add_kick ? 0.5 * c->p.h / c->mass : 0.0;
    st = fetch(c, {error_range(c), {c->b.vel, n * sizeof(float4)}, {c->b.fout, add_kick ? n * sizeof(float4) : 0}},
               [&](int k, size_t off, size_t bytes, const char *p) {
                   if (k == 0)
                       return take_errors(c, p);
                   if (add_kick && c->sticky)
                       return;
                   const float4 *w = reinterpret_cast<const float4 *>(p);
                   const size_t i0 = off / sizeof(float4), m = bytes / sizeof(float4);
                   for (size_t u = 0; u < m; ++u) {
                       double *o = v + 3 * (i0 + u);
                       if (c->fixed[i0 + u]) {
                           o[0] = o[1] = o[2] = 0.0;
                       } else if (k == 1) {
                           o[0] = (double)w[u].x;
                           o[1] = (double)w[u].y;
                           o[2] = (double)w[u].z;
                       } else {
                           o[0] += hk * (double)w[u].x;
                           o[1] += hk * (double)w[u].y;
                           o[2] += hk * (double)w[u].z;
                       }
                   }
               });
    return st != SOP_OK ? st : error_status(c);
}

sop_status sop_set_tempering(sop_ctx *c, int32_t n_rep, const double *kbt, int64_t exchange_every,
                             const int32_t *tidx)
{
    if (!c)
        return SOP_E_ARG;
    if (c->schedule != SOP_SCHEDULE_BATCHED || !c->bound)
        return fail(c, SOP_E_STATE, "replica exchange runs on a bound batched schedule");
    if (n_rep < 1 || !kbt || exchange_every < 0 || c->n_traj % n_rep != 0)
        return fail(c, SOP_E_ARG, "n_rep must divide the trajectory count; exchange_every >= 0");
    for (int k = 0; k < n_rep; ++k)
        if (!(kbt[k] > 0.0) || !std::isfinite(kbt[k]))
            return fail(c, SOP_E_ARG, "temperatures must be positive");
    const int T = c->n_traj;
    std::vector<int> ti(T);
    std::vector<float> ts(T);
    for (int t = 0; t < T; ++t)
        ti[t] = tidx ? tidx[t] : t % n_rep;
    for (int g = 0; g < T / n_rep; ++g) {  // each group a permutation of 0..n_rep-1
        std::vector<char> seen(n_rep, 0);
        for (int m = 0; m < n_rep; ++m) {
            const int v = ti[g * n_rep + m];
            if (v < 0 || v >= n_rep || seen[v])
                return fail(c, SOP_E_ARG, "temperature indices are not a permutation in each group");
            seen[v] = 1;
        }
    }
    for (int t = 0; t < T; ++t)
        ts[t] = (float)std::sqrt(kbt[ti[t]] / c->p.kBT);
    c->re_rep = n_rep;
    c->re_kbt.assign(kbt, kbt + n_rep);
    c->re_every = exchange_every;
    c->re_last = -1;
    hipStream_t s = c->stream;
    HIP_TRY(c, hipMemcpyAsync(c->b.re_kbt, kbt, n_rep * sizeof(double), hipMemcpyHostToDevice, s));
    HIP_TRY(c, hipMemcpyAsync(c->b.re_tidx, ti.data(), T * sizeof(int), hipMemcpyHostToDevice, s));
    HIP_TRY(c, hipMemcpyAsync(c->b.re_tscale, ts.data(), T * sizeof(float), hipMemcpyHostToDevice, s));
    HIP_TRY(c, hipMemsetAsync(c->b.re_stats, 0, 2 * (size_t)T * sizeof(unsigned long long), s));
    HIP_TRY(c, hipStreamSynchronize(s));
    destroy_graphs(c);
    return SOP_OK;
}

sop_status sop_get_tempering(sop_ctx *c, int32_t *tidx, int64_t *accepted, int64_t *attempted)
{
    sop_status st = need_ready(c);
    if (st != SOP_OK)
        return st;
    if (c->re_rep < 1)
        return fail(c, SOP_E_STATE, "no replica exchange set");
    const size_t T = (size_t)c->n_traj;
    const int R = c->re_rep;
    std::vector<unsigned long long> stv(2 * T);
    st = fetch(c, {error_range(c), {c->b.re_stats, 2 * T * sizeof(unsigned long long)},
                   {c->b.re_tidx, tidx ? T * sizeof(int) : 0}},
               [&](int k, size_t off, size_t bytes, const char *p) {
                   if (k == 0)
                       take_errors(c, p);
                   else
                       std::memcpy((k == 1 ? reinterpret_cast<char *>(stv.data()) : reinterpret_cast<char *>(tidx)) + off,
                                   p, bytes);
               });
    if (st != SOP_OK)
        return st;
    for (int k = 0; k + 1 < R; ++k) {
        if (accepted)
            accepted[k] = (int64_t)stv[2 * k];
        if (attempted)
            attempted[k] = (int64_t)stv[2 * k + 1];
    }
    return error_status(c);
}

sop_status sop_set_list_skin(sop_ctx *c, double skin)
{
    if (!c || !(skin >= 0.0) || !std::isfinite(skin) || skin > 4.0 * c->p.r_list)
        return SOP_E_ARG;
    if (skin == c->skin)
        return SOP_OK;
    c->skin = skin;
    c->list_valid = false;
    c->skin_checked = c->binned_at = -1;
    destroy_graphs(c);  // the radius, the cell grid and the check are kernel arguments
    if (c->coords)
        set_grid(c, c->xyz_set.data());  // the cell edge follows the skin radius
    if (c->bound && c->coords)
        HIP_TRY(c, hipMemcpyAsync(c->b.traj_cell, c->traj_cell.data(), c->n_traj * sizeof(int4),
                                  hipMemcpyHostToDevice, c->stream));
    return SOP_OK;
}

sop_status sop_get_list_skin(const sop_ctx *c, double *skin)
{
    if (!c || !skin)
        return SOP_E_ARG;
    *skin = c->skin;
    return SOP_OK;
}

sop_status sop_get_list_stats(sop_ctx *c, int64_t *rebuilds, int64_t *skin_builds)
{
    sop_status st = need_ready(c);
    if (st != SOP_OK)
        return st;
    unsigned long long v[2] = {0, 0};
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    HIP_TRY(c, hipMemcpy(v, c->b.list_stats, sizeof(v), hipMemcpyDeviceToHost));
    if (rebuilds)
        *rebuilds = (int64_t)v[0];
    if (skin_builds)
        *skin_builds = (int64_t)v[1];
    return SOP_OK;
}

sop_status sop_set_graph_steps(sop_ctx *c, int32_t k)
{
    if (!c || k < 0)
        return SOP_E_ARG;
    if (k != c->graph_steps)
        destroy_graphs(c);  // captured graphs hold the old span
    c->graph_steps = k;
    return SOP_OK;
}

sop_status sop_set_energy_interval(sop_ctx *c, int64_t k)
{
    if (!c || k < 0)
        return SOP_E_ARG;
    if (k != c->energy_every)
        destroy_graphs(c);  // batched graphs hold the interval as a kernel argument
    c->energy_every = k;
    return SOP_OK;
}

sop_status sop_workspace_size(const sop_ctx *c, size_t *bytes)
{
    if (!c || !bytes)
        return SOP_E_ARG;
    if (!c->topo)
        return SOP_E_STATE;
    *bytes = layout(c, nullptr, nullptr);
    return SOP_OK;
}

sop_status sop_bind_workspace(sop_ctx *c, void *dev, size_t bytes)
{
    if (!c)
        return SOP_E_ARG;
    if (!c->topo)
        return fail(c, SOP_E_STATE, "load a topology first");
    const size_t need = layout(c, nullptr, nullptr);
    if (!dev || ((uintptr_t)dev & 255) || bytes < need)
        return fail(c, SOP_E_WORKSPACE, "workspace null, not 256-byte aligned, or smaller than " +
                                            std::to_string(need) + " bytes");
    if (c->schedule == SOP_SCHEDULE_BATCHED && c->max_len > 1024)
        return fail(c, SOP_E_ARG, "the batched schedule holds trajectories of at most 1024 residues");
    destroy_graphs(c);
    c->bound = false;
    c->coords = false;
    c->list_valid = false;
    c->ws = dev;
    c->ws_bytes = bytes;
    layout(c, (char *)dev, &c->b);
    const sop_status pinned = make_pin(c);
    if (pinned != SOP_OK)
        return pinned;
    if (c->schedule == SOP_SCHEDULE_BATCHED) {
        c->batch_wg = pick_batch_wg(c);
        if (c->batch_wg < c->max_len)
            return fail(c, SOP_E_ARG, "batch workgroup smaller than the longest trajectory");
        make_packs(c);
        const sop_status st = upload_packs(c);
        if (st != SOP_OK)
            return st;
    }
    const DevBufs &b = c->b;
    const size_t n = (size_t)c->n_res;
    hipStream_t s = c->stream;
    HIP_TRY(c, hipMemcpyAsync(b.trow, c->trow.data(), n * sizeof(int2), hipMemcpyHostToDevice, s));
    if (!c->tent.empty())
        HIP_TRY(c, hipMemcpyAsync(b.tent, c->tent.data(), c->tent.size() * sizeof(float2),
                                  hipMemcpyHostToDevice, s));
    HIP_TRY(c, hipMemcpyAsync(b.traj_lo, c->traj_lo.data(), n * sizeof(int), hipMemcpyHostToDevice, s));
    HIP_TRY(c, hipMemcpyAsync(b.traj_hi, c->traj_hi.data(), n * sizeof(int), hipMemcpyHostToDevice, s));
    HIP_TRY(c, hipMemcpyAsync(b.pull_slot, c->pull_slot.data(), n * sizeof(int), hipMemcpyHostToDevice, s));
    if (!c->pulls.empty())
        HIP_TRY(c, hipMemcpyAsync(b.pulls, c->pulls.data(), c->pulls.size() * sizeof(PullDev),
                                  hipMemcpyHostToDevice, s));
    HIP_TRY(c, hipMemcpyAsync(b.stream_ids, c->stream_ids.data(), c->n_traj * sizeof(unsigned),
                              hipMemcpyHostToDevice, s));
    {
        std::vector<uint2> key(n);
        for (size_t i = 0; i < n; ++i) {
            key[i].x = (unsigned)c->local[i] | (c->fixed[i] ? 0x80000000u : 0u);
            key[i].y = c->stream_ids[c->traj_of[i]];
        }
        HIP_TRY(c, hipMemcpy(b.noise_key, key.data(), n * sizeof(uint2), hipMemcpyHostToDevice));
    }
    HIP_TRY(c, hipMemcpyAsync(b.res_offsets, c->res_offsets.data(), (c->n_traj + 1) * sizeof(long long),
                              hipMemcpyHostToDevice, s));
    HIP_TRY(c, hipMemsetAsync(b.list_cnt, 0, n * sizeof(int), s));
    if (c->schedule == SOP_SCHEDULE_PLAIN) {
        size_t n_tiles_max = 0;
        for (int k = 0; k < 3; ++k) {
            const size_t nt = c->tiles[k].size() - 1;
            n_tiles_max = std::max(n_tiles_max, nt);
            HIP_TRY(c, hipMemcpyAsync(b.tile_first[k], c->tiles[k].data(), c->tiles[k].size() * sizeof(int),
                                      hipMemcpyHostToDevice, s));
        }
        HIP_TRY(c, hipMemsetAsync(b.tile_top, 0, n_tiles_max * sizeof(int4), s));
        HIP_TRY(c, hipMemsetAsync(b.err + MOVED, 0, 2 * sizeof(unsigned), s));
        HIP_TRY(c, hipMemsetAsync(b.cell_count, 0, (size_t)c->n_cells_cap * sizeof(int), s));
        HIP_TRY(c, hipMemsetAsync(b.facc, 0, n * sizeof(float4), s));
        HIP_TRY(c, hipMemsetAsync(b.vel, 0, n * sizeof(float4), s));
        HIP_TRY(c, hipMemsetAsync(b.skin_ord, 0, n_tiles_max * 256 * sizeof(unsigned short), s));
        HIP_TRY(c, hipMemsetAsync(b.eacc, 0, n * sizeof(double4), s));
        HIP_TRY(c, hipMemsetAsync(b.stage_cnt, 0, n_tiles_max * sizeof(int), s));
    }
    HIP_TRY(c, hipMemsetAsync(b.res_energy, 0, n * RES_E * sizeof(double), s));
    HIP_TRY(c, hipMemcpyAsync(b.chunk_lo, c->chunk_lo.data(), c->chunk_lo.size() * sizeof(int),
                              hipMemcpyHostToDevice, s));
    HIP_TRY(c, hipMemcpyAsync(b.chunk_first, c->chunk_first.data(), c->chunk_first.size() * sizeof(int),
                              hipMemcpyHostToDevice, s));
    HIP_TRY(c, hipMemsetAsync(b.energy, 0, (size_t)c->n_traj * SOP_NTERMS * sizeof(double), s));
    HIP_TRY(c, hipMemsetAsync(b.f_ext, 0, (size_t)c->n_traj * sizeof(double), s));
    HIP_TRY(c, hipMemsetAsync(b.err, 0, sizeof(unsigned), s));
    HIP_TRY(c, hipMemsetAsync(b.skin_flag, 0, sizeof(unsigned), s));
    HIP_TRY(c, hipMemsetAsync(b.list_stats, 0, 2 * sizeof(unsigned long long), s));
    HIP_TRY(c, hipStreamSynchronize(s));
    c->skin_checked = c->binned_at = -1;
    c->bound = true;
    c->sticky = 0;
    c->energy_step = -1;
    return SOP_OK;
}

sop_status sop_set_coordinates(sop_ctx *c, const double *xyz)
{
    if (!c || !xyz)
        return SOP_E_ARG;
    if (!c->topo || !c->bound)
        return fail(c, SOP_E_STATE, "load a topology and bind a workspace first");
    const long long n = c->n_res;
    for (long long k = 0; k < 3 * n; ++k)
        if (!std::isfinite(xyz[k]))
            return fail(c, SOP_E_ARG, "non-finite coordinate");
    c->xyz_set.assign(xyz, xyz + 3 * n);
    set_grid(c, xyz);
    destroy_graphs(c);  // the grid is a kernel argument of captured rebuilds
    hipStream_t s = c->stream;
    // {hi, tag}, {lo, trajectory} of a piece of the residues in one half of the
    // host memory while the piece before is on its way from the other
    const long long piece = (long long)(c->pin_half / (2 * sizeof(float4)));
    for (long long i0 = 0, h = 0; i0 < n; i0 += piece, h ^= 1) {
        const long long m = std::min(piece, n - i0);
        float4 *pv = reinterpret_cast<float4 *>(c->pin + h * c->pin_half);
        for (long long u = 0; u < m; ++u) {
            const double *x = xyz + 3 * (i0 + u);
            const unsigned tag = (unsigned)c->local[i0 + u] | (c->fixed[i0 + u] ? 0x80000000u : 0u);
            const int tr = c->traj_of[i0 + u];
            float tw, lw;
            std::memcpy(&tw, &tag, 4);
            std::memcpy(&lw, &tr, 4);
            const float4 hi{(float)x[0], (float)x[1], (float)x[2], tw};
            pv[2 * u] = hi;
            pv[2 * u + 1] = float4{(float)(x[0] - (double)hi.x), (float)(x[1] - (double)hi.y),
                                   (float)(x[2] - (double)hi.z), lw};
        }
        if (i0 > 0)
            HIP_TRY(c, hipStreamSynchronize(s));
        HIP_TRY(c, hipMemcpyAsync(c->b.pos[0] + 2 * i0, pv, 2 * m * sizeof(float4), hipMemcpyHostToDevice, s));
    }
    HIP_TRY(c, hipMemcpyAsync(c->b.pos[1], c->b.pos[0], 2 * n * sizeof(float4), hipMemcpyDeviceToDevice, s));
    HIP_TRY(c, hipMemcpyAsync(c->b.traj_cell, c->traj_cell.data(), c->n_traj * sizeof(int4),
                              hipMemcpyHostToDevice, s));
    HIP_TRY(c, hipMemsetAsync(c->b.err, 0, sizeof(unsigned), s));
    if (c->schedule == SOP_SCHEDULE_PLAIN)
        HIP_TRY(c, hipMemsetAsync(c->b.vel, 0, n * sizeof(float4), s));  // new coordinates, zero velocities
    HIP_TRY(c, hipStreamSynchronize(s));
    c->ud_half = true;
    c->cur = 0;
    c->sticky = 0;
    c->coords = true;
    c->list_valid = false;
    c->skin_checked = c->binned_at = -1;
    c->last_error.clear();
    return SOP_OK;
}

sop_status sop_get_coordinates(sop_ctx *c, double *xyz)
{
    sop_status st = need_ready(c);
    if (st != SOP_OK)
        return st;
    if (!xyz)
        return fail(c, SOP_E_ARG, "null output");
    st = fetch(c, {error_range(c), {c->b.pos[c->cur], 2 * (size_t)c->n_res * sizeof(float4)}},
               [&](int k, size_t off, size_t bytes, const char *p) {
                   if (k == 0)
                       return take_errors(c, p);
                   const float4 *w = reinterpret_cast<const float4 *>(p);
                   double *o = xyz + 3 * (off / (2 * sizeof(float4)));
                   for (size_t u = 0; u < bytes / (2 * sizeof(float4)); ++u) {
                       o[3 * u + 0] = (double)w[2 * u].x + (double)w[2 * u + 1].x;
                       o[3 * u + 1] = (double)w[2 * u].y + (double)w[2 * u + 1].y;
                       o[3 * u + 2] = (double)w[2 * u].z + (double)w[2 * u + 1].z;
                   }
               });
    return st != SOP_OK ? st : error_status(c);
}

sop_status sop_set_step(sop_ctx *c, int64_t step)
{
    if (!c || step < 0)
        return SOP_E_ARG;
    c->step = step;
    c->list_valid = false;
    c->skin_checked = c->binned_at = -1;
    return SOP_OK;
}

sop_status sop_get_step(const sop_ctx *c, int64_t *step)
{
    if (!c || !step)
        return SOP_E_ARG;
    *step = c->step;
    return SOP_OK;
}

sop_status sop_build_pairlist(sop_ctx *c)
{
    sop_status st = need_ready(c);
    if (st != SOP_OK)
        return st;
    if (c->schedule == SOP_SCHEDULE_BATCHED)
        batch_launch(c, c->stream, 1, 1, 1, nullptr, c->step);  // rebuild + one force evaluation
    else
        rebuild(c, c->stream, false);
    HIP_TRY(c, hipGetLastError());
    c->list_valid = true;
    return SOP_OK;
}

sop_status sop_get_pairlist(sop_ctx *c, int64_t cap, int32_t *ij, int64_t *n_pairs)
{
    sop_status st = need_ready(c);
    if (st != SOP_OK)
        return st;
    if (!n_pairs || cap < 0 || (cap > 0 && !ij))
        return fail(c, SOP_E_ARG, "bad pairlist arguments");
    if (!c->list_valid)
        return fail(c, SOP_E_STATE, "no list built since the coordinates were set");
    st = check_device_errors(c);
    if (st != SOP_OK)
        return st;
    const long long n = c->n_res;
    std::vector<std::pair<int, int>> pairs;
    if (c->schedule == SOP_SCHEDULE_BATCHED) {
        std::vector<int> cnt(n);
        HIP_TRY(c, hipMemcpy(cnt.data(), c->b.list_cnt, n * sizeof(int), hipMemcpyDeviceToHost));
        std::vector<unsigned short> list((size_t)n * c->cap);
        HIP_TRY(c, hipMemcpy(list.data(), c->b.list16, list.size() * sizeof(unsigned short),
                             hipMemcpyDeviceToHost));
        // rows hold local slots of the residue's pack
        for (int pk = 0; pk < n_packs(c); ++pk) {
            const int off = c->pack_off[pk], m = c->pack_off[pk + 1] - off;
            for (int t = 0; t < m; ++t) {
                const int i = c->slot_res[off + t];
                for (int k = 0; k < std::min(cnt[i], c->cap); ++k) {
                    const int sl = list[(size_t)i * c->cap + k] >> 4;
                    if (sl >= m)
                        return fail(c, SOP_E_LIST_OVERFLOW, "list entry outside its pack");
                    const int j = c->slot_res[off + sl];
                    if (i < j)
                        pairs.push_back({i, j});
                }
            }
        }
    } else {
        // rows hold slots of their tile, in lane order; the tile's stage maps slots to ids
        const int T = c->tile, SM = STAGE_MAX;
        const auto &tl = c->tiles[tile_index(T)];
        const int n_tiles = (int)tl.size() - 1, nl = lanes_for(T, n_tiles), W = T * nl / 256;
        const int chunks = lane_chunks(c->cap, nl);
        std::vector<unsigned short> list((size_t)n_tiles * W * chunks * 1024);
        std::vector<unsigned short> llen((size_t)n_tiles * W * 256);
        std::vector<unsigned char> grho((size_t)n_tiles * T);
        std::vector<int> stage(n_tiles * (size_t)SM), stage_cnt(n_tiles);
        HIP_TRY(c, hipMemcpy(list.data(), c->b.flist16, list.size() * sizeof(unsigned short),
                             hipMemcpyDeviceToHost));
        HIP_TRY(c, hipMemcpy(llen.data(), c->b.llen, llen.size() * sizeof(unsigned short), hipMemcpyDeviceToHost));
        HIP_TRY(c, hipMemcpy(grho.data(), c->b.grho, grho.size(), hipMemcpyDeviceToHost));
        HIP_TRY(c, hipMemcpy(stage.data(), c->b.stage, stage.size() * sizeof(int), hipMemcpyDeviceToHost));
        HIP_TRY(c, hipMemcpy(stage_cnt.data(), c->b.stage_cnt, n_tiles * sizeof(int), hipMemcpyDeviceToHost));
        for (int tile = 0; tile < n_tiles; ++tile)
            for (int w = 0; w < W; ++w)
                for (int lane = 0; lane < 256; ++lane) {
                    const int wg = tile * W + w;
                    const int i = tl[tile] + grho[(size_t)wg * (256 / nl) + lane / nl];
                    for (int k = 0; k < std::min((int)llen[(size_t)wg * 256 + lane], 4 * chunks); ++k) {
                        const int sl = list[chunk_index(wg, k / 4, lane, chunks) * 4 + k % 4] >> 2;
                        if (sl >= stage_cnt[tile])
                            return fail(c, SOP_E_LIST_OVERFLOW, "list entry outside its tile's staging set");
                        const int j = stage[(size_t)tile * SM + sl];
                        if (i < j)
                            pairs.push_back({i, j});
                    }
                }
    }
    std::sort(pairs.begin(), pairs.end());
    *n_pairs = (int64_t)pairs.size();
    if ((int64_t)pairs.size() > cap)
        return fail(c, SOP_E_ARG, "output capacity too small");
    for (size_t k = 0; k < pairs.size(); ++k) {
        ij[2 * k] = pairs[k].first;
        ij[2 * k + 1] = pairs[k].second;
    }
    return SOP_OK;
}

sop_status sop_compute_forces(sop_ctx *c, double *f, double *energies, double *f_ext)
{
    sop_status st = need_ready(c);
    if (st != SOP_OK)
        return st;
    const bool stale = !c->list_valid || c->step % c->p.list_every == 0;
    if (c->schedule == SOP_SCHEDULE_BATCHED) {
        batch_launch(c, c->stream, 1, stale ? 1 : 0, 1, nullptr, c->step);
    } else {
        if (stale)
            rebuild(c, c->stream, false);
        launch_step(c->b, c->cur, (int)c->n_res, c->cap, c->tile, step_consts(c), fix_consts(c), c->tip,
                    c->pulls.empty() ? 0 : 1, true, 1, nullptr, c->step, 0.0f, c->stream, c->force_mode);
        launch_reduce_energy(c->b, c->n_traj, c->stream);
    }
    c->list_valid = true;
    HIP_TRY(c, hipGetLastError());
    const size_t n = (size_t)c->n_res, T = (size_t)c->n_traj;
    st = fetch(c, {error_range(c), {c->b.fout, f ? n * sizeof(float4) : 0},
                   {c->b.energy, energies ? T * SOP_NTERMS * sizeof(double) : 0},
                   {c->b.f_ext, f_ext ? T * sizeof(double) : 0}},
               [&](int k, size_t off, size_t bytes, const char *p) {
                   if (k == 0)
                       return take_errors(c, p);
                   if (c->sticky)
                       return;
                   if (k > 1) {
                       std::memcpy(reinterpret_cast<char *>(k == 2 ? energies : f_ext) + off, p, bytes);
                       return;
                   }
                   const float4 *w = reinterpret_cast<const float4 *>(p);
                   double *o = f + 3 * (off / sizeof(float4));
                   for (size_t u = 0; u < bytes / sizeof(float4); ++u) {
                       o[3 * u] = w[u].x;
                       o[3 * u + 1] = w[u].y;
                       o[3 * u + 2] = w[u].z;
                   }
               });
    if (st == SOP_OK)
        st = error_status(c);
    if (st == SOP_OK)
        c->energy_step = c->step;
    return st;
}

sop_status sop_step(sop_ctx *c, int64_t n_steps)
{
    sop_status st = need_ready(c);
    if (st != SOP_OK)
        return st;
    if (n_steps < 0)
        return fail(c, SOP_E_ARG, "negative step count");
    if (c->sticky)
        return fail(c, status_from_bits(c->sticky), bits_message(c->sticky));
    if (c->schedule == SOP_SCHEDULE_BATCHED) {
        const long long K = c->batch_steps;
        const long long X = c->re_rep > 1 ? c->re_every : 0;
        bool base_set = false;
        long long q = 0;
        while (q < n_steps) {
            if (X > 0 && c->step % X == 0 && c->re_last != c->step) {
                // replica exchange before this step's update: energies of
                // the current positions, then one round of swaps
                batch_launch(c, c->stream, 1, c->list_valid ? 0 : 1, 1, nullptr, c->step);
                c->list_valid = true;
                c->energy_step = c->step;
                launch_exchange(c->b, c->re_rep, (int)(c->n_traj / c->re_rep), c->p.kBT, c->step / X,
                                (unsigned)(c->p.seed & 0xffffffffu), (unsigned)(c->p.seed >> 32), c->stream);
                c->re_last = c->step;
                base_set = false;
            }
            long long k = std::min<long long>(K, n_steps - q);
            if (X > 0)
                k = std::min<long long>(k, X - c->step % X);  // stop at the next exchange
            k = std::min<long long>(k, record_span(c, c->step));
            const long long rec = last_record(c, c->step, k);
            if (c->graph_steps > 0 && c->list_valid && k == K && X == 0) {
                const int rg = rec >= 0 ? 1 : 0;
                if (!c->bgraphs[c->cur][rg]) {
                    st = capture_batch_graph(c, c->cur, rg);
                    if (st != SOP_OK)
                        return st;
                }
                if (!base_set) {
                    launch_set_step(c->b.step_base, c->step, c->stream);
                    base_set = true;
                }
                HIP_TRY(c, hipGraphLaunch(c->bgraphs[c->cur][rg], c->stream));
            } else {
                batch_launch(c, c->stream, (int)k, c->list_valid ? 0 : 1, 0, nullptr, c->step, rec >= 0);
                base_set = false;
            }
            if (rec >= 0)
                c->energy_step = rec;
            c->list_valid = true;
            c->cur ^= 1;
            c->step += k;
            q += k;
        }
        HIP_TRY(c, hipGetLastError());
        return SOP_OK;
    }
    const int L = c->p.list_every;
    const long long E = c->energy_every;
    const long long span = (long long)L * std::max(c->graph_steps, 1);
    // graphs replay whole list periods and record energies only at their
    // first step: with an energy interval (a multiple of the span) a graph
    // starts only on a multiple of the span, so no record step falls inside
    const bool graphs_ok = c->graph_steps > 0 && (E == 0 || E % span == 0);
    const long long align = E > 0 ? span : L;
    bool base_set = false;
    long long q = 0;
    while (q < n_steps) {
        if (graphs_ok && c->step % align == 0 && n_steps - q >= span &&
            !(c->integrator == SOP_INTEGRATOR_UNDERDAMPED && c->ud_half)) {
            const int en = (E > 0 && c->step % E == 0) ? 1 : 0;
            const int m = long_factor(c);
            const bool lng = m > 1 && c->graph_runs >= LONG_AFTER && n_steps - q >= m * span &&
                             (E == 0 || E - c->step % E >= m * span);
            const long long run = lng ? m * span : span;
            hipGraphExec_t &ex = (lng ? c->long_graphs : c->graphs)[c->cur][en];
            if (!ex) {
                st = capture_graph(c, c->cur, en, (lng ? m : 1) * c->graph_steps, &ex);
                if (st != SOP_OK)
                    return st;
            }
            if (c->graph_runs < LONG_AFTER)
                ++c->graph_runs;
            if (!base_set) {
                launch_set_step(c->b.step_next, c->step, c->stream);
                base_set = true;
            }
            // the graph's first rebuild relies on the cells holding the
            // current positions and on the displacement check
            if (c->binned_at != c->step)
                launch_bin_all(c->b, c->cur, (int)c->n_res, c->grid, fix_consts(c), c->stream);
            if (c->skin_checked != c->step)
                launch_force_skin(c->b, c->stream);
            HIP_TRY(c, hipGraphLaunch(ex, c->stream));
            if (en)
                c->energy_step = c->step;
            c->list_valid = true;
            c->step += run;
            c->skin_checked = c->binned_at = c->step;
            if (run & 1)
                c->cur ^= 1;
            q += run;
            continue;
        }
        const bool en = E > 0 && c->step % E == 0;
        const bool chk = checks_skin(c, c->step);
        bool fused = false;
        if (!c->list_valid || c->step % L == 0) {
            fused = fuses_filter(c, chk);
            rebuild(c, c->stream, false, false, !fused);
            c->list_valid = true;
        }
        one_step(c, c->stream, nullptr, c->step, en, chk, fused);
        c->ud_half = false;
        if (en)
            c->energy_step = c->step;
        c->cur ^= 1;
        ++c->step;
        if (chk)
            c->skin_checked = c->binned_at = c->step;
        ++q;
        base_set = false;
    }
    HIP_TRY(c, hipGetLastError());
    return SOP_OK;
}

sop_status sop_step_timed(sop_ctx *c, int64_t n_steps, double *ms_out)
{
    sop_status st = need_ready(c);
    if (st != SOP_OK)
        return st;
    if (n_steps < 0 || !ms_out)
        return fail(c, SOP_E_ARG, "bad timing arguments");
    if (c->sticky)
        return fail(c, status_from_bits(c->sticky), bits_message(c->sticky));
    hipEvent_t ev[4];
    for (auto &e : ev)
        HIP_TRY(c, hipEventCreate(&e));
    if (c->schedule == SOP_SCHEDULE_BATCHED) {
        double sum = 0.0;
        long long cnt = 0, q = 0;
        sop_status out = SOP_OK;
        while (q < n_steps) {
            // the launches that sop_step makes; the last counts only if whole
            const long long whole = std::min<long long>(c->batch_steps, record_span(c, c->step));
            const long long k = std::min(whole, (long long)(n_steps - q));
            const long long rec = last_record(c, c->step, k);
            (void)hipEventRecord(ev[0], c->stream);
            batch_launch(c, c->stream, (int)k, c->list_valid ? 0 : 1, 0, nullptr, c->step, rec >= 0);
            (void)hipEventRecord(ev[1], c->stream);
            hipError_t e = hipEventSynchronize(ev[1]);
            if (e != hipSuccess) {
                out = hip_fail(c, e, "hipEventSynchronize");
                break;
            }
            float ms = 0.0f;
            if (k == whole && hipEventElapsedTime(&ms, ev[0], ev[1]) == hipSuccess) {
                sum += ms;
                cnt += k;
            }
            if (rec >= 0)
                c->energy_step = rec;
            c->list_valid = true;
            c->cur ^= 1;
            c->step += k;
            q += k;
        }
        for (auto &e : ev)
            (void)hipEventDestroy(e);
        ms_out[0] = cnt ? sum / (double)cnt * (double)c->batch_steps : 0.0;
        ms_out[1] = 0.0;
        ms_out[2] = (double)c->batch_steps;
        if (out == SOP_OK)
            HIP_TRY(c, hipGetLastError());
        return out;
    }
    // Plain schedule: each kernel group is captured n_steps times back to back
    // in one graph (the step kernel reuses the current list; the rebuild
    // re-bins the same positions), so the events around the graph launch see
    // kernel time plus the short gaps between graph nodes.  The positions and
    // the error word are saved first and restored afterwards: steps on a
    // stale list may trip the error checks, which must not outlive the timing.
    for (auto &e : ev)
        (void)hipEventDestroy(e);
    const long long K = n_steps;
    ms_out[0] = ms_out[1] = ms_out[2] = 0.0;
    if (K == 0)
        return SOP_OK;
    const size_t bytes = 2 * (size_t)c->n_res * sizeof(float4);
    hipStream_t s = c->stream;
    unsigned err_saved = 0;
    HIP_TRY(c, hipStreamSynchronize(s));
    HIP_TRY(c, hipMemcpy(&err_saved, c->b.err, sizeof(unsigned), hipMemcpyDeviceToHost));
    HIP_TRY(c, hipMemcpyAsync(c->b.pos_save, c->b.pos[c->cur], bytes, hipMemcpyDeviceToDevice, s));
    if (!c->list_valid) {
        rebuild(c, s, false);
        c->list_valid = true;
    }
    if (!c->cap_stream)
        HIP_TRY(c, hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking));
    hipEvent_t e0, e1;
    HIP_TRY(c, hipEventCreate(&e0));
    HIP_TRY(c, hipEventCreate(&e1));
    sop_status out = SOP_OK;
    // kind 0: step kernels; 1: rebuilds with the skin build; 2: rebuilds
    // that only filter the skin rows (the skin stays valid in between)
    const int kinds = c->schedule == SOP_SCHEDULE_PLAIN ? 3 : 2;
    for (int kind = 0; kind < kinds && out == SOP_OK; ++kind) {
        const int saved = c->cur;
        hipGraph_t g = nullptr;
        hipError_t e = hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeRelaxed);
        if (e != hipSuccess) {
            out = hip_fail(c, e, "hipStreamBeginCapture");
            break;
        }
        // the steps run on past the list's period: whatever they move, the
        // kernel timed is the ordinary one
        FixDev fix = fix_consts(c);
        fix.move = 0x7fffffffu;
        fix.jump = 3.0e38f;
        for (long long q = 0; q < K; ++q) {
            if (kind == 0) {
                launch_step(c->b, c->cur, (int)c->n_res, c->cap, c->tile, step_consts(c), fix, c->tip,
                            c->pulls.empty() ? 0 : 1, false, 0, nullptr, c->step + q, 0.0f,
                            c->cap_stream, c->force_mode, 0.0f);
                c->cur ^= 1;
            } else {
                // kind 1: a search from freshly binned positions; kind 2:
                // the filter alone (the skin stays valid)
                c->skin_checked = c->binned_at = -1;
                rebuild(c, c->cap_stream, false, kind == 2);
            }
        }
        e = hipStreamEndCapture(c->cap_stream, &g);
        c->cur = saved;
        if (e != hipSuccess) {
            out = hip_fail(c, e, "hipStreamEndCapture");
            break;
        }
        hipGraphExec_t ex = nullptr;
        e = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
        (void)hipGraphDestroy(g);
        if (e != hipSuccess) {
            out = hip_fail(c, e, "hipGraphInstantiate");
            break;
        }
        float ms = 0.0f;
        for (int rep = 0; rep < 2 && e == hipSuccess; ++rep) {  // the first replay warms up
            (void)hipEventRecord(e0, s);
            e = hipGraphLaunch(ex, s);
            (void)hipEventRecord(e1, s);
            if (e == hipSuccess)
                e = hipEventSynchronize(e1);
        }
        if (e == hipSuccess)
            e = hipEventElapsedTime(&ms, e0, e1);
        (void)hipGraphExecDestroy(ex);
        if (e != hipSuccess) {
            out = hip_fail(c, e, "timed graph");
            break;
        }
        ms_out[kind] = (double)ms / (double)K;
        // back to the saved positions; the next list is built from them
        HIP_TRY(c, hipMemcpyAsync(c->b.pos[c->cur], c->b.pos_save, bytes, hipMemcpyDeviceToDevice, s));
        if (kind == 0) {
            c->skin_checked = c->binned_at = -1;
            rebuild(c, s, false);
        }
    }
    c->skin_checked = c->binned_at = -1;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    c->list_valid = false;
    if (out == SOP_OK) {
        HIP_TRY(c, hipStreamSynchronize(s));
        HIP_TRY(c, hipMemcpy(c->b.err, &err_saved, sizeof(unsigned), hipMemcpyHostToDevice));
    }
    return out;
}

sop_status sop_get_energies(sop_ctx *c, double *energies, int64_t *step)
{
    sop_status st = need_ready(c);
    if (st != SOP_OK)
        return st;
    st = fetch(c, {error_range(c), {c->b.energy, energies ? (size_t)c->n_traj * SOP_NTERMS * sizeof(double) : 0}},
               [&](int k, size_t off, size_t bytes, const char *p) {
                   if (k == 0)
                       take_errors(c, p);
                   else if (!c->sticky)
                       std::memcpy(reinterpret_cast<char *>(energies) + off, p, bytes);
               });
    if (st == SOP_OK)
        st = error_status(c);
    if (st == SOP_OK && step)
        *step = c->energy_step;
    return st;
}

sop_status sop_get_external_force(sop_ctx *c, double *f_ext)
{
    sop_status st = need_ready(c);
    if (st != SOP_OK)
        return st;
    if (!f_ext)
        return fail(c, SOP_E_ARG, "null output");
    st = fetch(c, {error_range(c), {c->b.f_ext, (size_t)c->n_traj * sizeof(double)}},
               [&](int k, size_t off, size_t bytes, const char *p) {
                   if (k == 0)
                       take_errors(c, p);
                   else if (!c->sticky)
                       std::memcpy(reinterpret_cast<char *>(f_ext) + off, p, bytes);
               });
    return st != SOP_OK ? st : error_status(c);
}

sop_status sop_sample_noise(sop_ctx *c, int64_t step, uint32_t *words, double *g)
{
    sop_status st = need_ready(c);
    if (st != SOP_OK)
        return st;
    if (step < 0)
        return fail(c, SOP_E_ARG, "negative step");
    // fout is scratch outside a force evaluation
    launch_noise(c->b, c->cur, (int)c->n_res, step_consts(c), step, c->b.words, c->b.fout, c->stream);
    HIP_TRY(c, hipGetLastError());
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    const long long n = c->n_res;
    if (words)
        HIP_TRY(c, hipMemcpy(words, c->b.words, n * sizeof(uint4), hipMemcpyDeviceToHost));
    if (g) {
        std::vector<float4> gv(n);
        HIP_TRY(c, hipMemcpy(gv.data(), c->b.fout, n * sizeof(float4), hipMemcpyDeviceToHost));
        for (long long i = 0; i < n; ++i) {
            g[3 * i] = gv[i].x;
            g[3 * i + 1] = gv[i].y;
            g[3 * i + 2] = gv[i].z;
        }
    }
    return SOP_OK;
}

}  // extern "C"

namespace {

// FNV-1a digest of what the schedule's speed depends on.
unsigned long long topology_digest(const sop_ctx *c)
{
    unsigned long long h = 1469598103934665603ull;
    auto mix = [&](unsigned long long v) {
        for (int k = 0; k < 8; ++k) {
            h ^= (v >> (8 * k)) & 0xff;
            h *= 1099511628211ull;
        }
    };
    mix((unsigned long long)c->n_res);
    mix((unsigned long long)c->n_traj);
    for (long long v : c->res_offsets)
        mix((unsigned long long)v);
    for (const int2 &r : c->trow)
        mix((unsigned long long)(unsigned)r.y);
    mix((unsigned long long)c->cap);
    mix((unsigned long long)c->p.list_every);
    return h;
}

std::string cache_key(const sop_ctx *c)
{
    int dev = 0;
    hipDeviceProp_t prop{};
    std::string arch = "unknown";
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
        arch = prop.gcnArchName;
    char buf[160];
    std::snprintf(buf, sizeof buf, "%s|%d|%016llx", arch.c_str(), c->schedule, topology_digest(c));
    return buf;
}

// Cache lines: <key> <a> <b>   (plain schedule: a = tile, b = force mode; batched: a = wg,
// b = steps)
bool cache_lookup(const char *path, const std::string &key, int *a, int *b)
{
    if (!path)
        return false;
    FILE *f = std::fopen(path, "r");
    if (!f)
        return false;
    char k[200];
    int x, y;
    bool found = false;
    while (std::fscanf(f, "%199s %d %d", k, &x, &y) == 3)
        if (key == k) {
            *a = x;
            *b = y;
            found = true;
        }
    std::fclose(f);
    return found;
}

void cache_store(const char *path, const std::string &key, int a, int b)
{
    if (!path)
        return;
    FILE *f = std::fopen(path, "a");
    if (!f)
        return;
    std::fprintf(f, "%s %d %d\n", key.c_str(), a, b);
    std::fclose(f);
}

// Residue-steps per second of `steps` steps from the saved state.
// A candidate slower than a third of `best` (residue-steps/s; 0: none yet)
// is stopped after the first eighth of its steps.
sop_status trial(sop_ctx *c, long long steps, double *rate, double best = 0.0)
{
    const size_t bytes = 2 * (size_t)c->n_res * sizeof(float4);
    HIP_TRY(c, hipMemcpyAsync(c->b.pos[c->cur], c->b.pos_save, bytes, hipMemcpyDeviceToDevice, c->stream));
    const long long step0 = c->step;
    c->list_valid = false;
    c->skin_checked = c->binned_at = -1;
    hipEvent_t e0, e1;
    HIP_TRY(c, hipEventCreate(&e0));
    HIP_TRY(c, hipEventCreate(&e1));
    sop_status st = sop_step(c, 2 * c->p.list_every);  // warm up: capture graphs, touch caches
    const long long L2 = 2 * c->p.list_every;
    const long long chunk = std::max<long long>(L2, (steps / 8 / L2) * L2);
    long long done = 0;
    float ms = 0.0f;
    if (st == SOP_OK)
        (void)hipEventRecord(e0, c->stream);
    while (st == SOP_OK && done < steps) {
        const long long k = std::min(chunk, steps - done);
        st = sop_step(c, k);
        done += k;
        (void)hipEventRecord(e1, c->stream);
        if (st != SOP_OK || hipEventSynchronize(e1) != hipSuccess ||
            hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
            ms = 0.0f;
            break;
        }
        const double r = ms > 0 ? (double)c->n_res * (double)done / (1e-3 * ms) : 0.0;
        if (best > 0.0 && r < best / 3.0)
            break;  // clearly slower: no need for the rest
    }
    *rate = ms > 0 ? (double)c->n_res * (double)done / (1e-3 * ms) : 0.0;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    // back to the saved state (the trial advanced the layer parity too)
    HIP_TRY(c, hipMemcpyAsync(c->b.pos[c->cur], c->b.pos_save, bytes, hipMemcpyDeviceToDevice, c->stream));
    c->step = step0;
    c->list_valid = false;
    c->skin_checked = c->binned_at = -1;
    return st;
}

}  // namespace

extern "C" {

sop_status sop_autotune(sop_ctx *c, double budget_ms, const char *cache_path)
{
    sop_status st = need_ready(c);
    if (st != SOP_OK)
        return st;
    if (c->sticky)
        return fail(c, status_from_bits(c->sticky), bits_message(c->sticky));
    const std::string key = cache_key(c);
    int a = 0, b = 0;
    if (cache_lookup(cache_path, key, &a, &b)) {
        if (c->schedule == SOP_SCHEDULE_BATCHED)
            return sop_set_batch(c, a, b);
        const sop_status s1 = sop_set_tile(c, a);
        return s1 != SOP_OK ? s1 : sop_set_force_mode(c, b);
    }
    const size_t bytes = 2 * (size_t)c->n_res * sizeof(float4);
    HIP_TRY(c, hipMemcpyAsync(c->b.pos_save, c->b.pos[c->cur], bytes, hipMemcpyDeviceToDevice, c->stream));
    const long long saved_energy_step = c->energy_step;
    std::vector<std::pair<int, int>> cand;
    if (c->schedule == SOP_SCHEDULE_BATCHED) {
        for (int wg : {256, 512, 1024})
            if (wg >= c->max_len)
                for (int k : {20, 50, 100, 200})
                    cand.push_back({wg, k});
    } else {
        for (int mode : {SOP_FORCES_PARTICLE, SOP_FORCES_PAIR})
            for (int tl : {64, 128, 256})
                cand.push_back({tl, mode});
    }
    // steps per trial from the budget, using the current schedule's speed as a guide
    double rate0 = 0.0;
    st = trial(c, 4 * c->p.list_every, &rate0);
    if (st != SOP_OK)
        return st;
    const double per_trial_ms = std::max(1.0, budget_ms / (double)cand.size());
    long long steps = (long long)(rate0 * 1e-3 * per_trial_ms / (double)c->n_res);
    steps = std::max<long long>(2 * c->p.list_every, (steps / (2 * c->p.list_every)) * 2 * c->p.list_every);
    if (c->schedule == SOP_SCHEDULE_BATCHED)
        steps = std::max<long long>(steps, 400);
    double best = -1.0;
    std::pair<int, int> pick = cand.front();
    for (const auto &cd : cand) {
        if (c->schedule == SOP_SCHEDULE_BATCHED) {
            st = sop_set_batch(c, cd.first, cd.second);
        } else {
            st = sop_set_tile(c, cd.first);
            if (st == SOP_OK)
                st = sop_set_force_mode(c, cd.second);
        }
        if (st != SOP_OK)
            return st;
        double rate = 0.0;
        st = trial(c, steps, &rate, best);
        if (st != SOP_OK)
            return st;
        if (rate > best) {
            best = rate;
            pick = cd;
        }
    }
    if (c->schedule == SOP_SCHEDULE_BATCHED) {
        st = sop_set_batch(c, pick.first, pick.second);
    } else {
        st = sop_set_tile(c, pick.first);
        if (st == SOP_OK)
            st = sop_set_force_mode(c, pick.second);
    }
    if (st != SOP_OK)
        return st;
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    c->energy_step = saved_energy_step;
    cache_store(cache_path, key, pick.first, pick.second);
    return check_device_errors(c);
}

sop_status sop_synchronize(sop_ctx *c)
{
    if (!c)
        return SOP_E_ARG;
    return check_device_errors(c);
}

}  // extern "C"
