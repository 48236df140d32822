// Triplet construction on the GPU: hashed uniform grid, fixed-radius query with local
// voxelisation (Sec. 3.2 "Definition"; fixed radius search of Sec. 4.1), and the reordering of
// Sec. 3.3.2 done as a counting sort on the composite key (k, centre): the query's count pass is
// the histogram, a prefix sum gives every (k, centre) run its place, the fill pass writes each
// triplet straight to its final position with ties ordered by the other index.
//
// This file is compiled with -ffp-contract=off: the inclusion test and the cell index are a fixed
// sequence of binary64 operations (see pcpp.h) and must not be fused.
#include <math.h>

#include "pcpp_internal.h"

namespace pcpp {

namespace {

constexpr unsigned long long EMPTY_KEY = ~0ull;
constexpr int CELL_BIAS = 1 << 20;
constexpr double CELL_CLAMP = (double)((1 << 20) - 2);   // +-1 stencil steps stay inside 21 bits

__device__ inline uint32_t hash_key(unsigned long long k)
{
    k ^= k >> 33; k *= 0xff51afd7ed558ccdULL;
    k ^= k >> 33; k *= 0xc4ceb9fe1a85ec53ULL;
    k ^= k >> 33;
    return (uint32_t)k;
}

__device__ inline int grid_coord(float p, double inv_g)
{
    double u = floor((double)p * inv_g);
    u = fmin(fmax(u, -CELL_CLAMP), CELL_CLAMP);      // NaN falls to a bound; no out-of-range key
    return (int)u;
}

__device__ inline unsigned long long pack_key(int cx, int cy, int cz)
{
    return ((unsigned long long)(uint32_t)(cx + CELL_BIAS) << 42) |
           ((unsigned long long)(uint32_t)(cy + CELL_BIAS) << 21) |
           (unsigned long long)(uint32_t)(cz + CELL_BIAS);
}

// Which cloud of a batch a point belongs to: the largest b with off[b] <= idx (off has n_batches + 1 entries).
__device__ inline int find_batch(const int32_t *__restrict__ off, int n_batches, int idx)
{
    int lo = 0, hi = n_batches - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= idx) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Voxel of a coordinate in a global voxelisation of pitch v (voxel mode): floor(p / v) in binary64.
__device__ inline double voxel_of(float p, double v) { return floor(__ddiv_rn((double)p, v)); }

__device__ inline int floor_div(int a, int b) { return a >= 0 ? a / b : -((-a + b - 1) / b); }

// How points map to cells of the hashed grid.  Ball mode: cells of pitch 1 / inv_g (a hair above the radius).
// Voxel mode: cells of hp = max(h, 1) voxels per axis, so that voxels at most h apart lie in adjacent cells.
// With batches the cloud's number is mixed into the key: equal keys of different clouds are possible but harmless,
// because a centre only accepts candidates of its own cloud (their index range) and never probes two cells whose
// keys the mixing could make equal (it is a bijection within one cloud).
struct GridMap {
    double inv_g;
    double vox;       // voxel pitch, voxel mode only
    int hp;
    int voxel_mode;
};

__device__ inline void grid_cell3(float fx, float fy, float fz, const GridMap &m, int &gx, int &gy, int &gz)
{
    if (m.voxel_mode) {
        const double lim = CELL_CLAMP * (double)m.hp;
        gx = floor_div((int)fmin(fmax(voxel_of(fx, m.vox), -lim), lim), m.hp);
        gy = floor_div((int)fmin(fmax(voxel_of(fy, m.vox), -lim), lim), m.hp);
        gz = floor_div((int)fmin(fmax(voxel_of(fz, m.vox), -lim), lim), m.hp);
    } else {
        gx = grid_coord(fx, m.inv_g);
        gy = grid_coord(fy, m.inv_g);
        gz = grid_coord(fz, m.inv_g);
    }
}

template <bool EXT>
__device__ inline void grid_cell(float fx, float fy, float fz, const GridMap &m, int &gx, int &gy, int &gz)
{
    if constexpr (EXT) {
        grid_cell3(fx, fy, fz, m, gx, gy, gz);
    } else {
        gx = grid_coord(fx, m.inv_g); gy = grid_coord(fy, m.inv_g); gz = grid_coord(fz, m.inv_g);
    }
}

__device__ inline unsigned long long mix_batch(unsigned long long key, int batch)
{
    key ^= (unsigned long long)(batch + 1) * 0x9E3779B97F4A7C15ull;
    return key == EMPTY_KEY ? key - 1ull : key;
}

// ---- hashed grid over the candidate set ------------------------------------------------------

// empty table: no keys, zero populations (slots + 1 entries, the input of the prefix sum);
// the first call of a build also zeroes the status words of all its prefix sums
__global__ __launch_bounds__(256) void grid_clear(unsigned long long *__restrict__ keys, uint32_t *__restrict__ cnt,
                                                  int64_t slots,
                                                  unsigned long long *__restrict__ scan_status, int64_t scan_words)
{
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i <= slots; i += stride) {
        cnt[i] = 0u;
        if (i < slots) keys[i] = EMPTY_KEY;
    }
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < scan_words; i += stride) scan_status[i] = 0ull;
}

__global__ __launch_bounds__(256) void grid_insert(const float *__restrict__ xyz, int64_t n, GridMap gm,
                                                   const int32_t *__restrict__ batch_off, int n_batches,
                                                   unsigned long long *__restrict__ keys,
                                                   uint32_t *__restrict__ slot_cnt, uint32_t mask,
                                                   uint2 *__restrict__ point_at)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    int gx, gy, gz;
    grid_cell3(xyz[3 * p], xyz[3 * p + 1], xyz[3 * p + 2], gm, gx, gy, gz);
    unsigned long long key = pack_key(gx, gy, gz);
    if (batch_off) key = mix_batch(key, find_batch(batch_off, n_batches, (int)p));
    uint32_t slot = hash_key(key) & mask;
    // the table has at least twice as many slots as points, so an empty slot is always reached
    for (;;) {
        // (most points find their cell's key there already: a read is cheaper than a swap)
        unsigned long long prev = __hip_atomic_load(&keys[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (prev == EMPTY_KEY) prev = atomicCAS(&keys[slot], EMPTY_KEY, key);
        if (prev == EMPTY_KEY || prev == key) break;
        slot = (slot + 1) & mask;
    }
    point_at[p] = make_uint2(slot, atomicAdd(&slot_cnt[slot], 1u));      // its slot, and its place there
}

__global__ __launch_bounds__(256) void grid_scatter(const float *__restrict__ xyz, int64_t n,
                                                    const uint2 *__restrict__ point_at,
                                                    const uint32_t *__restrict__ slot_start, float4 *__restrict__ pts,
                                                    const uint32_t *__restrict__ err)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n || *err) return;                       // err: the slot offsets come from a prefix sum that gave up
    const uint2 at = point_at[p];
    const uint32_t pos = slot_start[at.x] + at.y;
    pts[pos] = make_float4(xyz[3 * p], xyz[3 * p + 1], xyz[3 * p + 2], __int_as_float((int)p));
}

struct GridView {
    const unsigned long long *keys;   // NULL: no grid, every candidate is looked at (small clouds)
    const uint32_t *slot_start;   // [slots + 1]
    const float4 *pts;            // candidates grouped by grid cell; .w carries the original index
    uint32_t mask;
    GridMap map;
    const float *xyz;             // without a grid: the candidates [n][3]
    int n;

    __device__ inline float4 candidate(uint32_t at) const
    {
        if (keys) return pts[at];
        return make_float4(xyz[3 * (size_t)at], xyz[3 * (size_t)at + 1], xyz[3 * (size_t)at + 2], __int_as_float((int)at));
    }
};

// Ball mode (Sec. 3.2 "Definition"): R, r2, inv_cell.  Voxel mode (the degraded operator of Sec. 3.2, "Voxel
// Convolution as a Special Case"): neighbours are the points whose voxel differs from the centre's by at most
// h = (t - 1) / 2 along every axis, the cell is the voxel offset (input minus output) plus h.
// Batches: c_off / d_off are the offsets of the clouds in the centre set and in the candidate set.
struct QueryParams {
    double R;         // (double)radius, or the voxel pitch
    double r2;        // R * R
    double inv_cell;  // t / (2 R)
    double sign;      // offset input minus output = sign (candidate - centre): 1 where the centres are outputs, -1 inputs
    int t;
    int voxel_mode, h;
    const int32_t *c_off, *d_off;
    int n_batches;
};

__device__ inline uint32_t wave_incl_scan_u32(uint32_t v)
{
    // DPP moves inside the adds (all 64 lanes must be active): shifts inside rows of 16 lanes, then the rows' last lanes to
    // the rows behind them; no trip through LDS
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);
    return v;
}

// A value that the compiler has to work out at this place: what rarely taken code derives from it is not kept in registers
// all along the loops around it (the fill pass spilled twenty for that).
__device__ inline int here(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

__device__ inline uint32_t lane_value(uint32_t v, int lane) { return (uint32_t)__builtin_amdgcn_readlane((int)v, lane); }
__device__ inline float lane_value(float v, int lane) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane)); }

// The block's LDS traffic done, then its barrier.  No wait for memory: what the passes below read ahead stays on its way, and
// nobody waits for stores; the waves of a block share nothing but LDS.
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Candidates around one grid cell, held across the lanes of a wave: lane j < 27 owns stencil cell j.
// Every method must be called by all 64 lanes of the wave (it uses cross-lane reads).
struct Stencil {
    uint32_t my_start;       // lane j: first candidate of stencil cell j
    uint32_t my_excl;        // lane j: candidates in cells before j
    uint32_t total;

    // (gx, gy, gz): the middle cell; batch: the cloud's number, or -1 where there is one cloud
    __device__ inline void open(int gx, int gy, int gz, int batch, const GridView &g, int lane)
    {
        uint32_t cnt = 0;
        my_start = 0;
        if (!g.keys) {                     // one cell that holds all candidates
            if (lane == 0) cnt = (uint32_t)g.n;
        } else if (lane < 27) {
            unsigned long long key = pack_key(gx + lane / 9 - 1, gy + (lane / 3) % 3 - 1, gz + lane % 3 - 1);
            if (batch >= 0) key = mix_batch(key, batch);
            uint32_t slot = hash_key(key) & g.mask;
            for (;;) {
                const unsigned long long kk = g.keys[slot];
                if (kk == key) {
                    my_start = g.slot_start[slot];
                    cnt = g.slot_start[slot + 1] - my_start;
                    break;
                }
                if (kk == EMPTY_KEY) break;
                slot = (slot + 1) & g.mask;
            }
        }
        const uint32_t incl = wave_incl_scan_u32(cnt);
        my_excl = incl - cnt;
        total = lane_value(incl, 63);
    }

    // where candidate number idx < total (idx may differ per lane) lies among g.pts
    __device__ inline uint32_t place(uint32_t idx) const
    {
        int j = 0;
#pragma unroll
        for (int step = 16; step >= 1; step >>= 1) {
            const int c = j + step;
            const int cc = c <= 26 ? c : 26;
            const uint32_t e = __shfl(my_excl, cc, 64);
            if (c <= 26 && e <= idx) j = c;
        }
        const uint32_t s = __shfl(my_start, j, 64);
        const uint32_t e = __shfl(my_excl, j, 64);
        return s + (idx - e);
    }
};

// d = candidate - centre, in binary64, no contraction: the test of the ball, which does not depend on its sign
__device__ inline bool inside_ball(double dx, double dy, double dz, const QueryParams &q)
{
    return __dadd_rn(__dadd_rn(__dmul_rn(dx, dx), __dmul_rn(dy, dy)), __dmul_rn(dz, dz)) <= q.r2;
}

// Kernel cell of the offset d = input - output of a neighbour.  A neighbour's |d| exceeds R by rounding at most, so
// (d + R) t / (2 R) lies above -1 and cutting the fraction off is floor and the clamp at 0 in one.
__device__ inline int ball_cell(double dx, double dy, double dz, const QueryParams &q)
{
    const int tm1 = q.t - 1;
    const int kx = (int)__dmul_rn(__dadd_rn(dx, q.R), q.inv_cell);
    const int ky = (int)__dmul_rn(__dadd_rn(dy, q.R), q.inv_cell);
    const int kz = (int)__dmul_rn(__dadd_rn(dz, q.R), q.inv_cell);
    return __mul24(__mul24(kx < tm1 ? kx : tm1, q.t) + (ky < tm1 ? ky : tm1), q.t) + (kz < tm1 ? kz : tm1);
}

// Voxel mode: the offset of the voxels is an exact small integer in binary64
__device__ inline bool inside_cube(double ox, double oy, double oz, const QueryParams &q)
{
    const double h = (double)q.h;
    return fabs(ox) <= h && fabs(oy) <= h && fabs(oz) <= h;
}
__device__ inline int cube_cell(double ox, double oy, double oz, const QueryParams &q)
{
    return (((int)ox + q.h) * q.t + (int)oy + q.h) * q.t + (int)oz + q.h;
}

// One centre's search by a whole wave.  EXT: the voxel operator and batches of clouds are compiled in (the plain search,
// which is bound by instruction issue, does without their tests).
template <bool EXT>
struct Candidates {
    double cx, cy, cz;       // centre coordinate (ball mode) or its voxel (voxel mode)
    Stencil st;
    int d_lo, d_hi;          // candidates of the centre's own cloud: indices [d_lo, d_hi)

    __device__ inline void open(const float *__restrict__ centres, int64_t a, const GridView &g, const QueryParams &q,
                                int lane)
    {
        const float fx = centres[3 * a], fy = centres[3 * a + 1], fz = centres[3 * a + 2];
        if (EXT && q.voxel_mode) { cx = voxel_of(fx, q.R); cy = voxel_of(fy, q.R); cz = voxel_of(fz, q.R); }
        else { cx = (double)fx; cy = (double)fy; cz = (double)fz; }
        int batch = -1;
        d_lo = 0; d_hi = 0x7fffffff;
        if (EXT && q.c_off) {
            batch = find_batch(q.c_off, q.n_batches, (int)a);
            d_lo = q.d_off[batch]; d_hi = q.d_off[batch + 1];
        }
        int gx, gy, gz;
        grid_cell<EXT>(fx, fy, fz, g.map, gx, gy, gz);
        st.open(gx, gy, gz, batch, g, lane);
    }

    // Candidate number idx (idx may differ per lane).  Returns whether it is a neighbour; b = its original index, k = its
    // kernel cell, k2 = the cell of the opposite offset, i.e. the cell this pair falls in when the roles are swapped.
    __device__ inline bool fetch(uint32_t idx, const GridView &g, const QueryParams &q, int &b, int &k, int &k2) const
    {
        const bool in_range = idx < st.total;
        const uint32_t at = st.place(in_range ? idx : 0u);
        bool hit = false;
        b = 0; k = 0; k2 = 0;
        if (in_range) {
            const float4 p = g.candidate(at);
            b = __float_as_int(p.w);
            if (EXT && q.voxel_mode) {
                const double ox = q.sign * (voxel_of(p.x, q.R) - cx), oy = q.sign * (voxel_of(p.y, q.R) - cy), oz = q.sign * (voxel_of(p.z, q.R) - cz);
                hit = inside_cube(ox, oy, oz, q) && b >= d_lo && b < d_hi;
                if (hit) { k = cube_cell(ox, oy, oz, q); k2 = cube_cell(-ox, -oy, -oz, q); }
                return hit;
            }
            const double dx = q.sign * __dsub_rn((double)p.x, cx), dy = q.sign * __dsub_rn((double)p.y, cy), dz = q.sign * __dsub_rn((double)p.z, cz);
            hit = inside_ball(dx, dy, dz, q) && (!EXT || (b >= d_lo && b < d_hi));
            if (hit) { k = ball_cell(dx, dy, dz, q); k2 = ball_cell(-dx, -dy, -dz, q); }
        }
        return hit;
    }
};

constexpr uint32_t KEEP_MAX = 512;        // largest stride of the neighbour lists
constexpr int HIT_INDEX_BITS = 24;        // a stored hit = cell << 24 | candidate index
constexpr uint32_t HIT_INDEX_MASK = (1u << HIT_INDEX_BITS) - 1u;

// The neighbour lists of one side's centres.  found[c] says how many neighbours centre c has, up to `stride`, whose list lies at
// c stride; or, with LONG_LIST set, where its list lies behind those, in units of LONG_UNIT words and behind a word that says how many
// there are.  The search hands out that room where it finds a list that is too long.  A centre that finds none left has its number with
// NO_LIST set, and the passes search it again: in the smallest workspace, or when there are more triplets than the call has room for.
constexpr uint32_t LONG_LIST = 0x80000000u, NO_LIST = 0xc0000000u, LONG_UNIT = 4;
__device__ inline bool has_no_list(uint32_t f) { return (f & NO_LIST) == NO_LIST; }
__device__ inline bool has_long_list(uint32_t f) { return (f & NO_LIST) == LONG_LIST; }
struct Lists {
    uint32_t *hits;               // cell << 24 | index, in arrival order; NULL: no lists at all
    uint32_t *found;              // [n_centres]; without lists the count pass writes the numbers, or a search that only counts
    uint32_t stride;
    size_t long_from;

    __device__ inline size_t long_at(uint32_t f) const { return long_from + (size_t)(f & ~LONG_LIST) * LONG_UNIT; }
};

// ---- search: every centre's neighbours, in arrival order ----------------------------------------
// into the lists of the side where the centres are outputs, or `mirror` where they are inputs.  A cloud queried against itself
// has both: the pair (centre c, candidate b) is also the pair (c, b) of the side with the roles swapped, in the cell of the opposite
// offset, at the same place of its lists.
// A wave takes `per_wave` consecutive centres of `order`, which holds the centres grouped by grid cell (without it: in index
// order), and those of one cell together: the stencil is probed and the candidates are read, placed and converted once for
// all of them, 256 at a time in registers, and a centre costs its binary64 tests, the cells of its neighbours and the stores.
// The vector ALU issues in 84 % of the cycles (1 M points of a ground scene, 32 neighbours in 125 cells, shuffled); the candidates, whose
// cells the hash scatters, come from memory, 1.7 GB of them.  One search per centre, in the order of the tiles and with the tiles'
// tables in LDS: 1215 us; now 325.
// Centres with a long list are searched a second time here, where they still share their candidates, and not by the later passes, one
// wave per centre: 20 000 points with a quarter of them in a blob, two sides, 2.9 M triplets, the build with both further
// searches 457 us, so 241; without a grid 2896 points, one side, 350 and 66.
constexpr int GROUP_SETS = 4;             // sets of 64 candidates in registers
constexpr int64_t SEARCH_WAVES = 8192;    // waves wanted before a wave takes more centres

struct SearchArgs {
    const float4 *order;
    const float *centres;
    int64_t n_centres;
    GridView g;
    QueryParams q;
    Lists lists;
    uint32_t *mirror;
    unsigned long long long_units;       // room for lists longer than the stride
    unsigned long long *long_used;       // how much of it has been handed out (NULL: every centre has its own, for all candidates)
    int per_wave;
    uint32_t *err;
    unsigned long long *clear_from;      // without a grid: what its clearing kernel would have cleared
    int64_t clear_words;
};

// FORM: centres are outputs, centres are inputs (the offset input minus output is the other way round), or both in one.
enum Form { OUTPUTS, INPUTS, BOTH };

// a neighbour at offset d = candidate - centre (of their voxels in voxel mode)
template <Form FORM, bool EXT>
__device__ inline void store_hit(const SearchArgs &a, size_t at, double dx, double dy, double dz, uint32_t b)
{
    const bool cube = EXT && a.q.voxel_mode;
    if constexpr (FORM != INPUTS) {
        const int k = cube ? cube_cell(dx, dy, dz, a.q) : ball_cell(dx, dy, dz, a.q);
        a.lists.hits[at] = ((uint32_t)k << HIT_INDEX_BITS) | b;
    }
    if constexpr (FORM != OUTPUTS) {
        const int k = cube ? cube_cell(-dx, -dy, -dz, a.q) : ball_cell(-dx, -dy, -dz, a.q);
        a.mirror[at] = ((uint32_t)k << HIT_INDEX_BITS) | b;
    }
}

// a long list's word in front
template <Form FORM>
__device__ inline void store_length(const SearchArgs &a, size_t at, uint32_t n)
{
    if constexpr (FORM != INPUTS) a.lists.hits[at] = n;
    if constexpr (FORM != OUTPUTS) a.mirror[at] = n;
}

template <Form FORM, bool EXT>
__global__ __launch_bounds__(256, 6) void search_cells(const SearchArgs a)
{
    const int lane = threadIdx.x & 63;
    const int64_t wave = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t base = wave * a.per_wave;
    if (*a.err || base >= a.n_centres) return;     // wave-uniform (nothing below is shared between waves)
    // this lane's centre
    const int64_t at = base + lane;
    const bool mine = lane < a.per_wave && at < a.n_centres;
    float fx = 0.f, fy = 0.f, fz = 0.f;
    int index = 0, batch = -1, gx = 0, gy = 0, gz = 0;
    if (mine) {
        if (a.order) {
            const float4 p = a.order[at];
            fx = p.x; fy = p.y; fz = p.z; index = __float_as_int(p.w);
        } else {
            fx = a.centres[3 * at]; fy = a.centres[3 * at + 1]; fz = a.centres[3 * at + 2]; index = (int)at;
        }
        grid_cell<EXT>(fx, fy, fz, a.g.map, gx, gy, gz);
        if (EXT && a.q.c_off) batch = find_batch(a.q.c_off, a.q.n_batches, index);
    }
    const unsigned long long below = (1ull << lane) - 1ull;
    uint32_t filled_of = 0;                        // where the next neighbour of this lane's centre goes in its list, or among the long lists
    unsigned long long open = __ballot(mine);
    // once over the candidates for all centres, once more for those whose list turned out to be a long one
    for (bool again = false;; again = true) {
        const uint32_t limit = again ? 0xffffffffu : a.lists.stride;
        while (open) {
            const int lead = __builtin_ctzll(open);
            const int lx = (int)lane_value((uint32_t)gx, lead), ly = (int)lane_value((uint32_t)gy, lead), lz = (int)lane_value((uint32_t)gz, lead);
            const int lb = EXT ? (int)lane_value((uint32_t)batch, lead) : -1;
            const unsigned long long group = __ballot(gx == lx && gy == ly && gz == lz && (!EXT || batch == lb)) & open;
            open &= ~group;
            Stencil st;
            st.open(lx, ly, lz, lb, a.g, lane);
            int d_lo = 0, d_hi = 0x7fffffff;
            if (EXT && a.q.c_off) { d_lo = a.q.d_off[lb]; d_hi = a.q.d_off[lb + 1]; }
            for (uint32_t first = 0; first < st.total; first += 64 * GROUP_SETS) {
                double px[GROUP_SETS], py[GROUP_SETS], pz[GROUP_SETS];
                uint32_t pb[GROUP_SETS];
#pragma unroll
                for (int s = 0; s < GROUP_SETS; ++s) {
                    px[s] = INFINITY; py[s] = 0.0; pz[s] = 0.0; pb[s] = 0u;       // infinitely far: no neighbour of any centre
                    const uint32_t idx = first + 64u * s + (uint32_t)lane;
                    if (first + 64u * s < st.total) {  // wave-uniform
                        const uint32_t pos = st.place(idx < st.total ? idx : 0u);
                        if (idx < st.total) {
                            const float4 p = a.g.pts[pos];
                            pb[s] = (uint32_t)__float_as_int(p.w);
                            if (!EXT || ((int)pb[s] >= d_lo && (int)pb[s] < d_hi)) {
                                if (EXT && a.q.voxel_mode) { px[s] = voxel_of(p.x, a.q.R); py[s] = voxel_of(p.y, a.q.R); pz[s] = voxel_of(p.z, a.q.R); }
                                else { px[s] = (double)p.x; py[s] = (double)p.y; pz[s] = (double)p.z; }
                            }
                        }
                    }
                }
                for (unsigned long long rest = group; rest; rest &= rest - 1) {
                    const int c = __builtin_ctzll(rest);
                    const float sx = lane_value(fx, c), sy = lane_value(fy, c), sz = lane_value(fz, c);
                    double cx, cy, cz;
                    if (EXT && a.q.voxel_mode) { cx = voxel_of(sx, a.q.R); cy = voxel_of(sy, a.q.R); cz = voxel_of(sz, a.q.R); }
                    else { cx = (double)sx; cy = (double)sy; cz = (double)sz; }
                    const size_t row = again ? a.lists.long_from : (size_t)lane_value((uint32_t)index, c) * a.lists.stride;
                    uint32_t filled = lane_value(filled_of, c);
#pragma unroll
                    for (int s = 0; s < GROUP_SETS; ++s) {
                        if (first + 64u * s >= st.total) break;                   // wave-uniform
                        const double dx = __dsub_rn(px[s], cx), dy = __dsub_rn(py[s], cy), dz = __dsub_rn(pz[s], cz);
                        const bool hit = EXT && a.q.voxel_mode ? inside_cube(dx, dy, dz, a.q) : inside_ball(dx, dy, dz, a.q);
                        const unsigned long long m = __ballot(hit);
                        const uint32_t slot = filled + (uint32_t)__popcll(m & below);
                        filled += (uint32_t)__popcll(m);
                        if (hit && slot < limit) store_hit<FORM, EXT>(a, row + slot, dx, dy, dz, pb[s]);
                    }
                    if (lane == c) filled_of = filled;
                }
            }
        }
        if (again) break;
        uint32_t found = filled_of;
        if (mine && a.lists.hits && filled_of > a.lists.stride) {
            const uint32_t units = (filled_of + LONG_UNIT) / LONG_UNIT;          // (its length in front)
            const unsigned long long from = a.long_units ? atomicAdd(a.long_used, (unsigned long long)units) : 0ull;
            found = filled_of | NO_LIST;
            if (from + units <= a.long_units) {
                found = (uint32_t)from | LONG_LIST;
                store_length<FORM>(a, a.lists.long_at(found), filled_of);
                filled_of = (uint32_t)from * LONG_UNIT + 1u;
            }
        }
        if (mine) a.lists.found[index] = found;
        open = __ballot(mine && has_long_list(found));
        if (!open) break;
    }
}

// The same for small clouds, without a grid: every centre looks at every candidate, one wave per centre, and a test in 32 bits
// passes over those that are far away (its bound leaves room for its rounding: a difference of two coordinates and a sum of
// three squares are off by less than 2^-21 together, and by less than 1e-37 where they underflow).
constexpr int ALL_CHUNK = 4096;           // candidates in LDS at a time

template <Form FORM, bool EXT>
__global__ __launch_bounds__(256) void search_all(const SearchArgs a)
{
    constexpr int LOADS = 24;
    extern __shared__ float cand[];                // [ALL_CHUNK][3], or as many as there are
    const int tid = threadIdx.x, lane = tid & 63;
    if (blockIdx.x == 0)
        for (int64_t i = tid; i < a.clear_words; i += 256) a.clear_from[i] = 0ull;
    const int64_t index = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool on = index < a.n_centres;           // wave-uniform
    float fx = 0.f, fy = 0.f, fz = 0.f;
    int d_lo = 0, d_hi = a.g.n;
    if (on) {
        fx = a.centres[3 * index]; fy = a.centres[3 * index + 1]; fz = a.centres[3 * index + 2];
        if (EXT && a.q.c_off) {
            const int batch = find_batch(a.q.c_off, a.q.n_batches, (int)index);
            d_lo = a.q.d_off[batch]; d_hi = a.q.d_off[batch + 1];
        }
    } else {
        d_hi = 0;
    }
    const bool cube = EXT && a.q.voxel_mode;
    double cx = fx, cy = fy, cz = fz;
    if (cube) { cx = voxel_of(fx, a.q.R); cy = voxel_of(fy, a.q.R); cz = voxel_of(fz, a.q.R); }
    const float near2 = (float)(a.q.r2 * (1.0 + 1.0 / 1048576.0)) + 1e-37f;
    const unsigned long long below = (1ull << lane) - 1ull;
    // once over the candidates, and once more if the list turned out to be a long one
    uint32_t filled = 0;
    bool is_long = false;
    uint32_t long_of = 0;
    for (bool again = false;; again = true) {
        const size_t row = again ? a.lists.long_at(long_of) + 1 : (size_t)index * a.lists.stride;
        const uint32_t limit = again ? 0xffffffffu : a.lists.stride;
        for (int c0 = 0; c0 < a.g.n; c0 += ALL_CHUNK) {
            const int m = a.g.n - c0 < ALL_CHUNK ? a.g.n - c0 : ALL_CHUNK;
            if (!again || a.g.n > ALL_CHUNK) {             // (otherwise they are all there still)
                if (again || c0 > 0) __syncthreads();
                for (int i0 = tid; i0 < 3 * m; i0 += 256 * LOADS) {        // (all of a step's loads on their way at a time)
                    float v[LOADS];
#pragma unroll
                    for (int j = 0; j < LOADS; ++j) v[j] = i0 + 256 * j < 3 * m ? a.g.xyz[3 * (size_t)c0 + i0 + 256 * j] : 0.f;
#pragma unroll
                    for (int j = 0; j < LOADS; ++j)
                        if (i0 + 256 * j < 3 * m) cand[i0 + 256 * j] = v[j];
                }
                __syncthreads();
            }
            if (again && !is_long) continue;               // (wave-uniform)
            const int lo = d_lo > c0 ? (d_lo - c0) & ~63 : 0, hi = d_hi - c0 < m ? d_hi - c0 : m;     // the centre's own cloud
            for (int first = lo; first < hi; first += 64 * GROUP_SETS) {
                float x[GROUP_SETS], y[GROUP_SETS], z[GROUP_SETS];
                bool in[GROUP_SETS], near[GROUP_SETS], any = false;
#pragma unroll
                for (int s = 0; s < GROUP_SETS; ++s) {
                    const int i = first + 64 * s + lane;
                    in[s] = i < hi && (!EXT || c0 + i >= d_lo);
                    const int at = 3 * (in[s] ? i : first);
                    x[s] = cand[at]; y[s] = cand[at + 1]; z[s] = cand[at + 2];
                }
#pragma unroll
                for (int s = 0; s < GROUP_SETS; ++s) {
                    const float ax = x[s] - fx, ay = y[s] - fy, az = z[s] - fz;
                    near[s] = in[s] && (cube || ax * ax + ay * ay + az * az <= near2);
                    any = any || near[s];
                }
                if (!__ballot(any)) continue;
#pragma unroll
                for (int s = 0; s < GROUP_SETS; ++s) {
                    if (!__ballot(near[s])) continue;
                    double dx, dy, dz;
                    if (cube) { dx = voxel_of(x[s], a.q.R) - cx; dy = voxel_of(y[s], a.q.R) - cy; dz = voxel_of(z[s], a.q.R) - cz; }
                    else { dx = __dsub_rn((double)x[s], cx); dy = __dsub_rn((double)y[s], cy); dz = __dsub_rn((double)z[s], cz); }
                    const bool hit = in[s] && (cube ? inside_cube(dx, dy, dz, a.q) : inside_ball(dx, dy, dz, a.q));
                    const unsigned long long mask = __ballot(hit);
                    const uint32_t slot = filled + (uint32_t)__popcll(mask & below);
                    filled += (uint32_t)__popcll(mask);
                    if (hit && slot < limit) store_hit<FORM, EXT>(a, row + slot, dx, dy, dz, (uint32_t)(c0 + first + 64 * s + lane));
                }
            }
        }
        if (again) break;
        // (wave-uniform, as the numbers are)
        const bool past = on && a.lists.hits && filled > a.lists.stride;
        uint32_t found = filled;
        if (past && !a.long_used) {
            long_of = (uint32_t)index * (((uint32_t)a.g.n + LONG_UNIT) / LONG_UNIT);
            is_long = true;
        } else if (past) {
            const uint32_t units = (filled + LONG_UNIT) / LONG_UNIT;
            unsigned long long from = 0ull;
            if (lane == 0) from = atomicAdd(a.long_used, (unsigned long long)units);
            from = __shfl(from, 0, 64);
            is_long = from + units <= a.long_units;
            long_of = (uint32_t)from;
            found = filled | NO_LIST;
        }
        if (is_long) found = long_of | LONG_LIST;
        if (on && lane == 0) {
            a.lists.found[index] = found;
            if (is_long) store_length<FORM>(a, a.lists.long_at(long_of), filled);
        }
        if (a.g.n > ALL_CHUNK ? !__syncthreads_or(is_long) : !is_long) break;
        filled = 0u;
    }
}

// ---- one side's order of the triplets -------------------------------------------------------------
// The public list (centres = outputs in index order) and the plan's sides.  Tile = 64 consecutive slots.
//   perm     centre index of each slot (NULL: slots are centre indices); lists are indexed by centre
//   lists    the centres' neighbours as the search left them.  Without lists both passes search again (the count pass writes the
//            numbers of neighbours, and where mirror_sums is given, the sums of the swapped side too)
//   sums     [K * n_tiles]      k-major: neighbours of tile's centres in cell k
//   ptr      [K * n_tiles + 1]  exclusive prefix sum of `sums`
struct FillOut {
    // Where the fill pass writes.  out_c / out_b / out_k: centre index, candidate index, cell of each triplet (any may
    // be NULL).  With tail_index >= 0 the candidate indices go to the tail_index-th |T|-sized array behind `tail`
    // instead (each align_up(|T| * 4) bytes, |T| read from the prefix sum's last entry), with GATHER_LAST set on the
    // last triplet of every run.  Nothing is written when |T| exceeds out_cap (the pass is
    // queued before the host has compared the count with what the caller provided).
    int32_t *out_c, *out_b, *out_k;
    char *tail;
    int tail_index;
    uint32_t out_cap;
};
struct Side {
    const float *centres;
    const int32_t *perm;
    int64_t n_centres, n_tiles;
    GridView g;
    QueryParams q;
    Lists lists;
    uint32_t *sums, *mirror_sums;
    const uint32_t *ptr;
    uint32_t *run_start;          // [n_tiles][K][TILE], NULL: not wanted
    unsigned long long *rows;     // [n_tiles][mask_words(K)], which rows of run_start are written (NULL: all)
    int64_t *seg_out;             // [K + 1], NULL: not wanted
    FillOut out;
};
constexpr int MAX_SIDES = 3;
struct Sides { Side s[MAX_SIDES]; };

// What the fill pass keeps in LDS of a tile's centres.
struct TileCentres {
    uint32_t off[TILE + 1];       // neighbours of the centres before each
    int32_t at[TILE];             // its own index
    uint32_t found[TILE];
    uint32_t searched;            // centres without a list: whether there are any

    __device__ inline uint32_t n(int al) const { return off[al + 1] - off[al]; }
    // by wave 0; a barrier follows
    __device__ inline void open(const Side &s, int64_t tile, int lane)
    {
        const int64_t slot = tile * TILE + lane;
        const bool on = slot < s.n_centres;
        const int32_t c = on ? (s.perm ? s.perm[slot] : (int32_t)slot) : 0;
        const uint32_t f = on ? s.lists.found[c] : 0u;
        uint32_t m = f & LONG_LIST ? f & ~NO_LIST : f;
        if (has_long_list(f)) m = s.lists.hits[s.lists.long_at(f)];
        const unsigned long long none = __ballot(on && (!s.lists.hits || has_no_list(f)));
        const uint32_t incl = wave_incl_scan_u32(m);
        at[lane] = c;
        found[lane] = f;
        off[lane] = incl - m;
        if (lane == TILE - 1) off[TILE] = incl;
        if (lane == 0) searched = none != 0ull;
    }
    // the centre that a neighbour of the tile belongs to, for a thread that goes through consecutive ones
    struct Cursor { int al; uint32_t end; };
    __device__ inline Cursor cursor(uint32_t p) const
    {
        int al = 0;
#pragma unroll
        for (int step = TILE / 2; step >= 1; step >>= 1)
            if (off[al + step] <= p) al += step;
        return Cursor{al, off[al + 1]};
    }
    __device__ inline void advance(Cursor &c, uint32_t p) const
    {
        while (p >= c.end) {               // (p is below the tile's number of neighbours)
            ++c.al;
            c.end = off[c.al + 1];
        }
    }
};

// The tile of a block.  Blocks go round the eight XCDs; of many tiles, 16 consecutive ones (a cache line of an offset table's
// row) go to one XCD, whose L2 then reads the line once and completes the lines that the ends of their output share.
constexpr int XCD_TILES = 16, NUM_XCD = 8;
__host__ __device__ inline bool tiles_by_xcd(int64_t n_tiles) { return n_tiles >= 32 * XCD_TILES * NUM_XCD; }
__device__ inline int64_t tile_of_block(int64_t block, int64_t n_tiles)
{
    if (!tiles_by_xcd(n_tiles)) return block;
    const int64_t r = block / NUM_XCD;
    return (r / XCD_TILES * NUM_XCD + block % NUM_XCD) * XCD_TILES + r % XCD_TILES;
}
// ... and how many blocks n_tiles tiles take (the last ones may find no tile)
inline int64_t blocks_of_tiles(int64_t n_tiles)
{
    return tiles_by_xcd(n_tiles) ? ceil_div(n_tiles, XCD_TILES * NUM_XCD) * (XCD_TILES * NUM_XCD) : n_tiles;
}

// ---- pass 1: neighbours per (cell, tile) ----------------------------------------------------------
// Eight lanes read a centre's list, four words each at a time.  Consecutive neighbours often fall in one cell, so that every
// lane of a half wave has a column of counters of its own.  A block takes several consecutive tiles where there are enough for
// the device, so that the sums of its tiles lie side by side in its stores: one tile per block stored six million words one by one
// (three sides of 1 M points with 32 neighbours: 236 us, so 155).  The three reads that depend on each other (centre, length, list)
// are on their way two, one and one tile ahead, as a block has no other to wait beside (with one tile per block that changed nothing).
constexpr int COUNT_THREADS = 8 * TILE;
// Without lists (2^24 points and more, most calls with the smallest workspace) this pass and the next search, one wave per centre.  The
// latency of a search wants company: with few tiles sixteen waves per tile (20 000 -> 5 000 points, 23 neighbours, 27 cells, smallest
// workspace: the build 104 us with eight waves here and four in the next pass, so 62); with many there is enough, and small
// blocks wait less (250 000 points, 21 neighbours: 486 us, with sixteen waves 551).
constexpr int64_t MANY_TILES = 2048;
constexpr int SEARCH_THREADS = 1024;
constexpr int64_t COUNT_BLOCKS = 2048;                     // blocks wanted before a block takes more tiles
constexpr int COUNT_COLS = 32, COUNT_PITCH = COUNT_COLS + 1;
constexpr int COUNT_TILES = 16;                            // at most that many tiles per block, whose sums are written together
constexpr size_t count_lds_bytes(int K, bool mirror) { return (size_t)K * (COUNT_PITCH + COUNT_TILES) * sizeof(uint32_t) * (mirror ? 2 : 1); }
typedef uint32_t list_words __attribute__((ext_vector_type(4), aligned(4)));     // (a list may start at any word)

template <bool EXT>
__global__ __launch_bounds__(SEARCH_THREADS, 8) void tile_count(const Sides sides, int K, int tiles_per_block, const uint32_t *__restrict__ err)
{
    extern __shared__ uint32_t tbl[];                      // [K][COUNT_PITCH] and [K][COUNT_TILES], each twice with mirror_sums
    __shared__ uint32_t searched[2];                       // tile's parity: a centre of it has no list
    const Side &s = sides.s[blockIdx.y];
    const int64_t t0 = (int64_t)blockIdx.x * tiles_per_block;
    const int64_t t1 = t0 + tiles_per_block < s.n_tiles ? t0 + tiles_per_block : s.n_tiles;
    if (*err || t0 >= t1) return;                          // block-uniform: the grid's offsets are not to be trusted
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int PITCH = COUNT_PITCH;
    const int threads = blockDim.x, waves = threads >> 6;
    const bool mirror = s.mirror_sums != nullptr;
    uint32_t *tbl2 = tbl + K * PITCH, *col = tbl + (tid & 31);
    uint32_t *sums = tbl + K * PITCH * (mirror ? 2 : 1), *sums2 = sums + K * COUNT_TILES;
    const int al = tid >> 3, l = tid & 7;
    auto centre_of = [&](int64_t tile) -> int32_t {        // -1: none
        const int64_t slot = tile * TILE + al;
        return al < TILE && tile < t1 && slot < s.n_centres ? (s.perm ? s.perm[slot] : (int32_t)slot) : -1;
    };
    auto found_of = [&](int32_t c) -> uint32_t { return c >= 0 && s.lists.hits ? s.lists.found[c] : 0u; };
    auto words_of = [&](size_t list, uint32_t n, uint32_t e) -> list_words {
        // (a last piece may read past the list, not past the room behind the lists)
        return e < n ? *reinterpret_cast<const list_words *>(s.lists.hits + list + e) : list_words{0u, 0u, 0u, 0u};
    };
    // (the few long lists are not read ahead)
    auto ahead_of = [&](int32_t c, uint32_t f) -> list_words { return words_of((size_t)c * s.lists.stride, f & LONG_LIST ? 0u : f, 4u * l); };
    int32_t c_now = centre_of(t0), c_next = centre_of(t0 + 1), c_after = centre_of(t0 + 2);
    uint32_t f_now = found_of(c_now), f_next = found_of(c_next);
    list_words w_now = ahead_of(c_now, f_now);
    for (int i = tid; i < K * PITCH * (mirror ? 2 : 1); i += threads) tbl[i] = 0u;
    if (tid < 2) searched[tid] = 0u;
    lds_barrier();
    for (int64_t tile = t0; tile < t1; ++tile) {
        const list_words w_next = ahead_of(c_next, f_next);
        const uint32_t f_after = found_of(c_after);
        const int32_t c_third = centre_of(tile + 3);
        uint32_t n = f_now;
        size_t list = (size_t)c_now * s.lists.stride;
        list_words w = w_now;
        if (f_now & LONG_LIST) {
            n = 0u;
            if (has_long_list(f_now)) {
                list = s.lists.long_at(f_now) + 1;
                n = s.lists.hits[list - 1];
                w = words_of(list, n, 4u * l);
            }
        }
        for (uint32_t e = 4u * l; e < n;) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (e + j < n) atomicAdd(&col[(w[j] >> HIT_INDEX_BITS) * PITCH], 1u);
            e += 32u;
            if (e < n) w = words_of(list, n, e);
        }
        if (c_now >= 0 && (!s.lists.hits || has_no_list(f_now))) searched[tile & 1] = 1u;
        lds_barrier();
        if (tid == 0) searched[(tile + 1) & 1] = 0u;       // (read before the last barrier, written behind the next)
        if (searched[tile & 1]) {                          // (block-uniform)
            // centres without a list: searched, one wave per centre
            for (int a = wave; a < TILE; a += waves) {
                const int64_t slot = tile * TILE + a;
                if (slot >= s.n_centres) break;            // wave-uniform
                const int64_t c = s.perm ? (int64_t)s.perm[slot] : slot;
                if (s.lists.hits && !has_no_list((uint32_t)__builtin_amdgcn_readfirstlane((int)s.lists.found[c]))) continue;
                Candidates<EXT> cand;
                cand.open(s.centres, c, s.g, s.q, lane);
                uint32_t found = 0;
                for (uint32_t base = 0; base < cand.st.total; base += 64) {
                    int b, k, k2;
                    const bool hit = cand.fetch(base + lane, s.g, s.q, b, k, k2);
                    if (hit) {
                        atomicAdd(&col[k * PITCH], 1u);
                        if (mirror) atomicAdd(&tbl2[k2 * PITCH + (tid & 31)], 1u);
                    }
                    found += (uint32_t)__popcll(__ballot(hit));
                }
                if (!s.lists.hits && lane == 0) s.lists.found[c] = found;
            }
            lds_barrier();
        }
        for (int i = tid; i < 4 * K; i += threads) { // four threads per cell, which also clear its counters
            const int k = i >> 2;
            auto row_sum = [&](uint32_t *row) -> uint32_t {
                uint32_t v = 0u;
#pragma unroll
                for (int j = 0; j < COUNT_COLS / 4; ++j) { v += row[j]; row[j] = 0u; }
                v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xb1, 0xf, 0xf, true);       // neighbours in the group of four
                return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4e, 0xf, 0xf, true);
            };
            const uint32_t at = (uint32_t)(k * PITCH + (i & 3) * (COUNT_COLS / 4));
            const uint32_t v = row_sum(tbl + at), v2 = mirror ? row_sum(tbl2 + at) : 0u;
            if ((i & 3) == 0) {
                sums[k * COUNT_TILES + (int)(tile - t0)] = v;
                if (mirror) sums2[k * COUNT_TILES + (int)(tile - t0)] = v2;
            }
        }
        lds_barrier();
        c_now = c_next; f_now = f_next; w_now = w_next;
        c_next = c_after; f_next = f_after;
        c_after = c_third;
    }
    for (int i = tid; i < K * COUNT_TILES; i += threads) {
        const int64_t tile = t0 + i % COUNT_TILES, at = (int64_t)(i / COUNT_TILES) * s.n_tiles + tile;
        if (tile < t1) {
            s.sums[at] = sums[i];
            if (mirror) s.mirror_sums[at] = sums2[i];
        }
    }
}

// ---- pass 2: write every triplet to its place in (k, centre, other) order ----------------------
// One block per tile.  A thread takes up to FILL_ROUNDS neighbours of the tile's centres; an LDS add per neighbour counts its
// (cell, centre) run and hands it a place there, in whatever order; the counts become run starts; the neighbours go to a list
// in LDS, run by run; and a neighbour's rank among the smaller candidate indices of its run is its final place, so ties between
// equal (k, centre) are ordered by the other index without any global sort.  The list lies in (cell, centre) order, as the
// output does, so that a wave's stores cover a few contiguous pieces of the output.  Tiles with more neighbours than the list holds are done some
// centres at a time.
//   LDS: [K][FILL_PITCH] runs, two centres to a word (a list has fewer than 2^16 places); [K] first triplet of the tile (or of
//   its part) in cell k; [K] how many there are; [K] where they start in the list; [K] whether run_start wants the row; the list: candidate index, (cell | centre << 8)
// With 125 cells the vector ALU issues in 70 % of the cycles and 2 GB pass at 2.9 TB/s (1 M points, three sides: 660 us); a fifth of
// the vector instructions less changed nothing, the rows of run_start that nobody reads left out took 766 to 660.
constexpr int FILL_PITCH = TILE / 2 + 1;  // (a half wave works on one centre, i.e. one column)
constexpr int FILL_ROUNDS = 8;           // places of the list per thread
constexpr size_t fill_table_bytes(int K) { return (size_t)K * (FILL_PITCH + 4) * sizeof(uint32_t); }
// A block's threads and places.  Small blocks wait less at the phases' barriers (eight clouds of 100 000 points, 27 cells: the
// build 680 us with 256 threads, 713 with 512), as long as the neighbours of a tile, `load` as a guess, fit their list.
struct FillShape { int threads; uint32_t list_cap; size_t lds; };
constexpr FillShape fill_shape_of(int K, int threads)
{
    const size_t most = (size_t)(threads / 256 * 20 - 1) * 1024, table = fill_table_bytes(K);       // (160 KB per CU)
    size_t n = table < most ? (most - table) / 6 / 2 * 2 : 0;
    if (n > (size_t)FILL_ROUNDS * threads) n = (size_t)FILL_ROUNDS * threads;
    return FillShape{threads, (uint32_t)n, table + n * 6};
}
constexpr FillShape fill_shape(int K, int64_t load)
{
    for (int threads = 256; threads < 1024; threads *= 2)
        if ((int64_t)fill_shape_of(K, threads).list_cap >= load && fill_shape_of(K, threads).list_cap >= 1024) return fill_shape_of(K, threads);
    return fill_shape_of(K, 1024);
}
static_assert(fill_shape_of(MAX_K, 1024).list_cap >= 4096, "the list has room beside the largest table");
static_assert(FILL_ROUNDS * 1024 < 65536, "runs count in 16 bits");

template <bool EXT>
__global__ __launch_bounds__(1024, 8) void tile_fill(const Sides sides, int K, int64_t most_tiles, uint32_t list_cap,
                                                    const uint32_t *__restrict__ err)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t tbl[];
    __shared__ TileCentres tc;
    const Side &s = sides.s[blockIdx.y];
    const int64_t tile = tile_of_block(blockIdx.x, most_tiles);
    if (*err || tile >= s.n_tiles) return;                 // block-uniform: a prefix sum of this build gave up
    uint32_t *first = tbl + K * FILL_PITCH, *row_n = first + K, *to_list = row_n + K, *read = to_list + K, *list = read + K;
    uint16_t *list_at = reinterpret_cast<uint16_t *>(list + list_cap);
    const int threads = blockDim.x, n_waves = threads >> 6;
    int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t total = s.ptr[(size_t)K * s.n_tiles];
    // start of every cell's segment (Sec. 3.3.2): the offset of its first tile; entry K is |T|
    if (s.seg_out && tile == 0)
        for (int k = tid; k <= K; k += threads) s.seg_out[k] = (int64_t)s.ptr[(size_t)k * s.n_tiles];
    if (total > s.out.out_cap) return;                     // no room: the call is going to say so
    const uint32_t out_cap = s.out.out_cap;
    int32_t *out_b = s.out.out_b;
    const bool flag_last = s.out.tail_index >= 0;
    if (flag_last)
        out_b = reinterpret_cast<int32_t *>(s.out.tail + (size_t)s.out.tail_index * (((size_t)total * 4 + 255) / 256 * 256));
    int32_t *out_c = s.out.out_c, *out_k = s.out.out_k;
    auto clear = [&]() {
        for (uint32_t i = tid; i < (uint32_t)(K * FILL_PITCH) / 4u; i += threads) reinterpret_cast<uint4 *>(tbl)[i] = make_uint4(0u, 0u, 0u, 0u);
        if (tid < ((K * FILL_PITCH) & 3)) tbl[((K * FILL_PITCH) & ~3) + tid] = 0u;
    };
    auto emit = [&](uint32_t pos, int al, int k, uint32_t b, bool last) {
        if (pos >= out_cap) return;
        if (out_c) out_c[pos] = tc.at[al];
        if (out_b) out_b[pos] = (int32_t)(flag_last && last ? b | GATHER_LAST : b);
        if (out_k) out_k[pos] = k;
    };
    clear();
    // In spatial order the rows of run_start that no kernel reads are not written either: those of cells without a triplet in
    // this tile and in the one beside it (a kernel that takes tiles in pairs reads both rows of a cell; 1 M points of a ground
    // scene, 125 cells: six rows in ten).  In index order nearly all cells hold one, and a kernel that need not look at the
    // tiles' bounds starts sooner (64 -> 128 strided layer: 1 %).
    const int64_t pair = tile & ~(int64_t)1, pair_end = pair + 2 < s.n_tiles ? pair + 2 : s.n_tiles;
    for (int k0 = 64 * wave; k0 < K; k0 += threads) {
        const int k = k0 + lane;
        bool wanted = false;
        if (k < K) {
            const uint32_t *ptr = s.ptr + (size_t)k * s.n_tiles;
            first[k] = ptr[tile];
            wanted = !s.rows || ptr[pair] != ptr[pair_end];
            read[k] = wanted;
        }
        const unsigned long long mask = __ballot(wanted);
        if (s.rows && lane == 0) s.rows[tile * mask_words(K) + (k0 >> 6)] = mask;
    }
    if (wave == 0) tc.open(s, tile, lane);
    lds_barrier();
    const uint32_t upto = tc.off[lane + 1];
    char *run_start = s.run_start ? reinterpret_cast<char *>(s.run_start + (size_t)tile * K * TILE) : nullptr;
    // as many centres at a time as the list holds: usually all of them
    int c0 = 0;
    for (;;) {
        tid = here(tid);
        lane = tid & 63;
        const uint32_t before = c0 > 0 ? lane_value(upto, c0 - 1) : 0u;
        const int c1 = c0 + (int)__popcll(__ballot(lane >= c0 && upto - before <= list_cap));
        if (c1 == c0) {
            // a centre with more neighbours than the list holds: rank each one by scanning the candidates again
            for (int k = tid; k < K; k += threads) row_n[k] = 0u;
            lds_barrier();
            Candidates<EXT> cand;
            cand.open(s.centres, tc.at[c0], s.g, s.q, lane);
            for (uint32_t base = (uint32_t)wave * 64u; base < cand.st.total; base += (uint32_t)threads) {
                int b, k, k2;
                if (cand.fetch(base + lane, s.g, s.q, b, k, k2)) atomicAdd(&row_n[k], 1u);
            }
            lds_barrier();
            for (uint32_t base = (uint32_t)wave * 64u; base < cand.st.total; base += (uint32_t)threads) {
                int b, k, k2;
                const bool hit = cand.fetch(base + lane, s.g, s.q, b, k, k2);
                uint32_t rank = 0;
                for (uint32_t other = 0; other < cand.st.total; ++other) {
                    int b2, k3, k4;
                    const bool hit2 = cand.fetch(other, s.g, s.q, b2, k3, k4);
                    rank += (hit2 && k3 == k && b2 < b) ? 1u : 0u;
                }
                if (hit) emit(first[k] + rank, c0, k, (uint32_t)b, rank + 1u == row_n[k]);
            }
            if (run_start)
                for (int k = tid; k < K; k += threads)
                    if (read[k]) reinterpret_cast<uint32_t *>(run_start)[k * TILE + c0] = first[k];
            lds_barrier();
            for (int k = tid; k < K; k += threads) first[k] += row_n[k];
            if (++c0 == TILE) break;
            lds_barrier();
            continue;
        }
        const uint32_t n = lane_value(upto, c1 - 1) - before;
        // ---- neighbours without a list: searched again, one wave per centre, left in the list for the threads that take them --
        if (tc.searched) {                                 // (block-uniform)
            for (int al = c0 + wave; al < c1; al += n_waves) {
                if (__builtin_amdgcn_readfirstlane((int)(tc.n(al) == 0u || (s.lists.hits && !has_no_list(tc.found[al]))))) continue;
                const int lane = here(tid & 63);
                Candidates<EXT> cand;
                cand.open(s.centres, tc.at[al], s.g, s.q, lane);
                uint32_t at = tc.off[al] - before;
                for (uint32_t base = 0; base < cand.st.total; base += 64) {
                    int b, k, k2;
                    const bool hit = cand.fetch(base + lane, s.g, s.q, b, k, k2);
                    const unsigned long long mask = __ballot(hit);
                    const uint32_t p = at + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
                    if (hit && p < list_cap) {
                        list[p] = (uint32_t)b;
                        list_at[p] = (uint16_t)k;
                    }
                    at += (uint32_t)__popcll(mask);
                }
            }
            lds_barrier();
        }
        // ---- a thread's consecutive neighbours: candidate index; cell | centre << 8 | place in the run << 14 -----------------
        const int rounds = (int)((n + (uint32_t)threads - 1u) / (uint32_t)threads);       // at most FILL_ROUNDS
        const uint32_t p0 = (uint32_t)(tid * rounds), mine = p0 < n ? (n - p0 < (uint32_t)rounds ? n - p0 : (uint32_t)rounds) : 0u;
        uint32_t b_of[FILL_ROUNDS], at_of[FILL_ROUNDS];
        if (mine > 0u) {
            TileCentres::Cursor c = tc.cursor(p0 + before);
#pragma unroll
            for (int j = 0; j < FILL_ROUNDS; ++j) {
                b_of[j] = at_of[j] = 0u;
                if (j < rounds && (uint32_t)j < mine) {    // (the first: block-uniform)
                    const uint32_t p = p0 + before + j;
                    tc.advance(c, p);
                    at_of[j] = (uint32_t)c.al << 8;
                    const uint32_t first = tc.off[c.al];
                    size_t at = (size_t)tc.at[c.al] * s.lists.stride;
                    bool listed = c.end - first <= s.lists.stride;
                    if (!listed && has_long_list(tc.found[c.al])) {
                        at = s.lists.long_at(tc.found[c.al]) + 1;
                        listed = true;
                    }
                    if (listed) {
                        b_of[j] = s.lists.hits[at + (p - first)];
                    } else {
                        b_of[j] = list[p0 + j];
                        at_of[j] |= list_at[p0 + j] | 1u << 31;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < FILL_ROUNDS; ++j)
                if (j < rounds && (uint32_t)j < mine) {
                    if (!(at_of[j] >> 31)) {
                        at_of[j] |= b_of[j] >> HIT_INDEX_BITS;
                        b_of[j] &= HIT_INDEX_MASK;
                    }
                    const uint32_t al = (at_of[j] >> 8) & 63u, sh = 16u * (al & 1u);
                    const uint32_t was = atomicAdd(&tbl[(at_of[j] & 255u) * FILL_PITCH + (al >> 1)], 1u << sh);
                    at_of[j] = (at_of[j] & 0x3fffu) | ((was >> sh) & 0xffffu) << 14;
                }
        }
        lds_barrier();
        // ---- counts -> starts within the part's triplets of the cell, eight cells per wave --------------------------------
        for (int k0 = 8 * wave; k0 < K; k0 += 8 * n_waves) {
            const int k = k0 + (lane >> 3), l = lane & 7;  // eight lanes per cell, eight centres per lane
            uint32_t *word = tbl + (k < K ? k : K - 1) * FILL_PITCH + 4 * l;
            uint32_t v[4], s0[4], s1[4], sum = 0u;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = word[i];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                s0[i] = sum;
                s1[i] = sum + (v[i] & 0xffffu);
                sum = s1[i] + (v[i] >> 16);
            }
            uint32_t incl = sum;                           // over the eight lanes: shifts inside a row of sixteen, which holds two cells
            const uint32_t u1 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x111, 0xf, 0xf, true);
            incl += l >= 1 ? u1 : 0u;
            const uint32_t u2 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x112, 0xf, 0xf, true);
            incl += l >= 2 ? u2 : 0u;
            const uint32_t u4 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, 0x114, 0xf, 0xf, true);
            incl += l >= 4 ? u4 : 0u;
            const uint32_t lead = incl - sum;
            if (k < K) {
#pragma unroll
                for (int i = 0; i < 4; ++i) word[i] = (lead + s0[i]) | (lead + s1[i]) << 16;
                if (l == 7) { row_n[k] = incl; word[4] = incl; }
                if (run_start && read[k]) {
                    const uint32_t f = first[k] + lead, at = (uint32_t)(k * TILE + 8 * l) * 4u;
                    if (c0 == 0 && c1 == TILE) {
#pragma unroll
                        for (int i = 0; i < 2; ++i)
                            *reinterpret_cast<uint4 *>(run_start + at + 16 * i) = make_uint4(f + s0[2 * i], f + s1[2 * i], f + s0[2 * i + 1], f + s1[2 * i + 1]);
                    } else {
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            if (8 * l + i >= c0 && 8 * l + i < c1) *reinterpret_cast<uint32_t *>(run_start + at + 4 * i) = f + (i & 1 ? s1[i / 2] : s0[i / 2]);
                    }
                }
            }
        }
        lds_barrier();
        // ---- places ----------------------------------------------------------------------------------------------------
        if (wave == 0) {
            uint32_t run = 0;
            for (int k0 = 0; k0 < K; k0 += 64) {
                const int k = k0 + lane;
                const uint32_t m = k < K ? row_n[k] : 0u;
                const uint32_t incl = wave_incl_scan_u32(m);
                if (k < K) to_list[k] = run + incl - m;
                run += lane_value(incl, 63);
            }
        }
        lds_barrier();
#pragma unroll
        for (int j = 0; j < FILL_ROUNDS; ++j)
            if (j < rounds && (uint32_t)j < mine) {
                const uint32_t k = at_of[j] & 255u, al = (at_of[j] >> 8) & 63u;
                const uint32_t place = to_list[k] + ((tbl[k * FILL_PITCH + (al >> 1)] >> (16u * (al & 1u))) & 0xffffu) + (at_of[j] >> 14);
                list[place] = b_of[j];
                list_at[place] = (uint16_t)(at_of[j] & 0x3fffu);
            }
        lds_barrier();
        // ---- ranks, and out ----------------------------------------------------------------------------------------------
        for (uint32_t p = tid; p < n; p += threads) {
            const uint32_t b = list[p], at = list_at[p];
            const int k = (int)(at & 255u), al = (int)(at >> 8);
            const uint32_t *word = tbl + k * FILL_PITCH + (al >> 1);       // (behind the last centre: the end of its run)
            const uint32_t bounds = __builtin_amdgcn_alignbit(word[1], word[0], 16u * (al & 1u));
            const uint32_t prev = bounds & 0xffffu, m = (bounds >> 16) - prev;
            const uint32_t *run = list + to_list[k] + prev;
            uint32_t rank = 0;
            for (uint32_t j = 0; j < m; j += 4) {          // (reads past the run stay inside the block's LDS)
#pragma unroll
                for (int i = 0; i < 4; ++i) rank += (uint32_t)(run[j + i] < b) & (uint32_t)(j + i < m);
            }
            emit(first[k] + prev + rank, al, k, b, rank + 1u == m);
        }
        if (c1 == TILE) break;
        lds_barrier();
        clear();
        for (int k = tid; k < K; k += threads) first[k] += row_n[k];
        lds_barrier();
        c0 = c1;
    }
}

// ---- voxel-grid down-sampling that keeps original coordinates (Sec. 4.1) ----------------------------------------
// One point per occupied voxel of pitch v: the one with the lowest index.  The voxels go through the same kind of
// hash table as the search grid; every slot keeps the lowest index inserted into it.

__global__ __launch_bounds__(256) void sub_clear(unsigned long long *__restrict__ keys, int *__restrict__ lowest,
                                                 int64_t slots, unsigned long long *__restrict__ zero_from,
                                                 int64_t zero_words)
{
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < slots; i += stride) {
        keys[i] = EMPTY_KEY;
        lowest[i] = 0x7fffffff;
    }
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < zero_words; i += stride) zero_from[i] = 0ull;
}

__global__ __launch_bounds__(256) void sub_insert(const float *__restrict__ xyz, int64_t n, double v,
                                                  unsigned long long *__restrict__ keys, int *__restrict__ lowest,
                                                  uint32_t mask, uint32_t *__restrict__ point_slot)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    int c[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) c[a] = (int)fmin(fmax(voxel_of(xyz[3 * p + a], v), -CELL_CLAMP), CELL_CLAMP);
    const unsigned long long key = pack_key(c[0], c[1], c[2]);
    uint32_t slot = hash_key(key) & mask;
    for (;;) {
        unsigned long long prev = atomicCAS(&keys[slot], EMPTY_KEY, key);
        if (prev == EMPTY_KEY || prev == key) break;
        slot = (slot + 1) & mask;
    }
    atomicMin(&lowest[slot], (int)p);
    point_slot[p] = slot;
}

__global__ __launch_bounds__(256) void sub_flag(int64_t n, const int *__restrict__ lowest,
                                                const uint32_t *__restrict__ point_slot, uint32_t *__restrict__ flag)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) flag[p] = lowest[point_slot[p]] == (int)p ? 1u : 0u;
}

// pos = exclusive prefix sum of the flags, computed in place over them: a point is kept iff pos[p + 1] > pos[p]
__global__ __launch_bounds__(256) void sub_scatter(int64_t n, const uint32_t *__restrict__ pos, int32_t *__restrict__ kept,
                                                   const uint32_t *__restrict__ err)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n || *err) return;
    if (pos[p + 1] != pos[p]) kept[pos[p]] = (int32_t)p;
}

// ---- host side ------------------------------------------------------------------------------

struct GridScratch {
    size_t keys_off, cnt_off, point_at_off, pts_off, end;
    int64_t slots;
};

int64_t grid_slots(int64_t n)
{
    int64_t s = 64;
    while (s < 2 * n) s <<= 1;
    return s;
}

struct SubScratch {
    size_t err_off, total_off, scan_off, keys_off, lowest_off, slot_off, flag_off, end;
    int64_t slots;
};

SubScratch sub_scratch(int64_t n)
{
    SubScratch s;
    s.slots = grid_slots(n);
    size_t off = 0;
    s.err_off = off;    off += 256;
    s.total_off = off;  off += 256;
    s.scan_off = off;   off += scan_scratch_bytes(n > 0 ? n : 1);
    s.keys_off = off;   off += align_up((size_t)s.slots * 8);
    s.lowest_off = off; off += align_up((size_t)s.slots * 4);
    s.slot_off = off;   off += align_up((size_t)(n > 0 ? n : 1) * 4);
    s.flag_off = off;   off += align_up((size_t)(n + 1) * 4);
    s.end = off;
    return s;
}

GridScratch grid_scratch(size_t base, int64_t n)
{
    GridScratch s;
    s.slots = grid_slots(n);
    size_t off = base;
    s.keys_off = off;        off += align_up((size_t)s.slots * 8);
    s.cnt_off = off;         off += align_up((size_t)(s.slots + 1) * 4);
    s.point_at_off = off;    off += align_up((size_t)(n > 0 ? n : 1) * 8);
    s.pts_off = off;         off += align_up((size_t)(n > 0 ? n : 1) * 16);
    s.end = off;
    return s;
}

// prefix sums of one build, each with status words of its own: the two grids, the public (k, o, i) list, the
// two sides of a spatial plan (or the input-gradient side of a plain one), and the passes of two spatial sorts
constexpr int SCAN_GRID_IN = 0, SCAN_GRID_OUT = 1, SCAN_PUBLIC = 2, SCAN_FWD_SIDE = 3, SCAN_BWD_SIDE = 4,
              SCAN_SORT_OUT = 5, SCAN_SORT_IN = SCAN_SORT_OUT + SPATIAL_ORDER_SCANS,
              N_SCANS = SCAN_SORT_IN + SPATIAL_ORDER_SCANS;

struct BuildScratch {
    GridScratch grid_in, grid_out;
    size_t err_off;                  // one word: raised by a prefix sum whose wait ran out
    size_t total_off;                // |T| as the prefix sum leaves it, when the caller's landing word is pageable
    size_t scan_off;                 // status words of the prefix sums: N_SCANS regions of scan_stride bytes
    size_t scan_stride;
    size_t fwd_ptr_off, bwd_ptr_off; // per-(k, tile) sums; of the public list, their offsets
    size_t fwd_tbl_off = 0, bwd_tbl_off = 0;         // K words per centre of a tile: neighbour lists in the smallest workspace
    size_t sort_off;                 // scratch of the spatial sorts
    size_t end;                      // what a call needs
    // The centres' neighbour lists.  How many neighbours each has lies where the grids kept their points' places.
    struct SideLists {
        bool on = false;
        uint32_t stride = 0;
        size_t found_off = 0, hits_off = 0;
        int64_t long_units = 0;          // room behind the lists of the stride
    };
    SideLists fwd, bwd;
    bool grid = true;
    bool own_rows = false;           // without a grid: room for all candidates of each centre
    size_t end_with_lists;
};

// Small clouds do without a grid: every centre looks at every candidate, which takes less than the four launches of a grid
// (with one and without, us: 2048 points, build and forward pass, 82 and 72; the build of 2800 points 62 and 58; of 4096, past
// the line, 65 and 78).
constexpr int64_t NO_GRID_POINTS = 8192, NO_GRID_PAIRS = (int64_t)1 << 23;     // most that a search without a grid looks at
bool small_clouds(int64_t n_in, int64_t n_out)
{
    return n_in > 0 && n_out > 0 && n_in <= NO_GRID_POINTS && n_out <= NO_GRID_POINTS && n_in * n_out <= NO_GRID_PAIRS;
}

// Stride of the lists: twice the mean neighbour count, within [32, most]; longer ones lie further apart (three times the mean: builds
// of 0.8 and 1 M points 2.5 % slower).  In crowded clouds, which are mostly uneven ones, `most`: a centre with more neighbours is
// searched a second time to fill its long list (115 200 points of a spinning lidar, 162 neighbours, up to 460 and more, both sides: 714 us
// with 256, 654 so; 30 000 points with 338 neighbours 434 and 306).
constexpr int64_t CROWDED = 128, MIN_STRIDE = 32;
uint32_t hit_stride_for(int64_t capacity, int64_t n_centres, int64_t most)
{
    if (n_centres <= 0 || capacity <= 0) return 0;
    const int64_t mean = ceil_div(capacity, n_centres);
    int64_t s = mean >= CROWDED ? most : (2 * mean + 15) / 16 * 16;
    if (s < MIN_STRIDE) s = MIN_STRIDE;
    if (s > most) s = most;
    return (uint32_t)s;
}

constexpr int64_t LARGE_CLOUD = 1 << 16;
constexpr int64_t LIST_SLACK = 4;        // words that a read of four words may take past the last list
// Room for the long lists of a call with `capacity` triplets, in units: a list of n > 32 words takes at most (n + 4) / 4.
constexpr int64_t long_units_for(int64_t capacity) { return (capacity + capacity / 8) / LONG_UNIT + 1; }
static_assert(8 * (int64_t)LONG_UNIT <= MIN_STRIDE, "the lengths and the unused words of long lists are an eighth at most");

BuildScratch build_scratch(int64_t n_in, int64_t n_out, int K, bool tables = true)
{
    BuildScratch b;
    b.grid_in = grid_scratch(0, n_in);
    b.grid_out = grid_scratch(b.grid_in.end, n_out);
    size_t off = b.grid_out.end;
    const int64_t nt_o = ceil_div(n_out, TILE), nt_i = ceil_div(n_in, TILE);
    int64_t scan_n = b.grid_in.slots > b.grid_out.slots ? b.grid_in.slots : b.grid_out.slots;
    if ((int64_t)K * nt_o > scan_n) scan_n = (int64_t)K * nt_o;
    if ((int64_t)K * nt_i > scan_n) scan_n = (int64_t)K * nt_i;
    const int64_t n_max = n_in > n_out ? n_in : n_out;
    if (spatial_order_scan_items(n_max) > scan_n) scan_n = spatial_order_scan_items(n_max);
    b.err_off = off;     off += 256;
    b.total_off = off;   off += 256;
    b.scan_stride = scan_scratch_bytes(scan_n);
    b.scan_off = off;    off += N_SCANS * b.scan_stride;
    b.fwd_ptr_off = off; off += align_up((size_t)(K * nt_o + 1) * 4);
    b.fwd_tbl_off = off;
    if (tables) off += align_up((size_t)(nt_o > 0 ? nt_o : 1) * K * TILE * 4);
    b.bwd_ptr_off = off; off += align_up((size_t)(K * nt_i + 1) * 4);
    b.bwd_tbl_off = off;
    if (tables) off += align_up((size_t)(nt_i > 0 ? nt_i : 1) * K * TILE * 4);
    b.sort_off = off;    off += spatial_order_scratch_bytes(n_max);
    b.end = off;
    b.end_with_lists = off;
    b.fwd.found_off = b.grid_out.point_at_off;
    b.bwd.found_off = b.grid_in.point_at_off;
    return b;
}

// Lists with a stride of at most `most` words in place of the tables, and room for the longer ones: for all neighbours that a call
// has room for, or (own_rows) for all candidates of each centre, which needs no counter that a launch in front would have to clear.
BuildScratch build_scratch_with_lists(int64_t n_in, int64_t n_out, int K, int64_t capacity, int64_t most, bool own_rows)
{
    BuildScratch b = build_scratch(n_in, n_out, K, false);
    b.grid = !small_clouds(n_in, n_out);
    b.own_rows = own_rows;
    auto side = [&](BuildScratch::SideLists &l, int64_t n_centres, int64_t n_candidates) {
        l.hits_off = b.end_with_lists;
        if (n_centres <= 0) return;
        l.stride = hit_stride_for(capacity, n_centres, most);
        l.on = l.stride > 0;
        const int64_t all = n_centres * ((n_candidates + LONG_UNIT) / LONG_UNIT), needed = long_units_for(capacity);
        l.long_units = l.stride >= n_candidates ? 0 : own_rows || all < needed ? all : needed;
        b.end_with_lists += align_up((size_t)(n_centres * l.stride + l.long_units * LONG_UNIT + LIST_SLACK) * 4);
    };
    side(b.fwd, n_out, n_in);
    side(b.bwd, n_in, n_out);
    b.end = build_scratch(n_in, n_out, K).end;             // (no call does with less)
    if (b.end_with_lists < b.end) b.end_with_lists = b.end;
    return b;
}

// Whether most centres of an even cloud have no more than `stride` neighbours: long lists cost a second search, and the counter of
// their room takes one wave after the other (400 000 centres: 1000 us).
bool enough_for_most(int64_t stride, int64_t capacity, int64_t n_centres) { return 4 * stride >= 5 * ceil_div(capacity, n_centres); }

// The scratch of a call whose workspace has `bytes` bytes: as long lists as fit, or lists inside the tables of
// the smallest workspace; a side whose neighbours have no room there does without.
BuildScratch build_scratch_within(int64_t n_in, int64_t n_out, int K, int64_t capacity, size_t bytes)
{
    BuildScratch b = build_scratch(n_in, n_out, K);
    // stored hits carry the candidate index in HIT_INDEX_BITS bits; places among the long lists take 30
    if (capacity <= 0 || n_in >= (1 << HIT_INDEX_BITS) || n_out >= (1 << HIT_INDEX_BITS)) return b;
    if (capacity > INT32_MAX) capacity = INT32_MAX;
    const bool small = small_clouds(n_in, n_out);
    if (small) {
        const BuildScratch l = build_scratch_with_lists(n_in, n_out, K, capacity, KEEP_MAX, true);
        if (bytes >= l.end_with_lists) return l;
    }
    for (int64_t most = KEEP_MAX; most >= 32; most /= 2) {
        const BuildScratch l = build_scratch_with_lists(n_in, n_out, K, capacity, most, false);
        if (most < KEEP_MAX && ((n_out > 0 && !enough_for_most(l.fwd.stride, capacity, n_out)) || (n_in > 0 && !enough_for_most(l.bwd.stride, capacity, n_in))))
            break;
        if (bytes >= l.end_with_lists) return l;
    }
    // Inside the tables.  Without a grid a centre without a list costs a search of all candidates in each pass, so that there must be room
    // for every list; with one, three quarters of the room are for the lists of the stride.  Large clouds, where the passes that
    // search wait less, gain from whatever has a list (400 000 points with 24 neighbours, 27 cells, one side: 1062 us without, 673 so).
    auto side = [&](BuildScratch::SideLists &l, int64_t n_centres, size_t table, bool whole) -> bool {
        if (n_centres <= 0) return true;
        const int64_t room = ceil_div(n_centres, TILE) * TILE * K - LIST_SLACK, mean = ceil_div(capacity, n_centres);
        int64_t stride = whole ? (room - long_units_for(capacity) * LONG_UNIT) / n_centres : room / n_centres * 3 / 4;
        if (stride > 2 * mean) stride = 2 * mean;
        const bool most = stride > 0 && enough_for_most(stride, capacity, n_centres), some = !whole && n_centres >= LARGE_CLOUD && K >= 27;
        if (!most && !some) return false;
        if (!most) stride = room / n_centres;
        l.on = true;
        l.stride = (uint32_t)stride;
        l.long_units = most ? (room - n_centres * stride) / LONG_UNIT : 0;
        l.hits_off = table;
        return true;
    };
    if (small && side(b.fwd, n_out, b.fwd_tbl_off, true) && side(b.bwd, n_in, b.bwd_tbl_off, true)) {
        b.grid = false;
        return b;
    }
    b.fwd.on = b.bwd.on = false;
    side(b.fwd, n_out, b.fwd_tbl_off, false);
    side(b.bwd, n_in, b.bwd_tbl_off, false);
    return b;
}

// What the query for a workspace with lists answers.
size_t build_bytes_for(int64_t n_in, int64_t n_out, int K, int64_t capacity)
{
    if (capacity <= 0 || n_in >= (1 << HIT_INDEX_BITS) || n_out >= (1 << HIT_INDEX_BITS)) return build_scratch(n_in, n_out, K).end;
    return build_scratch_with_lists(n_in, n_out, K, capacity < INT32_MAX ? capacity : INT32_MAX, KEEP_MAX, small_clouds(n_in, n_out)).end_with_lists;
}

// scan_scratch: the status words of this grid's prefix sum.  clear_words > 0: the first grid of a build, whose
// clearing kernel also zeroes the error word and the status words of all the build's prefix sums (they follow
// the error word in the workspace).
int build_grid(const float *xyz, int64_t n, const GridMap &gm, const int32_t *batch_off, int n_batches, char *ws,
               const GridScratch &gs, void *scan_scratch, unsigned long long *clear_from, int64_t clear_words,
               uint32_t *err, GridView *view, hipStream_t stream)
{
    auto *keys = reinterpret_cast<unsigned long long *>(ws + gs.keys_off);
    auto *cnt = reinterpret_cast<uint32_t *>(ws + gs.cnt_off);
    auto *point_at = reinterpret_cast<uint2 *>(ws + gs.point_at_off);
    auto *pts = reinterpret_cast<float4 *>(ws + gs.pts_off);
    int rc;
    {
        int64_t blocks = ceil_div(gs.slots + 1, 256);
        if (blocks > 4096) blocks = 4096;
        grid_clear<<<(unsigned)blocks, 256, 0, stream>>>(keys, cnt, gs.slots, clear_from, clear_words);
        PCPP_HIP_CHECK(hipGetLastError());
    }
    if (n > 0) {
        const unsigned blocks = (unsigned)ceil_div(n, 256);
        grid_insert<<<blocks, 256, 0, stream>>>(xyz, n, gm, batch_off, n_batches, keys, cnt, (uint32_t)(gs.slots - 1),
                                                point_at);
        PCPP_HIP_CHECK(hipGetLastError());
    }
    if ((rc = scan_exclusive_u32(cnt, cnt, gs.slots, scan_scratch, nullptr, err, stream)) != PCPP_OK) return rc;
    if (n > 0) {
        const unsigned blocks = (unsigned)ceil_div(n, 256);
        grid_scatter<<<blocks, 256, 0, stream>>>(xyz, n, point_at, cnt, pts, err);
        PCPP_HIP_CHECK(hipGetLastError());
    }
    view->keys = keys;
    view->slot_start = cnt;
    view->pts = pts;
    view->mask = (uint32_t)(gs.slots - 1);
    view->map = gm;
    view->xyz = xyz;
    view->n = (int)n;
    return PCPP_OK;
}

// The event that tells the host that |T| has landed; created and destroyed inside one call.
struct CallEvent {
    hipEvent_t ev = nullptr;
    ~CallEvent() { if (ev) (void)hipEventDestroy(ev); }
};

}  // namespace

PlanLayout plan_layout(int64_t n_in, int64_t n_out, int K, int64_t n_triplets, int flags)
{
    PlanLayout p;
    const bool spatial = (flags & PCPP_PLAN_SPATIAL) != 0;
    size_t off = 256;   // header (reserved)
    auto side = [&](SideLayout &s, int64_t n_centres, bool with_gather) {
        s.n_centres = n_centres;
        s.n_tiles = ceil_div(n_centres, TILE);
        s.perm_off = off;
        if (spatial) off += align_up((size_t)(n_centres > 0 ? n_centres : 1) * 4);
        s.tile_ptr_off = off;  off += align_up((size_t)(K * s.n_tiles + 1) * 4);
        s.run_start_off = off; off += align_up((size_t)(s.n_tiles > 0 ? s.n_tiles : 1) * K * TILE * 4);
        s.rows_off = off;
        if (spatial) off += align_up((size_t)(s.n_tiles > 0 ? s.n_tiles : 1) * mask_words(K) * 8);
        if (with_gather) s.gather_index = p.n_tail++;
    };
    if (flags & PCPP_PLAN_FWD) side(p.fwd, n_out, spatial);
    if (flags & PCPP_PLAN_BWD_INPUT) side(p.bwd, n_in, true);
    p.tail_off = off;
    const size_t each = align_up((size_t)(n_triplets > 0 ? n_triplets : 1) * 4);
    if (p.fwd.gather_index >= 0) p.fwd.gather_off = off + (size_t)p.fwd.gather_index * each;
    if (p.bwd.gather_index >= 0) p.bwd.gather_off = off + (size_t)p.bwd.gather_index * each;
    p.bytes = off + (size_t)p.n_tail * each;
    return p;
}

}  // namespace pcpp

using namespace pcpp;

extern "C" {

size_t pcpp_build_triplets_workspace_bytes(int64_t n_in, int64_t n_out, int t)
{
    if (n_in < 0 || n_out < 0 || t < 1 || t > PCPP_MAX_T) return 0;
    return build_scratch(n_in, n_out, t * t * t).end;
}

size_t pcpp_build_triplets_workspace_bytes_for(int64_t n_in, int64_t n_out, int t, int64_t capacity)
{
    if (n_in < 0 || n_out < 0 || t < 1 || t > PCPP_MAX_T || capacity < 0) return 0;
    return build_bytes_for(n_in, n_out, t * t * t, capacity);
}

size_t pcpp_plan_bytes(int64_t n_in, int64_t n_out, int t, int64_t n_triplets, int plan_flags)
{
    if (n_in < 0 || n_out < 0 || t < 1 || t > PCPP_MAX_T || n_triplets < 0) return 0;
    return plan_layout(n_in, n_out, t * t * t, n_triplets, plan_flags & PLAN_FLAG_MASK).bytes;
}

int pcpp_build_triplets(const float *in_xyz, int64_t n_in, const float *out_xyz, int64_t n_out,
                        float radius, int t,
                        int32_t *tri_o, int32_t *tri_i, int32_t *tri_k, int64_t capacity,
                        int64_t *seg_offsets, int64_t *n_triplets,
                        void *plan, size_t plan_bytes, int plan_flags,
                        void *workspace, size_t workspace_bytes, void *stream_)
{
    return pcpp_build_triplets_batched(in_xyz, n_in, out_xyz, n_out, nullptr, nullptr, 1, radius, t, tri_o, tri_i, tri_k,
                                       capacity, seg_offsets, n_triplets, plan, plan_bytes, plan_flags, workspace,
                                       workspace_bytes, stream_);
}

int pcpp_build_triplets_batched(const float *in_xyz, int64_t n_in, const float *out_xyz, int64_t n_out,
                                const int32_t *in_batch_offsets, const int32_t *out_batch_offsets, int n_batches,
                                float radius, int t,
                                int32_t *tri_o, int32_t *tri_i, int32_t *tri_k, int64_t capacity,
                                int64_t *seg_offsets, int64_t *n_triplets,
                                void *plan, size_t plan_bytes, int plan_flags,
                                void *workspace, size_t workspace_bytes, void *stream_)
{
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    if (n_batches < 1 || n_batches > 65536 || ((in_batch_offsets == nullptr) != (out_batch_offsets == nullptr)) ||
        (n_batches > 1 && !in_batch_offsets)) {
        set_error("pcpp_build_triplets_batched: n_batches must be in 1..65536 and both offset arrays given (or neither, "
                  "for one cloud)");
        return PCPP_ERR_INVALID_ARG;
    }
    if (n_in < 0 || n_out < 0 || (n_in > 0 && !in_xyz) || (n_out > 0 && !out_xyz) || !n_triplets) {
        set_error("pcpp_build_triplets: null pointer or negative size");
        return PCPP_ERR_INVALID_ARG;
    }
    if (n_in >= INT32_MAX || n_out >= INT32_MAX) {
        set_error("pcpp_build_triplets: point counts must be below 2^31");
        return PCPP_ERR_UNSUPPORTED;
    }
    if (!(radius > 0.0f) || !isfinite(radius)) {
        set_error("pcpp_build_triplets: radius must be finite and positive");
        return PCPP_ERR_INVALID_ARG;
    }
    if (t < 1 || t > PCPP_MAX_T) {
        set_error("pcpp_build_triplets: t must be in 1..%d", PCPP_MAX_T);
        return PCPP_ERR_INVALID_ARG;
    }
    const int n_null = (tri_o == nullptr) + (tri_i == nullptr) + (tri_k == nullptr);
    if (n_null != 0 && n_null != 3) {
        set_error("pcpp_build_triplets: tri_o, tri_i, tri_k must be all NULL or all non-NULL");
        return PCPP_ERR_INVALID_ARG;
    }
    const bool count_only = n_null == 3;
    if (!count_only && (capacity < 0 || !seg_offsets)) {
        set_error("pcpp_build_triplets: seg_offsets is NULL or capacity negative");
        return PCPP_ERR_INVALID_ARG;
    }
    const int test_flags = plan_flags & (PCPP_BUILD_TEST_SHORT_LISTS | PCPP_BUILD_TEST_WIDE_KEYS);
    if (plan_flags & ~(PLAN_FLAG_MASK | PCPP_BUILD_TEST_SHORT_LISTS | PCPP_BUILD_TEST_WIDE_KEYS | PCPP_BUILD_VOXEL)) {
        set_error("pcpp_build_triplets: unknown bits in plan_flags");
        return PCPP_ERR_INVALID_ARG;
    }
    const bool voxel = (plan_flags & PCPP_BUILD_VOXEL) != 0;
    const bool ext = voxel || in_batch_offsets != nullptr;     // the search kernels with the variants compiled in
    if (voxel && t % 2 == 0) {
        set_error("pcpp_build_triplets: the voxel operator needs an odd t (a centre voxel)");
        return PCPP_ERR_INVALID_ARG;
    }
    plan_flags &= PLAN_FLAG_MASK;
    if (plan && !(plan_flags & PCPP_PLAN_FWD)) {
        set_error("pcpp_build_triplets: plan_flags must include PCPP_PLAN_FWD");
        return PCPP_ERR_INVALID_ARG;
    }
    const int K = t * t * t;
    const bool wide_keys = (test_flags & PCPP_BUILD_TEST_WIDE_KEYS) != 0;
    const BuildScratch bs = build_scratch_within(n_in, n_out, K, count_only || wide_keys ? -1 : capacity, workspace_bytes);
    if (!workspace || workspace_bytes < bs.end || (reinterpret_cast<uintptr_t>(workspace) & 255)) {
        set_error("pcpp_build_triplets: workspace missing, misaligned or smaller than %zu bytes", bs.end);
        return PCPP_ERR_WORKSPACE;
    }
    if (plan && (reinterpret_cast<uintptr_t>(plan) & 255)) {
        set_error("pcpp_build_triplets: plan must be 256-byte aligned");
        return PCPP_ERR_WORKSPACE;
    }
    *n_triplets = 0;
    char *ws = static_cast<char *>(workspace);
    uint32_t *err = reinterpret_cast<uint32_t *>(ws + bs.err_off);
    auto scan_scratch = [&](int which) -> void * { return ws + bs.scan_off + (size_t)which * bs.scan_stride; };

    // Where |T| lands.  Pinned host memory is written by the device itself (the prefix sum's last block), so the
    // host can pick the count up while the second pass is already running; pageable memory gets it through a
    // blocking copy before that pass is queued.
    unsigned long long *total_dev = reinterpret_cast<unsigned long long *>(ws + bs.total_off);
    bool pinned = false;
    {
        hipPointerAttribute_t attr;
        if (hipPointerGetAttributes(&attr, n_triplets) == hipSuccess && attr.type == hipMemoryTypeHost &&
            attr.devicePointer) {
            total_dev = static_cast<unsigned long long *>(attr.devicePointer);
            pinned = true;
        } else {
            (void)hipGetLastError();                 // an unregistered pointer is reported as an error; it is not one
        }
    }

    // grid pitch a hair above r so that, with the binary64 cell computation, any accepted pair lies
    // in adjacent grid cells (27-cell stencil is conservative)
    const double R = (double)radius;
    GridMap gm;
    gm.inv_g = 1.0 / (R * (1.0 + 1.0 / 1048576.0));
    gm.vox = R;
    gm.hp = (t - 1) / 2 > 1 ? (t - 1) / 2 : 1;
    gm.voxel_mode = voxel ? 1 : 0;
    QueryParams q;
    q.R = R;
    q.r2 = R * R;
    q.inv_cell = (double)t / (2.0 * R);
    q.t = t;
    q.sign = 1.0;
    q.voxel_mode = voxel ? 1 : 0;
    q.h = (t - 1) / 2;
    q.c_off = out_batch_offsets;         // forward orientation: centres = outputs, candidates = inputs
    q.d_off = in_batch_offsets;
    q.n_batches = n_batches;
    QueryParams qs = q;                  // roles swapped: centres = inputs, candidates = outputs
    qs.sign = -1.0;
    qs.c_off = in_batch_offsets;
    qs.d_off = out_batch_offsets;

    const int64_t nt_o = ceil_div(n_out, TILE), nt_i = ceil_div(n_in, TILE);
    const bool want_plan = plan && !count_only;
    const bool want_bwd = want_plan && (plan_flags & PCPP_PLAN_BWD_INPUT);
    const bool spatial = want_plan && (plan_flags & PCPP_PLAN_SPATIAL);
    const bool self = out_xyz == in_xyz && n_out == n_in && in_batch_offsets == out_batch_offsets;

    // the offsets of everything but the |T|-sized arrays do not depend on |T|
    const PlanLayout pl = want_plan ? plan_layout(n_in, n_out, K, 0, plan_flags) : PlanLayout{};
    if (want_plan && plan_bytes < pl.bytes) {
        set_error("pcpp_build_triplets: plan buffer has %zu bytes, needs at least %zu", plan_bytes, pl.bytes);
        return PCPP_ERR_WORKSPACE;
    }
    char *pb = static_cast<char *>(plan);
    auto words = [](char *base, size_t off) { return reinterpret_cast<uint32_t *>(base + off); };

    // ---- the candidates ----------------------------------------------------------------------------------------
    const bool f_lists = bs.fwd.on, b_lists = want_bwd && bs.bwd.on, no_grid = count_only ? small_clouds(n_in, n_out) : !bs.grid;
    int rc;
    GridView grid_in{nullptr, nullptr, nullptr, 0u, gm, in_xyz, (int)n_in};
    // the error word, the total and all status words (contiguous) start at zero: the clearing kernel of the first grid sees to it
    auto *clear_from = reinterpret_cast<unsigned long long *>(ws + bs.err_off);
    const int64_t clear_words = (int64_t)((512 + N_SCANS * bs.scan_stride) / sizeof(unsigned long long));
    const bool clear_first = no_grid && !count_only && !bs.own_rows;       // (its blocks share a counter)
    if (clear_first && (rc = fill_u64(clear_from, 0ull, clear_words, stream)) != PCPP_OK) return rc;
    if (!no_grid)
        if ((rc = build_grid(in_xyz, n_in, gm, in_batch_offsets, n_batches, ws, bs.grid_in, scan_scratch(SCAN_GRID_IN), clear_from,
                             clear_words, err, &grid_in, stream)) != PCPP_OK)
            return rc;
    GridView grid_out = grid_in;
    if (want_bwd && !self) {
        if (no_grid) grid_out = GridView{nullptr, nullptr, nullptr, 0u, gm, out_xyz, (int)n_out};
        else if ((rc = build_grid(out_xyz, n_out, gm, out_batch_offsets, n_batches, ws, bs.grid_out, scan_scratch(SCAN_GRID_OUT),
                                  nullptr, 0, err, &grid_out, stream)) != PCPP_OK)
            return rc;
    }

    // ---- |T| ------------------------------------------------------------------------------------------------------
    CallEvent landed;
    unsigned long long total = 0;
    bool have_total = false;
    auto wait_total = [&]() -> int {
        if (!have_total) {
            if (pinned) {
                PCPP_HIP_CHECK(hipEventSynchronize(landed.ev));
                total = *reinterpret_cast<volatile unsigned long long *>(n_triplets);
            } else {
                PCPP_HIP_CHECK(hipMemcpyAsync(&total, total_dev, sizeof(total), hipMemcpyDeviceToHost, stream));
                PCPP_HIP_CHECK(hipStreamSynchronize(stream));
            }
            have_total = true;
        }
        if (total == ~0ull) {
            *n_triplets = 0;
            set_error("pcpp_build_triplets: a wait inside a device-wide prefix sum ran out");
            return PCPP_ERR_HIP;
        }
        *n_triplets = (int64_t)total;
        if (total >= (unsigned long long)INT32_MAX) {
            set_error("pcpp_build_triplets: %llu triplets; the library indexes at most 2^31-1", total);
            return PCPP_ERR_UNSUPPORTED;
        }
        return PCPP_OK;
    };
    // the last prefix sum is queued
    auto total_queued = [&]() -> int {
        if (!pinned) return wait_total();
        PCPP_HIP_CHECK(hipEventCreateWithFlags(&landed.ev, hipEventDisableTiming));
        PCPP_HIP_CHECK(hipEventRecord(landed.ev, stream));
        return PCPP_OK;
    };

    // ---- every centre's neighbours ----------------------------------------------------------------------------
    // Centres = outputs, candidates = inputs; for the input gradient centres = inputs, candidates = outputs: the same
    // predicate with the roles swapped, so the set is identical and only the grouping changes to (k, i, o).  A cloud
    // queried against itself is searched once for both.
    auto lists_of = [&](const BuildScratch::SideLists &l, bool on, int64_t n_centres) {
        return Lists{on ? words(ws, l.hits_off) : nullptr, words(ws, l.found_off), on ? l.stride : 0u,
                     (size_t)n_centres * l.stride};
    };
    const Lists f_l = lists_of(bs.fwd, f_lists, n_out);
    Lists b_l = lists_of(bs.bwd, b_lists, n_in);
    if (self) b_l.found = f_l.found;               // (one search or count for both)
    unsigned long long *long_used = reinterpret_cast<unsigned long long *>(ws + bs.err_off + 64);      // of the two searches; cleared with the error word
    auto search = [&](Form form, const float4 *order, const float *centres, int64_t n, const GridView &g, const QueryParams &qp) -> int {
        if (n <= 0) return PCPP_OK;
        int per_wave = 1;                          // centres: as many as leave enough waves for the device
        while (per_wave < 32 && n / (2 * per_wave) >= SEARCH_WAVES) per_wave *= 2;
        const bool in = form == INPUTS;
        const SearchArgs sa{order, centres, n, g, qp, in ? b_l : f_l, b_l.hits, (unsigned long long)(in ? bs.bwd : bs.fwd).long_units,
                            no_grid && bs.own_rows ? nullptr : long_used + (in ? 1 : 0), per_wave, err, clear_from, in || clear_first ? 0 : clear_words};
        const size_t lds = no_grid ? (size_t)(g.n < ALL_CHUNK ? g.n : ALL_CHUNK) * 3 * sizeof(float) : 0;
        auto pick = [&](auto cells, auto cells_ext, auto all, auto all_ext) { return no_grid ? (ext ? all_ext : all) : (ext ? cells_ext : cells); };
        auto kern = form == BOTH ? pick(search_cells<BOTH, false>, search_cells<BOTH, true>, search_all<BOTH, false>, search_all<BOTH, true>)
                    : form == INPUTS ? pick(search_cells<INPUTS, false>, search_cells<INPUTS, true>, search_all<INPUTS, false>, search_all<INPUTS, true>)
                                     : pick(search_cells<OUTPUTS, false>, search_cells<OUTPUTS, true>, search_all<OUTPUTS, false>, search_all<OUTPUTS, true>);
        if (lds > (size_t)32 * 1024)
            if (int r = raise_lds_limit(reinterpret_cast<const void *>(kern), lds)) return r;
        kern<<<(unsigned)ceil_div(ceil_div(n, no_grid ? 1 : per_wave), 4), 256, lds, stream>>>(sa);
        PCPP_HIP_CHECK(hipGetLastError());
        return PCPP_OK;
    };
    if (f_lists)
        if ((rc = search(self && b_lists ? BOTH : OUTPUTS, self ? grid_in.pts : (want_bwd ? grid_out.pts : nullptr), out_xyz, n_out,
                         grid_in, q)) != PCPP_OK)
            return rc;
    if (b_lists && !self)
        if ((rc = search(INPUTS, grid_in.pts, in_xyz, n_in, grid_out, qs)) != PCPP_OK) return rc;

    if (count_only) {
        // how many neighbours each output has, and their sum (as numbers per cell and tile, whose search takes one wave per centre: 20 000
        // points with 23 neighbours 70 us, so 51; 400 000 622 and 211)
        if ((rc = search(OUTPUTS, self ? grid_in.pts : nullptr, out_xyz, n_out, grid_in, q)) != PCPP_OK) return rc;
        if ((rc = scan_exclusive_u32(f_l.found, f_l.found, n_out, scan_scratch(SCAN_PUBLIC), total_dev, err, stream)) != PCPP_OK) return rc;
        if ((rc = total_queued()) != PCPP_OK) return rc;
        return wait_total();
    }

    // ---- the centres' orders --------------------------------------------------------------------------------------
    const int32_t *perm_o = nullptr, *perm_i = nullptr;
    if (spatial) {
        // cells of half the radius: a tile of 64 centres then spans a few radii at the densities the layers see
        const double pitch = 0.5 * R;
        int32_t *po = reinterpret_cast<int32_t *>(pb + pl.fwd.perm_off);
        if ((rc = spatial_order(out_xyz, n_out, pitch, po, ws + bs.sort_off, scan_scratch(SCAN_SORT_OUT), bs.scan_stride,
                                err, stream)) != PCPP_OK)
            return rc;
        perm_o = po;
        if (want_bwd) {
            int32_t *pi = reinterpret_cast<int32_t *>(pb + pl.bwd.perm_off);
            if (self) {
                PCPP_HIP_CHECK(hipMemcpyAsync(pi, po, (size_t)n_in * 4, hipMemcpyDeviceToDevice, stream));
            } else if ((rc = spatial_order(in_xyz, n_in, pitch, pi, ws + bs.sort_off, scan_scratch(SCAN_SORT_IN),
                                           bs.scan_stride, err, stream)) != PCPP_OK) {
                return rc;
            }
            perm_i = pi;
        }
    }

    // ---- the sides: the public list in index order, the plan's forward side where that differs, its input-gradient side ----
    const uint32_t tri_cap = (uint32_t)(capacity < (int64_t)INT32_MAX ? capacity : (int64_t)INT32_MAX);
    // how many triplets the |T|-sized arrays of the plan have room for
    uint32_t tail_cap = 0;
    if (want_plan && pl.n_tail > 0) {
        const size_t room = (plan_bytes - pl.tail_off) / (size_t)pl.n_tail / 256 * 256 / 4;
        tail_cap = (uint32_t)(room < (size_t)tri_cap ? room : (size_t)tri_cap);
    }
    Sides sides{};
    ScanJob jobs[MAX_SIDES] = {};
    int n_sides = 0;
    auto add_side = [&](bool outputs, const int32_t *perm, uint32_t *sums, uint32_t *ptr, int which, unsigned long long *total64,
                        uint32_t *run_start, unsigned long long *rows, int64_t *seg, const FillOut &out) {
        Side &d = sides.s[n_sides];
        d.centres = outputs ? out_xyz : in_xyz;
        d.perm = perm;
        d.n_centres = outputs ? n_out : n_in;
        d.n_tiles = outputs ? nt_o : nt_i;
        d.g = outputs ? grid_in : grid_out;
        d.q = outputs ? q : qs;
        d.lists = outputs ? f_l : b_l;
        d.sums = sums; d.mirror_sums = nullptr;
        d.ptr = ptr;
        d.run_start = run_start; d.rows = rows; d.seg_out = seg;
        d.out = out;
        jobs[n_sides++] = ScanJob{sums, ptr, (int64_t)K * d.n_tiles, scan_scratch(which), total64};
    };
    // (the sums of a plan's side lie in its own offset table, which the prefix sum replaces in place)
    uint32_t *f_ptr = want_plan ? words(pb, pl.fwd.tile_ptr_off) : nullptr, *b_ptr = want_bwd ? words(pb, pl.bwd.tile_ptr_off) : nullptr;
    auto rows_of = [&](const SideLayout &l) { return spatial ? reinterpret_cast<unsigned long long *>(pb + l.rows_off) : nullptr; };
    uint32_t *pub_ptr = want_plan && !spatial ? f_ptr : words(ws, bs.fwd_ptr_off);
    add_side(true, nullptr, pub_ptr, pub_ptr, SCAN_PUBLIC, total_dev, want_plan && !spatial ? words(pb, pl.fwd.run_start_off) : nullptr,
             nullptr, nt_o == 0 ? nullptr : seg_offsets, FillOut{tri_o, tri_i, tri_k, nullptr, -1, tri_cap});
    if (spatial)
        add_side(true, perm_o, f_ptr, f_ptr, SCAN_FWD_SIDE, nullptr, words(pb, pl.fwd.run_start_off), rows_of(pl.fwd), nullptr,
                 FillOut{nullptr, nullptr, nullptr, pb + pl.tail_off, pl.fwd.gather_index, tail_cap});
    int counted = n_sides;
    if (want_bwd) {
        add_side(false, perm_i, b_ptr, b_ptr, SCAN_BWD_SIDE, nullptr, words(pb, pl.bwd.run_start_off), rows_of(pl.bwd), nullptr,
                 FillOut{nullptr, nullptr, nullptr, pb + pl.tail_off, pl.bwd.gather_index, tail_cap});
        // without lists one search counts both sides of a cloud against itself (same tiles on both)
        if (self && !b_lists) sides.s[counted - 1].mirror_sums = b_ptr;
        else counted = n_sides;
    }
    const int64_t most_tiles = want_bwd && nt_i > nt_o ? nt_i : nt_o;
    if (most_tiles > 0) {
        int64_t per_block = most_tiles * counted / COUNT_BLOCKS;
        per_block = per_block < 1 ? 1 : (per_block > COUNT_TILES ? COUNT_TILES : per_block);
        const dim3 grid((unsigned)ceil_div(most_tiles, per_block), (unsigned)counted);
        const size_t lds = count_lds_bytes(K, sides.s[counted - 1].mirror_sums != nullptr);
        if (lds > (size_t)32 * 1024)                   // (both sides of 125 cells 49 KB, of 216 cells 85 KB)
            if ((rc = raise_lds_limit(ext ? reinterpret_cast<const void *>(&tile_count<true>) : reinterpret_cast<const void *>(&tile_count<false>),
                                      lds)) != PCPP_OK)
                return rc;
        int threads = COUNT_THREADS;
        for (int i = 0; i < counted; ++i)
            if (!sides.s[i].lists.hits && sides.s[i].n_tiles < MANY_TILES) threads = SEARCH_THREADS;
        if (ext) tile_count<true><<<grid, threads, lds, stream>>>(sides, K, (int)per_block, err);
        else tile_count<false><<<grid, threads, lds, stream>>>(sides, K, (int)per_block, err);
        PCPP_HIP_CHECK(hipGetLastError());
    }
    if ((rc = scan_exclusive_u32_jobs(jobs, n_sides, err, stream)) != PCPP_OK) return rc;
    if ((rc = total_queued()) != PCPP_OK) return rc;
    if (nt_o == 0) {
        // no outputs: every run starts at 0
        if ((rc = fill_u64(reinterpret_cast<unsigned long long *>(seg_offsets), 0ull, K + 1, stream)) != PCPP_OK) return rc;
    }
    for (int from = 0; from < n_sides;) {
        // sides whose tiles ask for blocks of one size go in one launch (capacities are on the generous side)
        auto shape_of = [&](const Side &d) {
            return d.lists.hits || d.n_tiles >= MANY_TILES ? fill_shape(K, ceil_div(capacity, d.n_tiles > 0 ? d.n_tiles : 1) * 2 / 3) : fill_shape_of(K, SEARCH_THREADS);
        };
        FillShape shape = shape_of(sides.s[from]);
        Sides part{};
        int n = 0;
        int64_t tiles = 0;
        for (; from < n_sides && shape_of(sides.s[from]).threads == shape.threads; ++from) {
            part.s[n++] = sides.s[from];
            if (sides.s[from].n_tiles > tiles) tiles = sides.s[from].n_tiles;
        }
        if (tiles == 0) continue;
        if (test_flags & PCPP_BUILD_TEST_SHORT_LISTS) shape.list_cap = 40;
        if (shape.lds > (size_t)32 * 1024)
            if ((rc = raise_lds_limit(ext ? reinterpret_cast<const void *>(&tile_fill<true>) : reinterpret_cast<const void *>(&tile_fill<false>),
                                      shape.lds)) != PCPP_OK)
                return rc;
        const dim3 grid((unsigned)blocks_of_tiles(tiles), (unsigned)n);
        if (ext) tile_fill<true><<<grid, shape.threads, shape.lds, stream>>>(part, K, tiles, shape.list_cap, err);
        else tile_fill<false><<<grid, shape.threads, shape.lds, stream>>>(part, K, tiles, shape.list_cap, err);
        PCPP_HIP_CHECK(hipGetLastError());
    }
    // everything is queued; now compare the count with what the caller provided
    if ((rc = wait_total()) != PCPP_OK) return rc;
    if ((int64_t)total > capacity) {
        set_error("pcpp_build_triplets: %llu triplets but capacity is %lld", total, (long long)capacity);
        return PCPP_ERR_CAPACITY;
    }
    if (plan) {
        const size_t need = plan_layout(n_in, n_out, K, (int64_t)total, plan_flags).bytes;
        if (plan_bytes < need) {
            set_error("pcpp_build_triplets: plan buffer has %zu bytes, needs %zu", plan_bytes, need);
            return PCPP_ERR_WORKSPACE;
        }
    }
    return PCPP_OK;
}

size_t pcpp_voxel_subsample_workspace_bytes(int64_t n)
{
    if (n < 0 || n >= INT32_MAX) return 0;
    return sub_scratch(n).end;
}

int pcpp_voxel_subsample(const float *xyz, int64_t n, float pitch, int32_t *kept, int64_t *n_kept, void *workspace,
                         size_t workspace_bytes, void *stream_)
{
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    if (n < 0 || (n > 0 && (!xyz || !kept)) || !n_kept) {
        set_error("pcpp_voxel_subsample: null pointer or negative size");
        return PCPP_ERR_INVALID_ARG;
    }
    if (n >= INT32_MAX) {
        set_error("pcpp_voxel_subsample: point count must be below 2^31");
        return PCPP_ERR_UNSUPPORTED;
    }
    if (!(pitch > 0.0f) || !isfinite(pitch)) {
        set_error("pcpp_voxel_subsample: pitch must be finite and positive");
        return PCPP_ERR_INVALID_ARG;
    }
    const SubScratch ss = sub_scratch(n);
    if (!workspace || workspace_bytes < ss.end || (reinterpret_cast<uintptr_t>(workspace) & 255)) {
        set_error("pcpp_voxel_subsample: workspace missing, misaligned or smaller than %zu bytes", ss.end);
        return PCPP_ERR_WORKSPACE;
    }
    *n_kept = 0;
    if (n == 0) return PCPP_OK;
    char *ws = static_cast<char *>(workspace);
    auto *keys = reinterpret_cast<unsigned long long *>(ws + ss.keys_off);
    int *lowest = reinterpret_cast<int *>(ws + ss.lowest_off);
    auto *point_slot = reinterpret_cast<uint32_t *>(ws + ss.slot_off);
    auto *flag = reinterpret_cast<uint32_t *>(ws + ss.flag_off);
    auto *err = reinterpret_cast<uint32_t *>(ws + ss.err_off);
    unsigned long long *total_dev = reinterpret_cast<unsigned long long *>(ws + ss.total_off);
    bool pinned = false;
    {
        hipPointerAttribute_t attr;
        if (hipPointerGetAttributes(&attr, n_kept) == hipSuccess && attr.type == hipMemoryTypeHost && attr.devicePointer) {
            total_dev = static_cast<unsigned long long *>(attr.devicePointer);
            pinned = true;
        } else {
            (void)hipGetLastError();
        }
    }
    int64_t blocks = ceil_div(ss.slots, 256);
    if (blocks > 4096) blocks = 4096;
    // the error word, the landing word and the prefix sum's status words are contiguous at the start of the workspace
    sub_clear<<<(unsigned)blocks, 256, 0, stream>>>(keys, lowest, ss.slots, reinterpret_cast<unsigned long long *>(ws),
                                                    (int64_t)(ss.keys_off / sizeof(unsigned long long)));
    const unsigned pb = (unsigned)ceil_div(n, 256);
    sub_insert<<<pb, 256, 0, stream>>>(xyz, n, (double)pitch, keys, lowest, (uint32_t)(ss.slots - 1), point_slot);
    sub_flag<<<pb, 256, 0, stream>>>(n, lowest, point_slot, flag);
    PCPP_HIP_CHECK(hipGetLastError());
    int rc;
    if ((rc = scan_exclusive_u32(flag, flag, n, ws + ss.scan_off, total_dev, err, stream)) != PCPP_OK) return rc;
    sub_scatter<<<pb, 256, 0, stream>>>(n, flag, kept, err);
    PCPP_HIP_CHECK(hipGetLastError());
    unsigned long long total = 0;
    if (pinned) {
        PCPP_HIP_CHECK(hipStreamSynchronize(stream));
        total = *reinterpret_cast<volatile unsigned long long *>(n_kept);
    } else {
        PCPP_HIP_CHECK(hipMemcpyAsync(&total, total_dev, sizeof(total), hipMemcpyDeviceToHost, stream));
        PCPP_HIP_CHECK(hipStreamSynchronize(stream));
    }
    if (total == ~0ull) {
        *n_kept = 0;
        set_error("pcpp_voxel_subsample: a wait inside a device-wide prefix sum ran out");
        return PCPP_ERR_HIP;
    }
    *n_kept = (int64_t)total;
    return PCPP_OK;
}

}  // extern "C"
