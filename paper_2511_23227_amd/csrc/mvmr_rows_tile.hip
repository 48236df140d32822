// MVMR rows kernel for any channel counts (Eq. (1) forward; Sec. 3.3.3 input gradient with W^T), fp32 or bf16 storage,
// both factors on the bf16 matrix cores.
//
// Eq. (1) is linear, so out[o] = sum_k W[k] S_k[o] with S_k[o] = the sum of x[i] over the (k, o) run.  A block owns up
// to 64 consecutive slots of the plan's centre order (one tile or a part of it) and walks the kernel cells that hold a
// triplet for any of them.
//   stage A   one wave per (cell, part of 16 GA centres): S^T [channel][centre] = X_g^T [channel][triplet] .
//             Sel^T [triplet][centre], X_g = the part's source rows of the cell, 32 triplets at a time, each row read once
//             and densely (mvmr_stage.h), Sel = 0/1 from the run bounds through an LDS table of eight-bit masks.  Products
//             with 1.0 are exact, so this is the fp32 sum of the rows; run lengths never cause divergence.  The sums go to
//             stage B as three bf16 terms that add up to the fp32 value exactly (EXACT), or, in the bf16 layers that
//             bf16_sums() lists, rounded to bf16 once.
//   stage B   acc^T [destination][centre] += W[k] [destination][channel] . S^T [channel][centre]; W comes straight from
//             memory / L2 in fragment order.  fp32 layers keep the six products of weight 2^-16 or more relative to the
//             leading one.
// Split form (SPLITK): a wave takes every NW-th cell of its block's 16 GA centres and all destination channels, and the
// waves' sums are added in wave order at the end.  The registers that stage A leaves are the operands of stage B as they
// are (W is packed in that order of the channels), so the loop has no barrier and S never goes through LDS (through LDS:
// 87 us instead of 80 for a 32 -> 32 fp32 layer of 2.4 M triplets, 280 instead of 253 for 128 -> 64 bf16 of 18 M).
// Cooperative form: the waves of a block share the S tiles of a round of cells in LDS (two sets, one barrier per round),
// and each owns 16 DTW destination channels of its centre groups: W is read once per 64 centres and the accumulators
// stay small, so several blocks per CU hide the gathers.
// Where a sum has many steps, the products of the smaller terms have sums of their own (APART), which reach the accumulators
// as ordinary additions: the matrix cores cut the low bits of an addend far below the accumulator, and with values of one sign
// these cuts add up (relative errors with one accumulator, apart, and of fp32 sums on the vector ALUs, all values positive:
// 256 -> 256 fp32, 1.5 M triplets, 8.9e-6, 4.2e-7, 1.06e-6; 512 -> 256 bf16 with 270 neighbours 2.1e-6, 6.4e-7, 1.6e-6).
// What bounds it: with 32 to 64 channels in fp32 the vector instructions, most of which split rows and sums into terms (32 ->
// 32: issued in 73 % of the cycles), in bf16 the rows' way through the L1 caches (a 64 -> 64 layer of 17 M triplets moves 2.2 GB of
// them in 141 us, 0.67 L1 accesses per cycle and CU, matrix pipe 13 %); with more channels W's way from L2.  Layers whose channel
// counts are no power of two, which the vector ALUs had served before: 20 -> 36 fp32, 0.49 M triplets, 29 us (349); 128 -> 128 bf16,
// 0.97 M triplets, 130 us (7938).
// Every destination row is written once, by one block: no atomics, fixed summation order.
//
// v_mfma_f32_16x16x32_bf16: A: lane (M = l%16, g = l/16) holds A[M][8g .. 8g+7]; B: lane (N = l%16, g) holds
// B[8g .. 8g+7][N]; D: lane l, register j -> M = 4g + j, N = l%16.
#include "mvmr_stage.h"
#include "mvmr_walk.h"

namespace pcpp {

namespace {

// packed[(((k * ndt + d) * nks + ks) * planes + p) * 64 + lane], element e
//     = term p of W(k, dst 16 d + lane%16, channel at place 32 ks + 16 (e/4) + 4 (lane/16) + e%4 of the chunks' operand
// tiles), zero where there is none: in this order of the reduction index the sums of stage A, as the matrix cores leave
// them in registers, are operands of stage B.  W(k, d, s) at w[k*c_dst*c_src + d*stride_d + s*stride_s] (covers W as stored and its transpose)
template <bool F32, bool NARROW>
__global__ __launch_bounds__(256) void pack_w_tile_kernel(const void *__restrict__ w_, v4u *__restrict__ packed, int K,
                                                          int c_src, int c_dst, int nks, int ndt, int chk, int stride_d,
                                                          int stride_s)
{
    const int64_t piece = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (piece >= (int64_t)K * ndt * nks * 64) return;
    const int lane = (int)(piece & 63);
    int64_t r = piece >> 6;
    const int ks = (int)(r % nks); r /= nks;
    const int d = 16 * (int)(r % ndt) + (lane & 15);
    const int k = (int)(r / ndt);
    const int s0 = 32 * ks + 4 * (lane >> 4);
    const size_t base = (size_t)k * c_dst * c_src + (size_t)d * stride_d;
    uint32_t t[3][8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int at_place = s0 + 16 * (e >> 2) + (e & 3), chunk = at_place / chk, place = at_place % chk;
        int ch;
        if constexpr (F32) ch = Direct<2, NARROW>::channel(chunk, place, c_src);
        else if (chk == 32) ch = Stage<4, NARROW>::channel(chunk, place, c_src);
        else ch = Stage<8, NARROW>::channel(chunk, place, c_src);
        const bool ok = d < c_dst && ch >= 0;
        const size_t at = base + (size_t)ch * stride_s;
        if constexpr (F32) {
            const float x = ok ? static_cast<const float *>(w_)[at] : 0.f;
            t[0][e] = __float_as_uint(x) & 0xffff0000u;
            const float r1 = x - __uint_as_float(t[0][e]);
            t[1][e] = __float_as_uint(r1) & 0xffff0000u;
            t[2][e] = __float_as_uint(r1 - __uint_as_float(t[1][e]));
        } else {
            t[0][e] = ok ? (uint32_t)static_cast<const uint16_t *>(w_)[at] << 16 : 0u;
        }
    }
    constexpr int PL = F32 ? 3 : 1;
#pragma unroll
    for (int p = 0; p < PL; ++p) {
        v4u v;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = __builtin_amdgcn_perm(t[p][2 * q + 1], t[p][2 * q], 0x07060302u);
        packed[((piece >> 6) * PL + p) * 64 + lane] = v;
    }
}

struct TileArgs {
    const void *feat;
    const v4u *w;
    void *dst;
    const int32_t *gather;
    PlanSideView side;
    int64_t n_centres;
    uint32_t feat_bytes, gather_bytes, row_bytes;
    int K, c_src, c_dst, n_chunks, ndt;
    int out_bf16;
};

template <bool F32, bool EXACT, int RL, bool NARROW, int GA, int NP, int NW, int WD, int DTW, bool SPLITK>
struct TileCfg {
    using St = std::conditional_t<F32, Direct<2, NARROW>, Stage<RL, NARROW>>;
    static constexpr int CHK = St::CHK, KS = CHK / 32, PL = St::PL, PLS = EXACT ? 3 : 1;     // terms of a row or of W, of a sum
    static_assert(!F32 || EXACT, "fp32 layers keep fp32 sums");
    static constexpr int NG = GA * NP, CR = NW / NP;
    static constexpr int WC = SPLITK ? 1 : NW / WD, GW = NG / WC;
    static constexpr int NBUF = (SPLITK || CR == 1) ? 1 : 2;              // sets of S tiles (one: a second barrier per step)
    static constexpr uint32_t PITCH = CHK * 2 * PLS + 16, PART = GA * 16 * PITCH;      // multiples of 256
    // a wave's staged rows lie where its sums will go, if they fit
    static constexpr bool STAGE_IN_S = SPLITK || PART >= St::BYTES;
    static constexpr uint32_t STILE = SPLITK ? St::BYTES : NP * PART;
    static constexpr uint32_t ACT = MAX_K + 1;                              // words of the list of active cells
    static constexpr uint32_t RUNS = 16 * GA + 1;
    static constexpr uint32_t OFF_ACT = 4096, OFF_BND = OFF_ACT + 4 * ACT, OFF_RUNS = OFF_BND + 4 * (NP + 1) * MAX_K;
    static constexpr uint32_t OFF_S = (OFF_RUNS + 4 * NW * RUNS + 255) / 256 * 256;
    static constexpr uint32_t RED = SPLITK ? NW * NG * 4 * 64 * 4 : 0;      // partial sums of one destination tile
    static constexpr uint32_t S_BYTES = NBUF * CR * STILE, OFF_STAGE = OFF_S + S_BYTES;
    static constexpr uint32_t ALL = S_BYTES + (STAGE_IN_S ? 0 : NW * St::BYTES);
    static constexpr uint32_t LDS = OFF_S + (ALL > RED ? ALL : RED);
    static_assert(PART % 256 == 0 && St::BYTES % 256 == 0, "alignment of the staged rows");
};

template <bool F32, bool EXACT, int RL, bool NARROW, int GA, int NP, int NW, int WD, int DTW, bool SPLITK, bool APART>
__global__ __launch_bounds__(NW * 64) void rows_tile_kernel(const TileArgs a)
{
    using C = TileCfg<F32, EXACT, RL, NARROW, GA, NP, NW, WD, DTW, SPLITK>;
    using St = typename C::St;
    constexpr int CHK = C::CHK, KS = C::KS, PL = C::PL, PLS = C::PLS, NT = St::NT, NG = C::NG, CR = C::CR, GW = C::GW;
    constexpr uint32_t PITCH = C::PITCH, STILE = C::STILE;
    constexpr int W_REGS = DTW * KS * PL * 4, CELLS = SPLITK ? 1 : CR;       // of one cell; cells of a round that this wave multiplies
    constexpr bool W_EARLY = W_REGS * CELLS <= 64;
    constexpr int CW = W_EARLY ? CELLS : 1;
    static_assert(!APART || EXACT, "rounded sums have one term");
    static_assert(NG <= 4 && (SPLITK ? (WD == 1 && NP == 1 && NW >= NG) : NW % WD == 0 && NG % (NW / WD) == 0), "shape");
    extern __shared__ __attribute__((aligned(256))) char lds[];
    v4u *sel_tab = reinterpret_cast<v4u *>(lds);
    int *act = reinterpret_cast<int *>(lds + C::OFF_ACT);
    uint32_t *bnd = reinterpret_cast<uint32_t *>(lds + C::OFF_BND);          // [NP + 1][MAX_K]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint32_t *runs = reinterpret_cast<uint32_t *>(lds + C::OFF_RUNS) + wave * C::RUNS;
    char *S = lds + C::OFF_S;
    const int m = lane & 15, g = lane >> 4;
    constexpr int PER_TILE = 4 / NG;                     // blocks per tile of 64 centres
    const int64_t blk = blockIdx.x;
    const int64_t tile = blk / PER_TILE;
    const int sub0 = (int)(blk % PER_TILE) * (NG * 16);
    const int d_base = (int)blockIdx.y * (WD * DTW);     // first destination tile of the block
    const int part = wave % NP, cslot = wave / NP;
    const uint32_t *run_tile = a.side.run_start + (size_t)tile * a.K * TILE;

    for (int b = threadIdx.x; b < 256; b += NW * 64) {   // mask of eight triplets -> eight bf16 values 0 / 1
        v4u v;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            v[q] = (((b >> (2 * q)) & 1) ? 0x3f80u : 0u) | (((b >> (2 * q + 1)) & 1) ? 0x3f800000u : 0u);
        sel_tab[b] = v;
    }
    if (wave == 0) {                                     // cells with a triplet among the block's centres, and their bounds
        int cnt = 0;
        for (int kb = 0; kb < a.K; kb += 64) {
            const int k = kb + lane;
            // (asked of tile_ptr, whose words lie in a cache line per cell, layers on spatial plans took 1 .. 4 % longer)
            const unsigned long long rows = a.side.rows ? a.side.rows[tile * mask_words(a.K) + (kb >> 6)] : ~0ull;
            uint32_t b[NP + 1];
#pragma unroll
            for (int p = 0; p <= NP; ++p) {
                const int slot = sub0 + 16 * GA * p;
                b[p] = 0u;
                if (k < a.K) b[p] = slot < TILE ? run_tile[(size_t)k * TILE + slot] : a.side.tile_ptr[(size_t)k * a.side.n_tiles + tile + 1];
            }
            const bool on = ((rows >> lane) & 1ull) && k < a.K && b[0] != b[NP];
            const unsigned long long msk = __ballot(on);
            const int at = cnt + __popcll(msk & ((1ull << lane) - 1ull));
            if (on) {
                act[at] = k;
#pragma unroll
                for (int p = 0; p <= NP; ++p) bnd[p * MAX_K + at] = b[p];
            }
            cnt += __popcll(msk);
        }
        if (lane == 0) act[MAX_K] = cnt;
    }
    __syncthreads();
    const int n_act = __builtin_amdgcn_readfirstlane(act[MAX_K]);

    const __amdgpu_buffer_rsrc_t frs = make_rsrc(a.feat, a.feat_bytes), grs = make_rsrc(a.gather, a.gather_bytes);

    // Position of a window of 32 triplets in this wave's stream: cell j of the active list, chunk of channels, window w of
    // the part's n triplets [bs, bs + n).  A part without triplets (also past the list's end) has one window all the same,
    // which reads nothing: the number of requests between any two points of the stream is then the same on every path, and
    // the compiler can wait for older ones without waiting for younger ones.
    struct Cursor { int j, chunk; uint32_t w, bs, n; };
    auto bounds = [&](int j, uint32_t &bs, uint32_t &n) {
        const int jj = j < n_act ? j : 0;
        bs = __builtin_amdgcn_readfirstlane(bnd[part * MAX_K + jj]);
        n = j < n_act ? __builtin_amdgcn_readfirstlane(bnd[(part + 1) * MAX_K + jj]) - bs : 0u;
    };
    auto advance = [&](Cursor &c) {
        c.w += (uint32_t)WINDOW;
        if (c.w < c.n) return;
        c.w = 0u;
        if (++c.chunk < a.n_chunks) return;
        c.chunk = 0;
        c.j += CR;
        bounds(c.j, c.bs, c.n);
    };
    // The gather word of a window's triplet, requested a window ahead of the row and not touched in between.  Triplets
    // past the part's end get an offset past the buffer: their reads return zeros and cost no traffic.
    St st;
    uint32_t raw;
    const uint32_t tl = St::triplet_of_lane(m, g);
    auto load_indices = [&](const Cursor &c) {
        raw = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(grs, (int)index_offset(c.bs + c.w, tl), 0, 0);
    };
    auto load_rows = [&](const Cursor &c) {
        const uint32_t offs = tl < c.n - c.w ? (raw & GATHER_INDEX) * a.row_bytes : OOB_OFFSET;
        st.set_chunk(c.chunk, a.c_src, lane);
        st.load(frs, offs, a.c_src);
    };
    // starts of the part's runs (lane <-> centre), relative to the part's first triplet
    auto load_runs = [&](int j) -> uint32_t {
        const int k = act[j < n_act ? j : (n_act > 0 ? n_act - 1 : 0)];
        const int c = lane < 16 * GA ? lane : 0;
        return run_tile[(size_t)k * TILE + sub0 + part * 16 * GA + c];
    };

    v4f acc[GW][DTW];
#pragma unroll
    for (int i = 0; i < GW; ++i)
#pragma unroll
        for (int d = 0; d < DTW; ++d) acc[i][d] = v4f{0.f, 0.f, 0.f, 0.f};

    const int wd = SPLITK ? 0 : wave % WD, wc = SPLITK ? 0 : wave / WD;
    const int dt0 = d_base + wd * DTW;
    const int nks = a.n_chunks * KS;
    const int rounds = (n_act + CR - 1) / CR;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds;

    if (n_act > 0) {
        Cursor nx{cslot, 0, 0u, 0u, 0u};
        bounds(cslot, nx.bs, nx.n);
        uint32_t st_next = load_runs(cslot);
        load_indices(nx);
        load_rows(nx);
        advance(nx);
        load_indices(nx);
        int buf = 0;
        for (int r = 0; r < rounds; ++r) {
            const int j = r * CR + cslot;
            uint32_t bs, n;
            bounds(j, bs, n);
            __builtin_amdgcn_wave_barrier();
            if (lane < 16 * GA) runs[lane] = st_next - bs;
            if (lane == 0) runs[16 * GA] = n;
            asm volatile("" ::: "memory");             // (the next request stays behind the last use of its register)
            st_next = load_runs(j + CR);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            int chunk = 0;
            do {
                const uint32_t my_part = C::OFF_S + (uint32_t)(buf * CR + cslot) * STILE + (uint32_t)part * C::PART;
                st.init(lds0 + (C::STAGE_IN_S ? my_part : C::OFF_STAGE + (uint32_t)wave * St::BYTES), lane);
                // ---- stage A -------------------------------------------------------------------------------
                // W of the round's cells, requested in front of the rows that are requested below: it arrives during stage A
                v4u wf[CW][DTW][KS][PL];
                auto load_w = [&](int cc, int at) {
                    const int jc = SPLITK ? j : r * CR + cc;
                    const int k = __builtin_amdgcn_readfirstlane(act[jc < n_act ? jc : n_act - 1]);
#pragma unroll
                    for (int d = 0; d < DTW; ++d) {
                        const int dt = dt0 + d < a.ndt ? dt0 + d : a.ndt - 1;
                        const v4u *wp = a.w + (((size_t)k * a.ndt + dt) * nks + (size_t)chunk * KS) * (PL * 64) + lane;
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                            for (int pl = 0; pl < PL; ++pl) wf[at][d][ks][pl] = wp[(ks * PL + pl) * 64];
                    }
                };
                if constexpr (W_EARLY) {
#pragma unroll
                    for (int cc = 0; cc < CW; ++cc) load_w(cc, cc);
                }
                v4f d1[GA][NT];
#pragma unroll
                for (int i = 0; i < GA; ++i)
#pragma unroll
                    for (int t = 0; t < NT; ++t) d1[i][t] = v4f{0.f, 0.f, 0.f, 0.f};
                uint32_t w = 0u;
                do {
                    st.store();
                    load_rows(nx);
                    advance(nx);
                    load_indices(nx);
                    // selection operands: lane (centre m, g), element e = 1 when triplet w + 8 g + e is in the centre's run
                    v4u sel[GA];
#pragma unroll
                    for (int i = 0; i < GA; ++i) {
                        const int base = (int)w + 8 * g;
                        int lo = (int)runs[16 * i + m] - base, hi = (int)runs[16 * i + m + 1] - base;
                        lo = lo < 0 ? 0 : (lo > 8 ? 8 : lo);
                        hi = hi < 0 ? 0 : (hi > 8 ? 8 : hi);
                        sel[i] = sel_tab[((1u << hi) - 1u) & ~((1u << lo) - 1u)];
                    }
#pragma unroll
                    for (int pl = 0; pl < PL; ++pl) {
                        v4u x[NT];
                        st.tiles(pl, 0, x);
#pragma unroll
                        for (int i = 0; i < GA; ++i)
#pragma unroll
                            for (int t = 0; t < NT; ++t)
                                d1[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, x[t]), __builtin_bit_cast(v8bf, sel[i]),
                                                                                   d1[i][t], 0, 0, 0);
                    }
                    __builtin_amdgcn_wave_barrier();
                    w += (uint32_t)WINDOW;
                } while (w < n);
                // the sums as operands: lane (centre m, g) holds the places 16 t + 4 g .. + 3 of tile t, and takes those of two
                // tiles as its share of a reduction step
                v4u own[GA][KS][PLS];
#pragma unroll
                for (int i = 0; i < GA; ++i)
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float x0 = d1[i][2 * ks + q / 2][2 * (q & 1)], x1 = d1[i][2 * ks + q / 2][2 * (q & 1) + 1];
                            if constexpr (!EXACT) {
                                own[i][ks][0][q] = cvt_pk_bf16(x0, x1);
                            } else {
                                uint32_t p1, p2, p3;
                                split_pair(x0, x1, p1, p2, p3);
                                own[i][ks][0][q] = p1; own[i][ks][PLS / 2][q] = p2; own[i][ks][PLS - 1][q] = p3;
                            }
                        }
                if constexpr (!SPLITK) {
                    if (j < n_act) {
                        char *sp = lds + my_part + (uint32_t)m * PITCH + (uint32_t)(16 * g);
#pragma unroll
                        for (int i = 0; i < GA; ++i)
#pragma unroll
                            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                                for (int pl = 0; pl < PLS; ++pl)
                                    *reinterpret_cast<v4u *>(sp + (uint32_t)(16 * i) * PITCH + pl * CHK * 2 + ks * 64) = own[i][ks][pl];
                    }
                    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                }
                // ---- stage B -------------------------------------------------------------------------------
#pragma unroll
                for (int cc = 0; cc < (SPLITK ? 1 : CR); ++cc) {
                    const int jc = SPLITK ? j : r * CR + cc;
                    if (jc < n_act) {                    // wave-uniform
                        const char *sb = S + (size_t)(buf * CR + cc) * STILE + (uint32_t)(wc * GW * 16 + m) * PITCH + (uint32_t)(16 * g);
                        constexpr bool EARLY = W_EARLY;
                        if constexpr (!EARLY) load_w(cc, 0);
                        const int wi = EARLY ? cc : 0;
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                            for (int i = 0; i < GW; ++i) {
                                v8bf sv[PLS];
#pragma unroll
                                for (int pl = 0; pl < PLS; ++pl) {
                                    if constexpr (SPLITK) sv[pl] = __builtin_bit_cast(v8bf, own[i][ks][pl]);
                                    else sv[pl] = __builtin_bit_cast(v8bf, *reinterpret_cast<const v4u *>(sb + (uint32_t)(16 * i) * PITCH + pl * CHK * 2 + ks * 64));
                                }
#pragma unroll
                                for (int d = 0; d < DTW; ++d) {
                                    auto mm = [&](int ws, int ss) {
                                        acc[i][d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, wf[wi][d][ks][ws]), sv[ss], acc[i][d], 0, 0, 0);
                                    };
                                    if constexpr (APART) {           // (smallest first)
                                        v4f lo = {0.f, 0.f, 0.f, 0.f};
                                        auto ml = [&](int ws, int ss) {
                                            lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, wf[wi][d][ks][ws]), sv[ss], lo, 0, 0, 0);
                                        };
                                        ml(0, PLS - 1);
                                        if constexpr (F32) { ml(PL - 1, 0); ml(PL / 2, PL / 2); }
                                        ml(0, PLS / 2);
                                        if constexpr (F32) ml(PL / 2, 0);
                                        mm(0, 0);
                                        acc[i][d] += lo;
                                    }
                                    else if constexpr (F32) { mm(0, PL - 1); mm(PL - 1, 0); mm(PL / 2, PL / 2); mm(0, PL / 2); mm(PL / 2, 0); mm(0, 0); }
                                    else if constexpr (EXACT) { mm(0, PLS - 1); mm(0, PLS / 2); mm(0, 0); }
                                    else mm(0, 0);
                                }
                            }
                    }
                }
                if constexpr (!SPLITK && C::NBUF == 2) buf ^= 1;
                else if constexpr (!SPLITK) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            } while (++chunk < a.n_chunks);
        }
    }

    // ---- every row once ------------------------------------------------------------------------------------------
    // lane (centre m, g) holds destination channels 16 dt + 4 g .. + 3
    auto store = [&](int group, int dt, const v4f &v) {
        const int64_t slot = tile * TILE + sub0 + 16 * group + m;
        if (slot >= a.n_centres || dt >= a.ndt) return;
        const int64_t row = a.side.perm ? (int64_t)a.side.perm[slot] : slot;
        const int d = 16 * dt + 4 * g;
        const size_t at = (size_t)row * a.c_dst + d;
        if ((a.c_dst & 3) == 0) {
            if (d >= a.c_dst) return;
            if (a.out_bf16) {
                const uint32_t lo = cvt_pk_bf16(v[0], v[1]), hi = cvt_pk_bf16(v[2], v[3]);
                *reinterpret_cast<uint64_t *>(static_cast<uint16_t *>(a.dst) + at) = (uint64_t)hi << 32 | lo;
            } else {
                *reinterpret_cast<v4f *>(static_cast<float *>(a.dst) + at) = v;
            }
        } else {
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                if (d + jj >= a.c_dst) break;
                if (a.out_bf16) static_cast<uint16_t *>(a.dst)[at + jj] = (uint16_t)(cvt_pk_bf16(v[jj], 0.f) & 0xffffu);
                else static_cast<float *>(a.dst)[at + jj] = v[jj];
            }
        }
    };
    if constexpr (SPLITK) {
        v4f *red = reinterpret_cast<v4f *>(S);           // [NW][NG][64]
#pragma unroll
        for (int d = 0; d < DTW; ++d) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NG; ++i) red[(wave * NG + i) * 64 + lane] = acc[i][d];
            __syncthreads();
            if (wave < NG) {
                v4f v = red[wave * 64 + lane];
                for (int u = 1; u < NW; ++u) v += red[(u * NG + wave) * 64 + lane];
                store(wave, d_base + d, v);
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < GW; ++i)
#pragma unroll
            for (int d = 0; d < DTW; ++d) store(wc * GW + i, dt0 + d, acc[i][d]);
    }
}

// fp32, split form: small products apart from more than this many steps (cells times chunks) of a wave on.  The error of one
// accumulator grows with the steps (all values positive: 7 steps, 32 -> 32 with 27 cells and 330 neighbours, 1.2e-7; 16 steps,
// 32 -> 32 with 64 cells, 2.3e-7; 28 steps, 128 -> 128, 4.6e-7; 128 steps, 1024 -> 64, 2.7e-6), that of fp32 sums on the vector ALUs
// with the square root (2.6e-7, 7.6e-7, 8.0e-7, 1.6e-6).  Apart: below 1.4e-7 at all of them, and up to 3 % of the time
// (20 -> 36, 0.49 M triplets: 99 and 102 us for the whole training step).  The cooperative form always has them apart when fp32.
// bf16: in crowded layers of the cooperative form, where sums have low terms (8 % of its time; 128 -> 256 with 37
// neighbours, not crowded: 3.7e-7, vector ALUs 7.0e-7), and in all layers of more than 128 destination channels in the split form, which
// takes that form's place on small clouds (128 -> 256, 3000 points: 1.1e-7, cooperative 3.0e-7).  The waves of the other split
// forms add up too few (1024 -> 64, 216 cells, crowded: 7.3e-7, vector ALUs 7.2e-6).
// Eight waves for 65 .. 128 destination channels, which larger clouds have four for: from half as many steps on, so that no layer has
// larger errors than with four (128 -> 128, 27 cells, 12 steps: one accumulator 2.5e-7 and, values of one sign, 1.1e-7; apart 1.35e-7
// and 7.5e-8; four waves, apart, 1.6e-7 and 9.4e-8).  4000 points, 128 -> 128: 49.6 us apart, 57.1 in one accumulator.
constexpr int64_t APART_FROM = 16;

template <bool F32, bool EXACT, int RL, bool NARROW, int GA, int NP, int NW, int WD, int DTW, bool SPLITK, bool APART = F32 && !SPLITK>
int launch_tile(const TileArgs &t, hipStream_t stream)
{
    using C = TileCfg<F32, EXACT, RL, NARROW, GA, NP, NW, WD, DTW, SPLITK>;
    if constexpr (F32 && SPLITK && !APART)
        if (ceil_div(t.K, NW) * t.n_chunks > (NW == 8 && DTW == 8 ? APART_FROM / 2 : APART_FROM))
            return launch_tile<F32, EXACT, RL, NARROW, GA, NP, NW, WD, DTW, SPLITK, true>(t, stream);
    auto kern = rows_tile_kernel<F32, EXACT, RL, NARROW, GA, NP, NW, WD, DTW, SPLITK, APART>;
    if (C::LDS > 64 * 1024)
        if (int rc = raise_lds_limit(reinterpret_cast<const void *>(kern), C::LDS)) return rc;
    const dim3 grid((unsigned)(t.side.n_tiles * (4 / C::NG)), (unsigned)ceil_div(t.ndt, WD * DTW));
    kern<<<grid, NW * 64, C::LDS, stream>>>(t);
    PCPP_HIP_CHECK(hipGetLastError());
    return PCPP_OK;
}

// Which form, by measurement over layers of 16 .. 256 channels and 2 000 .. 400 000 points (times in us).  A cell is crowded
// when it has more than 48 triplets per 32 centres on average, i.e. more than a window and a half.
//   - small clouds: split over more waves and 16 centres per block, up to 128 channels about as far as all waves fit on the device
//     at once (2 to 5 per SIMD by the registers of the form; a second round costs more than the longer chains of fewer waves).  The
//     wider layers' lines are where the times cross and lie beyond: 256 -> 256 bf16 with 16 centres (170 registers, a block per CU)
//     has up to 384 blocks, with 32 (222) up to 768.
//     Up to 64 destination channels, 8192 centres: eight waves (fp32 with 33 .. 64 channels from 6144 on with 32 centres: 8000
//     points, 64 -> 64 36.4, 29.5).  2048 points, 16 -> 16 fp32: 8.4, four waves 10.5, 32 centres 12.1, cooperative 27.  8000
//     points, 64 -> 64 bf16: 12.2 / 13.2 / 14.5 / 29.  Four waves up to 12288 centres in fp32 and, with eight lanes to a row, exact
//     bf16 (32 centres before): 12 000 points, 20 -> 36 fp32 35.1 -> 29.8, 128 -> 64 with 125 cells in bf16 100.9 -> 83.7.
//     65 .. 128 channels: eight waves, up to 4096 centres 16 per block, up to 8192 32.  2000 points, 128 -> 128 bf16 39.8 -> 26.7;
//     4000 points, 64 -> 128 fp32 46.2 -> 30.5; 8000 points 47.7 -> 37.7 (four waves, 32 centres before; at 12 000 points 59.1,
//     eight 65.6).
//     Wider: blocks of 128 destination channels, each with its own sums.  Up to 6144 / 12288 / 24576 centres times such blocks
//     eight waves with 16 centres, four and eight with 32.  2000 points, 256 -> 256 bf16 117 -> 39, fp32 460 -> 87; 5000, 128 ->
//     256 126 -> 52; 12 000 129 -> 88 (cooperative before; exact sums keep their small products apart as they did there; at 30 000
//     points 153, four waves with 32 centres 168, eight 208).
//     One cell (1 x 1 x 1 kernels) keeps one wave of a split block at work.  Wide layers take that form only while there are few
//     blocks (2000 points with 60 neighbours, 256 -> 256 bf16 45.4, cooperative 51.3; 2500 with 40 55.9, 35.4; 9000 188, 48; 300 ->
//     200 fp32, 2500 points 104, 183, 9000 593, 223), crowded ones with rounded sums up to 8192 centres (20 000 points with 40
//     neighbours, 64 -> 64: 24.2, 18.5; 400 000 with 12 in spatial order 103, 73).
//     Exact bf16 sums to 65 .. 128 channels on large clouds have two waves, of which one is idle, instead of four (128 -> 128,
//     150 000 points with 40 neighbours: 230, 396).
//   - exact sums, up to 128 destination channels: split over four waves, 32 centres, since the terms of a sum would take three
//     times the LDS (40 000 points, 128 -> 128 bf16: 130 per direction; cooperative, 16 centres per wave, about 165)
//     fp32, 17 .. 32 destination channels, more than 65536 centres with up to 16 neighbours: 64 centres, which fill a window better
//     (32 -> 32, 200 000 points with 10 neighbours: 120, 32 centres 132; 100 000 with 13.5: 74, 78; with 24: 90, 86; 24 000 with
//     14.5, too few blocks: 28.6, 24.6).
//     (With more cells two waves are up to 4 % faster on large bf16 clouds, but each adds up twice as much: 128 -> 128, 300 000
//     points, relative error 2.0e-7, four waves 1.5e-7; values of one sign 1.4e-7 and 8.7e-8.)
//   - rounded sums, up to 64: the same (strided layer's input gradient, 128 -> 64: 253, 16 centres 346, cooperative 312).
//     More than 131072 centres and up to 27 cells: two waves, whose sums are added half as often; the rounding of the sums is
//     10 000 times the error of the longer ones (64 -> 64, 400 000 points with 10 neighbours 229, 204, with 24 264, 246, in spatial
//     order 250, 215; 150 000 points with 10: 104, 98).
//     Crowded: 16 centres, which fill their windows, over two waves, or four where the cloud is too small to fill the device with
//     that (64 -> 64, cooperative with 16 centres per wave / four waves / two: 115 000 points with 148 neighbours 162 / 145 / 141
//     and in spatial order 178 / 146 / 143; 57 600 with 74 71 / 57 / 54; 150 000 with 48 in spatial order 152 / 143 / 128; 40 000
//     with 50 61 / 53 / 57; 10 000 with 50 41 / 19 / 24).  Two chunks of rows (128 -> 64) need more than 80 triplets per 32 centres
//     for it: 25 000 points with 100 neighbours 113 / 78 / 78 (32 centres 88), 60 000 with 60 135 / 142 / 145 (127).
//     More than 131072 centres and up to 27 cells: 32 centres over two waves up to 256 triplets per 32 centres (400 000 points, 64
//     -> 64, 43 neighbours cooperative 372, 16 centres 394, 32 343; in spatial order 293 and 249), with two chunks up to 128 in
//     spatial order (400 000 points with 70 neighbours: 788, 861, 663; in index order 200 000 with 32: 240, 231, 246).  Above 256
//     with two chunks in index order the cooperative form, whose blocks read W a quarter as often (400 000 points with 560
//     neighbours: 3756, 4626; in spatial order 3435, 3540).
//   - rounded sums to 65 .. 128 channels: split up to 32768 centres, crowded from 16384 on: over two waves (25 000 points with 368
//     neighbours, 64 -> 128: 52, four waves 61; 12 500 points with 80: 46, 37); above, cooperative, 32 centres per wave, crowded:
//     16 (strided layer, 64 -> 128: 97, split 107).
//   - wider: cooperative, so that W is read once per 64 centres; 32 centres per wave (100 000 points, 125 cells, 128 -> 256 with
//     rounded sums: 777; 16 centres 958, split 864), 16 where the exact bf16 sums of 32 would leave a CU one block, and in crowded
//     layers with rounded sums (115 000 points with 148 neighbours, 256 -> 256: 907 in spatial order and 860 in index order, 32
//     centres 1102 and 1026; 100 000 points with 24 neighbours, not crowded: 673, 32 centres 618).
template <bool F32, bool EXACT, int RL, bool NARROW, int GA, int NW>
int launch_tile_split(const TileArgs &t, hipStream_t stream)
{
    if constexpr (EXACT) {                               // (layers with rounded sums have four tiles or more)
        if (t.ndt == 1) return launch_tile<F32, EXACT, RL, NARROW, GA, 1, NW, 1, 1, true>(t, stream);
        if (t.ndt == 2) return launch_tile<F32, EXACT, RL, NARROW, GA, 1, NW, 1, 2, true>(t, stream);
    }
    return launch_tile<F32, EXACT, RL, NARROW, GA, 1, NW, 1, 4, true>(t, stream);
}

template <bool F32, bool EXACT, int RL, bool NARROW>
int launch_tile_form(const TileArgs &t, hipStream_t stream)
{
    const bool cells = t.K > 1;                          // (one cell: see above)
    if (t.ndt <= 4) {
        if constexpr (F32)
            if (t.ndt > 2 && t.n_centres > 6144 && t.n_centres <= 8192) return launch_tile<F32, EXACT, RL, NARROW, 2, 1, 8, 1, 4, true>(t, stream);
        if (t.n_centres <= 8192) return launch_tile_split<F32, EXACT, RL, NARROW, 1, 8>(t, stream);
        if constexpr (EXACT && (F32 || RL == 8))
            if (t.n_centres <= 12288) return launch_tile_split<F32, EXACT, RL, NARROW, 1, 4>(t, stream);
    } else if (t.ndt <= 8) {
        if (t.n_centres <= 4096) return launch_tile<F32, EXACT, RL, NARROW, 1, 1, 8, 1, 8, true>(t, stream);
        if (t.n_centres <= 8192) return launch_tile<F32, EXACT, RL, NARROW, 2, 1, 8, 1, 8, true>(t, stream);
    } else {
        const int64_t parts = t.n_centres * ceil_div(t.ndt, 8);
        if (parts <= (cells || F32 ? 6144 : 4096)) return launch_tile<F32, EXACT, RL, NARROW, 1, 1, 8, 1, 8, true, EXACT>(t, stream);
        if (cells && parts <= 12288) return launch_tile<F32, EXACT, RL, NARROW, 2, 1, 4, 1, 8, true, EXACT>(t, stream);
        if (cells && parts <= 24576) return launch_tile<F32, EXACT, RL, NARROW, 2, 1, 8, 1, 8, true, EXACT>(t, stream);
    }
    const int64_t per_cell = t.n_centres * (int64_t)t.K, triplets = (int64_t)(t.gather_bytes / 4);
    const bool crowded = triplets * 32 > 48 * per_cell;
    if constexpr (EXACT) {
        if constexpr (F32)
            if (t.ndt == 2 && t.n_centres > 65536 && triplets <= 16 * t.n_centres)
                return launch_tile<F32, EXACT, RL, NARROW, 4, 1, 4, 1, 2, true>(t, stream);
        if (t.ndt <= 4) return launch_tile_split<F32, EXACT, RL, NARROW, 2, 4>(t, stream);
        if constexpr (!F32)
            if (!cells && t.ndt <= 8 && t.n_centres > 131072) return launch_tile<F32, EXACT, RL, NARROW, 2, 1, 2, 1, 8, true>(t, stream);
        if (t.ndt <= 8) return launch_tile<F32, EXACT, RL, NARROW, 2, 1, 4, 1, 8, true>(t, stream);
        if constexpr (F32) return launch_tile<F32, EXACT, RL, NARROW, 2, 2, 4, 4, 4, false>(t, stream);
        else return crowded ? launch_tile<F32, EXACT, RL, NARROW, 1, 4, 4, 4, 4, false, true>(t, stream)
                            : launch_tile<F32, EXACT, RL, NARROW, 1, 4, 4, 4, 4, false>(t, stream);
    } else {
        if (t.ndt <= 4) {
            const bool large = t.n_centres > 131072, spatial = t.side.perm != nullptr, one = t.n_chunks == 1, two = large && t.K <= 27;
            if ((crowded && !cells) || (large && !one && !spatial && triplets > 8 * per_cell))
                return launch_tile<F32, EXACT, RL, NARROW, 1, 4, 4, 4, 1, false>(t, stream);
            int most = one ? 48 : 80;                    // triplets per cell and 32 centres for the forms with 32 centres
            if (two && cells && (one || spatial)) most = one ? 256 : 128;
            if (triplets * 32 <= most * per_cell)
                return two ? launch_tile<F32, EXACT, RL, NARROW, 2, 1, 2, 1, 4, true>(t, stream)
                           : launch_tile<F32, EXACT, RL, NARROW, 2, 1, 4, 1, 4, true>(t, stream);
            return t.n_centres > 49152 ? launch_tile<F32, EXACT, RL, NARROW, 1, 1, 2, 1, 4, true>(t, stream)
                                       : launch_tile<F32, EXACT, RL, NARROW, 1, 1, 4, 1, 4, true>(t, stream);
        }
        if (t.ndt <= 8) {
            if (t.n_centres <= 32768)
                return crowded && t.n_centres > 16384 ? launch_tile<F32, EXACT, RL, NARROW, 2, 1, 2, 1, 8, true>(t, stream)
                                                      : launch_tile<F32, EXACT, RL, NARROW, 2, 1, 4, 1, 8, true>(t, stream);
            return crowded ? launch_tile<F32, EXACT, RL, NARROW, 1, 4, 4, 4, 2, false>(t, stream)
                           : launch_tile<F32, EXACT, RL, NARROW, 2, 2, 4, 4, 2, false>(t, stream);
        }
        return crowded ? launch_tile<F32, EXACT, RL, NARROW, 1, 4, 4, 4, 4, false>(t, stream)
                       : launch_tile<F32, EXACT, RL, NARROW, 2, 2, 4, 4, 4, false>(t, stream);
    }
}

}  // namespace

bool mvmr_rows_tile_usable(const MvmrArgs &a)
{
    // row and index reads go through buffer descriptors of less than 4 GiB
    return a.n_triplets > 0 && (size_t)a.n_triplets * 4 <= MAX_BUFFER_BYTES &&
           (size_t)a.n_src * a.c_src * (a.in_dtype == PCPP_F32 ? 4 : 2) <= MAX_BUFFER_BYTES;
}

int mvmr_rows_tile_pack_w(const void *w, void *packed, int K, int c_src, int c_dst, int stride_d, int stride_s, int dtype,
                          hipStream_t stream)
{
    const bool f32 = dtype == PCPP_F32;
    const TileShape s = tile_shape(f32, c_src, c_dst);
    const int nks = s.n_chunks * s.chk / 32;
    const unsigned blocks = (unsigned)ceil_div((int64_t)K * s.ndt * nks * 64, 256);
    auto kern = f32 ? (s.narrow ? pack_w_tile_kernel<true, true> : pack_w_tile_kernel<true, false>)
                    : (s.narrow ? pack_w_tile_kernel<false, true> : pack_w_tile_kernel<false, false>);
    kern<<<blocks, 256, 0, stream>>>(w, static_cast<v4u *>(packed), K, c_src, c_dst, nks, s.ndt, s.chk, stride_d, stride_s);
    PCPP_HIP_CHECK(hipGetLastError());
    return PCPP_OK;
}

// bf16 layers whose run sums are rounded to bf16 once before they meet W: 64 -> 64, 64 -> 128 and 128 -> 64 with up to 64
// cells, and 256 -> 256.  That is these layers' precision (relative error 1.6e-3 against exact sums), and a third of stage
// B's matrix products.  All other layers keep the fp32 sums as three terms (1e-7 to 1e-6, growing with the length of the sums).
static bool bf16_sums(int K, int c_src, int c_dst)
{
    if (c_src == 256 && c_dst == 256) return true;
    return K <= 64 && ((c_src == 64 && (c_dst == 64 || c_dst == 128)) || (c_src == 128 && c_dst == 64));
}

// a.w must be the weights packed by mvmr_rows_tile_pack_w
int mvmr_rows_tile(const MvmrArgs &a, hipStream_t stream)
{
    const bool f32 = a.in_dtype == PCPP_F32;
    const TileShape s = tile_shape(f32, a.c_src, a.c_dst);
    TileArgs t{};
    t.feat = a.feat; t.w = static_cast<const v4u *>(a.w); t.dst = a.dst; t.gather = a.gather; t.side = a.side;
    t.n_centres = a.n_centres;
    t.row_bytes = (uint32_t)a.c_src * (f32 ? 4 : 2);
    t.feat_bytes = (uint32_t)((size_t)a.n_src * t.row_bytes);
    t.gather_bytes = (uint32_t)((size_t)a.n_triplets * 4);
    t.K = a.K; t.c_src = a.c_src; t.c_dst = a.c_dst; t.n_chunks = s.n_chunks; t.ndt = s.ndt;
    t.out_bf16 = a.out_dtype == PCPP_BF16;
    if (f32) return s.narrow ? launch_tile_form<true, true, 4, true>(t, stream) : launch_tile_form<true, true, 4, false>(t, stream);
    if (s.rl == 4) return s.narrow ? launch_tile_form<false, true, 4, true>(t, stream) : launch_tile_form<false, true, 4, false>(t, stream);
    return bf16_sums(a.K, a.c_src, a.c_dst) ? launch_tile_form<false, false, 8, false>(t, stream) : launch_tile_form<false, true, 8, false>(t, stream);
}

}  // namespace pcpp
