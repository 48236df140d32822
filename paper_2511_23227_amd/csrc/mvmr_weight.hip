// Weight gradient (VVOR), Eq. (5) of Sec. 3.3.3, on the matrix cores: dW[k] = sum over cell k's run of
// dy[o] (x) x[i].  The (k, o, i) ordered triplet list is cut into equal chunks, one per block (per sub-block of dW for
// wide layers); the reduction index of the MFMA is the triplet; chunk partial sums go to the workspace and are
// added in a fixed order by a second kernel: no atomics, reproducible.
//
// Block c owns triplets [c*chunk, (c+1)*chunk) of the list.  A chunk usually lies inside one cell's run; where a run starts
// inside the chunk the accumulator is flushed and restarted.  Slots of the partial buffer:
//   slot c               sum for the cell of the chunk's first triplet
//   slot n_chunks + k    sum for cell k over the part of its run that starts inside a chunk
//
// v_mfma_f32_16x16x32_bf16: A: lane (M = l%16, g = l/16) holds A[M][8g .. 8g+7]; B: lane (N = l%16, g) holds
// B[8g .. 8g+7][N]; D: lane l, register j -> M = 4g + j, N = l%16.

#include "mvmr_stage.h"
#include "mvmr_walk.h"

namespace pcpp {

namespace {

constexpr int WAVES = 4;

typedef uint32_t v2u __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------------------------
// bf16 256 -> 256: one block of eight waves per chunk, wave w owning the 128 x 64 sub-block (output channels
// 128 (w / 4) .., input channels 64 (w % 4) ..) of dW[k].  With 128 accumulator registers a wave has no room
// to keep rows in flight, and two waves per SIMD hide little of a gather's latency.  Here the block fetches every
// row of a batch of 32 triplets once (x[i] and dy[o]: 32 x 1 KB) with loads that write straight into LDS
// (global_load_lds_dwordx4: lane l of the wave writes bytes 16 l .. 16 l + 15 behind the address in M0, so one
// instruction moves two rows), into a ring of four batch buffers: rows in flight cost no registers, and the
// batches s + 1 .. s + 4 are on their way while batch s is multiplied.  The triplets' indices travel the same way
// (global_load_lds_dword into a small ring per wave), two batches ahead of their rows.
//   step s:  request the indices of batch s + 6 | first half of batch s (output channels co0 .. co0 + 63, operands
//            read during step s - 1), the LDS reads for the second half under way | wait for the rows of batch
//            s + 1, zero its dy rows past the batch's end | barrier | read the first operands of batch s + 1; second
//            half of batch s meanwhile, with one request for rows of batch s + 4 behind every four MFMAs (into the
//            buffer that batch s has just left: every wave read its last operands of it before the barrier) |
//            wait for the indices of batch s + 5, read them into registers
// The requests are spread between the MFMAs because a request can wait hundreds of cycles for room in the memory
// pipeline and the wave issues in order: bunched at the head of the step they kept the matrix pipe idle (5.1 ->
// 4.7 ms on a million-point cloud); with the operands of the next batch read during the second half, LDS reads and
// MFMAs of the block's lock-stepped waves overlap.  The rows' time in flight matters as well: requested in the second
// half of a step for the batch four ahead they have two and a half steps (4.55 ms), half a step less costs 6 %.
// Wave w moves rows 4 w .. 4 w + 3 of x and of dy.  The compiler does not see these loads, so the waits are written
// by hand; they are exact because every step issues the same five memory instructions per wave, in the same order
// (one for indices, four for rows; a batch that is short or empty re-reads its last triplet, or triplet 0): behind
// the rows to wait for, eleven younger instructions may still be outstanding, behind the indices nine.  (The partial
// sums' stores and the rare reads of a cell's bounds, which the compiler does see, only make these waits stricter.)
// A batch never crosses the end of a cell's run.  Lane (m, g) reads 8 bytes = channels 4m .. 4m+3 (+ 64 per 64-channel
// group) of the rows of triplets 8g .. 8g+7; element q of those four channels of the eight triplets is one MFMA operand:
// row / column m of operand (group, q) is channel 64 group + 4m + q.
// ---------------------------------------------------------------------------------------------
constexpr int LDS_WAVES = 8;
constexpr int LDS_GROUP_PITCH = 8 * 512 + 128;    // eight rows of 512 B, then 128 B: the rows r, r + 8, r + 16, r + 24 that
                                                  // one LDS read touches start in different banks
constexpr int LDS_BATCH_BYTES = 8 * LDS_GROUP_PITCH;   // 32 rows of x (four groups) then 32 rows of dy
constexpr int LDS_NBUF = 4;                        // batch buffers: batch s in s % 4
constexpr int LDS_INDEX_BYTES = LDS_WAVES * LDS_NBUF * 256;   // per wave and batch: 64 words, word 4 a + r = index of
                                                              // row 4 w + r in tri_i (a = 0) or tri_o (a = 1)
constexpr int LDS_WEIGHT_BYTES = LDS_NBUF * LDS_BATCH_BYTES + LDS_INDEX_BYTES;

// 16 bytes per lane from `src` (per lane) to LDS byte address `lds` + 16 lane (`lds` wave-uniform).  The address
// travels in M0, which the statement overwrites without saying so (the compiler reserves the register and refuses it
// as a clobber); nothing else in a compute kernel for this target lives in M0 (LDS instructions need none here).
__device__ inline void load_to_lds_b128(const void *src, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds) : "memory");
}
// 4 bytes per lane to `lds` + 4 lane
__device__ inline void load_to_lds_b32(const void *src, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(src), "s"(lds) : "memory");
}

__global__ __launch_bounds__(LDS_WAVES * 64, 2) void weight_lds_kernel(const uint16_t *__restrict__ x,
                                                                        const uint16_t *__restrict__ dy,
                                                                        float *__restrict__ part,
                                                                        const int32_t *__restrict__ tri_o,
                                                                        const int32_t *__restrict__ tri_i,
                                                                        const int64_t *__restrict__ seg, int K,
                                                                        int64_t n_triplets, int chunk, int64_t n_chunks)
{
    constexpr int C = 256, ROW = C * 2, GP = LDS_GROUP_PITCH, X_OFF = 0, DY_OFF = 4 * GP;   // row r: (r / 8) GP + (r % 8) ROW
    extern __shared__ __attribute__((aligned(16))) unsigned char stage[];        // four batches, then the index rings
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m = lane & 15, g = lane >> 4;
    const int ci0 = (wave & 3) * 64, co0 = (wave >> 2) * 128;
    const int64_t chunk_id = blockIdx.x;
    const int64_t p0 = chunk_id * chunk;                                          // positions below are relative to it
    const uint32_t q_end = (uint32_t)((p0 + chunk < n_triplets ? p0 + chunk : n_triplets) - p0);

    // cell of the first triplet: the k with seg[k] <= p0 < seg[k+1]
    int k = 0;
    for (int kb = 0; kb < K; kb += 64) {
        const int kk = kb + lane;
        const bool hit = kk < K && seg[kk] <= p0 && p0 < seg[kk + 1];
        const unsigned long long msk = __ballot(hit);
        if (msk) { k = kb + __ffsll((long long)msk) - 1; break; }
    }
    k = __builtin_amdgcn_readfirstlane(k);
    // A batch travels through the steps as one word: triplets | ends its run << 8 | cell << 16 (0: no batch).  run_end:
    // end of cell k's run inside the chunk, read from seg only when the cell changes.
    auto end_of = [&](int kk) -> uint32_t {
        const int64_t e = seg[kk + 1] - p0;
        return e < (int64_t)q_end ? (uint32_t)e : q_end;
    };
    uint32_t q = 0, run_end = end_of(k);
    uint32_t q5 = 0;                              // first triplet of the batch that next_batch returned last
    auto next_batch = [&]() -> uint32_t {
        while (q < q_end) {
            if (run_end <= q) {                       // next cell (empty runs are passed over)
                ++k;
                run_end = end_of(k);
                continue;
            }
            const uint32_t n = run_end - q < 32u ? run_end - q : 32u;
            q5 = q;
            q += n;
            return n | (q == run_end ? 256u : 0u) | ((uint32_t)k << 16);
        }
        q5 = 0;
        return 0u;
    };

    // mover role of this lane: rows 4 wave + 2 j + half (j = 0, 1), bytes 16 piece .. of the row
    const int half = lane >> 5, piece = lane & 31;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)(stage);
    const uint32_t ring0 = lds0 + LDS_NBUF * LDS_BATCH_BYTES + wave * (LDS_NBUF * 256);
    const unsigned char *ring = stage + LDS_NBUF * LDS_BATCH_BYTES + wave * (LDS_NBUF * 256);
    const unsigned char *xb = reinterpret_cast<const unsigned char *>(x) + piece * 16;
    const unsigned char *dyb = reinterpret_cast<const unsigned char *>(dy) + piece * 16;
    // index requests: lane -> (array, row lane % 4)
    const int32_t *tri_lane = (((lane >> 2) & 1) ? tri_o : tri_i) + p0;
    const int r_lane = 4 * wave + (lane & 3);

    // the first steps request rows before any index has arrived: they read zeros (row 0) from the ring
    *reinterpret_cast<v4u *>(stage + LDS_NBUF * LDS_BATCH_BYTES + wave * (LDS_NBUF * 256) + lane * 16) = v4u{0u, 0u, 0u, 0u};
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");

    uint32_t w0 = 0, w1 = 0, w2 = 0, w3 = 0, w4 = 0, w5 = 0, w6 = next_batch();      // batches s .. s + 6
    int cur = 0;                                  // buffer of batch s

    v4f acc[2][4][4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int d = 0; d < 4; ++d) acc[a][b][d] = v4f{0.f, 0.f, 0.f, 0.f};
    bool first = true;

    // operands of batch s that are read during step s - 1: the x side as MFMA operands, the dy rows of the first half
    v4u bv[4];
    v2u dyw0[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) bv[e] = v4u{0u, 0u, 0u, 0u};
#pragma unroll
    for (int e = 0; e < 8; ++e) dyw0[e] = v2u{0u, 0u};
    int32_t ix[2] = {0, 0}, io[2] = {0, 0};     // rows 4 wave + 2 j + half of the batch whose rows are requested next
    // acc[qo][qd] += dy(16 channels)^T . x over the batch's 32 triplets; dyw: this lane's words of the dy rows
    auto multiply = [&](int qo, int qd, const v2u (&dyw)[8]) __attribute__((always_inline)) {
        v4u av;
#pragma unroll
        for (int wd = 0; wd < 4; ++wd)
            av[wd] = __builtin_amdgcn_perm(dyw[2 * wd + 1][qd >> 1], dyw[2 * wd][qd >> 1],
                                           (qd & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
        for (int qs = 0; qs < 4; ++qs)
            acc[qo][qd][qs] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(v8bf, av), __builtin_bit_cast(v8bf, bv[qs]), acc[qo][qd][qs], 0, 0, 0);
    };

    // one step; COMPUTE = false for the six steps that fill the pipeline (no batch s yet).  Once a batch has reached
    // the front, every step has one until the chunk is used up, and nothing is left behind the last one.
    auto step = [&](auto compute) __attribute__((always_inline)) {
        constexpr bool COMPUTE = decltype(compute)::value;
        // indices of batch s + 6
        {
            const int n6 = (int)(w6 & 255u);
            int t = (int)q5 + (r_lane < n6 ? r_lane : n6 - 1);
            if (t < 0) t = 0;
            load_to_lds_b32(tri_lane + t, (uint32_t)__builtin_amdgcn_readfirstlane((int)(ring0 + ((cur + 6) & 3) * 256)));
        }
        // first half of batch s (output channels co0 .. co0 + 63; its operands were read one step ago).  The reads for the
        // second half go first.
        const unsigned char *buf = stage + cur * LDS_BATCH_BYTES;
        v2u dyw1[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            dyw1[e] = *reinterpret_cast<const v2u *>(buf + DY_OFF + g * GP + e * ROW + (co0 + 64 + 4 * m) * 2);
        if constexpr (COMPUTE) {
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) multiply(0, qd, dyw0);
        }
        // the rows of batch s + 1 have arrived; past its end the dy rows become zeros (the x rows there repeat the
        // batch's last triplet)
        asm volatile("s_waitcnt vmcnt(11)" ::: "memory");
        {
            const int n1 = (int)(w1 & 255u);
            if (n1 > 0 && n1 < 32) {
                unsigned char *dst = stage + ((cur + 1) & 3) * LDS_BATCH_BYTES + DY_OFF + piece * 16;
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int r = 4 * wave + 2 * j + half;
                    if (r >= n1) *reinterpret_cast<v4u *>(dst + (r >> 3) * GP + (r & 7) * ROW) = v4u{0u, 0u, 0u, 0u};
                }
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        // batch s + 1 is complete in LDS: ask for its first operands, multiply the second half of batch s meanwhile
        const unsigned char *nbuf = stage + ((cur + 1) & 3) * LDS_BATCH_BYTES;
        v2u xw[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            xw[e] = *reinterpret_cast<const v2u *>(nbuf + X_OFF + g * GP + e * ROW + (ci0 + 4 * m) * 2);
        v2u dyn[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            dyn[e] = *reinterpret_cast<const v2u *>(nbuf + DY_OFF + g * GP + e * ROW + (co0 + 4 * m) * 2);
        {
            // rows of batch s + 4 into the buffer that batch s has just left (every wave has read its last operands
            // of it before the barrier), one request behind every four MFMAs of the second half: a request can wait long for
            // room in the memory pipeline, and the matrix pipe should have work meanwhile
            const uint32_t dst = lds0 + (uint32_t)cur * LDS_BATCH_BYTES + (uint32_t)((wave >> 1) * GP + 4 * (wave & 1) * ROW);
            auto request = [&](int i) __attribute__((always_inline)) {
                const int j = i >> 1;
                if (i & 1)
                    load_to_lds_b128(dyb + (size_t)io[j] * ROW,
                                     (uint32_t)__builtin_amdgcn_readfirstlane((int)(dst + DY_OFF + 2 * j * ROW)));
                else
                    load_to_lds_b128(xb + (size_t)ix[j] * ROW,
                                     (uint32_t)__builtin_amdgcn_readfirstlane((int)(dst + X_OFF + 2 * j * ROW)));
            };
#pragma unroll
            for (int qd = 0; qd < 4; ++qd) {
                if constexpr (COMPUTE) multiply(1, qd, dyw1);
                request(qd);
            }
        }
        if constexpr (COMPUTE) {
            if (w0 & 256u) {
                // flush: lane (m, g), register j of acc[qo][qd][qs] is dW[co0 + 64 qo + 4 (4g + j) + qd][ci0 + 4m + qs]
                float *dstp = part + (size_t)(first ? chunk_id : n_chunks + (w0 >> 16)) * C * C;
#pragma unroll
                for (int qo = 0; qo < 2; ++qo)
#pragma unroll
                    for (int qd = 0; qd < 4; ++qd)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const int co = co0 + 64 * qo + 4 * (4 * g + j) + qd;
                            const int ci = ci0 + 4 * m;
                            *reinterpret_cast<v4f *>(dstp + (size_t)co * C + ci) =
                                v4f{acc[qo][qd][0][j], acc[qo][qd][1][j], acc[qo][qd][2][j], acc[qo][qd][3][j]};
                            acc[qo][qd][0][j] = acc[qo][qd][1][j] = acc[qo][qd][2][j] = acc[qo][qd][3][j] = 0.f;
                        }
                first = false;
            }
        }
#pragma unroll
        for (int qs = 0; qs < 4; ++qs)
#pragma unroll
            for (int wd = 0; wd < 4; ++wd)
                bv[qs][wd] = __builtin_amdgcn_perm(xw[2 * wd + 1][qs >> 1], xw[2 * wd][qs >> 1],
                                                   (qs & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
        for (int e = 0; e < 8; ++e) dyw0[e] = dyn[e];
        // the indices of batch s + 5 (asked for at the head of the step before) into registers for the next step's row
        // requests
        asm volatile("s_waitcnt vmcnt(9)" ::: "memory");
        {
            const unsigned char *words = ring + ((cur + 5) & 3) * 256;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                ix[j] = *reinterpret_cast<const int32_t *>(words + 4 * (2 * j + half));
                io[j] = *reinterpret_cast<const int32_t *>(words + 4 * (4 + 2 * j + half));
            }
        }
        w0 = w1; w1 = w2; w2 = w3; w3 = w4; w4 = w5; w5 = w6; w6 = next_batch();
        cur = (cur + 1) & 3;
    };
    for (int f = 0; f < 6; ++f) step(std::false_type{});
    while (w0) step(std::true_type{});
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // nothing of this wave is still on its way into LDS
}

// ---------------------------------------------------------------------------------------------
// Any channel counts, fp32 or bf16.  A block of four waves owns a chunk of the triplet list and a sub-block of dW, up to
// 128 x 64 channels (bf16) or 64 x 64 (fp32); the waves take the chunk's batches of 32 triplets in turn and their sums
// are added through LDS, in wave order, where the sub-block is flushed (so there are a quarter as many partial sums as
// waves).  The rows of a batch reach the matrix cores as mvmr_stage.h describes: dy as operand A, x as operand B, the
// triplet as the reduction index.  fp32 rows are three bf16 terms there, and the six products of weight 2^-16 or more
// relative to the leading one are kept (the rest is below 2^-24 of it).
// Triplets past the batch's end get an offset past the buffer, whose reads return zeros and cost no traffic.  The rows
// of the next batch are requested as soon as this one's have been passed on, so they are on their way while the matrix
// cores work; the indices are requested a batch ahead of them.
// What bounds it: bf16, the L1 cache, which serves four lanes per access (64 -> 64, 17 M triplets: 4 accesses per row of
// 128 bytes with 8 bytes per lane, 294 us; 2 with 16 bytes, 220); fp32, the vector instructions that split
// the rows into terms.  Before, with one wave per chunk, rows read as dwords or 8-byte pieces, fp32 products on the fp32
// matrix instructions, and the partial sums: 331 + 35 us for that layer (now 220 + 7), 84 + 11 for a 32 -> 32 fp32 layer
// with 2.4 M triplets (58 + 7), 146 + 24 for 64 -> 128 with 4.6 M (113 + 8), and on the vector ALUs 1715 for 128 -> 64 with
// 2.3 M (77 + 8).
// ---------------------------------------------------------------------------------------------
struct WeightArgs {
    const void *x, *dy;
    float *part;
    const int32_t *tri_o, *tri_i;
    const int64_t *seg;
    int64_t n_triplets, n_chunks;
    uint32_t x_bytes, dy_bytes, tri_bytes;
    int K, c_in, c_out, chunk, n_sub_in, n_sub;
};

// Waves per SIMD that the register allocation must leave room for.  fp32 sub-blocks of 64 x 32: three, with ten registers kept in
// scratch memory (168 in use); two without that are no faster (20 -> 36, 0.49 M triplets, whole training step: 99.2 us, 99.7).  128 x 64
// channels, bf16: two, with four registers in scratch memory (254 in use); one would halve the rows in flight.
template <typename SO, typename SI> constexpr int any_min_waves() {
    if (SO::NT * SI::NT >= 16 || SO::CHK + SI::CHK > 128) return 2;
    return SO::PL > 1 && SO::NT * SI::NT >= 8 ? 3 : 4;
}

// Triplets that are summed in registers at most, so that no sum in 32 bits loses more than those of the kernels for fp32 sums on
// the vector ALUs or of one wave per chunk did: chunks hold no more while the partial sums stay below 256 MB, and beyond
// that the sums of a run go to its slot part by part.  Relative errors with chunks of any length, now, and of those kernels: 64 ->
// 64 bf16, 16 M triplets (15 900 each), 3.8e-7, 2.7e-7, 3.1e-7; 512 -> 512 bf16, 1 M (30 700), 4.9e-7, 2.6e-7, 6.4e-7.  The
// former takes 365 us instead of 375, the latter, with 4 chunks for each before, 718 instead of 690.
constexpr uint32_t SEGMENT = 8192;

// fp32 chunks, within the same 256 MB (32 -> 32, 2.4 M triplets: 231 us for the whole step with 768, 237 with 512).
constexpr int F32_CHUNK = 768;

// SO, SI: how the rows of dy and x reach the matrix cores
template <typename SO, typename SI>
__global__ __launch_bounds__(WAVES * 64, (any_min_waves<SO, SI>())) void weight_any_kernel(const WeightArgs a)
{
    constexpr int ES = SO::ES, NTO = SO::NT, NTI = SI::NT, PL = SO::PL;
    constexpr bool F32 = PL > 1;
    static_assert(SEGMENT % (WINDOW * WAVES) == 0, "the waves' batches of a run continue across segments");
    extern __shared__ __attribute__((aligned(256))) char lds[];       // staged rows, [WAVES]; the sums of one row of tiles
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int m = lane & 15, g = lane >> 4;
    // the sub-blocks of a chunk, which read the same rows, run on the same XCD (blocks go round the eight XCDs)
    const int64_t per = 8 * (int64_t)a.n_sub;
    const int64_t chunk_id = (int64_t)blockIdx.x / per * 8 + blockIdx.x % 8;
    const int sub = (int)((int64_t)blockIdx.x % per / 8);
    if (chunk_id >= a.n_chunks) return;                   // whole block, before any barrier
    const int sub_i = sub % a.n_sub_in, sub_o = sub / a.n_sub_in;
    const int64_t p0 = chunk_id * a.chunk;                // positions below are relative to it
    const uint32_t p_end = (uint32_t)((p0 + a.chunk < a.n_triplets ? p0 + a.chunk : a.n_triplets) - p0);
    const __amdgpu_buffer_rsrc_t xrs = make_rsrc(a.x, a.x_bytes), drs = make_rsrc(a.dy, a.dy_bytes);
    const __amdgpu_buffer_rsrc_t irs = make_rsrc(a.tri_i, a.tri_bytes), ors = make_rsrc(a.tri_o, a.tri_bytes);
    const uint32_t xrow = (uint32_t)a.c_in * ES, drow = (uint32_t)a.c_out * ES;
    SO so;
    SI si;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds + (uint32_t)wave * (SO::BYTES + SI::BYTES);
    so.init(lds0, lane);
    si.init(lds0 + SO::BYTES, lane);
    so.set_chunk(sub_o, a.c_out, lane);
    si.set_chunk(sub_i, a.c_in, lane);

    // cell of the first triplet: the k with seg[k] <= p0 < seg[k+1]
    int k = 0;
    for (int kb = 0; kb < a.K; kb += 64) {
        const int kk = kb + lane;
        const bool hit = kk < a.K && a.seg[kk] <= p0 && p0 < a.seg[kk + 1];
        const unsigned long long msk = __ballot(hit);
        if (msk) { k = kb + __ffsll((long long)msk) - 1; break; }
    }
    k = __builtin_amdgcn_readfirstlane(k);

    // indices of the batch whose rows are requested next, as they come: not touched before a whole batch has been multiplied
    uint32_t ri, ro;
    const uint32_t ti = SI::triplet_of_lane(m, g), to = SO::triplet_of_lane(m, g);
    auto load_indices = [&](uint32_t pos) {
        const uint32_t first = (uint32_t)p0 + pos;         // (up to 286 words past the list: the walk runs two batches ahead)
        ri = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(irs, (int)index_offset(first, ti), 0, 0);
        ro = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(ors, (int)index_offset(first, to), 0, 0);
    };
    auto load_rows = [&](uint32_t n) {
        const uint32_t oi = ti < n ? ri * xrow : OOB_OFFSET, oo = to < n ? ro * drow : OOB_OFFSET;
        so.load(drs, oo, a.c_out);
        si.load(xrs, oi, a.c_in);
    };
    auto end_of = [&](int kk) -> uint32_t {               // end of cell kk's run inside the chunk
        const int64_t e = a.seg[kk + 1] - p0;
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)(e < (int64_t)p_end ? (uint32_t)e : p_end));
    };
    auto settle = [&](BatchCursor &c, uint32_t start) { settle_batch(c, start, p_end, (uint32_t)(WINDOW * wave), end_of); };
    auto left = [&](const BatchCursor &c) -> uint32_t { return c.pos < c.end ? (c.end - c.pos < (uint32_t)WINDOW ? c.end - c.pos : (uint32_t)WINDOW) : 0u; };
    BatchCursor nx{0u, end_of(k), k};
    settle(nx, (uint32_t)(WINDOW * wave));
    load_indices(nx.pos);
    load_rows(left(nx));
    settle(nx, nx.pos + WINDOW * WAVES);
    load_indices(nx.pos);

    bool first = true, more = false;                      // more: of the run whose sums so far are in its slot
    uint32_t p = 0u;
    while (p < p_end) {
        const uint32_t r_end = end_of(k);
        if (r_end <= p) { ++k; continue; }                // empty run
        const uint32_t q_end = r_end - p > SEGMENT ? p + SEGMENT : r_end;
        v4f acc[NTO][NTI];
#pragma unroll
        for (int o = 0; o < NTO; ++o)
#pragma unroll
            for (int i = 0; i < NTI; ++i) acc[o][i] = v4f{0.f, 0.f, 0.f, 0.f};
        for (uint32_t b = p + (uint32_t)(WINDOW * wave); b < q_end; b += WINDOW * WAVES) {
            so.store();
            si.store();
            load_rows(left(nx));
            settle(nx, nx.pos + WINDOW * WAVES);
            load_indices(nx.pos);
            if constexpr (!F32) {
                constexpr int AT = NTO < 4 ? NTO : 4, BT = NTI < 4 ? NTI : 4;      // tiles of operands held at a time
#pragma unroll
                for (int i0 = 0; i0 < NTI; i0 += BT) {
                    v4u bx[BT];
                    si.tiles(0, i0, bx);
#pragma unroll
                    for (int o0 = 0; o0 < NTO; o0 += AT) {
                        v4u av[AT];
                        so.tiles(0, o0, av);
#pragma unroll
                        for (int o = 0; o < AT; ++o)
#pragma unroll
                            for (int i = 0; i < BT; ++i)
                                acc[o0 + o][i0 + i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                    __builtin_bit_cast(v8bf, av[o]), __builtin_bit_cast(v8bf, bx[i]), acc[o0 + o][i0 + i], 0, 0, 0);
                    }
                }
            } else {
                v4u bx[PL][NTI];
#pragma unroll
                for (int pl = 0; pl < PL; ++pl) si.tiles(pl, 0, bx[pl]);
                auto mm = [&](const v4u &av, int q, int i, const v4f &c) {
                    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, av), __builtin_bit_cast(v8bf, bx[q][i]), c, 0, 0, 0);
                };
                // The five products with a smaller term in a sum of their own: against a long sum the matrix cores cut their low bits,
                // and with crowded cells or values of one sign these cuts add up (relative errors in one accumulator, apart, and
                // of one wave per chunk or fp32 sums on the vector ALUs: 20 -> 36, one cell, 6.6 M triplets, 1.4e-6, 2.3e-7, 5.0e-7;
                // 256 -> 256, 4.8 M, chunks of 4736, values of one sign, 9.3e-7, 6.3e-8, 1.5e-7).  The time is the same for 32 -> 32,
                // 1.5 us more of 42 for 20 -> 36 with 0.49 M triplets, 3260 and 3370 us for 256 -> 256.
                v4u av[PL][NTO];
#pragma unroll
                for (int pl = 0; pl < PL; ++pl) so.tiles(pl, 0, av[pl]);
#pragma unroll
                for (int o = 0; o < NTO; ++o)
#pragma unroll
                    for (int i = 0; i < NTI; ++i) {
                        v4f lo = {0.f, 0.f, 0.f, 0.f};
                        lo = mm(av[2][o], 0, i, mm(av[0][o], 2, i, lo));
                        lo = mm(av[0][o], 1, i, mm(av[1][o], 1, i, lo));
                        lo = mm(av[1][o], 0, i, lo);
                        acc[o][i] = mm(av[0][o], 0, i, acc[o][i]) + lo;
                    }
            }
            __builtin_amdgcn_wave_barrier();
        }
        // flush: the four waves' sums, one row of tiles at a time
        float *dstp = a.part + (size_t)(first ? chunk_id : a.n_chunks + k) * a.c_out * a.c_in;
        float (*red)[NTI][64][4] = reinterpret_cast<float (*)[NTI][64][4]>(lds);
        const int el = threadIdx.x >> 2, ej = threadIdx.x & 3;            // lane and register of the values this thread adds
#pragma unroll
        for (int o = 0; o < NTO; ++o) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NTI; ++i) *reinterpret_cast<v4f *>(red[wave][i][lane]) = acc[o][i];
            __syncthreads();
            const int co = SO::channel(sub_o, 16 * o + 4 * (el >> 4) + ej, a.c_out);
#pragma unroll
            for (int i = 0; i < NTI; ++i) {
                const int ci = SI::channel(sub_i, 16 * i + (el & 15), a.c_in);
                float v = red[0][i][el][ej];
#pragma unroll
                for (int w = 1; w < WAVES; ++w) v += red[w][i][el][ej];
                if (co >= 0 && ci >= 0) {
                    float *at = dstp + (size_t)co * a.c_in + ci;
                    *at = more ? *at + v : v;              // (written by this thread)
                }
            }
        }
        __syncthreads();                                   // (the next rows go where these sums lie)
        p = q_end;
        more = q_end < r_end;
        if (!more) {
            first = false;
            ++k;
        }
    }
}

// dw[k][e] = (partial of the run's head, if it starts inside a chunk) + partials of the chunks whose first
// triplet lies in run k.  A block of WAVES waves owns 64 VEC consecutive elements of one cell: wave w adds chunks
// c0 + w, c0 + w + WAVES, ... in ascending order, 32 at a time (each read is 256 VEC contiguous bytes), then these sums, and the
// waves' sums are added in order of w, so the result is reproducible.  (One long sum per wave loses precision: 20 -> 36 fp32, one
// cell, 6.6 M triplets, 8562 chunks: relative error 1.65e-6, by 32 2.3e-7, vector ALUs 5.0e-7.)  grid = (ceil(c_out*c_in / 64 VEC), K)
// Bound by the latency of the reads of one wave behind the other in small layers, which have few blocks, and by memory in large
// ones.  With four waves and one element per lane / as launch_reduce chooses, us: 32 -> 32 with 247 chunks a cell 15.3 / 6.3; 64 ->
// 64 with 100 10.8 / 8.8; 64 -> 128 with 60 8.4 / 7.7 (one element, sixteen waves: 15.3); 256 -> 256, 2046 chunks in all, 172 / 111.
template <int VEC, int WAVES_>
__global__ __launch_bounds__(WAVES_ * 64) void weight_reduce(const float *__restrict__ part, float *__restrict__ dw,
                                                             const int64_t *__restrict__ seg, int n_elem, int chunk,
                                                             int64_t n_chunks)
{
    typedef float vec __attribute__((ext_vector_type(VEC)));
    __shared__ vec sums[WAVES_][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int e = (blockIdx.x * 64 + lane) * VEC;                       // (VEC divides n_elem)
    const int k = blockIdx.y;
    const int64_t s = seg[k], t = seg[k + 1];
    vec v = 0.f, sum = 0.f;
    if (t > s && e < n_elem) {
        const int64_t c0 = (s + chunk - 1) / chunk, c1 = (t + chunk - 1) / chunk;
        auto of = [&](int64_t c) -> vec { return *reinterpret_cast<const vec *>(part + (size_t)c * n_elem + e); };
        int64_t c = c0 + wave;
        int n = 0;
        for (; c + 3 * WAVES_ < c1; c += 4 * WAVES_) {                  // four independent reads in flight
            const vec v0 = of(c), v1 = of(c + WAVES_), v2 = of(c + 2 * WAVES_), v3 = of(c + 3 * WAVES_);
            v += (v0 + v1) + (v2 + v3);
            if (++n % 8 == 0) { sum += v; v = 0.f; }
        }
        for (; c < c1; c += WAVES_) v += of(c);
    }
    sums[wave][lane] = sum + v;
    __syncthreads();
    if (wave == 0 && e < n_elem) {
        vec r = 0.f;
        if (t > s && s % chunk != 0) r = *reinterpret_cast<const vec *>(part + (size_t)(n_chunks + k) * n_elem + e);
#pragma unroll
        for (int w = 0; w < WAVES_; ++w) r += sums[w][lane];
        *reinterpret_cast<vec *>(dw + (size_t)k * n_elem + e) = r;
    }
}

// Triplets per chunk of weight_lds_kernel.  Its blocks, one per chunk, are spread evenly over the CUs and run at a fixed
// rate per CU, so a launch takes as long as the CU with the most blocks: the chunk length is chosen so that the number of
// blocks is a whole multiple m of the CU count, with about a thousand triplets per chunk and at most 2048 chunks (each has
// 256 KB of partial sums).  Clouds too small for one block per CU keep chunks of 512.
constexpr int64_t DEVICE_CUS = 256, LDS_MAX_CHUNKS = 2048;           // MI355X

int lds_chunk(int64_t n_triplets)
{
    int64_t m = (n_triplets + DEVICE_CUS * 500) / (DEVICE_CUS * 1000);   // nearest whole number of rounds
    if (m > LDS_MAX_CHUNKS / DEVICE_CUS) m = LDS_MAX_CHUNKS / DEVICE_CUS;
    if (m < 1 || n_triplets < DEVICE_CUS * 512) return 512;
    const int64_t chunk = ceil_div(n_triplets, DEVICE_CUS * m);
    return (int)((chunk + 31) / 32 * 32);
}

bool lds_shape(int in_dtype, int c_in, int c_out) { return in_dtype == PCPP_BF16 && c_in == 256 && c_out == 256; }

int launch_reduce(const float *part, float *dw, const int64_t *seg, int n_elem, int K, int chunk, int64_t n_chunks, hipStream_t stream)
{
    // Waves and elements per lane, by size of dW, number of blocks and chunks per cell (of the mean cell: on a surface half the cells hold
    // none).  Measured over 700 layers (64 .. 65 536 elements, 1 .. 216 cells, 0.3 .. 5000 chunks a cell); figures: the whole weight
    // gradient, us.
    // * Four elements per lane, which takes rows of dW at multiples of 16 bytes: a quarter of the blocks and of the requests.  Wide
    //   layers (128 -> 128, 216 cells, less than a chunk each: one element 50, four 38), and narrower ones with more waves where there
    //   are chunks for them (64 -> 64, 216 cells: one chunk each 22.2 with one element, 19.5 with four, 20.7 with eight waves; 4.5
    //   chunks 33.4, 31.6, 31.2).  Past 256 chunks a cell it is the chain of a wave that takes the time (64 -> 64, one cell, 972
    //   chunks: 31.5; one element and sixteen waves 24.8).
    // * One element per lane: sixteen waves from 4 chunks a cell on where the device holds all blocks at a time (8 -> 8, one cell, 1020
    //   chunks: four waves 39.4, sixteen 26.3; 16 -> 16, 125 cells, 8 chunks: 29.6 and 28.5).  With more blocks waves without a chunk
    //   take up room (127 -> 129, 216 cells, less than a chunk each: 59 with four, 121 with sixteen; 8 cells, 18 chunks: 28.5 and
    //   32.5), and the chains are worth more waves only when they are long (47 -> 61, 27 cells, 36 chunks: 32.8 with four, 31.9 with eight).
    const int64_t per_cell = n_chunks / K, blocks = ceil_div(n_elem, 64) * K;
    if (n_elem >= 4096 && n_elem % 4 == 0 && (reinterpret_cast<uintptr_t>(dw) & 15) == 0 && per_cell < 256) {
        const dim3 grid((unsigned)ceil_div(n_elem, 256), (unsigned)K);
        if (per_cell < (n_elem >= 16384 ? 32 : 4)) weight_reduce<4, 4><<<grid, 256, 0, stream>>>(part, dw, seg, n_elem, chunk, n_chunks);
        else weight_reduce<4, 8><<<grid, 512, 0, stream>>>(part, dw, seg, n_elem, chunk, n_chunks);
    } else {
        const dim3 grid((unsigned)ceil_div(n_elem, 64), (unsigned)K);
        if (per_cell >= (blocks <= 512 ? 4 : 64)) weight_reduce<1, 16><<<grid, 1024, 0, stream>>>(part, dw, seg, n_elem, chunk, n_chunks);
        else if (per_cell >= 20) weight_reduce<1, 8><<<grid, 512, 0, stream>>>(part, dw, seg, n_elem, chunk, n_chunks);
        else weight_reduce<1, 4><<<grid, 256, 0, stream>>>(part, dw, seg, n_elem, chunk, n_chunks);
    }
    PCPP_HIP_CHECK(hipGetLastError());
    return PCPP_OK;
}

// (16-byte row reads: the entry point has checked that x and dy are 16-byte aligned, and rows are 512 bytes)
int launch_weight_lds(const MvmrArgs &a, float *dw, const int32_t *tri_o, const int64_t *seg, float *part, hipStream_t stream)
{
    const int chunk = lds_chunk(a.n_triplets);
    const int64_t n_chunks = ceil_div(a.n_triplets, chunk);
    if (n_chunks > 0) {
        if (int rc = raise_lds_limit(reinterpret_cast<const void *>(&weight_lds_kernel), LDS_WEIGHT_BYTES)) return rc;
        weight_lds_kernel<<<(unsigned)n_chunks, LDS_WAVES * 64, LDS_WEIGHT_BYTES, stream>>>(
            static_cast<const uint16_t *>(a.feat), static_cast<const uint16_t *>(a.dense), part, tri_o, a.gather, seg, a.K,
            a.n_triplets, chunk, n_chunks);
        PCPP_HIP_CHECK(hipGetLastError());
    }
    return launch_reduce(part, dw, seg, a.c_src * a.c_dst, a.K, chunk, n_chunks, stream);
}

// The sub-block of dW that a block of weight_any_kernel owns, as channels of each side, and the chunk of the list.
// Enough blocks of up to 128 x 64 channels for four per CU, unless that would leave a wave fewer than two batches, and chunks no longer
// than the above.  (With half as many chunks the blocks' fixed cost and their partial sums halve, 128 -> 128 bf16 with 0.95 M triplets
// 74 us, 67, but a wave adds up twice as much: relative error 1.4e-7, 1.8e-7; 64 -> 64 fp32 with 0.35 M 39 us, 33, and 1.2e-7, 1.3e-7.)
// Sub-blocks of 128 x 64 channels read fewer rows, 64 x 64, of the same chunks, have three waves per SIMD for two: the latter up to
// 1.2 M triplets times the sub-blocks of 128 x 64 (128 -> 128, 0.14 M: 29.8 us, 128 x 64 37.1; 0.35 M: 42.7, 47.8; 0.58 M: 54.1, 57.7;
// 64 -> 128, 0.35 M: 33.8, 41.8; 0.93 M: 52.8, 59.4; 192 -> 128, 0.35 M: 51.9, 56.8; 0.57 M: 75.7, 70.4; 384 -> 320, 0.06 M: 59.1, 70.1).
// Beyond, where sub-blocks are many, it is the rows that count (512 -> 512, 0.39 M: 375, 300; 1024 -> 1024, 0.58 M: 2992, 1693).  Rows
// that are no multiple of 16 bytes cost more: 0.7 M (117 -> 211, 0.14 M: 57.2, 56.5; 0.22 M: 75.8, 67.2; 67 -> 91, 0.34 M: 47.8, 50.0; 0.49 M:
// 63.8, 57.4; 169 -> 123, 0.22 M: 56.7, 58.0; 0.34 M: 72.5, 66.0).
struct AnyShape { int co, ci, n_sub_in, n_sub, chunk; int64_t n_chunks; };

AnyShape any_shape(bool f32, int64_t n_triplets, int c_in, int c_out)
{
    AnyShape s;
    auto sub_blocks = [&](int widest) {
        auto channels = [&](int c) { return c <= 32 ? 32 : (c <= 64 || widest == 64 ? 64 : 128); };
        s.co = channels(c_out);
        s.ci = channels(c_in);
        if (s.co == 128 && s.ci == 128) s.ci = 64;         // 128 x 64 channels: 128 accumulator registers
        s.n_sub_in = (int)ceil_div(c_in, s.ci);
        return s.n_sub = s.n_sub_in * (int)ceil_div(c_out, s.co);
    };
    const int64_t n_sub = sub_blocks(f32 ? 64 : 128);
    if (!f32 && n_triplets * n_sub <= (c_in % 8 == 0 && c_out % 8 == 0 ? 1200000 : 700000)) sub_blocks(64);
    int64_t want = 1024 / n_sub;
    if (want < 8) want = 8;
    const int64_t short_chunks = ceil_div(n_triplets, f32 ? F32_CHUNK : SEGMENT), room = ((int64_t)1 << 26) / ((int64_t)c_in * c_out);
    if (short_chunks > want && want < room) want = short_chunks < room ? short_chunks : room;
    int64_t chunk = ceil_div(n_triplets > 0 ? n_triplets : 1, want);
    if (chunk < 2 * WINDOW * WAVES) chunk = 2 * WINDOW * WAVES;
    s.chunk = (int)((chunk + WINDOW * WAVES - 1) / (WINDOW * WAVES) * (WINDOW * WAVES));
    s.n_chunks = ceil_div(n_triplets, s.chunk);
    return s;
}

bool any_usable(int64_t n_in, int64_t n_out, int64_t n_triplets, int c_in, int c_out, int in_dtype)
{
    const size_t es = in_dtype == PCPP_F32 ? 4 : 2;
    return n_triplets > 0 && (size_t)n_triplets * 4 <= MAX_BUFFER_BYTES && (size_t)n_in * c_in * es <= MAX_BUFFER_BYTES &&
           (size_t)n_out * c_out * es <= MAX_BUFFER_BYTES;
}

template <typename SO, typename SI>
int launch_any(const WeightArgs &w, float *dw, hipStream_t stream)
{
    constexpr size_t staged = WAVES * (SO::BYTES + SI::BYTES), sums = WAVES * SI::NT * 64 * 4 * sizeof(float);
    constexpr size_t lds = staged > sums ? staged : sums;
    const int64_t blocks = ceil_div(w.n_chunks, 8) * 8 * w.n_sub;
    weight_any_kernel<SO, SI><<<(unsigned)blocks, WAVES * 64, lds, stream>>>(w);
    PCPP_HIP_CHECK(hipGetLastError());
    return launch_reduce(w.part, dw, w.seg, w.c_in * w.c_out, w.K, w.chunk, w.n_chunks, stream);
}

template <typename SO>
int launch_any_in(const WeightArgs &w, float *dw, int ci, hipStream_t stream)
{
    if constexpr (SO::PL > 1) {
        if (w.c_in < 2) return launch_any<SO, Direct<2, true>>(w, dw, stream);
        return ci == 32 ? launch_any<SO, Direct<2, false>>(w, dw, stream) : launch_any<SO, Direct<4, false>>(w, dw, stream);
    } else {
        if (w.c_in < 8) return launch_any<SO, Stage<4, true>>(w, dw, stream);
        if (ci == 32) return launch_any<SO, Stage<4, false>>(w, dw, stream);
        if constexpr (SO::CHK < 128)
            if (ci == 128) return launch_any<SO, Stage<16, false>>(w, dw, stream);
        return launch_any<SO, Stage<8, false>>(w, dw, stream);
    }
}

int launch_weight_any(const MvmrArgs &a, float *dw, const int32_t *tri_o, const int64_t *seg, float *part, hipStream_t stream)
{
    const bool f32 = a.in_dtype == PCPP_F32;
    const AnyShape s = any_shape(f32, a.n_triplets, a.c_src, a.c_dst);
    const size_t es = f32 ? 4 : 2;
    WeightArgs w{};
    w.x = a.feat; w.dy = a.dense; w.part = part;
    w.tri_o = tri_o; w.tri_i = a.gather; w.seg = seg;
    w.n_triplets = a.n_triplets; w.n_chunks = s.n_chunks;
    w.x_bytes = (uint32_t)((size_t)a.n_src * a.c_src * es); w.dy_bytes = (uint32_t)((size_t)a.n_centres * a.c_dst * es);
    w.tri_bytes = (uint32_t)((size_t)a.n_triplets * 4);
    w.K = a.K; w.c_in = a.c_src; w.c_out = a.c_dst; w.chunk = s.chunk; w.n_sub_in = s.n_sub_in; w.n_sub = s.n_sub;
    if (f32) {
        if (a.c_dst < 2) return launch_any_in<Direct<2, true>>(w, dw, s.ci, stream);
        return s.co == 32 ? launch_any_in<Direct<2, false>>(w, dw, s.ci, stream) : launch_any_in<Direct<4, false>>(w, dw, s.ci, stream);
    }
    if (a.c_dst < 8) return launch_any_in<Stage<4, true>>(w, dw, s.ci, stream);
    if (s.co == 32) return launch_any_in<Stage<4, false>>(w, dw, s.ci, stream);
    return s.co == 64 ? launch_any_in<Stage<8, false>>(w, dw, s.ci, stream) : launch_any_in<Stage<16, false>>(w, dw, s.ci, stream);
}

}  // namespace

// c_src = c_in (x), c_dst = c_out (dy, passed as `dense`); gather = tri_i
int mvmr_weight_mfma(const MvmrArgs &a, float *dw, const int32_t *tri_o, const int64_t *seg, void *workspace,
                     size_t workspace_bytes, hipStream_t stream, bool *handled)
{
    const bool lds = lds_shape(a.in_dtype, a.c_src, a.c_dst);
    *handled = lds || any_usable(a.n_src, a.n_centres, a.n_triplets, a.c_src, a.c_dst, a.in_dtype);
    if (!*handled) return PCPP_OK;
    const size_t need = mvmr_weight_mfma_workspace_bytes(a.n_triplets, a.c_src, a.c_dst, a.K, a.in_dtype);
    if (workspace_bytes < need) {
        set_error("pcpp_mvmr_bwd_weight: workspace has %zu bytes, needs %zu", workspace_bytes, need);
        return PCPP_ERR_WORKSPACE;
    }
    float *part = static_cast<float *>(workspace);
    // 256 -> 256: 31 + 22 us for 0.12 M triplets, 576 + 132 for 4.6 M, 4382 + 174 for 32 M (weight_any_kernel and its sums:
    // 54 + 21, 700 + 19, 8278 + 81, since each row is read by four sub-blocks)
    return lds ? launch_weight_lds(a, dw, tri_o, seg, part, stream) : launch_weight_any(a, dw, tri_o, seg, part, stream);
}

size_t mvmr_weight_mfma_workspace_bytes(int64_t n_triplets, int c_in, int c_out, int K, int in_dtype)
{
    const int64_t slots = lds_shape(in_dtype, c_in, c_out) ? ceil_div(n_triplets, lds_chunk(n_triplets))
                                                           : any_shape(in_dtype == PCPP_F32, n_triplets, c_in, c_out).n_chunks;
    return align_up((size_t)(slots + K) * c_in * c_out * sizeof(float));
}

}  // namespace pcpp
