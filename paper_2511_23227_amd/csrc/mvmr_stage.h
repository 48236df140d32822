// Gathered rows on their way to the matrix cores, shared by the rows and weight-gradient kernels that take any channel
// counts; not part of the C ABI.
//
// A wave takes 32 triplets (a window) at a time; the 16x16x32 MFMA wants the eight triplets of a lane's share of the
// reduction side by side for one channel, so rows have to be transposed on the way.
//
// bf16 rows (Stage) are read 16 bytes per lane, go row by row to a piece of LDS of the wave's own, and come back transposed
// (ds_read_b64_tr_b16).  The L1 cache serves four lanes per access whatever their width, so narrower reads leave it idle: a
// 64 -> 64 layer with 17 M triplets takes 158 us forward and 223 us for the weight gradient with them, 183 and 294 with 8
// bytes per lane and the transposition in registers.
//   ds_read_b64_tr_b16, inside each group of sixteen lanes: lane i receives element i % 4 of the 8 bytes that the lanes
//   4 j + i / 4, j = 0 .. 3, point to, i.e. channel i of four rows whose sixteen channels are read by four lanes each.
// LDS layout: 32 rows of ROWB = 64, 128 or 256 bytes; the 32-byte units of a row are exchanged by XOR with unit(row), so
// that the sixteen rows that one transposed read touches spread evenly over the banks (each is used twice, the least
// there is) and the 16-byte writes of whole rows do too.
//
// fp32 rows (Direct) are split exactly into three bf16 terms.  Three planes through LDS cost more than the L1 gains (32 ->
// 32, 2.4 M triplets: 98 us against 87 forward, 66 against 56 for the weight gradient), so a lane reads NV channels of
// eight rows and forms the operands in its registers.
#pragma once

#include <type_traits>

#include "mvmr_rows_common.h"

namespace pcpp {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4s lds_v4s;

constexpr int WINDOW = 32;                        // triplets

// Two floats as three pairs of bf16 whose sums they are exactly: 8 + 8 + 8 significant bits, each term the high half of
// what the ones before leave.  (v_dot2c_f32_bf16 gives what is left without masks, exactly, in seven instructions instead
// of eleven; it made no layer faster.)
__device__ static inline void split_pair(float x0, float x1, uint32_t &p1, uint32_t &p2, uint32_t &p3)
{
    const uint32_t a1 = __float_as_uint(x0) & 0xffff0000u, b1 = __float_as_uint(x1) & 0xffff0000u;
    const float ra = x0 - __uint_as_float(a1), rb = x1 - __uint_as_float(b1);
    const uint32_t a2 = __float_as_uint(ra) & 0xffff0000u, b2 = __float_as_uint(rb) & 0xffff0000u;
    p1 = __builtin_amdgcn_perm(b1, a1, 0x07060302u);
    p2 = __builtin_amdgcn_perm(b2, a2, 0x07060302u);
    p3 = __builtin_amdgcn_perm(__float_as_uint(rb - __uint_as_float(b2)), __float_as_uint(ra - __uint_as_float(a2)), 0x07060302u);
}

// bf16 rows.  RL lanes read a row (or the chunk of it that is staged), 64 / RL rows per load instruction.  NARROW: rows
// of fewer channels than a lane reads.
template <int RL, bool NARROW>
struct Stage {
    static constexpr int ES = 2, NV = 8;                             // bytes of a channel, channels per lane
    static constexpr int CHK = RL * NV, NT = CHK / 16, PL = 1;
    static constexpr int NI = RL / 2, RPI = 64 / RL;                 // load instructions per window, rows per instruction
    static constexpr uint32_t ROWB = CHK * 2, BYTES = WINDOW * ROWB;
    static_assert(CHK % 32 == 0 && (ROWB == 64 || ROWB == 128 || ROWB == 256), "row width");

    // exchange of the 32-byte units of row r
    __device__ static inline uint32_t unit(uint32_t r)
    {
        return ROWB == 64 ? (r >> 3) & 1u : (ROWB == 128 ? ((r >> 1) & 1u) | ((r >> 2) & 2u) : (r & 3u) | ((r >> 1) & 4u));
    }
    // The triplet whose source row lane (m, g) looks up (m < 8; the other lanes repeat them).
    __device__ static inline uint32_t triplet_of_lane(int m, int g)
    {
        const uint32_t e = (uint32_t)m & 7u;
        return RL == 4 ? 16u * (e >> 2) + 4u * (uint32_t)g + (e & 3u) : (RL == 8 ? 8u * (e >> 1) + 2u * (uint32_t)g + (e & 1u) : 4u * e + (uint32_t)g);
    }

    uint32_t x[NI][4];                            // rows in flight
    uint32_t w_at[2];                             // LDS addresses this lane writes to: even and odd exchanges
    uint32_t r_at;                                // ... and reads from, of unit 0, rows 8 g + 4 h + m / 4 at h = 0
    uint32_t col;                                 // byte of the row that this lane reads from

    __device__ inline void init(uint32_t lds, int lane)
    {
        const uint32_t m = (uint32_t)lane & 15u, g = (uint32_t)lane >> 4;
        const uint32_t r = (uint32_t)lane / RL, q = (uint32_t)lane % RL;
        const uint32_t byte = q * 16u, u = unit(r);         // rows of later instructions: RPI i + r
        w_at[0] = lds + r * ROWB + (byte ^ (32u * u));
        w_at[1] = lds + r * ROWB + (byte ^ (32u * (u ^ unit(8u))));
        const uint32_t rr = 8u * g + (m >> 2);
        r_at = lds + rr * ROWB + 32u * unit(rr) + 8u * (m & 3u);
    }
    // this lane's place in chunk `chunk` of rows of c channels
    __device__ inline void set_chunk(int chunk, int c, int lane)
    {
        const int pos = chunk * RL + lane % RL;
        if constexpr (NARROW) col = pos == 0 ? 0u : OOB_OFFSET;
        else col = pos * NV < c ? (uint32_t)lane_channel(pos, NV, c) * ES : 0u;   // (no channel: repeats the row's first ones)
    }
    // The channel at place `at` of chunk `chunk`, -1: none, or one that the lane before has read already.
    __device__ static inline int channel(int chunk, int at, int c)
    {
        const int place = chunk * CHK + at;
        if constexpr (NARROW) return place < c ? place : -1;
        const int pos = place / NV, ch = lane_channel(pos, NV, c) + place % NV;
        return pos * NV < c && ch >= pos * NV ? ch : -1;
    }
    // Requests of instruction I; offs: lane (m, g) holds the offset of triplet_of_lane's row.  A row's offset reaches its
    // lanes by the DPP broadcast inside the add that forms the address.
    template <int I> __device__ inline void load_one(const __amdgpu_buffer_rsrc_t &rs, uint32_t offs, int c)
    {
        uint32_t at = 0u;
        constexpr int P = 16 / RL;                // rows per sixteen lanes
        if constexpr (P == 1) {
            at = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)offs, 0x150 + I, 0xf, 0xf, true);
        } else if constexpr (P == 2) {
            at = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)offs, 0x150 + 2 * I, 0xf, 0xf, true);
            at = (uint32_t)__builtin_amdgcn_update_dpp((int)at, (int)offs, 0x150 + 2 * I + 1, 0xf, 0xc, false);
        } else {
            at = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)offs, 0x150 + 4 * I, 0xf, 0xf, true);
            at = (uint32_t)__builtin_amdgcn_update_dpp((int)at, (int)offs, 0x150 + 4 * I + 1, 0xf, 0x2, false);
            at = (uint32_t)__builtin_amdgcn_update_dpp((int)at, (int)offs, 0x150 + 4 * I + 2, 0xf, 0x4, false);
            at = (uint32_t)__builtin_amdgcn_update_dpp((int)at, (int)offs, 0x150 + 4 * I + 3, 0xf, 0x8, false);
        }
        if constexpr (NARROW) {
            // fewer channels than a lane reads: one at a time (a whole piece could go past the tensor's end)
            at = col == 0u ? at : OOB_OFFSET;
#pragma unroll
            for (int e = 0; e < NV; ++e) {
                const int off = (int)(e < c ? at + (uint32_t)(e * ES) : OOB_OFFSET);
                const uint32_t v = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, off, 0, 0);
                x[I][e >> 1] = (e & 1) ? x[I][e >> 1] | v << 16 : v;
            }
        } else {
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(at + col), 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) x[I][i] = v[i];
        }
    }
    __device__ inline void load(const __amdgpu_buffer_rsrc_t &rs, uint32_t offs, int c)
    {
        load_one<0>(rs, offs, c);
        load_one<1>(rs, offs, c);
        if constexpr (NI > 2) { load_one<(NI > 2 ? 2 : 0)>(rs, offs, c); load_one<(NI > 2 ? 3 : 0)>(rs, offs, c); }
        if constexpr (NI > 4) {
            load_one<(NI > 4 ? 4 : 0)>(rs, offs, c); load_one<(NI > 4 ? 5 : 0)>(rs, offs, c);
            load_one<(NI > 4 ? 6 : 0)>(rs, offs, c); load_one<(NI > 4 ? 7 : 0)>(rs, offs, c);
        }
    }
    // rows to LDS.  The statement at the end keeps the next requests behind the last use of the registers that they fill:
    // ahead of it the compiler would give them other registers, and wait for the rows in order to copy them over.
    __device__ inline void store() const
    {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            // row RPI i + r: exchanged like row r, with unit(8) on top where bit 3 of the row comes from i
            const uint32_t at = (RPI == 16 ? w_at[0] : w_at[(RPI * i >> 3) & 1]) + (uint32_t)(RPI * i) * ROWB;
            *reinterpret_cast<__attribute__((address_space(3))) v4u *>(at) = v4u{x[i][0], x[i][1], x[i][2], x[i][3]};
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();
    }
    // operand tiles t0 .. t0 + N - 1: lane (m, g) gets channel 16 t + m of the triplets 8 g .. 8 g + 7.  (All requested before
    // the first is used; and the next rows are not stored before these have been read.)
    template <int N> __device__ inline void tiles(int, int t0, v4u (&out)[N]) const
    {
#pragma unroll
        for (int t = 0; t < N; ++t) {
            const uint32_t at = (r_at ^ (32u * (uint32_t)(t0 + t))) ;
            const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_v4s *>(at));
            const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_v4s *>(at + 4 * ROWB));
            out[t] = __builtin_bit_cast(v4u, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
#pragma unroll
        for (int t = 0; t < N; ++t) asm volatile("" : "+v"(out[t]) :: "memory");
    }
};

// fp32 rows.  Sixteen lanes read a row (or a chunk of it), NV = 2 or 4 channels each; lane (m, g) reads the rows of the
// triplets 8 g .. 8 g + 7.  Operand tile t holds the channels NV m + t.
template <int NV_, bool NARROW>
struct Direct {
    static constexpr int ES = 4, NV = NV_, CHK = 16 * NV, NT = NV, PL = 3;
    static constexpr uint32_t BYTES = 0;
    __device__ static inline uint32_t triplet_of_lane(int m, int g) { return 8u * (uint32_t)g + ((uint32_t)m & 7u); }

    uint32_t x[8][NV];                            // rows in flight
    v4u op[PL][NT];
    uint32_t col;

    __device__ inline void init(uint32_t, int) {}
    __device__ inline void set_chunk(int chunk, int c, int lane)
    {
        const int pos = chunk * 16 + (lane & 15);
        if constexpr (NARROW) col = pos == 0 ? 0u : OOB_OFFSET;
        else col = pos * NV < c ? (uint32_t)lane_channel(pos, NV, c) * ES : 0u;   // (no channel: repeats the row's first ones)
    }
    __device__ static inline int channel(int chunk, int at, int c)
    {
        const int pos = chunk * 16 + at % 16;
        if constexpr (NARROW) return pos == 0 && at / 16 < c ? at / 16 : -1;
        const int ch = lane_channel(pos, NV, c) + at / 16;
        return pos * NV < c && ch >= pos * NV ? ch : -1;
    }
    template <int E> __device__ inline void load_one(const __amdgpu_buffer_rsrc_t &rs, uint32_t offs, int c)
    {
        const uint32_t at = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)offs, 0x150 + E, 0xf, 0xf, true);
        if constexpr (NARROW) {
#pragma unroll
            for (int e = 0; e < NV; ++e)
                x[E][e] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(e < c && col == 0u ? at + (uint32_t)(e * ES) : OOB_OFFSET), 0, 0);
        } else if constexpr (NV == 2) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)(at + col), 0, 0);
            x[E][0] = v[0]; x[E][1] = v[1];
        } else {
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(at + col), 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) x[E][i] = v[i];
        }
    }
    __device__ inline void load(const __amdgpu_buffer_rsrc_t &rs, uint32_t offs, int c)
    {
        load_one<0>(rs, offs, c); load_one<1>(rs, offs, c); load_one<2>(rs, offs, c); load_one<3>(rs, offs, c);
        load_one<4>(rs, offs, c); load_one<5>(rs, offs, c); load_one<6>(rs, offs, c); load_one<7>(rs, offs, c);
    }
    // The operands.  The statement keeps the next requests behind the last use of their registers, as in Stage.
    __device__ inline void store()
    {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t p1, p2, p3;
                split_pair(__uint_as_float(x[2 * q][t]), __uint_as_float(x[2 * q + 1][t]), p1, p2, p3);
                op[0][t][q] = p1; op[1][t][q] = p2; op[2][t][q] = p3;
            }
#pragma unroll
        for (int p = 0; p < PL; ++p)
#pragma unroll
            for (int t = 0; t < NT; ++t) asm volatile("" : "+v"(op[p][t]) :: "memory");
    }
    template <int N> __device__ inline void tiles(int p, int t0, v4u (&out)[N]) const
    {
#pragma unroll
        for (int t = 0; t < N; ++t) out[t] = op[p][t0 + t];
    }
};

}  // namespace pcpp
