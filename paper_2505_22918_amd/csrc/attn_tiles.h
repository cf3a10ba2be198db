// The two-tile walk shared by the attention kernels (attn.hip, attn_dense.hip): one wave
// holds 64 queries as two tiles of 32 and takes 32-key chunks of K and V from LDS.
//
//   S^T = K Q^T          v_mfma_f32_32x32x16_bf16, keys x queries
//   online softmax       fp32, exp2 with log2(e)/sqrt(D) folded in
//   O^T += V^T P^T       v_mfma_f32_32x32x16_bf16, head-dim x queries
//
// Computing the transposed products keeps every query in one lane column: the
// 32x32 accumulator of S^T hands each lane 16 keys of one query, which are
// exactly the 8+8 key values the B operand of the P V product needs, so P
// never leaves registers.  The rows of the V^T operand are permuted so that
// each lane's 16 accumulator values of O^T are 16 consecutive head dims of
// its query.
//
// The tiles run half a step apart: while the vector unit takes the softmax of one
// tile's chunk, the matrix cores form the other tile's next scores and its last
// P V product, one MFMA for every two scores.  No MFMA of a phase depends on its
// softmax, each tile's scores stay in one set of registers (the rare rescale finds them
// there), and K and V operands are read once for both tiles.
//
// 72-wide heads.  The 8 head dims past 64 take one k-step of Q K^T (half of it zeros) and
// one 16x16x32 product per 16 queries of P V, both tiles into one accumulator (a
// tile's V operand is zero in the rows of the other): 320 matrix cycles a chunk and tile
// instead of 352 with a third 32-row tile, and 233-243 registers instead of 370-420, so
// these heads too run two waves per SIMD.  The zeros never meet a NaN or an infinity,
// so that one query row's cannot reach another's.
//
// Softmax.  The running max starts at the first chunk's max and moves only
// when a chunk's probabilities against it reach 2^64 (far below fp32 and bf16
// overflow); that rare case rescales O and l and recomputes the chunk.  Without
// statistics no per-chunk max is taken: the overflow test reads the chunk's row sum.
#pragma once

#include <type_traits>

#include "attn_common.h"

namespace rt {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

#define RT_FENCE __builtin_amdgcn_sched_barrier(0)

// hides a lane constant's value, so that what derives from it is formed anew
// (one v_xad_u32 per read) instead of held in registers throughout the walk: 72-wide
// heads need the registers; 64-wide dense walks are 2.5 % faster without
__device__ __forceinline__ int fresh(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

__device__ __forceinline__ f32x16 mma(const bf16x8& x, const bf16x8& y, const f32x16& z) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, z, 0, 0, 0);
}

// STATS: the exact row max is tracked.  F32_SUM: l sums the fp32 probabilities (where l, m
// or rho are outputs); otherwise, where l only normalises O, the bf16 ones P V multiplies,
// two per v_dot2c_f32_bf16, so that numerator and denominator use the same weights.
// ZERO: LDS offset of 16 zero bytes at it and 8 rows on (72-wide heads).
template <int D, bool STATS, bool F32_SUM, int ZERO>
struct Tiles {
    using G = Geo<D>;
    static constexpr int DS = 4;                // 16-wide k-steps of Q K^T (and a tail step)
    static constexpr int ROWB = G::SLOTS * 16;  // LDS bytes per K / V row (= 2 * D)
    static constexpr bool TAIL = D == 72;       // 8 head dims past the two 32-row tiles of O^T
    static_assert(ROWB == 2 * D, "rows are unpadded");

    lds_u8* lds;
    int lane, l32, hi;
    int k_rd, v_rd, t_rd;
    int T, full_lim;
    float c2;  // log2(e) / sqrt(D)
    // Of a 72-wide head's last 8 dims, tile Q's queries sit in lanes of half Q, with
    // zeros in the other half and in K's there.
    bf16x8 qop[2][DS], qtl[2];
    f32x16 oacc[2][2];
    f32x4 tacc[2];  // tail of O^T for 16 queries: rows 0-7 tile 0's dims, 8-15 tile 1's
    float m_run[2], m_top[2], l_run[2];
    uint32_t pk[2][8];   // bf16 probabilities of the chunk before
    f32x16 s0, s1;       // scores of the two query tiles
    bf16x8 kop[DS];      // K operands: chunk t (tile 0 has used it) or t + 1
    bf16x8 vop[4];       // V^T operands (dt, ks) of the chunk before, or of chunk t
    bf16x8 kt1, vt1;     // the tails of both, for query tile 1
    bf16x8 kt0, vt0;     // and for tile 0, read by its own phase

    // the lane's constants, formed anew: after the walk, so that none is held throughout it
    __device__ __forceinline__ void lanes() {
        lane = fresh(__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)));
        l32 = lane & 31;
        hi = lane >> 5;
    }
    __device__ __forceinline__ void init(lds_u8* smem, int T_, float scale_log2) {
        lds = smem;
        lanes();
        T = T_;
        full_lim = (T - 32) * (D * 2);
        c2 = scale_log2;
        // K A-operand reads: row l32, head-dim chunk 2s + hi
        k_rd = l32 * ROWB + ((hi ^ kswz<D>(l32)) * 16);
        // V^T A-operand transpose reads.  In a group of 16 lanes (G4 = lane / 16),
        // lane L supplies key row 4*hi + L/4 (+16ks, +8 for the second read) at the
        // 4 head dims starting at 32dt + 16(L & 1) + 8(G4 & 1) + 4((L >> 1) & 1).
        // Lane 4a + b of the group then receives 4 consecutive keys of head dim
        // 32dt + 16(a & 1) + 8(G4 & 1) + 4(a >> 1) + b, which puts head dim
        // 32dt + 16h + 4j + i on O^T accumulator row 8j + 4h + i: lane (h, col)
        // accumulates head dims 32dt + 16h .. +15 of query col.
        const int G4 = lane >> 4, L = lane & 15;
        {
            const int r = 4 * hi + (L >> 2);
            const int d = 16 * (L & 1) + 8 * (G4 & 1) + 4 * ((L >> 1) & 1);
            v_rd = r * ROWB + (((d >> 3) ^ vswz<D>(r)) * 16) + (d & 7) * 2;
        }
        // the tail's: lane group g of 16 takes keys 16 (g & 1) + 4 (g >> 1) + (0 .. 3, 8 .. 11)
        t_rd = TAIL ? (16 * (G4 & 1) + 4 * (G4 >> 1) + (L >> 2)) * ROWB + (64 + 4 * (L & 1)) * 2 : 0;
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
            m_run[qt] = -1e30f;  // finite: a fully masked chunk then yields p = 0, not NaN
            m_top[qt] = -INFINITY;
            l_run[qt] = 0.f;
            oacc[qt][0] = oacc[qt][1] = f32x16{};
            tacc[qt] = f32x4{};
#pragma unroll
            for (int x = 0; x < 8; ++x) pk[qt][x] = 0u;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) vop[k] = bf16x8{};
        kt0 = kt1 = vt0 = vt1 = qtl[0] = qtl[1] = bf16x8{};
    }

    // Q^T operands: lane holds query l32 of tile qt, head dims 16s + 8hi .. +7 (zero past
    // row nrow).  Plain loads: the compiler waits before their first use.
    __device__ __forceinline__ void load_q(const uint16_t* rows, int nrow) {
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc((void*)rows, (short)0, nrow * D * 2, 0x00020000);
        auto load = [&](int off) {
            return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
        };
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
            const int row = (qt * 32 + l32) * (D * 2);
#pragma unroll
            for (int s = 0; s < DS; ++s) qop[qt][s] = load(row + (2 * s + hi) * 16);
            if (TAIL) qtl[qt] = load(hi == qt ? row + 128 : kOob);
        }
    }
    // Q has landed: no wait of the compiler's in the walk
    __device__ __forceinline__ void settle_q() {
#pragma unroll
        for (int s = 0; s < DS; ++s) asm volatile("" : "+v"(qop[0][s]), "+v"(qop[1][s]));
        if (TAIL) asm volatile("" : "+v"(qtl[0]), "+v"(qtl[1]));
    }

    // row max of one chunk; lane holds keys 8j + 4hi + i for acc index 4j + i, the
    // other 16 keys of its query sit in lane l ^ 32
    static __device__ __forceinline__ float chunk_max(const f32x16& sc) {
        float mx = fmaxf(fmaxf(sc[0], sc[1]), sc[2]);
#pragma unroll
        for (int x = 3; x < 15; x += 2) mx = fmaxf(fmaxf(mx, sc[x]), sc[x + 1]);
        mx = fmaxf(mx, sc[15]);
        return pair_max(mx);
    }
    // keys past T score -inf.  cb: byte offset of the chunk in the head's K; chunks at
    // offsets up to full_lim hold 32 keys below T.
    __device__ __forceinline__ void mask(int cb, f32x16& sc) {
        if (cb <= full_lim) return;
        const int lim = T - cb / (D * 2) - 4 * hi;
#pragma unroll
        for (int x = 0; x < 16; ++x) {
            if (8 * (x >> 2) + (x & 3) >= lim) sc[x] = -INFINITY;
        }
    }
    static __device__ __forceinline__ bf16x8 pk_op(const uint32_t (&p)[8], int ks) {
        return __builtin_bit_cast(bf16x8, u32x4{p[4 * ks], p[4 * ks + 1], p[4 * ks + 2], p[4 * ks + 3]});
    }
    // LDS addresses: of swizzled rows, chunk 2s + hi sits at the first one's slot
    // with bits 1.. flipped by s, and V's second 32 head dims at slot ^ 4.
    __device__ __forceinline__ bf16x8 tr_read(const lds_u8* p) {
        const bf16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)p);
        const bf16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p + 8 * ROWB));
        return __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
    }
    __device__ __forceinline__ bf16x8 v_read(int vb, int vo, int dt, int ks) {
        return tr_read(lds + (G::SWZ ? (vb ^ (64 * dt)) + vo : vb + vo + 64 * dt) + 16 * ks * ROWB);
    }
    // the tail's V^T operand for query tile Q: 8 dims at its rows, zeros at the other's
    __device__ __forceinline__ bf16x8 t_read(int vo, int Q) {
        return tr_read(lds + (((lane >> 1) & 1) == Q ? vo + t_rd : ZERO));
    }
    __device__ __forceinline__ bf16x8 k_read(int kb, int ko, int s) {
        return *(const lds_bf16x8*)(lds + (G::SWZ ? (kb ^ (32 * s)) + ko : kb + ko + 32 * s));
    }
    // tail K operand of query tile Q: the row's last chunk in lanes of half Q, else zeros
    __device__ __forceinline__ bf16x8 k_tail(int kb, int ko, int Q) {
        return *(const lds_bf16x8*)(lds + (hi == Q ? kb + ko + 128 - 16 * Q : ZERO));
    }
    // The 8-dim tails of O^T: a 16x16x32 product per tile and 16 queries, both tiles
    // into one accumulator.  Swapping the odd 16-lane rows of the first 8 keys'
    // registers with the even rows of the others' turns the two 16-key operands
    // of a 32-query tile into the two 32-key operands of its 16-query halves.
    __device__ __forceinline__ void tail_mma(const bf16x8& x, const uint32_t (&p)[8]) {
        uint32_t y[8];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            auto s = __builtin_amdgcn_permlane16_swap(p[r], p[4 + r], false, false);
            y[r] = s[0];
            y[4 + r] = s[1];
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) tacc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, pk_op(y, h), tacc[h], 0, 0, 0);
    }
    static __device__ __forceinline__ float bf16_sum(const uint32_t (&p)[8]) {
        const bf16x2 one2 = {(__bf16)1.0f, (__bf16)1.0f};
        float a0 = 0.f, a1 = 0.f;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            a0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, p[x]), one2, a0, false);
            a1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, p[4 + x]), one2, a1, false);
        }
        return a0 + a1;
    }
    // per-query values of the tiles as the tail accumulators' lanes hold them: lane l has
    // query 16 h + l % 16 of tile l / 32, dims 64 + 4 (l / 16 % 2) ..
    __device__ __forceinline__ float tail_bcast(float x0, float x1, int h) {
        const int src = (16 * h + (lane & 15)) << 2;
        const int y0 = __builtin_amdgcn_ds_bpermute(src, __float_as_uint(x0));
        const int y1 = __builtin_amdgcn_ds_bpermute(src, __float_as_uint(x1));
        return __uint_as_float(hi ? y1 : y0);
    }

    // scores of query tile Q against the chunk whose operands kop holds (its tail: LDS
    // offset ko; its rows: byte offset cb)
    __device__ __forceinline__ f32x16 scores(int Q, int ko, int cb) {
        f32x16 x = {};
#pragma unroll
        for (int s = 0; s < DS; ++s) x = mma(kop[s], qop[Q][s], x);
        if (TAIL) x = mma(k_tail(k_rd, ko, Q), qtl[Q], x);
        mask(cb, x);
        return x;
    }
    // operands of the walk's first chunk, and tile 0's scores
    __device__ __forceinline__ void first_chunk(int ko, int cb) {
#pragma unroll
        for (int s = 0; s < DS; ++s) kop[s] = k_read(k_rd, ko, s);
        if (TAIL) kt1 = k_tail(k_rd, ko, 1);
        s0 = scores(0, ko, cb);
    }
    // both tiles start from their first chunk's max; tile 1's scores of it stay in s1
    __device__ __forceinline__ void first_max(int ko, int cb) {
        s1 = scores(1, ko, cb);
        m_run[0] = fmaxf(chunk_max(s0), -1e30f);
        m_run[1] = fmaxf(chunk_max(s1), -1e30f);
    }

    // One phase: the softmax of query tile Q's chunk t runs on the VALU while the
    // matrix cores form the other tile's next scores and its last P V:
    //   Q = 0: S_1(t) = K(t) Q_1,       O_1 += V(t-1) P_1(t-1); the operands of
    //          chunks t+1 (K, at LDS offset ko) and t (V, at vo) are read behind
    //          their last use
    //   Q = 1: S_0(t+1) = K(t+1) Q_0,   O_0 += V(t) P_0(t); the tails' operands
    //          of both tiles are read
    // (QK, PV false at the ends of a walk: no scores to form, no P V pending).
    // nb: byte offset of the chunk the other tile scores.  Where the wave does not
    // score the block (!on), its probabilities are exp2(-inf) = 0; scores of
    // non-finite keys, whose probabilities are not, end up in the rare branch.
    template <int Q, bool QK = true, bool PV = true>
    __device__ __forceinline__ void phase(bool on, int nb, int ko, int vo) {
        constexpr int R = 1 - Q;
        f32x16& sc = Q ? s1 : s0;
        f32x16& sn = Q ? s0 : s1;
        const float mc = on ? m_run[Q] * c2 : INFINITY;
        const int kb = TAIL ? fresh(k_rd) : k_rd, vb = TAIL ? fresh(v_rd) : v_rd;
        if (TAIL && Q == 1) {
            if (QK) kt0 = k_tail(kb, ko, 0);
            vt0 = t_read(vo, 0);
        }
        // fp32 row sums in the order of the sparse walk: groups of four, groups 0
        // and 2 in one chain, 1 and 3 in the other
        float sa = 0.f, sb = 0.f, part = 0.f;
        // The chain of a score (scale, exp2, sum and pack) is spread over three slots,
        // so that nothing issued in one waits for another of the same.
        float f[16], e[16];
        auto scale = [&](int x) {
            if (STATS) m_top[Q] = fmaxf(fmaxf(m_top[Q], sc[x]), sc[x + 1]);
            f[x] = __builtin_fmaf(sc[x], c2, -mc);
            f[x + 1] = __builtin_fmaf(sc[x + 1], c2, -mc);
        };
        auto expo = [&](int x) {
            e[x] = __builtin_amdgcn_exp2f(f[x]);
            e[x + 1] = __builtin_amdgcn_exp2f(f[x + 1]);
        };
        auto keep = [&](int x) {
            if (F32_SUM) {
                part = x % 4 == 0 ? e[x] + e[x + 1] : part + (e[x] + e[x + 1]);
                if (x == 2) sa = part;
                if (x == 6) sb = part;
                if (x == 10) sa += part;
                if (x == 14) sb += part;
            }
            pk[Q][x / 2] = pack_bf16(e[x], e[x + 1]);
        };
        auto slot = [&](int j) {
            expo(2 * j);
            if (j < 7) scale(2 * j + 2);
            if (j > 0) keep(2 * j - 2);
        };
        scale(0);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            RT_FENCE;
            if (QK) sn = mma(kop[k], qop[R][k], k == 0 ? f32x16{} : sn);
            RT_FENCE;  // reads stay behind the operand's last use: no second set of registers
            if (Q == 0) kop[k] = k_read(kb, ko, k);
            slot(2 * k);
            RT_FENCE;
            if (PV) oacc[R][k & 1] = mma(vop[k], pk_op(pk[R], k >> 1), oacc[R][k & 1]);
            RT_FENCE;
            if (Q == 0) vop[k] = v_read(vb, vo, k & 1, k >> 1);
            slot(2 * k + 1);
        }
        RT_FENCE;
        keep(14);
        // the max is taken here, not moved behind the last read of the scores
        if (STATS) asm volatile("" : "+v"(m_top[Q]));
        if (TAIL) {
            if (QK) sn = mma(Q ? kt0 : kt1, qtl[R], sn);
            if (PV) tail_mma(Q ? vt0 : vt1, pk[R]);
            RT_FENCE;
            if (Q == 1) {
                kt1 = k_tail(kb, ko, 1);
                vt1 = t_read(vo, 1);
            }
        }
        float ls = F32_SUM ? sa + sb : bf16_sum(pk[Q]);
        if (__builtin_amdgcn_ballot_w64(!(ls < kJump))) {
            if (!on) {
#pragma unroll
                for (int x = 0; x < 8; ++x) pk[Q][x] = 0u;
                ls = 0.f;
            } else {
                // A probability reached 2^64: O and l move to the chunk's max.  The tails'
                // product would carry a NaN probability into the other tile (zero rows of V
                // times NaN): l alone takes it, and with l the row's output is NaN.
                auto number = [](float p) { return TAIL ? fminf(p, 2.0f) : p; };  // 2 for a NaN
                const float mnew = fmaxf(m_run[Q], chunk_max(sc));
                const float alpha = __builtin_amdgcn_exp2f((m_run[Q] - mnew) * c2);
                l_run[Q] *= alpha;
                oacc[Q][0] *= alpha;
                oacc[Q][1] *= alpha;
                if (TAIL) {
                    tacc[0] *= tail_bcast(Q ? 1.f : alpha, Q ? alpha : 1.f, 0);
                    tacc[1] *= tail_bcast(Q ? 1.f : alpha, Q ? alpha : 1.f, 1);
                }
                m_run[Q] = mnew;
                const float mn = mnew * c2;
#pragma unroll
                for (int x = 0; x < 16; x += 4) {
                    RT_FENCE;
#pragma unroll
                    for (int y = 0; y < 4; ++y) e[y] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[x + y], c2, -mn));
                    pk[Q][x / 2] = pack_bf16(number(e[0]), number(e[1]));
                    pk[Q][x / 2 + 1] = pack_bf16(number(e[2]), number(e[3]));
                    part = (e[0] + e[1]) + (e[2] + e[3]);
                    if (x == 0) sa = part;
                    if (x == 4) sb = part;
                    if (x == 8) sa += part;
                    if (x == 12) sb += part;
                }
                RT_FENCE;
                ls = sa + sb;
                if (!F32_SUM && !(TAIL && ls != ls)) ls = bf16_sum(pk[Q]);
            }
        }
        l_run[Q] += ls;
        if (QK) mask(nb, sn);
    }

    // the pending P V of tile 1
    __device__ __forceinline__ void pv1() {
#pragma unroll
        for (int k = 0; k < 4; ++k) oacc[1][k & 1] = mma(vop[k], pk_op(pk[1], k >> 1), oacc[1][k & 1]);
        if (TAIL) tail_mma(vt1, pk[1]);
    }
};

}  // namespace
}  // namespace rt
