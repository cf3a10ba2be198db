// Attention over every key block of a head (gfx950, CDNA4): dense attention with
// row statistics, and the dropped keys of a caching step.
//
//   rt_attn_full   Eq.1 with the Eq.4 denominator
//   rt_attn_cache  App. A.3: after the sparse walk (attn.hip) has left O_s and the kept
//                  keys' statistics, the other keys, then O_full, rho (Eq.8), R (Eq.10)
//
// Every query block of a head reads the whole K and V of that head, so a
// workgroup of W waves (64 query rows each, two waves per SIMD) shares one K and one V
// ring in LDS, three 64-key stages each, filled by all its waves with
// buffer_load ... lds; one barrier per 64 keys, two stages of lead.  With a ring
// per wave the chunk loads kept the vector-memory path 84-92 % busy.
//
// Products, operand layouts and softmax are those of attn.hip: S^T = K Q^T and
// O^T += V^T P^T by v_mfma_f32_32x32x16_bf16, each query in one lane column, P in
// registers.  A wave holds two 32-query tiles and runs them half a step apart:
// while the vector unit takes the softmax of one tile's chunk, the matrix cores
// form the other tile's next scores and its last P V product, one MFMA for every two
// scores.  No MFMA of a phase depends on its softmax, each tile's scores stay in
// one set of registers (the rare rescale finds them there), and K and V operands
// are read once for both tiles.
//
// 72-wide heads.  The 8 head dims past 64 take one k-step of Q K^T (tile 0's query
// values in the lower half of the lanes, tile 1's in the upper) and one 16x16x32
// product per 16 queries of P V, both tiles into one accumulator: 320 matrix cycles a
// chunk and tile instead of 352 with a third 32-row tile, and 233-237 registers instead of
// 370-420, so these heads too run two waves per SIMD.
//
// Bound by the vector unit's issue slots (an MFMA takes about 8 of its cycles
// beside its own; 131 instructions per 32-key chunk and 64 rows) and by power:
// with zero queries, keys and values the same instructions run 21 % faster, as a
// large bf16 product does.  Measured, before -> now: PixArt-Sigma-2K dense with
// statistics (32 heads, 16384 tokens, D = 72) 3998 -> 2582 us (0.96 PFLOP/s of real
// dims), CogVideoX caching step (60 heads, 17776 tokens, D = 64) 5739 -> 5266 us, of
// which the sparse walk is 235; PixArt-Sigma-1024 caching step 289 -> 201 us.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "attn_common.h"
#include "kernels.h"

namespace rt {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kOff = 0x60000000;  // buffer offset past every record, also after small additions
constexpr int kAct = 1;           // flags in the low bits of a block offset: this wave scores the block
constexpr int kEnd = 2;           // past the last block
constexpr int kFlags = 3;

template <int D, int W, bool STATS, bool CACHE>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_dense(AttnArgs a) {
    using G = Geo<D>;
    constexpr int DS = 4;                    // 16-wide k-steps of Q K^T (and a tail step)
    constexpr int ROWB = G::SLOTS * 16;      // LDS bytes per K / V row (= 2 * D)
    constexpr int HALF = 32 * ROWB;          // one 32-key chunk
    constexpr int PAIR = 2 * HALF;           // one ring stage: two chunks
    constexpr int NS = 3;                    // ring stages
    constexpr int SL = 64 * G::SLOTS;        // 16-byte slots per stage and tensor
    constexpr int NFULL = SL / (64 * W);     // whole DMA instructions per wave
    constexpr int REM = (SL - NFULL * 64 * W) / W;  // lanes of one more
    constexpr int NDMA = NFULL + (REM ? 1 : 0);
    constexpr bool TAIL = D == 72;           // 8 head dims past the two 32-row tiles of O^T
    constexpr int BLK = 64 * 2 * D;          // bytes of a 64-key block
    constexpr bool BF16_SUM = !STATS && !CACHE;
    static_assert(ROWB == 2 * D, "rows are unpadded");

    // rings; a chunk of zeros (V of blocks a wave does not score, and the tails' operands)
    constexpr int ZERO = 2 * NS * PAIR;
    constexpr int ZLEN = TAIL || CACHE ? HALF + 256 : 0;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[ZERO + ZLEN];
    lds_u8* const lds = (lds_u8*)smem;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;

    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l32 = lane & 31;
    const int hi = lane >> 5;

    const int g = blockIdx.x;
    const int item = (g & 7) * a.per_xcd + (g >> 3);
    if (item >= a.n_items) return;
    const int T = a.T;
    const int n64 = (T + 63) >> 6;
    const int n_tile = (n64 + W - 1) / W;
    const int bh = item / n_tile;
    const int tile = item - bh * n_tile;
    const int qb = tile * W + w;
    const bool live = qb < n64;
    const size_t head_off = (size_t)bh * (size_t)T * D;
    const int row0 = qb * 64;
    const int nrow = live ? (T - row0 < 64 ? T - row0 : 64) : 0;

    // ---- per-lane offsets ---------------------------------------------------------------
    // DMA: instruction n of wave w fills 16-byte slots base_n + lane of a stage, row
    // r = slot / SLOTS, from head-dim chunk (slot % SLOTS) ^ swizzle(r) of key row r.
    // Unswizzled rows (72-wide) are contiguous: source and LDS offsets agree.  Of
    // swizzled ones an instruction covers rows 8 (nW + w) .. + 7, so source
    // offsets of one wave's instructions differ by a constant.
    auto dma_base = [&](int n) { return n < NFULL ? (n * W + w) * 1024 : (NFULL * W * 64 + w * REM) * 16; };
    int kdma = lane * 16, vdma = lane * 16;
    if (G::SWZ) {
        const int r = lane >> 3, s = lane & 7;
        kdma = r * ROWB + ((s ^ kswz<D>(r)) * 16);
        vdma = r * ROWB + ((s ^ vswz<D>(r)) * 16);
    }
    // K A-operand reads: row l32, head-dim chunk 2s + hi
    const int k_rd = l32 * ROWB + ((hi ^ kswz<D>(l32)) * 16);
    // V^T transpose reads, as in attn.hip
    int v_rd;
    {
        const int G4 = lane >> 4, L = lane & 15;
        const int r = 4 * hi + (L >> 2);
        const int d = 16 * (L & 1) + 8 * (G4 & 1) + 4 * ((L >> 1) & 1);
        v_rd = r * ROWB + (((d >> 3) ^ vswz<D>(r)) * 16) + (d & 7) * 2;
    }
    // the tail's: lane group g of 16 takes keys 16 (g & 1) + 4 (g >> 1) + (0 .. 3, 8 .. 11)
    int t_rd = 0;
    if (TAIL) {
        const int G4 = lane >> 4, L = lane & 15;
        t_rd = (16 * (G4 & 1) + 4 * (G4 >> 1) + (L >> 2)) * ROWB + (64 + 4 * (L & 1)) * 2;
    }
    const i32x4 k_rs = buffer_rsrc(a.k + head_off, T * D * 2);
    const i32x4 v_rs = buffer_rsrc(a.v + head_off, T * D * 2);

    // ---- queries ------------------------------------------------------------------------
    // Of a 72-wide head's last 8 dims, lanes of half 0 hold query tile 0's and lanes of
    // half 1 tile 1's: each tile's tail product has zeros in K for the other half.
    bf16x8 qop[2][DS], qtl = {};
    {
        const __amdgpu_buffer_rsrc_t q_rs = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(a.q + head_off + (size_t)row0 * D), (short)0, nrow * D * 2, 0x00020000);
        auto load = [&](int row, int ch) {
            return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(q_rs, row * (D * 2) + ch * 16, 0, 0));
        };
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
#pragma unroll
            for (int s = 0; s < DS; ++s) qop[qt][s] = load(qt * 32 + l32, 2 * s + hi);
        }
        if (TAIL) qtl = load(hi * 32 + l32, 8);
    }
    for (int i = threadIdx.x * 16; i < ZLEN; i += 64 * W * 16) *(lds_u32x4*)(lds + ZERO + i) = u32x4{};

    // ---- the walk: key blocks 0, 1, ..; a caching step scores those its mask drops --------
    // The first 64 entries of the wave's CSR row sit in one VGPR (lane i: entry i), so
    // that stepping through them costs no load in the walk.
    int kept = -1, k_beg = 0, n_kept = 0, k_i = 0, k_next = -1;
    auto entry = [&](int i) -> int {  // -1 past the row
        return i >= n_kept ? -1
                           : (i < 64 ? __builtin_amdgcn_readlane(kept, i) : ((csr_ptr)a.col_idx)[k_beg + i]);
    };
    if (CACHE && live) {
        const int mid = a.n_masks <= 1 ? 0 : (a.n_masks == a.heads ? bh % a.heads : bh);
        const csr_ptr rp = (csr_ptr)a.row_ptr + (size_t)mid * (n64 + 1);
        int b = rp[qb], e = rp[qb + 1];
        b = b < 0 ? 0 : (b > a.nnz ? a.nnz : b);
        e = e < b ? b : (e > a.nnz ? a.nnz : e);
        k_beg = b;
        n_kept = e - b;
        if (lane < n_kept) kept = a.col_idx[k_beg + lane];
        k_next = entry(0);
    }
    int nxt_blk = 0;
    auto gen = [&]() -> int {  // byte offset of the next block, with its flags
        const int c = nxt_blk++;
        if (c >= n64) return kOff | kEnd;
        int act = kAct;
        if (CACHE) {
            if (k_i < n_kept) {
                while (k_next < c && ++k_i < n_kept) k_next = entry(k_i);
                if (k_i < n_kept && k_next == c) {
                    act = 0;
                    k_next = entry(++k_i);
                }
            }
            if (!live) act = 0;
        }
        return c * BLK | act;
    };

    // Ring stage p holds the 64 K rows past block p's first 32 (its second half and block
    // p + 1's first half) and the V rows of block p: what the walk reads while it
    // scores block p.  Rows past T read as zeros.
    auto dma = [&](const i32x4& rs, int off, int dst) {
#pragma unroll
        for (int n = 0; n < NDMA; ++n) {
            if (n < NFULL || lane < REM)
                dma16(__builtin_amdgcn_readfirstlane(lds0 + dst + dma_base(n)), off + dma_base(n), rs);
        }
    };
    auto issue = [&](int dst, int x) {
        dma(k_rs, kdma + x + HALF, dst);
        dma(v_rs, vdma + x, NS * PAIR + dst);
    };
    auto barrier = [&]() {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // b0 is the block being scored, b1 the next one
    int b0 = gen();
    int b1 = gen();
    dma(k_rs, kdma - HALF, 2 * PAIR);  // block 0's first half, behind 32 rows of zeros
    issue(0, 0);
    issue(PAIR, BLK);
    wait_vm<2 * NDMA>();
    // Q has landed as well (it was issued first): no wait of the compiler's in the walk
#pragma unroll
    for (int s = 0; s < DS; ++s) asm volatile("" : "+v"(qop[0][s]), "+v"(qop[1][s]));
    if (TAIL) asm volatile("" : "+v"(qtl));
    barrier();

    const float c2 = a.scale_log2;
    f32x16 oacc[2][2];
    f32x4 tacc[2];  // tail of O^T for 16 queries: rows 0-7 tile 0's dims, 8-15 tile 1's
    float m_run[2], m_top[2], l_run[2];
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
        m_run[qt] = -1e30f;
        m_top[qt] = -INFINITY;
        l_run[qt] = 0.f;
        oacc[qt][0] = oacc[qt][1] = f32x16{};
        tacc[qt] = f32x4{};
    }
    uint32_t pk[2][8];  // bf16 probabilities of the chunk before
#pragma unroll
    for (int x = 0; x < 8; ++x) pk[0][x] = pk[1][x] = 0u;

    auto chunk_max = [&](const f32x16& sc) {
        float mx = fmaxf(fmaxf(sc[0], sc[1]), sc[2]);
#pragma unroll
        for (int x = 3; x < 15; x += 2) mx = fmaxf(fmaxf(mx, sc[x]), sc[x + 1]);
        mx = fmaxf(mx, sc[15]);
        return pair_max(mx);
    };
    const int full_lim = (T - 32) * (D * 2);
    auto mask = [&](int cb, f32x16& sc) {  // cb: byte offset of the chunk
        const int lim = T - cb / (D * 2) - 4 * hi;
#pragma unroll
        for (int x = 0; x < 16; ++x) {
            if (8 * (x >> 2) + (x & 3) >= lim) sc[x] = -INFINITY;
        }
    };
    auto pk_op = [&](const uint32_t (&p)[8], int ks) {
        return __builtin_bit_cast(bf16x8, u32x4{p[4 * ks], p[4 * ks + 1], p[4 * ks + 2], p[4 * ks + 3]});
    };
    // LDS addresses: of swizzled rows, chunk 2s + hi sits at the first one's slot
    // with bits 1.. flipped by s, and V's second 32 head dims at slot ^ 4.
    auto v_read = [&](int vb, int vo, int dt, int ks) -> bf16x8 {
        const lds_u8* Vs = lds + (G::SWZ ? (vb ^ (64 * dt)) + vo : vb + vo + 64 * dt) + 16 * ks * ROWB;
        const bf16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)Vs);
        const bf16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(Vs + 8 * ROWB));
        return __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    // the tail's V^T operand for query tile Q: 8 dims at its rows, zeros at the other's
    auto t_read = [&](int vo, int Q) -> bf16x8 {
        const lds_u8* Vs = lds + (((lane >> 1) & 1) == Q ? vo + t_rd : ZERO);
        const bf16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)Vs);
        const bf16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(Vs + 8 * ROWB));
        return __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    auto k_read = [&](int kb, int ko, int s) -> bf16x8 {
        return *(const lds_bf16x8*)(lds + (G::SWZ ? (kb ^ (32 * s)) + ko : kb + ko + 32 * s));
    };
    // tail K operand of query tile Q: the row's last chunk in lanes of half Q, else zeros
    auto k_tail = [&](int kb, int ko, int Q) -> bf16x8 {
        return *(const lds_bf16x8*)(lds + (hi == Q ? kb + ko + 128 - 16 * Q : ZERO));
    };
    // hides a lane constant's value, so that what derives from it is formed anew
    // (one v_xad_u32 per read) instead of held in registers throughout the walk
    auto fresh = [](int x) {
        asm volatile("" : "+v"(x));
        return x;
    };
#define RT_FENCE __builtin_amdgcn_sched_barrier(0)
    auto mma = [](const bf16x8& x, const bf16x8& y, const f32x16& z) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, z, 0, 0, 0);
    };
    // The 8-dim tails of O^T: a 16x16x32 product per tile and 16 queries, both tiles
    // into one accumulator.  Swapping the odd 16-lane rows of the first 8 keys'
    // registers with the even rows of the others' turns the two 16-key operands
    // of a 32-query tile into the two 32-key operands of its 16-query halves.
    auto tail_mma = [&](const bf16x8& x, const uint32_t (&p)[8]) {
        uint32_t y[8];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            auto s = __builtin_amdgcn_permlane16_swap(p[r], p[4 + r], false, false);
            y[r] = s[0];
            y[4 + r] = s[1];
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) tacc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, pk_op(y, h), tacc[h], 0, 0, 0);
    };
    auto bf16_sum = [&](const uint32_t (&p)[8]) -> float {
        const bf16x2 one2 = {(__bf16)1.0f, (__bf16)1.0f};
        float a0 = 0.f, a1 = 0.f;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            a0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, p[x]), one2, a0, false);
            a1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, p[4 + x]), one2, a1, false);
        }
        return a0 + a1;
    };
    // per-query values of the tiles as the tail accumulators' lanes hold them: lane l has
    // query 16 h + l % 16 of tile l / 32, dims 64 + 4 (l / 16 % 2) ..
    auto tail_bcast = [&](float x0, float x1, int h) {
        const int src = (16 * h + (lane & 15)) << 2;
        const int y0 = __builtin_amdgcn_ds_bpermute(src, __float_as_uint(x0));
        const int y1 = __builtin_amdgcn_ds_bpermute(src, __float_as_uint(x1));
        return __uint_as_float(hi ? y1 : y0);
    };

    f32x16 s0, s1;  // scores of the two query tiles
    bf16x8 kop[DS];  // K operands: chunk t (tile 0 has used it) or t + 1
    bf16x8 vop[4];   // V^T operands (dt, ks) of the chunk before, or of chunk t
    bf16x8 kt1 = {}, vt1 = {};  // the tails of both, for query tile 1
    auto scores = [&](int Q, int ko, int cb) {
        f32x16 x = {};
#pragma unroll
        for (int s = 0; s < DS; ++s) x = mma(kop[s], qop[Q][s], x);
        if (TAIL) x = mma(k_tail(k_rd, ko, Q), qtl, x);
        if (cb > full_lim) mask(cb, x);
        return x;
    };
    auto k_fetch = [&](int ko) {
#pragma unroll
        for (int s = 0; s < DS; ++s) kop[s] = k_read(k_rd, ko, s);
        if (TAIL) kt1 = k_tail(k_rd, ko, 1);
    };
    k_fetch(2 * PAIR + HALF);
    s0 = scores(0, 2 * PAIR + HALF, b0 & ~kFlags);
    // Both tiles start from their first chunk's max.  A caching step starts from the max
    // m of the kept keys, which the sparse walk before it left with their exp-sum l
    // against it in the first 8 bytes of the residual row.
    const bool has_in = CACHE && n_kept > 0;
    auto kept_stat = [&](int qt, int i) {
        const int row = row0 + qt * 32 + l32;
        return row < T ? reinterpret_cast<const float*>(a.resid_out + head_off + (size_t)row * D)[i] : 0.f;
    };
    if (has_in) {
        m_run[0] = fmaxf(kept_stat(0, 0), -1e30f);
        m_run[1] = fmaxf(kept_stat(1, 0), -1e30f);
        if (STATS) {
            m_top[0] = m_run[0];
            m_top[1] = m_run[1];
        }
    } else {
        m_run[0] = fmaxf(chunk_max(s0), -1e30f);
        m_run[1] = fmaxf(chunk_max(scores(1, 2 * PAIR + HALF, b0 & ~kFlags)), -1e30f);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) vop[k] = bf16x8{};
    barrier();
    issue(2 * PAIR, 2 * BLK);
    int ahead = 3 * BLK;  // the next block to load

    int st = 0;  // LDS offset of the ring stage in use
    // The next stage has landed for every wave and this one has been read by
    // every wave; its refill goes out.
    auto turn = [&]() {
        wait_vm<2 * NDMA>();
        barrier();
        issue(st, ahead);
        ahead += BLK;
        b0 = b1;
        b1 = gen();
        st = st == 2 * PAIR ? 0 : st + PAIR;
    };

    // One phase: the softmax of query tile Q's chunk t runs on the VALU while the
    // matrix cores form the other tile's next scores and its last P V:
    //   Q = 0: S_1(t) = K(t) Q_1,       O_1 += V(t-1) P_1(t-1); the operands of
    //          chunks t+1 (K, at LDS offset ko) and t (V, at vo) are read behind
    //          their last use
    //   Q = 1: S_0(t+1) = K(t+1) Q_0,   O_0 += V(t) P_0(t); the tails' operands
    //          of both tiles are read
    // nb: byte offset of the chunk the other tile scores.  Where the wave does not
    // score the block (!on), its probabilities are exp2(-inf) = 0; scores of
    // non-finite keys, whose probabilities are not, end up in the rare branch.
    auto phase = [&](auto tile, bool on, int nb, int ko, int vo) {
        constexpr int Q = decltype(tile)::value, R = 1 - Q;
        f32x16& sc = Q ? s1 : s0;
        f32x16& sn = Q ? s0 : s1;
        const float mc = on ? m_run[Q] * c2 : INFINITY;
        const int kb = Q == 0 || TAIL ? fresh(k_rd) : 0, vb = Q == 0 ? fresh(v_rd) : 0;
        bf16x8 kt = kt1, vt = vt1;
        if (TAIL && Q == 1) {
            kt = k_tail(kb, ko, 0);
            vt = t_read(vo, 0);
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
            if (!BF16_SUM) {
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
            sn = mma(kop[k], qop[R][k], k == 0 ? f32x16{} : sn);
            RT_FENCE;  // reads stay behind the operand's last use: no second set of registers
            if (Q == 0) kop[k] = k_read(kb, ko, k);
            slot(2 * k);
            RT_FENCE;
            oacc[R][k & 1] = mma(vop[k], pk_op(pk[R], k >> 1), oacc[R][k & 1]);
            RT_FENCE;
            if (Q == 0) vop[k] = v_read(vb, vo, k & 1, k >> 1);
            slot(2 * k + 1);
        }
        RT_FENCE;
        keep(14);
        // the max is taken here, not moved behind the last read of the scores
        if (STATS) asm volatile("" : "+v"(m_top[Q]));
        if (TAIL) {
            sn = mma(kt, qtl, sn);
            tail_mma(vt, pk[R]);
            RT_FENCE;
            if (Q == 1) {
                kt1 = k_tail(kb, ko, 1);
                vt1 = t_read(vo, 1);
            }
        }
        float ls = BF16_SUM ? bf16_sum(pk[Q]) : sa + sb;
        if (__builtin_amdgcn_ballot_w64(!(ls < kJump))) {
            if (!on) {
#pragma unroll
                for (int x = 0; x < 8; ++x) pk[Q][x] = 0u;
                ls = 0.f;
            } else {
                // A probability reached 2^64: O and l move to the chunk's max.
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
                    pk[Q][x / 2] = pack_bf16(e[0], e[1]);
                    pk[Q][x / 2 + 1] = pack_bf16(e[2], e[3]);
                    part = (e[0] + e[1]) + (e[2] + e[3]);
                    if (x == 0) sa = part;
                    if (x == 4) sb = part;
                    if (x == 8) sa += part;
                    if (x == 12) sb += part;
                }
                RT_FENCE;
                ls = sa + sb;
                if (BF16_SUM) ls = bf16_sum(pk[Q]);
            }
        }
        l_run[Q] += ls;
        if (nb > full_lim) mask(nb, sn);
    };

    auto pv1 = [&]() {  // the pending P V of tile 1
#pragma unroll
        for (int k = 0; k < 4; ++k) oacc[1][k & 1] = mma(vop[k], pk_op(pk[1], k >> 1), oacc[1][k & 1]);
        if (TAIL) tail_mma(vt1, pk[1]);
    };
    using t0 = std::integral_constant<int, 0>;
    using t1 = std::integral_constant<int, 1>;
    while (!(b0 & kEnd)) {
        const int cur = b0 & ~kFlags;
        const bool on = !CACHE || (b0 & kAct);
        const int va = on ? NS * PAIR + st : ZERO, vb = on ? NS * PAIR + st + HALF : ZERO;
        phase(t0{}, on, cur, st, va);
        phase(t1{}, on, cur + HALF, st, va);
        phase(t0{}, on, cur + HALF, st + HALF, vb);
        phase(t1{}, on, b1 & ~kFlags, st + HALF, vb);
        turn();
    }
    pv1();
    wait_vm<0>();  // nothing may land in LDS after the workgroup has ended
    if (!live) return;

    // ---- epilogue -------------------------------------------------------------------------
    // lane (hi, l32) holds 16 head dims 32 dt + 16 hi .. of query l32 per tile and dt,
    // and in the tail lanes 0 .. 31 hold 4 head dims of query 16 h + lane % 16
    const bool split = CACHE && n_kept < n64;
    float inv2[2], rho2[2];
    // four output values of one row from accumulators, 1 / l, rho and O_s
    auto out4 = [&](const float* acc, float iv, float rh, const uint32_t* os, uint32_t* o2, uint32_t* r2) {
        float r[4], of[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float x = acc[e] * iv;
            if (CACHE) {
                const float osv = (e & 1) ? hi_f(os[e >> 1]) : lo_f(os[e >> 1]);
                r[e] = split ? (a.rho_out ? x : __builtin_fmaf(rh - 1.0f, osv, x)) : 0.f;
                of[e] = __builtin_fmaf(rh, osv, x);
            } else {
                of[e] = x;
            }
        }
        o2[0] = pack_bf16(of[0], of[1]);
        o2[1] = pack_bf16(of[2], of[3]);
        if (CACHE) {
            r2[0] = pack_bf16(r[0], r[1]);
            r2[1] = pack_bf16(r[2], r[3]);
        }
    };
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
        const int row = row0 + qt * 32 + l32;
        const float ls = pair_sum(l_run[qt]);
        float li = 0.f;
        if (has_in) li = kept_stat(qt, 1) * __builtin_amdgcn_exp2f((kept_stat(qt, 0) - m_run[qt]) * c2);
        const float lf = CACHE ? li + ls : ls;
        const float inv = 1.0f / lf;
        const float rho = split ? li / lf : 1.0f;  // exactly 1 when every block is kept
        inv2[qt] = inv;
        rho2[qt] = rho;
        if (STATS) m_top[qt] = pair_max(m_top[qt]);
        if (hi == 0 && row < T) {
            const size_t si = (size_t)bh * T + row;
            if (CACHE && a.rho_out) a.rho_out[si] = rho;
            if (STATS) {
                if (a.row_max) a.row_max[si] = m_top[qt] * a.scale_nat;
                if (a.row_sum) a.row_sum[si] = lf * __builtin_amdgcn_exp2f((m_run[qt] - m_top[qt]) * c2);
            }
        }
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (row < T) {
                    const size_t off = head_off + (size_t)row * D + 8 * (4 * dt + 2 * hi + u);
                    u32x4 os = {};
                    if (has_in) os = *reinterpret_cast<const u32x4*>(a.o + off);
                    float acc[8];
                    uint32_t o[4], r[4], osw[4] = {os[0], os[1], os[2], os[3]};
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[e] = oacc[qt][dt][8 * u + e];
                    out4(acc, inv, rho, osw, o, r);
                    out4(acc + 4, inv, rho, osw + 2, o + 2, r + 2);
                    if (CACHE)
                        *reinterpret_cast<u32x4*>(a.resid_out + off) = u32x4{r[0], r[1], r[2], r[3]};
                    *reinterpret_cast<u32x4*>(a.o + off) = u32x4{o[0], o[1], o[2], o[3]};
                }
            }
        }
    }
    if (TAIL) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float iv = tail_bcast(inv2[0], inv2[1], h), rh = tail_bcast(rho2[0], rho2[1], h);
            const int row = row0 + 32 * hi + 16 * h + (lane & 15);
            if (row < T) {
                const size_t off = head_off + (size_t)row * D + 64 + 4 * ((lane >> 4) & 1);
                uint32_t os[2] = {0u, 0u}, o[2], r[2];
                if (has_in) {
                    os[0] = reinterpret_cast<const uint32_t*>(a.o + off)[0];
                    os[1] = reinterpret_cast<const uint32_t*>(a.o + off)[1];
                }
                const float acc[4] = {tacc[h][0], tacc[h][1], tacc[h][2], tacc[h][3]};
                out4(acc, iv, rh, os, o, r);
                if (CACHE) {
                    reinterpret_cast<uint32_t*>(a.resid_out + off)[0] = r[0];
                    reinterpret_cast<uint32_t*>(a.resid_out + off)[1] = r[1];
                }
                reinterpret_cast<uint32_t*>(a.o + off)[0] = o[0];
                reinterpret_cast<uint32_t*>(a.o + off)[1] = o[1];
            }
        }
    }
}

template <int D, int W, bool STATS, bool CACHE>
hipError_t launch_one(AttnArgs a, hipStream_t stream) {
    const int64_t n64 = ((int64_t)a.T + 63) / 64;
    const int64_t n_bh = a.n_items / a.n_blk;
    a.n_items = (int32_t)(n_bh * ((n64 + W - 1) / W));
    a.per_xcd = (a.n_items + 7) / 8;
    hipLaunchKernelGGL((attn_dense<D, W, STATS, CACHE>), dim3(8 * a.per_xcd), dim3(64 * W), 0, stream, a);
    return hipGetLastError();
}

template <int D, int W>
hipError_t launch_dw(const AttnArgs& a, bool cache, hipStream_t stream) {
    const bool stats = a.row_max != nullptr || a.row_sum != nullptr;
    if (cache) return stats ? launch_one<D, W, true, true>(a, stream) : launch_one<D, W, false, true>(a, stream);
    return stats ? launch_one<D, W, true, false>(a, stream) : launch_one<D, W, false, false>(a, stream);
}

}  // namespace

hipError_t launch_attention_dense(const AttnArgs& a, int D, bool cache, hipStream_t stream) {
    return D == 64 ? launch_dw<64, 4>(a, cache, stream) : launch_dw<72, 4>(a, cache, stream);
}

}  // namespace rt
