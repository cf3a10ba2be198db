// Attention over every key block of a head (gfx950, CDNA4): dense attention with
// row statistics, and the dropped keys of a caching step.
//
//   rt_attn_full   Eq.1 with the Eq.4 denominator
//   rt_attn_cache  App. A.3: after the sparse walk (attn.hip) has left O_s and the kept
//                  keys' statistics, the other keys, then O_full, rho (Eq.8), R (Eq.10)
//
// Every query block of a head reads the whole K and V of that head, so a
// workgroup of four waves (64 query rows each, two waves per SIMD) shares one K and one V
// ring in LDS, three 64-key stages each, filled by all its waves with
// buffer_load ... lds; one barrier per 64 keys, two stages of lead.  With a ring
// per wave the chunk loads kept the vector-memory path 84-92 % busy.
//
// The walk itself is attn_tiles.h's.
//
// Bound by the vector unit's issue slots (an MFMA takes about 8 of its cycles
// beside its own; 131 instructions per 32-key chunk and 64 rows) and by power:
// with zero queries, keys and values the same instructions run 21 % faster, as a
// large bf16 product does.  Measured, before -> now: PixArt-Sigma-2K dense with
// statistics (32 heads, 16384 tokens, D = 72) 3925 -> 2534 us (0.98 PFLOP/s of real
// dims), CogVideoX caching step (60 heads, 17776 tokens, D = 64) 5511 -> 4918 us, of
// which the sparse walk is 225; PixArt-Sigma-1024 caching step 289 -> 192 us.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_tiles.h"
#include "kernels.h"

namespace rt {
namespace {

constexpr int kOff = 0x60000000;  // buffer offset past every record, also after small additions
constexpr int kAct = 1;           // flags in the low bits of a block offset: this wave scores the block
constexpr int kEnd = 2;           // past the last block
constexpr int kFlags = 3;
constexpr int W = 4;              // waves of a workgroup: one to each SIMD of a CU

template <int D, bool STATS, bool CACHE>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_dense(AttnArgs a) {
    using G = Geo<D>;
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
    static_assert(ROWB == 2 * D, "rows are unpadded");

    // rings; a chunk of zeros (V of blocks a wave does not score, and the tails' operands)
    constexpr int ZERO = 2 * NS * PAIR;
    constexpr int ZLEN = TAIL || CACHE ? HALF + 256 : 0;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[ZERO + ZLEN];
    lds_u8* const lds = (lds_u8*)smem;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;

    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

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
    const i32x4 k_rs = buffer_rsrc(a.k + head_off, T * D * 2);
    const i32x4 v_rs = buffer_rsrc(a.v + head_off, T * D * 2);

    Tiles<D, STATS, STATS || CACHE, ZERO> t;
    t.init(lds, T, a.scale_log2);
    t.load_q(a.q + head_off + (size_t)row0 * D, nrow);
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
    t.settle_q();  // issued first
    barrier();
    t.first_chunk(2 * PAIR + HALF, b0 & ~kFlags);
    // Both tiles start from their first chunk's max.  A caching step goes on from the running
    // max of the sparse walk before it, which left it with the kept keys' exp-sum against it
    // in the first 8 bytes of the residual row: the probabilities round as in one walk.
    const bool has_in = CACHE && n_kept > 0;
    auto kept_stat = [&](int qt, int i) {
        const int row = row0 + qt * 32 + t.l32;
        return row < T ? reinterpret_cast<const float*>(a.resid_out + head_off + (size_t)row * D)[i] : 0.f;
    };
    if (has_in) {
        t.m_run[0] = kept_stat(0, 0);
        t.m_run[1] = kept_stat(1, 0);
    } else {
        t.first_max(2 * PAIR + HALF, b0 & ~kFlags);
    }
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

    while (!(b0 & kEnd)) {
        const int cur = b0 & ~kFlags;
        const bool on = !CACHE || (b0 & kAct);
        const int va = on ? NS * PAIR + st : ZERO, vb = on ? NS * PAIR + st + HALF : ZERO;
        t.template phase<0>(on, cur, st, va);
        t.template phase<1>(on, cur + HALF, st, va);
        t.template phase<0>(on, cur + HALF, st + HALF, vb);
        t.template phase<1>(on, b1 & ~kFlags, st + HALF, vb);
        turn();
    }
    t.pv1();
    wait_vm<0>();  // nothing may land in LDS after the workgroup has ended
    if (!live) return;

    // ---- epilogue -------------------------------------------------------------------------
    t.lanes();
    // lane (hi, l32) holds 16 head dims 32 dt + 16 hi .. of query l32 per tile and dt,
    // and in the tail 4 head dims of query 16 h + lane % 16 of tile hi
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
        const int row = row0 + qt * 32 + t.l32;
        const float ls = pair_sum(t.l_run[qt]);
        float li = 0.f;
        if (has_in) li = kept_stat(qt, 1) * __builtin_amdgcn_exp2f((kept_stat(qt, 0) - t.m_run[qt]) * a.scale_log2);
        const float lf = CACHE ? li + ls : ls;
        const float inv = 1.0f / lf;
        const float rho = split ? li / lf : 1.0f;  // exactly 1 when every block is kept
        inv2[qt] = inv;
        rho2[qt] = rho;
        if (STATS) t.m_top[qt] = pair_max(t.m_top[qt]);
        if (t.hi == 0 && row < T) {
            const size_t si = (size_t)bh * T + row;
            if (CACHE && a.rho_out) a.rho_out[si] = rho;
            if (STATS) {
                if (a.row_max) a.row_max[si] = t.m_top[qt] * a.scale_nat;
                if (a.row_sum) a.row_sum[si] = lf * __builtin_amdgcn_exp2f((t.m_run[qt] - t.m_top[qt]) * a.scale_log2);
            }
        }
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (row < T) {
                    const size_t off = head_off + (size_t)row * D + 8 * (4 * dt + 2 * t.hi + u);
                    u32x4 os = {};
                    if (has_in) os = *reinterpret_cast<const u32x4*>(a.o + off);
                    float acc[8];
                    uint32_t o[4], r[4], osw[4] = {os[0], os[1], os[2], os[3]};
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[e] = t.oacc[qt][dt][8 * u + e];
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
            const float iv = t.tail_bcast(inv2[0], inv2[1], h), rh = t.tail_bcast(rho2[0], rho2[1], h);
            const int row = row0 + 32 * t.hi + 16 * h + (t.lane & 15);
            if (row < T) {
                const size_t off = head_off + (size_t)row * D + 64 + 4 * ((t.lane >> 4) & 1);
                uint32_t os[2] = {0u, 0u}, o[2], r[2];
                if (has_in) {
                    os[0] = reinterpret_cast<const uint32_t*>(a.o + off)[0];
                    os[1] = reinterpret_cast<const uint32_t*>(a.o + off)[1];
                }
                const float acc[4] = {t.tacc[h][0], t.tacc[h][1], t.tacc[h][2], t.tacc[h][3]};
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

template <int D, bool STATS, bool CACHE>
hipError_t launch_one(AttnArgs a, hipStream_t stream) {
    const int64_t n64 = ((int64_t)a.T + 63) / 64;
    const int64_t n_bh = a.n_items / a.n_blk;
    a.n_items = (int32_t)(n_bh * ((n64 + W - 1) / W));
    a.per_xcd = (a.n_items + 7) / 8;
    hipLaunchKernelGGL((attn_dense<D, STATS, CACHE>), dim3(8 * a.per_xcd), dim3(64 * W), 0, stream, a);
    return hipGetLastError();
}

template <int D>
hipError_t launch_d(const AttnArgs& a, bool cache, hipStream_t stream) {
    const bool stats = a.row_max != nullptr || a.row_sum != nullptr;
    if (cache) return stats ? launch_one<D, true, true>(a, stream) : launch_one<D, false, true>(a, stream);
    return stats ? launch_one<D, true, false>(a, stream) : launch_one<D, false, false>(a, stream);
}

}  // namespace

hipError_t launch_attention_dense(const AttnArgs& a, int D, bool cache, hipStream_t stream) {
    return D == 64 ? launch_d<64>(a, cache, stream) : launch_d<72>(a, cache, stream);
}

}  // namespace rt
