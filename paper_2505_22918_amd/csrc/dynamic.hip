// Dynamic block mask (gfx950): the kept key blocks chosen at run time from the
// step's own Q and K, one mask per (batch, head), in the stacked CSR layout the
// attention kernels take (n_masks = B*H).
//
// The paper keeps a static mask and names run-time masks as future work,
// adapted to attention statistics or token importance (Sec.6, App. A.2); the
// dynamic methods it cites pool Q K^T into blocks and keep the top-scoring
// blocks (Sec.2).  The rule built here, per (batch, head) and query block qb:
//   score(qb, kb) = sum_d Qsum_qb[d] * Kmean_kb[d]
// with Qsum the fp32 sum of qb's rows (one addition per row, ascending), Kmean
// the fp32 sum of kb's rows (same order) divided by its token count, and the
// dot product accumulated in fp32 over ascending d by fused multiply-adds (one
// rounding a term).  qb keeps itself (Eq.5 needs a non-empty kept set) and
// the keep - 1 best other blocks (higher score first, ties to the lower index,
// a NaN score ranked last); rows are stored ascending.  Every fp32 operation is
// fixed, so the choice is reproducible bit for bit.
//
//   pool_kernel    one workgroup per (batch, head, block): the block's Q and K
//                  rows are staged in LDS with 16-byte loads, then lane d < D
//                  sums Q column d over the rows in ascending order and lane
//                  128 + d does the same for K and divides by the token count.
//                  Writes qsum [B*H][n_blk][D] and, per 64-block tile, kmean as
//                  [D / 4][blocks of the tile][4], the order a wave reads it in.
//                  Bound by HBM: CogVideoX shape 43 us for 273 MB.
//   select_kernel  one workgroup per (batch, head) and a few query blocks, a wave per
//                  tile of 64 key blocks (up to 8 waves) and two rows per wave (one where
//                  a row has more than 512 blocks) while the scores fit 40 KB of
//                  LDS.  A lane keeps its key block's mean in
//                  registers and takes the query values from scalar registers, so
//                  that a term of a score is one vector instruction and no LDS read.
//                  Then one wave per row selects: up to 512 blocks with the keys in
//                  registers, the threshold found bit by bit with ballots (ends when
//                  exactly as many keys are above it as are to be kept); longer rows by
//                  four radix passes over LDS histograms, whose cost per bit does
//                  not grow with the registers.  The kept blocks go out in
//                  ascending order at the row's closed-form offset (every row
//                  keeps exactly min(keep, n_blk)).
// Bound by the latency of the scalar loads and the L2 reads of the key means.  CogVideoX
// shape (60 heads, 278 blocks, keep 9), before -> now: selection 65 -> 35 us (10 of them
// the selection proper), the build 102-109 -> 84 us; one and four rows per wave 37 and
// 41 us; key means read row by row instead of by tiles 40 us.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>

#include "kernels.h"

#pragma clang fp contract(off)

namespace rt {
namespace {

constexpr int kPoolThreads = 256;
constexpr int kSelWaves = 8;             // most waves of a select workgroup
constexpr int kSelRegs = 8;              // up to 64 times as many blocks are selected in registers
constexpr int kSelScoreBytes = 40 << 10; // LDS for the scores of one workgroup
constexpr int kMaxD = 72;
constexpr int kPoolRows = 64;                      // largest block

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) float* float_cptr;

__global__ __launch_bounds__(kPoolThreads) void pool_kernel(const uint16_t* __restrict__ q,
                                                            const uint16_t* __restrict__ k, int T, int D,
                                                            int block, int n_blk, float* __restrict__ qsum,
                                                            float* __restrict__ kmean) {
    // the block's rows of Q, then of K, row-major as in HBM (2D bytes per row)
    __shared__ __attribute__((aligned(16))) uint16_t tile[2][kPoolRows * kMaxD];
    const int bh = blockIdx.x / n_blk;
    const int b = blockIdx.x - bh * n_blk;
    const int t = threadIdx.x;
    const int r0 = b * block;
    const int cnt = min(block, T - r0);
    const size_t base = ((size_t)bh * T + r0) * D;
    // 16-byte pieces of the block's rows: cnt * D / 8 per tensor (D is a multiple of 8)
    const int n16 = cnt * D / 8;
    const u32x4* qs = reinterpret_cast<const u32x4*>(q + base);
    const u32x4* ks = reinterpret_cast<const u32x4*>(k + base);
    u32x4* tq = reinterpret_cast<u32x4*>(tile[0]);
    u32x4* tk = reinterpret_cast<u32x4*>(tile[1]);
    for (int i = t; i < n16; i += kPoolThreads) {
        tq[i] = qs[i];
        tk[i] = ks[i];
    }
    __syncthreads();
    const bool is_q = t < 128;
    const int d = is_q ? t : t - 128;
    if (d >= D) return;
    const uint16_t* col = tile[is_q ? 0 : 1] + d;
    float acc = 0.0f;
    for (int r = 0; r < cnt; ++r) acc = __fadd_rn(acc, bf16_to_f32(col[r * D]));
    if (is_q) {
        qsum[((size_t)bh * n_blk + b) * D + d] = acc;
    } else {
        const int t0 = b & ~63;
        const int nt = n_blk - t0 < 64 ? n_blk - t0 : 64;
        kmean[((size_t)bh * n_blk + t0) * D + ((d >> 2) * nt + (b - t0)) * 4 + (d & 3)] = __fdiv_rn(acc, (float)cnt);
    }
}

// Selection order as one unsigned key, larger = better: a NaN score counts as
// -inf and -0 as +0 (so keys are equal exactly when the fp32 scores compare
// equal), and the float's bits are mapped so that unsigned order is numeric
// order.  Equal keys go to the lower block index.
__device__ __forceinline__ uint32_t order_key(float x) {
    if (x != x) x = -INFINITY;
    if (x == 0.0f) x = 0.0f;
    const uint32_t u = __float_as_uint(x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Number of lanes below this one whose bit is set in the wave mask m.
__device__ __forceinline__ int lanes_below(unsigned long long m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Orders the wave's LDS accesses before and after this point (one wave only:
// LDS executes a wave's instructions in issue order).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Scores of the key blocks t0 + lane against `rows` pooled queries, into sc[row][kb].
template <int D>
__device__ __forceinline__ void score_tile(const float* __restrict__ qrow, const float* __restrict__ kh, int t0,
                                           int n_blk, int rows, float* sc, int lane) {
    float k[D];
    const int nt = n_blk - t0 < 64 ? n_blk - t0 : 64;
    const int kb = t0 + lane;
    const u32x4* src = reinterpret_cast<const u32x4*>(kh + (size_t)t0 * D) + (lane < nt ? lane : nt - 1);
#pragma unroll
    for (int i = 0; i < D / 4; ++i) {
        const u32x4 x = src[i * nt];
#pragma unroll
        for (int e = 0; e < 4; ++e) k[4 * i + e] = __uint_as_float(x[e]);
    }
    const float_cptr q = (float_cptr)qrow;
    for (int r = 0; r < rows; r += 2) {  // two rows at a time: two chains of sums
        const int r1 = r + 1 < rows ? r + 1 : r;
        float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            s0 = __builtin_fmaf(q[r * D + d], k[d], s0);
            s1 = __builtin_fmaf(q[r1 * D + d], k[d], s1);
        }
        if (kb < n_blk) {
            sc[r * n_blk + kb] = s0;
            sc[r1 * n_blk + kb] = s1;
        }
    }
}

// The keep - 1 best blocks other than the diagonal, by the value of their keys: thr, the
// key of the worst of them, and how many blocks holding exactly thr are kept.
struct Cut {
    uint32_t thr;
    int rem;
};

// Up to 64 N candidates, key u[i] of block lane + 64 i in registers (0, below every
// score's key, where there is none): thr bit by bit from the top, counting the keys
// at or above it by ballots, until exactly `need` are.
template <int N>
__device__ __forceinline__ Cut cut_in_registers(const uint32_t (&u)[N], int need) {
    uint32_t thr = 0;
    for (uint32_t bit = 0x80000000u; bit; bit >>= 1) {
        int cnt = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) cnt += __popcll(__ballot(u[i] >= (thr | bit)));
        if (cnt >= need) thr |= bit;
        if (cnt == need) break;
    }
    int above = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) above += __popcll(__ballot(u[i] > thr));
    return {thr, need - above};
}

// Any number of candidates, scores in LDS: radix selection, four passes of 8-bit digits
// from the top over a wave's histogram.
__device__ __forceinline__ Cut cut_by_radix(const float* row, int n_blk, int qb, int need, int* hw, int lane) {
    const int n_round = (n_blk + 63) / 64;
    uint32_t thr = 0, thr_mask = 0;  // digits of the threshold found so far
    int rem = need;                   // blocks still to keep at the threshold
    for (int shift = 24; shift >= 0; shift -= 8) {
#pragma unroll
        for (int j = 0; j < 4; ++j) hw[4 * lane + j] = 0;
        wave_lds_sync();
        for (int i = 0; i < n_round; ++i) {
            const int c = lane + 64 * i;
            if (c < n_blk && c != qb) {
                const uint32_t key = order_key(row[c]);
                if ((key & thr_mask) == thr) atomicAdd(&hw[(key >> shift) & 255u], 1);
            }
        }
        wave_lds_sync();
        // lane L holds bins 4L .. 4L+3; S(t) counts the blocks with digit >= t
        // and the threshold's digit is the t with S(t+1) < rem <= S(t)
        int h[4], sum = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            h[j] = hw[4 * lane + j];
            sum += h[j];
        }
        int incl = sum;  // inclusive sum over lanes 0 .. lane
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(incl, d, 64);
            if (lane >= d) incl += y;
        }
        const int tot = __shfl(incl, 63, 64);
        int s_t = tot - incl;  // bins above this lane's four
        int dig = -1, nrem = 0;
#pragma unroll
        for (int j = 3; j >= 0; --j) {
            s_t += h[j];
            if (h[j] > 0 && s_t >= rem && s_t - h[j] < rem) {
                dig = 4 * lane + j;
                nrem = rem - (s_t - h[j]);
            }
        }
        const unsigned long long found = __ballot(dig >= 0);
        const int src = __builtin_ctzll(found);  // exactly one lane finds it
        thr |= (uint32_t)__shfl(dig, src, 64) << shift;
        thr_mask |= 255u << shift;
        rem = __shfl(nrem, src, 64);
    }
    return {thr, rem};
}

// N: 64-block tiles of a row selected in registers, 0 for any number by radix passes.
// n_wave, the waves of the workgroup, is an argument: blockDim would bring the hidden
// kernel arguments in, whose filling costs the host 0.4 us a launch.
template <int D, int N>
__global__ __launch_bounds__(64 * kSelWaves) void select_kernel(const float* __restrict__ qsum,
                                                                const float* __restrict__ kmean, int n_blk, int keep,
                                                                int rows, int n_wave, int32_t* __restrict__ row_ptr,
                                                                int32_t* __restrict__ col_idx) {
    // scores of the workgroup's rows: rows x n_blk floats, then (radix) the waves' histograms
    extern __shared__ float sc[];
    const int n_grp = (n_blk + rows - 1) / rows;
    const int bh = blockIdx.x / n_grp;
    const int qb0 = (blockIdx.x - bh * n_grp) * rows;
    const int n_row = n_blk - qb0 < rows ? n_blk - qb0 : rows;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kk = keep < n_blk ? keep : n_blk;
    const int need = kk - 1;  // other blocks to keep, < n_blk
    const float* kh = kmean + (size_t)bh * n_blk * D;
    const float* qrow = qsum + ((size_t)bh * n_blk + qb0) * D;
    for (int t = w; t * 64 < n_blk; t += n_wave) score_tile<D>(qrow, kh, t * 64, n_blk, n_row, sc, lane);
    __syncthreads();
    // one wave per row
    for (int r = w; r < n_row; r += n_wave) {
        const int qb = qb0 + r;
        const float* row = sc + r * n_blk;
        const size_t row_off = ((size_t)bh * n_blk + qb) * kk;
        int n_tie = 0, n_out = 0;
        // kept blocks in ascending order, ties at the threshold to the lowest indices
        auto emit = [&](int c, uint32_t key, const Cut& cut) {
            bool kept = false, tie = false;
            if (c < n_blk) {
                if (c == qb || need >= n_blk - 1) {
                    kept = true;
                } else if (need > 0) {
                    tie = key == cut.thr;
                    kept = key > cut.thr;
                }
            }
            const unsigned long long tm = __ballot(tie);
            if (tie) kept = n_tie + lanes_below(tm) < cut.rem;
            n_tie += __popcll(tm);
            const unsigned long long km = __ballot(kept);
            const int pos = n_out + lanes_below(km);
            if (kept && pos < kk) col_idx[row_off + pos] = c;  // exactly kk kept (total order)
            n_out += __popcll(km);
        };
        const bool choose = need > 0 && need < n_blk - 1;
        Cut cut = {0u, 0};
        if constexpr (N > 0) {
            uint32_t u[N];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int c = lane + 64 * i;
                u[i] = c < n_blk && c != qb ? order_key(row[c]) : 0u;
            }
            if (choose) cut = cut_in_registers(u, need);
#pragma unroll
            for (int i = 0; i < N; ++i) emit(lane + 64 * i, u[i], cut);
        } else {
            if (choose) cut = cut_by_radix(row, n_blk, qb, need, reinterpret_cast<int*>(sc + rows * n_blk) + 256 * w, lane);
            for (int i = 0; 64 * i < n_blk; ++i) {
                const int c = lane + 64 * i;
                emit(c, c < n_blk ? order_key(row[c]) : 0u, cut);
            }
        }
        if (lane == 0) {
            row_ptr[(size_t)bh * (n_blk + 1) + qb] = (int32_t)row_off;
            if (qb == n_blk - 1) row_ptr[(size_t)bh * (n_blk + 1) + n_blk] = (int32_t)(row_off + kk);
        }
    }
}

constexpr int kMaxDevices = 64;
std::atomic<float*> g_scratch_ptr[kMaxDevices];

}  // namespace

// Library-owned workspace of rt_dynamic_index_noalloc, for callers that cannot
// allocate: the pooled query sums and key means, 2 * B*H*n_blk*D floats at most
// kDynScratchFloats (16 MiB).  Each GPU holds its own copy until the process
// ends.  In host code `scratch` names a host-side stand-in, never the device
// memory: its device address comes from hipGetSymbolAddress, once per device.
static __device__ __align__(256) float scratch[kDynScratchFloats];

hipError_t dynamic_scratch(float** ptr) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    float* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (p == nullptr) {
        // first call on this device, with it current: its copy's address
        void* addr = nullptr;
        e = hipGetSymbolAddress(&addr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        p = static_cast<float*>(addr);
        g_scratch_ptr[dev].store(p, std::memory_order_release);
    }
    *ptr = p;
    return hipSuccess;
}

hipError_t launch_dynamic_index(const DynIndexArgs& a, hipStream_t stream) {
    const int n_bh = a.B * a.H;
    hipLaunchKernelGGL(pool_kernel, dim3(n_bh * a.n_blk), dim3(kPoolThreads), 0, stream, a.q, a.k, a.T, a.D,
                       a.block, a.n_blk, a.qsum, a.kmean);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // A wave per 64 key blocks and, while their scores fit, two rows per wave; one where radix
    // passes select, whose latency two rows in turn double (556 blocks, D = 64, 1 head:
    // 20.6 us, two rows 35.6; 60 heads 161 and 169).
    const int n_tile = (a.n_blk + 63) / 64;
    const int waves = n_tile < kSelWaves ? n_tile : kSelWaves;
    int rows = (n_tile > kSelRegs ? 1 : 2) * waves;
    const int fit = (int)(kSelScoreBytes / (a.n_blk * sizeof(float)));  // >= 2: n_blk <= 4096
    if (rows > fit) rows = fit;
    const int n_grp = (a.n_blk + rows - 1) / rows;
    const size_t lds = (size_t)rows * a.n_blk * sizeof(float) + (a.n_blk > 64 * kSelRegs ? waves * 1024 : 0);
    const dim3 grid(n_bh * n_grp), block(64 * waves);
    auto go = [&](auto tiles) {
        constexpr int N = decltype(tiles)::value;
        if (a.D == 64)
            hipLaunchKernelGGL((select_kernel<64, N>), grid, block, lds, stream, a.qsum, a.kmean, a.n_blk, a.keep, rows,
                               waves, a.row_ptr, a.col_idx);
        else
            hipLaunchKernelGGL((select_kernel<72, N>), grid, block, lds, stream, a.qsum, a.kmean, a.n_blk, a.keep, rows,
                               waves, a.row_ptr, a.col_idx);
    };
    static_assert(kSelRegs == 8, "one case for each count of tiles");
    switch (n_tile) {  // a row's keys take as many registers as it has tiles
        case 1: go(std::integral_constant<int, 1>{}); break;
        case 2: go(std::integral_constant<int, 2>{}); break;
        case 3: go(std::integral_constant<int, 3>{}); break;
        case 4: go(std::integral_constant<int, 4>{}); break;
        case 5: go(std::integral_constant<int, 5>{}); break;
        case 6: go(std::integral_constant<int, 6>{}); break;
        case 7: go(std::integral_constant<int, 7>{}); break;
        case 8: go(std::integral_constant<int, 8>{}); break;
        default: go(std::integral_constant<int, 0>{});
    }
    return hipGetLastError();
}

}  // namespace rt
