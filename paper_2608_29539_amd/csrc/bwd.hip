// bwd.hip -- backward pass of the layer with the selection held fixed
// (App. B, backward traversal of the query-sparse global branch; the chain
// rule through Eqs. contextnorm, output-fusion and branch-attention):
//
//   fusion_bwd_kernel  ContextNorm + fusion backward per (token, head): the
//                      gradients of the raw branch outputs dO^L, dO^G (bf16,
//                      the operand of the attention backward), the row sums
//                      Delta = dO . O, each row's term of dL/dp, partial gain
//                      gradients, and a compact copy of the selected rows of
//                      Q^G (so the global branch's query tiles are contiguous).
//   bwd_reduce_kernel  dL/dp_t = sum over heads of the row terms, column sums
//                      of the gain-gradient partials, the zeros of dq_g.
//   bwd_dq_kernel      dQ of one branch.  Rows: local = every token (keys of
//                      its window), global = the selected rows in rank order
//                      (keys 0..pos).  Lane = query: S^T = K Q^T and
//                      dP^T = V dO^T with Q, dO in registers, then
//                      dQ^T += K^T dS^T with K^T read transposed from LDS.
//   bwd_dkv_kernel     dK, dV of one branch over dense KV blocks.  Lane = key:
//                      S = Q K^T, dP = dO V^T with K, V in registers, then
//                      dV^T += dO^T P and dK^T += Q^T dS with dO^T, Q^T read
//                      transposed from LDS.  A KV block of the global branch
//                      starts at the first compacted query row that can see
//                      it (binary search of sel_idx), so its loop covers only
//                      rows at or after the block, and only the first one or
//                      two query tiles need the causal mask.
//
// Softmax recomputation: P = 2^(c s - lse) with c = scale log2(e) and lse
// the forward's base-2 log-sum-exp; dS = P (dP - Delta).  P and dS are
// rounded to bf16 for the MFMAs, accumulation is fp32, and the outputs are
// fp32 (dQ, dK scaled by the softmax scale at the end).
//
// LDS tile layout (Q, dO, K, V tiles of 64 rows x d bf16, unpadded): the
// 16-byte chunk j of row r is stored at chunk j ^ swz(r).  The swizzle makes
// both access patterns conflict-free: the fragment reads (16 lanes read 16
// consecutive rows, one chunk each) and the transpose reads (32 lanes read
// 4 consecutive rows, 64 contiguous bytes each).
#include "logo_internal.h"
#include "attn_common.h"
#include "bwd_rules.h"

#include <type_traits>
#include <utility>

namespace logo {
namespace {

// f(integral_constant 0) ... f(integral_constant N - 1): unrolled by
// construction, so that every index is a compile-time constant.
template <int... I, class F>
__device__ __forceinline__ void static_for_seq(std::integer_sequence<int, I...>, F &&f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for_seq(std::make_integer_sequence<int, N>{}, f);
}

constexpr int kBwdWaves = 4;
static_assert(kBwdWaves * kWaveKeys == kKeysPerWg, "keys of a dK / dV workgroup");

template <int D>
__device__ __forceinline__ constexpr int swz(int r) {
    return D == 128 ? (((r & 3) << 2) | ((r >> 2) & 3))
                    : ((((r >> 1) & 1) << 2) | ((r >> 2) & 3));
}
// Byte offset of element col (a multiple of 4) of row r in a swizzled tile.
template <int D>
__device__ __forceinline__ int swz_off(int r, int col) {
    return r * D * 2 + (((col >> 3) ^ swz<D>(r)) << 4) + (col & 7) * 2;
}

// Global -> LDS staging of one swizzled 64-row tile by the 4 waves: LDS slot
// s (16 bytes) holds chunk (s % C) ^ swz(row) of row s / C, C = d / 8.  The
// per-lane byte offsets inside a tile are fixed and computed once.
template <int D>
struct TileDma {
    static constexpr int kInst = kTileRows * (D / 8) / 64;
    static constexpr int kPerWave = kInst / kBwdWaves;
    int voff[kPerWave];
};
template <int D>
__device__ __forceinline__ void tile_dma_plan(TileDma<D> &d, int wave, int lane, int row_bytes) {
#pragma unroll
    for (int i = 0; i < TileDma<D>::kPerWave; i++) {
        const int slot = (i * kBwdWaves + wave) * 64 + lane;
        const int row = slot / (D / 8), p = slot % (D / 8);
        d.voff[i] = row * row_bytes + ((p ^ swz<D>(row)) << 4);
    }
}
// dst: the LDS address of the tile (lds_addr_of)
// (tile_dma_part: the i-th of the wave's loads)
template <int D>
__device__ __forceinline__ void tile_dma_part(uint32_t dst, const TileDma<D> &d, u32x4 r, int wave,
                                              int i) {
    lds_load16_at(r, dst + (i * kBwdWaves + wave) * 1024, d.voff[i]);
}
template <int D>
__device__ __forceinline__ void tile_dma(uint32_t dst, const TileDma<D> &d, u32x4 r, int wave) {
#pragma unroll
    for (int i = 0; i < TileDma<D>::kPerWave; i++)
        lds_load16_at(r, dst + (i * kBwdWaves + wave) * 1024, d.voff[i]);
}

// Per-lane LDS offsets of the two fragment kinds inside a tile:
//   row: A/B operand rows  (row m = lane % 32, columns 16 ss + 8 g .. +7)
//   tr : transposed operand, column block cb, first / second read (rows
//        4 g + (lane % 16) / 4 and 8 further)
template <int D>
struct FragOffsets {
    int row[D / 16];
    int tr0[D / 32], tr1[D / 32];
};
template <int D>
__device__ __forceinline__ void frag_offsets(FragOffsets<D> &o, int lane) {
    const int m = lane & 31, g = lane >> 5;
#pragma unroll
    for (int ss = 0; ss < D / 16; ss++)
        o.row[ss] = swz_off<D>(m, ss * 16 + g * 8);
    const int tr_row = 4 * g + ((lane & 15) >> 2);
    const int tr_col = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
#pragma unroll
    for (int cb = 0; cb < D / 32; cb++) {
        o.tr0[cb] = swz_off<D>(tr_row, cb * 32 + tr_col);
        o.tr1[cb] = swz_off<D>(tr_row + 8, cb * 32 + tr_col);
    }
}
__device__ __forceinline__ bf16x8 frag_at(const char *tile, int off) {
    return *(const bf16x8 *)(tile + off);
}
// Transposed fragment of rows row0 .. row0+15 (row0 a multiple of 16),
// column block cb: lane l holds column 32 cb + l % 32 of rows
// row0 + 4 g + 0..3 and row0 + 8 + 4 g + 0..3 -- the order in which an
// accumulator's lane holds those rows.
template <int D>
__device__ __forceinline__ bf16x8 frag_tr(const char *tile, const FragOffsets<D> &o, int row0,
                                          int cb) {
    const char *t = tile + row0 * D * 2;
    return lds_tr_pair(t + o.tr0[cb], t + o.tr1[cb]);
}

__device__ __forceinline__ bf16x8 pack8(const bf16x2 (&w)[8], int half) {
    bf16x8 f;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        f[2 * j] = w[half * 4 + j][0];
        f[2 * j + 1] = w[half * 4 + j][1];
    }
    return f;
}

// ---------------------------------------------------------------------------
// dQ
// ---------------------------------------------------------------------------
// Two waves per SIMD, bound by MFMA issue and, over long runs, by the power
// budget (1.7 GHz at 64% of the matrix cycles).  Dense causal, 8192 tokens,
// 32 / 8 heads, d = 128: 690 us (1195 TFLOP/s executed), against 731 us with
// each half's softmax between its own products, 4 spilled registers and a
// branch per tile; 4096 selected rows of 32768 tokens: 1460 against 1629 us.
template <int D, int MODE>
__global__ __launch_bounds__(kBwdWaves * 64) __attribute__((amdgpu_waves_per_eu(2)))
void bwd_dq_kernel(const BwdArgs a) {
    constexpr int kTileBytes = kTileRows * D * 2;
    // two buffers of (K tile, V tile)
    __shared__ __attribute__((aligned(16))) char stile[2][2][kTileBytes];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = uni(tid >> 6);
    const int g = lane >> 5, m = lane & 31;
    const int bid = blockIdx.x;
    const int hg = bid % a.n_hg, rest = bid / a.n_hg;
    const int b = uni(rest % a.num_seqs);
    const int jt = a.ntile_max - 1 - rest / a.num_seqs;     // longest rows first
    const int base = uni(a.cu_seqlens[b]);
    const int T = uni(a.cu_seqlens[b + 1] - base);
    int row0 = base, nrows = T;
    if (MODE == kModeGlobal) {
        row0 = uni(a.cu_sel[b]);
        nrows = uni(max(0, min(a.cu_sel[b + 1], a.cap) - row0));
    }
    const int t0 = jt * a.tpw;
    if (t0 >= nrows)
        return;
    const int nvalid = min(a.tpw, nrows - t0);
    const int hw = wave % a.hpw, tb = wave / a.hpw;
    const int head = hg * a.hpw + hw;
    const int kvh = (hg * a.hpw) / a.group;
    auto pos_of = [&](int r) { return (MODE == kModeGlobal ? a.sel_idx[r] : r) - base; };
    const int ri = tb * 32 + m;
    const bool valid = ri < nvalid;
    const int r = row0 + t0 + (valid ? ri : nvalid - 1);
    const int pos = pos_of(r);
    const bool wave_valid = tb * 32 < nvalid;
    const int wpmin = __builtin_amdgcn_readfirstlane(pos);
    const int wpmax = __builtin_amdgcn_readlane(pos, 31);
    const int wg_pmin = uni(pos_of(row0 + t0));
    const int wg_pmax = uni(pos_of(row0 + t0 + nvalid - 1));

    bf16x8 qf[D / 16], dof[D / 16];
    {
        const int64_t off = ((int64_t)r * a.hq + head) * D + g * 8;
#pragma unroll
        for (int ss = 0; ss < D / 16; ss++) {
            qf[ss] = *(const bf16x8 *)(a.q + off + ss * 16);
            dof[ss] = *(const bf16x8 *)(a.dout + off + ss * 16);
        }
    }
    const float lse = a.lse[(int64_t)head * a.row_stride + r];
    const float ndlt = a.ndelta[(int64_t)head * a.row_stride + r];
    const float c = a.scale_log2;

    const int w = a.window;
    const int lo = (MODE == kModeLocal) ? max(0, wg_pmin - w + 1) : 0;
    const int kb_lo = lo / kTileRows, kb_hi = wg_pmax / kTileRows;
    int kb_first = kb_lo, kb_last = min(wpmax / kTileRows, kb_hi);
    if (MODE == kModeLocal)
        kb_first = max(kb_lo, max(0, wpmin - w + 1) / kTileRows);
    if (!wave_valid) {
        kb_first = kb_hi + 1;
        kb_last = kb_hi;
    }
    // tiles that need the real-position mask: past the causal edge of the
    // wave's first row, or (local) before the window edge of its last row
    const int kb_c = (wpmin + 1) / kTileRows - 1;
    int kb_w = kb_first;
    if (MODE == kModeLocal && wpmax - w + 1 > 0)
        kb_w = max(kb_w, (wpmax - w + 1 + kTileRows - 1) / kTileRows);

    const int row_bytes = a.hkv * D * 2;
    const uint16_t *kbase = a.k + ((int64_t)base * a.hkv + kvh) * D;
    const uint16_t *vbase = a.v + ((int64_t)base * a.hkv + kvh) * D;
    TileDma<D> dma;
    tile_dma_plan<D>(dma, wave, lane, row_bytes);
    FragOffsets<D> fo;
    frag_offsets<D>(fo, lane);
    auto stage = [&](int kb_, int buf) __attribute__((always_inline)) {
        const int k0 = kb_ * kTileRows;
        const int nb = max(0, min(kTileRows, T - k0)) * row_bytes;
        const uint32_t dst = lds_addr_of(&stile[0][0][0]) + buf * 2 * kTileBytes;
        tile_dma<D>(dst, dma, raw_rsrc(kbase + (int64_t)k0 * a.hkv * D, nb), wave);
        tile_dma<D>(dst + kTileBytes, dma, raw_rsrc(vbase + (int64_t)k0 * a.hkv * D, nb), wave);
    };

    f32x16 acc[D / 32];
#pragma unroll
    for (int cb = 0; cb < D / 32; cb++)
        acc[cb] = f32x16{};

    // One 64-key tile: 3 D / 8 MFMAs in four blocks, the two 32-key halves
    // skewed so that each half's softmax has independent MFMAs beside it:
    //   S, dP (half 0) | S, dP (half 1) + softmax (half 0) |
    //   dQ (half 0) + softmax (half 1) | dQ (half 1)
    // Chunk n holds the LDS reads of MFMA n + kAhead's operand, MFMA n and a
    // slice of a softmax; the scheduler may not move anything between chunks.
    constexpr int NM = D / 8;                // MFMAs of a block of S and dP
    constexpr int kAhead = 3;                // operand fragments in flight
    auto compute = [&](int kb_, auto masked) __attribute__((always_inline)) {
        const int k0 = kb_ * kTileRows;
        f32x16 s[2], dp[2];
        float p[2][2];
        bf16x2 dsw[2][8];
        bf16x8 fr[kAhead + 1];
        // MFMA n: its LDS operand, and the product
        auto load = [&](int n) __attribute__((always_inline)) {
            if (n < 2 * NM) {
                const int sb = n / NM, i = n % NM;
                return frag_at(stile[0][i & 1] + sb * 32 * D * 2, fo.row[i / 2]);
            }
            const int i = n - 2 * NM, sb = i / (NM / 2), j = i % (NM / 2);
            return frag_tr<D>(stile[0][0], fo, sb * 32 + (j / (NM / 4)) * 16, j % (NM / 4));
        };
        auto mfma = [&](int n) __attribute__((always_inline)) {
            const bf16x8 f = fr[n % (kAhead + 1)];
            if (n < 2 * NM) {
                const int sb = n / NM, i = n % NM;
                if (i % 2 == 0)
                    s[sb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, qf[i / 2], s[sb], 0, 0, 0);
                else
                    dp[sb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, dof[i / 2], dp[sb], 0, 0, 0);
            } else {
                const int i = n - 2 * NM, sb = i / (NM / 2), j = i % (NM / 2), cb = j % (NM / 4);
                acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, pack8(dsw[sb], j / (NM / 4)),
                                                                  acc[cb], 0, 0, 0);
            }
        };
        // softmax backward of half sb, element pair j: P = 2^(c S - lse),
        // then dS = P (dP - Delta) rounded to bf16.  Lane: query column;
        // element i: key k0 + 32 sb + 8 (i/4) + 4 g + i%4.
        auto soft_p = [&](int sb, int j) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 2; e++) {
                const int i = 2 * j + e;
                float x = fmaf(s[sb][i], c, -lse);
                if constexpr (decltype(masked)::value) {
                    const int key = k0 + sb * 32 + (i >> 2) * 8 + g * 4 + (i & 3);
                    bool ok = key <= pos;
                    if (MODE == kModeLocal)
                        ok = ok & (key > pos - w);
                    x = ok ? x : kNegInf;                // P = 0
                }
                p[sb][e] = __builtin_amdgcn_exp2f(x);
            }
        };
        auto soft_ds = [&](int sb, int j) __attribute__((always_inline)) {
            dsw[sb][j] = cvt_bf16x2(p[sb][0] * (dp[sb][2 * j] + ndlt), p[sb][1] * (dp[sb][2 * j + 1] + ndlt));
        };
        s[0] = s[1] = dp[0] = dp[1] = f32x16{};
#pragma unroll
        for (int n = 0; n < kAhead; n++)
            fr[n] = load(n);
        __builtin_amdgcn_sched_barrier(0);
        static_for<3 * NM>([&](auto nc) __attribute__((always_inline)) {
            constexpr int n = decltype(nc)::value;
            if constexpr (n + kAhead < 3 * NM)
                fr[(n + kAhead) % (kAhead + 1)] = load(n + kAhead);
            mfma(n);
            // half 0: one pair every NM / 8 chunks; half 1: twice as dense
            static_for<8>([&](auto jc) __attribute__((always_inline)) {
                constexpr int j = decltype(jc)::value;
                constexpr int a0 = NM + 1 + j * (NM / 8), a1 = 2 * NM + 1 + j * NM / 16;
                if constexpr (n == a0 + 1)
                    soft_ds(0, j);
                if constexpr (n == a0)
                    soft_p(0, j);
                if constexpr (NM == 8 && n == a1) {
                    soft_p(1, j);
                    soft_ds(1, j);
                }
                if constexpr (NM != 8 && n == a1 + 1)
                    soft_ds(1, j);
                if constexpr (NM != 8 && n == a1)
                    soft_p(1, j);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    using T_ = std::true_type;
    using F_ = std::false_type;
    // Step kb (buffer (kb - kb_lo) % 2): stage tile kb+1 into the other
    // buffer, run `work` on tile kb, then wait for the staged loads and
    // barrier.  The fragment offsets point into the current buffer.
    auto step = [&](int kb_, auto &&work) __attribute__((always_inline)) {
        if (kb_ < kb_hi)
            stage(kb_ + 1, ((kb_ - kb_lo) & 1) ^ 1);
        work();
        dma_wait_barrier();
#pragma unroll
        for (int i = 0; i < D / 16; i++)
            fo.row[i] ^= 2 * kTileBytes;
#pragma unroll
        for (int i = 0; i < D / 32; i++) {
            fo.tr0[i] ^= 2 * kTileBytes;
            fo.tr1[i] ^= 2 * kTileBytes;
        }
    };
    stage(kb_lo, 0);
    dma_wait_barrier();
    // Loops of a single kind each: tiles only the other waves see, window
    // edge, unmasked, diagonal.
    int kb = kb_lo;
    for (; kb < kb_first && kb <= kb_hi; kb++)
        step(kb, [] {});
    for (; kb <= kb_last && kb < kb_w; kb++)
        step(kb, [&]() __attribute__((always_inline)) { compute(kb, T_{}); });
    for (; kb <= kb_last && kb <= kb_c; kb++)
        step(kb, [&]() __attribute__((always_inline)) { compute(kb, F_{}); });
    for (; kb <= kb_last; kb++)
        step(kb, [&]() __attribute__((always_inline)) { compute(kb, T_{}); });
    for (; kb <= kb_hi; kb++)
        step(kb, [] {});

    if (!(wave_valid && valid))
        return;
    const int tok = pos + base;
    float *op = a.dq + ((int64_t)tok * a.hq + head) * D + g * 4;
#pragma unroll
    for (int cb = 0; cb < D / 32; cb++)
#pragma unroll
        for (int qd = 0; qd < 4; qd++) {
            f32x4 v = {acc[cb][qd * 4 + 0], acc[cb][qd * 4 + 1], acc[cb][qd * 4 + 2],
                       acc[cb][qd * 4 + 3]};
            v *= a.scale;
            if (a.acc_q)
                v += *(const f32x4 *)(op + cb * 32 + qd * 8);
            *(f32x4 *)(op + cb * 32 + qd * 8) = v;
        }
}

// ---------------------------------------------------------------------------
// dK, dV
// ---------------------------------------------------------------------------
// One wave per SIMD (32 keys: K and V fragments in AGPRs, dK and dV in the
// accumulators, both halves' scores in VGPRs).  What bounds it, by leaving
// parts out (dense causal, 8192 tokens, 32 / 8 heads, d = 128, 960 us): the
// MFMAs and the softmax 680 us, the LDS reads of one fragment per MFMA
// another 200 (each costs the wave ~6 cycles of issue, however far ahead it
// is made), the tile loads 80-100.  It took 1140 us with each half's softmax
// between its own products, the score accumulators in AGPRs (a copy per value
// read) and the row scalars staged through registers; dK, dV of the selected
// rows of 32768 tokens: 2430 -> 2080 us, of the local branch: 1300 -> 1083.
template <int D, int MODE>
__global__ __launch_bounds__(kBwdWaves * 64) __attribute__((amdgpu_waves_per_eu(1, 1)))
void bwd_dkv_kernel(const BwdArgs a) {
    constexpr int kTileBytes = kTileRows * D * 2;
    constexpr int kBufs = 3;
    // buffers of (Q tile, dO tile) and the rows' scalars: lse, -Delta, (global)
    // token index; the fourth row is a place for a load that keeps the waves'
    // numbers of loads equal
    __shared__ __attribute__((aligned(16))) char stile[kBufs][2][kTileBytes];
    __shared__ __attribute__((aligned(16))) float srow[kBufs][4][kTileRows];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = uni(tid >> 6);
    const int g = lane >> 5, m = lane & 31;
    const int bid = blockIdx.x;
    const int kvh = bid % a.hkv, rest = bid / a.hkv;
    const int b = uni(rest % a.num_seqs);
    const int jt = rest / a.num_seqs;                        // early blocks (most rows) first
    const int base = uni(a.cu_seqlens[b]);
    const int T = uni(a.cu_seqlens[b + 1] - base);
    const int k0 = jt * kKeysPerWg;
    if (k0 >= T)
        return;
    const int j0 = k0 + wave * 32;                           // this wave's first key
    const int key = j0 + m;                                  // this lane's key (column)
    const int w = a.window;

    bf16x8 kf[D / 16], vf[D / 16];
    {
        const int jl = min(key, T - 1);
        const int64_t off = ((int64_t)(base + jl) * a.hkv + kvh) * D + g * 8;
#pragma unroll
        for (int ss = 0; ss < D / 16; ss++) {
            kf[ss] = *(const bf16x8 *)(a.k + off + ss * 16);
            vf[ss] = *(const bf16x8 *)(a.v + off + ss * 16);
        }
    }

    // At d = 128 the fragments live in AGPRs, where the products read them in
    // place: left to itself the compiler fills the VGPRs first and copies
    // fragments back and forth in the loop.
    if constexpr (D == 128) {
#pragma unroll
        for (int ss = 0; ss < D / 16; ss++)
            asm volatile("" : "+a"(kf[ss]), "+a"(vf[ss]));
    }

    // Rows that can see a key of this block: local, positions k0 .. k0+127+w-1;
    // global, the compacted rows from the first one at or after k0.
    int r_begin, r_end;
    if (MODE == kModeGlobal) {
        const int s0 = uni(a.cu_sel[b]);
        const int s1 = uni(max(s0, min(a.cu_sel[b + 1], a.cap)));
        int lo_ = s0, hi_ = s1;
        while (lo_ < hi_) {
            const int mid = (lo_ + hi_) >> 1;
            if (uni(a.sel_idx[mid]) - base < k0)
                lo_ = mid + 1;
            else
                hi_ = mid;
        }
        r_begin = lo_;
        r_end = s1;
    } else {
        r_begin = base + k0;
        r_end = base + local_row_end(T, k0, w);
    }
    const int nblk = (r_end - r_begin + kTileRows - 1) / kTileRows;
    const int nsteps = nblk * a.group;                       // every head of the KV group

    // The 64-row tiles q of a head that this wave computes, qf .. ql, and
    // among them the ones that need no mask, qa .. qb - 1.  (The same for every
    // head.)
    const DkvTiles tiles = dkv_tiles<MODE == kModeLocal>(
        r_end - r_begin,
        [&](int i) {
            const int r = r_begin + i;
            return (MODE == kModeGlobal ? uni(a.sel_idx[r]) : r) - base;
        },
        T, k0, j0, w);
    const int qf = tiles.first, ql = tiles.last, qa = tiles.full, qb = tiles.full_end;

    const int row_bytes = a.hq * D * 2;
    TileDma<D> dma;
    tile_dma_plan<D>(dma, wave, lane, row_bytes);
    FragOffsets<D> fo;
    frag_offsets<D>(fo, lane);
    // Staging of tile q of head hh into buffer buf, all of it global -> LDS:
    // the Q / dO tiles, and the rows' lse (wave 0), -Delta (wave 1) and token
    // index (wave 2).  Rows past the tile's end read as zeros, which no row
    // uses.  (Scalars that pass through a register of the wave instead make
    // it wait for them in the middle of the step: 1209 against 1003 us for
    // the dense backward at 8192 tokens, 32 / 8 heads, d = 128.)
    constexpr int kLoads = 2 * TileDma<D>::kPerWave + 1;     // of each wave
    const uint32_t lds_tile = lds_addr_of(&stile[0][0][0]), lds_row = lds_addr_of(&srow[0][0][0]);
    struct Stage {
        u32x4 q, dout, row;
        uint32_t tile, rows;
    };
    auto stage_of = [&](int hh, int q, int buf) __attribute__((always_inline)) {
        const int head = kvh * a.group + hh;
        const int r0 = r_begin + q * kTileRows, nv = min(kTileRows, r_end - r0);
        const int64_t off = ((int64_t)r0 * a.hq + head) * D;
        const int64_t ro = (int64_t)head * a.row_stride + r0;
        const void *src = wave == 1 ? a.ndelta + ro : a.lse + ro;
        if (MODE == kModeGlobal && wave == 2)
            src = a.sel_idx + r0;
        return Stage{raw_rsrc(a.q + off, nv * row_bytes), raw_rsrc(a.dout + off, nv * row_bytes),
                     raw_rsrc(src, nv * 4), lds_tile + buf * 2 * kTileBytes,
                     lds_row + (buf * 4 + wave) * kTileRows * 4};
    };
    // the i-th of the wave's loads
    auto stage_part = [&](const Stage &sg, int i) __attribute__((always_inline)) {
        constexpr int P = TileDma<D>::kPerWave;
        if (i < P)
            tile_dma_part<D>(sg.tile, dma, sg.q, wave, i);
        else if (i < 2 * P)
            tile_dma_part<D>(sg.tile + kTileBytes, dma, sg.dout, wave, i - P);
        else
            lds_load4_at(sg.row, sg.rows, lane * 4);
    };
    auto stage_all = [&](const Stage &sg) __attribute__((always_inline)) {
        static_for<kLoads>([&](auto i) { stage_part(sg, decltype(i)::value); });
    };

    f32x16 dk[D / 32], dv[D / 32];
#pragma unroll
    for (int cb = 0; cb < D / 32; cb++)
        dk[cb] = dv[cb] = f32x16{};
    const float c = a.scale_log2;

    // One 64-row tile: 4 D / 8 MFMAs in four blocks, the two 32-row halves
    // skewed so that each half's softmax has independent MFMAs beside it:
    //   S, dP (half 0) | S, dP (half 1) + softmax (half 0) |
    //   dV, dK (half 0) + softmax (half 1) | dV, dK (half 1)
    // One wave runs per SIMD (the accumulators and the K / V fragments take
    // the registers of two), so the overlap has to be in the instruction
    // order: chunk n holds the LDS reads of MFMA n + kAhead's operand, MFMA n
    // and a slice of a softmax, and the scheduler may not move anything
    // between chunks.
    constexpr int NM = D / 8;                // MFMAs of a block
    constexpr int kAhead = 3;                // operand fragments in flight
    auto compute = [&](int buf, int q, const Stage &sg, auto masked)
                       __attribute__((always_inline)) {
        const char *qt = stile[buf][0], *dt = stile[buf][1];
        const int r0 = r_begin + q * kTileRows, nv = min(kTileRows, r_end - r0);
        f32x16 s[2], dp[2];
        f32x4 l4[2][4];
        float p[2][16];
        bf16x2 pw[2][8], dsw[2][8];
        bf16x8 fr[kAhead + 1];
        // MFMA n: its LDS operand, and the product
        auto load = [&](int n) __attribute__((always_inline)) {
            const int qh = (n / NM) & 1, i = n % NM;
            const char *t = ((n < 2 * NM) == (i % 2 == 0)) ? qt : dt;
            if (n < 2 * NM)
                return frag_at(t + qh * 32 * D * 2, fo.row[i / 2]);
            return frag_tr<D>(t, fo, qh * 32 + (i / (NM / 2)) * 16, (i % (NM / 2)) / 2);
        };
        auto mfma = [&](int n) __attribute__((always_inline)) {
            const int qh = (n / NM) & 1, i = n % NM;
            const bf16x8 f = fr[n % (kAhead + 1)];
            if (n < 2 * NM) {
                if (i % 2 == 0)
                    s[qh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, kf[i / 2], s[qh], 0, 0, 0);
                else
                    dp[qh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, vf[i / 2], dp[qh], 0, 0, 0);
            } else {
                const int half = i / (NM / 2), cb = (i % (NM / 2)) / 2;
                if (i % 2 == 0)
                    dv[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, pack8(pw[qh], half),
                                                                     dv[cb], 0, 0, 0);
                else
                    dk[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, pack8(dsw[qh], half),
                                                                     dk[cb], 0, 0, 0);
            }
        };
        // softmax of half qh, element pair j: P = 2^(c S - lse), then dS =
        // P (dP - Delta) and both rounded to bf16.  Lane: key column; element
        // i: row qh*32 + 8 (i/4) + 4 g + i%4.
        auto soft_p = [&](int qh, int j) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 2; e++) {
                const int i = 2 * j + e;
                float x = fmaf(s[qh][i], c, -l4[qh][i / 4][i % 4]);
                if constexpr (decltype(masked)::value) {
                    const int qi = qh * 32 + (i >> 2) * 8 + g * 4 + (i & 3);
                    const int qpos = (MODE == kModeGlobal ? __float_as_int(srow[buf][2][qi]) : r0 + qi) - base;
                    const bool ok = (qi < nv) & row_sees_key<MODE == kModeLocal>(qpos, key, w);
                    x = ok ? x : kNegInf;                // P = 0
                }
                p[qh][i] = __builtin_amdgcn_exp2f(x);
            }
        };
        auto soft_ds = [&](int qh, int j) __attribute__((always_inline)) {
            pw[qh][j] = cvt_bf16x2(p[qh][2 * j], p[qh][2 * j + 1]);
            dsw[qh][j] = cvt_bf16x2(p[qh][2 * j] * dp[qh][2 * j], p[qh][2 * j + 1] * dp[qh][2 * j + 1]);
        };
        // S starts from zero, dP from -Delta
#pragma unroll
        for (int qh = 0; qh < 2; qh++) {
            s[qh] = f32x16{};
#pragma unroll
            for (int qd = 0; qd < 4; qd++) {
                const f32x4 d4 = *(const f32x4 *)&srow[buf][1][qh * 32 + qd * 8 + g * 4];
#pragma unroll
                for (int e = 0; e < 4; e++)
                    dp[qh][qd * 4 + e] = d4[e];
            }
        }
#pragma unroll
        for (int n = 0; n < kAhead; n++)
            fr[n] = load(n);
        __builtin_amdgcn_sched_barrier(0);
        static_for<4 * NM>([&](auto nc) __attribute__((always_inline)) {
            constexpr int n = decltype(nc)::value;
            if constexpr (n + kAhead < 4 * NM)
                fr[(n + kAhead) % (kAhead + 1)] = load(n + kAhead);
            // lse of each half's rows, four reads before its softmax
            constexpr int l0 = n - (NM - 4), l1 = n - (2 * NM - 4);
            if constexpr (l0 >= 0 && l0 < 4)
                l4[0][l0] = *(const f32x4 *)&srow[buf][0][l0 * 8 + g * 4];
            if constexpr (l1 >= 0 && l1 < 4)
                l4[1][l1] = *(const f32x4 *)&srow[buf][0][32 + l1 * 8 + g * 4];
            mfma(n);
            // one element pair every NM / 8 chunks, its P one chunk before its dS
            constexpr int st8 = NM / 8;
            constexpr int p0 = n - (NM + 1), p1 = n - (2 * NM + 1);
            if constexpr (p0 >= 0 && p0 % st8 == 0 && p0 / st8 < 8)
                soft_p(0, p0 / st8);
            if constexpr (p0 >= 1 && (p0 - 1) % st8 == 0 && (p0 - 1) / st8 < 8)
                soft_ds(0, (p0 - 1) / st8);
            if constexpr (p1 >= 0 && p1 % st8 == 0 && p1 / st8 < 8)
                soft_p(1, p1 / st8);
            if constexpr (p1 >= 1 && (p1 - 1) % st8 == 0 && (p1 - 1) / st8 < 8)
                soft_ds(1, (p1 - 1) / st8);
            // the loads of the tile two steps ahead, spread over the step: a
            // wave that issues them all at once waits for the address unit
            // with its matrix pipe idle
            constexpr int every = 4 * NM / kLoads;
            if constexpr (n % every == 2 && n / every < kLoads)
                stage_part(sg, n / every);
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    using T_ = std::true_type;
    using F_ = std::false_type;
    // Steps: the tiles from the last to the first, each for every head of the
    // group, so that all key blocks of a KV head walk the same rows at the
    // same time and find them in L2 (half of the L2 misses of the ascending
    // order with the heads outermost).  Each step stages the tile two steps
    // ahead, runs `work` on its own and then waits for the next one's.
    int st = 0, buf = 0, buf2 = 2;
    auto step = [&](int hh, int q, auto &&work) __attribute__((always_inline)) {
        const bool more = st + 2 < nsteps;
        // two (tile, head) pairs on: hh + 2 < 2 G, or 2 for G = 1; past the
        // last one the loads repeat its tile into a buffer no one reads
        const int h2 = hh + 2, up = h2 < a.group ? 0 : (h2 < 2 * a.group ? 1 : 2);
        const Stage sg = more ? stage_of(h2 - up * a.group, q - up, buf2) : stage_of(hh, q, buf2);
        work(sg);
        dma_wait_barrier_but<kLoads>();
        st++;
        buf = buf == kBufs - 1 ? 0 : buf + 1;
        buf2 = buf2 == kBufs - 1 ? 0 : buf2 + 1;
    };
    if (nsteps > 0)
        stage_all(stage_of(0, nblk - 1, 0));
    if (nsteps > 1) {
        stage_all(stage_of(a.group > 1 ? 1 : 0, a.group > 1 ? nblk - 1 : nblk - 2, 1));
        dma_wait_barrier_but<kLoads>();
    } else {
        dma_wait_barrier_but<0>();
    }
    // Loops of a single kind each, so that no loop body switches between
    // instantiations (which would copy the 2 x D / 2 accumulators).
    int q = nblk - 1;
    for (; q > ql || (q >= 0 && qf >= nblk); q--)
        for (int hh = 0; hh < a.group; hh++)
            step(hh, q, stage_all);
    for (; q >= qb && q >= qf; q--)
        for (int hh = 0; hh < a.group; hh++)
            step(hh, q, [&](const Stage &sg) __attribute__((always_inline)) { compute(buf, q, sg, T_{}); });
    for (; q >= qa; q--)
        for (int hh = 0; hh < a.group; hh++)
            step(hh, q, [&](const Stage &sg) __attribute__((always_inline)) { compute(buf, q, sg, F_{}); });
    for (; q >= qf; q--)
        for (int hh = 0; hh < a.group; hh++)
            step(hh, q, [&](const Stage &sg) __attribute__((always_inline)) { compute(buf, q, sg, T_{}); });
    for (; q >= 0; q--)
        for (int hh = 0; hh < a.group; hh++)
            step(hh, q, stage_all);
    // no load may be in flight to this workgroup's LDS when it ends
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);

    if (key >= T)
        return;
    const int64_t off = ((int64_t)(base + key) * a.hkv + kvh) * D + g * 4;
    float *kp = a.dk + off;
    float *vp = a.dv + off;
#pragma unroll
    for (int cb = 0; cb < D / 32; cb++)
#pragma unroll
        for (int qd = 0; qd < 4; qd++) {
            f32x4 vk = {dk[cb][qd * 4 + 0], dk[cb][qd * 4 + 1], dk[cb][qd * 4 + 2],
                        dk[cb][qd * 4 + 3]};
            f32x4 vv = {dv[cb][qd * 4 + 0], dv[cb][qd * 4 + 1], dv[cb][qd * 4 + 2],
                        dv[cb][qd * 4 + 3]};
            vk *= a.scale;
            const int o = cb * 32 + qd * 8;
            if (a.acc_k)
                vk += *(const f32x4 *)(kp + o);
            if (a.acc_v)
                vv += *(const f32x4 *)(vp + o);
            *(f32x4 *)(kp + o) = vk;
            *(f32x4 *)(vp + o) = vv;
        }
}

// ---------------------------------------------------------------------------
// ContextNorm + fusion backward
// ---------------------------------------------------------------------------
// Slots: a token's Hq x d values are S = Hq d / 8 slots of 8; thread t of a
// workgroup handles slots (t + 256 k) % S of token t0 + (t + 256 k) / S for
// k < KS, so with S <= 256 a pass covers 256 / S tokens and with S > 256 a
// token takes KS = S / 256 slot sets.  A (token, head) row is d / 8
// consecutive lanes; its sums are DPP lane exchanges within them.
template <int Ctrl>
__device__ __forceinline__ float dpp_mov(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), Ctrl, 0xF, 0xF, false));
}
template <int D>
__device__ __forceinline__ float row_sum(float x) {
    // DPP within each group of D / 8 lanes (16 or 8, aligned): the two quad
    // swaps, then the half-row mirror (lane i <- 7 - i of its 8) and, for 16
    // lanes, the row mirror (i <- 15 - i), each pairing the partial sums of
    // disjoint lane sets.
    static_assert(D / 8 == 16 || D / 8 == 8, "row of 8 or 16 lanes");
    x += dpp_mov<0xB1>(x);        // quad_perm [1,0,3,2]
    x += dpp_mov<0x4E>(x);        // quad_perm [2,3,0,1]
    x += dpp_mov<0x141>(x);       // row_half_mirror
    if constexpr (D / 8 == 16)
        x += dpp_mov<0x140>(x);   // row_mirror
    return x;
}

template <int D, int KS>
__global__ __launch_bounds__(256) void fusion_bwd_kernel(const FusionBwdArgs a) {
    const int S = a.hq * (D / 8);
    const int P = S >= 256 ? 1 : 256 / S;                   // tokens per pass
    const int t_begin = blockIdx.x * a.tokens_per_block;
    const int t_end = min(a.n, t_begin + a.tokens_per_block);
    float gl_acc[KS][8], gg_acc[KS][8];
#pragma unroll
    for (int k = 0; k < KS; k++)
#pragma unroll
        for (int e = 0; e < 8; e++)
            gl_acc[k][e] = gg_acc[k][e] = 0.f;

    for (int t0 = t_begin; t0 < t_end; t0 += P) {
#pragma unroll
        for (int k = 0; k < KS; k++) {
            const int v = threadIdx.x + 256 * k;
            const int toff = v / S, slot = v % S;
            const int tok = t0 + toff;
            if (toff >= P || tok >= t_end)
                continue;                                    // uniform over a row's lanes
            const int h = slot / (D / 8), c0 = (slot % (D / 8)) * 8;
            const bool lead = c0 == 0;
            const int64_t e0 = ((int64_t)tok * a.hq + h) * D + c0;
            const float p = a.gate[tok];
            const int rank = a.tok2sel[tok];
            float dr[8];
            {
                const u32x4 w4 = *(const u32x4 *)(a.dout + e0);
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const uint32_t wd = w4[i];
                    dr[2 * i] = __uint_as_float(wd << 16);
                    dr[2 * i + 1] = __uint_as_float(wd & 0xFFFF0000u);
                }
            }
            float side = 0.f;
            // branch 0: local (every token), branch 1: global (selected)
#pragma unroll
            for (int br = 0; br < 2; br++) {
                if (br == 1 && rank < 0)
                    break;
                const float *src = br ? a.og + ((int64_t)rank * a.hq + h) * D + c0 : a.ol + e0;
                const float *gn = br ? a.gain_g : a.gain_l;
                float o[8], gv[8];
                {
                    const f32x4 x0 = *(const f32x4 *)src, x1 = *(const f32x4 *)(src + 4);
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        o[e] = x0[e];
                        o[4 + e] = x1[e];
                    }
                }
#pragma unroll
                for (int e = 0; e < 8; e++)
                    gv[e] = gn ? gn[h * D + c0 + e] : 1.f;
                const float wgt = br ? p : (rank >= 0 ? 1.f - p : 1.f);
                float sq = 0.f, proj = 0.f, sd = 0.f;
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    sq = fmaf(o[e], o[e], sq);
                    proj = fmaf(gv[e] * dr[e], o[e], proj);
                    sd = fmaf(dr[e] * gv[e], o[e], sd);
                }
                sq = row_sum<D>(sq);
                proj = row_sum<D>(proj) * wgt;
                sd = row_sum<D>(sd);
                const float rr = sqrtf(sq / (float)D + a.eps);
                const float ir = 1.f / rr;
                const float k3 = proj * ir * ir * ir / (float)D;
                float dO[8], dl = 0.f;
                float *gacc = br ? gg_acc[k] : gl_acc[k];
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    dO[e] = gv[e] * wgt * dr[e] * ir - o[e] * k3;
                    gacc[e] = fmaf(wgt * dr[e] * ir, o[e], gacc[e]);
                }
                // The attention backward takes dO in bf16 (dP = dO V^T);
                // Delta = dO . O takes the same rounded values, so that
                // sum_j dS_j = sum_j P_j (dP_j - Delta) vanishes as it does
                // in exact arithmetic (with one visible key, dS = 0).
                const u32x4 dob = u32x4{pack_bf16x2(dO[0], dO[1]), pack_bf16x2(dO[2], dO[3]),
                                        pack_bf16x2(dO[4], dO[5]), pack_bf16x2(dO[6], dO[7])};
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    dl = fmaf(__uint_as_float(dob[i] << 16), o[2 * i], dl);
                    dl = fmaf(__uint_as_float(dob[i] & 0xFFFF0000u), o[2 * i + 1], dl);
                }
                dl = row_sum<D>(dl);
                side += (br ? 1.f : -1.f) * sd * ir;
                const int64_t row = br ? rank : tok;
                uint16_t *dst = (br ? a.dog : a.dol) + (row * a.hq + h) * D + c0;
                *(u32x4 *)dst = dob;
                if (lead)
                    (br ? a.ndelta_g : a.ndelta_l)[(int64_t)h * (br ? a.cap : a.n) + row] = -dl;
                if (br == 1)
                    *(u32x4 *)(a.qc + (row * a.hq + h) * D + c0) = *(const u32x4 *)(a.q_g + e0);
            }
            if (lead)
                a.side[(int64_t)tok * a.hq + h] = rank >= 0 ? side : 0.f;
        }
    }
    // gain-gradient partials: row blockIdx.x * P + toff of [rows][Hq d]
    const int cols = a.hq * D;
#pragma unroll
    for (int k = 0; k < KS; k++) {
        const int v = threadIdx.x + 256 * k;
        const int toff = v / S, slot = v % S;
        if (toff >= P)
            continue;
        const int64_t o = ((int64_t)blockIdx.x * P + toff) * cols + slot * 8;
#pragma unroll
        for (int e = 0; e < 8; e++) {
            if (a.part_l)
                a.part_l[o + e] = gl_acc[k][e];
            if (a.part_g)
                a.part_g[o + e] = gg_acc[k][e];
        }
    }
}

// Zeros, 16 bytes per thread and step (block blk of the range; n a multiple
// of 4, x 16-byte aligned).
constexpr int kZeroPerBlock = 256 * 4 * 4;
__device__ __forceinline__ void zero_block(float *x, int64_t n, int64_t blk) {
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const int64_t i = blk * kZeroPerBlock + (j * 256 + threadIdx.x) * 4;
        if (i < n)
            *(f32x4 *)(x + i) = f32x4{0.f, 0.f, 0.f, 0.f};
    }
}

// What follows the ContextNorm + fusion backward, in one launch (its parts
// are independent, and as five launches of 4-8 us each they cost a small
// training step more than its dQ kernel).  Workgroups in this order:
//   gate_blocks   dL/dp_t: sum over heads of the per-row terms (zero for
//                 unselected tokens), one token per thread
//   gain blocks   column sums of the [rows][cols] gain-gradient partials of
//                 each branch with an output, over row chunks of kGainChunk:
//                 workgroup (x, y) sums rows y*kGainChunk .. of 64 columns (the
//                 4 waves take every 4th row, then a fixed-order sum of the
//                 4) into row y of `out`.  Two passes reduce any row count up
//                 to kGainChunk^2 to one row.
//   zero_blocks   dq_g, which the global branch's dQ writes only at the
//                 selected rows
constexpr int kGainChunk = 64;
__global__ __launch_bounds__(256) void bwd_reduce_kernel(const BwdReduceArgs a) {
    __shared__ float red[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int blk = blockIdx.x;
    if (blk < a.gate_blocks) {
        const int t = blk * 256 + threadIdx.x;
        if (t < a.n) {
            float s = 0.f;
            for (int h = 0; h < a.hq; h++)
                s += a.side[(int64_t)t * a.hq + h];
            a.dgate[t] = s;
        }
        return;
    }
    blk -= a.gate_blocks;
    const int col_blocks = (a.cols + 63) / 64;
    for (int br = 0; br < 2; br++) {
        if (!a.out[br])
            continue;
        if (blk < col_blocks * a.chunks) {
            const int y = blk / col_blocks, col = (blk % col_blocks) * 64 + lane;
            const int r0 = y * kGainChunk, r1 = min(a.rows, r0 + kGainChunk);
            float s = 0.f;
            if (col < a.cols)
                for (int r = r0 + wave; r < r1; r += 4)
                    s += a.part[br][(int64_t)r * a.cols + col];
            red[wave][lane] = s;
            __syncthreads();
            if (wave == 0 && col < a.cols)
                a.out[br][(int64_t)y * a.cols + col] =
                    (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
            return;
        }
        blk -= col_blocks * a.chunks;
    }
    zero_block(a.zero, a.n_zero, blk);
}

// -Delta = -rowsum(dO * O) per (token, head) for plain attention (bf16 O and
// dO), written [Hq][N]; one thread per 8 elements, d / 8 lanes per row.
template <int D>
__global__ __launch_bounds__(256) void attn_delta_kernel(int64_t n_rows, int hq, int64_t n,
                                                         const uint16_t *o, const uint16_t *dout,
                                                         float *ndelta) {
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t row = g / (D / 8);
    const bool ok = row < n_rows;
    float acc = 0.f;
    if (ok) {
        const u32x4 a = *(const u32x4 *)(o + g * 8), b = *(const u32x4 *)(dout + g * 8);
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint32_t x = a[i], y = b[i];
            acc = fmaf(__uint_as_float(x << 16), __uint_as_float(y << 16), acc);
            acc = fmaf(__uint_as_float(x & 0xFFFF0000u), __uint_as_float(y & 0xFFFF0000u), acc);
        }
    }
    acc = row_sum<D>(acc);
    if (ok && (g % (D / 8)) == 0) {
        const int64_t t = row / hq;
        const int h = (int)(row % hq);
        ndelta[(int64_t)h * n + t] = -acc;
    }
}

// Inputs of the standalone query-sparse backward (and, in the workgroups from
// prep_blocks on, the zeros of dq, which dQ writes only at the selected rows;
// at 8192 of 16384 rows of 8 heads, d = 128, 21 us, in two launches 32): per
// (selected rank < the device count, head) row, the compact copy of the row of
// Q and -Delta = -dO . O (O fp32, dO bf16, both compact), written [Hq][cap].
// d / 8 lanes per row.
template <int D>
__global__ __launch_bounds__(256) void sparse_prep_kernel(int64_t n_rows, int hq, int64_t cap,
                                                          const int32_t *n_sel_dev,
                                                          const int32_t *sel_idx,
                                                          const uint16_t *q, const float *o,
                                                          const uint16_t *dout, uint16_t *qc,
                                                          float *ndelta, int64_t prep_blocks,
                                                          float *zero, int64_t n_zero) {
    if (blockIdx.x >= prep_blocks) {
        zero_block(zero, n_zero, blockIdx.x - prep_blocks);
        return;
    }
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t row = g / (D / 8);
    // rows of ranks at or past the selected count (read on the device) are
    // skipped: their sel_idx entries are not written by the selection
    const int64_t live = min((int64_t)n_sel_dev[0], cap) * hq;
    const bool ok = row < n_rows && row < live;
    float acc = 0.f;
    if (ok) {
        const int64_t r = row / hq;
        const int h = (int)(row % hq);
        const int c0 = (int)(g % (D / 8)) * 8;
        const u32x4 b = *(const u32x4 *)(dout + g * 8);
        const f32x4 o0 = *(const f32x4 *)(o + g * 8), o1 = *(const f32x4 *)(o + g * 8 + 4);
        const float of[8] = {o0[0], o0[1], o0[2], o0[3], o1[0], o1[1], o1[2], o1[3]};
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint32_t y = b[i];
            acc = fmaf(of[2 * i], __uint_as_float(y << 16), acc);
            acc = fmaf(of[2 * i + 1], __uint_as_float(y & 0xFFFF0000u), acc);
        }
        const int64_t tok = sel_idx[r];
        *(u32x4 *)(qc + g * 8) = *(const u32x4 *)(q + (tok * hq + h) * D + c0);
    }
    acc = row_sum<D>(acc);
    if (ok && (g % (D / 8)) == 0)
        ndelta[(int64_t)(row % hq) * cap + row / hq] = -acc;
}

template <int D>
hipError_t launch_fusion_bwd_d(const FusionBwdArgs &a, int grid, hipStream_t s) {
    const int S = a.hq * (D / 8);
    const int ks = S <= 256 ? 1 : S / 256;
    if (ks == 1)
        hipLaunchKernelGGL((fusion_bwd_kernel<D, 1>), dim3(grid), dim3(256), 0, s, a);
    else if (ks == 2)
        hipLaunchKernelGGL((fusion_bwd_kernel<D, 2>), dim3(grid), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL((fusion_bwd_kernel<D, 4>), dim3(grid), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace

int fusion_bwd_tokens_per_pass(int hq, int head_dim) {
    const int S = hq * head_dim / 8;
    return S >= 256 ? 1 : 256 / S;
}

bool fusion_bwd_supported(int hq, int head_dim) {
    const int S = hq * head_dim / 8;
    return S <= 256 ? true : (S % 256 == 0 && S / 256 <= 4 && (S / 256) != 3);
}

hipError_t launch_fusion_bwd(const FusionBwdArgs &a, int grid, int head_dim, hipStream_t s) {
    if (grid <= 0)
        return hipSuccess;
    return head_dim == 128 ? launch_fusion_bwd_d<128>(a, grid, s)
                           : launch_fusion_bwd_d<64>(a, grid, s);
}

int gain_grad_chunks(int rows) { return (rows + kGainChunk - 1) / kGainChunk; }

// tmp[br]: gain_grad_chunks(rows) x cols floats for each branch with an
// output (dgain[br] not NULL); dgate and zero may be NULL.
hipError_t launch_bwd_reduce(int n, int hq, const float *side, float *dgate, int rows, int cols,
                             const float *const part[2], float *const tmp[2],
                             float *const dgain[2], float *zero, int64_t n_zero, hipStream_t s) {
    BwdReduceArgs a;
    a.n = n;
    a.hq = hq;
    a.side = side;
    a.dgate = dgate;
    a.gate_blocks = dgate ? (n + 255) / 256 : 0;
    a.rows = rows;
    a.cols = cols;
    a.chunks = gain_grad_chunks(rows);
    if (a.chunks > kGainChunk)
        return hipErrorInvalidValue;               // two passes cover 4096 rows
    a.zero = zero;
    a.n_zero = zero ? n_zero : 0;
    const long long per_branch = (long long)((cols + 63) / 64) * a.chunks;
    long long grid = a.gate_blocks + (a.n_zero + kZeroPerBlock - 1) / kZeroPerBlock;
    for (int br = 0; br < 2; br++) {
        a.part[br] = part[br];
        a.out[br] = dgain[br] ? (a.chunks > 1 ? tmp[br] : dgain[br]) : nullptr;
        if (a.out[br])
            grid += per_branch;
    }
    if (grid == 0)
        return hipSuccess;
    hipLaunchKernelGGL(bwd_reduce_kernel, dim3((unsigned)grid), dim3(256), 0, s, a);
    if (a.chunks > 1 && (dgain[0] || dgain[1])) {
        grid = 0;
        for (int br = 0; br < 2; br++) {
            a.part[br] = tmp[br];
            a.out[br] = dgain[br];
            if (dgain[br])
                grid += (cols + 63) / 64;
        }
        a.gate_blocks = 0;
        a.n_zero = 0;
        a.rows = a.chunks;
        a.chunks = 1;
        hipLaunchKernelGGL(bwd_reduce_kernel, dim3((unsigned)grid), dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_attn_delta(int64_t n, int hq, int head_dim, const uint16_t *o,
                             const uint16_t *dout, float *ndelta, hipStream_t s) {
    const int64_t threads = n * hq * (head_dim / 8);
    if (threads <= 0)
        return hipSuccess;
    const dim3 grid((unsigned)((threads + 255) / 256));
    if (head_dim == 128)
        hipLaunchKernelGGL((attn_delta_kernel<128>), grid, dim3(256), 0, s, n * hq, hq, n, o, dout,
                           ndelta);
    else
        hipLaunchKernelGGL((attn_delta_kernel<64>), grid, dim3(256), 0, s, n * hq, hq, n, o, dout,
                           ndelta);
    return hipGetLastError();
}

hipError_t launch_sparse_prep(int64_t cap, int hq, int head_dim, const int32_t *n_sel_dev,
                              const int32_t *sel_idx, const uint16_t *q, const float *o,
                              const uint16_t *dout, uint16_t *qc, float *ndelta, float *zero,
                              int64_t n_zero, hipStream_t s) {
    const int64_t prep = (cap * hq * (head_dim / 8) + 255) / 256;
    const int64_t blocks = prep + (n_zero + kZeroPerBlock - 1) / kZeroPerBlock;
    if (blocks <= 0)
        return hipSuccess;
    const dim3 grid((unsigned)blocks);
    if (head_dim == 128)
        hipLaunchKernelGGL((sparse_prep_kernel<128>), grid, dim3(256), 0, s, cap * hq, hq, cap,
                           n_sel_dev, sel_idx, q, o, dout, qc, ndelta, prep, zero, n_zero);
    else
        hipLaunchKernelGGL((sparse_prep_kernel<64>), grid, dim3(256), 0, s, cap * hq, hq, cap,
                           n_sel_dev, sel_idx, q, o, dout, qc, ndelta, prep, zero, n_zero);
    return hipGetLastError();
}

hipError_t launch_bwd_dq(int mode, int head_dim, const BwdArgs &a, int grid, hipStream_t s) {
    if (grid <= 0)
        return hipSuccess;
    if (head_dim == 128) {
        if (mode == kModeLocal)
            hipLaunchKernelGGL((bwd_dq_kernel<128, kModeLocal>), dim3(grid), dim3(256), 0, s, a);
        else
            hipLaunchKernelGGL((bwd_dq_kernel<128, kModeGlobal>), dim3(grid), dim3(256), 0, s, a);
    } else {
        if (mode == kModeLocal)
            hipLaunchKernelGGL((bwd_dq_kernel<64, kModeLocal>), dim3(grid), dim3(256), 0, s, a);
        else
            hipLaunchKernelGGL((bwd_dq_kernel<64, kModeGlobal>), dim3(grid), dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_bwd_dkv(int mode, int head_dim, const BwdArgs &a, int grid, hipStream_t s) {
    if (grid <= 0)
        return hipSuccess;
    if (head_dim == 128) {
        if (mode == kModeLocal)
            hipLaunchKernelGGL((bwd_dkv_kernel<128, kModeLocal>), dim3(grid), dim3(256), 0, s, a);
        else
            hipLaunchKernelGGL((bwd_dkv_kernel<128, kModeGlobal>), dim3(grid), dim3(256), 0, s, a);
    } else {
        if (mode == kModeLocal)
            hipLaunchKernelGGL((bwd_dkv_kernel<64, kModeLocal>), dim3(grid), dim3(256), 0, s, a);
        else
            hipLaunchKernelGGL((bwd_dkv_kernel<64, kModeGlobal>), dim3(grid), dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

int bwd_keys_per_block() { return kKeysPerWg; }

}  // namespace logo
