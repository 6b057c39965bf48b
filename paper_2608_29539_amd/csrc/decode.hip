// decode.hip -- one autoregressive decoding step of the layer (Sec. 3.3 and
// App. B, Autoregressive Decoding).  Each of B sequences appends one token
// whose key and value are already the last row of its cache.  The token's
// query attends to the last min(L, w) cached keys (local branch); when its
// gate passes the threshold it also attends to the whole cache (global
// branch), and the two outputs are ContextNorm-ed and fused as in the layer.
//
// Only selected tokens do global work: every global work item tests its
// sequence's routing decision z_b = gate[b] > thr (fp32, strict) and an
// unselected one exits at once, so an unselected token costs one window of
// the cache (the paper's batched decoding instead launches the dense kernel
// for every row and masks).
//
//   decode_attn_kernel    split-KV attention, one workgroup per (branch,
//                         sequence, KV head, head group, chunk of keys):
//                         the GH query heads of one KV head share every K/V
//                         row read, sixteen lanes (one DPP row) cover one
//                         2d-byte row, and each of the 16 streams keeps two
//                         rows in flight.  Writes the chunk's unnormalised
//                         (O, m, l) per head.  One extra workgroup writes
//                         the compacted list of selected sequences and the
//                         count, where the caller asks for either.
//   decode_combine_kernel merges the chunks of each (sequence, head) in chunk
//                         order, applies ContextNorm to each branch and the
//                         fusion, and rounds once to bf16.
//
// The cache is read once per branch (HBM-bound); the arithmetic is fp32
// (bf16 dot products accumulate in fp32 with v_dot2), so no MFMA is needed.
#include "logo_internal.h"

namespace logo {
namespace {

constexpr int kDecThreads = 256;
constexpr int kLanesPerRow = 16;            // lanes that share one cached K / V row
constexpr int kStreams = kDecThreads / kLanesPerRow;   // keys per workgroup step
constexpr int kPrefetch = 2;                // rows in flight per stream
constexpr float kNegInfD = -__builtin_inff();
constexpr float kLazyD = 8.f;               // exp2-domain headroom of the running max

typedef uint32_t u32x4d __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2d __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// One lane's slice of a cached row: N 32-bit words (one 16- or 8-byte load).
// A struct rather than a dependent-size ext_vector_type: element reads of
// such a vector passed by value into a lambda compiled to element 0.
template <int N>
struct alignas(4 * N) Words {
    uint32_t w[N];
};

// Sum over the 16 lanes of a DPP row, returned in every lane: rotations by 8
// and 4 within the row, then the two quad swaps.
template <int Ctrl>
__device__ __forceinline__ float dpp_f(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), Ctrl, 0xF, 0xF, false));
}
__device__ __forceinline__ float row16_sum(float x) {
    x += dpp_f<0x128>(x);   // row_ror:8
    x += dpp_f<0x124>(x);   // row_ror:4
    x += dpp_f<0x4E>(x);    // quad_perm [2,3,0,1]
    x += dpp_f<0xB1>(x);    // quad_perm [1,0,3,2]
    return x;
}

// The token's routing decision z_b = gate[b] > thr (fp32, strict: a NaN
// gate or threshold selects nothing), taken identically by every workgroup
// that needs it.
__device__ __forceinline__ float decode_threshold(const DecodeArgs &a) {
    return a.sel_mode == 2 ? a.thr_dev[0] : a.thr_host;
}

// The compacted list of selected sequences (ascending) and the count, each
// where it is asked for: one workgroup, ballot + mbcnt ranks and a carry over
// chunks of kDecThreads sequences.
__device__ void build_active_list(const DecodeArgs &a) {
    __shared__ int s_cnt[kDecThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float thr = decode_threshold(a);
    int carry = 0;
    for (int c0 = 0; c0 < a.num_seqs; c0 += kDecThreads) {
        const int b = c0 + tid;
        const bool z = b < a.num_seqs && a.gate[b] > thr;
        const uint64_t m = __ballot(z);
        const int below = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                        __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
        if (lane == 0)
            s_cnt[wave] = (int)__popcll(m);
        __syncthreads();
        int before = carry, total = 0;
        for (int i = 0; i < kDecThreads / 64; i++) {
            if (i < wave)
                before += s_cnt[i];
            total += s_cnt[i];
        }
        if (z && a.act)
            a.act[before + below] = b;
        carry += total;
        __syncthreads();                         // s_cnt is rewritten by the next chunk
    }
    if (tid == 0 && a.n_act)
        a.n_act[0] = carry;
}

// (m, l, acc) of stream b merged into stream a (exp2 domain).
__device__ __forceinline__ void merge_into(float &ma, float &la, float &mb, float &lb, float *aa,
                                           const float *ab, int n) {
    const float M = fmaxf(ma, mb);
    const float Mc = M == kNegInfD ? 0.f : M;
    const float fa = __builtin_amdgcn_exp2f(ma - Mc), fb = __builtin_amdgcn_exp2f(mb - Mc);
    la = la * fa + lb * fb;
    for (int i = 0; i < n; i++)
        aa[i] = aa[i] * fa + ab[i] * fb;
    ma = M;
}

template <int D, int GH>
__global__ __launch_bounds__(kDecThreads) void decode_attn_kernel(const DecodeArgs a) {
    constexpr int DE = D / kLanesPerRow;  // d values per lane
    constexpr int DW = DE / 2;            // 32-bit words per lane (2 bf16 each)
    typedef Words<DW> frag_t;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int e = lane % kLanesPerRow, sid = tid / kLanesPerRow;

    // work item -> (branch, sequence, kv head, head group, chunk); the
    // workgroup past them builds the list of selected sequences instead
    const int per_row = a.hkv * a.nhg;
    int item = blockIdx.x;
    if (item == a.n_local_items + a.n_global_items) {
        build_active_list(a);
        return;
    }
    const bool global = item >= a.n_local_items;
    if (global)
        item -= a.n_local_items;
    const int nch = global ? a.chunks_global : a.chunks_local;
    const int c = item % nch;
    const int rest = item / nch;
    const int hgi = rest % a.nhg;
    const int kvh = (rest / a.nhg) % a.hkv;
    const int b = rest / per_row;                // sequence
    if (global && !(a.gate[b] > decode_threshold(a)))
        return;                                  // an unselected token: window only
    const int64_t base = a.cu[b];
    const int L = a.cu[b + 1] - (int)base;
    const int lo = global ? 0 : max(0, L - a.window);
    const int k0 = lo + c * a.kc;
    const int k1 = min(L, k0 + a.kc);
    if (k0 >= k1)
        return;                                  // a chunk past this sequence's keys
    // this item's partials: acc [item][GH][D], then all items' m, l
    float *out_part = (global ? a.part_global : a.part_local) + (int64_t)item * GH * D;
    float *out_ml = (global ? a.part_global + (int64_t)a.n_global_items * GH * D
                            : a.part_local + (int64_t)a.n_local_items * GH * D) +
                    (int64_t)item * GH * 2;
    const uint16_t *kc_ = global ? a.k_g : a.k;
    const uint16_t *vc_ = global ? a.v_g : a.v;
    const uint16_t *qv = global ? a.q_g : a.q;
    const int h0 = kvh * a.group + hgi * GH;     // first query head of the group

    // Query slices (bf16 pairs) of the GH heads.
    uint32_t q2[GH][DW];
#pragma unroll
    for (int hh = 0; hh < GH; hh++) {
        const uint32_t *qp = (const uint32_t *)(qv + ((int64_t)b * a.hq + h0 + hh) * D + e * DE);
#pragma unroll
        for (int i = 0; i < DW; i++)
            q2[hh][i] = qp[i];
    }
    float m[GH], l[GH], acc[GH][DE];
#pragma unroll
    for (int hh = 0; hh < GH; hh++) {
        m[hh] = kNegInfD;
        l[hh] = 0.f;
#pragma unroll
        for (int i = 0; i < DE; i++)
            acc[hh][i] = 0.f;
    }

    const int64_t row_stride = (int64_t)a.hkv * D;    // elements between cached tokens
    const uint16_t *kbase = kc_ + (base * a.hkv + kvh) * (int64_t)D + e * DE;
    const uint16_t *vbase = vc_ + (base * a.hkv + kvh) * (int64_t)D + e * DE;
    auto load_row = [&](const uint16_t *p, int j) {
        return *(const frag_t *)(p + (int64_t)j * row_stride);
    };
    // Online softmax update with key row (kw, vw).
    auto consume = [&](const frag_t kw, const frag_t vw) {
        float s[GH];
#pragma unroll
        for (int hh = 0; hh < GH; hh++) {
            float d0 = 0.f;
#pragma unroll
            for (int i = 0; i < DW; i++)
                d0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2d, q2[hh][i]),
                                                    __builtin_bit_cast(bf16x2d, kw.w[i]), d0, false);
            s[hh] = row16_sum(d0) * a.scale_log2;
        }
        float vf[DE];
#pragma unroll
        for (int i = 0; i < DW; i++) {
            vf[2 * i] = bf16_lo(vw.w[i]);
            vf[2 * i + 1] = bf16_hi(vw.w[i]);
        }
#pragma unroll
        for (int hh = 0; hh < GH; hh++) {
            if (s[hh] > m[hh] + kLazyD) {
                // the running max moves (always on the first key)
                const float alpha = __builtin_amdgcn_exp2f(m[hh] - s[hh]);
                l[hh] *= alpha;
#pragma unroll
                for (int i = 0; i < DE; i++)
                    acc[hh][i] *= alpha;
                m[hh] = s[hh];
            }
            const float p = __builtin_amdgcn_exp2f(s[hh] - m[hh]);
            l[hh] += p;
#pragma unroll
            for (int i = 0; i < DE; i++)
                acc[hh][i] = fmaf(p, vf[i], acc[hh][i]);
        }
    };

    // Each stream (16 lanes) walks keys k0 + sid, k0 + sid + kStreams, ...,
    // with kPrefetch rows in flight in a ring of registers (the ring index is
    // a compile-time constant: the loop body covers kPrefetch keys).
    int j = k0 + sid;
    frag_t kr[kPrefetch], vr[kPrefetch];
#pragma unroll
    for (int p = 0; p < kPrefetch; p++) {
        const int jp = j + p * kStreams;
        if (jp < k1) {
            kr[p] = load_row(kbase, jp);
            vr[p] = load_row(vbase, jp);
        }
    }
    for (; j < k1; j += kPrefetch * kStreams) {
#pragma unroll
        for (int p = 0; p < kPrefetch; p++) {
            const int jc = j + p * kStreams;
            if (jc < k1) {
                const frag_t kw = kr[p], vw = vr[p];
                const int jn = jc + kPrefetch * kStreams;
                if (jn < k1) {
                    kr[p] = load_row(kbase, jn);
                    vr[p] = load_row(vbase, jn);
                }
                consume(kw, vw);
            }
        }
    }

    // Merge the streams of the wave (lanes with the same e), then the waves.
#pragma unroll
    for (int hh = 0; hh < GH; hh++) {
#pragma unroll
        for (int sh = kLanesPerRow; sh < 64; sh <<= 1) {
            float mo = __shfl_xor(m[hh], sh, 64), lo_ = __shfl_xor(l[hh], sh, 64);
            float ao[DE];
#pragma unroll
            for (int i = 0; i < DE; i++)
                ao[i] = __shfl_xor(acc[hh][i], sh, 64);
            merge_into(m[hh], l[hh], mo, lo_, acc[hh], ao, DE);
        }
    }
    __shared__ float s_m[4][GH], s_l[4][GH];
    __shared__ float s_acc[4][GH][D];
    if (lane < kLanesPerRow) {
#pragma unroll
        for (int hh = 0; hh < GH; hh++) {
            if (lane == 0) {
                s_m[wave][hh] = m[hh];
                s_l[wave][hh] = l[hh];
            }
#pragma unroll
            for (int i = 0; i < DE; i++)
                s_acc[wave][hh][e * DE + i] = acc[hh][i];
        }
    }
    __syncthreads();
    // thread t < GH * D: head t / D, element t % D
    for (int t = tid; t < GH * D; t += kDecThreads) {
        const int hh = t / D, x = t % D;
        float M = s_m[0][hh], Lw = s_l[0][hh], A = s_acc[0][hh][x];
        for (int w2 = 1; w2 < 4; w2++) {
            float mb = s_m[w2][hh], lb = s_l[w2][hh];
            const float ab = s_acc[w2][hh][x];
            merge_into(M, Lw, mb, lb, &A, &ab, 1);
        }
        out_part[t] = A;
        if (x == 0) {
            out_ml[2 * hh] = M;
            out_ml[2 * hh + 1] = Lw;
        }
    }
}

// WPH waves per (sequence, query head), four waves per workgroup.  A branch's
// chunks are merged in one pass: the largest chunk maximum first (lane c of
// every wave holds chunks c and c + 64), then every chunk's weight
// 2^(m_c - M), then the weighted sum, in which the head's threads are 4 WPH
// chunk groups x 16 element groups (chunks cg, cg + 4 WPH, ..., D/16 elements
// in 16-byte loads), so a thread's chain is that share of the chunks; shuffles
// add a wave's four groups, LDS the waves.  Bound by the latency of that
// chain: with WPH = 4 the merge of 64 chunks (16 caches of 32K tokens, two
// selected, 32 heads of d = 128) takes 7.4 us, with one wave per head and
// 4-byte loads 8.7; with a few chunks per cache the one wave is the faster (a step of
// 64 caches of 2K tokens 82.0 against 84.4 us), so the launcher takes WPH = 4
// above 16 chunks.  At most 128 chunks per branch.
constexpr int kMaxChunks = 128;

constexpr int kWideMergeChunks = 16;

template <int D, int WPH>
__global__ __launch_bounds__(256) void decode_combine_kernel(const DecodeArgs a) {
    constexpr int EL = D / 16;                    // elements per thread
    typedef float f32x4c __attribute__((ext_vector_type(4)));
    __shared__ float s_w[4][2][kMaxChunks];
    __shared__ __attribute__((aligned(16))) float s_o[2][4][D];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int cg = (wave % WPH) * 4 + (lane >> 4), eg = lane & 15;
    const int job = blockIdx.x * (4 / WPH) + wave / WPH;
    if (WPH == 1 && job >= a.num_seqs * a.hq)
        return;                                   // whole wave: no barrier below
    const int b = job / a.hq, h = job % a.hq;
    const int L = a.cu[b + 1] - a.cu[b];
    // chunks of this sequence (clamped to the planned slots: max_seqlen bounds L)
    const int n_loc = min((min(L, a.window) + a.kc - 1) / a.kc, a.chunks_local);
    const int n_glb = min((L + a.kc - 1) / a.kc, a.chunks_global);
    const float p = a.gate[b];
    const bool sel = p > decode_threshold(a);
    const int kvh = h / a.group, hg = (h % a.group) / a.gh, hh = (h % a.group) % a.gh;
    // This wave's share of one branch's sum of 2^(m_c - M) O_c, in A (every
    // chunk group's lanes) and, for several waves, in s_o; returns the sum of
    // the weighted l (the same in every thread).
    auto branch = [&](int br, const float *parts, int64_t n_items, int nch, int chunks_stride,
                      float (&A)[EL]) {
        const int64_t item0 = (((int64_t)b * a.hkv + kvh) * a.nhg + hg) * chunks_stride;
        const float *acc = parts + (item0 * a.gh + hh) * D + eg * EL;
        const float *ml = parts + n_items * a.gh * D + (item0 * a.gh + hh) * 2;
        float *w = s_w[wave][br];
        // the first kPre chunks' elements are loaded before the weights exist
        constexpr int kPre = 4, EV = EL / 4;
        f32x4c pre[kPre][EV];
#pragma unroll
        for (int j = 0; j < kPre; j++) {
            const int c = cg + j * 4 * WPH;
            const float *pp = acc + (int64_t)c * a.gh * D;
            if (c < nch)
#pragma unroll
                for (int i = 0; i < EV; i++)
                    pre[j][i] = *(const f32x4c *)(pp + 4 * i);
        }
        float mc[2], lc[2];
        float M = kNegInfD;
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const int c = lane + 64 * i;
            mc[i] = c < nch ? ml[(int64_t)c * a.gh * 2] : kNegInfD;
            lc[i] = c < nch ? ml[(int64_t)c * a.gh * 2 + 1] : 0.f;
            M = fmaxf(M, mc[i]);
        }
#pragma unroll
        for (int sh = 1; sh < 64; sh <<= 1)
            M = fmaxf(M, __shfl_xor(M, sh, 64));
        const float Mc = M == kNegInfD ? 0.f : M;
        float lsum = 0.f;
#pragma unroll
        for (int i = 0; i < 2; i++) {
            const int c = lane + 64 * i;
            const float wc = c < nch ? __builtin_amdgcn_exp2f(mc[i] - Mc) : 0.f;
            w[c] = wc;
            lsum = fmaf(wc, lc[i], lsum);
        }
#pragma unroll
        for (int sh = 1; sh < 64; sh <<= 1)
            lsum += __shfl_xor(lsum, sh, 64);
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int i = 0; i < EL; i++)
            A[i] = 0.f;
        auto add = [&](float wc, int i, const f32x4c v) {
#pragma unroll
            for (int e = 0; e < 4; e++)
                A[4 * i + e] = fmaf(wc, v[e], A[4 * i + e]);
        };
#pragma unroll
        for (int j = 0; j < kPre; j++) {
            const int c = cg + j * 4 * WPH;
            if (c < nch) {
                const float wc = w[c];
#pragma unroll
                for (int i = 0; i < EV; i++)
                    add(wc, i, pre[j][i]);
            }
        }
#pragma unroll 2
        for (int c = cg + kPre * 4 * WPH; c < nch; c += 4 * WPH) {
            const float wc = w[c];
            const float *pp = acc + (int64_t)c * a.gh * D;
#pragma unroll
            for (int i = 0; i < EV; i++)
                add(wc, i, *(const f32x4c *)(pp + 4 * i));
        }
#pragma unroll
        for (int i = 0; i < EL; i++) {
            A[i] += __shfl_xor(A[i], 16, 64);
            A[i] += __shfl_xor(A[i], 32, 64);
            if (WPH > 1 && lane < 16)
                s_o[br][wave][eg * EL + i] = A[i];
        }
        return lsum;
    };
    float ol[EL], og[EL];
    const float l_loc = branch(0, a.part_local, a.n_local_items, n_loc, a.chunks_local, ol);
    float l_glb = 0.f;
    if (sel)                                      // (every wave of the head)
        l_glb = branch(1, a.part_global, a.n_global_items, n_glb, a.chunks_global, og);
    if constexpr (WPH > 1)
        __syncthreads();
    if (wave % WPH != 0 || lane >= 16)
        return;
    // the row's D values in 16 lanes: O / l, ContextNorm
    auto norm = [&](int br, float lsum, const float *gain, float (&o)[EL]) {
        const float inv = lsum > 0.f ? 1.f / lsum : 0.f;
        float ss = 0.f;
#pragma unroll
        for (int i = 0; i < EL; i++) {
            [[maybe_unused]] const int x = eg * EL + i;
            if constexpr (WPH == 4)
                o[i] = (s_o[br][0][x] + s_o[br][1][x]) + (s_o[br][2][x] + s_o[br][3][x]);
            o[i] *= inv;
            ss = fmaf(o[i], o[i], ss);
        }
#pragma unroll
        for (int sh = 1; sh < 16; sh <<= 1)
            ss += __shfl_xor(ss, sh, 64);
        const float rn = 1.f / sqrtf(ss / (float)D + a.eps);
#pragma unroll
        for (int i = 0; i < EL; i++)
            o[i] = o[i] * rn * (gain ? gain[h * D + eg * EL + i] : 1.f);
    };
    norm(0, l_loc, a.gain_local, ol);
    if (sel) {
        norm(1, l_glb, a.gain_global, og);
#pragma unroll
        for (int i = 0; i < EL; i++)
            ol[i] = (1.f - p) * ol[i] + p * og[i];
    }
    uint16_t *op = a.out + ((int64_t)b * a.hq + h) * D + eg * EL;
#pragma unroll
    for (int i = 0; i < EL; i++)
        op[i] = __builtin_bit_cast(uint16_t, (__bf16)ol[i]);
}

template <int D, int GH>
hipError_t launch_attn_gh(const DecodeArgs &a, hipStream_t s) {
    const int grid = a.n_local_items + a.n_global_items + (a.act || a.n_act);   // + the list builder
    hipLaunchKernelGGL((decode_attn_kernel<D, GH>), dim3(grid), dim3(kDecThreads), 0, s, a);
    return hipGetLastError();
}

template <int D>
hipError_t launch_attn_d(const DecodeArgs &a, hipStream_t s) {
    if (a.gh == 4)
        return launch_attn_gh<D, 4>(a, s);
    if (a.gh == 2)
        return launch_attn_gh<D, 2>(a, s);
    return launch_attn_gh<D, 1>(a, s);
}

}  // namespace

hipError_t launch_decode(const DecodeArgs &a, hipStream_t s) {
    hipError_t e = a.head_dim == 128 ? launch_attn_d<128>(a, s) : launch_attn_d<64>(a, s);
    if (e != hipSuccess)
        return e;
    const int jobs = a.num_seqs * a.hq;
    const bool wide = a.chunks_global > kWideMergeChunks;
    const dim3 grid(wide ? jobs : (jobs + 3) / 4);
    if (a.head_dim == 128) {
        if (wide)
            hipLaunchKernelGGL((decode_combine_kernel<128, 4>), grid, dim3(256), 0, s, a);
        else
            hipLaunchKernelGGL((decode_combine_kernel<128, 1>), grid, dim3(256), 0, s, a);
    } else {
        if (wide)
            hipLaunchKernelGGL((decode_combine_kernel<64, 4>), grid, dim3(256), 0, s, a);
        else
            hipLaunchKernelGGL((decode_combine_kernel<64, 1>), grid, dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace logo
