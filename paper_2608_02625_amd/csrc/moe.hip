// Mixture-of-experts routing for the refiner's FFN: router logits with
// softmax top-k, dispatch (per-expert row ranges + device tile table for the
// grouped GEMM) and the weighted combine back into the residual stream.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace {

// XOR key of the 16-byte chunks of a 128-byte LDS row: a fragment read of 32
// consecutive rows at one logical chunk hits distinct banks.
__device__ __forceinline__ int rkey(int row) { return (row & 7) ^ ((row >> 3) & 1); }

// Router logits z[t][e] = sum_c h[t][c] Wr[e][c], 64 tokens x 64 experts per
// workgroup (4 waves of 32x32) on v_mfma_f32_32x32x16_bf16.  K is cut into
// n_parts (2, 4 or 8) equal parts whose sums are added as a balanced tree,
// ((p0 + p1) + (p2 + p3)) + ..., so that the result has the same bits however
// the parts are spread over workgroups: blockIdx.z = s adds parts
// s * CH .. s * CH + CH - 1 and writes its subtree to out[s][T][E]; the top-k
// kernel adds the subtrees.
// A few hundred tokens would leave this to a handful of workgroups, each
// streaming all of Wr and walking d in one chain; with the parts on workgroups
// of their own the chain is n_parts times shorter.  Copies go global -> LDS (3
// stages of 64 columns), 48 KB, three workgroups per CU.
template <int CH>
__global__ __launch_bounds__(256) void router_logits_kernel(const bf16_t* __restrict__ h, const bf16_t* __restrict__ Wr,
                                                            int T, int d, int E, int part, float* __restrict__ out) {
    constexpr int NS = 3, BK = 64, ROW = BK * 2, HALF = 64 * ROW, STAGE = 2 * HALF;
    constexpr int NI = STAGE / 1024 / 4;             // 1 KB copies (8 rows) per wave and stage
    __shared__ __attribute__((aligned(16))) char smem[NS * STAGE];
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
    const int g = lane >> 5, j = lane & 31;
    const int t0 = blockIdx.x * 64, e0 = blockIdx.y * 64;
    const int k0 = blockIdx.z * CH * part;           // first column
    const int wt = wave >> 1, we = wave & 1;

    // Rows past T or E lie past the buffers' ranges: nothing is fetched for them.
    const buf_rsrc_t h_rsrc = make_rsrc(h + (int64_t)t0 * d, (int)min((int64_t)(T - t0) * d * 2, (int64_t)0x7fffffff));
    const buf_rsrc_t w_rsrc = make_rsrc(Wr + (int64_t)e0 * d, (E - e0) * d * 2);
    uint32_t off[NI];
#pragma unroll
    for (int p = 0; p < NI; ++p) {
        const int row = ((wave & 1) * NI + p) * 8 + lane / 8;     // waves 0, 1 copy token rows, 2, 3 expert rows
        off[p] = (uint32_t)(row * d * 2) + (uint32_t)(((lane % 8) ^ rkey(row)) * 16);
    }
    const lds_ptr_t lds = (lds_ptr_t)smem;
    typedef __attribute__((address_space(3))) char lds_char;
    typedef __attribute__((address_space(3))) const bf16x8 lds_frag;
    const int nk = CH * part / BK;
    auto issue = [&](int kt, int stage) {
        const int dst = stage * STAGE + wave * NI * 1024;
#pragma unroll
        for (int p = 0; p < NI; ++p)
            lds_dma16_buf(wave < 2 ? h_rsrc : w_rsrc, off[p], (k0 + kt * BK) * 2, (lds_ptr_t)((lds_char*)lds + dst + p * 1024));
    };
    f32x16 acc, tree[3];
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
    for (int l = 0; l < 3; ++l) tree[l] = acc;
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) issue(min(s, nk - 1), s);
    const int ha = (wt * 32 + j) * ROW, wa = HALF + (we * 32 + j) * ROW, key = rkey(j);
    const int per = part / BK;                       // K tiles per part
    int stage = 0, kt = 0;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        for (int q = 0; q < per; ++q, ++kt) {
            wait_vmcnt<NI * (NS - 2)>();             // own copies of K tile kt landed
            lds_barrier();                           // everyone's; the stage of K tile kt - 1 is free
            issue(min(kt + NS - 1, nk - 1), (stage + NS - 1) % NS);
            const int sb = stage * STAGE;
            stage = (stage + 1) % NS;
#pragma unroll
            for (int ks = 0; ks < BK / 16; ++ks) {
                const int co = ((2 * ks + g) ^ key) << 4;
                const bf16x8 hf = *(lds_frag*)((lds_char*)lds + sb + ha + co);
                const bf16x8 wf = *(lds_frag*)((lds_char*)lds + sb + wa + co);
                acc = mfma32x32x16(hf, wf, acc);
            }
        }
        // part c done: add the subtrees that end with it
        f32x16 v = acc;
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            if (((c >> l) & 1) == 0) {
                tree[l] = v;
                break;
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] += tree[l][e];
        }
        if (c == CH - 1) {
            // v[e]: token 8*(e/4) + 4*g + e%4 of the wave's 32, expert j
            const int ex = e0 + we * 32 + j;
            float* o = out + (int64_t)blockIdx.z * T * E;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int t = t0 + wt * 32 + 8 * (e >> 2) + 4 * g + (e & 3);
                if (t < T && ex < E) o[(int64_t)t * E + ex] = v[e];
            }
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    }
    wait_all_memory();                               // no copy may still land in LDS when the workgroup ends
}

// Largest of the wave's 64 unsigned values, on DPP lane moves.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
    auto step = [&](uint32_t o) { v = o > v ? o : v; };
    step((uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xF, 0xF, false));    // quad_perm [1,0,3,2]
    step((uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xF, 0xF, false));    // quad_perm [2,3,0,1]
    step((uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x141, 0xF, 0xF, false));   // row_half_mirror
    step((uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x140, 0xF, 0xF, false));   // row_mirror
    step((uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x142, 0xA, 0xF, false));   // row_bcast:15 into rows 1, 3
    step((uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x143, 0xC, 0xF, false));   // row_bcast:31 into rows 2, 3
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
#else
    return v;
#endif
}
__device__ __forceinline__ float lane_value(float v, int lane) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
#else
    return v;
#endif
}

// Softmax top-k of group_tokens tokens per workgroup (8 waves, one token per
// wave at a time; lane l owns experts l + 64q, E <= 64 NQ).  The logits are the
// tree sum of n_split subtrees.  A NaN logit counts as -inf, so that the order
// is total and every token receives exactly k distinct experts whatever its
// input.  Selections are taken one by one, the largest logit with ties to the
// lower id: the maximum of order-preserving keys over the wave, then the first
// owner of that key (a ballot per expert block): k maxima of about 25
// instructions each, where ranking every expert takes E compares per expert
// owned.  Bound by those instructions.  Logits + top-k + dispatch against one
// kernel of 32 tokens per workgroup that did both, us with each launch:
// 10240 tokens, 256 experts, d 4096: 57 + 21 + 14 against 228 + 100; 640
// tokens, 64 experts, d 2048: 6.2 + 6.2 + 6.7 against 21.5 + 7.2; 32768 tokens:
// 40 + 29 + 14 against 84 + 114.
// Lane r < k records selection r with its rank among this workgroup's
// selections of the same expert (LDS counter), and the workgroup's per-expert
// counts go to wg_counts[E][workgroup].  Ranks only order rows inside an
// expert's group.
template <int NQ>
__global__ __launch_bounds__(512) void router_topk_kernel(const float* __restrict__ parts, int n_split, int T, int E, int k,
                                                           int group_tokens, int32_t* __restrict__ ids,
                                                           float* __restrict__ wts, int32_t* __restrict__ pos,
                                                           int32_t* __restrict__ wg_counts, float* __restrict__ logits) {
    __shared__ int lcnt[64 * NQ];
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
    for (int e = threadIdx.x; e < 64 * NQ; e += 512) lcnt[e] = 0;
    __syncthreads();
    const int t_end = min((int)(blockIdx.x + 1) * group_tokens, T);
    const int64_t stride = (int64_t)T * E;
    for (int t = blockIdx.x * group_tokens + wave; t < t_end; t += 8) {
        float z[NQ], p[NQ];
        uint32_t key[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int e = lane + 64 * q;
            const float* r = parts + (int64_t)t * E + min(e, E - 1);
            float v;
            if (n_split == 8)
                v = ((r[0] + r[stride]) + (r[2 * stride] + r[3 * stride])) +
                    ((r[4 * stride] + r[5 * stride]) + (r[6 * stride] + r[7 * stride]));
            else if (n_split == 4)
                v = (r[0] + r[stride]) + (r[2 * stride] + r[3 * stride]);
            else if (n_split == 2)
                v = r[0] + r[stride];
            else
                v = r[0];
            if (logits && e < E) logits[(int64_t)t * E + e] = v;   // test hook
            v = (e < E && v == v) ? v + 0.f : -INFINITY;           // (+0.f: -0 and +0 compare equal)
            z[q] = v;
            const uint32_t b = __float_as_uint(v);
            key[q] = e < E ? b ^ ((b >> 31) ? 0xffffffffu : 0x80000000u) : 0u;   // 0: below every logit's key
        }
        float m = z[0];
#pragma unroll
        for (int q = 1; q < NQ; ++q) m = fmaxf(m, z[q]);
        m = wave_max_dpp(m);
        float own = 0.f;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            p[q] = lane + 64 * q < E ? __expf(z[q] - m) : 0.f;
            own += p[q];
        }
        const float sum = wave_sum_dpp(own);
        int sel = 0;
        float w = 0.f;                               // lane r < k: exp(z - m) of selection r
        for (int r = 0; r < k; ++r) {
            uint32_t best = key[0];
#pragma unroll
            for (int q = 1; q < NQ; ++q) best = key[q] > best ? key[q] : best;
            best = wave_max_u32(best);
            // first owner of the key: the lowest block that holds it, then its
            // lowest lane (one of the ballots is not empty)
            unsigned long long b = __ballot(key[NQ - 1] == best);
            int qs = NQ - 1;
#pragma unroll
            for (int q = NQ - 2; q >= 0; --q) {
                const unsigned long long bq = __ballot(key[q] == best);
                qs = bq ? q : qs;
                b = bq ? bq : b;
            }
            const int l = (int)__builtin_ctzll(b);
            float pq = p[0];
#pragma unroll
            for (int q = 1; q < NQ; ++q) pq = q == qs ? p[q] : pq;
            const float pv = lane_value(pq, l);
#pragma unroll
            for (int q = 0; q < NQ; ++q) key[q] = (q == qs && lane == l) ? 0u : key[q];
            sel = lane == r ? l + 64 * qs : sel;
            w = lane == r ? pv : w;
        }
        w /= sum;
        const float psum = wave_sum_dpp(w);
        if (lane < k) {
            const int64_t o = (int64_t)t * k + lane;
            ids[o] = sel;
            wts[o] = w / psum;
            pos[o] = atomicAdd(&lcnt[sel], 1);
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += 512) wg_counts[(int64_t)e * gridDim.x + blockIdx.x] = lcnt[e];
}

// Exclusive scan of n <= 512 non-negative ints held in LDS, by one wave;
// out[n] receives the total.
__device__ void wave_scan512(const int* in, int* out, int n) {
    const int lane = threadIdx.x & 63;
    int v[8], run = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int idx = lane * 8 + i;
        v[i] = idx < n ? in[idx] : 0;
        run += v[i];
    }
    int incl = run;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(incl, off, 64);
        if (lane >= off) incl += o;
    }
    int excl = incl - run;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int idx = lane * 8 + i;
        if (idx < n) out[idx] = excl;
        excl += v[i];
    }
    if (lane == 63) out[n] = incl;
}

// Dispatch: one workgroup per router workgroup w (its group_tokens tokens).
// Each workgroup derives from the per-expert counts wg_counts[E][nwg] what it
// needs itself: every group's size (all routed experts, then n_shared shared
// experts of T rows) and, per expert, how many of that expert's selections come
// from router workgroups before w (1024 / (64 NQ) threads per expert row, E <=
// 64 NQ, consecutive threads on consecutive counts, 16 loads at a time).
// Workgroup 0 also writes grp_off, the tile table of the grouped GEMM (entries
// as at kRasterBand) and its length.  The selections of the workgroup's tokens
// then get their rows: slot (in place of the rank) = grp_off[e] + those before w
// + rank, a_rows[slot] = token.  No workgroup waits for another; every one reads
// the whole table, so the host makes the groups large enough to keep it small
// (router_group_tokens).
template <int NQ>
__global__ __launch_bounds__(1024) void dispatch_kernel(const int32_t* __restrict__ ids, int T, int k, int E,
                                                       int n_shared, int nwg, int group_tokens, int bm,
                                                       const int32_t* __restrict__ wg_counts,
                                                       int32_t* __restrict__ grp_off, int2* __restrict__ tile_tab,
                                                       int32_t* __restrict__ n_tiles, int32_t* __restrict__ slot,
                                                       int32_t* __restrict__ a_rows) {
    __shared__ int tot[512], before[512], off[513], ntl[512], toff[513];
    const int w = blockIdx.x, G = E + n_shared;
    constexpr int TPR = 16 / NQ;                     // threads per expert row
    const int wave = threadIdx.x >> 6, q = threadIdx.x % TPR, e = threadIdx.x / TPR;
    int s_all = 0, s_pre = 0;
    if (e < E) {
        const int32_t* col = wg_counts + (int64_t)e * nwg;
        for (int v0 = q; v0 < nwg; v0 += 16 * TPR) {
            int c[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) c[u] = v0 + u * TPR < nwg ? col[v0 + u * TPR] : 0;
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                s_all += c[u];
                if (v0 + u * TPR < w) s_pre += c[u];
            }
        }
    }
#pragma unroll
    for (int o = 1; o < TPR; o <<= 1) {
        s_all += __shfl_xor(s_all, o, 64);
        s_pre += __shfl_xor(s_pre, o, 64);
    }
    if (e < E && q == 0) {
        tot[e] = s_all;
        before[e] = s_pre;
    }
    for (int gi = E + threadIdx.x; gi < G; gi += blockDim.x) tot[gi] = T;
    __syncthreads();
    for (int gi = threadIdx.x; gi < G; gi += blockDim.x) ntl[gi] = (tot[gi] + bm - 1) / bm;
    __syncthreads();
    if (wave == 0) wave_scan512(tot, off, G);
    else if (wave == 1) wave_scan512(ntl, toff, G);
    __syncthreads();
    if (w == 0) {
        for (int gi = threadIdx.x; gi <= G; gi += blockDim.x) grp_off[gi] = off[gi];
        if (threadIdx.x == 0) *n_tiles = toff[G];
        for (int gi = threadIdx.x; gi < G; gi += blockDim.x)
            for (int t = 0; t < ntl[gi]; ++t) {
                const int pos = t % kRasterBand, size = min(ntl[gi] - (t - pos), kRasterBand);
                // equal heights, in steps of 32 rows, that fit the group in its tiles
                const int height = ((tot[gi] + ntl[gi] - 1) / ntl[gi] + 31) & ~31;
                tile_tab[toff[gi] + t] = make_int2(gi | pos << 10 | size << 16 | (height >> 5) << 22, t * height);
            }
    }
    const int t0 = w * group_tokens;
    const int nt = min(group_tokens, T - t0);
    for (int il = threadIdx.x; il < nt * k; il += blockDim.x) {
        const int64_t i = (int64_t)t0 * k + il;
        const int ei = ids[i];
        const int sr = off[ei] + before[ei] + slot[i];
        slot[i] = sr;
        a_rows[sr] = t0 + il / k;
    }
    for (int il = threadIdx.x; il < nt * n_shared; il += blockDim.x) {
        const int t = t0 + il % nt, sh = il / nt;
        a_rows[off[E + sh] + t] = t;
    }
}

// x[t] += sum_j w[t][j] * Y[slot[t][j]] + sum_s Y[grp_off[E+s] + t], fixed order.
// With g_next, also the next block's input norm h[t] = bf16(x[t] / rms * g_next)
// (the same arithmetic, in the same order, as the stand-alone RMSNorm).
// NR = k + n_shared rows per token, a compile-time count so that all of a
// token's row loads are issued before the first is used.
template <int NR>
__global__ void combine_kernel(float* __restrict__ x, const bf16_t* __restrict__ Y,
                               const int32_t* __restrict__ slot, const float* __restrict__ w,
                               const int32_t* __restrict__ grp_off, int k, int E, int n_shared,
                               int d, const bf16_t* __restrict__ g_next, bf16_t* __restrict__ h_next, float eps,
                               int map_S, int map_P, int map_D) {
    const int t = blockIdx.x;
    const int64_t xrow = map_D > 0 ? (int64_t)(t / map_D) * map_S + map_P + t % map_D : t;
    int rows[NR];
    float wt[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        if (r < k) {
            rows[r] = slot[(int64_t)t * k + r];
            wt[r] = w[(int64_t)t * k + r];
        } else {
            rows[r] = grp_off[E + (r - k)] + t;
            wt[r] = 1.f;
        }
    }
    float* xr = x + xrow * d;
    float ss = 0.f;
    for (int i = threadIdx.x * 8; i < d; i += blockDim.x * 8) {
        u32x4 y[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) y[r] = *reinterpret_cast<const u32x4*>(Y + (int64_t)rows[r] * d + i);
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const float c = wt[r];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                acc[2 * q] += c * __uint_as_float(y[r][q] << 16);
                acc[2 * q + 1] += c * __uint_as_float(y[r][q] & 0xffff0000u);
            }
        }
        f32x4 a = *reinterpret_cast<const f32x4*>(xr + i);
        f32x4 b = *reinterpret_cast<const f32x4*>(xr + i + 4);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            a[q] += acc[q];
            b[q] += acc[q + 4];
        }
        *reinterpret_cast<f32x4*>(xr + i) = a;
        *reinterpret_cast<f32x4*>(xr + i + 4) = b;
        ss += a[0] * a[0] + a[1] * a[1] + a[2] * a[2] + a[3] * a[3];
        ss += b[0] * b[0] + b[1] * b[1] + b[2] * b[2] + b[3] * b[3];
    }
    if (g_next) rms_store_row(xr, g_next, h_next + (int64_t)t * d, d, block_rms_scale(ss, d, eps));
}

}  // namespace

int router_parts(int d) { return d % 512 == 0 ? 8 : d % 256 == 0 ? 4 : 2; }

// Enough workgroups for two per CU; more only adds partial logits to write and
// read back.
int router_splits(int T, int d, int E, int64_t capacity) {
    const int64_t wgs = (int64_t)((T + 63) / 64) * ((E + 63) / 64);
    int n = router_parts(d);
    while (n > 1 && (wgs * n > 512 || (int64_t)n * T * E * 4 > capacity)) n >>= 1;
    return n;
}

// The top-k of a token is about 2000 cycles of a SIMD, so small groups spread
// it, but the dispatch workgroups each read all groups' counts: at most 256
// groups.  top-k + dispatch, us with each launch (5.9): 640 tokens of 64 experts
// in groups of 8 (what run_layer asks for) 6.2 + 6.7, of 16 7.5 + 6.6, of 32 (its
// fallback) 10.8 + 6.6; 5120 tokens of 64 experts in 128 / 256 / 512 groups 12.6 +
// 7.8 / 9.5 + 8.2 / 9.6 + 9.5; 32768 in 128 / 256 / 512 / 1024 53 + 14 / 29 + 14 /
// 24 + 14 / 22 + 23; 10240 tokens of 256 experts 37 + 11 / 21 + 14 / 18 + 26 / 17 +
// 60.
int router_group_tokens(int T, int least) {
    const int64_t n = ((int64_t)T + least - 1) / least;
    return least * (int)((n + 255) / 256);
}

hipError_t launch_router_logits(const bf16_t* h, const bf16_t* Wr, int T, int d, int E, int n_split, float* parts,
                                hipStream_t st) {
    if (E < 1 || E > 256 || d % 128 != 0 || T < 1) return hipErrorInvalidValue;
    const int np = router_parts(d);
    if (n_split < 1 || np % n_split != 0) return hipErrorInvalidValue;
    const dim3 grid((T + 63) / 64, (E + 63) / 64, n_split);
#define ROUTER_CASE(CH)                                                                                       \
    case CH:                                                                                                  \
        hipLaunchKernelGGL(router_logits_kernel<CH>, grid, dim3(256), 0, st, h, Wr, T, d, E, d / np, parts); \
        break;
    switch (np / n_split) {
        ROUTER_CASE(1)
        ROUTER_CASE(2)
        ROUTER_CASE(4)
        ROUTER_CASE(8)
        default:
            return hipErrorInvalidValue;
    }
#undef ROUTER_CASE
    return hipGetLastError();
}

hipError_t launch_router_topk(const float* parts, int n_split, int T, int E, int k, int group_tokens, int32_t* ids, float* w,
                              int32_t* pos, int32_t* wg_counts, hipStream_t st, float* logits) {
    if (group_tokens < 1 || E < 1 || E > 256 || k < 1 || k > 8 || k > E || T < 1) return hipErrorInvalidValue;
    if (n_split != 1 && n_split != 2 && n_split != 4 && n_split != 8) return hipErrorInvalidValue;
    const int gt = group_tokens;
    const dim3 grid((T + gt - 1) / gt), block(512);
    if (E <= 64)
        hipLaunchKernelGGL(router_topk_kernel<1>, grid, block, 0, st, parts, n_split, T, E, k, gt, ids, w, pos, wg_counts,
                           logits);
    else if (E <= 128)
        hipLaunchKernelGGL(router_topk_kernel<2>, grid, block, 0, st, parts, n_split, T, E, k, gt, ids, w, pos, wg_counts,
                           logits);
    else
        hipLaunchKernelGGL(router_topk_kernel<4>, grid, block, 0, st, parts, n_split, T, E, k, gt, ids, w, pos, wg_counts,
                           logits);
    return hipGetLastError();
}

hipError_t launch_dispatch(const int32_t* ids, int T, int k, int E, int n_shared, int group_tokens, int bm,
                           const int32_t* wg_counts, int32_t* grp_off, int2* tile_tab, int32_t* n_tiles,
                           int32_t* slot, int32_t* a_rows, hipStream_t st) {
    if (E + n_shared > 512 || group_tokens < 1) return hipErrorInvalidValue;
    const int gt = group_tokens, nwg = (T + gt - 1) / gt;
    auto* kernel = E <= 64 ? dispatch_kernel<1> : E <= 128 ? dispatch_kernel<2> : dispatch_kernel<4>;
    hipLaunchKernelGGL(kernel, dim3(nwg), dim3(1024), 0, st, ids, T, k, E, n_shared, nwg, gt, bm, wg_counts, grp_off,
                       tile_tab, n_tiles, slot, a_rows);
    return hipGetLastError();
}

void launch_combine(float* x, const bf16_t* Y, const int32_t* slot, const float* w,
                    const int32_t* grp_off, int T, int k, int E, int n_shared, int d, const bf16_t* g_next,
                    bf16_t* h_next, float eps, hipStream_t st, int map_S, int map_P, int map_D) {
    const int nr = k + std::min(n_shared, 9 - k);
#define COMBINE_CASE(N)                                                                                    \
    case N:                                                                                                \
        hipLaunchKernelGGL(combine_kernel<N>, dim3(T), dim3(256), 0, st, x, Y, slot, w, grp_off, k, E, n_shared, d, \
                           g_next, h_next, eps, map_S, map_P, map_D);                                      \
        break;
    switch (nr) {
        COMBINE_CASE(1)
        COMBINE_CASE(2)
        COMBINE_CASE(3)
        COMBINE_CASE(4)
        COMBINE_CASE(5)
        COMBINE_CASE(6)
        COMBINE_CASE(7)
        COMBINE_CASE(8)
        COMBINE_CASE(9)
        default:
            break;
    }
#undef COMBINE_CASE
}
