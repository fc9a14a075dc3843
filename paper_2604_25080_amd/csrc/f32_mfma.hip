// The float32 path on CDNA4 matrix cores: GEMM and paged causal attention with the float32 MFMA
// 16x16x4 (a float32 multiply-add per term, the precision of the plain FMA kernels).
//
// One operand trick serves both.  An MFMA step multiplies four K terms, one per quarter of the
// wavefront; which four is free as long as both operands agree.  Lane quarter q therefore reads
// one float4 -- terms 16g + 4q .. 16g + 4q + 3 of its row -- and feeds it to four steps: 16-byte
// reads instead of 4-byte ones.  Every output element sees its K terms in the same order whatever
// the tile, so the tile choice never changes a result bit.
#include "kernels.h"
#include "cacheflow.h"

namespace cf {

typedef __attribute__((ext_vector_type(4))) float f32x4_t;

namespace {

__device__ __forceinline__ f32x4_t mfma4(float a, float b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

constexpr int GK = 32;                    // K per step: eight 16-byte chunks per LDS row

// acc[M,N] = A[M,K] * W[N,K]^T; block tile B x B, 4 wavefronts as 2x2, F x F fragments of 16x16
// each.  Bound by latency at the few-hundred-row, K = 256..688 sizes of a small float32 model: a
// K-step is 256 matrix cycles against ~1000 of memory latency, hence DEPTH K-steps in flight in
// registers; LDS rows are 128 bytes with the 16-byte chunk index XORed by the row.  96 rows through
// the projections of a 256-wide model: 48 -> 8 us a launch against the plain FMA kernel; 4000 rows
// through gate/up: 69 -> 17 us.
template <int EPI, int B, int DEPTH>
__global__ void __launch_bounds__(256)
gemm_f32_kernel(const float* __restrict__ A, const float* __restrict__ W, const float* __restrict__ W2,
                float* __restrict__ C, int M, int N, int K, int tiles_n) {
    constexpr bool SILU = EPI == EPI_SILU_MUL;
    constexpr int F = B / 32, LD = B / 32;                    // fragments per side; rows per thread
    constexpr int NB = SILU ? 2 : 1, TILE = B * GK;
    __shared__ __align__(16) float smem[2][(1 + NB) * TILE];
    const int m0 = blockIdx.x / tiles_n * B, n0 = blockIdx.x % tiles_n * B;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave >> 1) * (B / 2), wn = (wave & 1) * (B / 2);
    const int ld_row = tid >> 3, ld_c = tid & 7;
    const int fr = lane & 15, fq = lane >> 4;

    const float* pa[LD];
    const float* pb[LD];
    const float* pb2[LD];
    int lds_at[LD];
#pragma unroll
    for (int j = 0; j < LD; ++j) {
        const int r = ld_row + 32 * j;
        pa[j] = A + (int64_t)min(m0 + r, M - 1) * K;
        pb[j] = W + (int64_t)min(n0 + r, N - 1) * K;
        pb2[j] = SILU ? W2 + (int64_t)min(n0 + r, N - 1) * K : nullptr;
        lds_at[j] = r * GK + ((ld_c ^ (r & 7)) << 2);
    }
    f32x4_t ra[DEPTH][LD], rb[DEPTH][NB][LD];
    auto fetch = [&](int kt, f32x4_t (&xa)[LD], f32x4_t (&xb)[NB][LD]) {
        const int k = kt * GK + ld_c * 4;
        const bool in = k < K;                                // K is a multiple of 4
#pragma unroll
        for (int j = 0; j < LD; ++j) {
            const f32x4_t zero = {0.f, 0.f, 0.f, 0.f};
            xa[j] = in ? *reinterpret_cast<const f32x4_t*>(pa[j] + k) : zero;
            xb[0][j] = in ? *reinterpret_cast<const f32x4_t*>(pb[j] + k) : zero;
            if constexpr (SILU) xb[NB - 1][j] = in ? *reinterpret_cast<const f32x4_t*>(pb2[j] + k) : zero;
        }
    };
    auto stash = [&](float* buf, const f32x4_t (&xa)[LD], const f32x4_t (&xb)[NB][LD]) {
#pragma unroll
        for (int j = 0; j < LD; ++j) {
            *reinterpret_cast<f32x4_t*>(buf + lds_at[j]) = xa[j];
#pragma unroll
            for (int n = 0; n < NB; ++n) *reinterpret_cast<f32x4_t*>(buf + (1 + n) * TILE + lds_at[j]) = xb[n][j];
        }
    };
    // two chains per output, added at the end: half the dependent steps and a smaller rounding error
    f32x4_t acc[2][NB][F][F];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int i = 0; i < F; ++i)
#pragma unroll
                for (int j = 0; j < F; ++j) acc[h][n][i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    const int nk = (K + GK - 1) / GK;
    // register set t % DEPTH holds step t; steps past the end are zero and multiply nothing in
#pragma unroll
    for (int t = 0; t < DEPTH; ++t) fetch(t, ra[t], rb[t]);
    stash(smem[0], ra[0], rb[0]);
    fetch(DEPTH, ra[0], rb[0]);
    __syncthreads();
    for (int kt0 = 0; kt0 < nk; kt0 += DEPTH) {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            const int kt = kt0 + u;
            if (kt < nk) {                                    // the same for the whole workgroup
                const float* cur = smem[kt & 1];
                float* nxt = smem[(kt + 1) & 1];
#pragma unroll
                for (int g = 0; g < GK / 16; ++g) {
                    f32x4_t fa[F], fb[NB][F];
                    const int c = ((4 * g + fq) ^ (fr & 7)) << 2;  // fragment bases are multiples of 16 rows
#pragma unroll
                    for (int i = 0; i < F; ++i) {
                        fa[i] = *reinterpret_cast<const f32x4_t*>(cur + (wm + 16 * i + fr) * GK + c);
#pragma unroll
                        for (int n = 0; n < NB; ++n)
                            fb[n][i] = *reinterpret_cast<const f32x4_t*>(cur + (1 + n) * TILE + (wn + 16 * i + fr) * GK + c);
                    }
#pragma unroll
                    for (int s = 0; s < 4; ++s)
#pragma unroll
                        for (int n = 0; n < NB; ++n)
#pragma unroll
                            for (int i = 0; i < F; ++i)
#pragma unroll
                                for (int j = 0; j < F; ++j) acc[s & 1][n][i][j] = mfma4(fa[i][s], fb[n][j][s], acc[s & 1][n][i][j]);
                }
                constexpr int D = DEPTH;
                stash(nxt, ra[(u + 1) % D], rb[(u + 1) % D]);
                fetch(kt + 1 + D, ra[(u + 1) % D], rb[(u + 1) % D]);
                __syncthreads();
            }
        }
    }
    // accumulator register r of a fragment: row 4 * quarter + r, column lane % 16
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j) {
            const int gn = n0 + wn + 16 * j + fr;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int gm = m0 + wm + 16 * i + 4 * fq + r;
                if (gm < M && gn < N) {
                    float* o = C + (int64_t)gm * N + gn;
                    float v = acc[0][0][i][j][r] + acc[1][0][i][j][r];
                    if constexpr (EPI == EPI_ADD_F32) v += *o;
                    if constexpr (SILU) v = v / (1.0f + expf(-v)) * (acc[0][NB - 1][i][j][r] + acc[1][NB - 1][i][j][r]);
                    *o = v;
                }
            }
        }
}

template <int EPI>
void launch_f32(hipStream_t s, const float* A, const float* W, const float* W2, float* C, int M, int N, int K) {
    // 64x64 tiles once they give every CU a workgroup, else 32x32: four times the workgroups
    // (3600 rows, N 768: 26 us; at 1000 rows 10 us against 18 with the large tile)
    const int64_t tiles64 = (int64_t)((M + 63) / 64) * ((N + 63) / 64);
    if (tiles64 >= 256) {
        const int tn = (N + 63) / 64;
        gemm_f32_kernel<EPI, 64, 2><<<(unsigned)tiles64, 256, 0, s>>>(A, W, W2, C, M, N, K, tn);
    } else {
        const int tn = (N + 31) / 32;
        gemm_f32_kernel<EPI, 32, 4><<<(unsigned)((M + 31) / 32 * tn), 256, 0, s>>>(A, W, W2, C, M, N, K, tn);
    }
}

// Varlen causal attention over the float32 pages.  A workgroup takes 16 * NQ query rows of one work
// item and one head; its four wavefronts take the key pages in turn (page p goes to wavefront
// p % 4), each with its own running maximum, sum and output, merged through LDS at the end: at the
// sizes of a small model the launch has too few query blocks to fill the chip, so the keys of a
// block are what is spread.  Scores are computed transposed (S^T = K Q^T), which leaves them in the
// register layout that O^T = V^T P^T wants as its second operand; the V part of a page is already
// [head_dim][slot], so both K and V fragments are 16-byte reads straight from the page (no LDS: the
// wavefronts share no keys), one page ahead.  NQ = 2 halves the page reads per row, NQ = 1 doubles
// the workgroups; a row's result does not depend on it: keys past its position add exact zeros, whatever
// they hold (the test for that costs nothing measurable: a batch of 2.7 k rows 551 -> 535 us a call).
// What bounds it is the chain of pages of a long row: 2.7 k query rows over up to 2 k keys, 4 heads
// of 64: 6.0 ms -> 47 us a launch against the lane-per-key kernel; 64 rows: 240 -> 7 us.
template <int HD, int NQ>
__global__ void __launch_bounds__(256)
attention_f32_kernel(const float* __restrict__ q, float* __restrict__ out, const float* __restrict__ pool_layer,
                     const AttnWork* __restrict__ work, const int32_t* __restrict__ page_tables, int n_q_heads,
                     KvGeom g) {
    constexpr int ROWS = 16 * NQ, SUB = ATTN_BLOCK_ROWS / ROWS, G = HD / 16, PAD = 20;
    __shared__ __align__(16) float o_sh[4][ROWS][PAD];        // one 16-wide slice of head_dim at a time
    __shared__ float m_sh[4][ROWS], l_sh[4][ROWS];
    // the longest items are listed last: start with them
    const int blk = gridDim.x - 1 - blockIdx.x;
    const AttnWork w = work[blk / SUB];
    const int r0 = blk % SUB * ROWS;
    if (r0 >= w.n_rows) return;
    const int head = blockIdx.y, gk = head / (n_q_heads / g.n_kv_heads);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, fr = lane & 15, fq = lane >> 4;
    const int32_t* pt = page_tables + w.pt_off;
    const int n_keys = w.pos0 + min(r0 + ROWS, w.n_rows);     // keys the block's last row sees
    const int n_pages = (n_keys + CF_PAGE_TOKENS - 1) / CF_PAGE_TOKENS;

    f32x4_t qf[NQ][G];
    int qpos[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const int row = min(r0 + 16 * i + fr, w.n_rows - 1);  // padded rows repeat the last row
        qpos[i] = w.pos0 + row;
        const float* qrow = q + ((int64_t)(w.row0 + row) * n_q_heads + head) * HD;
#pragma unroll
        for (int t = 0; t < G; ++t) qf[i][t] = *reinterpret_cast<const f32x4_t*>(qrow + 16 * t + 4 * fq);
    }
    const int64_t k_off = (int64_t)gk * CF_PAGE_TOKENS * HD + fr * HD + 4 * fq;
    const int64_t v_off = (int64_t)g.n_kv_heads * CF_PAGE_TOKENS * HD + (int64_t)gk * HD * CF_PAGE_TOKENS +
                          fr * CF_PAGE_TOKENS + 4 * fq;
    f32x4_t kf[G], vf[G], kn[G], vn[G];
    auto fetch = [&](int p, f32x4_t (&k)[G], f32x4_t (&v)[G]) {
        const float* page = pool_layer + (int64_t)pt[min(p, n_pages - 1)] * g.page_elems;
#pragma unroll
        for (int t = 0; t < G; ++t) {
            k[t] = *reinterpret_cast<const f32x4_t*>(page + k_off + 16 * t);
            v[t] = *reinterpret_cast<const f32x4_t*>(page + v_off + 16 * t * CF_PAGE_TOKENS);
        }
    };
    f32x4_t o[NQ][G];
    float m_run[NQ], l_run[NQ];                                // running maximum times c, partial row sum
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        m_run[i] = -INFINITY;
        l_run[i] = 0.f;
#pragma unroll
        for (int t = 0; t < G; ++t) o[i][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    const float c = rsqrtf((float)HD) * 1.4426950408889634f;  // softmax in the log2 domain
    fetch(wave, kf, vf);
    for (int p = wave; p < n_pages; p += 4) {
        fetch(p + 4, kn, vn);
        const int key0 = p * CF_PAGE_TOKENS + 4 * fq;         // register r: key key0 + r
        if (p == n_pages - 1) {
            // slots past the last needed key may hold anything: zero them, 0 * NaN must not get in
#pragma unroll
            for (int t = 0; t < G; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) vf[t][r] = key0 + r < n_keys ? vf[t][r] : 0.f;
        }
        f32x4_t s[NQ], s2[NQ];                                // two chains, as in the GEMM
#pragma unroll
        for (int i = 0; i < NQ; ++i) s[i] = s2[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < G; ++t)
#pragma unroll
            for (int e = 0; e < 4; e += 2)
#pragma unroll
                for (int i = 0; i < NQ; ++i) {
                    s[i] = mfma4(kf[t][e], qf[i][t][e], s[i]);
                    s2[i] = mfma4(kf[t][e + 1], qf[i][t][e + 1], s2[i]);
                }
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
#pragma unroll
            for (int r = 0; r < 4; ++r) s[i][r] = key0 + r > qpos[i] ? -INFINITY : s[i][r] + s2[i][r];
            float mx = fmaxf(fmaxf(s[i][0], s[i][1]), fmaxf(s[i][2], s[i][3]));
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m_run[i], mx * c);
            const float m_use = m_new == -INFINITY ? 0.f : m_new;    // no visible key yet
            const float corr = __builtin_amdgcn_exp2f(m_run[i] - m_use);
            m_run[i] = m_new;
            float ps = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[i][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i][r], c, -m_use));
                ps += s[i][r];
            }
            l_run[i] = l_run[i] * corr + ps;
#pragma unroll
            for (int t = 0; t < G; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) o[i][t][r] *= corr;
        }
        // A page with keys that some row of the block does not see yet: their probabilities are zero, but
        // 0 * Inf or 0 * NaN must not get into that row.
        bool bad = false;
        if ((p + 1) * CF_PAGE_TOKENS - 1 > w.pos0 + r0) {
#pragma unroll
            for (int t = 0; t < G; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) bad |= !(fabsf(vf[t][r]) < INFINITY);
        }
        if (__builtin_amdgcn_ballot_w64(bad) == 0) {
#pragma unroll
            for (int t = 0; t < G; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < NQ; ++i) o[i][t] = mfma4(vf[t][e], s[i][e], o[i][t]);
        } else {
            // once per query row, with the keys past it out of V (a row is a column of the product)
#pragma unroll 1
            for (int row = 0; row < 16; ++row)
#pragma unroll
                for (int i = 0; i < NQ; ++i) {
                    const int seen = w.pos0 + min(r0 + 16 * i + row, w.n_rows - 1);
#pragma unroll
                    for (int t = 0; t < G; ++t) {
                        f32x4_t x = o[i][t];
#pragma unroll
                        for (int e = 0; e < 4; ++e) x = mfma4(key0 + e <= seen ? vf[t][e] : 0.f, s[i][e], x);
#pragma unroll
                        for (int r = 0; r < 4; ++r) o[i][t][r] = fr == row ? x[r] : o[i][t][r];
                    }
                }
        }
#pragma unroll
        for (int t = 0; t < G; ++t) { kf[t] = kn[t]; vf[t] = vn[t]; }
    }
    // ---- merge the four wavefronts
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        l_run[i] += __shfl_xor(l_run[i], 16);
        l_run[i] += __shfl_xor(l_run[i], 32);
        if (fq == 0) { m_sh[wave][16 * i + fr] = m_run[i]; l_sh[wave][16 * i + fr] = l_run[i]; }
    }
    __syncthreads();
    float f[NQ];                                              // this wavefront's share of a row, normalised
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const int r = 16 * i + fr;
        float m = m_sh[0][r];                                 // wavefront 0 has page 0: finite for every row
#pragma unroll
        for (int v = 1; v < 4; ++v) m = fmaxf(m, m_sh[v][r]);
        float l = 0.f;
#pragma unroll
        for (int v = 0; v < 4; ++v) l += l_sh[v][r] * __builtin_amdgcn_exp2f(m_sh[v][r] - m);
        f[i] = __builtin_amdgcn_exp2f(m_run[i] - m) / l;
    }
    // register r of slice t: head_dim 16 t + 4 quarter + r of query row lane % 16
    const int st_row = threadIdx.x >> 2, st_c = (threadIdx.x & 3) * 4;
#pragma unroll
    for (int t = 0; t < G; ++t) {
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            f32x4_t x = o[i][t];
#pragma unroll
            for (int r = 0; r < 4; ++r) x[r] *= f[i];
            *reinterpret_cast<f32x4_t*>(&o_sh[wave][16 * i + fr][4 * fq]) = x;
        }
        __syncthreads();
        if (st_row < ROWS && r0 + st_row < w.n_rows) {
            f32x4_t x = *reinterpret_cast<const f32x4_t*>(&o_sh[0][st_row][st_c]);
#pragma unroll
            for (int v = 1; v < 4; ++v) {
                const f32x4_t y = *reinterpret_cast<const f32x4_t*>(&o_sh[v][st_row][st_c]);
#pragma unroll
                for (int r = 0; r < 4; ++r) x[r] += y[r];
            }
            *reinterpret_cast<f32x4_t*>(out + ((int64_t)(w.row0 + r0 + st_row) * n_q_heads + head) * HD + 16 * t + st_c) = x;
        }
        __syncthreads();
    }
}

template <int HD, int NQ>
void launch_attn(hipStream_t s, const void* q, void* out, const void* pool_layer, const AttnWork* work, int n_work,
                 const int32_t* page_tables, int n_q_heads, KvGeom g) {
    const dim3 grid((unsigned)n_work * (ATTN_BLOCK_ROWS / (16 * NQ)), n_q_heads);
    attention_f32_kernel<HD, NQ><<<grid, 256, 0, s>>>((const float*)q, (float*)out, (const float*)pool_layer, work,
                                                       page_tables, n_q_heads, g);
}

}  // namespace

bool gemm_f32_supported(const void* A, const void* W, const void* W2, int K) {
    // 16-byte reads of whole rows
    return K % 4 == 0 && (((uintptr_t)A | (uintptr_t)W | (uintptr_t)W2) & 15) == 0;
}

void launch_gemm_f32(hipStream_t s, const void* A, const void* W, const void* W2, float* C, int M, int N, int K,
                     int epi) {
    if (M <= 0 || N <= 0) return;
    const float *a = (const float*)A, *w = (const float*)W, *w2 = (const float*)W2;
    switch (epi) {
        case EPI_ADD_F32: launch_f32<EPI_ADD_F32>(s, a, w, w2, C, M, N, K); break;
        case EPI_SILU_MUL: launch_f32<EPI_SILU_MUL>(s, a, w, w2, C, M, N, K); break;
        default: launch_f32<EPI_STORE_F32>(s, a, w, w2, C, M, N, K); break;    // STORE_T is the same for float
    }
}

void launch_attention_f32(hipStream_t s, const void* q, void* out, const void* pool_layer, const AttnWork* work,
                          int n_work, const int32_t* page_tables, int n_q_heads, KvGeom g) {
    if (n_work <= 0) return;
    // 32-row blocks once whole items of them would give every CU two workgroups, 16-row blocks below
    const bool two = (int64_t)n_work * (ATTN_BLOCK_ROWS / 32) * n_q_heads >= 512;
    if (g.head_dim == 128) {
        if (two) launch_attn<128, 2>(s, q, out, pool_layer, work, n_work, page_tables, n_q_heads, g);
        else launch_attn<128, 1>(s, q, out, pool_layer, work, n_work, page_tables, n_q_heads, g);
    } else {
        if (two) launch_attn<64, 2>(s, q, out, pool_layer, work, n_work, page_tables, n_q_heads, g);
        else launch_attn<64, 1>(s, q, out, pool_layer, work, n_work, page_tables, n_q_heads, g);
    }
}

}  // namespace cf
