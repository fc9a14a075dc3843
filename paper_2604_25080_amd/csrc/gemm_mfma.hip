// bf16 GEMM on CDNA4 matrix cores for the linear layers of recompute:
//   acc[M,N] = A[M,K] * W[N,K]^T   (both operands K-contiguous, float accumulate)
// with the layer's epilogue fused: float store (QKV, O-proj, down-proj, LM head), float add, bf16
// store, SiLU(gate)*up -> bf16 (gate/up pair), or -- for the QKV projection on the big tile -- RoPE
// on the accumulators with Q stored as bf16 and K/V written straight into their page slots.
//
// Tiling: 256x256 block tile, 8 wavefronts (4x2, two per SIMD), each a 64x128 wave tile = 4x8
// fragments of the MFMA 16x16x32; problems too small to fill the chip with such tiles use 128x128
// or 64x64 block tiles (4 wavefronts).  K is walked in steps of 64: operands go from global memory
// straight to LDS (no staging registers) into a ring of K-steps, one barrier per step.  LDS rows are
// K-contiguous (128 bytes, a whole cache line of the operand row) with the 16-byte chunk index
// XOR-swizzled by the row, so that the 16-byte fragment reads of a wavefront spread over all banks.
// Workgroups are renumbered so that the 32 workgroups resident on one XCD
// (one L2) cover an 8x4 patch of tiles.
//
// What bounds it: power and the waits for operands.  Under a full chip of MFMAs the clock falls to
// 1.7-1.9 GHz, so what counts is energy per product: registers-only loops over random operands
// sustain 1750 TFLOP/s with the 32x32x16 MFMA and 2025 with the 16x16x32 (half the accumulator
// traffic per product), 1590 against 1770 with the fragments read from LDS.  8192 rows of the 8B
// gate/up projection: 1.28 -> 1.45 PFLOP/s against one wavefront per SIMD, 32x32x16 and operands
// staged through registers; with the loads taken out of the loop 1.70, with all of them hitting L2
// 1.56 (74 % of the cycles multiply at 1.83 GHz).
#include <type_traits>

#include "kernels.h"
#include "per_device.h"
#include "rope.h"
#include "cacheflow.h"

namespace cf {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_t;   // native 16-byte register vector
typedef u32x4_t __attribute__((aligned(2))) u32x4_any_t;            // the same in memory, at any element

namespace {

constexpr int BK = 64;
constexpr int ROW_BYTES = BK * 2;         // one LDS row: 128 bytes = eight 16-byte chunks

__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
// two floats -> two bf16 (round to nearest even), low half = a
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
    f32x2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

__device__ __forceinline__ uint16_t f32_to_bf16_bits(float v) {
    uint32_t u = __float_as_uint(v);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

typedef __attribute__((address_space(3))) char* lds_ptr_t;

// Buffer descriptor of a run of bytes.
__device__ __forceinline__ u32x4_t buffer_rsrc(const void* base, unsigned bytes) {
    const uint64_t p = (uint64_t)(uintptr_t)base;
    u32x4_t r;
    r.x = __builtin_amdgcn_readfirstlane((unsigned)p);
    r.y = __builtin_amdgcn_readfirstlane((unsigned)(p >> 32) & 0xFFFFu);
    r.z = __builtin_amdgcn_readfirstlane(bytes);
    r.w = 0x00020000u;
    return r;
}
constexpr unsigned PAST_THE_END = 0x80000000u;    // no operand tile is that long: such an offset reads zero
// 16 bytes per lane from the buffer straight to LDS: lane i lands at lds + 16 i.  No register is
// written; whoever reads the LDS bytes waits for vmcnt first (wait_barrier below).  The LDS base goes in
// m0, which the compiler sets (an operand, not a write it does not know of).
__device__ __forceinline__ void load_to_lds(u32x4_t rsrc, unsigned voff, unsigned soff, unsigned lds) {
    asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" :: "v"(voff), "s"(rsrc), "s"(soff), "{m0}"(lds) : "memory");
}
// This wavefront's LDS reads are done and all but its last LEFT loads have landed; then everybody's.
template <int LEFT>
__device__ __forceinline__ void wait_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(LEFT) : "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// Stores a wave tile: fragment (i, j) of a lane is output row row0 + 16 i, columns col0 + 16 j + r; gate/up
// pair: the first FN/2 fragments are gate, the rest up.  INSIDE: the tile lies wholly in the matrix.
template <int EPI, int FM, int FN, bool INSIDE>
__device__ __forceinline__ void store_tile(const f32x4_t (&acc)[FM][FN], float* __restrict__ Cf, bf16* __restrict__ Dt,
                                           int M, int N, int row0, int col0) {
    constexpr bool SILU = (EPI == EPI_SILU_MUL);
    constexpr bool TO_F32 = (EPI == EPI_STORE_F32 || EPI == EPI_ADD_F32);
    constexpr int FN_OUT = SILU ? FN / 2 : FN;
    const bool vec_ok = (N & 3) == 0;             // row starts stay vector-aligned
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        const int gm = row0 + i * 16;
        if (!INSIDE && gm >= M) continue;
#pragma unroll
        for (int j = 0; j < FN_OUT; ++j) {
            const int gn = col0 + j * 16;
            const int64_t o = (int64_t)gm * N + gn;
            f32x4_t v = acc[i][j];
            if constexpr (SILU) {
                // silu(g) * u with the hardware exp2 and reciprocal (each within 1 ulp;
                // the result is rounded to bf16 right after)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    float e = __builtin_amdgcn_exp2f(v[t] * -1.4426950408889634f);
                    v[t] = v[t] * __builtin_amdgcn_rcpf(1.0f + e) * acc[i][j + FN / 2][t];
                }
            }
            if (vec_ok && (INSIDE || gn < N)) {
                if constexpr (TO_F32) {
                    f32x4_t* dst = reinterpret_cast<f32x4_t*>(Cf + o);
                    if constexpr (EPI == EPI_ADD_F32) {
                        const f32x4_t old = *dst;
#pragma unroll
                        for (int t = 0; t < 4; ++t) v[t] += old[t];
                    }
                    *dst = v;
                } else {
                    uint2 pk;
                    pk.x = pack_bf16x2(v[0], v[1]);
                    pk.y = pack_bf16x2(v[2], v[3]);
                    *reinterpret_cast<uint2*>(Dt + o) = pk;
                }
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (gn + t < N) {
                        if constexpr (EPI == EPI_ADD_F32) Cf[o + t] += v[t];
                        else if constexpr (TO_F32) Cf[o + t] = v[t];
                        else Dt[o + t].x = f32_to_bf16_bits(v[t]);
                    }
            }
        }
    }
}

// BM x BN block tile by NWM x NWN wavefronts; SA (SB) K-steps of A (B) in LDS.  DIRECT: operands go
// straight to LDS, which takes starts on whole dwords and tiles within 32-bit offsets; otherwise they
// go through registers (see Tile).
// `bid` of `nb` workgroups walk the tiles_m x tiles_n tiles whose origin is (m_off, n_off); M, N
// are the bounds of the whole matrix.
template <int EPI, int BM, int BN, int NWM, int NWN, int SA, int SB, bool DIRECT>
__device__ __forceinline__ void
gemm_mfma_body(char* smem, const bf16* __restrict__ A, const bf16* __restrict__ W,
               const bf16* __restrict__ W2, float* __restrict__ Cf, bf16* __restrict__ Dt, int M,
               int N, int K, int tiles_m, int tiles_n, int m_off, int n_off, int bid, int nb,
               const RopeEpilogue& rope) {
    constexpr bool SILU = (EPI == EPI_SILU_MUL);
    constexpr bool ROPE = (EPI == EPI_QKV_ROPE128 || EPI == EPI_QKV_ROPE64);
    constexpr int BN_OUT = SILU ? BN / 2 : BN;    // output columns per block
    constexpr int NW = NWM * NWN;
    constexpr int WM = BM / NWM, WN = BN / NWN;   // wave tile
    constexpr int FM = WM / 16, FN = WN / 16;     // MFMA fragments per wave tile
    constexpr int A_TILE = BM * ROW_BYTES, B_TILE = BN * ROW_BYTES;
    constexpr int S = SA < SB ? SA : SB, XA = SA - S, XB = SB - S, A_ALL = SA * A_TILE;
    static_assert(XA + XB <= 1, "at most one operand is a step deeper");
    constexpr int LA = BM / 8 / NW, LB = BN / 8 / NW;         // loads per wavefront: 8 rows each
    static_assert(LA * 8 * NW == BM && LB * 8 * NW == BN && (!SILU || LB % 2 == 0) && NW % 2 == 0, "loader shape");

    // ---- workgroup -> tile: XCD-contiguous renumbering, then 8-row groups
    int per = nb >> 3, rem = nb & 7, xcd = bid & 7, idx = bid >> 3;
    int pid = xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
    constexpr int GM = 8;             // = GROUP_M of the launcher
    int in_group = GM * tiles_n;
    int first_m = (pid / in_group) * GM;
    int gsz = min(tiles_m - first_m, GM);
    int tile_m = first_m + (pid % in_group) % gsz;
    int tile_n = (pid % in_group) / gsz;
    int m0 = m_off + tile_m * BM, n0 = n_off + tile_n * BN_OUT;
    constexpr bool BIG = (BM == 256);
    if constexpr (BIG) {
        // Edge tiles are shifted back inside the matrix (the host guarantees M >= BM and
        // N >= BN_OUT); the overlap is recomputed and stored twice with identical values.
        // This keeps every row of a tile a fixed stride apart, so the loader needs one
        // per-thread offset instead of one per row.
        m0 = min(m0, M - BM);
        n0 = min(n0, N - BN_OUT);
    }

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / NWN, wn = wave % NWN;

    // ---- loader: a load moves 8 rows of 128 bytes; wavefront w takes row groups w, w + NW, ...
    // LDS holds chunk c of a row at position c ^ swz(row); a load writes LDS linearly, so the lanes
    // permute their global addresses instead.  swz is the same for all of a lane's rows.
    const int ld_row = wave * 8 + (lane >> 3);
    const unsigned ld_col = ((lane & 7) ^ swz(ld_row)) << 4;
    const unsigned row_b = (unsigned)K * 2u;
    const bf16* w_tile = W + (int64_t)n0 * K;
    const bf16* w2_tile = SILU ? W2 + (int64_t)n0 * K : w_tile;
    const int rows_a = min(BM, M - m0), rows_b = min(BN_OUT, N - n0);
    const u32x4_t rs_a = buffer_rsrc(A + (int64_t)m0 * K, rows_a * row_b);
    const u32x4_t rs_b = buffer_rsrc(w_tile, rows_b * row_b);
    const u32x4_t rs_b2 = SILU ? buffer_rsrc(w2_tile, rows_b * row_b) : rs_b;
    const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_ptr_t)smem + (unsigned)wave * 1024u);
    constexpr int LB1 = SILU ? LB / 2 : LB;       // gate/up pair: the second half of B's rows are W2's
    unsigned va[BIG ? 1 : LA], vb[BIG ? 1 : LB1];
    if constexpr (BIG) {
        va[0] = vb[0] = ld_row * row_b + ld_col;
    } else {
#pragma unroll
        for (int j = 0; j < LA; ++j) va[j] = min(ld_row + j * NW * 8, rows_a - 1) * row_b + ld_col;
#pragma unroll
        for (int j = 0; j < LB1; ++j) vb[j] = min(ld_row + j * NW * 8, rows_b - 1) * row_b + ld_col;
    }
    // K need not be whole steps (big tile: it is): in the last one the lanes whose chunk lies past
    // the row's end ask for an offset outside the buffer, which reads as zero.
    const int nk = (K + BK - 1) / BK, last = !BIG && K % BK ? nk - 1 : -1;
    const unsigned past = (int)ld_col >= (K % BK) * 2 ? PAST_THE_END : 0u;
    // load j of the wavefront's LA (LB) loads of a step's A (B) rows
    auto dma_a = [&](int kt, int stage, int j) {
        const unsigned k_b = (unsigned)kt * ROW_BYTES;
        const unsigned v = va[BIG ? 0 : j];
        load_to_lds(rs_a, !BIG && kt == last ? v | past : v, BIG ? k_b + j * (NW * 8) * row_b : k_b,
                    lds0 + stage * A_TILE + j * (NW * 1024));
    };
    auto dma_b = [&](int kt, int stage, int j) {
        const unsigned k_b = (unsigned)kt * ROW_BYTES;
        const int jr = SILU ? j % LB1 : j;
        const unsigned v = vb[BIG ? 0 : jr];
        load_to_lds(SILU && j >= LB1 ? rs_b2 : rs_b, !BIG && kt == last ? v | past : v, BIG ? k_b + jr * (NW * 8) * row_b : k_b,
                    lds0 + A_ALL + stage * B_TILE + j * (NW * 1024));
    };

    // ---- fragment reads: lane reads row (lane % 16) of a 16-row fragment, chunk 4*kk + lane/16
    const int frow = lane & 15, fq = lane >> 4;
    const int fswz = swz(frow);                   // fragment bases are multiples of 16 rows
    const char* a_base = smem + (wm * WM + frow) * ROW_BYTES;
    const char* b_base = smem + A_ALL + frow * ROW_BYTES;
    auto read_a = [&](int stage, int kk, int i) {
        return *reinterpret_cast<const u32x4_t*>(a_base + stage * A_TILE + i * 16 * ROW_BYTES + (((4 * kk + fq) ^ fswz) << 4));
    };
    auto read_b = [&](int stage, int kk, int j) {
        // gate/up pair: the first FN/2 fragments are gate columns, the rest the same columns of up
        const int r = SILU ? ((j < FN / 2) ? wn * (WN / 2) + j * 16 : BN / 2 + wn * (WN / 2) + (j - FN / 2) * 16)
                           : wn * WN + j * 16;
        return *reinterpret_cast<const u32x4_t*>(b_base + stage * B_TILE + r * ROW_BYTES + (((4 * kk + fq) ^ fswz) << 4));
    };

    f32x4_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    u32x4_t fa0[FM], fb0[FN], fa1[FM], fb1[FN];
    // One row of fragments.  W's fragment goes first, which leaves the transposed product in the
    // accumulators: a lane owns four consecutive columns of one output row.
    auto mfma_row = [&](const u32x4_t (&fa)[FM], const u32x4_t (&fb)[FN], int i) {
#pragma unroll
        for (int j = 0; j < FN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, fb[j]),
                                                                __builtin_bit_cast(bf16x8_t, fa[i]), acc[i][j], 0, 0, 0);
    };
    auto read_frags = [&](u32x4_t (&fa)[FM], u32x4_t (&fb)[FN], int sa, int sb, int kk) {
#pragma unroll
        for (int j = 0; j < FN; ++j) fb[j] = read_b(sb, kk, j);
#pragma unroll
        for (int i = 0; i < FM; ++i) fa[i] = read_a(sa, kk, i);
    };

    if constexpr (!DIRECT) {
        // ---- through registers, two K-steps in LDS; the K order of an element, and so its bits, are those of
        // the loop below.  Past the row's end its last chunk is read again: its place in LDS is zeroed (in the
        // last step) or never multiplied (in a step past the end).
        static_assert(SA == 2 && SB == 2, "two K-steps in LDS");
        const int64_t row_bytes = (int64_t)K * 2;
        const char* a_tile = (const char*)(A + (int64_t)m0 * K);
        auto b_tile = [&](int j) { return (const char*)(SILU && j >= LB1 ? w2_tile : w_tile); };
        const char* pa[LA];
        const char* pb[LB];
        if constexpr (!BIG) {
#pragma unroll
            for (int j = 0; j < LA; ++j) pa[j] = a_tile + min(ld_row + j * NW * 8, rows_a - 1) * row_bytes;
#pragma unroll
            for (int j = 0; j < LB; ++j) pb[j] = b_tile(j) + min(ld_row + j % LB1 * NW * 8, rows_b - 1) * row_bytes;
        }
        auto get = [&](const char* tile, const char* row, int kt, int j) {
            if constexpr (BIG)                    // one base per tile, 32-bit offsets (host: K < 2^23)
                return *reinterpret_cast<const u32x4_any_t*>(tile + (va[0] + (j * (NW * 8) * row_b + (unsigned)min(kt, nk - 1) * ROW_BYTES)));
            else
                return *reinterpret_cast<const u32x4_any_t*>(row + min((int64_t)kt * ROW_BYTES + ld_col, row_bytes - 16));
        };
        auto get_a = [&](int kt, int j) { return get(a_tile, pa[j], kt, j); };
        auto get_b = [&](int kt, int j) { return get(b_tile(j), pb[j], kt, j % LB1); };
        char* const st = smem + (wave * 64 + lane) * 16;
        auto put = [&](char* at, u32x4_t v, int kt) {
            if (!BIG && kt == last && past) v = u32x4_t{0u, 0u, 0u, 0u};
            *reinterpret_cast<u32x4_t*>(at) = v;
        };
        auto put_a = [&](int kt, int j, u32x4_t v) { put(st + (kt & 1) * A_TILE + j * (NW * 1024), v, kt); };
        auto put_b = [&](int kt, int j, u32x4_t v) { put(st + A_ALL + (kt & 1) * B_TILE + j * (NW * 1024), v, kt); };
        if constexpr (BIG) {
            // Registers for four loads are left beside two wavefronts per SIMD: A and B take turns, half a step
            // between a load and its way to LDS.  B runs a step ahead of A, into the stage that the barrier
            // has just freed.
            static_assert(LA == LB && LA <= FM, "one load beside each row of MFMAs");
            u32x4_t r[LA];
            auto fill_b = [&](int kt) {
#pragma unroll
                for (int j = 0; j < LB; ++j) put_b(kt, j, get_b(kt, j));
            };
#pragma unroll
            for (int j = 0; j < LA; ++j) put_a(0, j, get_a(0, j));
            fill_b(0);
            fill_b(1);
#pragma unroll
            for (int j = 0; j < LA; ++j) r[j] = get_a(1, j);
            __syncthreads();
            read_frags(fa0, fb0, 0, 0, 0);
            constexpr int PJ = FN / FM;
            auto step = [&](int kt, auto parity) {    // parity of kt: the LDS offsets are constants
                constexpr int cur = parity.value;
#pragma unroll
                for (int i = 0; i < FM; ++i) {
#pragma unroll
                    for (int j = i * PJ; j < (i + 1) * PJ; ++j) fb1[j] = read_b(cur, 1, j);
                    fa1[i] = read_a(cur, 1, i);
                    if (i < LA) {
                        put_a(cur ^ 1, i, r[i]);
                        r[i] = get_b(kt + 2, i);
                    }
                    mfma_row(fa0, fb0, i);
                    __builtin_amdgcn_sched_barrier(0);
                }
                __syncthreads();
#pragma unroll
                for (int i = 0; i < FM; ++i) {
#pragma unroll
                    for (int j = i * PJ; j < (i + 1) * PJ; ++j) fb0[j] = read_b(cur ^ 1, 0, j);
                    fa0[i] = read_a(cur ^ 1, 0, i);
                    if (i < LA) {
                        put_b(cur, i, r[i]);
                        r[i] = get_a(kt + 2, i);
                    }
                    mfma_row(fa1, fb1, i);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            for (int kt = 0; kt < nk; kt += 2) {      // K is whole pairs of steps (host)
                step(kt, std::integral_constant<int, 0>{});
                step(kt + 1, std::integral_constant<int, 1>{});
            }
        } else {
            constexpr int D = BM == 128 ? 2 : 4;  // K-steps in flight in registers
            u32x4_t ra[D][LA], rb[D][LB];
#pragma unroll
            for (int t = 0; t <= D; ++t) {
                if (t == D) {
#pragma unroll
                    for (int j = 0; j < LA; ++j) put_a(0, j, ra[0][j]);
#pragma unroll
                    for (int j = 0; j < LB; ++j) put_b(0, j, rb[0][j]);
                }
#pragma unroll
                for (int j = 0; j < LA; ++j) ra[t % D][j] = get_a(t, j);
#pragma unroll
                for (int j = 0; j < LB; ++j) rb[t % D][j] = get_b(t, j);
            }
            __syncthreads();
            read_frags(fa0, fb0, 0, 0, 0);
            auto step = [&](int kt, auto set) {   // set: the registers that hold step kt + 1
                constexpr int X = set.value, PJ = (FN + FM - 1) / FM, PA = (LA + FM - 1) / FM, PB = (LB + FM - 1) / FM;
                const int cur = kt & 1;
#pragma unroll
                for (int i = 0; i < FM; ++i) {
                    // beside a row of MFMAs: the second half's fragments, and step kt + 1 goes to LDS and makes
                    // room for step kt + 1 + D
#pragma unroll
                    for (int j = i * PJ; j < (i + 1) * PJ && j < FN; ++j) fb1[j] = read_b(cur, 1, j);
                    fa1[i] = read_a(cur, 1, i);
#pragma unroll
                    for (int j = i * PA; j < (i + 1) * PA && j < LA; ++j) {
                        put_a(kt + 1, j, ra[X][j]);
                        ra[X][j] = get_a(kt + 1 + D, j);
                    }
#pragma unroll
                    for (int j = i * PB; j < (i + 1) * PB && j < LB; ++j) {
                        put_b(kt + 1, j, rb[X][j]);
                        rb[X][j] = get_b(kt + 1 + D, j);
                    }
                    mfma_row(fa0, fb0, i);
                }
                __syncthreads();
#pragma unroll
                for (int i = 0; i < FM; ++i) {
#pragma unroll
                    for (int j = i * PJ; j < (i + 1) * PJ && j < FN; ++j) fb0[j] = read_b(cur ^ 1, 0, j);
                    fa0[i] = read_a(cur ^ 1, 0, i);
                    mfma_row(fa1, fb1, i);
                }
            };
            // whole groups without a branch: across one the compiler moves the loads down to their use
            int kt = 0;
            for (; kt + D <= nk; kt += D) {
                step(kt, std::integral_constant<int, 1 % D>{});
                step(kt + 1, std::integral_constant<int, 2 % D>{});
                if constexpr (D > 2) {
                    step(kt + 2, std::integral_constant<int, 3 % D>{});
                    step(kt + 3, std::integral_constant<int, 0>{});
                }
            }
            if (kt < nk) step(kt++, std::integral_constant<int, 1 % D>{});
            if (D > 2 && kt < nk) step(kt++, std::integral_constant<int, 2 % D>{});
            if (D > 2 && kt < nk) step(kt++, std::integral_constant<int, 3 % D>{});
        }
    } else {
        // ---- main loop over K-steps of 64.  Step t sits in stage t % SA of A and t % SB of B.  Half-way
        // through step t every wavefront has read all of it (the second half's fragments are in
        // registers): one barrier says so, and that step t + 1 has landed; the stages are then refilled
        // with steps t + SA and t + SB.  Of an operand with a stage more the loads go last and stay in
        // flight over a second barrier.
        constexpr int LOADS = LA + LB, LEFT = (S - 2) * LOADS + XA * LA + XB * LB;
#pragma unroll
        for (int t = 0; t < SA || t < SB; ++t)
            if (t < nk) {
#pragma unroll
                for (int j = 0; j < LA && t < SA; ++j) dma_a(t, t, j);
#pragma unroll
                for (int j = 0; j < LB && t < SB; ++j) dma_b(t, t, j);
            }
        if (nk >= S + XA + XB) wait_barrier<LEFT + LOADS>();
        else wait_barrier<0>();
        read_frags(fa0, fb0, 0, 0, 0);
        int ca = 0, cb = 0;                           // the current step's stages
        // refill 2: both operands; 1: only the one without the extra stage; 0: none
        auto kstep = [&](int kt, auto refill) {
            constexpr int REFILL = refill.value;
            const int na = ca + 1 == SA ? 0 : ca + 1, nb_ = cb + 1 == SB ? 0 : cb + 1;
            read_frags(fa1, fb1, ca, cb, 1);
#pragma unroll
            for (int i = 0; i < FM; ++i) mfma_row(fa0, fb0, i);
            constexpr int RPM = (FM * FN) / (FM + FN);            // MFMAs per fragment read
#pragma unroll
            for (int u = 0; u < FM + FN; ++u) {
                __builtin_amdgcn_sched_group_barrier(0x8, RPM, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x8, FM * FN - RPM * (FM + FN), 0);
            if constexpr (REFILL == 2) wait_barrier<LEFT>();
            else wait_barrier<0>();
#pragma unroll
            for (int i = 0; i < FM; ++i) {
                // the next fragments and the refill, spread over the rows of MFMAs; the priority keeps
                // the other wavefront of the SIMD from breaking into the row (gate/up: +3 %)
                constexpr int PJ = (FN + FM - 1) / FM;
                constexpr int FIRST = XB ? LA : LB, N_REFILL = REFILL == 2 ? LOADS : REFILL == 1 ? FIRST : 0;
                constexpr int PD = (LOADS + FM - 1) / FM;
#pragma unroll
                for (int j = i * PJ; j < (i + 1) * PJ && j < FN; ++j) fb0[j] = read_b(nb_, 0, j);
                fa0[i] = read_a(na, 0, i);
#pragma unroll
                for (int j = i * PD; j < (i + 1) * PD && j < N_REFILL; ++j) {
                    if ((j < FIRST) == (XB > 0)) dma_a(kt + SA, ca, j < FIRST ? j : j - FIRST);
                    else dma_b(kt + SB, cb, j < FIRST ? j : j - FIRST);
                }
                __builtin_amdgcn_s_setprio(1);
                mfma_row(fa1, fb1, i);
                __builtin_amdgcn_s_setprio(0);
                __builtin_amdgcn_sched_barrier(0);
            }
            ca = na;
            cb = nb_;
        };
        int kt = 0;
        for (; kt + S + XA + XB < nk; ++kt) kstep(kt, std::integral_constant<int, 2>{});
        if constexpr (XA + XB > 0)
            if (kt + S < nk) kstep(kt++, std::integral_constant<int, 1>{});
        for (; kt < nk; ++kt) kstep(kt, std::integral_constant<int, 0>{});
    }

    // ---- epilogue.  Fragment (i, j): output row 16 i + lane % 16, columns 16 j + 4 (lane / 16) + r:
    // a lane stores its four columns as one vector.  The big tile lies wholly inside the matrix
    // (shifted back at the edges): no bounds tests.
    if constexpr (ROPE) {
        // QKV projection (big tile only, N a multiple of the tile): a wave tile spans whole
        // heads, and both elements (j, j + head_dim/2) of a rotation pair sit in the same lane,
        // HALF_F fragments apart.  Per row the lane looks up the position (angle) and the page
        // slot; whether a head is Q, K or V is the same for the whole wavefront.
        static_assert(BIG, "the fused QKV epilogue exists for the 256x256 tile only");
        constexpr int HD = (EPI == EPI_QKV_ROPE128) ? 128 : 64;
        constexpr int HALF_F = HD / 32;               // fragments per half head
        static_assert(WN % HD == 0, "wave tile must span whole heads");
        const int col_l = 4 * fq;
        const int nq = rope.n_q_heads * HD, nkv = rope.g.n_kv_heads * HD;
        bf16* pool = (bf16*)rope.pool_layer;
        // Loads first, and ahead of the stores they could alias with as far as the compiler
        // knows: the rows' positions and slots up front, then the angles of row group i + 1
        // while row group i is rotated and stored.
        int rpos[FM], rslot[FM];
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            const int gm = m0 + wm * WM + i * 16 + frow;
            rpos[i] = rope.pos[gm];
            rslot[i] = rope.slot[gm];
        }
        constexpr int NTAB = HALF_F * 2;              // float4 loads per row: 4 * HALF_F (cos, sin) pairs
        constexpr int FH = 2 * HALF_F;                // fragments per head
#define CF_LOAD_ANGLES(I, T)                                                                  \
        {                                                                                     \
            const float2* cs_ = rope.cos_sin + (int64_t)rpos[I] * (HD / 2) + col_l;           \
            _Pragma("unroll") for (int u = 0; u < HALF_F; ++u) {                              \
                T[2 * u] = *reinterpret_cast<const float4*>(cs_ + 16 * u);                    \
                T[2 * u + 1] = *reinterpret_cast<const float4*>(cs_ + 16 * u + 2);            \
            }                                                                                 \
        }
        // Head by head; Q, K or V is decided once per head, outside the row loop, so that each
        // branch is straight-line code over the row groups.
#pragma unroll
        for (int hh = 0; hh < WN / HD; ++hh) {
            // first column of this head (the same for every lane: kept in a scalar register)
            const int hc = __builtin_amdgcn_readfirstlane(n0 + wn * WN + hh * HD);
            if (hc < nq + nkv) {
                float4 tab[2][NTAB];
                CF_LOAD_ANGLES(0, tab[0]);
#pragma unroll
                for (int i = 0; i < FM; ++i) {
                    if (i + 1 < FM) CF_LOAD_ANGLES(i + 1, tab[(i + 1) & 1]);
                    const float4* tb = tab[i & 1];
                    const int gm = m0 + wm * WM + i * 16 + frow;
                    // Q row of the packed query buffer, or the K row [head][slot][HD] of the page
                    bf16* dst = hc < nq ? Dt + (int64_t)gm * nq + hc
                                        : pool + (int64_t)(rslot[i] / CF_PAGE_TOKENS) * rope.g.page_elems +
                                              ((int64_t)((hc - nq) / HD) * CF_PAGE_TOKENS + rslot[i] % CF_PAGE_TOKENS) * HD;
#pragma unroll
                    for (int jj = 0; jj < HALF_F; ++jj) {
                        const int cj = jj * 16 + col_l;                // pair index, multiple of 4
                        const float4 t0 = tb[2 * jj], t1 = tb[2 * jj + 1];
                        const float2 cc[4] = {{t0.x, t0.y}, {t0.z, t0.w}, {t1.x, t1.y}, {t1.z, t1.w}};
                        float y1[4], y2[4];
#pragma unroll
                        for (int t = 0; t < 4; ++t)
                            rope_rotate(acc[i][hh * FH + jj][t], acc[i][hh * FH + HALF_F + jj][t], cc[t], y1[t], y2[t]);
                        uint2 lo, hi;
                        lo.x = pack_bf16x2(y1[0], y1[1]); lo.y = pack_bf16x2(y1[2], y1[3]);
                        hi.x = pack_bf16x2(y2[0], y2[1]); hi.y = pack_bf16x2(y2[2], y2[3]);
                        *reinterpret_cast<uint2*>(dst + cj) = lo;
                        *reinterpret_cast<uint2*>(dst + cj + HD / 2) = hi;
                    }
                }
            } else {
                // V, stored transposed in the page: [head][HD][slot]; the 16 rows of a fragment
                // are mostly consecutive slots, so a store instruction still fills 32-byte runs
#pragma unroll
                for (int i = 0; i < FM; ++i) {
                    bf16* dst = pool + (int64_t)(rslot[i] / CF_PAGE_TOKENS) * rope.g.page_elems +
                                (int64_t)rope.g.n_kv_heads * CF_PAGE_TOKENS * HD +
                                (int64_t)((hc - nq - nkv) / HD) * HD * CF_PAGE_TOKENS + rslot[i] % CF_PAGE_TOKENS;
#pragma unroll
                    for (int j = 0; j < FH; ++j)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            dst[(j * 16 + col_l + r) * CF_PAGE_TOKENS].x = f32_to_bf16_bits(acc[i][hh * FH + j][r]);
                }
            }
        }
#undef CF_LOAD_ANGLES
    } else {
        store_tile<EPI, FM, FN, BIG>(acc, Cf, Dt, M, N, m0 + wm * WM + frow, n0 + wn * (SILU ? WN / 2 : WN) + 4 * fq);
    }
}

// The block tiles: wavefront grid and K-steps of A and B in LDS.  Of the 160 KB two steps of the
// big tile take 128; the third step of B lets its loads take two steps to land (down projection,
// K = 14336, 8192 rows: 1.33 -> 1.41 PFLOP/s; K = 4096: no change).
// Operands that cannot go straight to LDS (an odd element, rows of 2^22 elements and more) go through
// registers: unaligned 16-byte loads and the way back cost a fifth to a half (13 389 rows x 4096 x 14336: 1711 us
// against 1220; 1000 x 4096 x 4096: 57, 45; 33 x 6144 x 4096: 22, 15), the plain kernel 15 to 60 times that.
template <int TILE, bool DIRECT> struct Tile;
template <> struct Tile<256, true> { static constexpr int NWM = 4, NWN = 2, SA = 2, SB = 3; };
template <> struct Tile<128, true> { static constexpr int NWM = 2, NWN = 2, SA = 2, SB = 2; };
template <> struct Tile<64, true> { static constexpr int NWM = 2, NWN = 2, SA = 4, SB = 4; };
template <int TILE> struct Tile<TILE, false> { static constexpr int NWM = TILE == 256 ? 4 : 2, NWN = 2, SA = 2, SB = 2; };

template <int EPI, int B, bool DIRECT>
__global__ void __launch_bounds__((64 * Tile<B, DIRECT>::NWM * Tile<B, DIRECT>::NWN), 2)
gemm_mfma_kernel(const bf16* __restrict__ A, const bf16* __restrict__ W,
                 const bf16* __restrict__ W2, float* __restrict__ Cf, bf16* __restrict__ Dt, int M,
                 int N, int K, int tiles_m, int tiles_n, RopeEpilogue rope) {
    extern __shared__ __align__(16) char smem[];
    using T = Tile<B, DIRECT>;
    gemm_mfma_body<EPI, B, B, T::NWM, T::NWN, T::SA, T::SB, DIRECT>(
        smem, A, W, W2, Cf, Dt, M, N, K, tiles_m, tiles_n, 0, 0, (int)blockIdx.x, tiles_m * tiles_n, rope);
}

// Big tiles with a quartered tail.  With one 256x256 tile per CU at a time, a launch whose tile
// count is not a multiple of the CU count ends with a round in which most CUs idle for a whole
// tile time (5152 tiles on 256 CUs: 20 rounds and 32 tiles).  Here the first n_big workgroups
// take the big tiles in the usual order EXCEPT a rectangle at its end -- the last tail_cols
// tile columns of the last 8-row group -- and the remaining workgroups cover that rectangle
// with 128x128 tiles, four times as many and a quarter as long (done only when the rectangle has at
// most half a round of big tiles: two rounds of small ones for one big; us without and with it, N 4096,
// K 4096 -- 272 tiles, 16 of them past the last full round: 169, 125; 336 (80): 173, 159; 384 (128): 174, 168;
// 896 (128): 370, 365; K 1024, 384: 61, 58).  The K order of an output element does not depend on the tile
// shape, so the result bits are those of any other tiling.
template <int EPI>
__global__ void __launch_bounds__(512, 2)
gemm_mfma_tail_kernel(const bf16* __restrict__ A, const bf16* __restrict__ W,
                      const bf16* __restrict__ W2, float* __restrict__ Cf, bf16* __restrict__ Dt,
                      int M, int N, int K, int tiles_m, int tiles_n, int n_big, int tail_m_off,
                      int tail_n_off, int tail_tiles_m, int tail_tiles_n) {
    extern __shared__ __align__(16) char smem[];
    const RopeEpilogue none{};
    if ((int)blockIdx.x < n_big)
        gemm_mfma_body<EPI, 256, 256, 4, 2, Tile<256, true>::SA, Tile<256, true>::SB, true>(
            smem, A, W, W2, Cf, Dt, M, N, K, tiles_m, tiles_n, 0, 0, (int)blockIdx.x, n_big, none);
    else
        gemm_mfma_body<EPI, 128, 128, 4, 2, 4, 4, true>(smem, A, W, W2, Cf, Dt, M, N, K, tail_tiles_m, tail_tiles_n,
                                               tail_m_off, tail_n_off, (int)blockIdx.x - n_big,
                                               tail_tiles_m * tail_tiles_n, none);
}

// Few rows: every row of A in one tile (BM >= M), BN columns per workgroup, so that the weights are
// read once and by as many workgroups as N gives.  Bound by memory: what counts is the bytes in
// flight and the serial chain of a workgroup's K-steps, so a stage of the ring holds G K-steps behind
// ONE barrier, all of a stage's fragments are read into registers at once, and S stages are in flight.
// The K order of an output element is that of every other tile.
template <int EPI, int BM, int BN, int G, int S>
__global__ void __launch_bounds__(BM == 16 ? 128 : 256)
gemm_rows_kernel(const bf16* __restrict__ A, const bf16* __restrict__ W, float* __restrict__ Cf,
                 bf16* __restrict__ Dt, int M, int N, int K) {
    extern __shared__ __align__(16) char smem[];
    constexpr int NWM = BM == 16 ? 1 : 2, NWN = 2, NW = NWM * NWN;
    constexpr int FM = BM / NWM / 16, FN = BN / NWN / 16;
    constexpr int A_TILE = BM * ROW_BYTES, STEP_BYTES = (BM + BN) * ROW_BYTES, STAGE_BYTES = G * STEP_BYTES;
    constexpr int LA = BM / 8 / NW, LB = BN / 8 / NW, LOADS = G * (LA + LB);
    static_assert(LA * 8 * NW == BM && LB * 8 * NW == BN && EPI != EPI_SILU_MUL, "loader shape");
    static_assert((S - 1) * LOADS <= 63, "the counter of loads in flight has six bits");
    const int n0 = blockIdx.x * BN;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / NWN, wn = wave % NWN;
    const unsigned row_b = (unsigned)K * 2u;
    const int rows_a = M, rows_b = min(BN, N - n0);
    const u32x4_t rs_a = buffer_rsrc(A, rows_a * row_b);
    const u32x4_t rs_b = buffer_rsrc(W + (int64_t)n0 * K, rows_b * row_b);
    const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lds_ptr_t)smem + (unsigned)wave * 1024u);
    const int ld_row = wave * 8 + (lane >> 3);
    const unsigned ld_col = ((lane & 7) ^ swz(ld_row)) << 4;
    unsigned va[LA], vb[LB];
#pragma unroll
    for (int j = 0; j < LA; ++j) va[j] = min(ld_row + j * NW * 8, rows_a - 1) * row_b + ld_col;
#pragma unroll
    for (int j = 0; j < LB; ++j) vb[j] = min(ld_row + j * NW * 8, rows_b - 1) * row_b + ld_col;
    const int nk = (K + BK - 1) / BK, ns = (nk + G - 1) / G;
    const int last = K % BK ? nk - 1 : -1;        // a partial step, see gemm_mfma_body
    const unsigned past = (int)ld_col >= (K % BK) * 2 ? PAST_THE_END : 0u;
    auto refill = [&](int t, int stage) {         // steps past the end fetch the last one again, unused
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int step = min(t * G + g, nk - 1);
            const unsigned k_b = (unsigned)step * ROW_BYTES, at = lds0 + stage * STAGE_BYTES + g * STEP_BYTES;
#pragma unroll
            for (int j = 0; j < LA; ++j) load_to_lds(rs_a, step == last ? va[j] | past : va[j], k_b, at + j * (NW * 1024));
#pragma unroll
            for (int j = 0; j < LB; ++j) load_to_lds(rs_b, step == last ? vb[j] | past : vb[j], k_b, at + A_TILE + j * (NW * 1024));
        }
    };
    const int frow = lane & 15, fq = lane >> 4, fswz = swz(frow);
    f32x4_t acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    u32x4_t fa[2 * G][FM], fb[2 * G][FN];
#pragma unroll
    for (int t = 0; t < S; ++t) refill(t, t);
    wait_barrier<(S - 1) * LOADS>();
    int cur = 0;
    for (int t = 0; t < ns; ++t) {
        const char* st = smem + cur * STAGE_BYTES + frow * ROW_BYTES;
#pragma unroll
        for (int kk = 0; kk < 2 * G; ++kk) {
            const int at = (kk >> 1) * STEP_BYTES + (((4 * (kk & 1) + fq) ^ fswz) << 4);
#pragma unroll
            for (int i = 0; i < FM; ++i)
                fa[kk][i] = *reinterpret_cast<const u32x4_t*>(st + at + (wm * FM + i) * 16 * ROW_BYTES);
#pragma unroll
            for (int j = 0; j < FN; ++j)
                fb[kk][j] = *reinterpret_cast<const u32x4_t*>(st + at + A_TILE + (wn * FN + j) * 16 * ROW_BYTES);
        }
        wait_barrier<(S - 2) * LOADS>();          // stage read by all, the next one landed
        refill(t + S, cur);
#pragma unroll
        for (int kk = 0; kk < 2 * G; ++kk)
            if (t * G + (kk >> 1) < nk)           // the same for the whole launch
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, fb[kk][j]),
                                                                            __builtin_bit_cast(bf16x8_t, fa[kk][i]), acc[i][j], 0, 0, 0);
        cur = cur + 1 == S ? 0 : cur + 1;
    }
    // the refills past the end must not land after the workgroup's LDS is given away
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    store_tile<EPI, FM, FN, false>(acc, Cf, Dt, M, N, wm * FM * 16 + frow, n0 + wn * (BN / NWN) + 4 * fq);
}

constexpr int N_CUS = 256;            // MI355X
constexpr int GROUP_M = 8;            // tile rows per group of the tile order (see the body)

// Lets a kernel have `bytes` of LDS: an attribute of the kernel on one device.
void allow_lds(PerDevice& once, const void* kern, int bytes) {
    int device = -1;
    (void)hipGetDevice(&device);
    once.run(device, [&] { (void)hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); });
}

template <int EPI, int B, bool DIRECT>
void launch_tile(hipStream_t s, const void* A, const void* W, const void* W2, float* Cf, void* Dt,
                 int M, int N, int K, bool tail_ok = false, const RopeEpilogue& rope = RopeEpilogue{}) {
    constexpr int BN_OUT = (EPI == EPI_SILU_MUL) ? B / 2 : B;
    constexpr int LDS = (Tile<B, DIRECT>::SA + Tile<B, DIRECT>::SB) * B * ROW_BYTES;
    int tiles_m = (M + B - 1) / B, tiles_n = (N + BN_OUT - 1) / BN_OUT;
    if constexpr (B == 256 && DIRECT && EPI != EPI_ADD_F32 && EPI != EPI_QKV_ROPE128 && EPI != EPI_QKV_ROPE64) {
        // tail: the last nb % N_CUS tiles, rounded up to whole columns of the last row group
        const int nb = tiles_m * tiles_n, tail = nb % N_CUS;
        const int gsz = tiles_m - (tiles_m - 1) / GROUP_M * GROUP_M;       // rows of the last group
        const int cols = (tail + gsz - 1) / gsz;
        if (tail_ok && nb > N_CUS && tail > 0 && gsz * cols <= N_CUS / 2 && cols <= tiles_n) {
            static PerDevice configured;
            auto kern = gemm_mfma_tail_kernel<EPI>;
            allow_lds(configured, (const void*)kern, LDS);
            constexpr int SBN_OUT = (EPI == EPI_SILU_MUL) ? 64 : 128;
            const int m_off = (tiles_m - gsz) * B, n_off = (tiles_n - cols) * BN_OUT;
            const int tm = (M - m_off + 127) / 128, tn = (N - n_off + SBN_OUT - 1) / SBN_OUT;
            const int n_big = nb - gsz * cols;
            kern<<<n_big + tm * tn, 512, LDS, s>>>((const bf16*)A, (const bf16*)W, (const bf16*)W2, Cf, (bf16*)Dt,
                                                   M, N, K, tiles_m, tiles_n, n_big, m_off, n_off, tm, tn);
            return;
        }
    }
    static PerDevice configured;
    auto kern = gemm_mfma_kernel<EPI, B, DIRECT>;
    allow_lds(configured, (const void*)kern, LDS);
    kern<<<tiles_m * tiles_n, 64 * Tile<B, DIRECT>::NWM * Tile<B, DIRECT>::NWN, LDS, s>>>((const bf16*)A, (const bf16*)W, (const bf16*)W2, Cf,
                                             (bf16*)Dt, M, N, K, tiles_m, tiles_n, rope);
}

template <int EPI, int BM, int BN, int G, int S>
void launch_rows(hipStream_t s, const void* A, const void* W, float* Cf, void* Dt, int M, int N, int K) {
    constexpr int LDS = S * G * (BM + BN) * ROW_BYTES;
    static PerDevice configured;
    auto kern = gemm_rows_kernel<EPI, BM, BN, G, S>;
    allow_lds(configured, (const void*)kern, LDS);
    kern<<<(N + BN - 1) / BN, BM == 16 ? 128 : 256, LDS, s>>>((const bf16*)A, (const bf16*)W, Cf, (bf16*)Dt, M, N, K);
}

int g_force_tile = 0;   // 0 = heuristic; 256 / 128 / 64 = forced tile, 257 = 256 with the quartered tail
constexpr int ROWS_MAX_WG = 1024;     // workgroups of 32 columns up to which the few-row kernel is used

// The big tile once 128x128 tiles would take more than one round (two workgroups per CU): a round of
// big tiles, however empty, costs 1.6 of theirs (us at N 4096, K 4096 -- 2048 rows, 512 tiles: 58 against
// 77; 2560 rows, 640 tiles: 93 against 77; K 14336, 2560 rows: 325 against 243).
inline bool prefer_big(int M, int N, int bn_out128) {
    return (int64_t)((M + 127) / 128) * ((N + bn_out128 - 1) / bn_out128) > 2 * N_CUS;
}

template <int EPI, bool DIRECT>
void launch(hipStream_t s, const void* A, const void* W, const void* W2, float* Cf, void* Dt, int M,
            int N, int K) {
    constexpr int BN_OUT128 = EPI == EPI_SILU_MUL ? 64 : 128;
    const bool big = (g_force_tile ? g_force_tile >= 256 : prefer_big(M, N, BN_OUT128)) && K % (2 * BK) == 0 && K < (1 << 23) &&
                     M >= 256 && N >= 2 * BN_OUT128 && EPI != EPI_ADD_F32;
    if (big) { launch_tile<EPI, 256, DIRECT>(s, A, W, W2, Cf, Dt, M, N, K, g_force_tile == 0 || g_force_tile == 257); return; }
    // At most 32 rows: the few-row kernel, unless the weight is so wide (an LM head) that larger
    // column tiles fill the chip anyway (us, 64x64 tiles against it -- N 4096, K 14336, 16 rows: 42,
    // 23; N 1280, K 8192: 25, 14; N 6144, K 4096, 23 rows: 14, 10; N 128256: 188 with 128x128
    // tiles against 205).  The gate/up pair has twice the columns and does better on the 64 tile.
    if constexpr (EPI != EPI_SILU_MUL && DIRECT)
        if (g_force_tile == 0 && M <= 32 && N <= 32 * ROWS_MAX_WG) {
            if (M <= 16) launch_rows<EPI, 16, 32, 4, 3>(s, A, W, Cf, Dt, M, N, K);
            else launch_rows<EPI, 32, 32, 4, 3>(s, A, W, Cf, Dt, M, N, K);
            return;
        }
    // One and a half rounds of 64x64 tiles (two workgroups per CU) or fewer: quarter the tile (us, 128
    // against 64 tile -- gate/up 100 rows of 4096: 52, 45; 300 rows of 8192 x 3584: 67, 64; down 700 rows:
    // 131, 121; N 1280, K 8192 2048 rows: 70, 66; above it the large tile wins: 3072 of those rows 76,
    // 89).  The K order of every output element is the same for all tile shapes, so the result bits do
    // not depend on the choice.
    const int64_t tiles64 = (int64_t)((M + 63) / 64) * ((N + BN_OUT128 / 2 - 1) / (BN_OUT128 / 2));
    const bool small = g_force_tile ? g_force_tile == 64 : tiles64 <= 3 * N_CUS;
    if (small) launch_tile<EPI, 64, DIRECT>(s, A, W, W2, Cf, Dt, M, N, K);
    else launch_tile<EPI, 128, DIRECT>(s, A, W, W2, Cf, Dt, M, N, K);
}

}  // namespace

void gemm_mfma_force_tile(int t) { g_force_tile = t; }

bool gemm_mfma_qkv_rope_supported(int dtype, int M, int N, int K, int head_dim) {
    // the shapes for which the float-output QKV GEMM would take the big tile anyway, with whole
    // tiles along N (no shifted edge tile: head boundaries stay on wave-tile boundaries)
    const bool big = g_force_tile ? g_force_tile >= 256 : prefer_big(M, N, 128);
    return dtype == CF_BF16 && (head_dim == 128 || head_dim == 64) && big && M >= 256 && N >= 256 &&
           N % 256 == 0 && K >= 2 * BK && K % (2 * BK) == 0;
}

// Straight to LDS: the loads move whole dwords at 32-bit offsets within a tile's rows.
static bool direct_ok(const void* A, const void* W, const void* W2, int K) {
    return (((uintptr_t)A | (uintptr_t)W | (uintptr_t)W2) & 3) == 0 && K < (1 << 22);
}

void launch_gemm_mfma_qkv_rope(hipStream_t s, const void* A, const void* Wqkv, void* q_out, int M,
                               int N, int K, const RopeEpilogue& rope) {
    const bool direct = direct_ok(A, Wqkv, nullptr, K);
#define CF_QKV(EPI, DIRECT) launch_tile<EPI, 256, DIRECT>(s, A, Wqkv, nullptr, nullptr, q_out, M, N, K, false, rope)
    if (rope.g.head_dim == 128) { if (direct) CF_QKV(EPI_QKV_ROPE128, true); else CF_QKV(EPI_QKV_ROPE128, false); }
    else { if (direct) CF_QKV(EPI_QKV_ROPE64, true); else CF_QKV(EPI_QKV_ROPE64, false); }
#undef CF_QKV
}

bool gemm_mfma_supported(int dtype, int M, int N, int K, int epi) {
    (void)epi;
    return dtype == CF_BF16 && M > 0 && N > 0 && K >= BK && K % BK == 0;
}

bool gemm_mfma_takes(int dtype, int M, int N, int K) {
    return dtype == CF_BF16 && M > 0 && N > 0 && K >= BK && K % 8 == 0;
}

void launch_gemm_mfma(hipStream_t s, const void* A, const void* W, const void* W2, float* Cf,
                      void* Dt, int M, int N, int K, int epi) {
    const bool direct = direct_ok(A, W, W2, K);
#define CF_GEMM(EPI) if (direct) launch<EPI, true>(s, A, W, W2, Cf, Dt, M, N, K); else launch<EPI, false>(s, A, W, W2, Cf, Dt, M, N, K)
    switch (epi) {
        case EPI_STORE_F32: CF_GEMM(EPI_STORE_F32); break;
        case EPI_ADD_F32: CF_GEMM(EPI_ADD_F32); break;
        case EPI_STORE_T: CF_GEMM(EPI_STORE_T); break;
        default: CF_GEMM(EPI_SILU_MUL); break;
    }
#undef CF_GEMM
}

}  // namespace cf
