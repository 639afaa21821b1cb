// BF16 GEMM on gfx950 matrix cores: C[M,N] = A[M,K] * B[N,K]^T with fused epilogues.
//
// Both operands are K-contiguous, which is the layout v_mfma_f32_32x32x16_bf16 wants for A and
// for B alike (a lane supplies 8 consecutive k of one row / one column), so no tile is ever
// transposed on its way to the matrix core.  Weights are stored [N,K] by the packer for exactly this reason.
//
// Three kernels share the epilogues:
//
//  * gemm_fast<BM,BN,EPI,WM,NS> — the production path for K % 128 == 0.  256 threads = 4 wavefronts, 2x2 (WM = 2:
//    each owns a (BM/2)x(BN/2) tile, up to 4x4 MFMA tiles = 256 fp32 accumulators per lane) or stacked 4x1 (WM = 4);
//    one workgroup per CU, two for 128x192 and 128x128 on two stages.  k-tile 64: a row of a tile is
//    one 128-byte cache line.  Tiles go global -> LDS directly (buffer_load_dwordx4 ... lds, no staging registers) into
//    NS = 2 .. 8 LDS stages (more for smaller tiles; A of 192x256 and 256x192 has four and three) that are separate arrays, so the
//    compiler can tell the stage being filled from the one being read; the wait for a copy is an explicit s_waitcnt.  LDS rows are
//    128 bytes, unpadded (a wavefront's copy fills 1 KB = 8 rows contiguously); the 16-byte chunk index is
//    XOR-swizzled with (row/2)%8 on both sides, which keeps the b128 fragment reads conflict-free.  Per k-tile four
//    phases of up to 16 MFMAs, each interleaved with the fragment reads of the next phase through
//    sched_group_barrier, ONE bare s_barrier, and the copies of k-tiles up to NS ahead spread over the phases that follow it.
//    What bounds it: the copies (a loop of nothing else takes 80 us of the 102 for 4096^3 on 256x256 tiles, 137 of 148 on
//    128x128).  They come in at about 60 bytes per ns and compute unit where lines miss the L2, at twice that where they hit
//    (every k-tile among the first eight: 128x128 148 -> 121 us); tiles that share lines ask for them at the same time.
//  * gemm_generic<EPI> — any shape (K % 8 == 0): 128x128 tile, 64x64 per wavefront, staged through registers.
//  * gemm_few_rows<BM,BN,NS,EPI,NORM> — M <= 64: BN output columns per workgroup, reduction split over its 4 wavefronts.
//
// Accumulator layout of a 32x32 tile: lane l, register r -> column l%32, row 8*(r/4) + 4*(l/32) + r%4.
#include <type_traits>

#include "kernels.hpp"
#include "norm_device.hpp"

namespace dlk {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

namespace {

constexpr int BM = 128, BN = 128, BK = 64;
constexpr int LDS_LD = BK + 8;   // row stride in elements: 144 bytes keeps 16-byte alignment and staggers banks

// x * sigmoid(x); the quotient is a multiplication with the hardware reciprocal (1 ulp), not an IEEE division
__device__ __forceinline__ float silu_f(float x) { return x * __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }
// tanh form of GELU: 0.5 x (1 + tanh u) = x * sigmoid(2u), u = sqrt(2/pi) (x + 0.044715 x^3): one exponential and
// one reciprocal instead of a library tanh (which dominated the epilogue of the encoder's MLP GEMM)
__device__ __forceinline__ float gelu_tanh_f(float x) {
    const float c2 = 2.0f * 0.7978845608028654f;
    const float u2 = c2 * (x + 0.044715f * x * x * x);
    return x * __builtin_amdgcn_rcpf(1.0f + __expf(-u2));
}
__device__ __forceinline__ float bf16_to_f(bf16_t v) { return __uint_as_float(uint32_t(v) << 16); }
__device__ __forceinline__ bf16_t f_to_bf16(float f) {
    __bf16 b = (__bf16)f;   // hardware round-to-nearest-even
    return *reinterpret_cast<bf16_t*>(&b);
}

// (acc + bias) * factor as fmaf(acc, factor, bias * factor): factor 1 leaves acc + bias
__device__ __forceinline__ float col_factor(const GemmArgs& p, int n) { return n < p.scale_cols ? p.scale : 1.0f; }
// first column that goes to p.vt
__device__ __forceinline__ int first_vt_col(const GemmArgs& p) { return p.vt ? p.vt_col : p.N; }

// 16 bytes per lane from a buffer straight into LDS (buffer_load_dwordx4 ... offen lds): the address is the buffer's
// base (four scalar registers, set up once) + a per-lane 32-bit offset that never changes + a scalar offset that
// advances with the k-tile, so a copy costs the vector unit nothing (a flat 64-bit address per lane cost 1.5 vector
// additions per copy instruction, which a wavefront cannot overlap with its own MFMAs).  Offsets past the buffer's
// size read zeros.
#define DL_BLL16(rsrc, voff, soff, l)                                                                    \
    __builtin_amdgcn_raw_ptr_buffer_load_lds((rsrc), (__attribute__((address_space(3))) void*)(l), 16,  \
                                             int(voff), int(soff), 0, 0)
// third dword of a raw buffer resource on gfx9: 32-bit data format, no swizzle, offsets checked against the size
constexpr int kBufferFlags = 0x00020000;

// s_waitcnt with an explicit vector-memory count (6 bits, split 4 + 2 in the gfx9 encoding); expcnt is left
// unconstrained, lgkmcnt is either unconstrained or zero
#define DL_WAIT_VM(N) __builtin_amdgcn_s_waitcnt(((N) & 0xF) | (((N) >> 4) << 14) | (0x7 << 4) | (0xF << 8))
#define DL_WAIT_VM_LGKM0(N) __builtin_amdgcn_s_waitcnt(((N) & 0xF) | (((N) >> 4) << 14) | (0x7 << 4) | (0x0 << 8))

// The wait states between the last MFMAs of a main loop and the first read of their results, spelled out.  The compiler
// inserts them itself, but has been seen to count them for one predecessor only where several paths that end in MFMAs
// meet (accumulator register 0 was read too early there), so such paths end with this.
#define DL_MFMA_SETTLE()                       \
    do {                                       \
        __builtin_amdgcn_sched_barrier(0);     \
        asm volatile("s_nop 15\n\ts_nop 15"); \
        __builtin_amdgcn_sched_barrier(0);     \
    } while (0)

// LDS stages of a tile.  Every stage is a separate __shared__ array, so that the compiler can tell the stage that is being
// filled from the one that is being read; the pointers are only ever indexed with constants.
template <int NS>
struct Stages {
    bf16_t* s[NS];
};
#define DL_STAGE(X, i, ELEMS) __shared__ __attribute__((aligned(1024))) bf16_t X##_##i[ELEMS]
#define DL_STAGES(X, NS, ELEMS)                                                                    \
    Stages<NS> X{{}};                                                                             \
    if constexpr (NS > 0) { DL_STAGE(X, 0, ELEMS); X.s[0] = X##_0; }                                     \
    if constexpr (NS > 1) { DL_STAGE(X, 1, ELEMS); X.s[1] = X##_1; }                                     \
    if constexpr (NS > 2) { DL_STAGE(X, 2, ELEMS); X.s[2] = X##_2; }                                     \
    if constexpr (NS > 3) { DL_STAGE(X, 3, ELEMS); X.s[3] = X##_3; }                                     \
    if constexpr (NS > 4) { DL_STAGE(X, 4, ELEMS); X.s[4] = X##_4; }                                     \
    if constexpr (NS > 5) { DL_STAGE(X, 5, ELEMS); X.s[5] = X##_5; }                                     \
    if constexpr (NS > 6) { DL_STAGE(X, 6, ELEMS); X.s[6] = X##_6; }                                     \
    if constexpr (NS > 7) { DL_STAGE(X, 7, ELEMS); X.s[7] = X##_7; }

// ---- few rows (M <= 64): one pass over the weights, bound by how many of their bytes are on the way at a time.  A 256-thread
// workgroup owns BN output columns (for SwiGLU BN / 2 gate columns and the BN / 2 up columns that go with them) and all
// BM >= M rows; its four wavefronts take the 64-wide k-tiles round-robin, each through NS LDS stages of its own (BM + BN
// rows of 128 bytes, filled by global -> LDS copies, chunks swizzled as in fast_tile), so nothing in the main loop waits
// for another wavefront.  The four partial tiles meet in LDS and are summed in wavefront order.  A row's sums do not
// depend on BM, BN or NS.
// 16-column tiles put 256 workgroups on 4096 columns (32 columns and 128 workgroups, eight wavefronts each, with the tiles
// staged through registers: 36 us for the 100 MB of 4096 x 12288 at 19 rows; now 24); the rows of A come through the same
// ~40 bytes per clock and compute unit as the weights, hence BM = 16, 32 or 64 by the number of rows.  8B gate/up, 19 rows:
// 76 us (128x128 register-staged kernel) -> 39, against 32 for its weights at the rate of a streaming read.
// EPI_QKV_POST: a tile of q or k columns takes BN / 2 columns and their rotary partners dh / 2 further on, scales and rounds them like a
// plain product's, rotates and scatters them (a layer over 19 rows and 3072 cached: 122.2 us with the separate launch, now 119.8).
// NORM >= 0: A is the normalisation (KIND as in norm_rows) of fp32 rows, which every workgroup makes for itself and keeps in LDS, all
// k-tiles of it; only weights are staged.  The rows are requested in front of the first weights, and at most 64 KB of them (see
// norm_pays; more were not measured).
// Rows past M repeat row M - 1 and are not stored.  Needs K % 64 == 0, N % 16 == 0, 16-byte aligned rows.
struct NoPost {};
template <int EPI>
using PostArgs = std::conditional_t<EPI == EPI_QKV_POST, QkvPostArgs, NoPost>;
struct NoNorm {};
template <int NORM>
using NormArgs = std::conditional_t<(NORM >= 0), NormIn, NoNorm>;
// longest reduction of the kernel with NORM
constexpr int max_norm_k(int bm) { return 256 * (64 / bm); }
template <int BM, int BN, int NS, int EPI, int NORM>
__global__ __launch_bounds__(256) void gemm_few_rows(GemmArgs p, PostArgs<EPI> post, NormArgs<NORM> nrm) {
    constexpr bool NA = NORM >= 0;
    constexpr int W = 4, STG = (NA ? BN : BM + BN) * 64;  // wavefronts; elements of one wavefront's stage
    constexpr int JA = NA ? 0 : BM / 8, JB = BN / 8, TM = BM / 16, TN = BN / 16;
    typedef __attribute__((ext_vector_type(4))) float f32x4;
    DL_STAGES(st, NS, W * STG)
    extern __shared__ __attribute__((aligned(1024))) bf16_t normed[];    // NORM: [k-tile][row][64], chunks swizzled as in the stages
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nk = p.K >> 6;
    const int n_my = (nk - wave + W - 1) / W;            // k-tiles wave, wave + W, ... (0 when there are fewer than wavefronts)
    constexpr bool SW = EPI == EPI_SWIGLU_BF16;
    const int n0 = blockIdx.x * (SW ? BN / 2 : BN);      // first output column
    // row of B that feeds column c of the tile
    auto brow = [&](int c) {
        if constexpr (EPI == EPI_QKV_POST) {
            if (n0 >= p.vt_col) return n0 + c;
            const int hd = n0 / post.dh * post.dh, i0 = (n0 - hd) / 2;       // head's first row, first pair
            return hd + i0 + (c < BN / 2 ? c : (post.dh - BN) / 2 + c);
        }
        if (!SW) return n0 + c;
        const int f = n0 + (c < BN / 2 ? c : c - BN / 2);
        return (f / 32) * 64 + f % 32 + (c < BN / 2 ? 0 : 32);
    };
    // the host takes this kernel only for operands below 4 GB
    const int sizeA = int(uint32_t(size_t(p.M) * p.lda * 2)), sizeB = int(uint32_t(size_t(p.N) * p.ldb * 2));
    uint32_t offA[JA + 1], offB[JB];
#pragma unroll
    for (int j = 0; j < JA; ++j) {
        const int row = 8 * j + (lane >> 3), lc = (lane & 7) ^ ((row >> 1) & 7);
        offA[j] = uint32_t((size_t(min(row, p.M - 1)) * p.lda + lc * 8) * 2);
    }
#pragma unroll
    for (int j = 0; j < JB; ++j) {
        const int row = 8 * j + (lane >> 3), lc = (lane & 7) ^ ((row >> 1) & 7);
        offB[j] = uint32_t((size_t(brow(row)) * p.ldb + lc * 8) * 2);
    }
    // (a k-tile that is not there reads as zeros: a buffer of no size, which fetches nothing)
    auto copy = [&](bf16_t* S, int i, bool real) {
        const int kb = (wave + W * i) * 128;
        const __amdgpu_buffer_rsrc_t gA = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p.A), 0, real ? sizeA : 0, kBufferFlags);
        const __amdgpu_buffer_rsrc_t gB = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p.B), 0, real ? sizeB : 0, kBufferFlags);
        bf16_t* d = S + wave * STG;
#pragma unroll
        for (int j = 0; j < JB; ++j) DL_BLL16(gB, offB[j], real ? kb : 0, d + (JA + j) * 512);
#pragma unroll
        for (int j = 0; j < JA; ++j) DL_BLL16(gA, offA[j], real ? kb : 0, d + j * 512);
    };
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = {0.0f, 0.0f, 0.0f, 0.0f};
    // the i-th k-tile of this wavefront, REM more behind it (NS stands for NS or more): wait for its copies, read the
    // fragments, refill the stage, multiply
    const int lr = lane & 15, lg = lane >> 4;
    auto ktile = [&](bf16_t* S, int i, auto rem_c) {
        constexpr int REM = decltype(rem_c)::value;
        DL_WAIT_VM((REM < NS - 1 ? REM : NS - 1) * (JA + JB));
        __builtin_amdgcn_sched_barrier(0);
        const bf16_t* d = S + wave * STG;
        // a k-tile that is not there has zeros for B; NORM has none for A: an infinity of another k-tile must not meet them
        const bool there = !NA || wave + W * i < nk;
        const bf16_t* da = NA ? normed + (there ? wave + W * i : 0) * (BM * 64) : d;
        bf16x8 a[2][TM], b[2][TN];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int pc = ((4 * kk + lg) ^ ((lr >> 1) & 7)) * 8;
#pragma unroll
            for (int t = 0; t < TM; ++t) a[kk][t] = *reinterpret_cast<const bf16x8*>(da + (16 * t + lr) * 64 + pc);
#pragma unroll
            for (int t = 0; t < TN; ++t) b[kk][t] = *reinterpret_cast<const bf16x8*>(d + (8 * JA + 16 * t + lr) * 64 + pc);
        }
        if constexpr (REM >= NS) {
            __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0): the fragments are in registers, the stage is free
            __builtin_amdgcn_sched_barrier(0);
            copy(S, i + NS, true);
        }
        if (there) {
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int t = 0; t < TM; ++t)
#pragma unroll
                    for (int u = 0; u < TN; ++u) acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kk][t], b[kk][u], acc[t][u], 0, 0, 0);
        }
    };
    using std::integral_constant;
    auto run = [&](auto self, int i0, auto i_c, auto n_c, auto after_c) {
        constexpr int I = decltype(i_c)::value, N = decltype(n_c)::value, AFTER = decltype(after_c)::value;
        ktile(st.s[I % NS], i0 + I, integral_constant<int, (N - 1 - I + AFTER < NS ? N - 1 - I + AFTER : NS)>{});
        if constexpr (I + 1 < N) self(self, i0, integral_constant<int, I + 1>{}, n_c, after_c);
    };
    if constexpr (NA) {
        // a wavefront takes BM / 4 rows, four at a time: 16 lanes to a row, P 16-byte pieces a lane
        constexpr int P = max_norm_k(BM) / 64, G = BM / W / 4;
        const int nv = p.K >> 2, l16 = lane & 15;
        float4 v[G][P];
        uint2 gk[P], bk[P];
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const int i = l16 + 16 * j, ic = i < nv ? i : 0;
#pragma unroll
            for (int g = 0; g < G; ++g)
                v[g][j] = reinterpret_cast<const float4*>(nrm.x + size_t(min((wave * G + g) * 4 + (lane >> 4), p.M - 1)) * p.K)[ic];
            gk[j] = reinterpret_cast<const uint2*>(nrm.g)[ic];
            if (NORM == 1) bk[j] = reinterpret_cast<const uint2*>(nrm.b)[ic];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < NS; ++s) copy(st.s[s], s, s < n_my);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int row = (wave * G + g) * 4 + (lane >> 4);
            float mean = 0.0f, ss = 0.0f;
            if (NORM == 1) {
                float sum = 0.0f;
#pragma unroll
                for (int j = 0; j < P; ++j)
                    if (l16 + 16 * j < nv) sum += (v[g][j].x + v[g][j].y) + (v[g][j].z + v[g][j].w);
                mean = normdev::row16_sum(sum) / float(p.K);
            }
#pragma unroll
            for (int j = 0; j < P; ++j) {
                const float a0 = v[g][j].x - mean, a1 = v[g][j].y - mean, a2 = v[g][j].z - mean, a3 = v[g][j].w - mean;
                if (l16 + 16 * j < nv) ss += (a0 * a0 + a1 * a1) + (a2 * a2 + a3 * a3);
            }
            const float inv = rsqrtf(normdev::row16_sum(ss) / float(p.K) + nrm.eps);
#pragma unroll
            for (int j = 0; j < P; ++j) {
                const int i = l16 + 16 * j;
                float o[4] = {(v[g][j].x - mean) * inv * __uint_as_float(gk[j].x << 16), (v[g][j].y - mean) * inv * __uint_as_float(gk[j].x & 0xFFFF0000u),
                              (v[g][j].z - mean) * inv * __uint_as_float(gk[j].y << 16), (v[g][j].w - mean) * inv * __uint_as_float(gk[j].y & 0xFFFF0000u)};
                if (NORM == 1) {
                    o[0] += __uint_as_float(bk[j].x << 16);
                    o[1] += __uint_as_float(bk[j].x & 0xFFFF0000u);
                    o[2] += __uint_as_float(bk[j].y << 16);
                    o[3] += __uint_as_float(bk[j].y & 0xFFFF0000u);
                }
                if (i < nv)
                    *reinterpret_cast<uint2*>(normed + ((i >> 4) * BM + row) * 64 + ((((i >> 1) & 7) ^ ((row >> 1) & 7)) * 8 + (i & 1) * 4)) =
                        make_uint2(uint32_t(f_to_bf16(o[0])) | (uint32_t(f_to_bf16(o[1])) << 16), uint32_t(f_to_bf16(o[2])) | (uint32_t(f_to_bf16(o[3])) << 16));
            }
        }
        __syncthreads();
    } else {
#pragma unroll
        for (int s = 0; s < NS; ++s) copy(st.s[s], s, s < n_my);
    }
    const int n_run = n_my < NS ? NS : n_my;             // stages of zeros are multiplied as well: no path for fewer than NS
    int i0 = 0;
    for (; i0 + 2 * NS <= n_run; i0 += NS)
        run(run, i0, integral_constant<int, 0>{}, integral_constant<int, NS>{}, integral_constant<int, NS>{});
    auto rest = [&](auto self, auto n_c) {               // NS .. 2 NS - 1 are left
        constexpr int N = decltype(n_c)::value;
        if constexpr (N < 2 * NS) {
            if (n_run - i0 == N) {
                run(run, i0, integral_constant<int, 0>{}, n_c, integral_constant<int, 0>{});
                DL_MFMA_SETTLE();
            } else {
                self(self, integral_constant<int, N + 1>{});
            }
        }
    };
    rest(rest, integral_constant<int, NS>{});

    __syncthreads();                                     // everybody is done with the stages
    float* part = reinterpret_cast<float*>(NA ? normed : st.s[0]);
    static_assert(NA || W * BM * BN * 4 <= W * STG * 2, "the partial tiles fit one stage array (or the rows: K >= 128, 16 columns)");
    // accumulator of a 16x16 tile: lane l, register r -> column l % 16, row 4 (l / 16) + r
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
        for (int u = 0; u < TN; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) part[(wave * BM + 16 * t + 4 * lg + r) * BN + 16 * u + lr] = acc[t][u][r];
    __syncthreads();
    if constexpr (EPI == EPI_QKV_POST) {
        if (n0 < p.vt_col) {
            const int half = post.dh >> 1, hh = n0 / post.dh, i0 = (n0 - hh * post.dh) / 2, n_q = post.k_off / post.dh;
            for (int q = tid; q < BM * BN / 2; q += 256) {
                const int c = q % (BN / 2), m = q / (BN / 2), i = i0 + c, r0 = hh * post.dh + i;
                if (m >= p.M) return;
                float a = part[m * BN + c], b = part[m * BN + BN / 2 + c];
#pragma unroll
                for (int w = 1; w < W; ++w) {
                    a += part[(w * BM + m) * BN + c];
                    b += part[(w * BM + m) * BN + BN / 2 + c];
                }
                if (p.bias) {
                    a += bf16_to_f(p.bias[r0]);
                    b += bf16_to_f(p.bias[r0 + half]);
                }
                const float f = col_factor(p, r0);
                a = bf16_to_f(f_to_bf16(a * f));
                b = bf16_to_f(f_to_bf16(b * f));
                const int pos = post.pos0 + m;
                float sn = 0.0f, cs = 1.0f;
                if (post.theta > 0.0f) sincosf(float(pos) * exp2f(-2.0f * float(i) / float(post.dh) * log2f(post.theta)), &sn, &cs);
                bf16_t* dst = static_cast<bf16_t*>(p.out) + size_t(m) * p.ldo + r0;
                if (hh >= n_q && post.k_out) dst = post.k_out + size_t(hh - n_q) * post.k_head_stride + size_t(pos) * post.dh + i;
                dst[0] = f_to_bf16(a * cs - b * sn);
                dst[half] = f_to_bf16(a * sn + b * cs);
            }
            return;
        }
    }
    if constexpr (EPI == EPI_BF16 || EPI == EPI_QKV_POST) {
        if (n0 + BN > first_vt_col(p)) {
            // columns of p.vt among them: neighbouring threads take neighbouring rows
#pragma unroll
            for (int q = tid; q < BM * BN; q += 256) {
                const int m = q % BM, c = q / BM, nc = n0 + c;
                float s = part[m * BN + c];
#pragma unroll
                for (int w = 1; w < W; ++w) s += part[(w * BM + m) * BN + c];
                if (p.bias) s += bf16_to_f(p.bias[nc]);
                if (m >= p.M) continue;
                if (nc < p.scale_cols) s *= p.scale;
                if (nc >= p.vt_col) p.vt[size_t(nc - p.vt_col) * p.vt_ld + m] = f_to_bf16(s);
                else static_cast<bf16_t*>(p.out)[size_t(m) * p.ldo + nc] = f_to_bf16(s);
            }
            return;
        }
    }
    // PT adjacent outputs per thread (a 16 x 8 tile leaves the upper half of the threads without one: row >= BM >= M)
    constexpr int BO = SW ? BN / 2 : BN, PT = BM * BO > 256 ? BM * BO / 256 : 1;
    static_assert(BO % PT == 0, "outputs of a thread sit in one row");
    const int row = tid * PT / BO, c0 = tid * PT % BO, n = n0 + c0;
    if (row >= p.M) return;
    float v[PT], u[PT];
#pragma unroll
    for (int e = 0; e < PT; ++e) {
        v[e] = part[row * BN + c0 + e];
        if (SW) u[e] = part[row * BN + BO + c0 + e];
#pragma unroll
        for (int w = 1; w < W; ++w) {
            v[e] += part[(w * BM + row) * BN + c0 + e];
            if (SW) u[e] += part[(w * BM + row) * BN + BO + c0 + e];
        }
        if (SW) v[e] = silu_f(v[e]) * u[e];
        else if (p.bias) v[e] += bf16_to_f(p.bias[n + e]);
        if (EPI == EPI_BF16 && n + e < p.scale_cols) v[e] *= p.scale;
        if (EPI == EPI_GELU_BF16) v[e] = gelu_tanh_f(v[e]);
    }
    constexpr int VW = PT < 4 ? PT : 4;                  // outputs per access (the host checks the alignment of 4)
    if (EPI == EPI_RESID_F32 || EPI == EPI_F32) {
        typedef __attribute__((ext_vector_type(VW))) float fv;
        float* out = static_cast<float*>(p.out) + size_t(row) * p.ldo + n;
#pragma unroll
        for (int e = 0; e < PT; e += VW) {
            fv o;
            if constexpr (EPI == EPI_RESID_F32) o = *reinterpret_cast<const fv*>(p.resid + size_t(row) * p.ldr + n + e);
#pragma unroll
            for (int x = 0; x < VW; ++x) o[x] = EPI == EPI_RESID_F32 ? o[x] + v[e + x] : v[e + x];
            *reinterpret_cast<fv*>(out + e) = o;
        }
    } else {
        typedef __attribute__((ext_vector_type(VW))) uint16_t hv;
        bf16_t* out = static_cast<bf16_t*>(p.out) + size_t(row) * p.ldo + n;
#pragma unroll
        for (int e = 0; e < PT; e += VW) {
            hv o;
#pragma unroll
            for (int x = 0; x < VW; ++x) o[x] = f_to_bf16(v[e + x]);
            *reinterpret_cast<hv*>(out + e) = o;
        }
    }
}

// Stages for two workgroups per compute unit (64, 72 or 80 KB of LDS), so that one's start and end hide under the other's stream;
// also where there are not that many workgroups, more stages gain nothing.  Columns per workgroup: 16; 32 for 33 .. 64 rows
// where 16 would be more than one workgroup per compute unit (6144 x 4096, 64 rows: 23 -> 19 us, with three stages in 144 KB and
// one workgroup per compute unit; up to 32 rows A is too small a share of the traffic: 24576 x 4096, 19 rows: 39 with 16 columns, 41
// with 32).
template <int EPI>
void launch_few_rows(const GemmArgs& a, hipStream_t st, const PostArgs<EPI>& post = {}) {
    auto go = [&](auto bm, auto bn, auto ns) {
        hipLaunchKernelGGL((gemm_few_rows<decltype(bm)::value, decltype(bn)::value, decltype(ns)::value, EPI, -1>), dim3(a.N / bn), dim3(256), 0, st, a,
                           post, NoNorm{});
    };
    using std::integral_constant;
    const integral_constant<int, 16> c16{};
    const integral_constant<int, 32> c32{};
    const integral_constant<int, 64> c64{};
    if (a.M <= 16) go(c16, c16, integral_constant<int, 4>{});
    else if (a.M <= 32) go(c32, c16, integral_constant<int, 3>{});
    else if (a.N % 32 == 0 && a.N > 256 * 16) go(c64, c32, integral_constant<int, 3>{});
    else go(c64, c16, integral_constant<int, 2>{});
}

// With the normalisation: all k-tiles of a wavefront staged at once (K at most 256, 512 and 1024 for 64, 32 and 16 rows).
template <int EPI, int NORM>
void launch_few_rows_norm(const GemmArgs& a, const NormIn& n, hipStream_t st, const PostArgs<EPI>& post) {
    const int bm = a.M <= 16 ? 16 : (a.M <= 32 ? 32 : 64);
    const dim3 grid(a.N / 16), block(256);
    const size_t lds = size_t(a.K) * bm * 2;
    if (bm == 16) hipLaunchKernelGGL((gemm_few_rows<16, 16, 4, EPI, NORM>), grid, block, lds, st, a, post, n);
    else if (bm == 32) hipLaunchKernelGGL((gemm_few_rows<32, 16, 2, EPI, NORM>), grid, block, lds, st, a, post, n);
    else hipLaunchKernelGGL((gemm_few_rows<64, 16, 2, EPI, NORM>), grid, block, lds, st, a, post, n);
}
template <int EPI>
void launch_few_rows_norm(const GemmArgs& a, const NormIn& n, hipStream_t st, const PostArgs<EPI>& post = {}) {
    if (n.kind == 0) launch_few_rows_norm<EPI, 0>(a, n, st, post);
    else launch_few_rows_norm<EPI, 1>(a, n, st, post);
}

// Column tiles whose residual values are requested together: what fits next to the accumulators without spilling (TM = 3: all of
// them).  The 256x192 tile takes one at a time: two spilled 32 registers and took 169.0 us for 4096 x 4096 outputs, K = 4096, now
// 164.1; 472.8 for 3072 x 4096, K = 12288, now 456.4; 33.8 for 8192 x 1152, K = 1152, now 31.5.
constexpr int resid_batch(int tm, int tn) {
    const int fit = (300 - tm * tn * 16) / (tm * 16);
    return tm == 3 ? tn : (fit < 1 ? 1 : (fit > tn ? tn : fit));
}

// epilogue shared by the tiled kernels: accumulator tile (i, j) of a wavefront whose tile starts at (mw, nw)
// n_end: first column past the tile's own columns (the start of the next tile or the matrix edge)
template <int EPI, int TM, int TN>
__device__ __forceinline__ void store_tiles(const GemmArgs& p, f32x16 (&acc)[TM][TN], int mw, int nw, int lane, int n_end) {
    const int col_in = lane & 31, row_in = (lane >> 5) * 4;
    if (EPI == EPI_SWIGLU_BF16) {
        // even tile columns hold gate rows, the next odd one the matching up rows (packed in groups of 32)
        bf16_t* out = static_cast<bf16_t*>(p.out);
#pragma unroll
        for (int j = 0; j < TN; j += 2) {
            const int pn = nw + 32 * j + col_in;            // packed column of the gate value
            if (pn + 32 >= p.N) continue;
            const int f = (nw + 32 * j) / 2 + col_in;        // feature index
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int m = mw + 32 * i + 8 * (r >> 2) + row_in + (r & 3);
                    if (m < p.M) out[size_t(m) * p.ldo + f] = f_to_bf16(silu_f(acc[i][j][r]) * acc[i][j + 1][r]);
                }
        }
        return;
    }
    if (EPI == EPI_RESID_F32) {
        // out may be the same buffer as resid: every element is read and then written by the same lane only, so the
        // pointers are declared non-aliasing.  The residual values of a batch of accumulator tiles are all requested
        // before the first one is used - unpredicated, rows and columns clamped into the matrix - so that the
        // wavefront pays one memory round trip per batch instead of one per tile; only the stores are predicated.
        const float* __restrict__ resid = p.resid;
        float* __restrict__ out = static_cast<float*>(p.out);
        constexpr int JB = resid_batch(TM, TN);
#pragma unroll
        for (int j0 = 0; j0 < TN; j0 += JB) {
            float rv[JB][TM][16];
            float bias[JB];
#pragma unroll
            for (int jj = 0; jj < JB; ++jj) {
                const int j = j0 + jj;
                if (j >= TN) continue;
                const int nc = min(nw + 32 * j + col_in, n_end - 1);
                bias[jj] = p.bias ? bf16_to_f(p.bias[nc]) : 0.0f;
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int mc = min(mw + 32 * i + 8 * (r >> 2) + row_in + (r & 3), p.M - 1);
                        rv[jj][i][r] = resid[uint32_t(mc) * uint32_t(p.ldr) + uint32_t(nc)];   // < 2^31 elements (host checks)
                    }
            }
#pragma unroll
            for (int jj = 0; jj < JB; ++jj) {
                const int j = j0 + jj;
                if (j >= TN) continue;
                const int n = nw + 32 * j + col_in;
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const int m = mw + 32 * i + 8 * (r >> 2) + row_in + (r & 3);
                        if (m < p.M && n < n_end) out[uint32_t(m) * uint32_t(p.ldo) + uint32_t(n)] = rv[jj][i][r] + acc[i][j][r] + bias[jj];
                    }
            }
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int n = nw + 32 * j + col_in;
        if (n >= n_end) continue;
        const float f = EPI == EPI_BF16 ? col_factor(p, n) : 1.0f;
        const float bias = p.bias ? bf16_to_f(p.bias[n]) * f : 0.0f;
        if (EPI == EPI_BF16 && n >= first_vt_col(p)) {
            // a transposed column of a tile that also holds others: a lane has four consecutive rows per register group
            bf16_t* col = p.vt + size_t(n - p.vt_col) * p.vt_ld;
            const bool wide = p.vt_ld % 4 == 0 && reinterpret_cast<uintptr_t>(p.vt) % 8 == 0;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int m = mw + 32 * i + 8 * g + row_in;
                    bf16_t o[4];
#pragma unroll
                    for (int x = 0; x < 4; ++x) o[x] = f_to_bf16(acc[i][j][4 * g + x] + bias);
                    if (wide && m + 4 <= p.M) {
                        *reinterpret_cast<uint2*>(col + m) =
                            make_uint2(o[0] | (uint32_t(o[1]) << 16), o[2] | (uint32_t(o[3]) << 16));
                    } else {
#pragma unroll
                        for (int x = 0; x < 4; ++x)
                            if (m + x < p.M) col[m + x] = o[x];
                    }
                }
            continue;
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = mw + 32 * i + 8 * (r >> 2) + row_in + (r & 3);
                if (m >= p.M) continue;
                const float v = EPI == EPI_BF16 ? fmaf(acc[i][j][r], f, bias) : acc[i][j][r] + bias;
                if (EPI == EPI_BF16) {
                    static_cast<bf16_t*>(p.out)[size_t(m) * p.ldo + n] = f_to_bf16(v);
                } else if (EPI == EPI_GELU_BF16) {
                    static_cast<bf16_t*>(p.out)[size_t(m) * p.ldo + n] = f_to_bf16(gelu_tanh_f(v));
                } else {
                    static_cast<float*>(p.out)[size_t(m) * p.ldo + n] = v;
                }
            }
    }
}

// The same epilogues as the fast path stores them (residual: a wavefront tile that lies wholly inside the matrix only, see
// there).  The others go through a buffer over the wavefront tile's rows of the output: rows past M are out of range and not
// written, columns past the tile's get an offset that is, so nothing is predicated, and an element costs its arithmetic, its
// conversion and the store; a row's scalar offset is computed once for all of its column tiles, which are stored together.
// (host: the rows of a wavefront tile span less than 2 GB)
// (the largest wavefront tile has no registers for a factor per column, 32 would spill: one for all of its columns, see the caller)
template <int TM, int TN>
constexpr bool kColFactors = TM * TN < 16;
template <int EPI, int TM, int TN>
__device__ __forceinline__ void store_tiles_buf(const GemmArgs& p, f32x16 (&acc)[TM][TN], int mw, int nw, int lane, int n_end) {
    constexpr bool SW = EPI == EPI_SWIGLU_BF16;
    constexpr int E = EPI == EPI_F32 ? 4 : 2, JS = SW ? 2 : 1;
    const int col_in = lane & 31, row_in = (lane >> 5) * 4, rows = min(p.M - mw, 32 * TM);
    if (rows <= 0) return;
    const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(
        static_cast<uint8_t*>(p.out) + (size_t(mw) * p.ldo + (SW ? nw / 2 : nw)) * E, 0, int(uint32_t(rows) * uint32_t(p.ldo) * E), kBufferFlags);
    uint32_t off[TN];
    float bias[TN], f[TN];
#pragma unroll
    for (int j = 0; j < TN; j += JS) {
        const int n = nw + 32 * j + col_in;              // SwiGLU: the gate column, its up column is 32 further on
        off[j] = n + 32 * (JS - 1) < n_end ? uint32_t(row_in * p.ldo + 32 * (j / JS) + col_in) * E : 0x80000000u;
        f[j] = EPI == EPI_BF16 ? col_factor(p, kColFactors<TM, TN> ? n : nw) : 1.0f;
        bias[j] = !SW && p.bias ? bf16_to_f(p.bias[min(n, n_end - 1)]) * f[j] : 0.0f;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int so = (32 * i + 8 * (r >> 2) + (r & 3)) * p.ldo * E;
#pragma unroll
            for (int j = 0; j < TN; j += JS) {
                if constexpr (SW) {
                    __builtin_amdgcn_raw_buffer_store_b16(f_to_bf16(silu_f(acc[i][j][r]) * acc[i][j + 1][r]), out, int(off[j]), so, 0);
                } else {
                    const float v = EPI == EPI_BF16 ? fmaf(acc[i][j][r], f[j], bias[j]) : acc[i][j][r] + bias[j];
                    if constexpr (EPI == EPI_F32) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), out, int(off[j]), so, 0);
                    else __builtin_amdgcn_raw_buffer_store_b16(f_to_bf16(EPI == EPI_GELU_BF16 ? gelu_tanh_f(v) : v), out, int(off[j]), so, 0);
                }
            }
        }
}

// Residual epilogue of a wavefront tile that lies wholly inside the matrix (every tile of the 8B shapes): nothing is predicated.
template <int TM, int TN>
__device__ __forceinline__ void store_resid_full(const GemmArgs& p, f32x16 (&acc)[TM][TN], int mw, int nw, int lane) {
    const uint32_t col_in = lane & 31, row_in = (lane >> 5) * 4;
    const uint32_t lane_o = row_in * uint32_t(p.ldo) + col_in;          // output element offset of this lane
    float bias[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) bias[j] = p.bias ? bf16_to_f(p.bias[nw + 32 * j + col_in]) : 0.0f;
    // one base pointer each for resid and out, per-lane 32-bit element offsets that advance row by row with
    // additions (no scalar pointer per row: 48-64 of them next to the accumulators made the loads slower)
    const float* __restrict__ resid = p.resid + size_t(mw) * p.ldr + nw;
    float* __restrict__ out = static_cast<float*>(p.out) + size_t(mw) * p.ldo + nw;
    const uint32_t lane_r = row_in * uint32_t(p.ldr) + col_in;
    constexpr int JB = resid_batch(TM, TN);
#pragma unroll
    for (int j0 = 0; j0 < TN; j0 += JB) {
        float rv[JB][TM][16];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const uint32_t ro = lane_r + uint32_t(32 * i + 8 * (r >> 2) + (r & 3)) * uint32_t(p.ldr);
#pragma unroll
                for (int jj = 0; jj < JB; ++jj)
                    if (j0 + jj < TN) rv[jj][i][r] = resid[ro + 32 * (j0 + jj)];
            }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const uint32_t oo = lane_o + uint32_t(32 * i + 8 * (r >> 2) + (r & 3)) * uint32_t(p.ldo);
#pragma unroll
                for (int jj = 0; jj < JB; ++jj)
                    if (j0 + jj < TN) out[oo + 32 * (j0 + jj)] = rv[jj][i][r] + acc[i][j0 + jj][r] + bias[j0 + jj];
            }
    }
}

// Transposed accumulators (lane: one row of C per 32 x 32 tile, registers: columns) of columns that go to p.vt: 32 lanes
// write 32 consecutive positions of one V^T row, the 64-byte pieces that the other columns are written in.  Through a
// buffer over the wavefront tile's rows of V^T: what lies past the matrix is out of range and not written, so an element
// costs its conversion, a scalar addition and the store (N and vt_col are multiples of 8).
template <int TM, int TN>
__device__ __forceinline__ void store_tiles_vt(const GemmArgs& p, f32x16 (&acc)[TM][TN], int mw, int nw, int lane) {
    const int rows = min(p.N - nw, 32 * TN), g4 = (lane >> 5) * 4;
    if (rows <= 0 || mw >= p.M) return;
    const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(
        p.vt + ptrdiff_t(nw - p.vt_col) * p.vt_ld + mw, 0, int(uint32_t(size_t(rows) * p.vt_ld * 2)), kBufferFlags);
    uint32_t off[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = 32 * i + (lane & 31);
        off[i] = mw + m < p.M ? uint32_t(g4 * p.vt_ld + m) * 2u : 0x80000000u;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            float bias[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if (p.bias) {
#pragma unroll
                for (int x = 0; x < 4; ++x) bias[x] = bf16_to_f(p.bias[min(nw + 32 * j + 8 * g + g4, p.N - 4) + x]);
            }
#pragma unroll
            for (int x = 0; x < 4; ++x)
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    __builtin_amdgcn_raw_buffer_store_b16(f_to_bf16(acc[i][j][4 * g + x] + bias[x]), out, int(off[i]),
                                                          (32 * j + 8 * g + x) * p.vt_ld * 2, 0);
        }
}

// Any shape.  The epilogue is the shared one: it requests a batch of residual values before it uses the first; element by
// element, behind a predicate each, a lane made 64 round trips and 256 x 144 outputs, K = 144, took 23.3 us, now 8.4.
template <int EPI>
__global__ __launch_bounds__(256) void gemm_generic(GemmArgs p) {
    __shared__ __attribute__((aligned(16))) bf16_t sA[BM * LDS_LD];
    __shared__ __attribute__((aligned(16))) bf16_t sB[BN * LDS_LD];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int tiles_n = (p.N + BN - 1) / BN;
    const int m0 = (blockIdx.x / tiles_n) * BM, n0 = (blockIdx.x % tiles_n) * BN;

    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    u32x4 ra[4], rb[4];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = tid + 256 * i, row = c >> 3, kc = (c & 7) * 8;
            const int k = k0 + kc;
            u32x4 z = {0u, 0u, 0u, 0u};
            ra[i] = z;
            rb[i] = z;
            if (m0 + row < p.M && k < p.K)
                ra[i] = *reinterpret_cast<const u32x4*>(p.A + size_t(m0 + row) * p.lda + k);
            if (n0 + row < p.N && k < p.K)
                rb[i] = *reinterpret_cast<const u32x4*>(p.B + size_t(n0 + row) * p.ldb + k);
        }
    };
    auto stash = [&]() {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = tid + 256 * i, row = c >> 3, kc = (c & 7) * 8;
            *reinterpret_cast<u32x4*>(&sA[row * LDS_LD + kc]) = ra[i];
            *reinterpret_cast<u32x4*>(&sB[row * LDS_LD + kc]) = rb[i];
        }
    };

    const int nk = (p.K + BK - 1) / BK;
    fetch(0);
    for (int kt = 0; kt < nk; ++kt) {
        stash();
        __syncthreads();
        if (kt + 1 < nk) fetch((kt + 1) * BK);
        const int lr = lane & 31, lk = (lane >> 5) * 8;
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            bf16x8 a[2], b[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                a[i] = *reinterpret_cast<const bf16x8*>(&sA[(64 * wm + 32 * i + lr) * LDS_LD + 16 * kk + lk]);
                b[i] = *reinterpret_cast<const bf16x8*>(&sB[(64 * wn + 32 * i + lr) * LDS_LD + 16 * kk + lk]);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
    }

    store_tiles<EPI, 2, 2>(p, acc, m0 + 64 * wm, n0 + 64 * wn, lane, min(p.N, n0 + BN));
}

// blockIdx -> tile.  Workgroups are dealt round-robin to the 8 XCDs (each with its own L2): XCD x gets a
// contiguous range of the tile order, and inside it 8 row-tiles x consecutive column-tiles run together,
// so the tiles resident on one XCD share their A and B slabs in that XCD's L2.
__device__ __forceinline__ bool tile_of(int bid, int tiles_m, int tiles_n, int* tm, int* tn) {
    const int total = tiles_m * tiles_n;
    const int xcd = bid % 8, idx = bid / 8;
    const int per = (total + 7) / 8;
    const int lin = xcd * per + idx;
    if (idx >= per || lin >= total) return false;
    constexpr int GM = 8;
    const int grp = lin / (GM * tiles_n), r = lin % (GM * tiles_n);
    const int gm = min(GM, tiles_m - grp * GM);
    *tm = grp * GM + r % gm;
    *tn = r / gm;
    return true;
}

// scheduling request for one phase of a k-tile: NM MFMAs with the NR fragment reads spread evenly over all but the
// last RT of them (those cover the latency of the last read) and the NC global->LDS copies spread over all of them
template <int NM, int NR, int NC, int RT, int M>
struct SchedEven {
    static __device__ __forceinline__ void run() {
        if constexpr (M < NM) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            constexpr int span = NM - RT;
            constexpr int r = M < span ? ((M + 1) * NR / span - M * NR / span) : 0;
            if constexpr (r > 0) __builtin_amdgcn_sched_group_barrier(0x100, r, 0);
            constexpr int c = (M + 1) * NC / NM - M * NC / NM;
            if constexpr (c > 0) __builtin_amdgcn_sched_group_barrier(0x020, c, 0);
            SchedEven<NM, NR, NC, RT, M + 1>::run();
        }
    }
};

// One output tile with its top-left corner at (m0, n0).  sa, sb: SA >= SB LDS stages of at least BM * 64 and BN * 64 elements.
// The four wavefronts form a WM x (4 / WM) grid.  TR: the tile's columns go to p.vt; the operands of every MFMA change places
// (both have the same layout), which transposes the accumulators and leaves the sums as they are.
template <int BM, int BN, int EPI, int WM, int SA, int SB, bool TR>
__device__ __forceinline__ void fast_tile_any(const GemmArgs& p, int m0, int n0, Stages<SA> sa, Stages<SB> sb) {
    constexpr int BK = 64, WN = 4 / WM;
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
    constexpr int JA = BM / 32, JB = BN / 32;            // 1 KB copy blocks (8 rows x 128 B) per wavefront and k-tile
    constexpr int RT = TM * TN / 4;
    static_assert(BM % (32 * WM) == 0 && BN % (32 * WN) == 0, "whole MFMA tiles per wavefront");
    // the wavefront index is the same in every lane: as a scalar it keeps the LDS addresses of the copies (M0) and
    // everything else derived from it out of the vector unit
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    // copy sources: block b = wave + 4*j of a tile holds rows 8b..8b+7, 128 bytes (one cache line, 64 k) each;
    // lane L lands at row 8b + L/8, physical 16-byte chunk L%8, and therefore fetches logical chunk
    // (L%8) ^ ((row/2)%8): a b128 fragment read serves 16 lanes (16 consecutive rows, 256 bytes of banks) at a time,
    // two rows fill the 64 banks once, so the swizzle has to differ between the 8 row PAIRS (with row%8 the counters
    // showed every second LDS cycle of the kernel as a bank conflict).  Rows past the matrix edge are clamped: they produce values that the epilogue never stores.
    // Tiles in one row of tiles start at different blocks of their rows of A, tiles in one column at different blocks of B:
    // those that run on an XCD at the same time then ask its L2 for a line one after the other, and all but the first find it there.
    // (not on 256x256: there the MFMAs hide them, and 4096^3 with an fp32 output took 1.5 us more.  With / without on the other shapes,
    // geometric means over layers of 128 .. 1536 features: K of 1024 and more 0.99, at best 0.86; at K = 128 and 256 up to 0.05 us more, what the
    // offsets take before the first copy: 768 columns, K = 256, 6.24 -> 6.29 us on average, 6.34 with the chunk of every block computed anew.
    // A condition at run time costs short reductions the same.)
    constexpr bool ROT = BM * BN < 256 * 256;
    const int rotA = ROT ? n0 / BN * ((JA + 3) / 4) % JA : 0, rotB = ROT ? m0 / BM * ((JB + 3) / 4) % JB : 0;
    // a wavefront's blocks are four apart, so (row/2)%8 of a lane's row is the same in all of them
    const int lc = (lane & 7) ^ ((4 * wave + (lane >> 4)) & 7);
    uint32_t offA[JA], offB[JB];
    int blkA[JA], blkB[JB];
#pragma unroll
    for (int j = 0; j < JA; ++j) {
        blkA[j] = wave + 4 * (j + rotA < JA ? j + rotA : j + rotA - JA);
        offA[j] = uint32_t((size_t(min(m0 + 8 * blkA[j] + (lane >> 3), p.M - 1)) * p.lda + lc * 8) * 2);
    }
#pragma unroll
    for (int j = 0; j < JB; ++j) {
        blkB[j] = wave + 4 * (j + rotB < JB ? j + rotB : j + rotB - JB);
        offB[j] = uint32_t((size_t(min(n0 + 8 * blkB[j] + (lane >> 3), p.N - 1)) * p.ldb + lc * 8) * 2);
    }
    // the host only takes this path for operands below 4 GB
    const int sizeA = int(uint32_t(size_t(p.M) * p.lda * 2)), sizeB = int(uint32_t(size_t(p.N) * p.ldb * 2));
    // fragment read offsets (elements) inside a stage, one per 16-wide k step
    const int lr = lane & 31, g2 = lane >> 5;
    int rdA[4], rdB[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        const int pc = (2 * kk + g2) ^ ((lr >> 1) & 7);
        rdA[kk] = ((BM / WM) * wm + lr) * BK + pc * 8;
        rdB[kk] = ((BN / WN) * wn + lr) * BK + pc * 8;
    }

    bf16x8 a0[TM], b0[TN], a1[TM], b1[TN];
    const int nk = p.K / BK;                             // host guarantees K % 128 == 0: nk is even and >= 2
    // copies j0 .. j1 - 1 of a k-tile of A or B
    constexpr bool EXITS = SA != SB;
    // (a k-tile that is not there: a buffer of no size, which fetches nothing)
    auto copyA = [&](bf16_t* S, int kt, int j0, int j1) {
        const bool there = !EXITS || kt < nk;
        const __amdgpu_buffer_rsrc_t g = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p.A), 0, there ? sizeA : 0, kBufferFlags);
#pragma unroll
        for (int j = j0; j < j1; ++j) DL_BLL16(g, offA[j], there ? kt * (BK * 2) : 0, S + blkA[j] * 512);
    };
    auto copyB = [&](bf16_t* S, int kt, int j0, int j1) {
        const bool there = !EXITS || kt < nk;
        const __amdgpu_buffer_rsrc_t g = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(p.B), 0, there ? sizeB : 0, kBufferFlags);
#pragma unroll
        for (int j = j0; j < j1; ++j) DL_BLL16(g, offB[j], there ? kt * (BK * 2) : 0, S + blkB[j] * 512);
    };
    auto ldfrag = [&](bf16x8* a, bf16x8* b, const bf16_t* S, const bf16_t* R, int kk) {
#pragma unroll
        for (int i = 0; i < TM; ++i) a[i] = *reinterpret_cast<const bf16x8*>(S + rdA[kk] + 32 * i * BK);
#pragma unroll
        for (int j = 0; j < TN; ++j) b[j] = *reinterpret_cast<const bf16x8*>(R + rdB[kk] + 32 * j * BK);
    };
    // serpentine order over the accumulator tiles: from one MFMA to the next exactly one operand changes
    auto mma = [&](const bf16x8* a, const bf16x8* b) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int jj = 0; jj < TN; ++jj) {
                const int j = (i & 1) ? TN - 1 - jj : jj;
                acc[i][j] = TR ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j], a[i], acc[i][j], 0, 0, 0)
                               : __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
            }
    };
    auto interleave = [&](auto ncopy_c) {
        SchedEven<TM * TN, TM + TN, decltype(ncopy_c)::value, RT, 0>::run();
        __builtin_amdgcn_sched_barrier(0);
    };

    // One k-tile = four phases of TM*TN MFMAs (16-wide k steps), each overlapped with the fragment reads of the next
    // phase.  Before the last phase the wavefront waits for its own copies of k-tile kt+1 and for all of its LDS reads
    // and meets the others at the one barrier of the k-tile; past it (a) k-tile kt+1 has landed for everyone and
    // (b) nobody reads the stages of kt any more, so the copies into them start right there: B of kt+SB in the last phase and the
    // first of the next k-tile, A of kt+SA in the two that follow.  Four phases with a quarter of the copies each: a wavefront
    // that issues more at a time waits in front of the copy path, and its MFMAs with it (128x256 on three, 517 x 24576, K = 4096:
    // 111.1 -> 106.8 us; the 25 of 810 problems that take this shape 4 % faster, the shapes of at most 192x192 0 to 2.5 %).  On two stages
    // there is no time for that, a copy has to land within a k-tile: A goes with the last phase, B with the first (the other way round,
    // 256x256 with 4096^3 and an fp32 output took 2 us more, the one product that this was measured on).
    // 192x256 and 256x192 have two stages of the operand with more to copy and four or three of the other: half of the copies get a
    // k-tile or two more to land (192x256, 3072 x 4096: K = 12288 250.8 -> 234.2 us, K = 4096 91.8 -> 88.2; the 48 problems that take one of
    // the two 9 % faster).
    // REM = k-tiles after this one, capped at SA (the steady state): with too few left a copy has nothing to fetch; the wait
    // leaves the copies younger than k-tile kt+1 in flight.
    constexpr bool SPREAD = SA > 2;
    constexpr int B0 = SPREAD ? JB / 2 : 0, A1 = SPREAD ? JA / 2 : JA;
    constexpr int U = SA % SB == 0 ? SA : SA * SB;       // k-tiles until the stages come round
    auto ktile = [&](auto i_c, int kt, auto rem_c) {
        constexpr int I = decltype(i_c)::value, REM = decltype(rem_c)::value;
        constexpr bool kB = REM >= SB, kB1 = REM >= SB - 1, kA = REM >= SA - 1;
        bf16_t *ca = sa.s[I % SA], *cb = sb.s[I % SB], *pa = sa.s[(I + SA - 1) % SA], *pb = sb.s[(I + SB - 1) % SB];
        ldfrag(a1, b1, ca, cb, 1);
        if (kB1) copyB(pb, kt + SB - 1, B0, JB);
        mma(a0, b0);
        interleave(std::integral_constant<int, (kB1 ? JB - B0 : 0)>{});
        ldfrag(a0, b0, ca, cb, 2);
        if (SPREAD && kA) copyA(pa, kt + SA - 1, 0, A1);
        mma(a1, b1);
        interleave(std::integral_constant<int, (SPREAD && kA ? A1 : 0)>{});
        ldfrag(a1, b1, ca, cb, 3);
        if (kA) copyA(pa, kt + SA - 1, A1, JA);
        mma(a0, b0);
        interleave(std::integral_constant<int, (kA ? JA - A1 : 0)>{});
        if constexpr (REM >= 1) {
            // younger than k-tile kt+1's last copy: B of kt+2 .. kt+SB-1 and A of kt+2 (SA > SB: kt+1+SA-SB) .. kt+SA-1
            constexpr int nB = (REM - 1 < SB - 2 ? REM - 1 : SB - 2);
            constexpr int lo = SA > SB ? 1 + SA - SB : 2, hi = SA - 1 < REM ? SA - 1 : REM;
            DL_WAIT_VM_LGKM0((nB > 0 ? nB : 0) * JB + (hi >= lo ? hi - lo + 1 : 0) * JA);
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            ldfrag(a0, b0, sa.s[(I + 1) % SA], sb.s[(I + 1) % SB], 0);
            if (kB) copyB(cb, kt + SB, 0, B0);
            if (!SPREAD && kB) copyA(ca, kt + SA, 0, JA);
            mma(a1, b1);
            interleave(std::integral_constant<int, (kB ? (SPREAD ? B0 : JA) : 0)>{});
        } else {
            mma(a1, b1);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    using std::integral_constant;
    // the first copies in the order of the main loop, up to what the last phase of a k-tile -1 would have issued
#pragma unroll
    for (int s = 0; s < SA; ++s) {
        const int kb = s - (SA - SB);
        if (kb >= 0) copyB(sb.s[kb], kb, 0, s + 1 < SA ? JB : B0);
        if (s + 1 < SA || !SPREAD) copyA(sa.s[s], s, 0, JA);
    }
    // k-tile 0 has landed (this wavefront's share): behind B of k-tile 0 come A of SA - SB (SA == SB: 1) .. SA - 2 and B of 1 .. SB - 1,
    // on two stages A of 1
    DL_WAIT_VM(SPREAD ? (SA == SB ? SB - 2 : SB - 1) * JA + (SB - 2) * JB + B0 : JA);
    __builtin_amdgcn_s_barrier();
    ldfrag(a0, b0, sa.s[0], sb.s[0], 0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (EXITS) {
        // every k-tile like one of the steady state, left behind the last one, whose copies fetch nothing.  Code for every
        // remainder, as below, spilled accumulators here.
        auto turn = [&](auto self, int kt, auto i_c) -> bool {
            constexpr int I = decltype(i_c)::value;
            ktile(i_c, kt + I, integral_constant<int, SA>{});
            if (I % 2 == 1 && kt + I + 1 == nk) return true;
            if constexpr (I + 1 < U) return self(self, kt, integral_constant<int, I + 1>{});
            return false;
        };
        for (int kt = 0; !turn(turn, kt, integral_constant<int, 0>{}); kt += U) {}
        DL_MFMA_SETTLE();
        DL_WAIT_VM(0);                                   // nothing is on its way into the LDS when the workgroup ends
    } else {
        // k-tiles kt .. kt + N - 1, of which the last has `AFTER` k-tiles behind it; k-tile kt sits in stage 0
        auto run = [&](auto self, int kt, auto i_c, auto n_c, auto after_c) {
            constexpr int I = decltype(i_c)::value, N = decltype(n_c)::value, AFTER = decltype(after_c)::value;
            ktile(i_c, kt + I, integral_constant<int, (N - 1 - I + AFTER < SA ? N - 1 - I + AFTER : SA)>{});
            if constexpr (I + 1 < N) self(self, kt, integral_constant<int, I + 1>{}, n_c, after_c);
        };
        int kt = 0;
        for (; kt + 2 * SA <= nk; kt += SA)              // whole turns of the stages in the steady state
            run(run, kt, integral_constant<int, 0>{}, integral_constant<int, SA>{}, integral_constant<int, SA>{});
        // SA .. 2 SA - 1 are left (the host takes a tile only for nk >= SA; nk is even, so with an even SA the rest is too)
        auto rest = [&](auto self, auto n_c) {
            constexpr int N = decltype(n_c)::value;
            if constexpr (N < 2 * SA) {
                if ((SA % 2 == 1 || N % 2 == 0) && nk - kt == N) {
                    run(run, kt, integral_constant<int, 0>{}, n_c, integral_constant<int, 0>{});
                    DL_MFMA_SETTLE();
                } else {
                    self(self, integral_constant<int, N + 1>{});
                }
            }
        };
        rest(rest, integral_constant<int, SA>{});
    }

    const int mw = m0 + (BM / WM) * wm, nw = n0 + (BN / WN) * wn;
    const int n_end = min(p.N, n0 + BN);
    if constexpr (TR) {
        store_tiles_vt<TM, TN>(p, acc, mw, nw, lane);
    } else if constexpr (EPI == EPI_RESID_F32) {
        if (mw + BM / WM <= p.M && nw + BN / WN <= n_end) store_resid_full<TM, TN>(p, acc, mw, nw, lane);
        else store_tiles<EPI, TM, TN>(p, acc, mw, nw, lane, n_end);
    } else {
        // (a tile that keys share with values goes element by element, and where there is one factor for all columns of a
        // wavefront tile, one that queries share with keys)
        const bool mixed = EPI == EPI_BF16 && (n_end > first_vt_col(p) ||
                                               (!kColFactors<TM, TN> && nw < p.scale_cols && nw + BN / WN > p.scale_cols));
        if (mixed) store_tiles<EPI, TM, TN>(p, acc, mw, nw, lane, n_end);
        else store_tiles_buf<EPI, TM, TN>(p, acc, mw, nw, lane, n_end);
    }
}

// A tile whose columns all go to p.vt runs on transposed accumulators; one that also holds other columns writes its share
// of p.vt in 8-byte pieces (16 of the 512 tiles of 3072 x 6144).  The transposing launch that used to follow the product took
// 3.5 us at 731 x 3456 (the product 12.6, now 12.4 with its V^T columns), 6.0 at 4096 x 3456 (33.8, now 36.0), 5.2 at 3072 x
// 2048 (45.4, now 46.6).  With a predicate and a 64-bit address per element, as the other epilogues had, this one took more
// than the launch it replaces (4096 x 3456: 45.6).
template <int BM, int BN, int EPI, int WM, int SA, int SB>
__device__ __forceinline__ void fast_tile(const GemmArgs& p, int m0, int n0, Stages<SA> sa, Stages<SB> sb) {
    if constexpr (EPI == EPI_BF16) {
        if (n0 >= first_vt_col(p) && p.vt_ld < (1 << 23)) {      // (32-bit offsets inside a wavefront tile)
            fast_tile_any<BM, BN, EPI, WM, SA, SB, true>(p, m0, n0, sa, sb);
            return;
        }
    }
    fast_tile_any<BM, BN, EPI, WM, SA, SB, false>(p, m0, n0, sa, sb);
}

// Two-stage tiles of at most 128x192 leave room for two workgroups per compute unit (at most 80 KB of LDS and 128
// accumulators each): one's prologue and epilogue hide under the other's main loop.
constexpr bool two_per_cu(int bm, int bn, int ns) { return bm == 128 && bn <= 192 && ns == 2; }
// stages of A: all of the LDS where B has two
constexpr int stages_a(int bm, int bn, int ns) { return bm == 192 && bn == 256 ? 4 : (bm == 256 && bn == 192 ? 3 : ns); }
template <int BM, int BN, int EPI, int WM, int NS>
__global__ __launch_bounds__(256, two_per_cu(BM, BN, NS) ? 2 : 1) void gemm_fast(GemmArgs p) {
    DL_STAGES(sa, stages_a(BM, BN, NS), BM * 64)
    DL_STAGES(sb, NS, BN * 64)
    const int tiles_m = (p.M + BM - 1) / BM, tiles_n = (p.N + BN - 1) / BN;
    int tm, tn;
    if (!tile_of(blockIdx.x, tiles_m, tiles_n, &tm, &tn)) return;
    fast_tile<BM, BN, EPI, WM, stages_a(BM, BN, NS), NS>(p, tm * BM, tn * BN, sa, sb);
}

// 256x256 tiles whose count is r full rounds of 256 workgroups plus a remainder of at most half a round: the last
// `n_split` tiles are computed as two 128x256 halves each, so the final round holds twice as many workgroups of
// half the work and ends in half the time instead of leaving most compute units idle for a whole tile time.
// Block b < n_big computes whole tile b (in the XCD-aware order), block n_big + 2 j + h half h of tile n_big + j.
template <int EPI>
__global__ __launch_bounds__(256) void gemm_fast_split_tail(GemmArgs p, int n_big) {
    DL_STAGES(sa, 2, 256 * 64)
    DL_STAGES(sb, 2, 256 * 64)
    const int tiles_m = (p.M + 255) / 256, tiles_n = (p.N + 255) / 256;
    const int b = blockIdx.x;
    const int v = b < n_big ? b : n_big + ((b - n_big) >> 1);
    int tm, tn;
    if (!tile_of(v, tiles_m, tiles_n, &tm, &tn)) return;
    if (b < n_big) {
        fast_tile<256, 256, EPI, 2, 2, 2>(p, tm * 256, tn * 256, sa, sb);
    } else {
        const int m0 = tm * 256 + 128 * ((b - n_big) & 1);
        if (m0 < p.M) fast_tile<128, 256, EPI, 2, 2, 2>(p, m0, tn * 256, sa, sb);
    }
}

// tile_of deals tiles to 8 XCDs in equal shares: the split needs every virtual index below `tiles` to be valid
constexpr bool splits_tail(long tiles) { return tiles > 256 && tiles % 8 == 0 && tiles % 256 > 0 && tiles % 256 <= 128; }

template <int BM, int BN, int EPI, int WM, int NS>
void launch_fast(const GemmArgs& a, hipStream_t st) {
    const int tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
    if (BM == 256 && BN == 256) {
        if (splits_tail(tiles)) {
            const int rem = tiles % 256, n_big = tiles - rem;
            hipLaunchKernelGGL((gemm_fast_split_tail<EPI>), dim3(n_big + 2 * rem), dim3(256), 0, st, a, n_big);
            return;
        }
    }
    const int grid = (tiles + 7) / 8 * 8;
    hipLaunchKernelGGL((gemm_fast<BM, BN, EPI, WM, NS>), dim3(grid), dim3(256), 0, st, a);
}

// Tile shapes of the fast path.  A launch takes rounds x (edge + k-tiles x step): a round is one workgroup on every compute
// unit (two where they share it), edge what a tile spends outside its main loop with each epilogue, step the time of one 64-deep
// k-tile with all compute units busy, in us.  The constants are one fit to the times of every shape on 810 problems (M 66 .. 16384
// against 36 outputs of 256 .. 24576 columns and reductions of 256 .. 12288, weights cold, as launches in a row), weighted to
// the shapes that come near the fastest; an added constant for the launch (1.8) is left out, being the same for all.  (Inside a
// layer, at the clock that a whole pass settles at, the same launches take up to a fifth longer.)  Median error 7 %; the shape
// taken is 0.5 % (geometric mean) slower than the fastest, 1.7 % of the problems lose more than 10 %.  Fitted without 342 of
// the problems, the choice loses 0.9 % on these.  (On the times of the kernels as they are now, which the test holds, the same
// table loses 0.8 %, and 2.0 % of the problems more than 10 %: the copies that were spread since made 192x256 and 256x192 8 % faster,
// 128x256 4 %, the others by up to 1 %.)  (A table fitted to M up to 4096 without a column for the residual, with one entry set by
// hand, and blind to the split tail, lost 3.0 % on all and 3.4 % on these: 4096 x 1152 residual outputs, K = 1152, 23.4 us where
// 128x128 tiles take 20.0; K = 4352, 51.6 where 192x128 take 46.4.)
// What separates the shapes: a compute unit takes in about 40 bytes per clock through the global -> LDS path whatever the tile,
// so large tiles need fewer bytes per flop and win as soon as there are rounds of them; and a copy takes up to ~1.3 us to
// land (weights cold), more than a small tile's k-tile lasts, so tiles of at most 128x160 run on four to eight stages
// (all of the LDS, one workgroup per compute unit).  517 x 4096 outputs, K = 12288: 200 us with 192x192 tiles on two
// stages, 159 with 128x128 on two, 86 on five, 78 with 128x96 on five; 731 x 1152, K = 4352: 35 -> 17 us (64x64 on eight).
struct TileShape {
    int bm, bn, ns;
    float step, edge[EPI_F32 + 1];                       // by epilogue: plain, residual, SwiGLU, GELU, fp32
    // 96 and 160 columns are an odd number of MFMA tiles: the four wavefronts are stacked in M there
    constexpr int waves_m() const { return bn % 64 ? 4 : 2; }
};
constexpr TileShape kTiles[] = {
    {256, 256, 2, 1.438f, {5.5f, 13.1f, 5.4f, 11.1f, 6.7f}}, {192, 256, 2, 1.246f, {4.7f, 8.8f, 3.1f, 8.7f, 2.2f}},
    {256, 192, 2, 1.156f, {6.6f, 10.4f, 6.6f, 9.9f, 9.4f}},  {128, 256, 3, 0.809f, {5.7f, 8.0f, 4.6f, 9.2f, 6.6f}},
    {192, 192, 3, 0.867f, {9.4f, 11.9f, 9.4f, 8.3f, 6.4f}},  {192, 128, 4, 0.632f, {4.8f, 8.5f, 4.5f, 7.2f, 7.3f}},
    {128, 192, 2, 1.362f, {0.8f, 4.2f, 0.8f, 2.9f, 4.0f}},   {128, 128, 2, 1.008f, {1.1f, 2.8f, 0.9f, 3.8f, 1.4f}},
    {128, 160, 4, 0.666f, {3.9f, 6.3f, 3.9f, 5.7f, 2.9f}},   {128, 128, 5, 0.553f, {1.5f, 2.7f, 1.9f, 3.0f, 1.5f}},
    {128, 96, 5, 0.397f, {3.2f, 5.4f, 3.2f, 4.5f, 4.3f}},    {128, 64, 6, 0.335f, {1.9f, 3.2f, 1.9f, 2.7f, 1.7f}},
    {64, 128, 6, 0.419f, {1.5f, 1.4f, 1.3f, 2.4f, 1.1f}},    {64, 64, 8, 0.261f, {1.3f, 1.6f, 1.3f, 1.8f, 1.0f}},
};
// gate/up pairs sit in one wavefront: an even number of 32-wide tile columns per wavefront
constexpr bool even_cols(const TileShape& t) { return t.bn % 128 == 0; }

// A last round with a fraction x of its workgroups takes less than a whole one (they have the chip to themselves, and behind
// other rounds they do not start together): 0.71 + 0.29 x; 0.79, less behind full rounds, where two workgroups share a compute unit
// and at most every other place is taken (x <= 1/2), from there up to 1; the split tail 0.71.  Fitted with the table above.
float rounds_of(const TileShape& t, int M, int N) {
    const long tiles = long((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
    const bool two = two_per_cu(t.bm, t.bn, t.ns);
    const long slots = two ? 512 : 256, full = tiles / slots, rest = tiles % slots;
    if (rest == 0) return float(full);
    if (t.bm == 256 && t.bn == 256 && splits_tail(tiles)) return float(full) + 0.71f;
    const float x = float(rest) / float(slots);
    const float least = two ? 0.79f / (1.0f + 0.21f * float(full)) : 0.71f;
    const float part = two ? (x > 0.5f ? 2.0f * x - 1.0f : 0.0f) : x;
    return float(full) + least + (1.0f - least) * part;
}

// ldo: the rows of a wavefront tile must span less than 2 GB, 4 bytes an element (wider outputs take the lower tiles; there is
// always the 64 rows of 128x128 on two stages)
int pick_tile(int M, int N, int K, int ldo, int epi) {
    const int nk = K / 64;
    int best = 0;
    float best_cost = 1e30f;
    for (int c = 0; c < int(sizeof(kTiles) / sizeof(kTiles[0])); ++c) {
        const TileShape& t = kTiles[c];
        if (nk < t.ns || (epi == EPI_SWIGLU_BF16 && !even_cols(t)) || size_t(t.bm / t.waves_m()) * size_t(ldo) >= (1u << 29)) continue;
        const float cost = rounds_of(t, M, N) * (t.edge[epi] + float(nk) * t.step);
        if (cost < best_cost) { best_cost = cost; best = c; }
    }
    return best;
}

template <int EPI, int C = 0>
void dispatch_fast(int c, const GemmArgs& a, hipStream_t st) {
    if constexpr (C < int(sizeof(kTiles) / sizeof(kTiles[0]))) {
        constexpr TileShape t = kTiles[C];
        if (c != C) return dispatch_fast<EPI, C + 1>(c, a, st);
        if constexpr (EPI != EPI_SWIGLU_BF16 || even_cols(t)) launch_fast<t.bm, t.bn, EPI, t.waves_m(), t.ns>(a, st);
    }
}

template <int EPI>
void dispatch_fast(const GemmArgs& a, hipStream_t st) {
    dispatch_fast<EPI>(pick_tile(a.M, a.N, a.K, a.ldo, EPI), a, st);
}

bool takes_tiles(const GemmArgs& a) {
    // fast path: K in whole pairs of 64-wide steps, 16-byte aligned rows, more rows than the few-rows kernel takes and
    // columns for a tile
    // (33 .. 64 rows over more than 8192 columns: a 64-row tile of this path reads A for 64 or 128 columns at a time, and
    // there are enough such tiles; 24576 x 4096 gate/up, 64 rows: 54 us with the few-rows kernel, 44 with 64x128 tiles)
    return a.K >= 128 && a.K % 128 == 0 && a.lda % 8 == 0 && a.ldb % 8 == 0 &&
                      (a.M > 64 || (a.M > 32 && a.N > 8192)) && a.N >= 64 && a.ldo < (1 << 23) &&
                      size_t(a.M) * a.lda * 2 < (1ull << 32) && size_t(a.N) * a.ldb * 2 < (1ull << 32);
}

bool takes_few_rows(const GemmArgs& a) {
    // few rows: 4-wide accesses to the outputs, the residual and the rows
    const bool aligned_out = a.epi == EPI_RESID_F32 || a.epi == EPI_F32
                                 ? (a.ldo % 4 == 0 && reinterpret_cast<uintptr_t>(a.out) % 16 == 0 &&
                                    (a.epi != EPI_RESID_F32 ||
                                     (a.ldr % 4 == 0 && reinterpret_cast<uintptr_t>(a.resid) % 16 == 0)))
                                 : (a.ldo % 4 == 0 && reinterpret_cast<uintptr_t>(a.out) % 8 == 0);
    return a.M <= 64 && a.K >= 64 && a.K % 64 == 0 && a.N % (a.epi == EPI_SWIGLU_BF16 ? 64 : 16) == 0 &&
                          a.lda % 8 == 0 && a.ldb % 8 == 0 && aligned_out &&
                          reinterpret_cast<uintptr_t>(a.A) % 16 == 0 && reinterpret_cast<uintptr_t>(a.B) % 16 == 0 &&
                          size_t(a.M) * a.lda * 2 < (1ull << 32) && size_t(a.N) * a.ldb * 2 < (1ull << 32);
}

}  // namespace

namespace {
// (the product is one of gemm_few_rows' with the rotary epilogue)
bool takes_qkv_post(const GemmArgs& a, const QkvPostArgs& q) {
    return a.M >= 1 && a.N >= 1 && a.vt && !takes_tiles(a) && takes_few_rows(a) && q.dh % 32 == 0 && q.q_off == 0 && q.k_off % q.dh == 0 &&
           a.vt_col % q.dh == 0 && a.out == q.qkv && a.ldo == q.n_qkv;
}
}  // namespace

bool gemm_qkv_post(const GemmArgs& a, const QkvPostArgs& q, hipStream_t st) {
    if (!takes_qkv_post(a, q)) return false;
    launch_few_rows<EPI_QKV_POST>(a, st, q);
    return true;
}

// Every workgroup makes all rows for itself, which pays for the launch it saves while there is one workgroup to a compute unit and the
// rows are short.  A product that writes the rows, then normalisation and product in two launches / in one, us: 16 rows, K = 256,
// RMSNorm 4096 columns 8.2 / 6.9, 8192 8.0 / 8.0, 24576 11.0 / 12.9; LayerNorm 512 columns 7.9 / 7.4, 4096 7.6 / 7.7, 8192 8.2 / 9.1, 24576
// 11.2 / 15.7; 32 rows 12288 columns 10.0 / 10.2, 16384 10.8 / 11.5; 64 rows 8192 10.6 / 10.5.  16 rows, K = 1024: RMSNorm 2048 columns 7.8 / 7.9,
// 8192 8.6 / 8.8; LayerNorm 512 columns 8.0 / 8.3, 4096 8.0 / 8.7.
bool norm_pays(const GemmArgs& a, int kind) {
    if (a.M > 16 && a.K <= 256) return a.N <= 12288;
    return a.N <= 4096 && long(a.N) * a.K <= (kind == 1 && a.K > 512 ? 1L << 19 : 1L << 21);
}

bool gemm_takes_norm(const GemmArgs& a, const NormIn& n, const QkvPostArgs* q) {
    const int bm = a.M <= 16 ? 16 : (a.M <= 32 ? 32 : 64);
    return a.M > 1 && norm_pays(a, n.kind) && a.N >= 1 && !takes_tiles(a) && takes_few_rows(a) && a.K >= 128 && a.K <= max_norm_k(bm) && a.lda == a.K &&
           (reinterpret_cast<uintptr_t>(n.x) | reinterpret_cast<uintptr_t>(n.g) | reinterpret_cast<uintptr_t>(n.b)) % 16 == 0 &&
           (q ? takes_qkv_post(a, *q) : a.epi == EPI_BF16 || a.epi == EPI_SWIGLU_BF16 || a.epi == EPI_GELU_BF16);
}

void gemm_normed(const GemmArgs& a, const NormIn& n, const QkvPostArgs* q, hipStream_t st) {
    if (q) launch_few_rows_norm<EPI_QKV_POST>(a, n, st, *q);
    else if (a.epi == EPI_BF16) launch_few_rows_norm<EPI_BF16>(a, n, st);
    else if (a.epi == EPI_SWIGLU_BF16) launch_few_rows_norm<EPI_SWIGLU_BF16>(a, n, st);
    else launch_few_rows_norm<EPI_GELU_BF16>(a, n, st);
}

void gemm(const GemmArgs& a, hipStream_t st) {
    if (a.M <= 0 || a.N <= 0) return;
    // the residual epilogue addresses out and resid with 32-bit element offsets: split the rows of larger outputs
    if (a.epi == EPI_RESID_F32 && a.M > 1 &&
        (size_t(a.M) * size_t(a.ldo) >= (1ull << 31) || size_t(a.M) * size_t(a.ldr) >= (1ull << 31))) {
        const int m1 = a.M / 2;
        GemmArgs lo = a, hi = a;
        lo.M = m1;
        hi.M = a.M - m1;
        hi.A = a.A + size_t(m1) * a.lda;
        hi.out = static_cast<float*>(a.out) + size_t(m1) * a.ldo;
        hi.resid = a.resid + size_t(m1) * a.ldr;
        gemm(lo, st);
        gemm(hi, st);
        return;
    }
    if (takes_tiles(a)) {
        switch (a.epi) {
            case EPI_BF16: dispatch_fast<EPI_BF16>(a, st); return;
            case EPI_RESID_F32: dispatch_fast<EPI_RESID_F32>(a, st); return;
            case EPI_SWIGLU_BF16: dispatch_fast<EPI_SWIGLU_BF16>(a, st); return;
            case EPI_GELU_BF16: dispatch_fast<EPI_GELU_BF16>(a, st); return;
            case EPI_F32: dispatch_fast<EPI_F32>(a, st); return;
            default: break;
        }
    }
    if (takes_few_rows(a)) {
        switch (a.epi) {
            case EPI_BF16: launch_few_rows<EPI_BF16>(a, st); return;
            case EPI_RESID_F32: launch_few_rows<EPI_RESID_F32>(a, st); return;
            case EPI_SWIGLU_BF16: launch_few_rows<EPI_SWIGLU_BF16>(a, st); return;
            case EPI_GELU_BF16: launch_few_rows<EPI_GELU_BF16>(a, st); return;
            default: launch_few_rows<EPI_F32>(a, st); return;
        }
    }
    const int tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
    dim3 grid(tiles), block(256);
    switch (a.epi) {
        case EPI_BF16: hipLaunchKernelGGL(gemm_generic<EPI_BF16>, grid, block, 0, st, a); break;
        case EPI_RESID_F32: hipLaunchKernelGGL(gemm_generic<EPI_RESID_F32>, grid, block, 0, st, a); break;
        case EPI_SWIGLU_BF16: hipLaunchKernelGGL(gemm_generic<EPI_SWIGLU_BF16>, grid, block, 0, st, a); break;
        case EPI_GELU_BF16: hipLaunchKernelGGL(gemm_generic<EPI_GELU_BF16>, grid, block, 0, st, a); break;
        default: hipLaunchKernelGGL(gemm_generic<EPI_F32>, grid, block, 0, st, a); break;
    }
}

}  // namespace dlk

// For tests (host only): whether a product with contiguous operands takes the LDS-staged tiles, and which.
extern "C" __attribute__((visibility("default"))) int32_t dlk_gemm_tile(int32_t M, int32_t N, int32_t K, int32_t epi, int32_t* bm, int32_t* bn, int32_t* stages) {
    dlk::GemmArgs a{};
    a.lda = a.ldb = a.K = K;
    a.ldo = epi == dlk::EPI_SWIGLU_BF16 ? N / 2 : N;
    a.M = M;
    a.N = N;
    if (!dlk::takes_tiles(a)) return 0;
    const dlk::TileShape& t = dlk::kTiles[dlk::pick_tile(M, N, K, a.ldo, epi)];
    *bm = t.bm;
    *bn = t.bn;
    *stages = t.ns;
    return 1;
}
