// fp32 GEMM on the fp32 matrix instructions:  C[M,N] = epilogue(A[M,K] * B[N,K]^T), plain row-major weights.
//
// The fp32 configuration is small (hundreds of rows, hundreds of columns), so a product is bound by the
// serial walk over K and by how few workgroups there are, not by arithmetic.  A workgroup therefore takes a
// small tile (16 x 16, or 32 x 32 where that still gives two workgroups per CU) and its waves split K; the
// partial tiles meet in LDS and are added in wave order.  Both operands are K-contiguous, so they go
// straight from memory to registers: with v_mfma_f32_16x16x4_f32 a lane supplies one k of one row, and which
// four k an instruction takes is free as long as A and B agree, so a lane loads 4 consecutive k of its
// row (16 bytes) and feeds them to four instructions.  The instruction multiplies and adds in fp32 like fmaf.
//
// Measured against the 64 x 64 FMA tile of kernels_generic.hip: 4 x 256 <- 1024 133 -> 11 us, 4 x 768 <- 256
// 39 -> 6 us (a launch), 1 x 6144 <- 2048 264 -> 15 us, 1000 x 6144 <- 2048 754 -> 366 us, 4096 x 6144 <- 2048
// 2794 -> 1421 us (73 TFLOP/s, bound by the operand reads: a 32 x 32 tile fetches 4 bytes per 32 flop).
//
// NORM: the rows of A are normalised on the way.  Every workgroup reads whole rows of A (K is the row), so it sums their
// squares beside the product, multiplies the operand by the gain and the finished sums by the row's factor: the norm's
// launch, 2 - 3 us of a step of some 40, is saved for a few vector instructions per load.
#include "pd_internal.h"

namespace pd {

typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float silu_precise(float z) { return z / (1.0f + expf(-z)); }

// MB x MB blocks of 16 x 16 per workgroup, W waves along K, U 16-wide k-steps requested at a time
template <int MB, int W, int U, int EPI, bool NORM = false>
__global__ __launch_bounds__(64 * W) void gemm_f32_mfma_kernel(GemmArgs a)
{
    static_assert(!NORM || MB == 1, "one row per lane");
    constexpr int BT = 16 * MB, NM = EPI == EPI_SWIGLU ? 2 : 1;   // NM: weight matrices (gate and up)
    __shared__ f32x4 red[W][NM * MB * MB][64];
    __shared__ float sq[NORM ? W : 1][16];

    int row0, row_end, group = 0;
    if (a.group_offsets) {
        int acc = 0;
        row0 = -1;
        row_end = 0;
        for (int g = 0; g < a.n_groups; ++g) {
            const int lo = a.group_offsets[g], hi = a.group_offsets[g + 1];
            const int nt = (hi - lo + BT - 1) / BT;
            if ((int)blockIdx.y < acc + nt) {
                group = g;
                row0 = lo + ((int)blockIdx.y - acc) * BT;
                row_end = hi;
                break;
            }
            acc += nt;
        }
        if (row0 < 0) return;
    } else {
        row0 = blockIdx.y * BT;
        row_end = a.M;
    }
    const int col0 = blockIdx.x * BT;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l15 = lane & 15, kg = (lane >> 4) * 4;

    const float *ap[MB], *bp[NM][MB];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        int r = min(row0 + 16 * i + l15, row_end - 1);            // clamped rows and columns are never stored
        if (a.a_gather) r = a.a_gather[r];
        ap[i] = (const float *)a.A + (size_t)r * a.lda;
        const size_t c = (size_t)group * a.b_group_stride + (size_t)min(col0 + 16 * i + l15, a.N - 1) * a.ldb;
        bp[0][i] = (const float *)a.B + c;
        if (EPI == EPI_SWIGLU) bp[NM - 1][i] = (const float *)a.B1 + c;
    }

    f32x4 acc[NM][MB][MB];
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < MB; ++j) acc[m][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    float ss = 0.f;                                               // NORM: this lane's part of its row's sum of squares
    const int steps = (a.K + 15) / 16, per = (steps + W - 1) / W;
    const int s1 = min(steps, (wave + 1) * per);
    for (int s0 = wave * per; s0 < s1; s0 += U) {
        f32x4 fa[U][MB], fb[U][NM][MB], fg[NORM ? U : 1];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = (s0 + u) * 16 + kg, kc = min(k, a.K - 4);
            const bool ok = s0 + u < s1 && k < a.K;               // K is a multiple of 4: a chunk is all in or all out
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                const f32x4 va = *(const f32x4 *)(ap[i] + kc);
                fa[u][i] = ok ? va : zero;
                if (NORM) fg[u] = *(const f32x4 *)(a.norm_g + kc);
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    const f32x4 vb = *(const f32x4 *)(bp[m][i] + kc);
                    fb[u][m][i] = ok ? vb : zero;
                }
            }
        }
        if (NORM)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const f32x4 x = fa[u][0];
                ss += (x[0] * x[0] + x[1] * x[1]) + (x[2] * x[2] + x[3] * x[3]);
                fa[u][0] = x * fg[u];
            }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int m = 0; m < NM; ++m)
#pragma unroll
                    for (int i = 0; i < MB; ++i)
#pragma unroll
                        for (int j = 0; j < MB; ++j)
                            acc[m][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[u][i][e], fb[u][m][j][e], acc[m][i][j], 0, 0, 0);
    }

#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < MB; ++j) red[wave][(m * MB + i) * MB + j][lane] = acc[m][i][j];
    if (NORM) {
        ss += __shfl_xor(ss, 16, 64);
        ss += __shfl_xor(ss, 32, 64);
        if (lane < 16) sq[wave][lane] = ss;
    }
    __syncthreads();
    float *C = (float *)a.C;
    const float *R = (const float *)a.R;
    // a lane's four accumulators: column lane % 16, rows 4 (lane / 16) .. + 3 of the block
    for (int q = threadIdx.x; q < MB * MB * 64; q += 64 * W) {
        const int blk = q >> 6, l = q & 63;
        f32x4 v = red[0][blk][l], w = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int z = 1; z < W; ++z) v += red[z][blk][l];
        if (EPI == EPI_SWIGLU) {
            w = red[0][MB * MB * (NM - 1) + blk][l];
#pragma unroll
            for (int z = 1; z < W; ++z) w += red[z][MB * MB * (NM - 1) + blk][l];
        }
        const int c = col0 + 16 * (blk % MB) + (l & 15);
        if (c >= a.N) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = row0 + 16 * (blk / MB) + 4 * (l >> 4) + r;
            if (m >= row_end) break;
            float x = v[r];
            if (NORM) {
                float t = sq[0][4 * (l >> 4) + r];
#pragma unroll
                for (int z = 1; z < W; ++z) t += sq[z][4 * (l >> 4) + r];
                const float inv = rsqrtf(t / (float)a.K + a.norm_eps);
                x *= inv;
                w[r] *= inv;
            }
            if (EPI == EPI_RESIDUAL) x += R[(size_t)m * a.ldr + c];
            if (EPI == EPI_SWIGLU) x = silu_precise(x) * w[r];
            C[(size_t)m * a.ldc + c] = x;
        }
    }
}

// 16-byte operand loads: rows of both operands start on 16 bytes.  Row tiles go over a grid dimension, which holds
// 65535: with tiles of 32 rows that is half of what the plain form's 64-row tiles reach.
bool gemm_f32_mfma_supported(const GemmArgs &a)
{
    const long long row_tiles = ((long long)a.M + 31) / 32 + (a.group_offsets ? a.n_groups : 0);
    // Up to 64 k a wave has one of the four k-steps that it requests; with outputs enough to fill the chip several times
    // over that costs more than the plain form's 64 x 64 tiles do.  Plain -> this form, us, at K = 64 and 96: 10000 x 1000
    // 65 -> 83, 88 -> 70; 5000 x 5000 123 -> 181, 171 -> 141; 2000 x 1000 (2016 tiles) 22 -> 22, 29 -> 19; 1000 x 768 16 -> 12.
    if (a.K <= 64 && row_tiles * ((a.N + 31) / 32) >= 2048) return false;
    return row_tiles <= 65535 && a.M > 0 && a.N > 0 && a.K >= 4 && a.K % 4 == 0 && a.lda % 4 == 0 && a.ldb % 4 == 0 && a.b_group_stride % 4 == 0 &&
           (((uintptr_t)a.A | (uintptr_t)a.B | (uintptr_t)(a.epilogue == EPI_SWIGLU ? a.B1 : nullptr)) & 15) == 0;
}

// K is the whole row, and the small tiles are taken (see launch_gemm_f32_mfma)
static bool small_tiles(const GemmArgs &a) { return (long long)((a.M + 31) / 32) * ((a.N + 31) / 32) < 512; }
bool gemm_f32_norm_supported(const GemmArgs &a)
{
    return gemm_f32_mfma_supported(a) && small_tiles(a) && !a.a_gather && !a.group_offsets && a.epilogue != EPI_RESIDUAL &&
           ((uintptr_t)a.norm_g & 15) == 0;
}

template <int MB, int W, int U = 4>
static hipError_t launch_f32(const GemmArgs &a, hipStream_t s)
{
    const dim3 grid((unsigned)((a.N + 16 * MB - 1) / (16 * MB)),
                    (unsigned)((a.M + 16 * MB - 1) / (16 * MB) + (a.group_offsets ? a.n_groups : 0)));
    if constexpr (MB == 1)
        if (a.norm_g) {
            if (a.epilogue == EPI_SWIGLU) gemm_f32_mfma_kernel<1, W, U, EPI_SWIGLU, true><<<grid, 64 * W, 0, s>>>(a);
            else gemm_f32_mfma_kernel<1, W, U, EPI_NONE, true><<<grid, 64 * W, 0, s>>>(a);
            return hipGetLastError();
        }
    switch (a.epilogue) {
    case EPI_NONE: gemm_f32_mfma_kernel<MB, W, U, EPI_NONE><<<grid, 64 * W, 0, s>>>(a); break;
    case EPI_RESIDUAL: gemm_f32_mfma_kernel<MB, W, U, EPI_RESIDUAL><<<grid, 64 * W, 0, s>>>(a); break;
    default: gemm_f32_mfma_kernel<MB, W, U, EPI_SWIGLU><<<grid, 64 * W, 0, s>>>(a); break;
    }
    return hipGetLastError();
}

hipError_t launch_gemm_f32_mfma(const GemmArgs &a, hipStream_t s)
{
    // two workgroups per CU: below that the small tile's four times as many workgroups are worth its extra reads
    if (!small_tiles(a)) return launch_f32<2, 4>(a, s);
    // small tiles: eight waves once each of them has a full round of k-steps to itself
    if (a.K < 512) return launch_f32<1, 4>(a, s);
    // Eight k-steps at a time halve a wave's round trips, but requests past its last k-step are made and multiplied all the
    // same: only where four at a time would make as many.  us, four -> eight: gate/up of 1 row, K = 2048 18.9 -> 14.5, K = 1024
    // 10.3 -> 9.7, 500 rows K = 896 52 -> 46; where they are more, 40 rows: K = 512 11.8 -> 17.8, 1040 22.0 -> 26.2 (100 rows),
    // 1536 22.5 -> 28.2, 2304 35.1 -> 40.8.
    const int per = ((a.K + 15) / 16 + 7) / 8;
    return (per + 7) / 8 * 2 == (per + 3) / 4 ? launch_f32<1, 8, 8>(a, s) : launch_f32<1, 8>(a, s);
}

}  // namespace pd
