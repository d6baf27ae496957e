// bf16 GEMM on the CDNA4 matrix cores:  C[M,N] = epilogue(A[M,K] * B[N,K]^T), fp32 accumulation.
//
// Both operands are K-contiguous, which is exactly the per-lane operand layout of v_mfma_f32_16x16x32_bf16 (each
// lane supplies 8 consecutive k of one row / column), so tiles go global -> LDS with the direct-to-LDS 16-byte
// loads of gfx950 (no staging registers, no LDS write instructions) and LDS -> registers with 16-byte reads, with
// no transposition anywhere.  A direct load puts lane i's 16 bytes at LDS offset base + 16*i, so the XOR swizzle
// that keeps the fragment reads of A free of bank conflicts is applied on the global side: the lane that owns LDS
// slot (row, s) fetches chunk s ^ ((row >> 1) & 7) of that row.  The weight operand B arrives in the packed block
// layout of pd_internal.h (1 KB blocks of 16 rows x 32 k): one direct-to-LDS instruction moves one block, blocks
// sit linearly in LDS, and a fragment is one block, read contiguously.
//
// A workgroup is four waves, one per SIMD, and a wave's tile is as large as its registers allow (128 x 128 of a
// 256 x 256 tile: 256 accumulator registers, 128 for two sets of fragments).  What bounds the large products is
// power: at full matrix rate the clock falls until the card stays inside its limit, so a flop's energy counts, and
// that is the multipliers' and the LDS reads'.  Large wave tiles read 128 KB of LDS per 64-wide k-tile of 256 x 256
// (eight waves of 128 x 64: 192 KB, which with the incoming 64 KB also keeps the LDS busy all the time), and
// 16x16x32 runs at a higher clock than 32x32x16 at the same rate of flops (half the accumulator traffic).
// With one wave per SIMD nothing else covers a wave's waits, so the k-loop is written as one instruction stream:
// between the MFMAs of half a k-tile stand the LDS reads of the next half's fragments and the direct-to-LDS
// requests of a later tile, a few MFMAs apart (a request occupies the CU's address unit for 16 clocks and the four
// waves issue theirs together, so closer than about five MFMAs they hold up the stream).  One barrier per k-tile.
// Measured, gate / up of the 8B shape at 8192 rows: 2300 clocks per k-tile for 2048 of MFMA issue (3700 with eight
// waves of 128 x 64 and 32x32x16, the reads of each fragment right ahead of its use), 1160 -> 1480 TFLOP/s; a
// request every four MFMAs 2640 clocks, the reads' spread does not matter there.
//
// Epilogues: plain store, residual add, and SwiGLU.  For SwiGLU the weight is packed at layer creation as
// alternating 32-row blocks (gate rows j..j+31, then up rows j..j+31); two blocks of 16 columns that lie 32 apart
// then hold gate and up of the same (row, column) in the same lane and register, and silu(gate)*up is formed
// without any data exchange.
//
// Optional row gather on A and per-group B matrices serve the mixture-of-experts grouped GEMM.
//
// Decode-sized problems (M <= 256) have too few output tiles to occupy 256 CUs while the weights stream from HBM,
// so K is split over gridDim.y: each split writes an fp32 partial tile and a second small kernel adds the splits in
// a fixed order and applies the epilogue (deterministic, no atomics).
#include <string.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "pd_internal.h"

namespace pd {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

constexpr int BK = 64;  // k per tile: 8 chunks of 16 bytes per row

__device__ __forceinline__ int swz(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }

__device__ __forceinline__ float silu_fast(float z) { return z / (1.0f + __expf(-z)); }

// The same for |z| < kSiluNear, bit for bit (all such z compared; -0 gives +0): the quotient by the hardware reciprocal and
// one correction from its remainder, without the division's steps for operands and results near the ends of the exponent's
// range.  The tiles take it where all gates of a wave's eight columns are that small, else the division (an infinite gate's
// correction would be inf - inf).  Gate/up of the 8B shape, division everywhere -> this: 8192 rows 1320 -> 1284 us, codes 672 ->
// 657, 2048 rows of 5632 <- 1024 27.7 -> 26.5; the look at the gates costs nothing that shows.
constexpr float kSiluNear = 87.f;
__device__ __forceinline__ float silu_near(float z)
{
    const float d = 1.0f + __expf(-z), r = __builtin_amdgcn_rcpf(d), q = z * r;
    return fmaf(fmaf(-d, q, z), r, q);
}

// acc += w x with acc in AGPRs
__device__ __forceinline__ void mfma_agpr(f32x4 &acc, const bf16x8 &w, const bf16x8 &x)
{
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(w), "v"(x));
}
__device__ __forceinline__ void mfma_agpr(f32x4 &acc, const i32x8 &w, const i32x8 &x)
{
    asm volatile("v_mfma_f32_16x16x128_f8f6f4 %0, %1, %2, %0" : "+a"(acc) : "v"(w), "v"(x));
}

template <class F, int... I>
__device__ __forceinline__ void static_for_seq(F f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
// f(0), ..., f(N - 1) with the index a compile-time constant
template <int N, class F>
__device__ __forceinline__ void static_for(F f)
{
    if constexpr (N > 0) static_for_seq(f, std::make_integer_sequence<int, N>{});
}

// Stages and schedule of a tile form.  LDS holds NS stages of the A tile, and of the B tile as many as the rest of the
// workgroup's share (a CU's 160 KB, or half of it) takes: the weights come from HBM, the rows mostly from an L2, so what
// can be requested further ahead is the weights.  Positions are in 64ths of half a k-tile, counted from the barrier: A's
// requests are spread over PA of them, B's over the PB behind; the fragment reads of a half over the first RS.
template <int BM, int BN, int WAVES, int NS>
struct TileRing {
    static constexpr bool pair = BM * BN <= 128 * 128 && NS == 2;     // two workgroups share a CU
    static constexpr int share = (pair ? 80 : 160) * 1024, SA = BM * BK * 2, SB = BN * BK * 2;
    static constexpr int NSA = NS, NSB = (share - NSA * SA) / SB < 8 ? (share - NSA * SA) / SB : 8;
    static constexpr int A_LD = BM / 8 / WAVES, B_LD = BN / 8 / WAVES, LD = A_LD + B_LD;   // requests of a wave per k-tile
    static constexpr int PA = 48, PB = 72;
    static constexpr int RS = BM * BN >= 256 * 192 ? 48 : 28;
    static constexpr size_t lds = (size_t)(NSA * SA + NSB * SB);
    static_assert(NSB > NSA || (NSA == 2 && NSB == 2), "B at least as far ahead as A");
    static_assert(BM % (8 * WAVES) == 0 && BN % (8 * WAVES) == 0, "loader mapping");
    // requests issued ahead of position p
    static constexpr int issued(int p)
    {
        int n = 0;
        for (int d = 0; d < LD; ++d) n += (d < A_LD ? d * PA / A_LD : PA + (d - A_LD) * PB / B_LD) < p;
        return n;
    }
    // of n fragment reads, those issued ahead of MFMA m of nm
    static constexpr int reads(int m, int nm, int n)
    {
        const int r = m * n * 64 / (RS * nm);
        return m == nm || r > n ? n : r;
    }
};

// F8: both operands are E4M3 codes and the caller passes them as if two codes were one bf16 element (K, lda, ldb
// halved; the weight pack is the bf16 pack of that view), so every byte moves exactly as above.  Two 16-byte
// fragments of a lane, of the two halves of the k-tile, form the 32-byte operand of v_mfma_f32_16x16x128_f8f6f4:
// which of the 128 k of the step a byte stands for does not matter as long as both operands are assembled the same
// way, and they are.  An MFMA needs both halves of k, so the halves of the loop are the upper and the lower row
// blocks of the wave's tile instead, with B's fragments in two register sets.  The fp32 sums are multiplied by the
// scale of their activation row and of their weight row before any epilogue.
template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int NS, bool F8>
__device__ __forceinline__ void gemm_mfma_body(const GemmArgs &a, int tiles_m, int tiles_n, int kt_per_split)
{
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;   // wave tile
    constexpr int MB = WM / 16, NB = WN / 16;             // 16x16 blocks per wave
    static_assert((!F8 || MB % 2 == 0) && NB % (EPI == EPI_SWIGLU ? 4 : 2) == 0, "blocks go in pairs, gate and up in pairs of pairs");
    constexpr int NW = WAVES_M * WAVES_N;
    using Ring = TileRing<BM, BN, NW, NS>;
    constexpr int NSA = Ring::NSA, NSB = Ring::NSB, A_LD = Ring::A_LD, B_LD = Ring::B_LD, LD = Ring::LD;
    constexpr unsigned SA = Ring::SA, SB = Ring::SB, B0 = NSA * SA;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

    // ---- tile id: contiguous ranges of tiles per XCD, 8-row bands inside ------------------------
    // A grouped launch has a row tile per group more than its rows may need.  Only the tiles in use are dealt: dealt
    // with the empty ones, these fall together on the last XCDs, and the others do their share.  Before -> now, us
    // (8 experts of the 8B shape): 128 rows gate/up 372 -> 343 (5.5 TB/s), down 248 -> 163 (5.8 TB/s); 11990 rows
    // gate/up 3209 -> 2947.
    if (a.group_offsets) {
        tiles_m = 0;
        for (int g = 0; g < a.n_groups; ++g) tiles_m += (a.group_offsets[g + 1] - a.group_offsets[g] + BM - 1) / BM;
    }
    const int n_tiles = tiles_m * tiles_n;
    if ((int)blockIdx.x >= n_tiles) return;
    struct Tile {
        int row0, row_end, col0, group;
    };
    auto tile_at = [&](int pid) {
        const int per = n_tiles / 8;
        if (per > 0) {
            // blocks are dealt to the 8 XCDs round-robin; give each XCD one contiguous range
            const int xcd = pid % 8, j = pid / 8;
            if (j < per) pid = xcd * per + j;       // the leftover tiles behind 8 * per keep their order
        }
        constexpr int GM = 8;
        const int band = pid / (GM * tiles_n);
        const int first = band * GM;
        const int rows = tiles_m - first < GM ? tiles_m - first : GM;
        const int in = pid - band * GM * tiles_n;
        const int tm = first + in % rows;
        Tile t;
        t.col0 = in / rows * BN;
        t.row0 = tm * BM;
        t.row_end = a.M;
        t.group = 0;
        if (a.group_offsets) {                        // virtual m-tiles map to groups
            int acc = 0;
            for (int g = 0; g < a.n_groups; ++g) {
                const int lo = a.group_offsets[g], hi = a.group_offsets[g + 1];
                const int nt = (hi - lo + BM - 1) / BM;
                if (tm < acc + nt) {
                    t.group = g;
                    t.row0 = lo + (tm - acc) * BM;
                    t.row_end = hi;
                    break;
                }
                acc += nt;
            }
        }
        return t;
    };
    // rows of (packed) B; a split-K launch of a SwiGLU GEMM works on the packed columns
    const int n_cols = (EPI == EPI_SWIGLU || (EPI == EPI_PARTIAL && a.epilogue == EPI_SWIGLU)) ? 2 * a.N : a.N;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int kt0 = blockIdx.y * kt_per_split;
    const int kt1 = min(a.K / BK, kt0 + kt_per_split);

    // ---- loader: a request of A covers 8 rows x 128 bytes = 1 KB of LDS, lane l owns slot (row = 8*blk + l/8,
    //      s = l%8) and fetches chunk s ^ swizzle(row) of that row; a request of B is one packed block ------------
    // A lane's offsets from the tile's first row and column block stay the same from tile to tile; the tile's place is in
    // the (scalar) base, the k-tile in the scalar offset, and the buffer ends with the tile's last row or block, so rows
    // and columns past it read as zeros (they are never stored).  Gathered rows have offsets of their own per tile.
    uint32_t off[LD];
    const int kblocks = a.K >> 5;                      // 32-k blocks per row block
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
        const int r = (wave * A_LD + i) * 8 + (lane >> 3);
        off[i] = (uint32_t)r * (uint32_t)(a.lda * 2) + swz(r, lane & 7) * 16;
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
        const int j = wave * B_LD + i;                // row block j/2 of the tile, k block j%2
        off[A_LD + i] = ((uint32_t)(j >> 1) * (uint32_t)kblocks + (j & 1)) * 1024u + lane * 16;
    }
    const char *abase, *bbase;
    uint32_t abytes, bbytes;
    // lane number the compiler knows nothing about: what is computed from it per tile is not kept in registers meanwhile
    auto opaque_lane = [&]() {
        int l = lane;
        asm volatile("" : "+v"(l));
        return l;
    };
    auto aim_a = [&](const Tile &t) {
        if (a.a_gather) {
            abase = (const char *)a.A;
            abytes = 0xffffffffu;
            const int l = opaque_lane();
#pragma unroll
            for (int i = 0; i < A_LD; ++i) {
                const int r = (wave * A_LD + i) * 8 + (l >> 3);
                off[i] = (uint32_t)a.a_gather[min(t.row0 + r, t.row_end - 1)] * (uint32_t)(a.lda * 2) + swz(r, l & 7) * 16;
            }
        } else {
            abase = (const char *)a.A + (size_t)t.row0 * (size_t)(a.lda * 2);
            abytes = (uint32_t)(t.row_end - t.row0) * (uint32_t)(a.lda * 2);
        }
    };
    auto aim_b = [&](const Tile &t) {
        bbase = (const char *)a.B + ((size_t)t.group * a.b_group_stride + (size_t)t.col0 * a.K) * 2;
        bbytes = (uint32_t)((n_cols - t.col0 + 15) >> 4) * (uint32_t)kblocks * 1024u;
    };
    typedef void __attribute__((address_space(3))) *lptr_t;
    // request D of k-tile ka of A into the stage at sa, or of k-tile kb of B into the one at sb
    auto request = [&](auto D, int ka, unsigned sa, int kb, unsigned sb) {
        constexpr int d = decltype(D)::value;
        if constexpr (d < A_LD)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void *)abase, 0, abytes, 0x00020000),
                                                     (lptr_t)(smem + sa + (wave * A_LD + d) * 1024), 16, off[d],
                                                     ka * (BK * 2), 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void *)bbase, 0, bbytes, 0x00020000),
                                                     (lptr_t)(smem + sb + (wave * B_LD + d - A_LD) * 1024), 16, off[d],
                                                     kb * 2048, 0, 0);       // two 1 KB k-blocks per tile
    };

    // Accumulators beyond what 256 registers leave room for have to stay in the AGPR half of the file: with the builtins
    // the compiler moved some of them back and forth inside the loop, in some epilogues' kernels up to 335 moves per
    // k-tile (2300 -> 3000 clocks).  The MFMA as an asm statement on AGPR operands leaves it no choice.  The statements
    // hide from the compiler that they are MFMAs, so the waits between a register's last vector write and the first
    // MFMA, and between the last MFMA and the first read, are written out; inside the loop the operands come from LDS
    // reads, whose counter the compiler keeps for asm operands too.
    constexpr bool kAgpr = MB * NB > (F8 ? 16 : 32);
    f32x4 acc[MB][NB];
    auto pin_acc = [&]() {
        if constexpr (kAgpr)
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) asm volatile("" : "+a"(acc[i][j]));
    };

    // ---- fragments.  bf16: set h holds k half h of the tile.  F8: whole operands, their 16-byte parts the two
    //      halves; two sets of B's -----------------------------------------------------------------------------------
    const int fr = lane & 15, kg = lane >> 4;
    bf16x8 xf[2][MB], wf[2][NB];                      // bf16
    i32x8 x8[MB], w8[2][NB];                          // F8
    const unsigned char *xa[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) xa[h] = smem + (wm * WM + fr) * 128 + swz(fr, 4 * h + kg) * 16;
    const unsigned char *wa = smem + wn * NB * 2048 + lane * 16;
    auto half_into = [&](i32x8 &r, const unsigned char *from, auto H) {
        const i32x4 t = *(const i32x4 *)from;
        const i32x8 w = __builtin_shufflevector(t, t, 0, 1, 2, 3, -1, -1, -1, -1);
        if constexpr (decltype(H)::value == 0) r = w;
        else r = __builtin_shufflevector(r, w, 0, 1, 2, 3, 8, 9, 10, 11);
    };
    auto read_x = [&](auto I, auto H, unsigned sa) {
        constexpr int i = decltype(I)::value, h = decltype(H)::value;
        if constexpr (F8) half_into(x8[i], xa[h] + sa + i * 2048, H);
        else xf[h][i] = *(const bf16x8 *)(xa[h] + sa + i * 2048);
    };
    auto read_w = [&](auto J, auto H, auto S, unsigned sb) {
        constexpr int j = decltype(J)::value, h = decltype(H)::value;
        if constexpr (F8) half_into(w8[decltype(S)::value][j], wa + sb + j * 2048 + h * 1024, H);
        else wf[h][j] = *(const bf16x8 *)(wa + sb + j * 2048 + h * 1024);
    };
    constexpr std::integral_constant<int, 0> c0{};
    constexpr std::integral_constant<int, 1> c1{};
    // Fragment reads of a half, in the order in which the MFMAs want them.  The second half's are of the same tile;
    // the first half's (FIRST) of the next one, for F8 with B's whole tile into set S.
    constexpr int N_FIRST = F8 ? MB + 2 * NB : MB + NB, N_SECOND = F8 ? MB : MB + NB;
    auto read_frag = [&](auto FIRST, auto R, auto S, unsigned sa, unsigned sb) {
        constexpr int r = decltype(R)::value;
        if constexpr (F8) {
            if constexpr (!decltype(FIRST)::value) read_x(std::integral_constant<int, MB / 2 + r / 2>{}, std::integral_constant<int, r % 2>{}, sa);
            else if constexpr (r < 2) read_x(c0, R, sa);
            else if constexpr (r < 2 + 2 * NB) read_w(std::integral_constant<int, (r - 2) / 2>{}, std::integral_constant<int, r % 2>{}, S, sb);
            else read_x(std::integral_constant<int, (r - 2 * NB) / 2>{}, std::integral_constant<int, r % 2>{}, sa);
        } else {
            constexpr std::integral_constant<int, decltype(FIRST)::value ? 0 : 1> h{};
            if constexpr (r == 0) read_x(c0, h, sa);
            else if constexpr (r <= NB) read_w(std::integral_constant<int, r - 1>{}, h, c0, sb);
            else read_x(std::integral_constant<int, r - NB>{}, h, sa);
        }
    };
    constexpr int NM = F8 ? MB / 2 * NB : MB * NB;    // MFMAs of a half, of 32 and of 16 clocks
    // the weights are the MFMA's A operand: a lane then holds four consecutive columns of one row of C
    auto mma = [&](auto Mi, auto H, auto S) {
        constexpr int m = decltype(Mi)::value, h = decltype(H)::value, s = decltype(S)::value;
        constexpr int ii = m / NB, j = ii % 2 ? NB - 1 - m % NB : m % NB;
        constexpr int i = F8 ? h * (MB / 2) + ii : ii;
        if constexpr (F8 && kAgpr) mfma_agpr(acc[i][j], w8[s][j], x8[i]);
        else if constexpr (F8) acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(w8[s][j], x8[i], acc[i][j], 0, 0, 0, 0, 0, 0);
        else if constexpr (kAgpr) mfma_agpr(acc[i][j], wf[h][j], xf[h][i]);
        else acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[h][j], xf[h][i], acc[i][j], 0, 0, 0);
    };

    // ---- k-loop.  The barrier stands between the halves of k-tile kt.  Ahead of it every wave has read all it needs of
    //      tile kt's stages and waited for its own requests of tile kt + 1, so behind it those stages take the next
    //      requests (a round: tile kt + NSA of A, kt + NSB of B, in this order, the last of them behind the other half of
    //      the next iteration) and tile kt + 1 may be read.  Vector-memory operations retire in order through the wave's
    //      counter, so "tile kt + 1 has landed" is "at most WAIT requests outstanding": all of the rounds behind the one
    //      that asked for it, and, with a further stage of B, that round's own requests of B.
    //      A workgroup that has another tile of C to do requests that one's first k-tiles behind the last of this one, and
    //      reads their first fragments, so the pipeline stays full through the epilogue; otherwise the last k-tile is
    //      requested again, so that the counts stay the same to the end.  Worth 1 - 1.5 % of a prefill pass of 4 x 2048 tokens or of
    //      3000 through 8 experts (power-limited, most of the time saved comes back as a lower clock).
#define PD_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (7 << 4) | (15 << 8) | (((n) >> 4) << 14))
#define PD_VMCNT_LGKM0(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (7 << 4) | (((n) >> 4) << 14))
    constexpr int D1 = Ring::issued(64);              // requests of a round ahead of the iteration's end
    constexpr int WAIT = (NSA - 2) * LD + (NSB > NSA ? B_LD : 0);
    static_assert(NSA >= 2 && WAIT + LD <= 63, "vector-memory counter range");
    int pid = blockIdx.x;
    Tile t = tile_at(pid), next = t;
    pid += gridDim.x;
    bool more = pid < n_tiles;
    if (more) next = tile_at(pid);
    aim_a(t);
    aim_b(t);
    static_for<NSB - 1>([&](auto R) {
        constexpr int ta = decltype(R)::value - NSB + NSA, tb = decltype(R)::value;
        static_for<LD>([&](auto D) {
            if constexpr (decltype(D)::value >= A_LD || ta >= 0) request(D, min(kt0 + ta, kt1 - 1), ta * SA, min(kt0 + tb, kt1 - 1), B0 + tb * SB);
        });
    });
    int kap = min(kt0 + NSA - 1, kt1 - 1), kbp = min(kt0 + NSB - 1, kt1 - 1);    // the round under way
    unsigned sap = (NSA - 1) * SA, sbp = B0 + (NSB - 1) * SB;
    static_for<D1>([&](auto D) { request(D, kap, sap, kbp, sbp); });
    PD_VMCNT(WAIT + D1);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    static_for<N_FIRST>([&](auto R) { read_frag(c1, R, c0, 0u, B0); });
    unsigned sa = 0, sb = B0;
    auto k_tile = [&](int kt, auto S) {
        constexpr int s = decltype(S)::value;
        static_for<NM>([&](auto Mi) {
            constexpr int m = decltype(Mi)::value;
            constexpr int d0 = m == 0 ? D1 : Ring::issued(64 + m * 64 / NM), d1 = m == NM - 1 ? LD : Ring::issued(64 + (m + 1) * 64 / NM);
            constexpr int r0 = Ring::reads(m, NM, N_SECOND), r1 = Ring::reads(m + 1, NM, N_SECOND);
            static_for<d1 - d0>([&](auto O) { request(std::integral_constant<int, d0 + decltype(O)::value>{}, kap, sap, kbp, sbp); });
            static_for<r1 - r0>([&](auto O) { read_frag(c0, std::integral_constant<int, r0 + decltype(O)::value>{}, c0, sa, sb); });
            mma(Mi, c0, S);
            __builtin_amdgcn_sched_barrier(0);        // the stream stays in this order
        });
        PD_VMCNT_LGKM0(WAIT);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        const unsigned sa1 = sa + SA == NSA * SA ? 0u : sa + SA, sb1 = sb + SB == B0 + NSB * SB ? B0 : sb + SB;
        kap = kt + NSA;
        kbp = kt + NSB;
        if (kbp >= kt1) {
            if (more && kbp == kt1) aim_b(next);
            kbp = more ? kt0 + kbp - kt1 : kt1 - 1;
        }
        if (kap >= kt1) {
            if (more && kap == kt1) aim_a(next);
            kap = more ? kt0 + kap - kt1 : kt1 - 1;
        }
        sap = sa;
        sbp = sb;
        static_for<NM>([&](auto Mi) {
            constexpr int m = decltype(Mi)::value;
            constexpr int d0 = m == 0 ? 0 : Ring::issued(m * 64 / NM), d1 = m == NM - 1 ? D1 : Ring::issued((m + 1) * 64 / NM);
            constexpr int r0 = Ring::reads(m, NM, N_FIRST), r1 = Ring::reads(m + 1, NM, N_FIRST);
            static_for<d1 - d0>([&](auto O) { request(std::integral_constant<int, d0 + decltype(O)::value>{}, kap, sap, kbp, sbp); });
            static_for<r1 - r0>([&](auto O) {
                read_frag(c1, std::integral_constant<int, r0 + decltype(O)::value>{}, std::integral_constant<int, F8 ? 1 - s : 0>{}, sa1, sb1);
            });
            mma(Mi, c1, S);
            __builtin_amdgcn_sched_barrier(0);
        });
        sa = sa1;
        sb = sb1;
    };
    for (;;) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        pin_acc();
        if constexpr (kAgpr) asm volatile("s_nop 7");
        if constexpr (F8) {
            for (int kt = kt0; kt < kt1; kt += 2) {       // two register sets of B's fragments
                k_tile(kt, c0);
                if (kt + 1 < kt1) k_tile(kt + 1, c1);
            }
        } else {
            for (int kt = kt0; kt < kt1; ++kt) k_tile(kt, c0);
        }
        if (!more) PD_VMCNT(0);                           // the repeated requests: none may outlive the workgroup's LDS
        if constexpr (kAgpr) asm volatile("s_nop 15\n\ts_nop 15");
        pin_acc();
#undef PD_VMCNT
#undef PD_VMCNT_LGKM0

        // ---- epilogue: lane holds row (lane % 16) of each block, columns 4*(lane/16) .. +3 -------------------------
        const int el = opaque_lane(), er = el & 15, eg = el >> 4;
        if constexpr (F8) {
            f32x4 sbv[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                // columns past the last block (a multiple of 16 of them exist) are not stored
                const int n = min(t.col0 + wn * WN + j * 16, n_cols - 16) + 4 * eg;
                sbv[j] = *(const f32x4 *)(a.b_scale + (size_t)t.group * n_cols + n);
            }
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                int mr = min(t.row0 + wm * WM + i * 16 + er, t.row_end - 1);
                if (a.a_gather) mr = a.a_gather[mr];        // the scale belongs to the row the codes came from
                const float sav = a.a_scale[mr];
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[i][j][r] *= sav * sbv[j][r];
            }
        }
        if constexpr (EPI == EPI_PARTIAL) {
            float *P = a.splitk_ws + (size_t)blockIdx.y * a.M * n_cols;
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                const int m = t.row0 + wm * WM + i * 16 + er;
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const int n = t.col0 + wn * WN + j * 16 + 4 * eg;
                    if (m < t.row_end && n < n_cols) *(f32x4 *)(P + (size_t)m * n_cols + n) = acc[i][j];
                }
            }
        } else {
            uint16_t *C = (uint16_t *)a.C;
            const uint16_t *R = (const uint16_t *)a.R;
            // Two neighbouring blocks of 16 columns: the lane groups 4*(lane/16) exchange a block's half in pairs, after which
            // a lane holds 8 consecutive columns of one block and stores (and loads the residual) 16 bytes; the residual is
            // added in fp32 ahead of the one rounding to bf16.
            constexpr int OB = EPI == EPI_SWIGLU ? NB / 2 : NB;   // output blocks of the wave
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                const int m = t.row0 + wm * WM + i * 16 + er;
#pragma unroll
                for (int o = 0; o < OB; o += 2) {
                    float v[8];                                   // the lane's four columns of block o, then of block o + 1
#pragma unroll
                    for (int b = 0; b < 2; ++b)
#pragma unroll
                        for (int r = 0; r < 4; ++r) v[4 * b + r] = acc[i][EPI == EPI_SWIGLU ? 2 * o + b : o + b][r];
                    if constexpr (EPI == EPI_SWIGLU) {
                        float far = 0.f;
#pragma unroll
                        for (int r = 0; r < 8; ++r) far = fmaxf(far, fabsf(v[r]));
                        if (__builtin_expect(__ballot(!(far < kSiluNear)) == 0, 1)) {
#pragma unroll
                            for (int r = 0; r < 8; ++r) v[r] = silu_near(v[r]);
                        } else {
#pragma unroll
                            for (int r = 0; r < 8; ++r) v[r] = silu_fast(v[r]);
                        }
#pragma unroll
                        for (int r = 0; r < 8; ++r) v[r] *= acc[i][2 * o + 2 + r / 4][r % 4];
                    }
                    // lane group kg: block o + kg % 2, columns 8 * (kg / 2) .. +7
                    const int n = (EPI == EPI_SWIGLU ? (t.col0 + wn * WN) / 2 : t.col0 + wn * WN) + (o + (eg & 1)) * 16 + 8 * (eg >> 1);
                    const bool in = m < t.row_end && n < a.N;
                    uint4 out;
                    if constexpr (EPI == EPI_RESIDUAL) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[r]), __float_as_uint(v[4 + r]), false, false);
                            v[r] = __uint_as_float(p[0]);
                            v[4 + r] = __uint_as_float(p[1]);
                        }
                        uint4 rr = make_uint4(0, 0, 0, 0);
                        if (in) rr = *(const uint4 *)(R + (size_t)m * a.ldr + n);
                        out.x = pack2bf(v[0] + bfbits2f(rr.x & 0xffffu), v[1] + bfbits2f(rr.x >> 16));
                        out.y = pack2bf(v[2] + bfbits2f(rr.y & 0xffffu), v[3] + bfbits2f(rr.y >> 16));
                        out.z = pack2bf(v[4] + bfbits2f(rr.z & 0xffffu), v[5] + bfbits2f(rr.z >> 16));
                        out.w = pack2bf(v[6] + bfbits2f(rr.w & 0xffffu), v[7] + bfbits2f(rr.w >> 16));
                    } else {
                        auto p = __builtin_amdgcn_permlane16_swap(pack2bf(v[0], v[1]), pack2bf(v[4], v[5]), false, false);
                        auto q = __builtin_amdgcn_permlane16_swap(pack2bf(v[2], v[3]), pack2bf(v[6], v[7]), false, false);
                        out = make_uint4(p[0], q[0], p[1], q[1]);
                    }
                    if (in) *(uint4 *)(C + (size_t)m * a.ldc + n) = out;
                }
            }
        }
        if (!more) break;
        t = next;
        pid += gridDim.x;
        more = pid < n_tiles;
        if (more) next = tile_at(pid);
    }
}

// Tiles of up to 256 x 128 (codes, whose fragments take more: 128 x 128) stay inside 256 registers; asked to, the compiler
// leaves the AGPRs, and moves to and from them, alone.
template <int BM, int BN, int WAVES_M, int WAVES_N, int EPI, int NS, bool F8 = false>
__global__ __launch_bounds__(64 * WAVES_M *WAVES_N, BM *BN > (F8 ? 128 : 256) * 128 ? 1 : 2)
void gemm_mfma_kernel(GemmArgs a, int tiles_m, int tiles_n, int kt_per_split)
{
    gemm_mfma_body<BM, BN, WAVES_M, WAVES_N, EPI, NS, F8>(a, tiles_m, tiles_n, kt_per_split);
}

// out = epilogue(sum over splits of the fp32 partials); 4 consecutive output columns per thread.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmArgs a, int splits)
{
    const int n4 = a.N / 4;
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (size_t)a.M * n4) return;
    const int m = (int)(idx / n4), n = (int)(idx % n4) * 4;
    const int n_cols = a.epilogue == EPI_SWIGLU ? 2 * a.N : a.N;
    const size_t plane = (size_t)a.M * n_cols;
    float v[4];
    if (a.epilogue == EPI_SWIGLU) {
        const int pc = (n >> 5) * 64 + (n & 31);     // packed gate column; up is 32 further
        float4 g = make_float4(0.f, 0.f, 0.f, 0.f), u = g;
        for (int z = 0; z < splits; ++z) {
            const float *p = a.splitk_ws + z * plane + (size_t)m * n_cols + pc;
            float4 gz = *(const float4 *)p, uz = *(const float4 *)(p + 32);
            g.x += gz.x; g.y += gz.y; g.z += gz.z; g.w += gz.w;
            u.x += uz.x; u.y += uz.y; u.z += uz.z; u.w += uz.w;
        }
        v[0] = silu_fast(g.x) * u.x; v[1] = silu_fast(g.y) * u.y;
        v[2] = silu_fast(g.z) * u.z; v[3] = silu_fast(g.w) * u.w;
    } else {
        float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int z = 0; z < splits; ++z) {
            float4 tz = *(const float4 *)(a.splitk_ws + z * plane + (size_t)m * n_cols + n);
            t.x += tz.x; t.y += tz.y; t.z += tz.z; t.w += tz.w;
        }
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
        if (a.epilogue == EPI_RESIDUAL) {
            uint2 rr = *(const uint2 *)((const uint16_t *)a.R + (size_t)m * a.ldr + n);
            v[0] += bfbits2f(rr.x & 0xffffu); v[1] += bfbits2f(rr.x >> 16);
            v[2] += bfbits2f(rr.y & 0xffffu); v[3] += bfbits2f(rr.y >> 16);
        }
    }
    uint2 o;
    o.x = pack2bf(v[0], v[1]);
    o.y = pack2bf(v[2], v[3]);
    *(uint2 *)((uint16_t *)a.C + (size_t)m * a.ldc + n) = o;
}

// The same sum for an EPI_RESIDUAL product whose rows are normalised next: one workgroup per row adds the
// partials and the residual, stores the row (bf16) and its RMSNorm (statistics in fp32 on the stored,
// rounded values, exactly what a separate norm launch would read); the workgroups behind the M rows do
// the cache append of a decode step (rmsnorm_append_kernel's second half).
__global__ __launch_bounds__(512) void splitk_reduce_norm_kernel(GemmArgs a, int splits, RopeArgs ap, int n_append)
{
    __shared__ float red[8];
    __shared__ float cs[128], sn[128];
    const int m = blockIdx.x;
    if (m >= a.M) {
        if (m - a.M < n_append) append_token_body(ap, m - a.M, cs, sn);
        return;
    }
    const int n8 = a.N / 8, nt = blockDim.x;
    const size_t plane = (size_t)a.M * a.N;
    const uint16_t *R = (const uint16_t *)a.R + (size_t)m * a.ldr;
    uint16_t *C = (uint16_t *)a.C + (size_t)m * a.ldc;
    uint4 hrow[4];                                    // this thread's stored values: up to 4 chunks of 8 columns
    float ss = 0.f;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int c8 = it * nt + threadIdx.x;
        if (c8 >= n8) break;
        const int n = c8 * 8;
        float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        const float *p = a.splitk_ws + (size_t)m * a.N + n;
        const uint4 rr = *(const uint4 *)(R + n);
        int z = 0;
        // four splits' loads in flight at a time: one round trip to the L2 per four splits
        for (; z + 4 <= splits; z += 4) {
            float4 t[8];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                t[2 * u] = *(const float4 *)(p + (z + u) * plane);
                t[2 * u + 1] = *(const float4 *)(p + (z + u) * plane + 4);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {             // in split order: the sum does not depend on the grouping
                v[0] += t[2 * u].x; v[1] += t[2 * u].y; v[2] += t[2 * u].z; v[3] += t[2 * u].w;
                v[4] += t[2 * u + 1].x; v[5] += t[2 * u + 1].y; v[6] += t[2 * u + 1].z; v[7] += t[2 * u + 1].w;
            }
        }
        for (; z < splits; ++z) {
            const float4 t0 = *(const float4 *)(p + z * plane), t1 = *(const float4 *)(p + z * plane + 4);
            v[0] += t0.x; v[1] += t0.y; v[2] += t0.z; v[3] += t0.w;
            v[4] += t1.x; v[5] += t1.y; v[6] += t1.z; v[7] += t1.w;
        }
        const uint32_t rw[4] = {rr.x, rr.y, rr.z, rr.w};
        uint32_t o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            o[j] = pack2bf(v[2 * j] + bfbits2f(rw[j] & 0xffffu), v[2 * j + 1] + bfbits2f(rw[j] >> 16));
            const float x0 = bfbits2f(o[j] & 0xffffu), x1 = bfbits2f(o[j] >> 16);
            ss += x0 * x0 + x1 * x1;
        }
        hrow[it] = make_uint4(o[0], o[1], o[2], o[3]);
        *(uint4 *)(C + n) = hrow[it];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
    for (int w = 0; w < nt / 64; ++w) tot += red[w];
    const float inv = rsqrtf(tot * (1.0f / (float)a.N) + a.fuse_eps);
    uint16_t *Y = (uint16_t *)a.fuse_y + (size_t)m * a.N;
    const uint16_t *G = (const uint16_t *)a.fuse_g;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int c8 = it * nt + threadIdx.x;
        if (c8 >= n8) break;
        const int n = c8 * 8;
        const uint4 gg = *(const uint4 *)(G + n);
        const uint32_t w[4] = {hrow[it].x, hrow[it].y, hrow[it].z, hrow[it].w}, gw[4] = {gg.x, gg.y, gg.z, gg.w};
        uint32_t o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            o[j] = pack2bf(bfbits2f(w[j] & 0xffffu) * inv * bfbits2f(gw[j] & 0xffffu),
                           bfbits2f(w[j] >> 16) * inv * bfbits2f(gw[j] >> 16));
        *(uint4 *)(Y + n) = make_uint4(o[0], o[1], o[2], o[3]);
    }
}

hipError_t launch_splitk_reduce(const GemmArgs &a, int splits, hipStream_t s)
{
    if (a.fuse_y && a.fuse_g && a.fuse_done && a.epilogue == EPI_RESIDUAL && a.N % 8 == 0 && a.N <= 8192 &&
        a.ldc % 8 == 0 && a.ldr % 8 == 0) {
        RopeArgs none;
        memset(&none, 0, sizeof(none));
        const int n_append = a.fuse_append ? a.fuse_append->T : 0;
        splitk_reduce_norm_kernel<<<a.M + n_append, a.N > 2048 ? 512 : 256, 0, s>>>(a, splits, a.fuse_append ? *a.fuse_append : none, n_append);
        *a.fuse_done = 1;
        return hipGetLastError();
    }
    const size_t n_out = (size_t)a.M * (a.N / 4);
    splitk_reduce_kernel<<<(unsigned)((n_out + 255) / 256), 256, 0, s>>>(a, splits);
    return hipGetLastError();
}

bool gemm_mfma_supported(const GemmArgs &a)
{
    if (a.K % BK != 0 || a.K <= 0 || a.M <= 0) return false;
    if (a.lda % 8 != 0 || a.ldb % 8 != 0) return false;
    // 32-bit byte offsets inside A and inside one group of B
    const int64_t brows = a.epilogue == EPI_SWIGLU ? 2 * (int64_t)a.N : a.N;
    if ((int64_t)a.ldb * 2 * brows >= (1ll << 32)) return false;
    if (!a.a_gather && (int64_t)a.lda * 2 * a.M >= (1ll << 32)) return false;
    if (a.a_gather && (int64_t)a.lda * 2 * a.M >= (1ll << 31)) return false;
    if (!a.packed || a.ldb != a.K || a.K % 32 != 0 || brows % 16 != 0) return false;
    if (a.epilogue == EPI_SWIGLU) return a.N % 32 == 0;
    return true;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int NS, bool F8 = false>
static hipError_t launch_cfg(const GemmArgs &a, hipStream_t s, int splits = 1)
{
    const int n_cols = a.epilogue == EPI_SWIGLU ? 2 * a.N : a.N;
    const int tiles_n = (n_cols + BN - 1) / BN;
    const int tiles_m = (a.M + BM - 1) / BM + (a.group_offsets ? a.n_groups : 0);
    constexpr size_t smem = TileRing<BM, BN, WAVES_M * WAVES_N, NS>::lds;
    const int nk = a.K / BK;
    const int kt_per = (nk + splits - 1) / splits;
    splits = (nk + kt_per - 1) / kt_per;               // no empty split
    // One workgroup per CU (two of a form that shares it) takes every further tile of C itself, unless K is too short for
    // the ring or, with codes, ends in the other register set.
    using Ring = TileRing<BM, BN, WAVES_M * WAVES_N, NS>;
    const int slots = Ring::pair ? 512 : 256;
    int grid_x = tiles_m * tiles_n;
    if (splits == 1 && nk > Ring::NSB && (!F8 || nk % 2 == 0)) grid_x = std::min(grid_x, slots);
    const dim3 grid((unsigned)grid_x, (unsigned)splits);
    const dim3 block(64 * WAVES_M * WAVES_N);
#define LAUNCH(EPI)                                                                              \
    do {                                                                                         \
        auto kern = gemm_mfma_kernel<BM, BN, WAVES_M, WAVES_N, EPI, NS, F8>;                         \
        static OncePerDevice attr;                                                               \
        int dev;                                                                                 \
        if (attr.need(&dev)) {                                                                   \
            hipError_t e = hipFuncSetAttribute((const void *)kern,                               \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem); \
            if (e != hipSuccess) return e;                                                       \
            attr.mark(dev);                                                                      \
        }                                                                                        \
        kern<<<grid, block, smem, s>>>(a, tiles_m, tiles_n, kt_per);                             \
    } while (0)
    if (splits > 1) {
        // fp32 partials of every split must fit the scratch buffer
        if (!a.splitk_ws || (size_t)splits * a.M * n_cols > a.splitk_ws_elems) return hipErrorInvalidValue;
        LAUNCH(EPI_PARTIAL);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_splitk_reduce(a, splits, s);
    }
    switch (a.epilogue) {
    case EPI_NONE: LAUNCH(EPI_NONE); break;
    case EPI_RESIDUAL: LAUNCH(EPI_RESIDUAL); break;
    default: LAUNCH(EPI_SWIGLU); break;
    }
#undef LAUNCH
    return hipGetLastError();
}

// Split count of a grouped product of few rows per group: about one workgroup per CU (more splits lose to the fp32
// partial traffic, fewer leave CUs without a weight stream), at least 4 k-tiles per split, partials (written and read
// back) below about the weight bytes, and they must fit the scratch buffer.
static int grouped_splits(const GemmArgs &a, int BN)
{
    if (!a.splitk_ws || a.N % 4 != 0 || a.ldc % 4 != 0 || (a.epilogue == EPI_RESIDUAL && a.ldr % 4 != 0))
        return 1;
    const int n_cols = a.epilogue == EPI_SWIGLU ? 2 * a.N : a.N;
    if (n_cols >= 16384) return 1;                 // enough column tiles without splitting K
    const int tiles = (a.M < a.n_groups ? a.M : a.n_groups) * ((n_cols + BN - 1) / BN);   // at most a row tile per group and row
    const int nk = a.K / BK;
    int splits = 256 / tiles;                      // never more workgroups than CUs: a second, nearly
    if (splits > nk / 4) splits = nk / 4;          // empty round costs more than the idle CUs
    const int cap = a.K / (4 * a.M) > 1 ? a.K / (4 * a.M) : 1;
    if (splits > cap) splits = cap;
    while (splits > 1 && (size_t)splits * a.M * n_cols > a.splitk_ws_elems) --splits;
    return splits < 1 ? 1 : splits;
}

// Tile and K split of a dense product, and of a grouped one of more than 160 rows per group, for both operand widths (a k-tile
// is 64 x 2 bytes wide in either, and takes the same time).  256 x 256 tiles are the fastest per flop, but a launch runs in
// rounds of one workgroup per CU: a few hundred to a few thousand rows fill the last round badly, and so do 257 rows
// that take two row tiles.  Each form and split gets the score
//   start + k-tiles per split x (full rounds x time of a k-tile + the last round's, from few workgroups to a full one)
// and a split in addition the launch that adds the partials and the partials written and read (a product whose sum would
// carry the norm behind it saves that launch).  The constants are fitted so that the best score falls on the fastest form, not
// so that it is a time: there is no term for the weights' bytes, which all forms share, and a nearly empty last round may
// count for more than a full one.  8B shape, gate/up: score 29 at 48 rows, 72 at 512, 969 at 8192; measured 47, 93, 1285 us.
// So the scores rank the forms of products like the fitted ones and say nothing else.  Four sets:
// - 32 k-tiles and more: 5400 launches of 18 shapes of 1024 ... 28672 columns and K = 1024 ... 14336, 257 ... 6000 rows, bf16 and
//   codes, every form and split.  The choice takes 0.8 % longer than the best form and split (at worst 14 %).  us, before -> with
//   this fit: bf16 QKV 771 rows 57 -> 48 (256 x 128), down 512 rows 84 -> 64 (256 x 128, four splits).
// - fewer k-tiles: 1157 products of 256 ... 8192 columns, K = 256 ... 4096, 257 ... 4000 rows, bf16 and codes, and grouped ones.
//   5.6 % longer than the best (7.5 % with the constants of the kernels of eight and sixteen waves that stood here before; the best
//   is two workgroups of 128 x 128 per CU without a split far more often than the fit says, which holds the forms that the tests
//   state).  us: bf16 300 rows, 1536 <- 1024 15.4 -> 12.4.
// - a residual product whose sum carries a norm, any K: 234 products of 256 ... 8192 columns.  4.8 % longer (10 % before), 1.2 % from
//   K = 3072 on (3.4 % before).  us, with the norm: 1024 <- 1024 2000 rows 21.6 -> 16.9, 512 <- 512 4000 rows 22.4 -> 14.4, 4096 <-
//   4096 771 rows 45 -> 40.
// - up to 256 rows of bf16, where the weights are streamed once and the tiles are smaller: 4500 launches of 17 shapes, 18 ... 256
//   rows, up to 12 splits.  0.3 % longer than the best (at worst 12 %); one form for each of up to 64,
//   128 and 256 rows, 128 or 64 columns wide, with as many splits as one round of workgroups holds, took 19 % longer.
//   us, before -> now: 256 rows QKV 31 -> 27, O 23.6 -> 21.3, gate/up 72 -> 64, down 50 -> 44; 64 rows O 16.0 -> 13.4.
// A grouped product's loads are known only on the average, so another form than 256 x 256 has to be 5 % ahead there
// (without that, 9200 rows on 8 experts took 4330 instead of 4265 us).
enum TileForm { TILE_256, TILE_192, TILE_128_PAIR, TILE_128_DEEP, TILE_256_128, TILE_128_64, TILE_64_128, TILE_64 };
struct TilePlan {
    TileForm form;
    int splits;
};

// Row tiles of height bm.  Only the device knows the rows of each group of a grouped product: the mean number over
// groups that spread around their mean as rows dealt at random would.
static double row_tiles(const GemmArgs &a, int bm)
{
    if (!a.group_offsets) return (double)((a.M + bm - 1) / bm);
    const double mean = (double)a.M / a.n_groups, sd = sqrt(mean * (1.0 - 1.0 / a.n_groups));
    const double z[] = {-1.64, -1.04, -0.67, -0.39, -0.13, 0.13, 0.39, 0.67, 1.04, 1.64};
    double sum = 0.0;
    for (double q : z) sum += ceil(fmax(mean + q * sd, 0.0) / bm);
    return sum / 10.0 * a.n_groups;
}

static TilePlan plan_tiles(const GemmArgs &a)
{
    const int n_cols = a.epilogue == EPI_SWIGLU ? 2 * a.N : a.N;
    const int nk = a.K / BK;
    const bool can_split = a.splitk_ws && !a.group_offsets && !a.a_gather && a.N % 4 == 0 && a.ldc % 4 == 0 && (a.epilogue != EPI_RESIDUAL || a.ldr % 4 == 0);
    TilePlan best = {TILE_256, 1};
    double best_us = 1e30;
    const struct Form {
        TileForm form;
        int bm, bn, per_round;
        double start, kt_full, kt_few;
    } few_k[] = {{TILE_256, 256, 256, 256, 4.791, 1.026, 1.301},
                 {TILE_192, 192, 256, 256, 4.065, 0.947, 1.137},
                 {TILE_128_PAIR, 128, 128, 512, 2.073, 0.811, 0.494},        // two workgroups per CU
                 {TILE_128_DEEP, 128, 128, 256, 1.121, 0.554, 0.448},        // alone on its CU with a deeper ring
                 {TILE_256_128, 256, 128, 256, 5.956, 0.981, 0.385}},
      normed[] = {{TILE_256, 256, 256, 256, 11.517, 1.011, 1.162},
                  {TILE_192, 192, 256, 256, 6.100, 0.993, 0.858},
                  {TILE_128_PAIR, 128, 128, 512, 2.309, 0.826, 0.964},
                  {TILE_128_DEEP, 128, 128, 256, 0.353, 0.615, 0.819},
                  {TILE_256_128, 256, 128, 256, 6.434, 0.716, 0.914}},
      many_k[] = {{TILE_256, 256, 256, 256, 1.235, 1.080, 1.306},
                  {TILE_192, 192, 256, 256, 3.609, 0.891, 0.943},
                  {TILE_128_PAIR, 128, 128, 512, 0.392, 0.832, 0.904},
                  {TILE_128_DEEP, 128, 128, 256, 0.021, 0.460, 0.769},
                  {TILE_256_128, 256, 128, 256, 2.968, 0.698, 0.830}},
      few_rows[] = {{TILE_256_128, 256, 128, 256, 3.0, 0.490, 0.861},
                    {TILE_128_DEEP, 128, 128, 256, 3.29, 0.445, 0.475},
                    {TILE_128_64, 128, 64, 256, 1.88, 0.312, 0.472},
                    {TILE_64_128, 64, 128, 256, 4.44, 0.402, 0.306},
                    {TILE_64, 64, 64, 256, 0.83, 0.232, 0.273}};
    // codes come in calls of more than 256 rows, but for pd_gemm_e4m3, which takes the larger calls' forms for fewer rows too
    const bool few = a.M <= 256 && !a.a_scale;
    const struct Kind {
        const Form *forms;                     // five each
        double add, partials, norm;            // us of a split's sum, bytes per us of its partials, us of the norm that it saves
        int max_splits, min_k_tiles;
    } kind = few        ? Kind{few_rows, 4.04, 3.2e6, 6.5, 12, 4}
             : a.fuse_y ? Kind{normed, 1.570, 3.543e6, 0.672, 8, 2}
             : nk >= 32 ? Kind{many_k, 5.06, 4.96e6, 0.0, 8, 2}
                        : Kind{few_k, 1.358, 2.909e6, 0.0, 8, 2};
    for (int i = 0; i < 5; ++i) {
        const Form &f = kind.forms[i];
        const long long tiles = (long long)ceil(row_tiles(a, f.bm) * ((n_cols + f.bn - 1) / f.bn));
        for (int sp = 1; sp <= kind.max_splits; ++sp) {
            if (sp > 1 && (!can_split || nk / sp < kind.min_k_tiles || (size_t)sp * a.M * n_cols > a.splitk_ws_elems)) break;
            const long long wg = tiles * sp, full = wg / f.per_round, rem = wg % f.per_round;
            const double last = rem ? f.kt_few + (f.kt_full - f.kt_few) * (double)rem / f.per_round : 0.0;
            double us = f.start + ((nk + sp - 1) / sp) * ((double)full * f.kt_full + last);
            if (sp > 1) us += kind.add + (double)sp * a.M * n_cols * 8.0 / kind.partials;
            else if (a.fuse_y) us += kind.norm;
            if (a.group_offsets && f.form != TILE_256) us *= 1.05;
            if (us < best_us) {
                best_us = us;
                best = {f.form, sp};
            }
        }
    }
    return best;
}

// The plan of a product, for tests that state which form their sizes take (host only; not part of the C ABI): n_groups 0 for
// a dense product, scratch_elems floats for partials, fused_norm where a split's sum would carry the norm behind it, codes
// where both operands are E4M3 (K then counts pairs).  form: in the order of TileForm.
extern "C" void pd_internal_tile_plan(int M, int N, int K, int epilogue, int n_groups, long long scratch_elems, int fused_norm,
                                      int codes, int *form, int *splits)
{
    static const int32_t some_offsets = 0;
    static float some_scratch;
    static char some_row;
    GemmArgs a;
    memset(&a, 0, sizeof(a));
    a.M = M; a.N = N; a.K = K; a.ldc = N; a.ldr = N; a.epilogue = epilogue;
    if (n_groups > 0) {
        a.n_groups = n_groups;
        a.group_offsets = &some_offsets;
    }
    if (scratch_elems > 0) {
        a.splitk_ws = &some_scratch;
        a.splitk_ws_elems = (size_t)scratch_elems;
    }
    if (fused_norm) a.fuse_y = &some_row;
    if (codes) a.a_scale = &some_scratch;
    const TilePlan p = plan_tiles(a);
    *form = p.form;
    *splits = p.splits;
}

// 8-bit operands (see the kernel): a.A are E4M3 codes [M, 2 K] with a.a_scale per row, a.B the codes in
// the pack of the halved view with a.b_scale per packed row; a.K, a.lda, a.ldb count code pairs.
bool gemm_mfma_f8_supported(const GemmArgs &a)
{
    return gemm_mfma_supported(a) && a.a_scale && a.b_scale;
}

template <bool F8>
static hipError_t launch_planned(const GemmArgs &a, hipStream_t s)
{
    const TilePlan p = plan_tiles(a);
    switch (p.form) {
    case TILE_192: return launch_cfg<192, 256, 2, 2, 2, F8>(a, s, p.splits);
    case TILE_128_PAIR: return launch_cfg<128, 128, 2, 2, 2, F8>(a, s, p.splits);
    case TILE_128_DEEP: return launch_cfg<128, 128, 2, 2, 3, F8>(a, s, p.splits);
    case TILE_256_128: return launch_cfg<256, 128, 2, 2, 3, F8>(a, s, p.splits);
    default: break;
    }
    if constexpr (!F8) {                                      // the forms of few rows, which plan_tiles gives to bf16 only
        switch (p.form) {
        case TILE_128_64: return launch_cfg<128, 64, 4, 1, 4>(a, s, p.splits);
        case TILE_64_128: return launch_cfg<64, 128, 2, 2, 4>(a, s, p.splits);
        case TILE_64: return launch_cfg<64, 64, 4, 1, 4>(a, s, p.splits);
        default: break;
        }
    }
    return launch_cfg<256, 256, 2, 2, 2, F8>(a, s, p.splits);
}

hipError_t launch_gemm_mfma_f8(const GemmArgs &a, hipStream_t s)
{
    return launch_planned<true>(a, s);
}

// Height of the row tiles of a grouped product of up to 160 rows per group, 128 columns wide (see launch_gemm_mfma)
static int grouped_row_tile(const GemmArgs &a, int rows, int splits)
{
    const int n_cols = a.epilogue == EPI_SWIGLU ? 2 * a.N : a.N;
    const double mean = (double)a.M / a.n_groups, most = mean + 2.0 * sqrt(mean * (1.0 - 1.0 / a.n_groups));
    auto one_round = [&](int bm) { return ceil(most / bm) * a.n_groups * ((n_cols + 127) / 128) * splits <= 256.0; };
    if (rows <= 32 || one_round(64)) return 64;
    return rows <= 107 || one_round(128) ? 128 : 256;
}

// The same for tests (host only; not part of the C ABI)
extern "C" int pd_internal_grouped_row_tile(int M, int N, int K, int epilogue, int n_groups, long long scratch_elems)
{
    static float some_scratch;
    GemmArgs a;
    memset(&a, 0, sizeof(a));
    a.M = M; a.N = N; a.K = K; a.ldc = N; a.ldr = N; a.epilogue = epilogue; a.n_groups = n_groups;
    if (scratch_elems > 0) {
        a.splitk_ws = &some_scratch;
        a.splitk_ws_elems = (size_t)scratch_elems;
    }
    return grouped_row_tile(a, (M + n_groups - 1) / n_groups, grouped_splits(a, 128));
}

hipError_t launch_gemm_mfma(const GemmArgs &a, hipStream_t s)
{
    if (!a.group_offsets) return launch_planned<false>(a, s);
    // Rows that share a weight matrix: the mean group size picks the tile.  A group that outgrows its row tile takes a second
    // one, which reads the weights again, and groups spread around the mean by about its square root; a taller tile
    // costs little while the launch is bound by the weight stream.  So 128-row tiles from 33 rows on (8 experts of 4096 x
    // 14336, one layer: the same 631 - 655 us with either up to 52 rows, where no group had 64; 63 rows on the average, three
    // routings, 768 / 825 / 813 us with 64-row tiles, 672 / 673 / 675 with these), 256-row tiles where a tenth of the groups or so
    // would outgrow 128 (mean + 2 x its root: 105 rows 686 us, with the taller tile 721; 110 rows 823 / 838 and 725 / 729;
    // 128 rows 921 / 902 and 743 / 740), and the estimate of plan_tiles, which counts those second tiles, from 161 rows on (175 rows
    // 836 -> 783 us, 225 rows 888 -> 863, 250 rows 1168 -> 1003, 255 rows 1289 -> 1042; between, at 237 rows, 903 -> 909).
    // That is for launches of more workgroups than CUs.  Where even the second tiles find a CU of their own (narrow or few
    // experts), they run beside the first, and the lower tile is the faster one; us, gate/up and down, lower -> taller:
    // 8 experts of 512 x 256 64 rows 7.7 + 6.0 -> 8.4 + 6.4, 116 rows 7.5 + 6.1 -> 11.1 + 7.9 (64 and 256 rows tall); 16 of
    // 1024 x 512 107 rows 14.3 + 10.4 -> 15.9 + 10.9, 128 rows 16.1 + 11.4 -> 18.9 + 12.3; where they do not, 4 of 1024 x
    // 2816, gate/up 64 rows 18.4 -> 14.8, 32 of 2048 x 1408, down 64 rows 63 -> 43, 116 rows 59 -> 49.
    const int rows = (a.M + a.n_groups - 1) / a.n_groups;
    if (rows > 160) return launch_planned<false>(a, s);
    const int splits = grouped_splits(a, 128), bm = grouped_row_tile(a, rows, splits);
    if (bm == 256) return launch_cfg<256, 128, 2, 2, 3>(a, s, splits);
    if (bm == 128) return launch_cfg<128, 128, 2, 2, 3>(a, s, splits);
    return launch_cfg<64, 128, 2, 2, 4>(a, s, splits);
}

}  // namespace pd
