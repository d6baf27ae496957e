// Rotary embedding, cache write and value transposition of a prefill (bf16 rows, head_dim 128), a tile of 64
// cache positions of one sequence at a time.
//
// The work is a copy: q and k are read, rotated and written back, k and v go to the cache, v also to the
// transposed scratch that prefill attention reads.  A block per token (rope_kv_kernel) does it in 2-byte
// accesses, worst for values, whose cache block is transposed (positions innermost).  A tile is aligned to the
// cache's own blocks of positions, so here every access is 8 or 16 bytes, values turning once through LDS.  A
// workgroup takes the query heads of one K/V group, or its key and value head (or all of them, see the launcher);
// eight lanes share a row, lane i holding channels 8i .. 8i + 7 and their partners 64 higher, so cosines and sines
// are loaded once for all heads.
// Measured (8B shape, rope + transposition, which was a launch of its own, -> this kernel): 8192 rows 77 + 8 -> 44 us
// (218 MB: 5.0 TB/s), 5107 rows into an 8-bit cache 57 + 6 -> 32 us, 771 rows 15 + 5 -> 9 us, a 512-row chunk
// 11 -> 6.5 us.  The whole workgroup also for a few rows: with eight threads a row the values of 13 rows took eight
// dependent passes (a call of one 13-row prompt into an 8-bit cache 92.7 us, now 88.6; a launch per row before: 89.4).
#include "pd_internal.h"

namespace pd {

constexpr int kTileRow = 128 + 2;     // LDS row stride of the value tile (elements): columns fall on different banks

// Codes of f / scale, inv = e4m3_inverse(scale).
__device__ __forceinline__ uint2 encode_run(const float (&f)[8], double scale, float inv)
{
    return make_uint2(e4m3_encode2(f[0], f[1], scale, inv) | (e4m3_encode2(f[2], f[3], scale, inv) << 16),
                      e4m3_encode2(f[4], f[5], scale, inv) | (e4m3_encode2(f[6], f[7], scale, inv) << 16));
}

__device__ __forceinline__ uint4 pack8(const float (&f)[8])
{
    return make_uint4(pack2bf(f[0], f[1]), pack2bf(f[2], f[3]), pack2bf(f[4], f[5]), pack2bf(f[6], f[7]));
}

__device__ __forceinline__ void unpack8(uint4 v, float (&f)[8])
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        f[2 * j] = bfbits2f(w[j] & 0xffffu);
        f[2 * j + 1] = bfbits2f(w[j] >> 16);
    }
}

// Sequence of tile b where sequence s has the tiles from cu[s] / 64 + extra s up to the next one's first (enough for its
// rows: extra is 1 where they start on a tile, 2 where they start anywhere): the largest s whose first tile is at most
// b.  The lanes of a wave look at 64 sequences at once, so 4096 take two rounds.
__device__ __forceinline__ int tile_sequence(const RopeTiles &t, int extra, int b)
{
    const int lane = threadIdx.x & 63, step = (t.n_seqs + 63) / 64;
    int s = 0;
    if (step > 1) {
        const int i = lane * step;
        s = (__popcll(__ballot(i < t.n_seqs && (t.cu[i] >> 6) + extra * i <= b)) - 1) * step;
    }
    const int i = s + lane;
    s += __popcll(__ballot((step == 1 || lane < step) && i < t.n_seqs && (t.cu[i] >> 6) + extra * i <= b)) - 1;
    return __builtin_amdgcn_readfirstlane(s);
}

template <bool FP8>
__global__ __launch_bounds__(512) void rope_tile_kernel(RopeArgs a, RopeTiles t, int per_seq, int halves)
{
    __shared__ uint32_t tile32[64 * kTileRow / 2];
    uint16_t *tile = (uint16_t *)tile32;
    const int part = blockIdx.y + blockIdx.z * gridDim.y;          // a grid dimension holds 65535
    const int tid = threadIdx.x, g = halves ? part >> 1 : part;
    if (g >= a.Hkv) return;
    const bool queries = !halves || !(part & 1), kv = !halves || (part & 1);
    const int extra = t.prefix ? 2 : 1;
    const int s = per_seq ? (int)blockIdx.x / per_seq : tile_sequence(t, extra, blockIdx.x);
    const int row0 = t.cu[s], L = t.cu[s + 1] - row0, P = t.prefix ? t.prefix[s] : 0;
    const int nth = (int)blockIdx.x - (per_seq ? s * per_seq : (row0 >> 6) + extra * s);
    const int tb = ((P >> 6) + nth) << 6;
    const int lo = max(tb, P), hi = min(tb + 64, P + L);           // positions of this tile that the call brings
    if (lo >= hi) return;
    const int nt = blockDim.x, c8 = (tid & 7) * 8;
    uint16_t *rows = (uint16_t *)a.qkv + (size_t)row0 * a.ld;
    const int slot = a.tok_slot ? t.slots[s] : -1;
    const size_t plane = slot < 0 ? 0 : ((size_t)slot * a.Hkv + g) * a.max_len * 128;

    for (int pos = tb + (tid >> 3); pos < hi; pos += nt >> 3) {
        if (pos < lo) continue;
        uint16_t *row = rows + (size_t)(pos - P) * a.ld;
        float cs[8], sn[8];
        if (pos < a.table_len) {
            const float4 *f = (const float4 *)(a.table + (size_t)pos * 64 + c8);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float4 v = f[j];
                cs[2 * j] = v.x; sn[2 * j] = v.y; cs[2 * j + 1] = v.z; sn[2 * j + 1] = v.w;
            }
        } else {
            for (int j = 0; j < 8; ++j) {
                double sv, cv;
                sincos((double)pos * a.inv_freq[c8 + j], &sv, &cv);
                cs[j] = (float)cv;
                sn[j] = (float)sv;
            }
        }
        const int group = a.Hq / a.Hkv;
        const int nq = queries ? group : 0, n = nq + (kv ? 1 : 0);     // query heads first, then the key head
        // the rows of up to four heads are requested before the first is written back
        for (int h = 0; h < n; h += 4) {
            uint4 r0[4], r1[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (h + u < n) {
                    const uint16_t *p = row + (size_t)(h + u < nq ? g * group + h + u : a.Hq + g) * 128 + c8;
                    r0[u] = *(const uint4 *)p;
                    r1[u] = *(const uint4 *)(p + 64);
                }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (h + u >= n) break;
                float x0[8], x1[8], y0[8], y1[8];
                unpack8(r0[u], x0);
                unpack8(r1[u], x1);
#pragma unroll
                for (int j = 0; j < 8; ++j) rope_pair(x0[j], x1[j], cs[j], sn[j], y0[j], y1[j]);
                const uint4 o0 = pack8(y0), o1 = pack8(y1);
                uint16_t *p = row + (size_t)(h + u < nq ? g * group + h + u : a.Hq + g) * 128 + c8;
                *(uint4 *)p = o0;
                *(uint4 *)(p + 64) = o1;
                if (h + u < nq || slot < 0) continue;
                if (FP8) {
                    uint8_t *kp = (uint8_t *)a.k_cache + plane;
                    *(uint2 *)(kp + kblk8_off(pos, c8)) = encode_run(y0, a.k_scale, a.k_inv);
                    *(uint2 *)(kp + kblk8_off(pos, c8 + 64)) = encode_run(y1, a.k_scale, a.k_inv);
                } else {
                    uint16_t *kp = (uint16_t *)a.k_cache + plane;
                    *(uint4 *)(kp + (a.blocked ? kblk_off(pos, c8) : (size_t)pos * 128 + c8)) = o0;
                    *(uint4 *)(kp + (a.blocked ? kblk_off(pos, c8 + 64) : (size_t)pos * 128 + c8 + 64)) = o1;
                }
            }
        }
    }
    if (!kv || (slot < 0 && !t.vt)) return;

    // values: rows of the tile into LDS (zero where the call brings none), columns out of it
    const int n_read = min(64, hi - tb + 19);          // rows that the reads below touch
    for (int r = tid >> 3; r < n_read; r += nt >> 3) {
        const int pos = tb + r;
        const bool in = pos >= lo && pos < hi;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            uint4 v = make_uint4(0, 0, 0, 0);
            if (in) v = *(const uint4 *)(rows + (size_t)(pos - P) * a.ld + (size_t)(a.Hq + a.Hkv + g) * 128 + c8 + 64 * i);
            if (!FP8 && !a.blocked && in && slot >= 0) *(uint4 *)((uint16_t *)a.v_cache + plane + (size_t)pos * 128 + c8 + 64 * i) = v;
            uint32_t *d = tile32 + (r * kTileRow + c8 + 64 * i) / 2;
            d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
        }
    }
    __syncthreads();
    if (t.vt) {
        uint16_t *vt = t.vt + (size_t)g * 128 * t.vt_ld + t.pad_cu[s] + tb;
        for (int e = tid; e < 1024; e += nt) {
            const int d = e >> 3, p = (e & 7) * 8;
            uint32_t w[4] = {0u, 0u, 0u, 0u};
            if (tb + p < hi) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    w[j] = tile[(p + 2 * j) * kTileRow + d] | ((uint32_t)tile[(p + 2 * j + 1) * kTileRow + d] << 16);
            }
            *(uint4 *)(vt + (size_t)d * t.vt_ld + p) = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
    if (slot < 0 || !a.blocked) return;
    // run e of the cache's 64 positions: one channel, positions p .. p + 3 and p + 16 .. p + 19
    for (int e = tid; e < 1024; e += nt) {
        const int half = FP8 ? e & 1 : e >> 9;
        const int d = FP8 ? (e >> 7) * 16 + ((e >> 1) & 15) : (e >> 2) & 127, q = FP8 ? (e >> 5) & 3 : e & 3;
        const int p = half * 32 + 4 * q;
        if (tb + p >= hi) continue;
        const uint16_t *c = tile + p * kTileRow + d;
        uint16_t v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = c[((j & 3) + 16 * (j >> 2)) * kTileRow];
        const bool whole = tb + p >= lo && tb + p + 19 < hi;       // else positions of the run that are not new stay as they are
        if (FP8) {
            float f[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = bfbits2f(v[j]);
            const uint2 code = encode_run(f, a.v_scale, a.v_inv);
            uint8_t *vp = (uint8_t *)a.v_cache + plane + (size_t)(tb >> 6) * 8192 + (size_t)e * 8;
            if (whole) {
                *(uint2 *)vp = code;
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int at = tb + p + (j & 3) + 16 * (j >> 2);
                    if (at >= lo && at < hi) vp[j] = (uint8_t)((j < 4 ? code.x : code.y) >> (8 * (j & 3)));
                }
            }
        } else {
            uint16_t *vp = (uint16_t *)a.v_cache + plane + (size_t)(tb >> 5) * 4096 + (size_t)e * 8;
            if (whole) {
                *(uint4 *)vp = make_uint4(v[0] | ((uint32_t)v[1] << 16), v[2] | ((uint32_t)v[3] << 16),
                                          v[4] | ((uint32_t)v[5] << 16), v[6] | ((uint32_t)v[7] << 16));
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int at = tb + p + (j & 3) + 16 * (j >> 2);
                    if (at >= lo && at < hi) vp[j] = v[j];
                }
            }
        }
    }
}

bool rope_tile_supported(int dtype, const RopeArgs &a)
{
    return dtype == PD_BF16 && a.hd == 128 && a.ld % 8 == 0;
}

// Tiles are dealt in one grid dimension.  Sequences of similar lengths: the tiles of the longest for each, so that a
// block knows its sequence by a division.  Where that would be more than twice what the rows need (a long prompt among
// many short ones), a block searches (0.3 - 0.5 us).  8192 + 999 x 8 rows (8B shape) 115 us found, 3900 dealt by the
// longest; 8 sequences of 30 ... 2000 rows the same either way.
// Where tiles are mostly empty and there are blocks for the whole chip twice over, one block of 128 threads takes a
// group's query, key and value heads instead of two of 512: 4096 x 1 rows 420 -> 215 us, 512 x 16 rows 83 -> 60, 64 x 9
// behind a prefix 20 -> 14; 200 x 50 rows (28 a tile) 62 both ways, 64 rows 7.5 -> 17.
hipError_t launch_rope_tile(const RopeArgs &a, const RopeTiles &t, hipStream_t s)
{
    if (a.T <= 0) return hipSuccess;
    const int extra = t.prefix ? 2 : 1;
    const long long found = (a.T >> 6) + (long long)extra * t.n_seqs;
    int per_seq = (t.max_len + (t.prefix ? 126 : 63)) / 64;
    if ((long long)per_seq * t.n_seqs > 2 * found) per_seq = 0;
    const unsigned nx = (unsigned)(per_seq ? (long long)per_seq * t.n_seqs : found);
    const bool few_rows = a.T <= 16 * ((a.T >> 6) + (long long)t.n_seqs) && (long long)nx * a.Hkv >= 512;
    const int halves = few_rows ? 0 : 1, nt = few_rows ? 128 : 512;
    const unsigned parts = (unsigned)((1 + halves) * a.Hkv), ny = parts < 65535u ? parts : 65535u;
    const dim3 grid(nx, ny, (parts + ny - 1) / ny);
    if (a.fp8) rope_tile_kernel<true><<<grid, nt, 0, s>>>(a, t, per_seq, halves);
    else rope_tile_kernel<false><<<grid, nt, 0, s>>>(a, t, per_seq, halves);
    return hipGetLastError();
}

}  // namespace pd
