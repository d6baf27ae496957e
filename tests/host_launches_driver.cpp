// Driver for tests/test_host_launches.py: the library's host code on a stand-in for the HIP runtime.  The runtime's
// entry points that the library imports are defined here, and an executable's definitions come before a shared
// library's: "device" memory is host memory, a launch is counted and refused where the GPU would refuse its grid, and
// of the kernels only those that write sequence arrays and cache lengths are carried out.  Test infrastructure only.
//
// failures  every launch and every allocation of a prefill call or a decode step fails in turn: the call has to return an error, the
//           cache lengths on the device and on the host have to be what they were, and the same call has to
//           succeed afterwards with the lengths that it would have left at once.
//
// limits    a prefill call of nearly as many rows as a launch of a workgroup of 256 per row can have: no launch may be refused.
#include <hip/hip_runtime_api.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>
#include <vector>

#include "pd.h"

// ---- the stand-in runtime ---------------------------------------------------------------------------------------
// (the library registers its kernels before this executable's own static objects exist)
static std::map<const void *, std::string> &names()
{
    static std::map<const void *, std::string> m;
    return m;
}
static hipError_t g_last = hipSuccess;
static long g_launches, g_fail_launch = -1, g_mallocs, g_fail_malloc = -1;
static bool g_refused;                      // a launch that the GPU would refuse
static int32_t *g_written;                  // where the last write_ints launch stored
static struct { dim3 grid, block; size_t shared; hipStream_t stream; } g_config;

struct Chunk { int32_t v[960]; };           // the library's by-value arrays of 256 and 960 entries start alike
struct Dst4 { int32_t *dst[4]; int32_t start[5]; };

static void carry_out(const std::string &name, void **args)
{
    auto is = [&](const char *k) { return name.find(k) != std::string::npos; };
#define ARG(T, i) (*(T *)args[i])
    if (is("write_ints_kernel")) {
        g_written = ARG(int32_t *, 0);
        memcpy(g_written, ((const Chunk *)args[1])->v, sizeof(int32_t) * (size_t)ARG(int, 2));
    } else if (is("write_ints4_kernel") || is("prefill_meta_kernel") || is("prefill_meta_norm_kernel")) {
        const Dst4 &d = ARG(Dst4, 0);
        const int32_t *v = ((const Chunk *)args[1])->v;
        for (int k = 0; k < 4; ++k)
            for (int i = d.start[k]; i < d.start[k + 1]; ++i) d.dst[k][i - d.start[k]] = v[i];
        if (is("write_ints4_kernel")) return;
        int32_t *len = ARG(int32_t *, 7), *was = ARG(int32_t *, 8);
        for (int i = 0; len && i < ARG(int, 2); ++i) {
            const int s = v[d.start[2] + i];
            was[i] = len[s];
            len[s] = (ARG(int, 9) ? len[s] : 0) + v[i + 1] - v[i];
        }
    } else if (is("prefill_set_len_kernel")) {
        const int32_t *slots = ARG(const int32_t *, 0), *cu = ARG(const int32_t *, 1);
        int32_t *len = ARG(int32_t *, 3);
        for (int i = 0; i < ARG(int, 2); ++i) len[slots[i]] = (ARG(int, 4) ? len[slots[i]] : 0) + cu[i + 1] - cu[i];
    } else if (is("decode_meta_")) {
        const bool by_value = !is("decode_meta_kernel") && !is("ILb0");
        const int at = is("decode_meta_chunks_kernel") ? 1 : 0;      // the by-value slots' argument
        const int32_t *slots = by_value ? ((const Chunk *)args[at])->v : ARG(const int32_t *, 0);
        const int b0 = is("decode_meta_kernel") ? 1 : at + 2, B = ARG(int, b0);
        int32_t *len = ARG(int32_t *, b0 + 1), *pos = ARG(int32_t *, b0 + 2);
        for (int b = 0; b < B; ++b) {
            if (by_value) ARG(int32_t *, at + 1)[b] = slots[b];
            pos[b] = len[slots[b]]++;
        }
    } else if (is("restore_len_kernel")) {
        const int32_t *slots = ARG(const int32_t *, 0), *was = ARG(const int32_t *, 1);
        int32_t *len = ARG(int32_t *, 3);
        for (int i = 0; i < ARG(int, 2); ++i) len[slots[i]] = was[i];
    }
#undef ARG
}

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *, int *)
{
    names()[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream)
{
    g_config = {grid, block, shared, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *stream)
{
    *grid = g_config.grid; *block = g_config.block; *shared = g_config.shared; *stream = g_config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t shared, hipStream_t)
{
    const long id = g_launches++;
    const bool fits = (uint64_t)grid.x * block.x <= 0xffffffffull && grid.y <= 65535 && grid.z <= 65535 && grid.x && grid.y && grid.z &&
                      (uint64_t)block.x * block.y * block.z <= 1024 && shared <= 160 * 1024;
    if (!fits) {
        g_refused = true;
        printf("refused: %s grid %u %u %u block %u\n", names()[f].c_str(), grid.x, grid.y, grid.z, block.x);
    }
    if (!fits || id == g_fail_launch) return g_last = hipErrorInvalidConfiguration;
    carry_out(names()[f], args);
    return hipSuccess;
}
hipError_t hipGetLastError(void)
{
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "refused"; }
hipError_t hipMalloc(void **p, size_t n)
{
    if (g_mallocs++ == g_fail_malloc || !(*p = calloc(n ? n : 1, 1))) return g_last = hipErrorOutOfMemory;
    return hipSuccess;
}
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void *, int v, size_t) { return v ? hipErrorInvalidValue : hipSuccess; }   // allocations come cleared
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { static char scratch[64 << 20]; *p = scratch; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *) { return hipErrorNotSupported; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
}

// ---- the cases --------------------------------------------------------------------------------------------------
#define CHECK(x, ...)                                            \
    do {                                                         \
        if (!(x)) {                                              \
            printf("FAILED %s:%d %s: ", __FILE__, __LINE__, #x); \
            printf(__VA_ARGS__);                                 \
            printf("\n");                                        \
            exit(1);                                             \
        }                                                        \
    } while (0)

static pd_layer *make_layer(pd_dtype dtype, int d, int hq, int hkv, int hd, int f, int experts)
{
    pd_layer_config c;
    memset(&c, 0, sizeof(c));
    c.d_model = d; c.n_q_heads = hq; c.n_kv_heads = hkv; c.head_dim = hd; c.d_ff = f; c.n_experts = experts; c.top_k = experts ? 2 : 0;
    c.rms_eps = 1e-6f; c.rope_base = 1e4f; c.dtype = dtype;
    const size_t wide = (size_t)(experts ? experts : 1) * f > (size_t)hq * hd ? (size_t)(experts ? experts : 1) * f : (size_t)hq * hd;
    std::vector<float> some(wide * d + 4);
    pd_layer_weights w;
    const void *p = some.data();
    w.g_attn = w.w_q = w.w_k = w.w_v = w.w_o = w.g_ffn = w.w_gate = w.w_up = w.w_down = p;
    w.w_router = experts ? p : nullptr;
    pd_layer *L = nullptr;
    CHECK(pd_layer_create(&c, &w, &L) == PD_OK, "%s", pd_last_error());
    return L;
}

struct Case {
    const char *name;
    pd_dtype dtype;
    int d, hq, hkv, hd, f, experts;
    enum { PROMPTS, CHUNK, STEP, STEP_NOALLOC } kind;
    std::vector<int32_t> before, rows;      // cache lengths and new rows of the sequences
    int min_mallocs;                        // allocations that the call has to make beyond its workspace
};

static void failures(const Case &k)
{
    const int n = (int)k.rows.size(), max_len = n > 100 ? 64 : 4096;
    std::vector<int32_t> cu(1, 0), slots;
    for (int s = 0; s < n; ++s) {
        cu.push_back(cu.back() + k.rows[(size_t)s]);
        slots.push_back(n - 1 - s);
    }
    std::vector<float> x((size_t)cu.back() * k.d), out(x.size());
    pd_tokens tk;
    memset(&tk, 0, sizeof(tk));
    tk.hidden = x.data(); tk.n_seqs = n; tk.cu_seqlens = cu.data(); tk.slots = slots.data();
    pd_batch bt;
    memset(&bt, 0, sizeof(bt));
    bt.hidden = x.data(); bt.batch = n; bt.slots = slots.data();
    long launches = 0, mallocs = 0;
    for (long step = -1; step < launches + mallocs; ++step) {
        // a layer of its own each time: what an earlier call has allocated is there
        pd_layer *L = make_layer(k.dtype, k.d, k.hq, k.hkv, k.hd, k.f, k.experts);
        pd_kv_cache *c = nullptr;
        CHECK(pd_kv_cache_create(L, n, max_len, &c) == PD_OK, "%s", pd_last_error());
        for (int s = n - 1; s >= 0; --s) CHECK(pd_kv_cache_set_len(c, slots[(size_t)s], k.before[(size_t)s], nullptr) == PD_OK, "%s", pd_last_error());
        const int32_t *d_len = g_written - slots[0];
        CHECK(pd_layer_reserve(L, cu.back()) == PD_OK, "%s", pd_last_error());
        auto lens_are = [&](bool after) {
            for (int s = 0; s < n; ++s) {
                const int want = after ? (k.kind == Case::PROMPTS ? 0 : k.before[(size_t)s]) + k.rows[(size_t)s] : k.before[(size_t)s];
                int32_t h = -1;
                pd_kv_cache_len(c, slots[(size_t)s], &h);
                CHECK(d_len[slots[(size_t)s]] == want && h == want, "%s, step %ld of %ld launches + %ld allocations: sequence %d has %d on the device, %d on the host, not %d",
                      k.name, step, launches, mallocs, s, d_len[slots[(size_t)s]], h, want);
            }
        };
        auto call = [&] {
            switch (k.kind) {
            case Case::PROMPTS: return pd_prefill(L, &tk, c, out.data(), nullptr);
            case Case::CHUNK: return pd_prefill_chunk(L, &tk, c, out.data(), nullptr);
            case Case::STEP: return pd_decode_step(L, &bt, c, out.data(), nullptr);
            default: return pd_decode_step_noalloc(L, &bt, c, out.data(), nullptr);
            }
        };
        g_launches = g_mallocs = 0;
        g_fail_launch = step < launches ? step : -1;
        g_fail_malloc = step >= launches ? step - launches : -1;
        const pd_status st = call();
        g_fail_launch = g_fail_malloc = -1;
        if (step < 0) {
            CHECK(st == PD_OK, "%s: %s", k.name, pd_last_error());
            launches = g_launches;
            mallocs = g_mallocs;
            CHECK(launches >= 4 && mallocs >= k.min_mallocs, "%s: %ld launches, %ld allocations", k.name, launches, mallocs);
            lens_are(true);
        } else if (st != PD_OK) {
            lens_are(false);
            CHECK(call() == PD_OK, "%s", pd_last_error());
            lens_are(true);
        } else {                            // a larger scratch than needed was refused, and the needed one taken
            CHECK(step >= launches, "%s: launch %ld failed and the call did not say so", k.name, step);
            lens_are(true);
        }
        pd_kv_cache_destroy(c);
        pd_layer_destroy(L);
    }
    CHECK(!g_refused, "%s", k.name);
    printf("ok %s: %ld launches, %ld allocations\n", k.name, launches, mallocs);
}

static void limits()
{
    const int rows = 16720000, d = 64;      // 2^32 threads: 16777216 rows
    pd_layer *L = make_layer(PD_BF16, d, 1, 1, 64, 64, 0);
    void *x = calloc((size_t)rows * d, 2);
    const int32_t cu[2] = {0, rows};
    pd_tokens tk;
    memset(&tk, 0, sizeof(tk));
    tk.hidden = x; tk.n_seqs = 1; tk.cu_seqlens = cu;
    CHECK(x && pd_prefill(L, &tk, nullptr, x, nullptr) == PD_OK, "%s", pd_last_error());
    CHECK(!g_refused, "%d rows", rows);
    pd_layer_destroy(L);
    free(x);
}

int main(int argc, char **argv)
{
    if (argc != 2) return 2;
    if (!strcmp(argv[1], "limits")) {
        limits();
        return 0;
    }
    const std::vector<int32_t> four = {5, 0, 40, 7}, rows = {12, 1, 30, 9};
    std::vector<int32_t> long_before, short_rows, many_before(100, 3), many_rows(100, 2);
    for (int i = 0; i < 63; ++i) {
        long_before.push_back(700 + 13 * i);
        short_rows.push_back(8 - i % 3);
    }
    failures({"fp32 prompts", PD_F32, 64, 4, 2, 32, 128, 0, Case::PROMPTS, four, rows, 0});
    failures({"fp32 chunk", PD_F32, 64, 4, 2, 32, 128, 0, Case::CHUNK, four, rows, 0});
    failures({"bf16 prompts", PD_BF16, 256, 4, 2, 128, 512, 0, Case::PROMPTS, four, rows, 1});
    failures({"bf16 chunk", PD_BF16, 256, 4, 2, 128, 512, 0, Case::CHUNK, four, rows, 1});
    failures({"bf16 short chunk", PD_BF16, 256, 4, 2, 128, 512, 0, Case::CHUNK, four, {8, 1, 3, 2}, 0});
    failures({"bf16 short chunk that outgrows the workspace", PD_BF16, 256, 8, 8, 128, 512, 0, Case::CHUNK, long_before, short_rows, 1});
    failures({"bf16 plain cache", PD_BF16, 128, 4, 2, 64, 256, 0, Case::CHUNK, four, rows, 0});
    failures({"experts", PD_BF16, 256, 4, 2, 128, 512, 4, Case::CHUNK, four, rows, 1});
    failures({"more sequences than a launch's arguments hold", PD_BF16, 256, 4, 2, 128, 512, 0, Case::CHUNK, many_before, many_rows, 0});
    const std::vector<int32_t> ones(4, 1), many(300, 1), most(1000, 1);
    failures({"fp32 step", PD_F32, 64, 4, 2, 32, 128, 0, Case::STEP, four, ones, 0});
    failures({"fp32 step of many", PD_F32, 64, 4, 2, 32, 128, 0, Case::STEP, many, many, 0});
    failures({"bf16 step", PD_BF16, 256, 4, 2, 128, 512, 0, Case::STEP, four, ones, 0});
    failures({"bf16 step of many", PD_BF16, 256, 4, 2, 128, 512, 0, Case::STEP, many, many, 0});
    failures({"bf16 step of more than a launch's arguments hold", PD_BF16, 256, 4, 2, 128, 512, 0, Case::STEP, most, most, 0});
    failures({"bf16 step without allocations", PD_BF16, 256, 4, 2, 128, 512, 0, Case::STEP_NOALLOC, four, ones, 0});
    failures({"experts, step", PD_BF16, 256, 4, 2, 128, 512, 4, Case::STEP, four, ones, 0});
    return 0;
}
