// A host stand-in for the HIP runtime calls and kernel launchers that
// dv_engine.cpp uses, so that its order of allocations, clears, launches and
// waits can be looked at without a GPU.  Every call is logged as one line;
// "device" memory is host memory; launches compute nothing.  An allocation of
// fail_at bytes or more fails and, as in the runtime, leaves the error set until
// hipGetLastError takes it, which the launchers return.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>

#include "dv_internal.h"

static std::string g_log;
static size_t g_fail_at = ~(size_t)0, g_live = 0;
static hipError_t g_err = hipSuccess;

static void note(const char *what, const void *stream, size_t bytes = 0)
{
    char b[128];
    std::snprintf(b, sizeof b, "%s %zx %zu\n", what, (size_t)stream, bytes);
    g_log += b;
}

extern "C" {

void stub_reset(size_t fail_at)
{
    g_log.clear();
    g_fail_at = fail_at;
}
const char *stub_log() { return g_log.c_str(); }
size_t stub_live() { return g_live; }

hipError_t hipMalloc(void **p, size_t n)
{
    note("malloc", nullptr, n);
    if (n >= g_fail_at) return g_err = hipErrorOutOfMemory;
    size_t *m = static_cast<size_t *>(std::malloc(n + 64));
    *m = n;
    g_live += n;
    *p = reinterpret_cast<char *>(m) + 64;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    if (!p) return hipSuccess;
    size_t *m = reinterpret_cast<size_t *>(static_cast<char *>(p) - 64);
    note("free", nullptr, *m);
    g_live -= *m;
    std::free(m);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return (*p = std::calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { return *d = h, hipSuccess; }
hipError_t hipMemset(void *p, int v, size_t n) { return note("memset", nullptr, n), std::memset(p, v, n), hipSuccess; }
hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t s) { return note("memset", s, n), std::memset(p, v, n), hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { return std::memcpy(d, s, n), hipSuccess; }
hipError_t hipDeviceSynchronize() { return note("devsync", nullptr), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return note("sync", s), hipSuccess; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipGetLastError() { hipError_t e = g_err; return g_err = hipSuccess, e; }
const char *hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipEventCreate(hipEvent_t *) { return hipErrorNotSupported; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *, hipEvent_t, hipEvent_t) { return hipErrorNotSupported; }

}  // extern "C"

static hipError_t launched(const char *what, hipStream_t s) { return note(what, s), hipGetLastError(); }

hipError_t launch_pack(const GemmArgs &, int, int, void *, hipStream_t s) { return launched("pack", s); }
hipError_t launch_pack_scales(const GemmArgs &, int, float *, hipStream_t s) { return launched("pack", s); }
GemmShape gemm_shape(int rb) { return rb >= 4 ? GemmShape{4, 2} : GemmShape{4, 4}; }
int gemm_blocks_per_cu(int, int, int, int, int) { return 1; }
bool gemm_has_rb8(int, int, int) { return false; }
// (a launch of its own: returns its own status, not the last error)
hipError_t launch_gemm(const GemmArgs &, int, int, int, int, hipStream_t s, hipEvent_t, hipEvent_t) { return note("gemm", s), hipSuccess; }
hipError_t launch_embed_norm(const NormArgs &, int, int, hipStream_t s) { return launched("norm", s); }
hipError_t launch_attention(const AttnArgs &, int, hipStream_t s) { return launched("attention", s); }
hipError_t launch_accept(const AcceptArgs &, hipStream_t s) { return launched("accept", s); }
hipError_t launch_accept_sampled(const SampleArgs &, hipStream_t s) { return launched("sample", s); }
hipError_t noalloc_scratch(void **) { return hipErrorNotSupported; }
hipError_t launch_pf_embed(const int32_t *, const void *, int, int, int, const void *, float *, uint16_t *, float *, hipStream_t s)
{
    return launched("pf_embed", s);
}
PfPlan pf_plan(int, int MT, int, bool, int) { return PfPlan{1, MT > 8 ? 8 : (MT < 4 ? 4 : MT), (MT + 7) / 8, 2}; }
int pf_part_tiles(int NB, const PfPlan &p) { return (NB + 15) / 16 * p.n_tt * p.ks * 16 * p.tt; }
hipError_t launch_pf_gemm(const PfArgs &, const PfPlan &, int, hipStream_t s) { return launched("pf_gemm", s); }
hipError_t launch_attn_causal(const float *, const void *, const void *, int, int, int, int, int, int, int, uint16_t *, hipStream_t s)
{
    return launched("causal", s);
}
hipError_t launch_dgf_in(const float *, const void *, const DgfTokens &, int, int, int, uint16_t *, uint16_t *, hipStream_t s) { return launched("dgf", s); }
hipError_t launch_dgf_gate_in(const float *, const float *, int, int, int, uint16_t *, hipStream_t s) { return launched("dgf", s); }
hipError_t launch_dgf_mix(const float *, const float *, const float *, int, int, float *, hipStream_t s) { return launched("dgf", s); }
hipError_t launch_gather_rows(const float *, const RowIndex &, int, int, float *, hipStream_t s) { return launched("gather", s); }
hipError_t launch_topk_probs(const float *, int, const TopkArgs &, int, hipStream_t s) { return launched("topk", s); }
hipError_t launch_kv_commit(const CommitArgs &, int, hipStream_t s) { return launched("commit", s); }
