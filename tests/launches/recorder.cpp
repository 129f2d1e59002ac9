// Runs the library's host code on a machine without a GPU and prints what it would launch: this program defines the runtime
// calls that the library makes, and the dynamic linker finds them here before the HIP runtime's.  No kernel runs.
//
// stdin, a line per call: dir (3: forward with statistics, 4: the forward that allocates nothing) algo workspace_bytes, then the 13 fields
// of sn_conv_shape.  stdout per call: a line per launch
//   launch <kernel> <grid x y z> <threads> <dynamic LDS> <LDS limit set for the kernel, or -1> <workspace bytes it reaches, or -1>
// and `call <status> <plans of the channels-last product that were made>`.  What a launch reaches is known for the sum over slices (reduce_partials_kernel): the end of its slices.
#include <dlfcn.h>

#include <cstdint>
#include <cstdio>
#include <map>
#include <string>

#include "sn.h"

namespace {
struct Dim { uint32_t x, y, z; };
std::map<const void *, std::string> &names() { static std::map<const void *, std::string> m; return m; }
std::map<const void *, int> limits;
Dim grid, block;
size_t lds;
void *stream;
int plans;
const char *const ws = reinterpret_cast<const char *>(uintptr_t(1) << 44);   // nothing is there; nothing is read or written
}  // namespace

namespace sn {   // counted, and passed on
struct ConvGeom;
struct ChlastPlan;
bool chlast_plan(const ConvGeom &g, int dir, size_t budget, ChlastPlan *plan)
{
    static const auto next = reinterpret_cast<bool (*)(const ConvGeom &, int, size_t, ChlastPlan *)>(
        dlsym(RTLD_NEXT, "_ZN2sn11chlast_planERKNS_8ConvGeomEimPNS_10ChlastPlanE"));
    ++plans;
    return next(g, dir, budget, plan);
}
}  // namespace sn

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { names()[host] = name; }
int __hipPushCallConfiguration(Dim g, Dim b, size_t shared, void *s) { grid = g; block = b; lds = shared; stream = s; return 0; }
int __hipPopCallConfiguration(Dim *g, Dim *b, size_t *shared, void **s) { *g = grid; *b = block; *shared = lds; *s = stream; return 0; }
int hipFuncSetAttribute(const void *f, int attr, int value)
{
    if (attr == 8) limits[f] = value;   // hipFuncAttributeMaxDynamicSharedMemorySize
    return 0;
}
int hipGetLastError() { return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetSymbolAddress(void **p, const void *) { *p = const_cast<char *>(ws); return 0; }
int hipEventCreate(void **e) { *e = nullptr; return 0; }
int hipEventDestroy(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *, void *) { *ms = 1.f; return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipLaunchKernel(const void *f, Dim g, Dim b, void **args, size_t shared, void *)
{
    const std::string &name = names()[f];
    const auto limit = limits.find(f);
    long long reach = -1;
    if (name.find("reduce_partials_kernel") != std::string::npos) {   // (partial, dw, n, splits, ..): n float4 or n float
        const char *partial = *static_cast<const char **>(args[0]);
        const size_t n = *static_cast<size_t *>(args[2]) * (name.find("HIP_vector_type") != std::string::npos ? 16 : 4);
        if (partial >= ws && partial < ws + (size_t(1) << 43)) reach = partial - ws + (long long)n * *static_cast<int *>(args[3]);
    }
    std::printf("launch %s %u %u %u %u %zu %d %lld\n", name.c_str(), g.x, g.y, g.z, b.x * b.y * b.z, shared, limit == limits.end() ? -1 : limit->second, reach);
    return 0;
}
}

int main()
{
    int dir, algo;
    size_t ws_bytes;
    sn_conv_shape s;
    int32_t *f = &s.N;
    static_assert(sizeof(s) == 13 * sizeof(int32_t), "the fields that are read");
    while (std::scanf("%d %d %zu", &dir, &algo, &ws_bytes) == 3) {
        for (int i = 0; i < 13; ++i)
            if (std::scanf("%d", f + i) != 1) return 1;
        void *const w = ws_bytes ? const_cast<char *>(ws) : nullptr;
        const auto tensor = [](uintptr_t i) { return reinterpret_cast<void *>(i << 40); };
        const auto call = dir == SN_CONV_FWD ? sn_conv2d_fwd : dir == SN_CONV_BWD_DATA ? sn_conv2d_bwd_data : sn_conv2d_bwd_filter;
        plans = 0;
        float *const stats = static_cast<float *>(tensor(4));
        const int status = dir == 3 ? sn_conv2d_fwd_bn_stats(tensor(1), tensor(2), tensor(3), &s, (sn_conv_algo)algo, w, ws_bytes, stats, stats, 1e-5f,
                                                             tensor(5), sn_conv_bn_stats_scratch_bytes(&s), nullptr)
                           : dir == 4 ? sn_conv2d_fwd_noalloc(tensor(1), tensor(2), tensor(3), &s, nullptr)
                                      : call(tensor(1), tensor(2), tensor(3), &s, (sn_conv_algo)algo, w, ws_bytes, nullptr);
        std::printf("call %d %d\n", status, plans);
    }
    return 0;
}
