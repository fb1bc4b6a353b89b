// CPU-only view of what the engine launches: its host code against a stand-in for the HIP
// runtime that notes every kernel launch and runs none.  One call per line on stdin:
//   move path host_layout layers heads dim tokens elem chunk_layers max_copy_wgs wg_lanes vecs_per_lane cache_at pool_at n_out n_in
//   read layers heads dim tokens elem max_wgs n
// and on stdout a line per launch, "kernel key=value ...", then an empty line.  cache_at and
// pool_at are where the two begin behind a multiple of 4096 bytes; no slot follows the one before.
#include <cxxabi.h>

#include <map>
#include <string>

#include "../paper_2601_20309_amd/csrc/duplexkv.hip"

namespace {
std::map<const void *, std::string> names;
struct {
    dim3 g, b;
    size_t shared;
    hipStream_t s;
} next_launch;

void note(const void *f, dim3 g, dim3 b, void **args)
{
    const std::string &name = names[f];
    const unsigned waves = g.x * b.x / 64;
    std::printf("%s grid=%u lanes=%u waves=%u", name.c_str(), g.x, b.x, waves);
    if (name.rfind("kv_move", 0) == 0) {
        const MoveParams &p = *static_cast<MoveParams *>(args[0]);
        const unsigned steps = p.mix_q ? p.in.tiles : std::max(p.out.tiles, p.in.tiles);
        std::printf(" out=%u in=%u steps=%u drawn=%d whole=%u mask=%u through=%u", p.out.tiles, p.in.tiles, steps,
                    steps > (uint64_t)p.fixed_rounds * waves ? 1 : 0, p.full_tiles, p.line_mask, p.through);
    } else if (name.rfind("kv_stage", 0) == 0) {
        const dkv::StageParams &p = *static_cast<dkv::StageParams *>(args[0]);
        std::printf(" blocks=%u planes=%u", p.n, p.n_planes);
    } else if (name == "kv_reader_kernel" || name == "kv_reader_inline_kernel") {
        const dkv::ReadParams &p = *static_cast<dkv::ReadParams *>(args[0]);
        std::printf(" rows=%u tiles=%u", p.rows, p.tiles);
    }
    std::printf("\n");
}
}  // namespace

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, unsigned long, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *, void *, void *, void *, int *)
{
    std::string s = device;
    if (char *d = abi::__cxa_demangle(device, nullptr, nullptr, nullptr)) { s = d; std::free(d); }
    s = s.substr(0, s.find('<'));
    s = s.substr(0, s.find('('));
    const size_t at = s.find("kv_");
    names[host] = at == std::string::npos ? s : s.substr(at);
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t shared, hipStream_t s) { next_launch = {g, b, shared, s}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *shared, hipStream_t *s)
{
    *g = next_launch.g; *b = next_launch.b; *shared = next_launch.shared; *s = next_launch.s;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t, hipStream_t) { note(f, g, b, args); return hipSuccess; }
hipError_t hipExtLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t, hipStream_t, hipEvent_t, hipEvent_t, int)
{
    note(f, g, b, args);
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 100000; return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)8; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)8; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) { p->multiProcessorCount = 256; return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "none"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorInvalidSymbol; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::calloc(1, n); return hipSuccess; }
hipError_t hipMalloc(void **p, size_t) { *p = std::calloc(1, 64); return hipSuccess; }  // nothing is read or written there
hipError_t hipMemGetAddressRange(hipDeviceptr_t *base, size_t *n, hipDeviceptr_t) { *base = nullptr; *n = ~(size_t)0; return hipSuccess; }
hipError_t hipMemcpy2DAsync(void *, size_t, const void *, size_t, size_t, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipMemset(void *, int, size_t) { return hipSuccess; }
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *) { a->type = hipMemoryTypeHost; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)8; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *c) { *c = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
}

int main()
{
    char what[8];
    while (std::scanf("%7s", what) == 1) {
        const bool read = !std::strcmp(what, "read");
        kv_config c{};
        int no = 0, ni = 0, wgs = 0;
        long long cache_at = 0, pool_at = 0;
        const int got = read ? std::scanf("%d %d %d %d %d %d %d", &c.n_layers, &c.n_kv_heads, &c.head_dim, &c.block_size, &c.elem_bytes, &wgs, &ni)
                             : std::scanf("%d %d %d %d %d %d %d %d %d %d %d %lld %lld %d %d", &c.path, &c.host_layout, &c.n_layers, &c.n_kv_heads,
                                          &c.head_dim, &c.block_size, &c.elem_bytes, &c.chunk_layers, &c.max_copy_wgs, &c.wg_lanes,
                                          &c.vecs_per_lane, &cache_at, &pool_at, &no, &ni);
        if (got != (read ? 7 : 15)) return 2;
        c.n_hbm_blocks = no + ni + 1;
        c.n_host_slots = 2 * (no + ni) + 1;
        kv_engine *e = nullptr;
        int rc = kv_create(&e, &c, (void *)(0x100000 + cache_at), (void *)(0x100000 + pool_at), nullptr, nullptr);
        std::vector<int32_t> ids((size_t)(no + ni)), slots((size_t)(no + ni));
        for (int32_t i = 0; i < no + ni; i++) { ids[(size_t)i] = i; slots[(size_t)i] = 2 * i; }
        if (rc == KV_OK)
            rc = read ? kv_reader_start(e, ids.data(), ni, 1, wgs)
                      : kv_rotate(e, ids.data(), slots.data(), no, ids.data() + no, slots.data() + no, ni);
        if (rc != KV_OK) std::printf("refused rc=%d\n", rc);
        std::printf("\n");
        if (e) (void)kv_destroy(e);
    }
    return 0;
}
