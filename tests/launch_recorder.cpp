// Stands in for the HIP runtime underneath the built library, so that a test without a GPU sees what the library asks of it: every launch with its grid and its dynamic LDS, and
// every grant of LDS.  Device memory is addresses only; nothing runs.  Commands from stdin, one a line:
//   context <hidden> <heads> <head_dim> <mlp> <max_fresh> <max_tokens> <dtype>
//   block <type> <text rows> <image rows> <dtype of h> <flags> <n_all> <fp8>
//   step <edited> <tokens> <channels> <fresh text rows> <dtype> <block type>...   (up to the end of the line; every block with a conditioning vector; `edited` is the count that the call gets)
// Output: "grant <bytes> <kernel>" and "launch <x> <y> <z> <dynamic LDS> <kernel>", "rc <code> <message>" behind a command's calls.
#include <hip/hip_runtime_api.h>
#include <cxxabi.h>
#include <dlfcn.h>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>
#include "regione.h"

namespace {
std::map<const void*, std::string>& kernels() { static std::map<const void*, std::string> m; return m; }
struct Config { dim3 grid, block; size_t lds; hipStream_t stream; };
Config pushed;
uintptr_t next_address = uintptr_t{1} << 40;
int32_t* pinned;             // the context's words that the count of a step's partition and the number of the step arrive in
int32_t steps;
const char* name(const void* f) { return kernels().count(f) ? kernels()[f].c_str() : "unknown"; }
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* mangled, unsigned, void*, void*, void*, void*, int*) {
    int status = 0;
    char* plain = abi::__cxa_demangle(mangled, nullptr, nullptr, &status);
    kernels()[f] = plain && status == 0 ? plain : mangled;
    free(plain);
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) { pushed = {grid, block, lds, stream}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) { *grid = pushed.grid; *block = pushed.block; *lds = pushed.lds; *stream = pushed.stream; return hipSuccess; }
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void**, size_t lds, hipStream_t) { printf("launch %u %u %u %zu %s\n", grid.x, grid.y, grid.z, lds, name(f)); return hipSuccess; }
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute attr, int value) {
    if (attr == hipFuncAttributeMaxDynamicSharedMemorySize) printf("grant %d %s\n", value, name(f));
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { *p = reinterpret_cast<void*>(next_address); next_address += (n + 255) / 256 * 256; return hipSuccess; }
hipError_t hipFree(void*) { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = pinned = static_cast<int32_t*>(calloc(1, n)); steps = 0; return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { return hipMalloc(p, 1 << 20); }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = reinterpret_cast<hipEvent_t>(8); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = reinterpret_cast<hipStream_t>(8); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
}

int main(int, char** argv) {
    void* lib = dlopen(argv[1], RTLD_NOW | RTLD_LOCAL);
    if (!lib) { fprintf(stderr, "%s\n", dlerror()); return 2; }
    const auto create = reinterpret_cast<decltype(&regione_create)>(dlsym(lib, "regione_create"));
    const auto destroy = reinterpret_cast<decltype(&regione_destroy)>(dlsym(lib, "regione_destroy"));
    const auto block = reinterpret_cast<decltype(&regione_block_forward)>(dlsym(lib, "regione_block_forward"));
    const auto block_fp8 = reinterpret_cast<decltype(&regione_block_forward_fp8)>(dlsym(lib, "regione_block_forward_fp8"));
    const auto step = reinterpret_cast<decltype(&regione_region_step)>(dlsym(lib, "regione_region_step"));
    const auto error = reinterpret_cast<decltype(&regione_last_error)>(dlsym(lib, "regione_last_error"));
    auto device = [] { void* p = nullptr; (void)hipMalloc(&p, size_t{1} << 30); return p; };
    regione_ctx* ctx = nullptr;
    char cmd[32];
    while (scanf("%31s", cmd) == 1) {
        int rc = -1;
        if (!strcmp(cmd, "context")) {
            regione_dims d;
            if (scanf("%d %d %d %d %d %d %d", &d.hidden, &d.heads, &d.head_dim, &d.mlp, &d.max_fresh, &d.max_tokens, &d.compute_dtype) != 7) return 2;
            if (ctx) destroy(ctx);
            rc = create(&ctx, &d, nullptr);
        } else if (!strcmp(cmd, "block")) {
            int type, n_txt, n_img, dtype, flags, n_all, fp8;
            if (scanf("%d %d %d %d %d %d %d", &type, &n_txt, &n_img, &dtype, &flags, &n_all, &fp8) != 7) return 2;
            regione_block_weights w = {};
            regione_block_weights_fp8 w8 = {};
            for (regione_stream_weights* s : {&w.txt, &w.img})
                for (const void** p : {&s->w_qkv, &s->w_o, &s->w_1, &s->w_2}) *p = device();
            for (regione_stream_weights_fp8* s : {&w8.txt, &w8.img}) {
                s->w_qkv = s->w_o = s->w_1 = s->w_2 = static_cast<decltype(s->w_1)>(device());
                s->s_qkv = s->s_o = s->s_1 = s->s_2 = static_cast<const float*>(device());
            }
            void *h = device(), *out = device(), *k = device(), *v = device();
            const int32_t* slots = static_cast<const int32_t*>(device());
            rc = fp8 ? block_fp8(ctx, &w, &w8, type, h, out, dtype, n_txt + n_img, n_txt, slots, 0, k, v, n_all, flags, nullptr)
                     : block(ctx, &w, type, h, out, dtype, n_txt + n_img, n_txt, slots, 0, k, v, n_all, flags);
        } else if (!strcmp(cmd, "step")) {
            int edited, tokens, channels, n_txt, dtype, used = 0;
            char line[4096];
            if (scanf("%d %d %d %d %d", &edited, &tokens, &channels, &n_txt, &dtype) != 5 || !fgets(line, sizeof line, stdin)) return 2;
            std::vector<int32_t> types;
            int type;
            for (const char* p = line; sscanf(p, "%d%n", &type, &used) == 1; p += used) types.push_back(type);
            std::vector<regione_block_weights> blocks(types.size());
            std::vector<void*> caches(types.size());
            for (size_t i = 0; i < types.size(); ++i) {
                blocks[i] = {};
                for (regione_stream_weights* s : {&blocks[i].txt, &blocks[i].img})
                    for (const void** p : {&s->w_qkv, &s->w_o, &s->w_1, &s->w_2, &s->w_mod}) *p = device();
                blocks[i].cond = static_cast<const float*>(device());
                caches[i] = device();
            }
            regione_region_step_args a = {};
            a.x_t = device(); a.v = device(); a.x_ref = device(); a.n_tokens = tokens; a.c = channels; a.dtype = dtype; a.sigma_t = 0.5f; a.eta = 0.9f;
            a.mask = static_cast<uint8_t*>(device());
            for (int32_t** p : {&a.e_index, &a.u_index, &a.n_edited_dev, &a.slots}) *p = static_cast<int32_t*>(device());
            a.h_full = device(); a.h_dtype = dtype; a.n_txt_fresh = n_txt; a.h_rows = device(); a.h_rows_out = device();
            a.n_blocks = static_cast<int32_t>(types.size()); a.n_all = tokens + n_txt; a.slot_offset = n_txt;
            a.blocks = blocks.data(); a.block_types = types.data(); a.k_caches = caches.data(); a.v_caches = caches.data();
            a.w_head_packed = device(); a.dt = 0.04f; a.c_a = device(); a.x_e = device(); a.x_next_full = device(); a.h_next_full_opt = device();
            pinned[0] = edited; pinned[1] = ++steps;
            int32_t got = -1;
            rc = step(ctx, &a, &got);
            if (!rc && got != edited) return 3;
        } else {
            return 2;
        }
        printf("rc %d %s\n", rc, rc ? error() : "");
    }
    if (ctx) destroy(ctx);
    return 0;
}
