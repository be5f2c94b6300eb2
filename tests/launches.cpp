// The launches of the built library's calls, without a GPU: this program stands in for the HIP runtime, loads the library (argv[1]) and prints, for every line of standard input, the kernels that
// the call launches, by name, one after the other with " ; " between them.  For tests/test_launches.py.
//   step <step | forward | backward> <fp8> <M> <T> <D> <F> <flags> <n> [<n + 1 segment offsets>]   (n = 0: the plain step)
//   kernels           all that the library has
//   spmm <fp8> <M> <T> <N> <F>           wgrad <out_f_major> <M> <T> <F> <N>
#include <cxxabi.h>
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <map>
#include <string>
#include <vector>

#include "../include/sparseffn.h"

namespace {
std::map<const void*, std::string>& names() { static std::map<const void*, std::string> m; return m; }
std::vector<std::string> launched;
std::string readable(const std::string& name) {          // without the parameters
    int status = 0;
    char* s = abi::__cxa_demangle(name.c_str(), nullptr, nullptr, &status);
    const std::string r = s ? s : name;
    free(s);
    return r.substr(0, r.find('('));
}
}  // namespace
struct Dim3 { uint32_t x, y, z; };
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*, int*) { names()[host] = device; }
int __hipPushCallConfiguration(Dim3, Dim3, size_t, void*) { return 0; }
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) { *grid = *block = {1, 1, 1}; *lds = 0; *stream = nullptr; return 0; }
int hipLaunchKernel(const void* host, Dim3, Dim3, void**, size_t, void*) { launched.push_back(readable(names()[host])); return 0; }
int hipGetLastError() { return 0; }
}

int main(int argc, char** argv) {
    void* lib = argc == 2 ? dlopen(argv[1], RTLD_NOW | RTLD_LOCAL) : nullptr;
    if (!lib) { fprintf(stderr, "%s\n", argc == 2 ? dlerror() : "usage: launches LIBRARY"); return 1; }
#define CALL(f) ((decltype(&f))dlsym(lib, #f))
    uint16_t* const p = (uint16_t*)0x100000;      // never dereferenced
    uint8_t* const p8 = (uint8_t*)0x200000;
    float* const pf = (float*)0x300000;
    const size_t plenty = (size_t)1 << 45;
    const sffn_fp8_scales scales = {1.f, 1.f, 1.f, 1.f, 1.f, 1.f};
    char what[16], call[16];
    while (scanf("%15s", what) == 1) {
        launched.clear();
        int rc = -100;
        if (!strcmp(what, "kernels")) {
            for (const auto& k : names()) launched.push_back(readable(k.second));
            rc = SFFN_OK;
        } else if (!strcmp(what, "step")) {
            int fp8, n;
            sffn_cfg c;
            memset(&c, 0, sizeof(c));
            c.V = 64;
            if (scanf("%15s %d %d %ld %ld %ld %d %d", call, &fp8, &c.M, &c.T, &c.D, &c.F, &c.flags, &n) != 8) return 1;
            int64_t seg[65];
            for (int i = 0; n && i <= n; ++i) if (scanf("%ld", seg + i) != 1) return 1;
            void* const ws = (void*)((uintptr_t)1 << 40);
            sffn_buffers b;
            if ((fp8 ? CALL(sffn_fp8_buffer_sizes)(&c, n ? n : 1, &b) : CALL(sffn_buffer_sizes)(&c, n ? n : 1, &b)) != SFFN_OK) { printf("refused\n"); continue; }
            b.scratch = (void*)((uintptr_t)1 << 40); b.saved = (void*)((uintptr_t)2 << 40); b.weights = (void*)((uintptr_t)3 << 40);
            if (!strcmp(call, "step"))
                rc = fp8 ? (n ? CALL(ffn_sparse_step_fp8_grouped)(&c, &scales, n, seg, p, p, p, pf, p, p, p, p, p, ws, plenty, pf, nullptr) : CALL(ffn_sparse_step_fp8)(&c, &scales, p, p, p, pf, p, p, p, p, p, ws, plenty, pf, nullptr))
                         : (n ? CALL(ffn_sparse_step_grouped)(&c, n, seg, p, p, p, pf, p, p, p, p, p, ws, plenty, nullptr) : CALL(ffn_sparse_step)(&c, p, p, p, pf, p, p, p, p, p, ws, plenty, nullptr));
            else if (!strcmp(call, "forward"))
                rc = fp8 ? (n ? CALL(ffn_sparse_forward_fp8_grouped)(&c, &scales, n, seg, p, p, p, pf, p, &b, pf, nullptr) : CALL(ffn_sparse_forward_fp8)(&c, &scales, p, p, p, pf, p, &b, pf, nullptr))
                         : (n ? CALL(ffn_sparse_forward_grouped)(&c, n, seg, p, p, p, pf, p, &b, nullptr) : CALL(ffn_sparse_forward)(&c, p, p, p, pf, p, &b, nullptr));
            else if (!strcmp(call, "backward"))
                rc = fp8 ? (n ? CALL(ffn_sparse_backward_fp8_grouped)(&c, &scales, n, seg, p, p, p, p, &b, pf, nullptr) : CALL(ffn_sparse_backward_fp8)(&c, &scales, p, p, p, p, &b, pf, nullptr))
                         : (n ? CALL(ffn_sparse_backward_grouped)(&c, n, seg, p, p, p, p, p, &b, nullptr) : CALL(ffn_sparse_backward)(&c, p, p, p, p, p, &b, nullptr));
        } else {
            int a, M;
            int64_t T, N, F;
            if (scanf("%d %d %ld %ld %ld", &a, &M, &T, &N, &F) != 5) return 1;
            if (!strcmp(what, "spmm")) rc = a ? CALL(vnm_spmm_fp8)(p8, p8, p8, 1.f, p8, 1.f, 0, T, N, F, 64, M, p, (void*)p8, plenty, nullptr) : CALL(vnm_spmm)(p, p8, p8, p, F, 0, T, N, F, 64, M, p, (void*)p8, plenty, nullptr);
            else if (!strcmp(what, "wgrad")) rc = CALL(vnm_wgrad)(p, p8, p8, p, T, N, F, 64, M, a, p, (void*)p8, plenty, nullptr);
        }
        if (rc != SFFN_OK) { printf("refused %d %s\n", rc, CALL(sffn_last_error)()); continue; }
        for (size_t i = 0; i < launched.size(); ++i) printf("%s%s", i ? " ; " : "", launched[i].c_str());
        printf("\n");
    }
    return 0;
}
