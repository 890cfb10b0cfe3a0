// Stands in for the HIP runtime under the host code of the GEMM launchers: kernels are not run, the name and the grid of
// each launch are printed.  Reads one problem per line: epi M N K n_sel max_rows which acc_dbg (n_sel 0: a single matrix;
// epi -1: whether a linear on fp16 rows takes the one launch that forms its own codes; epi -2: column maxima of K x N weights).
#include <cstdarg>
#include <cstdio>
#include <map>
#include <string>

#include "haq_common.h"

static std::map<const void*, std::string>& kernels() {  // filled before this file's own constructors have run
    static std::map<const void*, std::string> m;
    return m;
}
static dim3 grid_, block_;

extern "C" {
void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { kernels()[host] = name; }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) {
    grid_ = grid;
    block_ = block;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* st) {
    *grid = grid_;
    *block = block_;
    *lds = 0;
    *st = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void**, size_t, hipStream_t) {
    if (kernels()[f].find("fill_zero") == std::string::npos) printf("%s %u\n", kernels()[f].c_str(), grid.x * grid.y);
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return ""; }
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
    *v = 256;  // compute units
    return hipSuccess;
}
}

namespace haq {
void set_error(const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vfprintf(stderr, fmt, ap);
    va_end(ap);
}
}  // namespace haq

int main() {
    int epi, dbg;
    static int32_t some;
    haq::GemmArgs a{};
    while (scanf("%d %d %d %d %d %d %d %d", &epi, &a.M, &a.N, &a.K, &a.n_sel, &a.max_rows, &a.which, &dbg) == 8) {
        if (epi == -1) {
            printf("%s 0\n", haq::fused_linear_fits(a.M, a.K, a.N) ? "fused_linear_kernel" : "none_kernel");
            continue;
        }
        if (epi == -2) {
            haq::launch_weight_colmax(nullptr, nullptr, 1, a.K, a.N, nullptr, nullptr);
            continue;
        }
        a.Npad = haq::round_up(a.N, haq::NPAD);
        a.R = 256 + haq::round_up(a.M > a.max_rows ? a.M : a.max_rows, 16);
        a.offsets = a.n_sel ? &some : nullptr;
        a.acc_dbg = dbg ? &some : nullptr;
        if (haq::launch_gemm(a, epi, nullptr) != HAQ_OK) printf("refused 0\n");
    }
    return 0;
}
