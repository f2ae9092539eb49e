// Prints the names of the kernels that calls of the library launch, without a GPU: this program's own functions take the place of the
// runtime's for the library it loads; they say that the device has 256 compute units, and launch nothing.
//
//   launched_kernels libtpq.so < calls
//
// One call a line, whose kernels are printed as one line (mangled names, in order; "-" and the code where the call was refused):
//   gemm E k G T K                          tpq_gemm_encode
//   decode E k G bits N T accum out_dtype   tpq_decode_reduce
//   static E k G bits N T accum out_dtype   tpq_decode_reduce_static
//   finalize E k N ranked                   tpq_calibrate_finalize
#include <dlfcn.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>

#include "tpq_internal.h"

#define TAKES_THE_PLACE extern "C" __attribute__((visibility("default")))

static std::map<const void *, std::string> &kernels()
{
    static std::map<const void *, std::string> m;
    return m;
}

TAKES_THE_PLACE void **__hipRegisterFatBinary(const void *)
{
    static void *handle;
    return &handle;
}
TAKES_THE_PLACE void __hipUnregisterFatBinary(void **) {}
TAKES_THE_PLACE void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    kernels()[host] = name;
}
TAKES_THE_PLACE void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
TAKES_THE_PLACE hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
TAKES_THE_PLACE hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
TAKES_THE_PLACE hipError_t hipGetLastError() { return hipSuccess; }
TAKES_THE_PLACE hipError_t hipGetDevice(int *dev)
{
    *dev = 0;
    return hipSuccess;
}
TAKES_THE_PLACE hipError_t hipDeviceGetAttribute(int *value, hipDeviceAttribute_t, int)
{
    *value = 256;
    return hipSuccess;
}
TAKES_THE_PLACE hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
TAKES_THE_PLACE hipError_t hipLaunchKernel(const void *kernel, dim3, dim3, void **, size_t, hipStream_t)
{
    printf("%s ", kernels()[kernel].c_str());
    return hipSuccess;
}

// made-up addresses, 2^40 apart (nothing looks at them)
template <typename T>
static T *at(int i)
{
    return reinterpret_cast<T *>((1ull + i) << 40);
}

int main(int argc, char **argv)
{
    void *lib = argc == 2 ? dlopen(argv[1], RTLD_NOW) : nullptr;
    if (!lib) {
        fprintf(stderr, "%s\n", argc == 2 ? dlerror() : "launched_kernels libtpq.so");
        return 2;
    }
#define TPQ_TAKE(name) const auto name = reinterpret_cast<decltype(&::name)>(dlsym(lib, #name))
    TPQ_TAKE(tpq_layout_init);
    TPQ_TAKE(tpq_gemm_encode);
    TPQ_TAKE(tpq_decode_reduce);
    TPQ_TAKE(tpq_decode_reduce_static);
    TPQ_TAKE(tpq_calibrate_finalize);
    TPQ_TAKE(tpq_calibrate_finalize_workspace_bytes);
    char line[256], what[16];
    while (fgets(line, sizeof line, stdin)) {
        long long v[8] = {};
        if (sscanf(line, "%15s %lld %lld %lld %lld %lld %lld %lld %lld", what, v, v + 1, v + 2, v + 3, v + 4, v + 5, v + 6, v + 7) < 5) return 3;
        const int E = static_cast<int>(v[0]), k = static_cast<int>(v[1]);
        tpq_layout L = {};
        int rc;
        if (!strcmp(what, "finalize")) {
            rc = tpq_calibrate_finalize(at<float>(0), at<float>(1), static_cast<int>(v[2]), E, k, at<float>(2), at<float>(3), at<int32_t>(4),
                                        v[3] ? at<int32_t>(5) : nullptr, at<void>(6), tpq_calibrate_finalize_workspace_bytes(E), nullptr);
        } else if (!strcmp(what, "gemm")) {
            if (tpq_layout_init(&L, E, k, static_cast<int>(v[2]), 4) != TPQ_OK) return 4;
            const int K = static_cast<int>(v[4]);
            rc = tpq_gemm_encode(&L, at<uint16_t>(0), v[3], K, K, at<uint16_t>(1), at<uint8_t>(2), at<uint16_t>(3), at<uint16_t>(4),
                                 at<uint16_t>(5), nullptr, 0, nullptr);
        } else {
            if (tpq_layout_init(&L, E, k, static_cast<int>(v[2]), static_cast<int>(v[3])) != TPQ_OK) return 4;
            const int N = static_cast<int>(v[4]);
            const uint8_t *codes[TPQ_MAX_RANKS];
            const uint16_t *rest[3][TPQ_MAX_RANKS];
            for (int i = 0; i < N; ++i) {
                codes[i] = at<uint8_t>(10 + 4 * i);
                for (int s = 0; s < 3; ++s) rest[s][i] = at<uint16_t>(11 + 4 * i + s);
            }
            if (!strcmp(what, "static"))
                rc = tpq_decode_reduce_static(&L, at<void>(0), N, v[5], codes, rest[2], at<float>(1), static_cast<int>(v[6]),
                                              static_cast<int>(v[7]), at<void>(2), E, nullptr);
            else
                rc = tpq_decode_reduce(&L, at<void>(0), N, v[5], codes, rest[0], rest[1], rest[2], static_cast<int>(v[6]),
                                       static_cast<int>(v[7]), at<void>(2), E, nullptr);
        }
        if (rc != TPQ_OK) printf("- %d", rc);
        printf("\n");
    }
    return 0;
}
