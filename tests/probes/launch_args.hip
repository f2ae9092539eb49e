// Prints what tpq_decode_reduce (fp32 output: column passes at any size) hands to its kernels, without a GPU: this program's own launch functions take the
// place of the runtime's for the library it loads; they read the argument block and launch nothing.
//
//   launch_args libtpq.so E k G bits N T pitch_outl
//
// The sections lie at made-up addresses (nothing looks at them): rank i's codes, scale, zero, outl at
// (1 + 4 i + s) * 2^40.  One line per launch: rows, pitch_outl, then the 8-rank groups' outl pointers in hex.
#include <dlfcn.h>
#include <stdio.h>
#include <stdlib.h>

#include "tpq_internal.h"

#define TAKES_THE_PLACE extern "C" __attribute__((visibility("default")))

TAKES_THE_PLACE hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
TAKES_THE_PLACE hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
TAKES_THE_PLACE hipError_t hipGetLastError() { return hipSuccess; }

TAKES_THE_PLACE hipError_t hipLaunchKernel(const void *, dim3, dim3, void **args, size_t, hipStream_t)
{
    const tpq::DecodeArgs &a = *static_cast<const tpq::DecodeArgs *>(args[0]);
    const tpq::RankPtrs &outl = *static_cast<const tpq::RankPtrs *>(args[4]);
    printf("%lld %lld", static_cast<long long>(a.T), static_cast<long long>(a.pitch_outl));
    for (int i = 0; i < (a.n_ranks + 7) / 8 * 8; ++i) printf(" %llx", static_cast<unsigned long long>(reinterpret_cast<uintptr_t>(outl.p[i])));
    printf("\n");
    return hipSuccess;
}

int main(int argc, char **argv)
{
    if (argc != 9) return 2;
    void *lib = dlopen(argv[1], RTLD_NOW);
    if (!lib) {
        fprintf(stderr, "%s\n", dlerror());
        return 3;
    }
    const auto init = reinterpret_cast<decltype(&tpq_layout_init)>(dlsym(lib, "tpq_layout_init"));
    const auto decode = reinterpret_cast<decltype(&tpq_decode_reduce)>(dlsym(lib, "tpq_decode_reduce"));
    tpq_layout L;
    if (init(&L, atoi(argv[2]), atoi(argv[3]), atoi(argv[4]), atoi(argv[5])) != TPQ_OK) return 4;
    const int N = atoi(argv[6]);
    L.pitch_outl = atoll(argv[8]);
    const uint8_t *codes[TPQ_MAX_RANKS];
    const uint16_t *rest[3][TPQ_MAX_RANKS];
    for (int i = 0; i < N; ++i) {
        codes[i] = reinterpret_cast<const uint8_t *>((1ull + 4 * i) << 40);
        for (int s = 0; s < 3; ++s) rest[s][i] = reinterpret_cast<const uint16_t *>((2ull + 4 * i + s) << 40);
    }
    return decode(&L, reinterpret_cast<void *>(1ull << 39), N, atoll(argv[7]), codes, rest[0], rest[1], rest[2], TPQ_ACC_FP32,
                  TPQ_OUT_FP32, reinterpret_cast<void *>(1ull << 38), L.E, nullptr) == TPQ_OK
               ? 0
               : 5;
}
