// A caller whose HIP runtime runs amap_rows_few_kernel on the CPU: the library's launch hands over the kernel's argument, every lane
// of every workgroup is walked with the kernel's own index functions, and the bytes are moved in the caller's memory.  What the call
// left there is compared with the permutation it asks for, so that the division of the workgroups among the pieces and which pieces
// count as alike are seen as well as the decode.  (No GPU.  A launch of another kernel is named and moves nothing.)
//   rows_few_replay <element bytes> <few | other> <maps>, a map: a,b,c,d,swap,order  [a,b,c,d] with the two dimensions of swap exchanged
//   (01 12 02; none: --) and the place of its output among the others in memory
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <memory>
#include <string>
#include <vector>

#include "amap.h"
#include "amap_index.hpp"

using namespace amap_dev;

static std::map<const void *, std::string> &names() {
    static std::map<const void *, std::string> m;
    return m;
}
static int few = 0, others = 0;

template <int N, int L>
static void walk(const RowsFew<N, L> &F, int es, uint32_t grid, uint32_t threads) {
    for (uint32_t block = 0; block < grid; ++block)
        for (uint32_t tid = 0; tid < threads; ++tid) {
            uint32_t b;
            const FewPiece p = rows_few_block(F, threads, block, b);
            for (uint32_t u = 0; u < (uint32_t)kRowsUnroll; ++u) {
                const uint32_t r = b * (threads * kRowsUnroll) + tid + u * threads;
                if (r >= F.n_units) continue;
                uint32_t d, s;
                rows_few_offsets(F, r, d, s);
                std::memcpy(p.dst + (size_t)d * es, p.src + (size_t)s * es, 16);
            }
        }
}

extern "C" {
void __hipRegisterFunction(void **, const void *kernel, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *, int *) { names()[kernel] = name; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetFuncBySymbol(hipFunction_t *f, const void *kernel) { return *f = (hipFunction_t)const_cast<void *>(kernel), hipSuccess; }
hipError_t hipModuleLaunchKernel(hipFunction_t f, unsigned gx, unsigned, unsigned, unsigned bx, unsigned, unsigned, unsigned, hipStream_t, void **args, void **) {
    const std::string &name = names()[(const void *)f];
    const size_t at = name.find("amap_rows_few_kernelILi");
    if (at == std::string::npos) return ++others, hipSuccess;
    const int es = name[at + strlen("amap_rows_few_kernelILi")] - '0';
    if (name.find("ELi1ELi5E", at) != std::string::npos)
        walk(*static_cast<const RowsOne *>(args[0]), es, gx, bx);
    else if (name.find("ELi3ELi4E", at) != std::string::npos)
        walk(*static_cast<const RowsThree *>(args[0]), es, gx, bx);
    else
        return hipErrorInvalidValue;
    return ++few, hipSuccess;
}
}

static int fail(const char *what) {
    std::printf("FAIL %s\n", what);
    return 1;
}

int main(int argc, char **argv) {
    if (argc < 4) return 2;
    const int es = std::atoi(argv[1]), n = argc - 3;
    const bool want_few = !std::strcmp(argv[2], "few");
    std::vector<amap_t *> maps(n);
    std::vector<int64_t> bytes(n), shape(4);
    std::vector<std::vector<int64_t>> perm(n);
    std::vector<int> order(n);
    for (int i = 0; i < n; ++i) {
        long long s[4];
        char swap[3];
        if (std::sscanf(argv[3 + i], "%lld,%lld,%lld,%lld,%2[-0-9],%d", s, s + 1, s + 2, s + 3, swap, &order[i]) != 6) return 2;
        shape.assign(s, s + 4);
        perm[i] = {0, 1, 2, 3};
        if (swap[0] != '-') std::swap(perm[i][swap[0] - '0'], perm[i][swap[1] - '0']);
        amap_src_desc src = {4, shape.data(), es == 2 ? AMAP_B16 : AMAP_B32};
        amap_op op;
        std::memset(&op, 0, sizeof(op));
        op.kind = AMAP_TRANSPOSE;
        op.n = 4;
        op.a = perm[i].data();
        if (amap_compose(&src, 1, &op, 1, &maps[i]) != AMAP_OK) return fail("compose");
        bytes[i] = shape[0] * shape[1] * shape[2] * shape[3] * es;   // (one source: as many in each)
    }
    // sources and outputs in one block of memory, guards of 256 bytes between them
    const int64_t room = (bytes[0] + 511) / 256 * 256;
    std::vector<char> memory((size_t)room * (n + 2) + 256);
    char *const base = memory.data() + (256 - (uintptr_t)memory.data() % 256) % 256;
    std::memset(base, 0x5A, (size_t)room * (n + 1));
    for (int64_t i = 0; i < bytes[0]; ++i) base[i] = (char)(i * 2654435761u >> 13);
    const void *src = base;
    std::vector<void *> dst(n);
    for (int i = 0; i < n; ++i) dst[i] = base + room * (1 + order[i]);
    if ((n == 1 ? amap_execute(&src, dst[0], maps[0], nullptr) : amap_execute_multi(&src, dst.data(), maps.data(), n, nullptr)) != AMAP_OK) return fail("execute");
    if (want_few ? few != 1 || others : few) return fail(want_few ? "another kernel" : "amap_rows_few_kernel");
    for (int i = 0; want_few && i < n; ++i) {
        const char *d = static_cast<const char *>(dst[i]);
        int64_t to[4], at = 0, stride[4] = {shape[1] * shape[2] * shape[3], shape[2] * shape[3], shape[3], 1};
        const std::vector<int64_t> &p = perm[i];
        for (to[0] = 0; to[0] < shape[p[0]]; ++to[0])
            for (to[1] = 0; to[1] < shape[p[1]]; ++to[1])
                for (to[2] = 0; to[2] < shape[p[2]]; ++to[2], at += shape[3]) {
                    int64_t from = 0;
                    for (int k = 0; k < 3; ++k) from += to[k] * stride[p[k]];
                    if (std::memcmp(d + at * es, base + from * es, (size_t)shape[3] * es)) return fail("a row");
                }
        for (int64_t k = bytes[i]; k < room; ++k)
            if (d[k] != 0x5A) return fail("behind the output");
    }
    for (amap_t *m : maps) amap_free(m);
    std::printf("OK\n");
    return 0;
}
