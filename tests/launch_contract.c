/* A caller whose HIP runtime is the few functions below: what the library asks of the runtime on its way to a launch, without a
 * GPU.  The definitions of the executable come before those of the real runtime.  Modes:
 *   devices  every launch of more than 64 KB of dynamic LDS finds the attribute set for its kernel on the current device, also on
 *            the second device that a thread uses, and after a device that refused it
 *   errors   an error that another call left on the thread neither fails a launch nor is cleared by it; the launch's own error
 *            fails the call and does not stay behind
 *   lookup   a kernel whose handle cannot be had is launched by its address, and the failed look-up leaves no error on the thread
 *   streams  a stream of a device that is not the current one: the launch, its kernel's handle and the LDS are that device's, and the
 *            caller's device is current again afterwards; a stream that cannot be asked is left to the launch
 *   names    writes "ran <kernel>" to stderr for every launch, behind what the library's trace says of it
 * A kernel's handle is looked up on the current device and is good there only; a launch by address finds the kernel on the stream's device.
 * (A stream here is its device + 1.) */
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "amap.h"

typedef struct { uint32_t x, y, z; } dim3_t;
enum { OK = 0, INVALID = 1, LEFT_BEHIND = 719, LAUNCH_FAILED = 700, NOT_FOUND = 500, MAX_LDS_ATTRIBUTE = 8 };

static int device = 0, last_error = OK, launches = 0, fail_launch = 0, refuse_attribute = 0, unreserved = 0, wide_launches = 0;
static int fail_lookup = 0, by_address = 0, lookups = 0, fail_stream = 0, fail_set = 0, device_calls = 0, ran_on = -1;
static struct { const void *kernel; int device, bytes; } reserved[256];
static int n_reserved = 0;

int hipGetDevice(int *d) { *d = device; return OK; }
int hipSetDevice(int d)
{
    ++device_calls;
    if (fail_set) return last_error = INVALID;
    device = d;
    return OK;
}
int hipStreamGetDevice(void *stream, int *d)
{
    ++device_calls;
    if (fail_stream) return last_error = INVALID;
    *d = stream ? (int)(uintptr_t)stream - 1 : device;
    return OK;
}
int hipDeviceGetAttribute(int *v, int attr, int d) { (void)attr; (void)d; *v = 256; return OK; }
int hipGetLastError(void) { const int e = last_error; last_error = OK; return e; }
int hipFuncSetAttribute(const void *kernel, int attr, int value)
{
    if (attr != MAX_LDS_ATTRIBUTE || refuse_attribute || n_reserved == 256) return last_error = INVALID;
    reserved[n_reserved].kernel = kernel;
    reserved[n_reserved].device = device;
    reserved[n_reserved++].bytes = value;
    return OK;
}
typedef struct { const void *kernel; int device; } handle_t;
static handle_t handles[256];
static int n_handles = 0;
int hipGetFuncBySymbol(handle_t **f, const void *kernel)
{
    ++lookups;
    if (fail_lookup || n_handles == 256) return last_error = NOT_FOUND;
    handles[n_handles].kernel = kernel;
    handles[n_handles].device = device;
    *f = &handles[n_handles++];
    return OK;
}
/* the kernels by name, as the library registers them when it is loaded */
static struct { const void *kernel; const char *name; } names[512];
static int n_names = 0, say_names = 0;
void __hipRegisterFunction(void **modules, const void *kernel, char *symbol, const char *name, unsigned threads, void *tid, void *bid, dim3_t *block,
                           dim3_t *grid, int *warp)
{
    (void)modules; (void)symbol; (void)threads; (void)tid; (void)bid; (void)block; (void)grid; (void)warp;
    if (n_names == 512) return;
    names[n_names].kernel = kernel;
    names[n_names++].name = name;
}
static int launch(const void *kernel, int on, unsigned grid, unsigned block, size_t lds, const void *stream)
{
    int found = lds <= 65536;
    if (fail_launch) return last_error = LAUNCH_FAILED;
    if (!grid || !block || on != (stream ? (int)(uintptr_t)stream - 1 : device)) return last_error = INVALID;
    ran_on = on;
    for (int i = 0; say_names && i < n_names; ++i)
        if (names[i].kernel == kernel) fprintf(stderr, "ran %s\n", names[i].name);
    for (int i = 0; i < n_reserved; ++i)
        found |= reserved[i].kernel == kernel && reserved[i].device == on && (size_t)reserved[i].bytes >= lds;
    unreserved += !found;
    wide_launches += lds > 65536;
    ++launches;
    return OK;
}
int hipLaunchKernel(const void *kernel, dim3_t grid, dim3_t block, void **args, size_t lds, void *stream)
{
    (void)args;
    ++by_address;
    return launch(kernel, stream ? (int)(uintptr_t)stream - 1 : device, grid.x, block.x, lds, stream);
}
int hipModuleLaunchKernel(const handle_t *f, unsigned gx, unsigned gy, unsigned gz, unsigned bx, unsigned by, unsigned bz, unsigned lds, void *stream,
                          void **args, void **extra)
{
    (void)args;
    if (gy != 1 || gz != 1 || by != 1 || bz != 1 || extra) return last_error = INVALID;
    return launch(f->kernel, f->device, gx, bx, lds, stream);
}

static amap_t *layout(int64_t a, int64_t b, int64_t c, int64_t d, int merge)
{
    const int64_t shape[4] = {a, b, c, d}, perm[4] = {0, 2, 1, 3}, rows[2] = {a * c, b * d};
    amap_src_desc src = {4, shape, AMAP_B16};
    amap_op ops[2];
    amap_t *m = NULL;
    memset(ops, 0, sizeof(ops));
    ops[0].kind = AMAP_TRANSPOSE; ops[0].n = 4; ops[0].a = perm;
    ops[1].kind = AMAP_RESHAPE;   ops[1].n = 2; ops[1].a = rows;
    return amap_compose(&src, 1, ops, merge ? 2 : 1, &m) == AMAP_OK ? m : NULL;
}

/* addresses that nothing reads */
static const void *const srcs[1] = {(const void *)((uintptr_t)1 << 40)};
static const void *const weight = (const void *)((uintptr_t)2 << 40);
static void *const out = (void *)((uintptr_t)3 << 40);

/* one product per GEMM kernel that asks for more than 64 KB: 64 x 128 tiles, 256 x 256 tiles, the general kernel */
static const struct { int64_t b, h, s, d, n; } products[3] = {{1, 20, 2341, 64, 760}, {16, 16, 512, 64, 4096}, {1, 9, 300, 8, 256}};

static amap_status product_on(int i, void *stream)
{
    amap_t *m = layout(products[i].b, products[i].h, products[i].s, products[i].d, 1);
    const amap_status st = m ? amap_gemm_gather(srcs, m, weight, NULL, products[i].n, NULL, out, stream) : AMAP_E_INVALID;
    amap_free(m);
    return st;
}
static amap_status product(int i) { return product_on(i, NULL); }

/* every way to a launch: the layout call, the call of several maps, the products */
enum { WAYS = 5 };
static amap_status way(int i, void *stream)
{
    amap_t *m;
    amap_status st = AMAP_E_INVALID;
    if (i >= 2) return product_on(i - 2, stream);
    if ((m = layout(2, 8, 64, 64, 0))) st = i == 0 ? amap_execute(srcs, out, m, stream) : amap_execute_multi(srcs, &out, (const amap_t *const *)&m, 1, stream);
    amap_free(m);
    return st;
}

#define EXPECT(x)                                             \
    do {                                                      \
        if (!(x)) {                                           \
            printf("FAIL line %d: %s\n", __LINE__, #x);       \
            return 1;                                         \
        }                                                     \
    } while (0)

int main(int argc, char **argv)
{
    launches = n_reserved = 0;
    if (argc == 2 && !strcmp(argv[1], "devices")) {
        const int walk[6] = {0, 0, 1, 0, 3, 1};
        for (int i = 0; i < 3; ++i) {
            device = 2;
            refuse_attribute = 1;
            EXPECT(product(i) == AMAP_E_HIP && launches == 0 && last_error == OK);
        }
        refuse_attribute = 0;
        for (int w = 0; w < 6; ++w)
            for (int i = 0; i < 3; ++i) {
                device = walk[w];
                EXPECT(product(i) == AMAP_OK);
                EXPECT(wide_launches == 3 * w + i + 1 && unreserved == 0);
            }
        device = 2;   /* refused before, asked again */
        for (int i = 0; i < 3; ++i) EXPECT(product(i) == AMAP_OK && unreserved == 0);
        const int asked = n_reserved, looked = lookups;
        for (int i = 0; i < 3; ++i) EXPECT(product(i) == AMAP_OK && n_reserved == asked && lookups == looked);   /* once per device is enough */
        EXPECT(by_address == 0);
    } else if (argc == 2 && !strcmp(argv[1], "errors")) {
        amap_t *m = layout(2, 8, 64, 64, 0);
        EXPECT(m);
        for (int i = -1; i < 3; ++i) {
            const int before = launches;
            last_error = LEFT_BEHIND;
            EXPECT((i < 0 ? amap_execute(srcs, out, m, NULL) : product(i)) == AMAP_OK);
            EXPECT(launches == before + 1 && last_error == LEFT_BEHIND);
            last_error = OK;
            fail_launch = 1;
            EXPECT((i < 0 ? amap_execute(srcs, out, m, NULL) : product(i)) == AMAP_E_HIP);
            EXPECT(last_error == OK && strlen(amap_last_error()) > 0);
            fail_launch = 0;
        }
        EXPECT(by_address == 0);
        amap_free(m);
    } else if (argc == 2 && !strcmp(argv[1], "lookup")) {
        amap_t *m = layout(2, 8, 64, 64, 0);
        EXPECT(m);
        fail_lookup = 1;
        for (int i = -1; i < 3; ++i) {
            EXPECT((i < 0 ? amap_execute(srcs, out, m, NULL) : product(i)) == AMAP_OK);
            EXPECT(by_address == i + 2 && last_error == OK);
        }
        fail_lookup = 0;   /* asked again, and found */
        for (int i = -1; i < 3; ++i) EXPECT((i < 0 ? amap_execute(srcs, out, m, NULL) : product(i)) == AMAP_OK);
        EXPECT(by_address == 4 && launches == 8 && last_error == OK);
        amap_free(m);
    } else if (argc == 2 && !strcmp(argv[1], "streams")) {
        for (int i = 0; i < WAYS; ++i)
            for (int k = 0; k < 9; ++k) {
                void *const stream = (void *)(uintptr_t)(k % 3 + 1);
                device = k / 3;
                EXPECT(way(i, stream) == AMAP_OK && ran_on == k % 3 && device == k / 3 && unreserved == 0 && last_error == OK);
                device_calls = 0;
                EXPECT(way(i, NULL) == AMAP_OK && ran_on == k / 3 && unreserved == 0 && device_calls == 0);
            }
        EXPECT(by_address == 0);
        device = 0;
        for (int i = 0; i < WAYS; ++i) {
            fail_launch = 1;   /* back on the caller's device after an error too */
            EXPECT(way(i, (void *)2) == AMAP_E_HIP && device == 0 && last_error == OK);
            fail_launch = 0;
            fail_stream = 1;
            EXPECT(way(i, (void *)1) == AMAP_OK && ran_on == 0 && last_error == OK);
            fail_stream = 0;
            fail_set = 1;
            EXPECT(way(i, (void *)2) == AMAP_E_HIP && device == 0 && last_error == OK);
            fail_set = 0;
        }
    } else if (argc == 2 && !strcmp(argv[1], "names")) {
        /* [a,b,c,d] with b and c exchanged; up to 32 MB and beyond, one map and several, rows of one element */
        const struct { int64_t a, b, c, d, n; } calls[] = {{2, 8, 64, 64, 1}, {64, 12, 512, 64, 1}, {2, 8, 64, 64, 3}, {32, 12, 512, 64, 2}, {2, 8, 64, 64, 4},
                                                           {8, 64, 4096, 1, 1}, {16, 288, 1225, 1, 1}, {3, 5, 7, 3, 1}};
        say_names = 1;
        for (unsigned i = 0; i < sizeof(calls) / sizeof(calls[0]); ++i) {
            amap_t *m = layout(calls[i].a, calls[i].b, calls[i].c, calls[i].d, 0);
            const amap_t *maps[4] = {m, m, m, m};
            void *const outs[4] = {out, (char *)out + (1 << 26), (char *)out + (2 << 26), (char *)out + (3 << 26)};
            EXPECT(m && (calls[i].n == 1 ? amap_execute(srcs, out, m, NULL) : amap_execute_multi(srcs, outs, maps, (int)calls[i].n, NULL)) == AMAP_OK);
            amap_free(m);
        }
    } else {
        return 2;
    }
    printf("OK\n");
    return 0;
}
