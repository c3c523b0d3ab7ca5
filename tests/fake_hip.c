/* Stand-ins for the HIP calls of a synchronous libfrnn call, for tests of its host side
 * without a GPU: several devices, each with an address of its own for the same pinned host
 * memory.  The kernel whose mangled name contains fake_kernel gets the address that it
 * writes the result to as argument number fake_arg; a synchronisation "runs" it, and the
 * result arrives only if that is the current device's address (or by a copy to the host,
 * where mapping fails).  The names of search kernels are kept for tests of the launch. */
#include <stddef.h>
#include <stdlib.h>
#include <string.h>

int fake_device, fake_arg, fake_map_fails, fake_copies;
unsigned fake_flags;
char fake_kernel[64], fake_result[128];
char fake_asked[256], fake_searched[256]; /* search kernels: asked for its occupancy, launched last */

typedef struct {
    unsigned x, y, z;
} dims;

static char *host;
static size_t host_bytes;
static const void *wanted;
static void *written;

static struct {
    const void *f;
    char name[256];
} searches[256];
static int n_searches;

static void name_of(const void *f, char *name) {
    for (int k = 0; k < n_searches; ++k)
        if (searches[k].f == f) strcpy(name, searches[k].name);
}

static char *address(int device) { return host + (size_t)(device + 1) * 4096; }

void **__hipRegisterFatBinary(const void *data) {
    static void *module;
    module = (void *)data;
    return &module;
}
void __hipUnregisterFatBinary(void **module) { (void)module; }
void __hipRegisterVar(void **m, void *v, char *h, char *n, int e, size_t s, int c, int g) {
    (void)m, (void)v, (void)h, (void)n, (void)e, (void)s, (void)c, (void)g;
}
void __hipRegisterFunction(void **m, const void *f, char *name, const char *n, unsigned t, void *a, void *b, void *c,
                           void *d, int *w) {
    (void)m, (void)n, (void)t, (void)a, (void)b, (void)c, (void)d, (void)w;
    if (fake_kernel[0] && strstr(name, fake_kernel)) wanted = f;
    if (strstr(name, "k_search") && strlen(name) < 256 && n_searches < 256) {
        searches[n_searches].f = f;
        strcpy(searches[n_searches++].name, name);
    }
}
int __hipPushCallConfiguration(dims g, dims b, size_t lds, void *stream) {
    (void)g, (void)b, (void)lds, (void)stream;
    return 0;
}
int __hipPopCallConfiguration(dims *g, dims *b, size_t *lds, void **stream) {
    memset(g, 0, sizeof *g), memset(b, 0, sizeof *b), *lds = 0, *stream = NULL;
    return 0;
}
int hipLaunchKernel(const void *f, dims g, dims b, void **args, size_t lds, void *stream) {
    (void)g, (void)b, (void)lds, (void)stream;
    name_of(f, fake_searched);
    if (f == wanted) memcpy(&written, args[fake_arg], sizeof written);
    return 0;
}
int hipGetDevice(int *d) {
    *d = fake_device;
    return 0;
}
int hipDeviceGetAttribute(int *v, int attribute, int device) {
    (void)attribute, (void)device;
    *v = 256;
    return 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *v, const void *f, int threads, size_t lds) {
    (void)threads, (void)lds;
    name_of(f, fake_asked);
    *v = 4;
    return 0;
}
int hipHostMalloc(void **p, size_t bytes, unsigned flags) {
    host = calloc(8, 4096);
    host_bytes = bytes;
    fake_flags = flags;
    *p = host;
    return 0;
}
int hipHostGetDevicePointer(void **d, void *h, unsigned flags) {
    (void)flags;
    if (h != host || fake_map_fails) return 1;
    *d = address(fake_device);
    return 0;
}
int hipMemcpyAsync(void *to, const void *from, size_t bytes, int kind, void *stream) {
    (void)from, (void)kind, (void)stream;
    ++fake_copies;
    memcpy(to, fake_result, bytes);
    return 0;
}
int hipGetLastError(void) { return 0; }
int hipStreamSynchronize(void *stream) {
    (void)stream;
    if (written == address(fake_device)) memcpy(host, fake_result, host_bytes);
    return 0;
}
