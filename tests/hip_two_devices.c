/* Stand-ins for the HIP runtime calls of the surrogate's host code, preloaded
 * over the real ones on a host without a GPU: two devices of host memory, and
 * kernels that do nothing but note the device that was current at their launch
 * (-1 if a synchronisation was on another device than the launch that follows). */
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_t;
static int current, synced = -1, launched[4096], n_launched;

int hipGetDevice(int *d) { *d = current; return 0; }
int hipSetDevice(int d) { if (d < 0 || d > 1) return 101; current = d; return 0; }
int hipMalloc(void **p, size_t n) { *p = calloc(n, 1); return *p ? 0 : 2; }
int hipFree(void *p) { free(p); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int k) { (void)k; memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { (void)k; (void)st; memcpy(d, s, n); return 0; }
int hipMemsetAsync(void *d, int v, size_t n, void *st) { (void)st; memset(d, v, n); return 0; }
int hipDeviceSynchronize(void) { synced = current; return 0; }
int hipStreamSynchronize(void *st) { (void)st; return 0; }
int hipGetLastError(void) { return 0; }
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t l, void *st)
{
    (void)g; (void)b; (void)l; (void)st;
    return 0;
}
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *l, void **st)
{
    const dim3_t one = {1, 1, 1};
    *g = *b = one;
    *l = 0;
    *st = NULL;
    return 0;
}
int hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **a, size_t l, void *st)
{
    (void)f; (void)g; (void)b; (void)a; (void)l; (void)st;
    if (n_launched < 4096) launched[n_launched++] = synced < 0 || synced == current ? current : -1;
    return 0;
}
int test_launches(void) { return n_launched; }
int test_launch_device(int i) { return launched[i]; }
void test_forget(void) { n_launched = 0; synced = -1; }
