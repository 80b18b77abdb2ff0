/* A HIP runtime that runs nothing, for tests of the library's host side on the
 * CPU: every buffer is host memory, a kernel launch is remembered, and the wait
 * for a stream writes the result that the last launched kernel (the fold of a
 * reduction: partials, count, mask, out) would have left. Load it with global
 * symbols before the library. */
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_;
int fake_malloc_fails, fake_sync_fails;
long fake_mallocs, fake_copies, fake_set_device;
double fake_value;
double *fake_out; /* where the last fold writes */

int hipGetDeviceCount(int *n) { *n = 1; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int d) { (void)d; fake_set_device++; return 0; }
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { return e ? "made to fail" : "no error"; }
int hipThreadExchangeStreamCaptureMode(int *mode) { static int now; int t = now; now = *mode; *mode = t; return 0; }

int hipHostMalloc(void **p, size_t bytes, unsigned flags)
{
    (void)flags;
    fake_mallocs++;
    if (fake_malloc_fails) return 2;
    *p = calloc(1, bytes);
    return 0;
}

int hipMemcpyAsync(void *dst, const void *src, size_t bytes, int kind, void *stream)
{
    (void)kind;
    (void)stream;
    fake_copies++;
    /* in stream order: after the kernel */
    for (int k = 0; k < 8; k++) fake_out[k] = fake_value + k;
    memcpy(dst, src, bytes);
    return 0;
}

int hipStreamSynchronize(void *stream)
{
    (void)stream;
    if (fake_sync_fails) return 719;
    for (int k = 0; k < 8; k++) fake_out[k] = fake_value + k;
    return 0;
}

int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t shm, void *s)
{
    (void)g; (void)b; (void)shm; (void)s;
    return 0;
}
int __hipPopCallConfiguration(dim3_ *g, dim3_ *b, size_t *shm, void **s)
{
    memset(g, 0, sizeof *g);
    memset(b, 0, sizeof *b);
    *shm = 0;
    *s = NULL;
    return 0;
}
int hipLaunchKernel(const void *f, dim3_ g, dim3_ b, void **args, size_t shm, void *s)
{
    (void)f; (void)g; (void)b; (void)shm; (void)s;
    fake_out = *(double **)args[3];
    return 0;
}
