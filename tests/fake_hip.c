/* A HIP runtime without a GPU, preloaded before libibm.so (tests/test_host_calls.py): device memory
   is the caller's host memory, copies and fills are done at once, kernels are not run.  Every call
   that does or awaits device work is written to the log as "name stream-or-object device". */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

static int device;
static FILE *out;
static struct {
    size_t bytes;
    char data[4096];
} reads[8];
static int nread;

typedef struct {
    int device;
} Event;

static void note(const char *what, const void *p, int dev) {
    if (!out) out = fopen(getenv("FAKE_HIP_LOG"), "w");
    fprintf(out, "%s %p %d\n", what, p, dev);
    fflush(out);
}

/* the next device-to-host copy of so many bytes delivers data (what the kernels would have left) */
void fake_hip_next_read(size_t bytes, const void *data) {
    reads[nread].bytes = bytes;
    memcpy(reads[nread++].data, data, bytes);
}
void fake_hip_mark(void) { note("mark", NULL, device); }

int hipGetDevice(int *d) {
    note("hipGetDevice", NULL, device);
    *d = device;
    return 0;
}
int hipSetDevice(int d) {
    device = d;
    return 0;
}
int hipDeviceGetAttribute(int *v, int attr, int d) {
    (void)attr;
    note("hipDeviceGetAttribute", NULL, d);
    *v = 256;
    return 0;
}
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { return e ? "fake error" : "no error"; }
int hipHostMalloc(void **p, size_t n, unsigned f) {
    (void)f;
    *p = calloc(1, n);
    return 0;
}
int hipHostFree(void *p) {
    free(p);
    return 0;
}
int hipMemcpyAsync(void *dst, const void *src, size_t n, int kind, void *s) {
    note("copy", s, device);
    memmove(dst, src, n);
    for (int q = 0; kind == 2 && q < nread; ++q)
        if (reads[q].bytes == n) {
            memcpy(dst, reads[q].data, n);
            reads[q] = reads[--nread];
            break;
        }
    return 0;
}
int hipMemsetAsync(void *p, int v, size_t n, void *s) {
    note("fill", s, device);
    memset(p, v, n);
    return 0;
}
int hipLaunchKernel(const void *f, uint64_t g0, uint32_t g1, uint64_t b0, uint32_t b1, void **a, size_t sh, void *s) {
    (void)f, (void)g0, (void)g1, (void)b0, (void)b1, (void)a, (void)sh;
    note("kernel", s, device);
    return 0;
}
int hipStreamSynchronize(void *s) {
    note("wait", s, device);
    return 0;
}
int hipEventCreateWithFlags(void **e, unsigned f) {
    (void)f;
    Event *v = malloc(sizeof(Event));
    v->device = device;
    *e = v;
    note("create", v, device);
    return 0;
}
int hipEventDestroy(void *e) {
    note("destroy", e, ((Event *)e)->device);
    return 0; /* kept, so that no later event has its address */
}
int hipEventRecord(void *e, void *s) {
    (void)s;
    note("record", e, device);
    return ((Event *)e)->device == device ? 0 : 400; /* invalid handle: the stream is another device's */
}
int hipEventSynchronize(void *e) {
    note("wait event", e, device);
    return 0;
}
int hipEventQuery(void *e) {
    (void)e;
    return 0;
}
