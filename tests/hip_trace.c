/* Stand-ins for the HIP runtime calls that libtensair makes, which only write down what was asked for: loaded with
 * RTLD_GLOBAL ahead of the library, they let its host side run on a machine without a GPU (nothing is executed on the
 * pointers it is given).  One line per call, read with hip_trace_take:
 *   launch <mangled kernel> <workgroups> <threads> <stream>     event <event> <stream>     wait <stream> <event>
 */
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;

static char *text;
static size_t used, room;
static struct { const void *f; char name[512]; } kernel[2048];
static int kernels, capturing;
static uintptr_t handles = 16;
static struct { dim3 grid, block; size_t lds; void *stream; } config;

static void say(const char *fmt, const char *name, unsigned long long a, unsigned long long b, unsigned long long c)
{
    if (room - used < 1024) {
        room = room ? 2 * room : 1 << 16;
        text = (char *)realloc(text, room);
        if (!text) abort();
    }
    used += (size_t)snprintf(text + used, room - used, fmt, name, a, b, c);
}

const char *hip_trace_take(void)
{
    say("%s", "", 0, 0, 0);
    used = 0;
    return text;
}
void hip_trace_capture(int on) { capturing = on; }

void **__hipRegisterFatBinary(const void *data) { (void)data; return (void **)&handles; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *var, char *host, char *dev, int ext, size_t size, int constant, int global)
{
    (void)m; (void)var; (void)host; (void)dev; (void)ext; (void)size; (void)constant; (void)global;
}
void __hipRegisterFunction(void **m, const void *f, char *name, const char *dev, unsigned limit, void *t, void *b, dim3 *bd,
                           dim3 *gd, int *ws)
{
    (void)m; (void)dev; (void)limit; (void)t; (void)b; (void)bd; (void)gd; (void)ws;
    if (kernels == (int)(sizeof(kernel) / sizeof(kernel[0]))) abort();
    kernel[kernels].f = f;
    snprintf(kernel[kernels++].name, sizeof(kernel[0].name), "%s", name);
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream)
{
    config.grid = grid;
    config.block = block;
    config.lds = lds;
    config.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream)
{
    *grid = config.grid;
    *block = config.block;
    *lds = config.lds;
    *stream = config.stream;
    return 0;
}
int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, void *stream)
{
    const char *name = "?";
    (void)args; (void)lds;
    for (int i = 0; i < kernels; ++i)
        if (kernel[i].f == f) name = kernel[i].name;
    say("launch %s %llu %llu %llu\n", name, (unsigned long long)grid.x * grid.y * grid.z,
        (unsigned long long)block.x * block.y * block.z, (unsigned long long)(uintptr_t)stream);
    return 0;
}
int hipEventCreate(void **e) { *e = (void *)(handles += 16); return 0; }
int hipEventCreateWithFlags(void **e, unsigned flags) { (void)flags; return hipEventCreate(e); }
int hipEventDestroy(void *e) { (void)e; return 0; }
int hipEventRecord(void *e, void *stream)
{
    say("%sevent %llu %llu\n", "", (uintptr_t)e, (uintptr_t)stream, 0);
    return 0;
}
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 0.f; return 0; }
int hipStreamCreateWithFlags(void **s, unsigned flags) { (void)flags; *s = (void *)(handles += 16); return 0; }
int hipStreamDestroy(void *s) { (void)s; return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipStreamWaitEvent(void *s, void *e, unsigned flags)
{
    (void)flags;
    say("%swait %llu %llu\n", "", (uintptr_t)s, (uintptr_t)e, 0);
    return 0;
}
int hipStreamIsCapturing(void *s, int *status) { (void)s; *status = capturing; return 0; }
int hipMemcpyAsync(void *dst, const void *src, size_t n, int kind, void *s)
{
    (void)dst; (void)src; (void)n; (void)kind; (void)s;
    return 0;
}
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetSymbolAddress(void **p, const void *sym) { (void)sym; *p = (void *)(uintptr_t)0x100000; return 0; }
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { (void)e; return "error"; }
