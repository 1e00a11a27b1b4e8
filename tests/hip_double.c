/* A stand-in for the HIP runtime, preloaded into a process without a GPU: it
 * records the calls the library makes, launches nothing, and fails the calls
 * it is told to fail.  Device pointers are never followed. */
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef int err_t;

static char g_log[1 << 20];
static size_t g_len;
static char g_fail[64];
static int g_fail_left, g_fail_after;
static err_t g_sticky;
static uint32_t g_word;          /* what a 4-byte copy to the host brings, once */
static uint32_t g_cu_mask[8];
static int g_mask_set;

static struct { const void* fn; char name[160]; } g_fns[512];
static int g_nfns;

static void note(const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    if (g_len < sizeof(g_log) - 256)
        g_len += (size_t)vsnprintf(g_log + g_len, 256, fmt, ap);
    va_end(ap);
}
static err_t call(const char* name)
{
    if (g_fail_left > 0 && !strcmp(name, g_fail) && g_fail_after-- <= 0) {
        --g_fail_left;
        g_sticky = 2;
        note("%s failed\n", name);
        return 2;
    }
    return 0;
}
static const char* fn_name(const void* f)
{
    for (int i = 0; i < g_nfns; ++i)
        if (g_fns[i].fn == f) return g_fns[i].name;
    return "?";
}

/* for the test */
const char* double_log(void) { return g_log; }
void double_clear(void) { g_len = 0; g_log[0] = 0; }
void double_fail(const char* name, int times, int after)
{
    snprintf(g_fail, sizeof(g_fail), "%s", name);
    g_fail_left = times;
    g_fail_after = after;
}
void double_word(uint32_t w) { g_word = w; }
void double_cu_mask(const uint32_t* m) { memcpy(g_cu_mask, m, sizeof(g_cu_mask)); g_mask_set = 1; }

/* registration and launches */
void** __hipRegisterFatBinary(const void* d) { static void* h; (void)d; return &h; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t s, int c, int g)
{
    (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g;
}
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned t,
                           void* a, void* b, void* c, void* d, int* w)
{
    (void)m; (void)dev; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
    if (g_nfns < 512) {
        g_fns[g_nfns].fn = host;
        snprintf(g_fns[g_nfns++].name, 160, "%s", name);
    }
}
static dim3_t g_grid, g_block;
static size_t g_lds;
static void* g_stream;
err_t __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void* stream)
{
    g_grid = grid; g_block = block; g_lds = lds; g_stream = stream;
    return 0;
}
err_t __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* lds, void** stream)
{
    *grid = g_grid; *block = g_block; *lds = g_lds; *stream = g_stream;
    return 0;
}
err_t hipLaunchKernel(const void* f, dim3_t grid, dim3_t block, void** args, size_t lds, void* s)
{
    (void)args; (void)s;
    note("launch %s grid %u block %u lds %zu\n", fn_name(f), grid.x, block.x, lds);
    return call("hipLaunchKernel");
}
err_t hipExtLaunchKernel(const void* f, dim3_t grid, dim3_t block, void** args, size_t lds, void* s,
                         void* e0, void* e1, int flags)
{
    (void)e0; (void)e1; (void)flags;
    return hipLaunchKernel(f, grid, block, args, lds, s);
}
err_t hipLaunchCooperativeKernel(const void* f, dim3_t grid, dim3_t block, void** args, unsigned lds,
                                 void* s)
{
    (void)args; (void)s;
    note("cooperative %s grid %u block %u lds %u\n", fn_name(f), grid.x, block.x, lds);
    return call("hipLaunchCooperativeKernel");
}
err_t hipFuncSetAttribute(const void* f, int attr, int v)
{
    note("hipFuncSetAttribute %s %d %d\n", fn_name(f), attr, v);
    return call("hipFuncSetAttribute");
}

/* memory, events, streams, device */
err_t hipMemcpyAsync(void* dst, const void* src, size_t n, int kind, void* s)
{
    (void)src; (void)s;
    note("hipMemcpyAsync %zu kind %d\n", n, kind);
    if (kind == 2) {
        memset(dst, 0, n);
        if (n == 4) {
            memcpy(dst, &g_word, 4);
            g_word = 0;
        }
    }
    return call("hipMemcpyAsync");
}
err_t hipHostMalloc(void** p, size_t n, unsigned flags)
{
    (void)flags;
    note("hipHostMalloc\n");
    const err_t e = call("hipHostMalloc");
    *p = e ? NULL : calloc(1, n);
    return e;
}
err_t hipHostFree(void* p) { free(p); return 0; }
static err_t new_event(const char* name, void** e)
{
    note("%s\n", name);
    const err_t r = call(name);
    *e = r ? NULL : malloc(1);
    return r;
}
err_t hipEventCreate(void** e) { return new_event("hipEventCreate", e); }
err_t hipEventCreateWithFlags(void** e, unsigned f) { (void)f; return new_event("hipEventCreateWithFlags", e); }
err_t hipEventDestroy(void* e) { free(e); return 0; }
err_t hipEventRecord(void* e, void* s) { (void)e; (void)s; note("hipEventRecord\n"); return call("hipEventRecord"); }
err_t hipEventSynchronize(void* e) { (void)e; return 0; }
err_t hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 1.0f; return 0; }
err_t hipStreamSynchronize(void* s) { (void)s; note("hipStreamSynchronize\n"); return 0; }
err_t hipStreamWaitEvent(void* s, void* e, unsigned f) { (void)s; (void)e; (void)f; return 0; }
err_t hipExtStreamGetCUMask(void* s, uint32_t n, uint32_t* m)
{
    (void)s;
    for (uint32_t i = 0; i < n; ++i) m[i] = i >= 8 ? 0u : g_mask_set ? g_cu_mask[i] : ~0u;
    return call("hipExtStreamGetCUMask");
}
err_t hipGetDevice(int* d) { *d = 0; return 0; }
err_t hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
err_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int b, size_t l)
{
    (void)f; (void)b; (void)l;
    *n = 4;
    return 0;
}
err_t hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = (void*)4096; return 0; }
const char* hipGetErrorString(err_t e) { return e ? "error" : "no error"; }
err_t hipGetLastError(void) { const err_t e = g_sticky; g_sticky = 0; return e; }
