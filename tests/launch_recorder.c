/* Stands in for the HIP runtime functions that the library imports, so that a process without a GPU can make calls: records
 * kernel launches and events in order, and refuses the launch it is told to.  Nothing runs and no pointer is followed. */
#include <stddef.h>
#include <stdio.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_t;

static const void *fn_of[4096];
static const char *name_of[4096];
static int functions, launches, fail_at, last_error;
static char text[1 << 16];
static size_t used;

void recorder_reset(int refuse) { launches = 0, fail_at = refuse, last_error = 0, used = 0, text[0] = 0; }
const char *recorder_text(void) { return text; }

static void line(const char *kind, const char *what, dim3_t g)
{
    if (used + 512 < sizeof text) used += (size_t)snprintf(text + used, 512, "%s %.400s %u %u %u\n", kind, what, g.x, g.y, g.z);
}

void **__hipRegisterFatBinary(const void *data) { static void *handle; (void)data; return &handle; }
void __hipUnregisterFatBinary(void **modules) { (void)modules; }
void __hipRegisterFunction(void **modules, const void *host, char *device, const char *name, unsigned limit, void *tid, void *bid, void *block,
                           void *grid, int *wave)
{
    (void)modules, (void)device, (void)limit, (void)tid, (void)bid, (void)block, (void)grid, (void)wave;
    if (functions < 4096) fn_of[functions] = host, name_of[functions++] = name;
}
void __hipRegisterVar(void **modules, void *var, char *host, char *name, int ext, size_t size, int constant, int global)
{
    (void)modules, (void)var, (void)host, (void)name, (void)ext, (void)size, (void)constant, (void)global;
}

static struct { dim3_t grid, block; size_t lds; void *stream; } config;
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void *stream)
{
    config.grid = grid, config.block = block, config.lds = lds, config.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *lds, void **stream)
{
    *grid = config.grid, *block = config.block, *lds = config.lds, *stream = config.stream;
    return 0;
}
int hipLaunchKernel(const void *fn, dim3_t grid, dim3_t block, void **args, size_t lds, void *stream)
{
    (void)block, (void)args, (void)lds, (void)stream;
    const char *name = "?";
    for (int i = 0; i < functions; ++i)
        if (fn_of[i] == fn) name = name_of[i];
    const int refused = ++launches == fail_at;
    line(refused ? "refused" : "launch", name, grid);
    if (refused) last_error = 719; /* hipErrorLaunchFailure */
    return refused ? 719 : 0;
}
int hipGetLastError(void)
{
    const int e = last_error;
    last_error = 0;
    return e;
}
int hipEventRecord(void *event, void *stream)
{
    char handle[32];
    (void)stream;
    snprintf(handle, sizeof handle, "%zu", (size_t)event);
    line("event", handle, (dim3_t){0, 0, 0});
    return 0;
}
int hipGetDevice(int *device) { *device = 0; return 0; }
int hipDeviceGetAttribute(int *value, int attribute, int device) { (void)attribute, (void)device; *value = 256; return 0; }
int hipFuncSetAttribute(const void *fn, int attribute, int value) { (void)fn, (void)attribute, (void)value; return 0; }
int hipGetSymbolAddress(void **address, const void *symbol) { (void)symbol; *address = (void *)((size_t)99 << 40); return 0; }
