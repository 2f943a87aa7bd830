/* Stand-ins for the HIP runtime calls that librealb.so makes, for CPU tests of its host side: every call succeeds at once and
 * the ordering-relevant ones (launches, event records, event waits) are written down, one per line, in calls_log().  No kernel
 * runs.  Loaded with RTLD_GLOBAL ahead of the library, so that its undefined symbols resolve here. */
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
enum { kNotReady = 600 };

static char* log_text;
static size_t log_len, log_cap;
static intptr_t next_handle = 0x1000;
static int last_error, capturing, events_done;
static char failing[128];

static void record(const char* line) {
    const size_t n = strlen(line);
    if (log_len + n + 2 > log_cap) {
        log_cap = 2 * (log_len + n + 2);
        log_text = realloc(log_text, log_cap);
    }
    memcpy(log_text + log_len, line, n);
    log_text[log_len + n] = '\n';
    log_text[log_len += n + 1] = 0;
}
const char* calls_log(void) { return log_text ? log_text : ""; }
void calls_clear(void) { log_len = 0; if (log_text) log_text[0] = 0; }
void calls_set_capturing(int on) { capturing = on; }
void calls_set_events_done(int on) { events_done = on; }
/* launches of kernels whose name holds this text fail ("": none) */
void calls_fail(const char* kernel) { snprintf(failing, sizeof failing, "%s", kernel); }

/* kernels: the host-side handle and the device name it was registered under */
static struct { const void* host; const char* name; }* kernels;
static size_t n_kernels, cap_kernels;
void** __hipRegisterFatBinary(const void* data) { static void* module; (void)data; return &module; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void** m, void* a, char* b, char* c, int d, size_t e, int f, int g) { (void)m; (void)a; (void)b; (void)c; (void)d; (void)e; (void)f; (void)g; }
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned limit, void* t, void* b, void* bd, void* gd, int* ws) {
    (void)m; (void)dev; (void)limit; (void)t; (void)b; (void)bd; (void)gd; (void)ws;
    if (n_kernels == cap_kernels) kernels = realloc(kernels, (cap_kernels = 2 * cap_kernels + 64) * sizeof *kernels);
    kernels[n_kernels].host = host;
    kernels[n_kernels++].name = strdup(name);
}

static dim3_t cfg_grid, cfg_block;
static size_t cfg_lds;
static void* cfg_stream;
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void* stream) { cfg_grid = grid; cfg_block = block; cfg_lds = lds; cfg_stream = stream; return 0; }
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* lds, void** stream) { *grid = cfg_grid; *block = cfg_block; *lds = cfg_lds; *stream = cfg_stream; return 0; }
int hipLaunchKernel(const void* f, dim3_t grid, dim3_t block, void** args, size_t lds, void* stream) {
    const char* name = "?";
    char line[512];
    (void)lds;
    for (size_t i = 0; i < n_kernels; ++i) if (kernels[i].host == f) name = kernels[i].name;
    int n = snprintf(line, sizeof line, "launch %s grid %u block %u stream %p", name, grid.x, block.x, stream);
    if (strstr(name, "ffn_") && n < (int)sizeof line) {      /* a GEMM: its parameters begin with the six operands */
        void* const* o = (void* const*)args[0];
        snprintf(line + n, sizeof line - n, " operands %p %p %p %p %p %p", o[0], o[1], o[2], o[3], o[4], o[5]);
    }
    record(line);
    /* the runtime's limit: fewer than 2^32 threads in a grid */
    if ((uint64_t)grid.x * block.x >= (1ull << 32) || (failing[0] && strstr(name, failing))) last_error = 9;
    return last_error;
}

int hipEventRecord(void* e, void* s) { char l[96]; snprintf(l, sizeof l, "record event %p stream %p", e, s); record(l); return 0; }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { char l[96]; (void)f; snprintf(l, sizeof l, "wait event %p stream %p", e, s); record(l); return 0; }
int hipStreamIsCapturing(void* s, int* status) { (void)s; *status = capturing; return 0; }
int hipEventQuery(void* e) { (void)e; return events_done ? 0 : kNotReady; }
int hipStreamQuery(void* s) { (void)s; return 0; }
int hipEventSynchronize(void* e) { (void)e; return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 0; return 0; }
int hipEventCreate(void** e) { *e = (void*)next_handle++; return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { (void)f; return hipEventCreate(e); }
int hipEventDestroy(void* e) { (void)e; return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = (void*)next_handle++; return 0; }
int hipStreamDestroy(void* s) { (void)s; return 0; }
int hipMalloc(void** p, size_t n) { *p = calloc(1, n ? n : 1); return *p ? 0 : 2; }
int hipFree(void* p) { free(p); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned f) { (void)f; return hipMalloc(p, n); }
int hipHostFree(void* p) { free(p); return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = (void*)next_handle++; return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) { (void)f; (void)a; (void)v; return 0; }
int hipGetLastError(void) { const int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int e) { return e == 9 ? "invalid configuration" : "error"; }
