/* The host side of the library without a GPU: this program defines the HIP functions that libnd.so calls
 * (its own definitions come before the HIP library's), so that a call of the C ABI checks its arguments,
 * plans, lays out its scratch and "launches" as it would, and nothing runs.  Device memory is reserved
 * address space that reads as zeros; what is copied to the host comes from there.
 *
 *   host_calls V E weighted free_bytes app num_roots [name=value ...]
 *
 * creates a graph of that shape on a device with free_bytes left (0: no limit), asks for the sizes of a
 * call, makes it through nd_sample_static, and prints what came back:
 *   create RC
 *   query RC WORKSPACE_BYTES STEPS
 *   static RC
 *   launch KERNEL GRID LDS (one line per launch, of the sampling call only; LDS: the dynamic bytes)
 *   device D               (current when the queries have returned)
 *   allocated BYTES        (live when the program ends, before the graph is destroyed)
 * Names: the fields of nd_params, fanout as a,b,c; queries=N (asks N times); fail_malloc=N (the first N
 * allocations of the queries fail); query_roots=N (sizes are asked for N roots; the call keeps its own); left=B (of the device's memory, B bytes are free when the first query
 * is made); device=D (current during the queries; the graph lies on device 0, and memory taken on another
 * is counted as elsewhere and ends the program with status 4); unused=B (asks for the statistics and the status of a workspace of bytes B that no call has used,
 * and prints "unused STATS_RC STATUS_RC"); empty=N (so many of the rows have no entries, as the kernel that checks the
 * offsets would have found); workspace=1 (the call is made through nd_sample with the scratch it asks for, and "call RC"
 * comes in the place of "static RC"); query_window=N (sizes are asked for with that sched_window; the call keeps its own).  A call that does not return within 20 seconds ends the program with SIGALRM. */
#define _GNU_SOURCE
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>
#include <unistd.h>

#include "../include/nd.h"

typedef struct { unsigned x, y, z; } dim3_t;
typedef struct { void* p; size_t n; } Block;

static Block blocks[256];
static int n_blocks, fail_malloc, trace, device, elsewhere;
static size_t live_bytes, free_limit;
static uint64_t empty_rows;
static struct { const void* f; const char* name; } kernels[1024];
static int n_kernels;

static void* reserve(size_t n) {
    void* p = mmap(NULL, n ? n : 1, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    return p == MAP_FAILED ? NULL : p;
}
int hipMalloc(void** p, size_t n) {
    *p = NULL;
    if (fail_malloc > 0) { --fail_malloc; return 2; }
    if (free_limit && live_bytes + n > free_limit) return 2;
    if (!(*p = reserve(n))) return 2;
    blocks[n_blocks].p = *p;
    blocks[n_blocks++].n = n;
    live_bytes += n;
    elsewhere |= device != 0;
    return 0;
}
int hipFree(void* p) {
    for (int i = 0; p && i < n_blocks; ++i)
        if (blocks[i].p == p) {
            munmap(p, blocks[i].n ? blocks[i].n : 1);
            live_bytes -= blocks[i].n;
            blocks[i] = blocks[--n_blocks];
        }
    return 0;
}
int hipMemGetInfo(size_t* avail, size_t* total) {
    *total = free_limit ? free_limit : (size_t)1 << 40;
    *avail = *total - live_bytes;
    return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* stream) {
    (void)stream;
    if (kind == 2) memcpy(d, s, n);
    if (kind == 2 && n == 24) ((uint64_t*)d)[2] = empty_rows;  /* flags, the longest row, the empty rows */
    return 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void* s) { (void)d; (void)v; (void)n; (void)s; return 0; }
int hipGetDevice(int* d) { *d = device; return 0; }
int hipSetDevice(int d) { device = d; return 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) { (void)f; (void)a; (void)v; return 0; }
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) { (void)e; return "error"; }
int hipGetSymbolAddress(void** p, const void* sym) { (void)sym; *p = reserve(ND_STATIC_SCRATCH_BYTES); return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = (void*)16; return 0; }
int hipStreamDestroy(void* s) { (void)s; return 0; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipThreadExchangeStreamCaptureMode(int* m) { (void)m; return 0; }
void** __hipRegisterFatBinary(const void* d) { (void)d; static void* m; return &m; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void) {}
void __hipRegisterFunction(void** m, const void* f, char* df, const char* name, unsigned tl, void* a, void* b, void* c,
                           void* d, int* w) {
    (void)m; (void)df; (void)tl; (void)a; (void)b; (void)c; (void)d; (void)w;
    kernels[n_kernels].f = f;
    kernels[n_kernels++].name = name;
}
static dim3_t c_grid, c_block;
static size_t c_lds;
static void* c_stream;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void* s) {
    c_grid = g; c_block = b; c_lds = lds; c_stream = s;
    return 0;
}
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* lds, void** s) {
    *g = c_grid; *b = c_block; *lds = c_lds; *s = c_stream;
    return 0;
}
int hipLaunchKernel(const void* f, dim3_t g, dim3_t b, void** args, size_t lds, void* s) {
    (void)b; (void)args; (void)s;
    for (int i = 0; trace && i < n_kernels; ++i)
        if (kernels[i].f == f) printf("launch %s %u %zu\n", kernels[i].name, g.x, lds);
    return 0;
}

int main(int argc, char** argv) {
    if (argc < 7) return 2;
    alarm(20);
    setvbuf(stdout, NULL, _IOLBF, 0);
    const long long V = atoll(argv[1]), E = atoll(argv[2]), roots = atoll(argv[6]);
    const int weighted = atoi(argv[3]), app = atoi(argv[5]);
    free_limit = (size_t)atoll(argv[4]);
    nd_params p;
    nd_params_init(&p);
    int fail = 0, unused = -1, queries = 1, query_device = 0, workspace = 0, query_window = 0, own_window = 1;
    long long left = -1, query_roots = roots;
    for (int i = 7; i < argc; ++i) {
        char* eq = strchr(argv[i], '=');
        if (!eq) return 2;
        *eq = 0;
        const char* v = eq + 1;
        const char* n = argv[i];
        if (!strcmp(n, "fanout")) {
            p.num_steps = 0;
            for (const char* c = v; c; c = strchr(c, ',') ? strchr(c, ',') + 1 : NULL) p.fanout[p.num_steps++] = atoi(c);
        } else if (!strcmp(n, "num_steps")) p.num_steps = atoi(v);
        else if (!strcmp(n, "unique_rounds")) p.unique_rounds = atoi(v);
        else if (!strcmp(n, "roots_per_sample")) p.roots_per_sample = atoi(v);
        else if (!strcmp(n, "sched_window")) p.sched_window = atoi(v);
        else if (!strcmp(n, "mode")) p.mode = atoi(v);
        else if (!strcmp(n, "use_weights")) p.use_weights = atoi(v);
        else if (!strcmp(n, "unused")) unused = atoi(v);
        else if (!strcmp(n, "fail_malloc")) fail = atoi(v);
        else if (!strcmp(n, "queries")) queries = atoi(v);
        else if (!strcmp(n, "query_roots")) query_roots = atoll(v);
        else if (!strcmp(n, "left")) left = atoll(v);
        else if (!strcmp(n, "empty")) empty_rows = (uint64_t)atoll(v);
        else if (!strcmp(n, "query_window")) { query_window = atoi(v); own_window = 0; }
        else if (!strcmp(n, "workspace")) workspace = atoi(v);
        else if (!strcmp(n, "device")) query_device = atoi(v);
        else return 2;
    }
    nd_graph* g = NULL;
    void* any = reserve(4096);  /* copied from in name only */
    int rc = nd_graph_create(&g, V, E, any, 1, any, weighted ? any : NULL, 1, NULL);
    printf("create %d\n", rc);
    if (rc != 0) return 0;
    int32_t steps = 0;
    static int64_t lens[ND_MAX_WALK_STEPS];
    size_t ws = 0;
    fail_malloc = fail;
    if (left >= 0) free_limit = live_bytes + (size_t)left;
    device = query_device;
    nd_params asked = p;
    if (!own_window) asked.sched_window = query_window;
    for (int i = 0; i < queries; ++i) rc = nd_sample_query(g, app, &asked, query_roots, &steps, lens, &ws);
    fail_malloc = 0;
    printf("query %d %zu %d\n", rc, ws, steps);
    printf("device %d\n", device);
    device = 0;
    static int32_t* out[ND_MAX_WALK_STEPS];
    for (int i = 0; i < ND_MAX_WALK_STEPS; ++i) out[i] = any;
    trace = 1;
    if (workspace) printf("call %d\n", nd_sample(g, app, &p, any, roots, 1, out, reserve(ws), ws, NULL));
    else printf("static %d\n", nd_sample_static(g, app, &p, any, roots, 1, out, any, NULL));
    trace = 0;
    if (unused >= 0) {
        const size_t n = 1 << 20;
        char* bytes = reserve(n);
        int64_t stats[4 * 8];
        memset(bytes, unused, n);
        const int stats_rc = nd_sample_stats(bytes, NULL, 4, stats);
        printf("unused %d %d\n", stats_rc, nd_sample_status(bytes, NULL));
    }
    printf("allocated %zu\n", live_bytes);
    nd_graph_destroy(g);
    return live_bytes != 0 ? 3 : elsewhere ? 4 : 0;
}
