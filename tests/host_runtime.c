/* The library's host side on a runtime of plain memory: this program defines the HIP calls that the
 * library imports, so allocations are counted (and refused beyond a limit) and kernel launches only
 * noted.  Arguments:
 *   DECISION BLCFA BPC CHUNK LIMIT FORM ACTION...
 * BPC 0: no launch shape is set.  LIMIT: bytes of device memory there are beyond what sfq_create
 * takes (0: no limit).  FORM: the tiles' field mode.  Actions, in order:
 *   reserve:N:T       sfq_reserve
 *   step:NxK,NxK,...  sfq_step of K tiles of N electrons, ...; noalloc: and plan: the same
 *   limit:B           another limit
 *   auto:             sfq_auto_launch
 * Each action prints its status, the handle's queue bytes, the most device memory in use beyond
 * sfq_create's so far in the action, and the blocks of the last streaming kernel. */
#include <hip/hip_runtime_api.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "sfq.h"

static size_t used, peak, limit, base;
static hipError_t last;
static unsigned grid_seen;
static struct { void* p; size_t n; } blocks[256];
static struct { const void* f; char name[96]; } fns[512];
static int nfns;

static hipError_t ret(hipError_t e)
{
    if (e != hipSuccess) last = e;
    return e;
}

hipError_t hipMalloc(void** p, size_t n)
{
    if (limit && used - base + n > limit) { *p = NULL; return ret(hipErrorOutOfMemory); }
    for (int k = 0; k < 256; ++k)
        if (!blocks[k].p) {
            *p = blocks[k].p = malloc(n);
            blocks[k].n = n;
            used += n;
            if (used > peak) peak = used;
            return hipSuccess;
        }
    return ret(hipErrorOutOfMemory);
}
hipError_t hipFree(void* p)
{
    for (int k = 0; p && k < 256; ++k)
        if (blocks[k].p == p) { used -= blocks[k].n; blocks[k].p = NULL; free(p); }
    return hipSuccess;
}
/* the last error stays until it is read */
hipError_t hipGetLastError(void) { const hipError_t e = last; last = hipSuccess; return e; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned f) { (void)f; *p = malloc(n); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned f) { (void)f; *d = h; return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k) { (void)k; memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void* d, int v, size_t n) { memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t s) { (void)d; (void)v; (void)n; (void)s; return hipSuccess; }
hipError_t hipSetDevice(int d) { (void)d; return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int d) { (void)d; memset(p, 0, sizeof *p); p->multiProcessorCount = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = (void*)0x10000; return hipSuccess; }
const char* hipGetErrorString(hipError_t e) { (void)e; return "error"; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned f) { (void)f; *e = (hipEvent_t)0x10; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { (void)e; (void)s; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) { (void)a; (void)b; *ms = 0; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned f) { (void)f; *s = (hipStream_t)0x20; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { (void)s; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned f) { (void)s; (void)e; (void)f; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* c) { (void)s; *c = hipStreamCaptureStatusNone; return hipSuccess; }

/* kernel registration and launches */
void** __hipRegisterFatBinary(const void* d) { (void)d; return (void**)0x30; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterVar(void** m, void* v, char* h, char* n, int e, size_t s, int c, int g)
{
    (void)m; (void)v; (void)h; (void)n; (void)e; (void)s; (void)c; (void)g;
}
void __hipRegisterFunction(void** m, const void* f, char* d, const char* name, unsigned t, void* a,
                           void* b, void* c, void* e, int* w)
{
    (void)m; (void)d; (void)t; (void)a; (void)b; (void)c; (void)e; (void)w;
    if (nfns < 512) {
        fns[nfns].f = f;
        snprintf(fns[nfns++].name, sizeof fns[0].name, "%s", name);
    }
}
static dim3 cfg_grid, cfg_block;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t st)
{
    (void)s; (void)st;
    cfg_grid = g;
    cfg_block = b;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st)
{
    *g = cfg_grid;
    *b = cfg_block;
    *s = 0;
    *st = NULL;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t s, hipStream_t st)
{
    (void)b; (void)args; (void)s; (void)st;
    for (int k = 0; k < nfns; ++k)
        if (fns[k].f == f && strstr(fns[k].name, "bulk_kernel")) grid_seen = g.x;
    return hipSuccess;
}

static sfq_tile tiles[SFQ_MAX_TILES];

static int fill(const char* spec, int form)
{
    static char some[256];  /* an address the host never reads, on a 256-byte boundary */
    double* a = (double*)(((size_t)some + 127) & ~(size_t)127);
    int nt = 0;
    for (const char* s = spec; s && *s;) {
        unsigned long long n;
        int k;
        if (sscanf(s, "%llux%d", &n, &k) != 2) exit(2);
        while (k-- > 0 && nt < SFQ_MAX_TILES) {
            sfq_tile* t = &tiles[nt++];
            memset(t, 0, sizeof *t);
            t->species = SFQ_ELECTRON;
            t->n = n;
            t->field_mode = form;
            t->px = a + nt % 16;  /* every start within a 128-byte line */
            t->py = t->pz = t->tau = t->fperp = t->dfperp = a;
            t->ex = t->ey = t->ez = t->bx = t->by = t->bz = t->px_prev = t->py_prev = t->pz_prev = a;
            t->wave_amp = t->wave_phase = a;
            t->wave_k[0] = t->wave_pol[1] = 1.0;
            t->uid = (const uint64_t*)a;
            t->just_created = (uint8_t*)a;
        }
        s = strchr(s, ',');
        if (s) ++s;
    }
    return nt;
}

int main(int argc, char** argv)
{
    if (argc < 8) return 2;
    sfq_config cfg;
    memset(&cfg, 0, sizeof cfg);
    cfg.ref_length = 1.2732395447351628e-07;
    cfg.dt = 0.02;
    cfg.decision = atoi(argv[1]);
    cfg.blcfa = atoi(argv[2]);
    const int bpc = atoi(argv[3]), form = atoi(argv[6]);
    sfq_handle h = NULL;
    if (sfq_create(&cfg, &h) != SFQ_OK) { printf("%s\n", sfq_last_error(NULL)); return 3; }
    if (bpc && sfq_set_launch(h, bpc, atoi(argv[4])) != SFQ_OK) return 4;
    base = used;
    limit = strtoull(argv[5], NULL, 10);
    static double made[8];
    static unsigned long long counts[3];
    static sfq_counters counters;
    for (int k = 7; k < argc; ++k) {
        const char* arg = strchr(argv[k], ':') + 1;
        int st = -1;
        peak = used;
        if (!strncmp(argv[k], "limit", 5)) {
            limit = strtoull(arg, NULL, 10);
            continue;
        } else if (!strncmp(argv[k], "auto", 4)) {
            st = sfq_auto_launch(h);
        } else if (!strncmp(argv[k], "reserve", 7)) {
            unsigned long long n;
            int t;
            if (sscanf(arg, "%llu:%d", &n, &t) != 2) return 2;
            st = sfq_reserve(h, n, t);
        } else {
            const sfq_products p = {made, made, made, made, (uint64_t*)made, (uint64_t*)made, 8};
            sfq_step_desc d;
            memset(&d, 0, sizeof d);
            d.ntiles = fill(arg, form);
            d.tiles = tiles;
            d.photons = d.electrons = d.positrons = p;
            d.product_counts = counts;
            d.counters = &counters;
            d.push = 1;
            grid_seen = 0;
            if (!strncmp(argv[k], "step", 4)) st = sfq_step(h, &d, NULL);
            else if (!strncmp(argv[k], "noalloc", 7)) st = sfq_step_noalloc(h, &d, NULL);
            else {
                sfq_plan p2 = NULL;
                st = sfq_plan_create(h, &d, 1, &p2);
                if (st == SFQ_OK) st = sfq_plan_launch(p2, NULL);
                if (p2) sfq_plan_destroy(p2);
            }
        }
        uint64_t q = 0;
        sfq_queue_bytes(h, &q);
        printf("%d %llu %zu %u\n", st, (unsigned long long)q, peak - base, grid_seen);
    }
    sfq_destroy(h);
    return 0;
}
