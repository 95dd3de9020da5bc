/* The HIP runtime calls of libsqn.so's host code, without a GPU: memory is
 * address ranges that nothing reads, a launch is noted by its kernel's name and
 * grid, and a launch takes the time the test set for it.  Loaded with its
 * symbols global ahead of the runtime, in a process of its own
 * (tests/fake_hip.py). */
#include <stdint.h>
#include <stdio.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
enum { OK = 0, INVALID_VALUE = 1, OUT_OF_MEMORY = 2, INVALID_CONFIGURATION = 9 };

static int last_error;
static int fail(int e) { return last_error = e; }
int hipGetLastError(void) { const int e = last_error; last_error = OK; return e; }
int hipGetDevice(int* d) { *d = 0; return OK; }
const char* hipGetErrorString(int e) { return e == OUT_OF_MEMORY ? "out of memory" : "error"; }

/* memory: ranges handed out in order, at most `limit` bytes at a time */
#define MAX_RANGES 4096
static struct { uintptr_t base; size_t size; } ranges[MAX_RANGES];
static int n_ranges;
static size_t used, limit = SIZE_MAX;
static uintptr_t next_base = (uintptr_t)1 << 44;
void fake_limit(size_t bytes) { limit = bytes; }
size_t fake_used(void) { return used; }

int hipMalloc(void** p, size_t size)
{
    if (n_ranges == MAX_RANGES || size > limit || used > limit - size)
        return fail(OUT_OF_MEMORY);
    ranges[n_ranges].base = next_base;
    ranges[n_ranges++].size = size;
    *p = (void*)next_base;
    next_base += (size + 8191) & ~(size_t)4095;
    used += size;
    return OK;
}

int hipFree(void* p)
{
    for (int k = 0; k < n_ranges; ++k)
        if (ranges[k].base == (uintptr_t)p) {
            used -= ranges[k].size;
            ranges[k] = ranges[--n_ranges];
            return OK;
        }
    return fail(INVALID_VALUE);
}

int hipMemGetAddressRange(void** base, size_t* size, void* p)
{
    for (int k = 0; k < n_ranges; ++k)
        if ((uintptr_t)p - ranges[k].base < ranges[k].size) {
            *base = (void*)ranges[k].base;
            *size = ranges[k].size;
            return OK;
        }
    return fail(INVALID_VALUE);
}

/* what was copied from the host: the last one's bytes */
static size_t copied;
static unsigned char copy[1 << 20];
size_t fake_copied(unsigned char* out) { memcpy(out, copy, sizeof(copy)); return copied; }
int hipMemcpyAsync(void* dst, const void* src, size_t n, int kind, void* stream)
{
    (void)dst, (void)stream;
    if (kind == 1) {
        copied = n;
        memcpy(copy, src, n < sizeof(copy) ? n : sizeof(copy));
    }
    return OK;
}
int hipStreamSynchronize(void* s) { (void)s; return OK; }

/* kernels by their host handles */
#define MAX_KERNELS 1024
static struct { const void* host; const char* name; } kernels[MAX_KERNELS];
static int n_kernels;
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned limit_, void* a, void* b,
                           dim3* c, dim3* d, int* e)
{
    if (strstr(name, "sqn") && n_kernels < MAX_KERNELS) {
        kernels[n_kernels].host = host;
        kernels[n_kernels++].name = name;
    }
    (void)m, (void)dev, (void)limit_, (void)a, (void)b, (void)c, (void)d, (void)e;
}

static dim3 grid_, block_;
static size_t shared_;
static void* stream_;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t n, void* s)
{
    grid_ = g, block_ = b, shared_ = n, stream_ = s;
    return OK;
}
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* n, void** s)
{
    *g = grid_, *b = block_, *n = shared_, *s = stream_;
    return OK;
}

/* launches: the log, and the clock they advance */
static char log_[1 << 22];
static size_t log_len;
static struct { char part[64]; double ms; } costs[64];
static int n_costs;
static double now;
const char* fake_log(void) { return log_; }
void fake_reset(void) { log_len = 0; log_[0] = 0; n_costs = 0; }
void fake_cost(const char* part, double ms)
{
    snprintf(costs[n_costs].part, sizeof(costs[0].part), "%s", part);
    costs[n_costs++].ms = ms;
}

int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t n, void* s)
{
    (void)n, (void)s;
    const char* name = "?";
    for (int k = 0; k < n_kernels; ++k)
        if (kernels[k].host == f)
            name = kernels[k].name;
    /* the runtime's bounds: at least one workgroup, fewer than 2^32 work items
     * per dimension */
    if (!g.x || !g.y || !g.z || b.x * b.y * b.z > 1024 || (uint64_t)g.x * b.x >> 32 || (uint64_t)g.y * b.y >> 32
        || (uint64_t)g.z * b.z >> 32)
        return fail(INVALID_CONFIGURATION);
    if (log_len < sizeof(log_) - 512)
        log_len += (size_t)snprintf(log_ + log_len, 512, "%s %u %u %u %u\n", name, g.x, g.y, g.z, b.x);
    if (strstr(name, "row_distance") && log_len < sizeof(log_) - 512)
        /* its scratch: (live, f, f_min, n_p, pitch) */
        log_len += (size_t)snprintf(log_ + log_len, 512, "scratch %llu %llu %d %d\n",
                                    (unsigned long long)*(uintptr_t*)args[1],
                                    (unsigned long long)*(uintptr_t*)args[2], *(int*)args[3], *(int*)args[4]);
    for (int k = 0; k < n_costs; ++k)
        if (strstr(name, costs[k].part)) {
            now += costs[k].ms;
            break;
        }
    return OK;
}

static double events[64];
static int n_events;
int hipEventCreate(void** e) { *e = &events[n_events++ % 64]; return OK; }
int hipEventDestroy(void* e) { (void)e; return OK; }
int hipEventRecord(void* e, void* s) { (void)s; *(double*)e = now; return OK; }
int hipEventSynchronize(void* e) { (void)e; return OK; }
int hipEventElapsedTime(float* ms, void* a, void* b) { *ms = (float)(*(double*)b - *(double*)a); return OK; }
