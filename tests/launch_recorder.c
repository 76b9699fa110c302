/* Stands in for the parts of the HIP runtime that launching a kernel and enqueueing a mini-batch need, on a machine without a GPU:
 * nothing runs, and the argument of every split-K reduction, which says where its product's partial sums lie, is kept, as are name, grid,
 * stream and LDS of every launch and the tickets that a gather convolution is handed. */
#include <stddef.h>
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3;
typedef struct { const void *part; void *dw, *db; size_t total_w, total; int splits, blocks; } splitk_args;

enum { GROUP = 6, KERNELS = 1024, RECORDS = 4096, LAUNCHES = 65536, GATHER_TICKETS = 19 };

static struct { const void *host; const char *name; } kernels[KERNELS];
static int n_kernels;
static struct { dim3 grid, block; size_t lds; void *stream; } config;
static splitk_args records[RECORDS];
static struct { const char *name; dim3 grid; void *stream; const void *tickets; size_t lds; } launches[LAUNCHES];
static int n_records, n_launches;
static void *handle;

void **__hipRegisterFatBinary(const void *data) { (void)data; return &handle; }
void __hipUnregisterFatBinary(void **modules) { (void)modules; }
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g) { (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g; }
void __hipRegisterFunction(void **m, const void *host, char *device, const char *name, unsigned limit, void *t, void *b, dim3 *bd, dim3 *gd, int *w)
{
    (void)m; (void)device; (void)limit; (void)t; (void)b; (void)bd; (void)gd; (void)w;
    if (n_kernels < KERNELS) { kernels[n_kernels].host = host; kernels[n_kernels++].name = name; }
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream)
{
    config.grid = grid; config.block = block; config.lds = lds; config.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream)
{
    *grid = config.grid; *block = config.block; *lds = config.lds; *stream = config.stream;
    return 0;
}
int hipGetLastError(void) { return 0; }
int hipFuncSetAttribute(const void *f, int attr, int value) { (void)f; (void)attr; (void)value; return 0; }
int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, void *stream)
{
    (void)block;
    const int at = n_launches < LAUNCHES ? n_launches : LAUNCHES - 1;
    launches[at].name = "?";
    launches[at].grid = grid;
    launches[at].stream = stream;
    launches[at].tickets = NULL;
    launches[at].lds = lds;
    n_launches++;
    for (int k = 0; k < n_kernels; ++k) {
        if (kernels[k].host != f) continue;
        launches[at].name = kernels[k].name;
        if (strstr(kernels[k].name, "k_gather_mfma")) launches[at].tickets = *(const void **)args[GATHER_TICKETS];
        if (!strstr(kernels[k].name, "k_splitk_reduce")) continue;
        const splitk_args *a = args[0];                     /* one of them, or GROUP and how many they are */
        int n = 1;
        if (strstr(kernels[k].name, "Group")) memcpy(&n, a + GROUP, sizeof n);
        for (int i = 0; i < n && n_records < RECORDS; ++i) records[n_records++] = a[i];
    }
    return 0;
}

int hipGetDevice(int *device) { *device = 0; return 0; }
int hipDeviceGetAttribute(int *value, int attr, int device) { (void)attr; (void)device; *value = 256; return 0; }      /* compute units */
int hipGetSymbolAddress(void **address, const void *symbol) { (void)symbol; *address = (void *)((size_t)1 << 50); return 0; }
int hipStreamSynchronize(void *stream) { (void)stream; return 0; }
int hipStreamWaitEvent(void *stream, void *event, unsigned flags) { (void)stream; (void)event; (void)flags; return 0; }
int hipEventCreateWithFlags(void **event, unsigned flags) { (void)flags; *event = &handle; return 0; }
int hipEventRecord(void *event, void *stream) { (void)event; (void)stream; return 0; }
int hipEventDestroy(void *event) { (void)event; return 0; }
int hipMemcpyAsync(void *to, const void *from, size_t n, int kind, void *stream) { (void)to; (void)from; (void)n; (void)kind; (void)stream; return 0; }

/* operator new of the library */
static long n_news;
void *_Znwm(size_t n) { n_news++; return malloc(n ? n : 1); }
void _ZdlPvm(void *p, size_t n) { (void)n; free(p); }
long recorder_news(void) { return n_news; }

void recorder_clear(void) { n_records = n_launches = 0; }
int recorder_launches(void) { return n_launches; }
const char *recorder_launch(int i, unsigned *grid, size_t *stream, size_t *tickets, size_t *lds)
{
    *lds = launches[i].lds;
    *stream = (size_t)launches[i].stream; *tickets = (size_t)launches[i].tickets;
    grid[0] = launches[i].grid.x; grid[1] = launches[i].grid.y; grid[2] = launches[i].grid.z;
    return launches[i].name;
}
int recorder_count(void) { return n_records; }
void recorder_get(int i, size_t *first, size_t *bytes)
{
    *first = (size_t)records[i].part;
    *bytes = (size_t)records[i].splits * records[i].total * sizeof(float);
}
