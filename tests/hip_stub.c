/* A HIP runtime that runs nothing and keeps a list: what libqg would launch, with which grid and arguments.
 * Loaded ahead of the library (tests/launches.py), so that launch plans can be looked at without a GPU.
 * A function keeps its limit of dynamic LDS per device, as the runtime's does: a launch
 * with more than 64 KB on a device where it was not asked for fails. */
#include <stddef.h>
#include <stdint.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
enum { MOST = 4096, ARGS = 4224, LDS_FREE = 64 << 10 };

static struct { const void *f; char name[256]; } known[1024];
static int n_known;
static struct { int kernel, device; dim3_t grid, block; size_t lds; unsigned char args[ARGS]; } launch[MOST];
static int n_launch;
static struct { const void *f; int device; int lds; } limit[1024];
static int n_limit, device, error;
static struct { dim3_t grid, block; size_t lds; void *stream; } call;

int stub_launches(void) { return n_launch; }
void stub_clear(void) { n_launch = 0; }
void stub_device(int d) { device = d; }
int stub_limits(void) { return n_limit; }
const char *stub_name(int i) { return known[launch[i].kernel].name; }
void stub_shape(int i, uint32_t *v)
{
    v[0] = launch[i].grid.x; v[1] = launch[i].grid.y; v[2] = launch[i].grid.z;
    v[3] = launch[i].block.x; v[4] = (uint32_t)launch[i].lds;
}
const void *stub_args(int i) { return launch[i].args; }

void **__hipRegisterFatBinary(const void *data) { static void *m; (void)data; return &m; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *v, char *a, char *b, int c, size_t d, int e, int f) { }
void __hipRegisterFunction(void **m, const void *f, char *df, const char *name, unsigned l, void *a, void *b, void *c, void *d, int *w)
{
    if (n_known == 1024) return;
    known[n_known].f = f;
    strncpy(known[n_known++].name, name, 255);
}
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void *st)
{
    call.grid = g; call.block = b; call.lds = lds; call.stream = st;
    return 0;
}
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *lds, void **st)
{
    *g = call.grid; *b = call.block; *lds = call.lds; *st = call.stream;
    return 0;
}
int hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **args, size_t lds, void *st)
{
    int k = 0, allowed = LDS_FREE;
    while (k < n_known && known[k].f != f) ++k;
    for (int i = 0; i < n_limit; ++i)
        if (limit[i].f == f && limit[i].device == device) allowed = limit[i].lds;
    if (k == n_known || n_launch == MOST || lds > (size_t)allowed) return error = 1;
    launch[n_launch].kernel = k; launch[n_launch].device = device;
    launch[n_launch].grid = g; launch[n_launch].block = b; launch[n_launch].lds = lds;
    /* the argument struct: QgCodesArgs, QgRowsI8Args, GemvArgs */
    if (strstr(known[k].name, "gemm_codes")) memcpy(launch[n_launch].args, args[0], 144);
    if (strstr(known[k].name, "gemm_rows_i8")) memcpy(launch[n_launch].args, args[0], 80);
    if (strstr(known[k].name, "gemv_")) memcpy(launch[n_launch].args, args[3], 4224);
    ++n_launch;
    return 0;
}
int hipFuncSetAttribute(const void *f, int attribute, int value)
{
    if (n_limit == 1024) return 1;
    limit[n_limit].f = f; limit[n_limit].device = device; limit[n_limit++].lds = value;
    return 0;
}
int hipGetLastError(void) { const int e = error; error = 0; return e; }
int hipGetDevice(int *d) { *d = device; return 0; }
int hipDeviceGetAttribute(int *v, int attribute, int d) { *v = 256; return 0; }      /* compute units: all that is asked for */
int hipFuncGetAttributes(void *a, const void *f) { memset(a, 0, 56); return 0; }     /* hipFuncAttributes */
int hipGetSymbolAddress(void **p, const void *s) { return 1; }
int hipEventCreate(void **e) { *e = &call; return 0; }
int hipEventDestroy(void *e) { return 0; }
int hipEventRecord(void *e, void *st) { return 0; }
int hipEventSynchronize(void *e) { return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { *ms = 1.0f; return 0; }
