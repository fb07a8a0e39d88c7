/* The HIP entry points that liblq.so imports, for tests of its host code without a device: nothing runs, launches are
   recorded by kernel name, and a launch or a function-attribute request can be made to fail.  Loaded with RTLD_GLOBAL before the
   library, so that its references bind here. */
#include <stddef.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_;
enum { MAX_KERNELS = 8192, MAX_LAUNCHES = 256 };
static struct { const void* host; const char* name; } kernels[MAX_KERNELS];
static int n_kernels, n_launches, n_attrs, fail_launch = -1, fail_attrs, last_error, device;
static const char* launched[MAX_LAUNCHES];
static double threads[MAX_LAUNCHES];
static struct { dim3_ grid, block; size_t lds; void* stream; } call;

void fake_reset(int failing_launch, int failing_attrs, int dev)
{
    n_launches = n_attrs = last_error = 0;
    fail_launch = failing_launch;
    fail_attrs = failing_attrs;
    device = dev;
}
int fake_launches(void) { return n_launches; }
int fake_attrs(void) { return n_attrs; }
const char* fake_launched(int i) { return launched[i]; }
double fake_threads(int i) { return threads[i]; }

void** __hipRegisterFatBinary(const void* data) { static void* handle; (void)data; return &handle; }
void __hipUnregisterFatBinary(void** modules) { (void)modules; }
void __hipRegisterFunction(void** modules, const void* host, char* device_name, const char* name, unsigned limit, void* tid, void* bid,
                           dim3_* block, dim3_* grid, int* wsize)
{
    (void)modules; (void)device_name; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)wsize;
    if (n_kernels < MAX_KERNELS) { kernels[n_kernels].host = host; kernels[n_kernels++].name = name; }
}
void __hipRegisterVar(void** modules, void* var, char* host_name, char* device_name, int ext, size_t size, int constant, int global)
{
    (void)modules; (void)var; (void)host_name; (void)device_name; (void)ext; (void)size; (void)constant; (void)global;
}
int __hipPushCallConfiguration(dim3_ grid, dim3_ block, size_t lds, void* stream)
{
    call.grid = grid; call.block = block; call.lds = lds; call.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3_* grid, dim3_* block, size_t* lds, void** stream)
{
    *grid = call.grid; *block = call.block; *lds = call.lds; *stream = call.stream;
    return 0;
}
int hipLaunchKernel(const void* f, dim3_ grid, dim3_ block, void** args, size_t lds, void* stream)
{
    (void)args; (void)lds; (void)stream;
    const char* name = "?";
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].host == f) name = kernels[i].name;
    if (n_launches < MAX_LAUNCHES) {
        launched[n_launches] = name;
        threads[n_launches] = (double)grid.x * grid.y * grid.z * block.x * block.y * block.z;
    }
    if (n_launches++ == fail_launch) return last_error = 719;
    return 0;
}
int hipFuncSetAttribute(const void* f, int attr, int value)
{
    (void)f; (void)attr; (void)value;
    ++n_attrs;
    if (fail_attrs > 0) { --fail_attrs; return last_error = 1; }
    return 0;
}
int hipGetLastError(void) { const int e = last_error; last_error = 0; return e; }
int hipGetDevice(int* dev) { *dev = device; return 0; }
int hipDeviceGetAttribute(int* value, int attr, int dev) { (void)attr; (void)dev; *value = 256; return 0; }
int hipGetSymbolAddress(void** p, const void* symbol) { (void)symbol; *p = (void*)256; return 0; }
int hipMemcpyAsync(void* dst, const void* src, size_t n, int kind, void* stream) { (void)dst; (void)src; (void)n; (void)kind; (void)stream; return 0; }
int hipStreamSynchronize(void* stream) { (void)stream; return 0; }
