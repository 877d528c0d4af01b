/* Stands in for the HIP runtime's launch functions (preloaded by tests/test_routes_host.py): every kernel launch is
 * written down by name and nothing runs, so that the launch sequence of a call can be looked at without a GPU.  Built with
 * gcc as a shared object; the signatures are those of hip_runtime_api.h. */
#include <stdint.h>
#include <stdio.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;

static struct { const void* fn; const char* name; } table[8192];
static int ntable;
static char log_buf[1 << 22];
static size_t log_len;
static dim3_t cfg_grid, cfg_block;
static size_t cfg_shmem;
static void* cfg_stream;

void** __hipRegisterFatBinary(const void* data) { (void)data; static void* handle; return &handle; }
void __hipUnregisterFatBinary(void** modules) { (void)modules; }
void __hipRegisterVar(void** m, void* var, char* h, char* d, int ext, size_t size, int constant, int global)
{
    (void)m; (void)var; (void)h; (void)d; (void)ext; (void)size; (void)constant; (void)global;
}
void __hipRegisterFunction(void** m, const void* fn, char* device_fn, const char* name, unsigned limit, void* tid,
                           void* bid, dim3_t* block, dim3_t* grid, int* wsize)
{
    (void)m; (void)device_fn; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)wsize;
    if (ntable < 8192) { table[ntable].fn = fn; table[ntable].name = name; ++ntable; }
}
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t shmem, void* stream)
{
    cfg_grid = grid; cfg_block = block; cfg_shmem = shmem; cfg_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* shmem, void** stream)
{
    *grid = cfg_grid; *block = cfg_block; *shmem = cfg_shmem; *stream = cfg_stream;
    return 0;
}
int hipLaunchKernel(const void* fn, dim3_t grid, dim3_t block, void** args, size_t shmem, void* stream)
{
    (void)grid; (void)block; (void)args; (void)shmem; (void)stream;
    const char* name = "?";
    for (int i = 0; i < ntable; ++i)
        if (table[i].fn == fn) name = table[i].name;
    const size_t n = strlen(name);
    if (log_len + n + 2 < sizeof(log_buf)) {
        memcpy(log_buf + log_len, name, n);
        log_len += n;
        log_buf[log_len++] = '\n';
        log_buf[log_len] = 0;
    }
    return 0;
}
int hipFuncSetAttribute(const void* fn, int attr, int value) { (void)fn; (void)attr; (void)value; return 0; }
int hipGetLastError(void) { return 0; }

/* What was launched since the last call of this function, one kernel name a line. */
const char* recorded_launches(void)
{
    static char out[sizeof(log_buf)];
    memcpy(out, log_buf, log_len);
    out[log_len] = 0;
    log_len = 0;
    return out;
}

/* Every kernel that was registered, one name a line. */
const char* registered_kernels(void)
{
    static char out[1 << 20];
    size_t n = 0;
    for (int i = 0; i < ntable; ++i) {
        const size_t l = strlen(table[i].name);
        if (n + l + 2 >= sizeof(out)) break;
        memcpy(out + n, table[i].name, l);
        n += l;
        out[n++] = '\n';
    }
    out[n] = 0;
    return out;
}
