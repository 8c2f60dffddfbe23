/* Preloaded into a process without a GPU: kernel launches are counted and do nothing, and launch number `fail_at` (from 0) fails
   the way the runtime reports it, by an error that hipGetLastError() returns once. */
#include <stddef.h>
#include <stdint.h>
typedef struct {
    uint32_t x, y, z;
} dim3_t;
static int launches, fail_at = -1, last_error;
static dim3_t grid, block;

void launch_stub_reset(int fail)
{
    launches = last_error = 0;
    fail_at = fail;
}
int launch_stub_count(void) { return launches; }

int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t shared, void *stream)
{
    (void)shared;
    (void)stream;
    grid = g;
    block = b;
    return 0;
}
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *shared, void **stream)
{
    *g = grid;
    *b = block;
    *shared = 0;
    *stream = 0;
    return 0;
}
int hipLaunchKernel(const void *kernel, dim3_t g, dim3_t b, void **args, size_t shared, void *stream)
{
    (void)kernel, (void)g, (void)b, (void)args, (void)shared, (void)stream;
    return launches++ == fail_at ? (last_error = 719) : 0;   /* hipErrorLaunchFailure */
}
int hipGetLastError(void)
{
    const int e = last_error;
    last_error = 0;
    return e;
}
