/* A stand-in for the launch calls of the HIP runtime, for tests of the library's host side on machines without a GPU: it
 * records every kernel launch (its function, grid, dynamic LDS and the first bytes of its first argument) and fails the launches it is
 * told to.  Loaded (RTLD_GLOBAL) before the library, so that these definitions come first. */
#include <stdint.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef struct { uint64_t func; uint32_t grid[3], block[3]; uint64_t head[2]; int failed; uint64_t shared; } launch_t;

enum { kMost = 4096, kOk = 0, kLaunchFailure = 719 };
static launch_t launches[kMost];
static int n_launches, fail_at = -1, last_error;
static dim3_t grid_, block_;
static size_t shared_;
static void* stream_;

int recorded(void) { return n_launches; }
const launch_t* launch_at(int i) { return &launches[i]; }
void fail_launch(int i) { fail_at = i; }             /* counted over all launches; -1: none */
void leave_error(int e) { last_error = e; }          /* as an earlier call's failure that nobody has asked for */

int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t shared, void* stream) {
    grid_ = grid; block_ = block; shared_ = shared; stream_ = stream;
    return kOk;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* shared, void** stream) {
    *grid = grid_; *block = block_; *shared = shared_; *stream = stream_;
    return kOk;
}
int hipLaunchKernel(const void* func, dim3_t grid, dim3_t block, void** args, size_t shared, void* stream) {
    (void)stream;
    launch_t l = {(uint64_t)(uintptr_t)func, {grid.x, grid.y, grid.z}, {block.x, block.y, block.z}, {0, 0}, n_launches == fail_at, shared};
    memcpy(l.head, args[0], sizeof l.head);
    if (n_launches < kMost) launches[n_launches] = l;
    ++n_launches;
    if (l.failed) last_error = kLaunchFailure;
    return l.failed ? kLaunchFailure : kOk;
}
int hipGetLastError(void) { const int e = last_error; last_error = kOk; return e; }
int hipGetDevice(int* d) { *d = 0; return kOk; }
int hipDeviceGetAttribute(int* v, int attr, int dev) { (void)attr; (void)dev; *v = 256; return kOk; }
int hipFuncSetAttribute(const void* f, int attr, int v) { (void)f; (void)attr; (void)v; return kOk; }
