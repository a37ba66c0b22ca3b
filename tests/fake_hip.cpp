// A HIP runtime without a device, for host tests: allocations are host memory, copies
// and fills happen at once, and kernel launches are recorded by name, grid and LDS bytes
// instead of run.  Loaded with RTLD_GLOBAL before the library, its symbols are the ones
// that the library binds to.  A chosen launch or copy can be made to fail.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

extern "C" {
struct Dim3 {
    uint32_t x, y, z;
};
struct Launch {
    const char *name;
    Dim3 grid;
    size_t lds;
};
enum { kOk = 0, kInvalid = 1, kLaunchFailure = 719 };

static std::map<const void *, std::string> &names()
{
    static auto *m = new std::map<const void *, std::string>;
    return *m;
}
static std::vector<Launch> launches;
static std::map<void *, size_t> allocs;
static int fail_launch = -1, fail_copy = -1, last = kOk;
static struct {
    Dim3 grid, block;
    size_t lds;
    void *stream;
} config;

// controls
void fake_reset() { launches.clear(); }
void fake_fail_launch(int n) { fail_launch = n; }  // the n-th launch from now on (0: the next) fails
void fake_fail_copy(int n) { fail_copy = n; }
int fake_launches() { return (int)launches.size(); }
const char *fake_name(int i) { return launches[i].name; }
long long fake_blocks(int i) { return (long long)launches[i].grid.x * launches[i].grid.y * launches[i].grid.z; }
long long fake_lds(int i) { return (long long)launches[i].lds; }
uint64_t fake_memory_hash()  // of everything allocated
{
    uint64_t h = 1469598103934665603ull;
    for (auto &a : allocs)
        for (size_t i = 0; i < a.second; ++i) h = (h ^ static_cast<unsigned char *>(a.first)[i]) * 1099511628211ull;
    return h;
}

static int result(int e) { return last = e; }  // the status of the last call, also where it succeeded

void **__hipRegisterFatBinary(const void *) { return new void *; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *)
{
    names()[host] = name;
}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void *stream)
{
    config = {grid, block, lds, stream};
    return kOk;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *lds, void **stream)
{
    *grid = config.grid;
    *block = config.block;
    *lds = config.lds;
    *stream = config.stream;
    return kOk;
}
int hipLaunchKernel(const void *f, Dim3 grid, Dim3, void **, size_t lds, void *)
{
    if (fail_launch >= 0 && fail_launch-- == 0) return result(kLaunchFailure);
    launches.push_back({names()[f].c_str(), grid, lds});
    return result(kOk);
}
int hipGetLastError()
{
    const int e = last;
    last = kOk;
    return e;
}
const char *hipGetErrorString(int e) { return e ? "error of the fake runtime" : "no error"; }
int hipMalloc(void **p, size_t n)
{
    *p = calloc(n ? n : 1, 1);
    allocs[*p] = n;
    return result(*p ? kOk : 2);
}
int hipFree(void *p)
{
    allocs.erase(p);
    free(p);
    return result(kOk);
}
int hipMemcpy(void *d, const void *s, size_t n, int)
{
    if (fail_copy >= 0 && fail_copy-- == 0) return result(kInvalid);
    memcpy(d, s, n);
    return result(kOk);
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *) { return hipMemcpy(d, s, n, kind); }
int hipMemsetAsync(void *d, int v, size_t n, void *)
{
    memset(d, v, n);
    return result(kOk);
}
int hipGetSymbolAddress(void **p, const void *)
{
    static void *scratch = malloc(256 << 20);  // the library's static scratch
    *p = scratch;
    return result(kOk);
}
int hipGetDevice(int *d)
{
    *d = 0;
    return result(kOk);
}
int hipDeviceGetAttribute(int *v, int, int)
{
    *v = 256;  // compute units
    return result(kOk);
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t)
{
    *n = 2;
    return result(kOk);
}
int hipDeviceSynchronize() { return result(kOk); }
int hipStreamSynchronize(void *) { return result(kOk); }
int hipEventCreate(void **e)
{
    *e = &last;
    return result(kOk);
}
int hipEventDestroy(void *) { return result(kOk); }
int hipEventRecord(void *, void *) { return result(kOk); }
int hipEventElapsedTime(float *ms, void *, void *)
{
    *ms = 0.0f;
    return result(kOk);
}
}
