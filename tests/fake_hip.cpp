// A HIP runtime of host memory for the host code's own tests: device memory is calloc'd
// and never handed out again, kernels are noted and not run.  fake_fail_at(n) refuses the
// n-th hipMalloc from now.  A kernel of split tiles given partial sums that are not live
// is counted by fake_bad().
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

struct D3 { uint32_t x, y, z; };
static std::map<char *, size_t> live;
static std::map<const void *, std::string> names;
static std::map<std::string, void *> vars;
static std::map<const void *, std::string> var_of;
static long fail_in = -1, refused = 0, units = 0, bad = 0, mallocs = 0;
static D3 cfg_g, cfg_b;
static size_t cfg_s;
static void *cfg_st;

static bool is_live(void *p)
{
    auto it = live.upper_bound((char *)p);
    return it != live.begin() && (char *)p < (--it)->first + it->second;
}

extern "C" {
void fake_fail_at(long n) { fail_in = n; }
long fake_refused() { return refused; }
long fake_units() { return units; }
long fake_bad() { return bad; }
long fake_mallocs() { return mallocs; }

int hipMalloc(void **p, size_t n)
{
    ++mallocs;
    if (fail_in >= 0 && fail_in-- == 0) {
        ++refused;
        *p = nullptr;
        return 2;
    }
    *p = calloc(1, n + 16);
    live[(char *)*p] = n + 16;
    return 0;
}
int hipFree(void *p)
{
    live.erase((char *)p);   // the memory itself stays: its address is not used twice
    return 0;
}
int hipHostMalloc(void **p, size_t n, unsigned) { *p = calloc(1, n + 16); return 0; }
int hipHostFree(void *p) { free(p); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) { memcpy(d, s, n); return 0; }
int hipMemGetInfo(size_t *f, size_t *t) { *f = *t = (size_t)1 << 32; return 0; }
int hipGetDeviceCount(int *n) { *n = 1; return 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return "refused"; }
int hipStreamCreateWithFlags(void **s, unsigned) { *s = malloc(1); return 0; }
int hipStreamDestroy(void *s) { free(s); return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipEventCreate(void **e) { *e = malloc(1); return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { *e = malloc(1); return 0; }
int hipEventDestroy(void *e) { free(e); return 0; }
int hipEventElapsedTime(float *t, void *, void *) { *t = 0; return 0; }
int hipEventQuery(void *) { return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipStreamBeginCapture(void *, int) { return 1; }
int hipStreamEndCapture(void *, void **) { return 1; }
int hipGraphInstantiate(void **, void *, void *, char *, size_t) { return 1; }
int hipGraphLaunch(void *, void *) { return 1; }
int hipGraphDestroy(void *) { return 0; }
int hipGraphExecDestroy(void *) { return 0; }

void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *n, unsigned, void *, void *, void *, void *,
                           int *)
{
    names[f] = n;
}
void __hipRegisterVar(void **, void *v, char *, char *n, int, size_t size, int, int)
{
    var_of[v] = n;
    vars[n] = calloc(1, size + 16);
    live[(char *)vars[n]] = size + 16;
}
int hipGetSymbolAddress(void **p, const void *v)
{
    *p = vars[var_of[v]];
    return *p ? 0 : 1;
}
int __hipPushCallConfiguration(D3 g, D3 b, size_t s, void *st)
{
    cfg_g = g, cfg_b = b, cfg_s = s, cfg_st = st;
    return 0;
}
int __hipPopCallConfiguration(D3 *g, D3 *b, size_t *s, void **st)
{
    *g = cfg_g, *b = cfg_b, *s = cfg_s, *st = cfg_st;
    return 0;
}
int hipLaunchKernel(const void *f, D3, D3, void **args, size_t, void *)
{
    const std::string &n = names[f];
    if (n.find("k_sep_unit") != std::string::npos || n.find("k_sep_add") != std::string::npos) {
        ++units;
        void **parts = (void **)args[2];   // SepParts by value: units, part
        if (!is_live(parts[0]) || !is_live(parts[1])) ++bad;
    }
    return 0;
}
}
