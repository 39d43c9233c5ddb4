// A HIP runtime for host tests of the library's launches: memory is host memory, a
// launch is recorded and not run, and device, launch errors and the dynamic LDS a
// kernel may use are the test's to set and see.  Linked into the test's program,
// whose symbols the library binds to before the real runtime's.
#pragma once
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <utility>
#include <vector>

namespace fake {

struct Dim {
    uint32_t x, y, z;
};
struct Launch {
    std::string name;
    int device;
    size_t lds;
    void **args;
};

int device = 0;
// (the library registers its kernels before this file's variables are made)
inline std::map<const void *, std::string> &kernels() {
    static auto *m = new std::map<const void *, std::string>;
    return *m;
}
std::map<std::pair<int, std::string>, size_t> lds_limit;  // (device, kernel)
std::vector<Launch> launches;
int refused = 0;                              // launches above the kernel's limit on the device
bool (*fail_launch)(const std::string &) = nullptr;  // which launches return an error
void (*on_launch)(const Launch &) = nullptr;
int last_error = 0;

struct Config {
    Dim grid, block;
    size_t lds;
    void *stream;
};
std::vector<Config> pushed;

inline int set(int e) {
    if (e) last_error = e;
    return e;
}

}  // namespace fake

#define HIP_FAKE extern "C" __attribute__((visibility("default"), used)) int

HIP_FAKE __hipPushCallConfiguration(fake::Dim g, fake::Dim b, size_t lds, void *s) {
    fake::pushed.push_back({g, b, lds, s});
    return 0;
}
HIP_FAKE __hipPopCallConfiguration(fake::Dim *g, fake::Dim *b, size_t *lds, void **s) {
    const fake::Config c = fake::pushed.back();
    fake::pushed.pop_back();
    *g = c.grid;
    *b = c.block;
    *lds = c.lds;
    *s = c.stream;
    return 0;
}
extern "C" __attribute__((visibility("default"), used)) void **__hipRegisterFatBinary(const void *) {
    static void *module;
    return &module;
}
extern "C" __attribute__((visibility("default"), used)) void __hipRegisterFunction(void **, const void *host, char *,
                                                                                   const char *name, unsigned, void *,
                                                                                   void *, void *, void *, int *) {
    fake::kernels()[host] = name;
}
extern "C" __attribute__((visibility("default"), used)) void __hipRegisterVar(void **, void *, char *, char *, int,
                                                                              size_t, int, int) {}
extern "C" __attribute__((visibility("default"), used)) void __hipUnregisterFatBinary(void **) {}

HIP_FAKE hipFuncSetAttribute(const void *f, int, int v) {
    fake::lds_limit[{fake::device, fake::kernels()[f]}] = (size_t)v;
    return 0;
}
HIP_FAKE hipLaunchKernel(const void *f, fake::Dim, fake::Dim, void **args, size_t lds, void *) {
    const std::string name = fake::kernels()[f];
    const fake::Launch l{name, fake::device, lds, args};
    const auto it = fake::lds_limit.find({fake::device, name});
    if (lds > (it == fake::lds_limit.end() ? 65536 : it->second)) {
        std::printf("device %d: %s with %zu bytes of LDS\n", fake::device, name.c_str(), lds);
        ++fake::refused;
        return fake::set(1);
    }
    if (fake::fail_launch && fake::fail_launch(name)) return fake::set(1);
    fake::launches.push_back(l);
    if (fake::on_launch) fake::on_launch(l);
    return 0;
}
HIP_FAKE hipGetLastError() {
    const int e = fake::last_error;
    fake::last_error = 0;
    return e;
}
extern "C" __attribute__((visibility("default"), used)) const char *hipGetErrorString(int) { return "fake error"; }
HIP_FAKE hipGetDevice(int *d) {
    *d = fake::device;
    return 0;
}
HIP_FAKE hipMalloc(void **p, size_t n) {
    *p = std::calloc(1, n ? n : 1);
    return *p ? 0 : 2;
}
HIP_FAKE hipFree(void *p) {
    std::free(p);
    return 0;
}
HIP_FAKE hipMemcpy(void *d, const void *s, size_t n, int) {
    std::memcpy(d, s, n);
    return 0;
}
HIP_FAKE hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) {
    std::memcpy(d, s, n);
    return 0;
}
HIP_FAKE hipMemset(void *d, int v, size_t n) {
    std::memset(d, v, n);
    return 0;
}
HIP_FAKE hipMemsetAsync(void *d, int v, size_t n, void *) {
    std::memset(d, v, n);
    return 0;
}
HIP_FAKE hipGetSymbolAddress(void **p, const void *) {
    static char symbol[256];
    *p = symbol;
    return 0;
}
HIP_FAKE hipDeviceSynchronize() { return 0; }
HIP_FAKE hipStreamSynchronize(void *) { return 0; }
HIP_FAKE hipStreamCreateWithFlags(void **s, unsigned) {
    *s = std::malloc(1);
    return 0;
}
HIP_FAKE hipStreamDestroy(void *s) {
    std::free(s);
    return 0;
}
HIP_FAKE hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
HIP_FAKE hipEventCreate(void **e) {
    *e = std::malloc(1);
    return 0;
}
HIP_FAKE hipEventCreateWithFlags(void **e, unsigned) { return hipEventCreate(e); }
HIP_FAKE hipEventDestroy(void *e) {
    std::free(e);
    return 0;
}
HIP_FAKE hipEventRecord(void *, void *) { return 0; }
HIP_FAKE hipEventSynchronize(void *) { return 0; }
HIP_FAKE hipEventElapsedTime(float *ms, void *, void *) {
    *ms = 1.f;
    return 0;
}
HIP_FAKE hipStreamBeginCapture(void *, int) { return 0; }
HIP_FAKE hipStreamEndCapture(void *, void **g) {
    *g = std::malloc(1);
    return 0;
}
HIP_FAKE hipGraphInstantiate(void **x, void *, void **, char *, size_t) {
    *x = std::malloc(1);
    return 0;
}
HIP_FAKE hipGraphLaunch(void *, void *) { return 0; }
HIP_FAKE hipGraphDestroy(void *g) {
    std::free(g);
    return 0;
}
HIP_FAKE hipGraphExecDestroy(void *g) {
    std::free(g);
    return 0;
}
