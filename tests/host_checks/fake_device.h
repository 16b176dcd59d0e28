// The HIP runtime and the kernel launchers as plain host code, for checks of the library's host files (she_api.cpp,
// she_host.cpp, she_circuits.cpp, she_leveled.cpp) without a GPU: device memory is host memory with a limit, copies are
// memcpy, every call that can fail can be told to, and the launchers that a check needs compute on the CPU.
#pragma once
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <vector>

#include "she_internal.h"

namespace fake {
inline std::map<char *, size_t> blocks;              // live device allocations
inline size_t held = 0, limit = ~(size_t)0;          // bytes in them, bytes there are
inline long calls = 0, fail_at = 0;                  // fallible calls so far, the one that fails (0: none)
inline hipError_t last_error = hipSuccess;           // sticky until hipGetLastError
inline std::function<void(const char *, size_t)> on_free;   // sees a block as it goes back
struct Rotations { size_t count, direct; const uint16_t *bar; bool mux, out; };
inline std::vector<Rotations> rotations;             // the launches of blind rotations so far

inline hipError_t result(hipError_t e) { if (e != hipSuccess) last_error = e; return e; }
inline hipError_t step() { return result(++calls == fail_at ? hipErrorUnknown : hipSuccess); }
}  // namespace fake

#define STEP() do { if (hipError_t e_ = fake::step()) return e_; } while (0)

extern "C" {
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t bytes)
{
    *p = nullptr;
    STEP();
    if (bytes > fake::limit - std::min(fake::held, fake::limit)) return fake::result(hipErrorOutOfMemory);
    *p = std::calloc(std::max<size_t>(bytes, 1), 1);
    fake::blocks[(char *)*p] = bytes;
    fake::held += bytes;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    if (!p) return hipSuccess;
    const auto b = fake::blocks.find((char *)p);
    if (b == fake::blocks.end()) { std::printf("hipFree of an unknown block\n"); std::abort(); }
    if (fake::on_free) fake::on_free(b->first, b->second);
    fake::held -= b->second;
    fake::blocks.erase(b);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { STEP(); std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    STEP();
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpy2D(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h, hipMemcpyKind)
{
    STEP();
    for (size_t r = 0; r < h; r++) std::memcpy((char *)d + r * dp, (const char *)s + r * sp, w);
    return hipSuccess;
}
hipError_t hipMemset(void *d, int v, size_t n) { STEP(); std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { STEP(); std::memset(d, v, n); return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return fake::step(); }
hipError_t hipStreamSynchronize(hipStream_t) { return fake::step(); }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)std::malloc(1); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { std::free((void *)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipGetLastError(void) { const hipError_t e = fake::last_error; fake::last_error = hipSuccess; return e; }
}

namespace she {
bool plan_supported(uint32_t) { return true; }
size_t twiddle_doubles(uint32_t) { return 2; }
void fill_twiddles(uint32_t, double *out) { out[0] = out[1] = 0; }
size_t half_twiddle_doubles(uint32_t) { return 0; }
void fill_half_twiddles(double *) {}
size_t bk_hat_elems(const she_params &) { return 1; }
hipError_t launch_bk_transform(const she_params &, const uint32_t *, const DeviceKeys &, hipStream_t) { return fake::step(); }
hipError_t launch_trgsw_transform(const she_params &, const DeviceKeys &, const uint32_t *, double2 *, const uint32_t *,
                                  size_t, hipStream_t) { return fake::step(); }
hipError_t launch_cmux(const she_params &, const DeviceKeys &, const double2 *, uint32_t *, const uint32_t *, const uint32_t *,
                       const uint32_t *, const uint32_t *, size_t, unsigned *, hipStream_t) { return fake::step(); }
hipError_t launch_lincomb(const she_params &, const CtSpace &, const uint8_t *, const uint32_t *, const uint32_t *,
                          const uint32_t *, size_t, const LevelWork &, hipStream_t) { return fake::step(); }
hipError_t launch_blind_rotate(const she_params &, const DeviceKeys &, const CtSpace &, const uint32_t *d_out, size_t count,
                               const LevelWork &W, unsigned *, hipStream_t, bool mux, size_t)
{
    fake::rotations.push_back({count, W.direct, W.bar, mux, d_out != nullptr});
    return fake::step();
}
hipError_t launch_mux_combine(const she_params &, const DeviceKeys &, const CtSpace &, const uint32_t *, size_t,
                              const LevelWork &, hipStream_t) { return fake::step(); }
hipError_t launch_key_switch(const she_params &, const DeviceKeys &, const CtSpace &, const uint32_t *, size_t,
                             const LevelWork &, hipStream_t) { return fake::step(); }
hipError_t launch_fp64_probe(int, double *, uint32_t, int, const double2 *, uint32_t, hipStream_t) { return fake::step(); }
hipError_t launch_lds_probe(int, uint32_t *, uint32_t, int, hipStream_t) { return fake::step(); }
hipError_t launch_copy_ct(const CtSpace &, const uint32_t *, const uint32_t *, size_t, uint32_t, hipStream_t) { return fake::step(); }
hipError_t noalloc_scratch(int, void **p, size_t *bytes) { *p = nullptr; *bytes = 0; return hipSuccess; }

// mask words k + i, no error of its own: every second sample is left to the host
hipError_t launch_fresh_samples(const CtSpace &cs, const uint32_t *ids, const uint8_t *bits, const uint8_t *key, uint32_t n,
                                uint64_t, double, size_t count, uint32_t *retry_count, uint32_t *retry, hipStream_t)
{
    STEP();
    for (size_t k = 0; k < count; k++) {
        uint32_t *dst = cs.pool + (size_t)ids[k] * cs.stride, sum = 0;
        for (uint32_t i = 0; i < n; i++) { dst[i] = (uint32_t)(k + i) << 20; sum += key[i] ? dst[i] : 0u; }
        dst[n] = sum + (bits[k] ? 1u << 29 : 0u - (1u << 29));
        if (k % 2) retry[(*retry_count)++] = (uint32_t)k;
    }
    return hipSuccess;
}
hipError_t launch_phase_bits(const CtSpace &cs, const uint32_t *ids, const uint8_t *key, uint32_t n, size_t count,
                             uint8_t *bits, hipStream_t)
{
    STEP();
    for (size_t k = 0; k < count; k++) {
        const uint32_t *ct = cs.pool + (size_t)ids[k] * cs.stride;
        uint32_t phase = ct[n];
        for (uint32_t i = 0; i < n; i++) phase -= key[i] ? ct[i] : 0u;
        bits[k] = (int32_t)phase > 0;
    }
    return hipSuccess;
}
hipError_t launch_clear_words(uint32_t *dst, size_t words, hipStream_t)
{
    STEP();
    std::fill(dst, dst + words, 0u);
    return hipSuccess;
}
hipError_t launch_trlwe_gather(const uint32_t *trlwe, uint32_t *dst, const uint32_t *ids, size_t count, uint32_t N, hipStream_t)
{
    STEP();
    for (size_t k = 0; k < count; k++)
        for (uint32_t w = 0; w < N / 2; w++) {
            const uint32_t c = w / (N / 4), q = w % (N / 4) / 64, j = c * N + 128 * q + w % 64;
            const uint32_t *v = trlwe + (size_t)ids[k] * 2 * N + 4 * w;
            uint32_t *d = dst + k * 2 * N + j;
            d[0] = v[0]; d[N / 2] = v[1]; d[64] = v[2]; d[64 + N / 2] = v[3];
        }
    return hipSuccess;
}
}  // namespace she
