// The library's host files on a fake device (fake_device.h):
//   1. a call that runs out of memory says so and leaves no error for the next launch (or the next call of another library in
//      the process) to find;
//   2. a context whose scratch has grown gives everything back.
#include <cstdint>
#include <vector>

#include "fake_device.h"

static int failures = 0;
#define CHECK(c, ...) do { if (!(c)) { failures++; std::printf(__VA_ARGS__); } } while (0)

static she_ctx *context(uint32_t N, uint32_t capacity)
{
    she_params P{};
    P.n = 4; P.N = N; P.k = 1; P.bg_bit = 7; P.l = 3; P.ks_t = 1; P.ks_basebit = 1;
    she_ctx *c = nullptr;
    if (she_keygen(&P, 3, capacity, &c)) { std::printf("keygen: %s\n", she_last_error(nullptr)); std::exit(1); }
    return c;
}

// without memory the call fails and nothing stays behind; with memory it works
template <class F> static void short_of_memory(const char *what, F &&call)
{
    fake::limit = fake::held;
    int rc = call();
    CHECK(rc == SHE_ENOMEM, "%s without memory returns %d\n", what, rc);
    CHECK(hipGetLastError() == hipSuccess, "%s leaves an error behind\n", what);
    fake::limit = ~(size_t)0;
    rc = call();
    CHECK(rc == SHE_OK, "%s with memory returns %d\n", what, rc);
}

int main()
{
    std::vector<uint32_t> a(64), b(64), s(64), out(64);
    std::vector<uint8_t> bits(64, 1), types(64, 0);
    for (uint32_t k = 0; k < 64; k++) { a[k] = k; b[k] = 63 - k; s[k] = k; out[k] = 64 + k; }
    she_ctx *c = context(256, 128);
    short_of_memory("she_encrypt_bits", [&] { return she_encrypt_bits(c, bits.data(), 64, 5, a.data()); });
    short_of_memory("she_eval_gates", [&] { return she_eval_gates(c, types.data(), a.data(), b.data(), out.data(), 8); });
    short_of_memory("she_eval_mux", [&] { return she_eval_mux(c, s.data(), a.data(), b.data(), out.data(), 16); });
    short_of_memory("she_leveled_init", [&] { return she_leveled_init(c, 2, 64); });
    for (uint32_t k = 0; k < 64; k++) { s[k] = 0; a[k] = k % 8; b[k] = 8 + k % 8; out[k] = 16 + k % 48; }
    short_of_memory("she_eval_cmux", [&] { return she_eval_cmux(c, s.data(), a.data(), b.data(), out.data(), 48); });
    she_free(c);
    CHECK(fake::held == 0, "%zu bytes are still held after she_free\n", fake::held);

    // gate levels grow the scratch that MUX levels share
    c = context(256, 128);
    for (uint32_t k = 0; k < 64; k++) { s[k] = k; a[k] = k; b[k] = 63 - k; out[k] = 64 + k; }
    for (size_t count : {4, 16, 64}) {
        CHECK(she_eval_mux(c, s.data(), a.data(), b.data(), out.data(), count / 4) == SHE_OK, "%zu MUX gates\n", count / 4);
        CHECK(she_eval_gates(c, types.data(), a.data(), b.data(), out.data(), count) == SHE_OK, "%zu gates\n", count);
    }
    she_free(c);
    CHECK(fake::held == 0, "%zu bytes are still held after she_free of a context whose scratch grew\n", fake::held);
    std::printf("failures %d\n", failures);
    return failures != 0;
}
