// she_encrypt_bits and she_decrypt on a fake device (fake_device.h): the secret key's bits and the plaintext bits that a
// call brings to the device, and the call's own host copies of them, are overwritten before the call returns, whether it
// succeeds or any one of its HIP calls fails; a block of device memory that is given back holds none of them either.
#include <malloc.h>

#include <cstdint>
#include <new>
#include <vector>

#include "fake_device.h"

namespace {
int failures = 0;
#define CHECK(c, ...) do { if (!(c)) { failures++; std::printf(__VA_ARGS__); } } while (0)

constexpr uint32_t n = 96, COUNT = 77;
uint8_t key[n], bits[COUNT];
bool watch_host = false;      // inside a call: its own host copies are looked at when they are freed
long host_copies = 0;

bool holds(const char *p, size_t size, const uint8_t *secret, size_t len)
{
    return size >= len && memmem(p, size, secret, len) != nullptr;
}
bool holds_secret(const char *p, size_t size) { return holds(p, size, key, n) || holds(p, size, bits, COUNT); }

void release(void *p)
{
    if (p && watch_host && holds_secret((const char *)p, malloc_usable_size(p))) host_copies++;
    std::free(p);
}
}  // namespace

void *operator new(size_t size) { if (void *p = std::malloc(size ? size : 1)) return p; throw std::bad_alloc(); }
void operator delete(void *p) noexcept { release(p); }
void operator delete(void *p, size_t) noexcept { release(p); }

int main()
{
    she_params P{};
    P.n = n; P.N = 256; P.k = 1; P.bg_bit = 7; P.l = 3; P.ks_t = 2; P.ks_basebit = 2; P.lwe_std = 0; P.bk_std = 0;
    she_ctx *c = nullptr;
    if (she_keygen(&P, 3, 200, &c)) { std::printf("keygen: %s\n", she_last_error(nullptr)); return 1; }
    she_export_keys(c, key, nullptr, nullptr, nullptr);
    uint32_t ids[COUNT];
    for (uint32_t k = 0; k < COUNT; k++) { bits[k] = (k * k + k / 3) % 2; ids[k] = 199 - 2 * k; }
    fake::on_free = [](const char *p, size_t size) { CHECK(!holds_secret(p, size), "a freed device block holds a secret\n"); };
    std::vector<uint8_t> back(COUNT);

    auto residue = [&](const char *call, long k) {
        for (const auto &b : fake::blocks)
            CHECK(!holds_secret(b.first, b.second), "%s, failing call %ld: device memory holds a secret\n", call, k);
        CHECK(!host_copies, "%s, failing call %ld: a host copy was freed as it was\n", call, k);
        host_copies = 0;
    };
    // every failing call in turn, until one run needs fewer calls than that and succeeds
    auto every_failure = [&](const char *call, auto run) {
        int succeeded = 0;
        for (long k = 1; k < 200 && !succeeded; k++) {
            fake::calls = 0; fake::fail_at = k;
            watch_host = true;
            const int rc = run();
            watch_host = false;
            fake::fail_at = 0;
            CHECK(rc == (fake::calls < k ? SHE_OK : SHE_EDEVICE), "%s, failing call %ld: %d\n", call, k, rc);
            residue(call, k);
            succeeded = rc == SHE_OK;
        }
        CHECK(succeeded, "%s never succeeded\n", call);
    };
    every_failure("encrypt", [&] { return she_encrypt_bits(c, bits, COUNT, 5, ids); });
    every_failure("decrypt", [&] {
        std::fill(back.begin(), back.end(), (uint8_t)2);
        const int rc = she_decrypt(c, ids, COUNT, back.data());
        if (rc == SHE_OK) CHECK(std::equal(back.begin(), back.end(), bits), "wrong bits\n");
        std::fill(back.begin(), back.end(), (uint8_t)2);                     // the caller's own array is not the library's to clear
        return rc;
    });
    she_free(c);
    CHECK(fake::blocks.empty(), "device memory left\n");
    std::printf("failures %d\n", failures);
    return failures != 0;
}
