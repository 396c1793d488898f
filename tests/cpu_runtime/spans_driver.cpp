// The spans of a drain against the definition (stream byte b lies at b modulo each ring's capacity) -- TEST INFRASTRUCTURE
// ONLY.  Places are compared as numbers; no ring of the larger sizes exists.
#include <cstdio>
#include <cstdlib>

#include "dmi_internal.h"

using namespace dmi;

static void check(uint64_t cap, uint64_t host_cap, uint64_t from, uint64_t nbytes)
{
    const uint8_t *const ring = reinterpret_cast<const uint8_t *>(uintptr_t(1) << 40);
    uint8_t *const host = reinterpret_cast<uint8_t *>(uintptr_t(1) << 44);
    for (uint64_t at = from, left = nbytes; left;) {
        DrainSpans d;
        const uint64_t n = drain_spans(ring, cap, host, host_cap, at, left, d);
        bool ok = n && n <= left && n <= kDrainMost && (n == left || n == kDrainMost);
        uint64_t b = at;
        for (const DrainSpan &s : d.span) {
            if (!s.n) continue;
            ok = ok && s.n % 64u == 0 && s.src == ring + b % cap && s.dst == host + b % host_cap &&
                 b % cap + s.n <= cap && b % host_cap + s.n <= host_cap;
            b += s.n;
        }
        if (!ok || b != at + n) {
            fprintf(stderr, "cap %llu host %llu from %llu nbytes %llu\n", (unsigned long long)cap, (unsigned long long)host_cap,
                    (unsigned long long)from, (unsigned long long)nbytes);
            exit(3);
        }
        at += n;
        left -= n;
    }
}

int main()
{
    for (uint64_t cap = 64; cap <= 64 * 9; cap += 64)
        for (uint64_t host = 64; host <= 64 * 9; host += 64)
            for (uint64_t from = 0; from < 64 * 40; from += 64)
                for (uint64_t n = 64; n <= cap && n <= host; n += 64) check(cap, host, from, n);
    const uint64_t G = 1ull << 30;
    for (const uint64_t cap : {G, 3 * G, 12 * G + 64, 100 * G})
        for (const uint64_t host : {G, 5 * G - 64, 16 * G})
            for (const uint64_t from : {uint64_t(0), cap - 64, host - 128, 977 * G + 64})
                for (const uint64_t n : {uint64_t(64), G - 64, G, G + 64, 4 * G + 4096})
                    if (n <= cap && n <= host) check(cap, host, from, n);
    fprintf(stderr, "passed\n");
    return 0;
}
