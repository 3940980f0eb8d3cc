// Selection keys (csrc/msao_keys.h) on the CPU: in range the exact key; out of
// range (z and d are the caller's) every key below the selection's range, every
// digit with a bin, and as many tokens listed for a digit as were counted.
// Used by tests/test_keys_cpu.py.
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>

#include "msao_keys.h"

using namespace msao;

static int bad = 0;
#define CHECK(x) do { if (!(x)) { if (++bad < 10) printf("FAIL line %d: %s\n", __LINE__, #x); } } while (0)

static void selection(std::mt19937_64& rng, int kind, uint32_t C, uint32_t E, uint64_t Ls, uint64_t Lt, bool in_range)
{
    const uint64_t kmax = kind == kKeyZ ? C : kind == kKeyE ? E : kind == kKeyFull ? Ls * C + Lt * E : kind == kKeyImp ? kImpKeyMax : 0;
    const int bits = key_bits(kmax), shift = first_shift(bits), N = 3000;
    CHECK(bits == 0 ? kmax == 0 : kmax >> (bits - 1) == 1);
    std::vector<uint32_t> z(N), d(N);
    for (int i = 0; i < N; ++i) {
        z[i] = in_range ? (uint32_t)(rng() % (C + 1)) : (uint32_t)rng();
        d[i] = in_range ? (uint32_t)(rng() % (E + 1)) : (uint32_t)rng() >> (rng() % 32);
        if (kind == kKeyImp && in_range) {
            float m = (float)(rng() % 1000001) / 1e6f;
            memcpy(&z[i], &m, 4);
        }
    }
    TokenKeys t;
    t.first = kind == kKeyZ || kind == kKeyFull || kind == kKeyImp ? z.data() : nullptr;
    t.d = kind == kKeyE || kind == kKeyFull ? d.data() : nullptr;
    t.kind = kind;
    t.Ms = kind == kKeyFull ? Ls : 1;
    t.Mt = kind == kKeyFull ? Lt : 1;
    t.E = E;
    t.mask = (1ull << bits) - 1;
    std::vector<uint32_t> counted(kRadixBins, 0), listed(kRadixBins, 0);
    for (int i = 0; i < N; ++i) {
        const uint64_t k = t.at(i);
        CHECK(k <= t.mask);
        if (kind != kKeyFull) CHECK(t.of_one(t.one() ? t.one()[i] : 0u) == k);
        if (in_range) {
            if (kind == kKeyZ) CHECK(k == z[i]);
            if (kind == kKeyE) CHECK(k == E - d[i]);
            if (kind == kKeyFull) CHECK(k == Ls * z[i] + Lt * (uint64_t)(E - d[i]));
            CHECK(k <= kmax);
        }
        CHECK(first_digit(k, shift) < (uint32_t)kRadixBins);
        if (first_digit(k, shift) < (uint32_t)kRadixBins) counted[first_digit(k, shift)]++;
    }
    for (int g = 0; g < kRadixBins; ++g)
        for (int i = 0; i < N; ++i)
            if (first_digit(t.at(i), shift) == (uint32_t)g) listed[g]++;
    CHECK(counted == listed);
}

int main()
{
    std::mt19937_64 rng(1);
    for (int in = 0; in < 2; ++in)
        for (uint32_t C : {8u, 40u, 512u, 1280u, 4096u, 65536u})
            for (uint32_t E : {C, 16u, 64u}) {
                selection(rng, kKeyZero, C, E, 0, 0, in != 0);
                selection(rng, kKeyZ, C, E, 10066330, 0, in != 0);
                selection(rng, kKeyE, C, E, 0, 6710886, in != 0);
                selection(rng, kKeyFull, C, E, 10066330, 6710886, in != 0);
                selection(rng, kKeyFull, C, E, 16777216ull * 64, 16777216ull * 65536, in != 0);
                selection(rng, kKeyImp, C, E, 0, 0, in != 0);
            }
    // importances: larger first, NaN and what is not above 0 last
    const float v[] = {1.0f, 0.999f, 0.5f, 1e-3f, 1e-20f, 1e-45f};
    uint32_t last = 0;
    for (float m : v) {
        uint32_t b;
        memcpy(&b, &m, 4);
        CHECK(imp_key(b) >= last && imp_key(b) < kImpKeyMax);
        last = imp_key(b);
    }
    for (float m : {0.0f, -0.0f, -1.0f, (float)NAN}) {
        uint32_t b;
        memcpy(&b, &m, 4);
        CHECK(imp_key(b) == kImpKeyMax);
    }
    printf(bad ? "%d checks failed\n" : "all keys as expected\n", bad);
    return bad ? 1 : 0;
}
