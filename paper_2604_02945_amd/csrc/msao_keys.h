// msao_keys.h -- selection keys and their first radix digit. Plain C++, for the
// kernels and for a check on the CPU.
#ifndef MSAO_KEYS_H
#define MSAO_KEYS_H

#include <stdint.h>

#ifdef __HIPCC__
#define MSAO_KEYS_FN __host__ __device__ __forceinline__
#else
#define MSAO_KEYS_FN inline
#endif

namespace msao {

// Key kinds of a selection: Ms z + Mt (E - d) in general, z or E - d alone
// when the other weight is 0 (the same order, a narrower range); or, in a
// learned run, a segment with a head ranked by its Eq. 3 importance.
enum : int { kKeyZero = 0, kKeyZ = 1, kKeyE = 2, kKeyFull = 3, kKeyImp = 4 };
constexpr uint32_t kImpKeyMax = 0x3F800000u;  // the bits of 1.0f
constexpr int kRadixBits = 11;
constexpr int kRadixBins = 1 << kRadixBits;

// A learned importance (its bits) as a key: larger importance first. It is a
// sigmoid, at most 1, and the bits of a positive float grow with its value, so
// their distance below those of 1 orders it downwards; NaN and values not above
// 0 take the largest key (importance 0). (30 bits instead of the complement's
// 32: the first digit then tells 16 values per octave apart instead of 4, and
// few enough keys share one to be ranked directly.)
MSAO_KEYS_FN uint32_t imp_key(uint32_t bits) { return bits - 1u < 0x7F800000u ? kImpKeyMax - bits : kImpKeyMax; }

// Bits of the keys 0 .. kmax, and the shift of their first digit.
MSAO_KEYS_FN int key_bits(uint64_t kmax) { return kmax > 0 ? 64 - __builtin_clzll((unsigned long long)kmax) : 0; }
MSAO_KEYS_FN int first_shift(int bits) { return bits > kRadixBits ? bits - kRadixBits : 0; }
MSAO_KEYS_FN uint32_t first_digit(uint64_t key, int shift) { return (uint32_t)(key >> shift); }

// The keys of a selection's tokens, key(i) = Ms z + Mt (E - d) of token i,
// order-equivalent to L_s z / C + L_t (E - d) / E (E = C for bit sampling,
// where Ms = L_s and Mt = L_t); when one weight is 0 the other term alone
// orders the tokens, so it is used unscaled; or the learned importance.
// `first`: the z values or importances; d: NULL where not used. z and d come
// from the caller and may be out of range: only the bits that the selection's
// largest key has are kept, so that every pass over the keys puts a token into
// the same digit, and every digit has a bin.
struct TokenKeys {
    const uint32_t* first;
    const uint32_t* d;
    int kind;
    uint64_t Ms, Mt;
    uint32_t E;
    uint64_t mask;
    MSAO_KEYS_FN uint64_t of(uint32_t z, uint32_t dd) const
    {
        if (kind == kKeyImp) return (uint64_t)imp_key(z) & mask;
        return (Ms * (uint64_t)z + (d ? Mt * (uint64_t)(E - dd) : 0ull)) & mask;
    }
    MSAO_KEYS_FN uint64_t at(int i) const { return of(first ? first[i] : 0u, d ? d[i] : 0u); }
    // The same for every kind but kKeyFull, whose keys alone need more than 32 bits
    // and two values: v is the token's entry of `one`.
    MSAO_KEYS_FN const uint32_t* one() const { return first ? first : d; }
    MSAO_KEYS_FN uint32_t of_one(uint32_t v) const
    {
        return (kind == kKeyImp ? imp_key(v) : kind == kKeyE ? E - v : v) & (uint32_t)mask;
    }
};

}  // namespace msao

#endif
