// A thread's answers to "which kernel runs this problem".  A search walks tables and models for up to tens of microseconds, a call
// asks up to three times (size query, workspace carve-out, launch), and a training loop asks for the layers of one network in turn,
// step after step: the calling thread keeps the answers it was given last, 512 of a kind, without locks.  A set of entries is made
// when the first of its problems comes and freed when the thread ends; without memory for it the answer is searched for each time.  (All
// sets in the thread's own storage were 309 KB to clear before its first answer, a backward-weight size query: 14 us in a new thread instead of
// 9, and the first forward query of a process 136 instead of 10.)
//
// A problem's place follows from all words of its key: multilinear hashing (Carter and Wegman; Dietzfelbinger's form for arithmetic
// modulo 2^64), the sum of the 32-bit words, each times a 64-bit constant of its own, of which the top bits name one of 64 sets of
// eight entries; the entry used longest ago makes room.  The products do not wait for each other.  Sizes of layers are multiples of 64
// more often than not: places from the low bits of a sum with small weights held 17 layers of a ResNet-50 in 9 of 64, each search
// undoing the last.  Measured, size query of backward-weight, bf16 NHWC, the layers in turn (us, such places -> these): 20 layers of
// ResNet-50 at batch 64 9.3 -> 0.12, at batch 256 11.5 -> 0.12, 36 of an inception network at batch 32 3.5 -> 0.12; one layer by itself
// 0.103 -> 0.112.
#pragma once
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <type_traits>
#include <utility>

namespace mxc {

extern thread_local long long g_plan_searches;      // searches the calling thread has made (mxc_plan_searches)

// The constant of word i: the i-th output of the SplitMix64 generator (Steele, Lea and Flood, 2014), made odd.
constexpr uint64_t hash_constant(int i)
{
    uint64_t z = (uint64_t)(i + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return (z ^ (z >> 31)) | 1;
}
template <typename Words> struct HashConstants;
template <int... I> struct HashConstants<std::integer_sequence<int, I...>> { static constexpr uint64_t of[] = {hash_constant(I)...}; };

template <typename Key, typename Value> class PlanCache {
    static_assert(std::has_unique_object_representations_v<Key> && sizeof(Key) % 4 == 0, "keys are mixed and compared as words: no padding");
    static_assert(std::is_trivially_copyable_v<Key> && std::is_trivial_v<Value>, "entries start as zeros, without a constructor to run");
    static constexpr int WORDS = sizeof(Key) / 4, SET_BITS = 6, WAYS = 8;
    struct Entry { uint32_t key[WORDS]; Value value; };
    struct Set { uint64_t tag[WAYS]; uint64_t used[WAYS], clock; Entry entry[WAYS]; };
    Set *sets_[1 << SET_BITS] = {};

public:
    PlanCache() = default;
    PlanCache(const PlanCache &) = delete;
    PlanCache &operator=(const PlanCache &) = delete;
    ~PlanCache()
    {
        for (Set *s : sets_) free(s);
    }
    // The answer kept for the key, or else that of `search`, which is then kept.
    template <typename F> Value get(const Key &k, F search)
    {
        uint32_t key[WORDS];
        memcpy(key, &k, sizeof key);
        uint64_t h = 0;
        for (int i = 0; i < WORDS; ++i) h += key[i] * HashConstants<std::make_integer_sequence<int, WORDS>>::of[i];
        Set *&made = sets_[h >> (64 - SET_BITS)];
        if (made == nullptr && (made = static_cast<Set *>(calloc(1, sizeof(Set)))) == nullptr) return search();
        Set &s = *made;
        h |= 1;                                      // no entry in use has tag 0
        for (int w = 0; w < WAYS; ++w)
            if (s.tag[w] == h && !memcmp(s.entry[w].key, key, sizeof key)) {
                s.used[w] = ++s.clock;
                return s.entry[w].value;
            }
        const Value v = search();
        int oldest = 0;
        for (int w = 1; w < WAYS; ++w)
            if (s.used[w] < s.used[oldest]) oldest = w;
        memcpy(s.entry[oldest].key, key, sizeof key);
        s.entry[oldest].value = v;
        s.tag[oldest] = h;
        s.used[oldest] = ++s.clock;
        return v;
    }
};

}  // namespace mxc
