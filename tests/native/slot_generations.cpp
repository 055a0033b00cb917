// Model of one exchange slot pair: units used by an exchange are read until they carry
// its generation, so none may carry it before this exchange writes it.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>

#include "hac_slots.h"

// First exchange at which a used unit already carries the generation, 0 = none.
static uint32_t stale(bool rule, uint32_t seed, uint32_t exchanges) {
    constexpr int kUnits = 130;
    static uint16_t gen[2][kUnits];
    std::memset(gen, 0, sizeof gen);
    std::mt19937 rng(seed);
    int used = 10;
    for (uint32_t e = 1; e < exchanges; ++e) {
        // Long runs of few units, single exchanges of many; at the wraps of the count too.
        used = (rng() & 1023u) == 0 || (e & 0xFFFFu) < 8 ? 10 + (int)(rng() % 121u) : 10;
        uint16_t *s = gen[e & 1u];
        for (int u = 0; u < used; ++u)
            if (s[u] == (uint16_t)e) return e;
        const int put = rule && hac::writes_whole_slot(e) ? kUnits : used;
        for (int u = 0; u < put; ++u) s[u] = (uint16_t)e;
    }
    return 0;
}

int main() {
    int plain = 0;
    for (uint32_t seed = 0; seed < 40; ++seed) {
        if (stale(true, seed, 300000)) return std::printf("stale words at seed %u\n", seed), 1;
        plain += stale(false, seed, 300000) != 0;
    }
    // The model does show the fault without the rule.
    std::printf("%s\n", plain ? "ok" : "model too weak");
    return plain ? 0 : 1;
}
