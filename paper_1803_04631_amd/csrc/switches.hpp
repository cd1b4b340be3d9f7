// Values of the environment switches (see mlda.h).  Host code only.
#pragma once
#include <errno.h>
#include <stdint.h>
#include <stdlib.h>

namespace mlda {

// n (up to 4) whole numbers with a comma between them, each within [lo, hi].  Any other text, and none: false, and nothing is stored.
inline bool switch_numbers(const char* text, int n, int64_t lo, int64_t hi, int64_t* numbers) {
    int64_t got[4];
    if (!text || n < 1 || n > 4) return false;
    for (int i = 0; i < n; ++i) {
        if (!(*text >= '0' && *text <= '9')) return false;
        char* end = nullptr;
        errno = 0;
        const long long v = strtoll(text, &end, 10);
        if (errno != 0 || v < lo || v > hi || *end != (i + 1 < n ? ',' : '\0')) return false;
        got[i] = (int64_t)v;
        text = end + 1;
    }
    for (int i = 0; i < n; ++i) numbers[i] = got[i];
    return true;
}

}  // namespace mlda
