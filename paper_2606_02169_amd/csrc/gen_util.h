// Helpers shared by the kernel generators (jit.cpp, window.cpp): literals and factor tables.
#pragma once

#include <cinttypes>
#include <cstdint>
#include <cstdio>
#include <string>
#include <vector>

#include "mrmf_internal.h"

namespace mrmf {

inline int64_t round_up(int64_t v, int64_t a) { return (v + a - 1) / a * a; }

inline std::string lit(double v, bool f32) {
    char buf[64];
    if (f32)
        std::snprintf(buf, sizeof buf, "%af", static_cast<double>(static_cast<float>(v)));
    else
        std::snprintf(buf, sizeof buf, "%a", v);
    return buf;
}

inline std::string ulit(uint64_t v) {
    char buf[32];
    std::snprintf(buf, sizeof buf, "%" PRIu64 "ull", v);
    return buf;
}

// Factor <n|O|n - q> of a local operator at target digit n, 0 where the source digit is outside 0..d-1.
inline std::vector<double> op_table(const mrmf_plan_t* p, int site, int op) {
    std::vector<double> t(p->d[site], 0.0);
    for (int n = 0; n < p->d[site]; ++n) t[n] = local_factor_host(p, site, op, n);
    return t;
}

}  // namespace mrmf
