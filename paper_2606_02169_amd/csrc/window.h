// The window form of the plan-specialized matvec (window.cpp).
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "mrmf_internal.h"

namespace mrmf {

constexpr int64_t kWindowLds = 163840;  // LDS of a compute unit: the staged rows and the tables of the uniform digits
constexpr int kWindowTab = 1024;        // most entries of those tables
constexpr int kWindowSum = 8;           // addends of an entry whose loads a thread issues together

// What a pass does with the rows it computes (H': the pass's terms).
constexpr int kPassSet = 0;       // y = H' x
constexpr int kPassAdd = 1;       // y += H' x
constexpr int kPassCheb = 2;      // p = ea H' x + eb x + eg y;  y = p;  acc += (ecr + i eci) p
constexpr int kPassChebPart = 3;  // y = ea H' x + eb x + eg y

struct WindowPass {
    std::vector<int> ord;      // the sites, most significant first: uniform, unrolled, inner
    int n_uni = 0, n_unr = 0;  // how many of them are uniform and unrolled
    std::vector<int> chans, diags;  // the pass's channels and diagonal terms (indices into the plan's lists)
    int mode = kPassSet;
    bool f32 = false, wide = false;
    int sched = 0;        // MRMF_SCHED_*
    int group = 8;        // gathers of a copy issued together, and LDS reads
    int waves = 0;        // > 0: ask the compiler for at least this many waves per SIMD
    int64_t dbuf_bytes = 49152;  // the staged rows are double-buffered while that takes no more LDS than this
    bool prefetch = true;  // the rows of the next super-tile are requested while the current one is computed
    std::string name, tag;  // kernel name; suffix of the pass's constants
};

// What a pass asks of a block: values that are worked out before its first super-tile, and gathers.
struct WindowCost {
    int coefs = 0;    // coefficients that are the same for every row
    int fills = 0;    // rounds of the block that fill the tables of the uniform digits
    int gathers = 0;  // of the first copy
    int varying = 0;  // of those, with a factor that differs between rows or super-tiles
    int tabled = 0;   // of those, with a factor read from the tables for every super-tile
};

// true when every term weight is real (the form has no complex coefficients)
bool window_real(const mrmf_plan_t* p);
std::string window_prelude(bool f32, bool wide);
// Source of one pass (after window_prelude, which several passes share); "" when the plan or its tile does not fit the
// form (tables, LDS).
std::string window_pass(const mrmf_plan_t* p, const WindowPass& w, int64_t* n_tiles, int64_t* rows, WindowCost* cost);

}  // namespace mrmf
