// Batched form: many independent lattices, each applied to a block of nvec c64 vectors, in one
// persistent launch.  Each lattice is the same target-driven gather (Sec. II) with its own digits
// (Sec. III, Eq. decode), channels and offsets (Sec. IV, Eq. sourceoffset) and ladder factors (App. A,
// App. B, App. C); the lattices only share the launch.
//
// Layout.  Lattice b's vectors are stored row-major as [D_b][nvec] at element offset off_b of X and Y
// (row F holds its nvec amplitudes contiguously, so one row is 8 * nvec bytes); offsets are multiples
// of 32 elements.
//
// Shared input (parameter sweeps: the same vectors under many couplings): every lattice reads block 0 of X,
// and the items are numbered tile by tile across the lattices instead of lattice by lattice.
//
// Work.  For a launch shape (R_max, block B), lattice b's rows are cut into tiles of T c rows: all states of its low
// sites (T = prod of the low d_i, the largest such product <= R_max) for c neighbouring digits of the next site (c = 1
// unless T <= R_max / 2, so that a tile is more than half full however large one site is).  An item is a tile; a block
// holds it in LDS (rows stored vector-major, so that consecutive threads read consecutive 8-byte words).  Items are
// numbered lattice by lattice.  Three schedules: runs - block v of the grid takes the contiguous item range
// [v I / G, (v+1) I / G), v chosen so that the blocks of one XCD (block b runs on XCD b mod 8) hold neighbouring ranges;
// windows - the grid sweeps windows of G consecutive items, the blocks of one XCD taking one eighth of each window side
// by side, so that the items an XCD works on at one time are neighbours and the gathers of one item find the rows its
// neighbours have just read in the XCD's L2 (at the price of reloading a lattice's descriptors whenever a block moves to
// another lattice); XCD chunks - XCD x sweeps the x-th eighth of every lattice's items with its blocks side by side, so
// that its L2 also holds the rows it read further back, while all XCDs work on one lattice, whose vectors the memory-side
// cache then holds (eighths of the whole list, each XCD in another lattice: 2.73 ms against 2.33 for windows in the case
// below, now 1.92 against 1.93).  With a shared input the strides are multiples of the lattice count, so that a block
// stays with one lattice.
//
// What a row costs.  The digits above the tile are the same for all its rows, so a wave works them out once per tile,
// one lane per site and then one lane per term: a channel whose sites lie above the tile is then either left out for the
// whole tile or a plain contiguous load with one coefficient, without work per row.  Digits inside the tile and the sums
// of its diagonal terms depend on the row of the tile alone and are laid out once per lattice.  Only the other terms
// (both sites in the tile: source in LDS; one inside, one above: gather) look their factors up per row.  The sums run in
// one order of the terms, whatever the tile, so every launch shape gives the same bits.
//
// Bound.  64 open chains of 8 to 16 sites (29.3 M rows, eight vectors; 10.5 GB fetched and 1.9 written, against 3.8 that
// every vector costs once): 2.39 ms with digits, factors and skips per row (2045 vector instructions per 64 rows, two
// waves per SIMD), 1.92 ms now, limited by the serial chain of a wave's item and by the gathers that miss the L2
// (6.4 TB/s).  What counts is waves: at 16 per CU (128 registers, of which eight vectors spill one, with complex weights
// and more than 64 terms 20; two gathers at a time, as three or four spill far more: 2.25 and 3.4 ms) against 12, 1.92 and
// 2.12 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "mrmf_internal.h"

namespace mrmf {
namespace {

constexpr int kBatchMaxLattices = 2048;
constexpr int kBatchMaxSites = 32;
constexpr int kBatchMaxBlock = 512;
constexpr int kBatchPoolMax = 2048;    // factor-table entries of one lattice (LDS)
constexpr int kBatchTileWords = 4096;  // 8-byte words of the LDS tile (32 KB): at most 4096 / nvec rows
constexpr int kBatchRmaxCands = 4;     // tile-row limits R_max = (64, 128, 256, 512) * 8 / nvec
constexpr int kBatchTermSets = 2;      // terms of one lattice, 64 to a set: one to a lane
constexpr int kBatchMaxTerms = 64 * kBatchTermSets;  // channels and diagonal terms
constexpr int kBatchMaxParams = 128;   // couplings of one lattice: no more than it has terms
constexpr int kBatchGather = 2;        // gathers issued together

struct alignas(16) BLat {
    int32_t N, n_chan, n_diag, theta_off;
    int32_t term_off, site_off, pool_off, pool_n;
    int64_t x_off, pad;
    int32_t item_beg[kBatchRmaxCands];    // per R_max candidate: first item of the lattice
    int32_t part_beg[kBatchRmaxCands];    // the same count of items per eighth of a lattice (rounded up)
    int32_t low_rows[kBatchRmaxCands];    // T
    int32_t low_sites[kBatchRmaxCands];   // number of low sites that T spans
    int32_t chunk[kBatchRmaxCands];       // c
    int32_t n_chunks[kBatchRmaxCands];    // ceil(d / c) of the next site d, 1 when c = 1
    int32_t n_local[kBatchRmaxCands];     // channels whose source lies in the tile (a prefix of the list)
    int32_t n_ldiag[kBatchRmaxCands];     // diagonal terms of the T rows' digits alone (a prefix of the list)
};
static_assert(sizeof(BLat) == 176, "BLat layout");

// n / m for n < 2^31 is umulhi(2 n, mul) >> shift (mul = ceil(2^(31 + shift) / m), shift = ceil(log2 m))
struct BDiv {
    uint32_t mul, shift;
};

struct alignas(16) BSite {
    int32_t d, pad;
    BDiv by_d, by_m, by_md;  // division by d, by the site's stride, by d times the stride
};
static_assert(sizeof(BSite) == 32, "BSite layout");

// One term: coefficient theta[param] * (wr + i wi) * pool[ta + n_a] * pool[tb + n_b]; source F - delta.
// A one-site term has b = -1 (its second factor is the pool's 1.0 entry at tb, digit 0).  low = number of
// low sites a tile must span for the term's sites to lie in it.
struct alignas(16) BTerm {
    int32_t a, b, ta, tb;
    int32_t param, delta, low, pad;
    float wr, wi, pad1, pad2;
};
static_assert(sizeof(BTerm) == 48, "BTerm layout");

struct BatchArgs {
    const BLat* lat;     // n_lat entries and one that holds the item counts
    const BSite* site;
    const BTerm* term;   // channels and diagonal terms of every lattice
    const float* pool;   // factor tables of every lattice
    int32_t n_lat;
    int32_t shared;  // every lattice reads its input rows from the one block at the start of X; items tile-major
};

__device__ __forceinline__ uint32_t div_by(uint32_t n, BDiv m) { return __umulhi(n << 1, m.mul) >> m.shift; }

__device__ __forceinline__ int lane_of(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
__device__ __forceinline__ float lane_of(float v, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// a product and a sum that are rounded each, never contracted, so that a term has one value wherever it is formed
__device__ __forceinline__ float mul_rn(float a, float b) {
#pragma clang fp contract(off)
    return a * b;
}
__device__ __forceinline__ float add_rn(float a, float b) {
#pragma clang fp contract(off)
    return a + b;
}

// digit of a field (shift | width << 5) of a row word; 0 for an empty field
__device__ __forceinline__ uint32_t digit_of(uint32_t word, int f) {
    return __builtin_amdgcn_ubfe(word, f & 31, f >> 5);
}

// Terms of the current lattice, lane k holding term k (a second set holds terms 64 and up).
struct LaneTerms {
    int tab;         // factor-table entries of the two sites at digit 0: a | b << 16
    int sites;       // a | b << 8 (b = a for a one-site term)
    int field;       // field of each site in the row word (shift | width << 5; width 0: the site is above the tile),
                     // a | b << 16; bit 31: one-site term
    int delta;
    float wr, wi;    // theta wr, theta wi
    // of the current tile
    int at;          // table entries at the digits of the tile's first row, a | b << 16
    float vr, vi;    // coefficient when both sites are above the tile
};

// f at the constants 0 .. N - 1
template <int N, typename F>
__device__ __forceinline__ void each(F&& f) {
    f(std::integral_constant<int, 0>{});
    if constexpr (N > 1) f(std::integral_constant<int, 1>{});
    if constexpr (N > 2) {
        f(std::integral_constant<int, 2>{});
        f(std::integral_constant<int, 3>{});
    }
}

// Two layouts of a wave's 64 rows.  By rows: lane l holds the NV amplitudes of one row (factors and LDS reads are per
// row).  By pieces: a row is NP pieces of two amplitudes (16 bytes; one of 8 bytes when NV = 1), NP neighbouring lanes
// hold a row and every lane NP rows, so that one load or store of the wave moves 64 consecutive pieces.  Loads by rows
// touch every line NP times, far enough apart in time that the L1 has lost it.  The lane groups of a row hold the same
// NP rows in both layouts, so that a transposition inside them leads from one to the other.
template <int NV>
struct Wave {
    static constexpr int NP = NV < 2 ? 1 : NV / 2;
    static constexpr int PW = NV < 2 ? 2 : 4;  // floats of a piece
    // padding of a vector's rows in LDS: the pieces of NP lanes then fall into different banks
    static constexpr int kPad = NV == 8 ? 4 : NV == 4 ? 8 : 0;
    // row i of lane group a; the rows of half a wave are distinct modulo 32 (no bank conflicts by rows)
    static __device__ __forceinline__ int row(int a, int i) { return (64 / NP) * i + (2 * i >= NP && NP > 1 ? a ^ (32 / NP) : a); }
    // what lane i of the lane group holds
    template <int I>
    static __device__ __forceinline__ int from(int v) {
        if constexpr (NP == 1) return v;
        constexpr int ctrl = NP == 4 ? I * 0x55 : I == 0 ? 0xA0 : 0xF5;  // quad_perm
        return __builtin_amdgcn_mov_dpp(v, ctrl, 0xf, 0xf, true);
    }
    // e[p] of lane j becomes e[j] of lane p
    static __device__ __forceinline__ void transpose(float (&e)[NP][PW], int lane) {
        if constexpr (NP >= 2) step<1, 0xB1>(e, lane);
        if constexpr (NP >= 4) step<2, 0x4E>(e, lane);
    }
    template <int S, int CTRL>
    static __device__ __forceinline__ void step(float (&e)[NP][PW], int lane) {
        const bool up = (lane & S) != 0;
#pragma unroll
        for (int p = 0; p < NP; ++p)
            if ((p & S) == 0) {
#pragma unroll
                for (int w = 0; w < PW; ++w) {
                    const float send = up ? e[p][w] : e[p + S][w];
                    const float got = __int_as_float(
                        __builtin_amdgcn_mov_dpp(__float_as_int(send), CTRL, 0xf, 0xf, true));
                    e[p][w] = up ? got : e[p][w];
                    e[p + S][w] = up ? e[p + S][w] : got;
                }
            }
    }
    static __device__ __forceinline__ void load(const float2* __restrict__ src, float (&v)[PW]) {
        if constexpr (PW == 2) {
            const float2 w = *src;
            v[0] = w.x;
            v[1] = w.y;
        } else {
            const float4 w = *reinterpret_cast<const float4*>(src);
            v[0] = w.x;
            v[1] = w.y;
            v[2] = w.z;
            v[3] = w.w;
        }
    }
    static __device__ __forceinline__ void store(float2* __restrict__ dst, const float (&v)[PW], bool stream) {
        using Vec = __attribute__((__vector_size__(PW * sizeof(float)))) float;
        Vec w;
#pragma unroll
        for (int e = 0; e < PW; ++e) w[e] = v[e];
        if (stream) __builtin_nontemporal_store(w, reinterpret_cast<Vec*>(dst));
        else *reinterpret_cast<Vec*>(dst) = w;
    }
};

template <int NV, bool CPLX, int kSets>
__global__ __launch_bounds__(kBatchMaxBlock, 4) void k_batch(BatchArgs A, const float* __restrict__ theta_all,
                                                        const float2* __restrict__ X, float2* __restrict__ Y,
                                                        int32_t rc, int32_t sched) {
    constexpr int kRows = kBatchTileWords / NV;
    using W = Wave<NV>;
    constexpr int NP = W::NP, PW = W::PW;
    extern __shared__ float pool[];              // factor tables of the current lattice
    __shared__ float2 xt[NV][kRows + W::kPad];
    __shared__ uint32_t rw[kRows];              // digits inside the tile, one field per site
    __shared__ float rd[CPLX ? 2 : 1][kRows];   // diagonal terms of the low digits
    __shared__ int32_t field[kBatchMaxSites];   // field of each site in the row word
    const int tid = threadIdx.x, B = blockDim.x, lane = tid & 63;
    const int la = lane / NP, lp = lane % NP;     // lane group, piece
    const int lrow = W::row(la, lp);              // by rows: row of the lane
    const int G = gridDim.x, bid = blockIdx.x, nl = A.n_lat;
    const bool shared = A.shared != 0;
    const int v = (G % 8 == 0) ? (bid % 8) * (G / 8) + bid / 8 : bid;
    // parts: XCD x sweeps the x-th eighth of every lattice
    const bool parts = sched == 2 && !shared && G % 8 == 0;
    const int32_t I = parts ? A.lat[nl].part_beg[rc] : A.lat[nl].item_beg[rc];
    int32_t i0, i1, step;
    // blocks side by side: with a shared input a stride that is a multiple of the lattice count keeps a block with one
    // lattice (the few blocks beyond it have no work), where the lattices are few enough for that
    const auto stride = [&](int n) { return shared && nl * 4 <= n ? n / nl * nl : n; };
    if (parts) {
        step = G / 8;
        i0 = bid / 8;
        i1 = I;
    } else if (sched == 2 && G % 8 == 0) {  // shared input: an eighth of the tiles, every lattice
        const int xcd = bid % 8;
        const int64_t C = (I / nl + 7) / 8 * nl;
        step = stride(G / 8);
        i1 = static_cast<int32_t>((xcd + 1) * C < I ? (xcd + 1) * C : I);
        i0 = bid / 8 < step ? static_cast<int32_t>(xcd * C < I ? xcd * C + bid / 8 : I) : I;
    } else if (sched != 0) {  // windows
        step = stride(G);
        i0 = v < step ? v : I;
        i1 = I;
    } else {  // runs
        i0 = static_cast<int32_t>(int64_t(v) * I / G);
        i1 = static_cast<int32_t>(int64_t(v + 1) * I / G);
        step = 1;
    }
    const auto first_item = [&](int l) { return parts ? A.lat[l].part_beg[rc] : A.lat[l].item_beg[rc]; };
    int lb = -1;
    // the current lattice's descriptor, kept in scalar registers (every field is block-uniform)
    int32_t N = 0, n_chan = 0, n_diag = 0, T = 1, ks = 0, n_loc = 0, n_ld = 0, chunk = 1, nch = 1, dp = 1;
    const float2* xb = X;
    float2* yb = Y;
    BSite site{};  // lane i: site i
    LaneTerms lt[kSets];
    int b = 0;
    int32_t beg = 0, end = 0, count = 0;  // items of lattice b (of an eighth of it), tiles of lattice b
    const auto tiles = [&](int l) {
        return __builtin_amdgcn_readfirstlane(A.lat[l + 1].item_beg[rc] - A.lat[l].item_beg[rc]);
    };
    if (!shared) {
        int lo = 0, hi = nl - 1;  // last lattice with its first item <= i0
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (first_item(mid) <= i0) lo = mid; else hi = mid - 1;
        }
        b = lo;
        beg = __builtin_amdgcn_readfirstlane(first_item(b));
        end = __builtin_amdgcn_readfirstlane(first_item(b + 1));
        count = tiles(b);
    }
    for (int32_t it = i0; it < i1; it += step) {
        // shared input: every lattice has the same tiles; item it is tile it / n of lattice it mod n, so the
        // items worked on together read the same input rows
        int32_t li;
        if (shared) {
            b = it % nl;
            li = it / nl;
        } else {
            while (it >= end) {
                ++b;
                beg = end;
                end = __builtin_amdgcn_readfirstlane(first_item(b + 1));
                count = tiles(b);
            }
            li = it - beg;
            if (parts) {
                li += bid % 8 * (end - beg);
                if (li >= count) continue;  // the last part is shorter
            }
        }
        b = __builtin_amdgcn_readfirstlane(b);
        li = __builtin_amdgcn_readfirstlane(li);
        __syncthreads();  // every thread is done with the previous item's tile (and tables)
        if (b != lb) {
            const BLat* L = A.lat + b;
            N = __builtin_amdgcn_readfirstlane(L->N);
            n_chan = __builtin_amdgcn_readfirstlane(L->n_chan);
            n_diag = __builtin_amdgcn_readfirstlane(L->n_diag);
            T = __builtin_amdgcn_readfirstlane(L->low_rows[rc]);
            ks = __builtin_amdgcn_readfirstlane(L->low_sites[rc]);
            chunk = __builtin_amdgcn_readfirstlane(L->chunk[rc]);
            nch = __builtin_amdgcn_readfirstlane(L->n_chunks[rc]);
            n_loc = __builtin_amdgcn_readfirstlane(L->n_local[rc]);
            n_ld = __builtin_amdgcn_readfirstlane(L->n_ldiag[rc]);
            const int64_t xo = L->x_off;
            xb = shared ? X : X + xo;
            yb = Y + xo;
            const int32_t po = L->pool_off, pn = L->pool_n, s0 = L->site_off, t0 = L->term_off, th0 = L->theta_off;
            for (int k = tid; k < pn; k += B) pool[k] = A.pool[po + k];
            site = A.site[s0 + (lane < N ? lane : 0)];
            const int inner = ks + (chunk > 1 ? 1 : 0);  // sites whose digit differs between the tile's rows
            dp = chunk > 1 ? lane_of(site.d, N - 1 - ks) : 1;
            if (tid < N) {
                int sh = 0, w = 0;
                for (int i = N - 1; i >= tid && i >= N - inner; --i) {
                    const int top = i == N - 1 - ks ? chunk : A.site[s0 + i].d;  // digits of the field: below top
                    sh += w;
                    w = 32 - __clz(top - 1);
                }
                field[tid] = tid >= N - inner ? sh | w << 5 : 0;
            }
            __syncthreads();
            for (int r = tid; r < T * chunk; r += B) {
                uint32_t f = r, word = 0;
                for (int i = N - 1; i >= N - ks; --i) {
                    const BSite s = A.site[s0 + i];
                    const uint32_t q = div_by(f, s.by_d);
                    word |= (f - q * static_cast<uint32_t>(s.d)) << (field[i] & 31);
                    f = q;
                }
                if (chunk > 1) word |= f << (field[N - 1 - ks] & 31);
                rw[r] = word;
                float dr = 0.f, di = 0.f;
                for (int k = 0; k < n_ld; ++k) {
                    const BTerm t = A.term[t0 + k];
                    const int fa = field[t.a], fb = t.b >= 0 ? field[t.b] : 0;
                    const float f2 = mul_rn(pool[t.ta + digit_of(word, fa)], pool[t.tb + digit_of(word, fb)]);
                    const float th = theta_all[th0 + t.param];
                    dr = add_rn(dr, mul_rn(mul_rn(th, t.wr), f2));
                    if (CPLX) di = add_rn(di, mul_rn(mul_rn(th, t.wi), f2));
                }
                rd[0][r] = dr;
                if constexpr (CPLX) rd[1][r] = di;
            }
#pragma unroll
            for (int q = 0; q < kSets; ++q) {
                const int k = q * 64 + lane;
                LaneTerms t{};
                t.field = 1 << 21 | 1 << 5;  // a lane without a term reads no factor
                if (k < n_diag + n_chan) {
                    const BTerm g = A.term[t0 + k];
                    t.tab = g.ta | g.tb << 16;
                    t.sites = g.a | (g.b >= 0 ? g.b : g.a) << 8;
                    t.field = field[g.a] | (g.b >= 0 ? field[g.b] << 16 : int(0x80000000u));
                    t.delta = g.delta;
                    t.wr = mul_rn(theta_all[th0 + g.param], g.wr);
                    if (CPLX) t.wi = mul_rn(theta_all[th0 + g.param], g.wi);
                }
                lt[q] = t;
            }
            lb = b;
        }
        const int32_t h = nch > 1 ? li / nch : li, g0 = (li - h * nch) * chunk;
        const int32_t r0 = (chunk > 1 ? h * dp + g0 : h) * T;
        const int32_t nr = (chunk > 1 && dp - g0 < chunk ? dp - g0 : chunk) * T;
        const float2* xr = xb + int64_t(r0) * NV;
        const auto fetch = [&](int32_t rb, float (&w)[NP][PW]) {
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int32_t r = rb + W::row(la, i) < nr ? rb + W::row(la, i) : nr - 1;
                W::load(xr + uint32_t(r * NV + 2 * lp), w[i]);
            }
        };
        const auto put = [&](int32_t rb, const float (&w)[NP][PW]) {
#pragma unroll
            for (int i = 0; i < NP; ++i) {  // rows beyond the last one repeat it
                const int32_t r = rb + W::row(la, i) < nr ? rb + W::row(la, i) : nr - 1;
#pragma unroll
                for (int e = 0; e < PW / 2; ++e) xt[2 * lp + e][r] = make_float2(w[i][2 * e], w[i][2 * e + 1]);
            }
        };
        const int32_t wave0 = __builtin_amdgcn_readfirstlane(tid - lane);
        float w0[NP][PW];
        if (wave0 < nr) fetch(wave0, w0);
        // the tile's first row: lane i its digit at site i, then every lane its terms
        const uint32_t qm = div_by(r0, site.by_m), qd = div_by(r0, site.by_md);
        const int dig = static_cast<int>(qm - qd * static_cast<uint32_t>(site.d));
        uint64_t todo[kSets], dtodo[kSets], uni[kSets];  // gathers, diagonal terms, terms without a digit in the tile
#pragma unroll
        for (int q = 0; q < kSets; ++q) {
            todo[q] = dtodo[q] = uni[q] = 0;
            if (q * 64 >= n_diag + n_chan) continue;
            LaneTerms& t = lt[q];
            const int k = q * 64 + lane;
            const int da = __shfl(dig, t.sites & 255, 64), db = __shfl(dig, t.sites >> 8, 64);
            t.at = t.tab + (t.field < 0 ? da : da | db << 16);
            const int wa = t.field >> 5 & 15, wb = t.field >> 21 & 15;
            const float f1 = wa ? 1.f : pool[t.at & 0xffff], f2 = wb ? 1.f : pool[t.at >> 16];
            const float f = mul_rn(f1, f2);
            t.vr = mul_rn(t.wr, f);
            if (CPLX) t.vi = mul_rn(t.wi, f);
            const bool on = f != 0.f;  // else a source digit above the tile is out of range (App. A)
            uni[q] = __ballot(!(wa | wb));
            dtodo[q] = __ballot(k >= n_ld && k < n_diag);
            todo[q] = __ballot(on && k >= n_diag + n_loc && k < n_diag + n_chan);
        }
        if (wave0 < nr) put(wave0, w0);
        for (int32_t rb = wave0 + B; rb < nr; rb += B) {
            fetch(rb, w0);
            put(rb, w0);
        }
        __syncthreads();
        // whole waves (terms are read across lanes); lanes beyond the last row repeat it
        for (int32_t rb = wave0; rb < nr; rb += B) {
            const int32_t r = rb + lrow < nr ? rb + lrow : nr - 1;
            int32_t pr[NP];  // by pieces: rows of the lane
#pragma unroll
            for (int i = 0; i < NP; ++i) pr[i] = rb + W::row(la, i) < nr ? rb + W::row(la, i) : nr - 1;
            const uint32_t word = rw[r];
            const auto factor = [&](int at, int field) {  // of a term at this row
                return mul_rn(pool[(at & 0xffff) + digit_of(word, field & 0xffff)],
                                 pool[(at >> 16) + digit_of(word, field >> 16 & 0x7fff)]);
            };
            const auto factor_of = [&](const LaneTerms& t, int k) { return factor(lane_of(t.at, k), lane_of(t.field, k)); };
            uint64_t left[kSets];
#pragma unroll
            for (int q = 0; q < kSets; ++q) left[q] = todo[q];
            float v[kBatchGather][NP][PW], acc[NP][PW];
            float cr[kBatchGather], ci[kBatchGather];  // by rows
            static_assert(kSets <= kBatchTermSets && kBatchTermSets == 2, "the last set is the first or the second");
            {
                // diagonal: the low digits' sum, then the other terms
                float ar[NV], ai[NV];
                const auto add = [&](float c, float d, float2 s, int q) {
                    ar[q] = fmaf(c, s.x, ar[q]);
                    ai[q] = fmaf(c, s.y, ai[q]);
                    if (CPLX) {
                        ar[q] = fmaf(-d, s.y, ar[q]);
                        ai[q] = fmaf(d, s.x, ai[q]);
                    }
                };
                float dr = rd[0][r], di = CPLX ? rd[CPLX ? 1 : 0][r] : 0.f;
#pragma unroll
                for (int q = 0; q < kSets; ++q)
                    for (uint64_t m = dtodo[q]; m; m &= m - 1) {
                        const int k = __builtin_ctzll(m);
                        float er = lane_of(lt[q].vr, k), ei = CPLX ? lane_of(lt[q].vi, k) : 0.f;
                        if (!(uni[q] >> k & 1)) {
                            const float f = factor_of(lt[q], k);
                            er = mul_rn(lane_of(lt[q].wr, k), f);
                            ei = CPLX ? mul_rn(lane_of(lt[q].wi, k), f) : 0.f;
                        }
                        dr = add_rn(dr, er);
                        if (CPLX) di = add_rn(di, ei);
                    }
#pragma unroll
                for (int q = 0; q < NV; ++q) {
                    const float2 s = xt[q][r];
                    ar[q] = mul_rn(dr, s.x);
                    ai[q] = mul_rn(dr, s.y);
                    if (CPLX) {
                        ar[q] = fmaf(-di, s.y, ar[q]);
                        ai[q] = fmaf(di, s.x, ai[q]);
                    }
                }
                // channels whose sites both lie among the low ones (the first n_loc): the source row is in LDS
                // (Eq. sourceoffset); an inadmissible source reads the row itself with coefficient 0
#pragma unroll
                for (int q = 0; q < kSets; ++q) {
                    const int k0 = q * 64 > n_diag ? q * 64 : n_diag;
                    const int k1 = (q + 1) * 64 < n_diag + n_loc ? (q + 1) * 64 : n_diag + n_loc;
                    float next = k0 < k1 ? factor_of(lt[q], k0 & 63) : 0.f;
#pragma unroll 1
                    for (int k = k0; k < k1; ++k) {
                        const float f = next;
                        if (k + 1 < k1) next = factor_of(lt[q], k + 1 & 63);  // under way during this term
                        const bool in = f != 0.f;
                        const float c = in ? mul_rn(lane_of(lt[q].wr, k & 63), f) : 0.f;
                        const float d = CPLX && in ? mul_rn(lane_of(lt[q].wi, k & 63), f) : 0.f;
                        const int32_t rs = in ? r - lane_of(lt[q].delta, k & 63) : r;
#pragma unroll
                        for (int e = 0; e < NV; ++e) add(c, d, xt[e][rs], e);
                    }
                }
#pragma unroll
                for (int p = 0; p < NP; ++p)
#pragma unroll
                    for (int e = 0; e < PW; ++e) acc[p][e] = e & 1 ? ai[2 * p + e / 2] : ar[2 * p + e / 2];
                W::transpose(acc, lane);
            }
            while (left[0] | left[kSets - 1]) {
                // the next gathers of the list, in its order
                int have = 0;
#pragma unroll
                for (int u = 0; u < kBatchGather; ++u) {
                    constexpr int kLast = kSets - 1;
                    const bool z = kSets == 1 || left[0] != 0;
                    const uint64_t m = z ? left[0] : left[kLast];
                    if (m == 0) continue;
                    const int k = __builtin_ctzll(m);
                    if (z) left[0] = m & (m - 1);
                    else left[kLast] = m & (m - 1);
                    const auto pick = [&](auto x) {
                        if constexpr (kSets == 1) return lane_of(x(lt[0]), k);
                        else return z ? lane_of(x(lt[0]), k) : lane_of(x(lt[kLast]), k);
                    };
#define MRMF_OF(field) pick([](const LaneTerms& t) { return t.field; })
                    const int delta = MRMF_OF(delta);
                    if ((z ? uni[0] : uni[kLast]) >> k & 1) {
                        const float2* src = xb + (int64_t(r0) - delta) * NV;
                        cr[u] = MRMF_OF(vr);
                        ci[u] = CPLX ? MRMF_OF(vi) : 0.f;
#pragma unroll
                        for (int i = 0; i < NP; ++i) W::load(src + uint32_t(pr[i] * NV + 2 * lp), v[u][i]);
                    } else {  // an inadmissible source reads the row itself with coefficient 0
                        const float f = factor(MRMF_OF(at), MRMF_OF(field));
                        const bool in = f != 0.f;
                        cr[u] = in ? mul_rn(MRMF_OF(wr), f) : 0.f;
                        ci[u] = CPLX && in ? mul_rn(MRMF_OF(wi), f) : 0.f;
                        const int off = in ? delta : 0;
                        each<NP>([&](auto I) {
                            const int64_t row = int64_t(r0) + pr[I] - W::template from<I>(off);
                            W::load(xb + row * NV + 2 * lp, v[u][I]);
                        });
                    }
                    have = u + 1;
#undef MRMF_OF
                }
#pragma unroll
                for (int u = 0; u < kBatchGather; ++u)
                    if (u < have) {
                        each<NP>([&](auto I) {
                            constexpr int i = I;
                            const float c = __int_as_float(W::template from<i>(__float_as_int(cr[u])));
                            const float d = CPLX ? __int_as_float(W::template from<i>(__float_as_int(ci[u]))) : 0.f;
#pragma unroll
                            for (int e = 0; e < PW; e += 2) {
                                acc[i][e] = fmaf(c, v[u][i][e], acc[i][e]);
                                acc[i][e + 1] = fmaf(c, v[u][i][e + 1], acc[i][e + 1]);
                                if (CPLX) {
                                    acc[i][e] = fmaf(-d, v[u][i][e + 1], acc[i][e]);
                                    acc[i][e + 1] = fmaf(d, v[u][i][e], acc[i][e + 1]);
                                }
                            }
                        });
                    }
            }
#pragma unroll
            for (int i = 0; i < NP; ++i)
                if (rb + W::row(la, i) < nr) W::store(yb + int64_t(r0 + pr[i]) * NV + 2 * lp, acc[i], !shared);
        }
    }
}

// Linear combination of parameter-group products: Y_k[i] = sum_p theta[k][p] G_p[i] for k < K, i < n (c64
// entries, real couplings).  A thread holds the P entries G_p[i] of its element in registers and writes
// every Y_k[i]; the couplings of the sweep sit in LDS.  Bound by the writes of the K outputs.
constexpr int kCombMaxP = 16;
constexpr int kCombTheta = 4096;  // couplings held in LDS at a time (16 KB)
constexpr int kCombBlock = 256;

template <int P>
__global__ __launch_bounds__(kCombBlock) void k_sweep_combine(const float* __restrict__ theta, int32_t K,
                                                              int64_t n, const float2* __restrict__ G,
                                                              int64_t g_stride, float2* __restrict__ Y,
                                                              int64_t y_stride) {
    __shared__ float th[kCombTheta];  // a chunk of the sweep's couplings, rows of P
    const int64_t i = int64_t(blockIdx.x) * kCombBlock + threadIdx.x;
    float2 g[P];
#pragma unroll
    for (int p = 0; p < P; ++p) g[p] = i < n ? G[p * g_stride + i] : make_float2(0.f, 0.f);
    const int kc = kCombTheta / P;  // sweep rows per chunk
    for (int k0 = 0; k0 < K; k0 += kc) {
        const int kn = K - k0 < kc ? K - k0 : kc;
        __syncthreads();
        for (int e = threadIdx.x; e < kn * P; e += kCombBlock) th[e] = theta[int64_t(k0) * P + e];
        __syncthreads();
        if (i < n)
            for (int k = 0; k < kn; ++k) {
                float yr = 0.f, yi = 0.f;
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    const float t = th[k * P + p];
                    yr += t * g[p].x;
                    yi += t * g[p].y;
                }
                Y[(k0 + k) * y_stride + i] = make_float2(yr, yi);
            }
    }
}

template <int P>
void launch_combine(const float* theta, int32_t K, int64_t n, const float2* G, int64_t gs, float2* Y, int64_t ys,
                    hipStream_t s) {
    const int64_t grid = (n + kCombBlock - 1) / kCombBlock;
    hipLaunchKernelGGL(k_sweep_combine<P>, dim3(static_cast<unsigned>(grid)), dim3(kCombBlock), 0, s, theta, K, n,
                       G, gs, Y, ys);
}

template <int NV>
void* batch_kernel_ptr(bool cplx, bool many) {
    if (many) return cplx ? reinterpret_cast<void*>(&k_batch<NV, true, 2>) : reinterpret_cast<void*>(&k_batch<NV, false, 2>);
    return cplx ? reinterpret_cast<void*>(&k_batch<NV, true, 1>) : reinterpret_cast<void*>(&k_batch<NV, false, 1>);
}

// many: a lattice of more than 64 terms
void* batch_kernel(int nvec, bool cplx, bool many) {
    switch (nvec) {
        case 1: return batch_kernel_ptr<1>(cplx, many);
        case 2: return batch_kernel_ptr<2>(cplx, many);
        case 4: return batch_kernel_ptr<4>(cplx, many);
        default: return batch_kernel_ptr<8>(cplx, many);
    }
}

// Factor table <n|O|n - q> at target digit n (0 where the source digit n - q is outside 0..d-1).
void factor_table(const mrmf_plan_t* p, int site, int op, std::vector<float>& out) {
    for (int n = 0; n < p->d[site]; ++n) out.push_back(static_cast<float>(local_factor_host(p, site, op, n)));
}

// Launch shapes tried by the autotuner: (R_max candidate index, block threads).  The last two are for one and two
// vectors, whose smallest tiles have 512 and 256 rows: eight rings of 7 spins 1, one vector, 21.4 -> 12.2 us.
struct Shape {
    int32_t rc, block;
};
const Shape kShapes[] = {{1, 128}, {2, 128}, {2, 256}, {3, 256}, {3, 512}, {0, 64}, {1, 256}, {0, 128}, {0, 256}, {0, 512}};
constexpr int kNumShapes = sizeof(kShapes) / sizeof(kShapes[0]);

BDiv div_of(int64_t m) {  // 1 <= m < 2^30
    BDiv v{0, 0};
    while ((int64_t(1) << v.shift) < m) ++v.shift;
    v.mul = static_cast<uint32_t>(((uint64_t(1) << (31 + v.shift)) + m - 1) / m);
    return v;
}

int32_t rmax_of(int rc, int nvec) { return (64 << rc) * 8 / nvec; }

// Launch shape until one is set, from the rows of all lattices: one row a thread in tiles of 256 rows (one vector: 512, the
// smallest there is), of 128 (eight vectors) up to 131072 rows and of the smallest size below 40960, where larger tiles
// leave the GPU short of them.  us, against tiles of 2048 / nvec rows for 256 threads: eight rings of 7 spins 1 (17496
// rows) 1 vector 12.2 (39.0), 4 vectors 9.8 (18.3), 8 vectors 10.4 (11.6); eight rings of 7 spins 3/2 (131072) 12.3 (52.0),
// 10.8 (16.5), 12.7 (15.0); eight rings of 12 spins 1/2 and 1 (373248) 27.9 (57.3), 26.5 (31.3), 29.1; the group products
// of nine spins 1 (59049) 8 vectors 9.4, in the smallest tiles 13.2.  From 2^22 rows on a thread's several rows cost less
// than more tiles (29 million, 4 vectors: 1801 against 1877 us).
Shape default_shape(int64_t rows, int nvec) {
    if (rows >= int64_t(1) << 22) return {2, 256};
    const int least = 512 / nvec;
    const int tile = rows < 160 * 256 ? least : std::max(least, nvec == 8 && rows <= 131072 ? 128 : 256);
    int rc = 0;
    while (rmax_of(rc, nvec) < tile) ++rc;
    return {rc, tile};
}

}  // namespace
}  // namespace mrmf

struct mrmf_batch_t {
    int32_t n = 0, nvec = 0;
    std::vector<int64_t> off;      // element offset of each lattice's block
    std::vector<int32_t> th_off;   // n + 1
    int64_t total = 0;             // elements, padded
    bool all_real = true;
    int32_t max_terms = 0, max_pool = 0;  // of a lattice
    std::vector<unsigned char> image;
    size_t off_lat = 0, off_site = 0, off_term = 0, off_pool = 0, ws_bytes = 0;
    int32_t rc = 0, block = 0;  // R_max candidate index and block threads
    int32_t sched = 0;            // MRMF_BATCH_SCHED_*
    int32_t grid = 0;
    bool shared = false;                     // mrmf_batch_share_input
    std::vector<std::vector<int32_t>> dims;  // local dimensions of each lattice
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    ~mrmf_batch_t() {
        if (exec) hipGraphExecDestroy(exec);
        if (graph) hipGraphDestroy(graph);
    }
};

namespace {

mrmf::BatchArgs batch_args(const mrmf_batch_t* b, const void* d_ws) {
    const unsigned char* w = static_cast<const unsigned char*>(d_ws);
    mrmf::BatchArgs a;
    a.lat = reinterpret_cast<const mrmf::BLat*>(w + b->off_lat);
    a.site = reinterpret_cast<const mrmf::BSite*>(w + b->off_site);
    a.term = reinterpret_cast<const mrmf::BTerm*>(w + b->off_term);
    a.pool = reinterpret_cast<const float*>(w + b->off_pool);
    a.n_lat = b->n;
    a.shared = b->shared ? 1 : 0;
    return a;
}

int batch_grid(const mrmf_batch_t* b) {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess) hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    // resident blocks per CU: 16 waves (four per SIMD at 128 registers), 160 KB of LDS
    const int rows = mrmf::kBatchTileWords / b->nvec;
    const int lds = mrmf::kBatchTileWords * 8 + 4 * (b->all_real ? 2 : 3) * rows + 1024 + 4 * b->max_pool;
    const int per_cu = std::max(1, std::min(16 * 64 / b->block, 163840 / lds));
    return cus * per_cu;
}

mrmf_status launch(mrmf_batch_t* b, const void* d_ws, const float* theta, const void* X, void* Y, hipStream_t s) {
    const mrmf::BatchArgs a = batch_args(b, d_ws);
    void* fn = mrmf::batch_kernel(b->nvec, !b->all_real, b->max_terms > 64);
    const int grid = batch_grid(b);
    b->grid = grid;
    int32_t rc = b->rc, sched = b->sched;
    const float2* xp = static_cast<const float2*>(X);
    float2* yp = static_cast<float2*>(Y);
    void* args[] = {const_cast<mrmf::BatchArgs*>(&a), &theta, &xp, &yp, &rc, &sched};
    return mrmf::hip_status(hipLaunchKernel(fn, dim3(grid), dim3(b->block), args, 4 * size_t(b->max_pool), s));
}

mrmf_status check_call(const mrmf_batch_t* b, const void* d_ws, const float* th, const void* X, const void* Y) {
    if (!b || !d_ws || !th || !X || !Y) return MRMF_E_INVALID_ARG;
    const size_t al = b->nvec >= 2 ? 16 : 8;  // rows are moved in 16-byte words when they hold two or more
    if (!mrmf::aligned(d_ws, 256) || !mrmf::aligned(X, al) || !mrmf::aligned(Y, al)) return MRMF_E_INVALID_ARG;
    const size_t bytes = size_t(b->total) * 8;
    const size_t x_bytes = b->shared ? size_t(b->off.size() > 1 ? b->off[1] : b->total) * 8 : bytes;
    if (mrmf::ranges_overlap(X, x_bytes, Y, bytes)) return MRMF_E_INVALID_ARG;
    return MRMF_OK;
}

// groups: lattice i keeps the terms of coupling i alone
mrmf_status create(int32_t n, const mrmf_plan* plans, int32_t nvec, bool groups, mrmf_batch* out) {
    using namespace mrmf;
    if (!out) return MRMF_E_INVALID_ARG;
    *out = nullptr;
    if (n < 1 || n > kBatchMaxLattices || !plans) return MRMF_E_INVALID_ARG;
    if (nvec != 1 && nvec != 2 && nvec != 4 && nvec != 8) return MRMF_E_INVALID_ARG;
    auto* b = new (std::nothrow) mrmf_batch_t();
    if (!b) return MRMF_E_INVALID_ARG;
    b->n = n;
    b->nvec = nvec;
    std::vector<BLat> lats(n + 1);  // the last one holds the item counts
    std::vector<BSite> sites;
    std::vector<BTerm> terms;
    std::vector<float> pool;
    int64_t off = 0, items[kBatchRmaxCands] = {}, parts[kBatchRmaxCands] = {};
    int32_t th = 0;
    for (int i = 0; i < n; ++i) {
        const mrmf_plan_t* p = plans[i];
        if (!p || p->N > kBatchMaxSites || p->D >= (int64_t(1) << 31) / 2 / nvec || p->n_params > kBatchMaxParams ||
            p->chans.size() + p->diags.size() > size_t(kBatchMaxTerms)) {
            delete b;
            return p ? MRMF_E_UNSUPPORTED : MRMF_E_INVALID_ARG;
        }
        BLat& L = lats[i];
        for (int rc = 0; rc < kBatchRmaxCands; ++rc) {  // tiles spanned by the low sites, <= R_max rows
            const int64_t rmax = rmax_of(rc, nvec);
            int64_t T = 1;
            int k = 0;
            while (k < p->N && T * p->d[p->N - 1 - k] <= rmax) T *= p->d[p->N - 1 - k++];
            L.low_rows[rc] = static_cast<int32_t>(T);
            L.low_sites[rc] = k;
            const int64_t d = k < p->N ? p->d[p->N - 1 - k] : 1, most = rmax / T;
            const int64_t nch = most >= 2 ? (d + most - 1) / most : d;
            L.chunk[rc] = most >= 2 ? static_cast<int32_t>((d + nch - 1) / nch) : 1;
            L.n_chunks[rc] = L.chunk[rc] > 1 ? static_cast<int32_t>(nch) : 1;
            L.item_beg[rc] = static_cast<int32_t>(items[rc]);
            const int64_t own = L.chunk[rc] > 1 ? p->D / (T * d) * nch : p->D / T;
            items[rc] += own;
            L.part_beg[rc] = static_cast<int32_t>(parts[rc]);
            parts[rc] += (own + 7) / 8;
        }
        b->dims.emplace_back(p->d.begin(), p->d.end());
        L.N = p->N;
        L.theta_off = th;
        L.x_off = off;
        L.site_off = static_cast<int32_t>(sites.size());
        for (int s = 0; s < p->N; ++s) {
            BSite bs{};
            bs.d = p->d[s];
            bs.by_d = div_of(p->d[s]);
            bs.by_m = div_of(p->M[s]);
            bs.by_md = div_of(p->M[s] * p->d[s]);
            sites.push_back(bs);
        }
        // factor pool of this lattice: entry 0 is 1.0 (second factor of a one-site term)
        std::vector<float> lp{1.0f};
        auto table = [&](int s, int op) {
            const int at = static_cast<int>(lp.size());
            factor_table(p, s, op, lp);
            return at;
        };
        auto add_term = [&](int a, int opa, int bsite, int opb, int param, double wr, double wi, int64_t delta) {
            BTerm t{};
            t.a = a;
            t.ta = table(a, opa);
            t.b = bsite;
            t.tb = bsite >= 0 ? table(bsite, opb) : 0;
            t.param = param;
            t.delta = static_cast<int32_t>(delta);
            t.low = p->N - (bsite >= 0 && bsite < a ? bsite : a);
            t.wr = static_cast<float>(wr);
            t.wi = static_cast<float>(wi);
            if (wi != 0.0) b->all_real = false;
            terms.push_back(t);
        };
        const size_t t0 = terms.size();
        L.term_off = static_cast<int32_t>(t0);
        for (const auto& g : p->diags)
            if (!groups || g.param == i) add_term(g.a, g.opa, g.b, g.opb, g.param, g.wr, g.wi, 0);
        const size_t t1 = terms.size();
        L.n_diag = static_cast<int32_t>(t1 - t0);
        for (const auto& c : p->chans)
            if (!groups || c.param == i) add_term(c.a, c.opa, c.b, c.opb, c.param, c.wr, c.wi, c.delta);
        L.n_chan = static_cast<int32_t>(terms.size() - t1);
        b->max_terms = std::max(b->max_terms, L.n_diag + L.n_chan);
        // by the number of low sites a tile must span (stable), so that for every tile size the diagonal terms of the
        // low digits and the channels whose source lies in the tile are prefixes of their lists
        const auto by_low = [](const BTerm& u, const BTerm& v) { return u.low < v.low; };
        std::stable_sort(terms.begin() + t0, terms.begin() + t1, by_low);
        std::stable_sort(terms.begin() + t1, terms.end(), by_low);
        for (int rc = 0; rc < kBatchRmaxCands; ++rc) {
            L.n_ldiag[rc] = L.n_local[rc] = 0;
            for (size_t k = t0; k < terms.size(); ++k)
                if (terms[k].low <= L.low_sites[rc]) ++(k < t1 ? L.n_ldiag[rc] : L.n_local[rc]);
        }
        if (lp.size() > size_t(kBatchPoolMax)) {
            delete b;
            return MRMF_E_UNSUPPORTED;
        }
        L.pool_off = static_cast<int32_t>(pool.size());
        L.pool_n = static_cast<int32_t>(lp.size());
        b->max_pool = std::max(b->max_pool, L.pool_n);
        pool.insert(pool.end(), lp.begin(), lp.end());
        b->off.push_back(off);
        b->th_off.push_back(th);
        off += (p->D * nvec + 31) / 32 * 32;
        th += p->n_params;
    }
    b->th_off.push_back(th);
    b->total = off;
    int64_t rows = 0;
    for (int i = 0; i < n; ++i) rows += plans[i]->D;
    const Shape shape = default_shape(rows, nvec);
    b->rc = shape.rc;
    b->block = shape.block;
    for (int rc = 0; rc < kBatchRmaxCands; ++rc) {
        if (items[rc] >= (int64_t(1) << 30)) {  // more rows than any memory holds
            delete b;
            return MRMF_E_OVERFLOW;
        }
        lats[n].item_beg[rc] = static_cast<int32_t>(items[rc]);
        lats[n].part_beg[rc] = static_cast<int32_t>(parts[rc]);
    }
    if (off * 8 >= (int64_t(1) << 62)) {
        delete b;
        return MRMF_E_OVERFLOW;
    }
    size_t o = 0;
    b->off_lat = o;
    o = align_up(o + sizeof(BLat) * lats.size(), 256);
    b->off_site = o;
    o = align_up(o + sizeof(BSite) * sites.size(), 256);
    b->off_term = o;
    o = align_up(o + sizeof(BTerm) * std::max<size_t>(1, terms.size()), 256);
    b->off_pool = o;
    o = align_up(o + sizeof(float) * pool.size(), 256);
    b->ws_bytes = o;
    b->image.assign(o, 0);
    std::memcpy(b->image.data() + b->off_lat, lats.data(), sizeof(BLat) * lats.size());
    std::memcpy(b->image.data() + b->off_site, sites.data(), sizeof(BSite) * sites.size());
    if (!terms.empty()) std::memcpy(b->image.data() + b->off_term, terms.data(), sizeof(BTerm) * terms.size());
    std::memcpy(b->image.data() + b->off_pool, pool.data(), sizeof(float) * pool.size());
    *out = b;
    return MRMF_OK;
}

}  // namespace

extern "C" {

mrmf_status mrmf_batch_create(int32_t n, const mrmf_plan* plans, int32_t nvec, mrmf_batch* out) {
    return create(n, plans, nvec, false, out);
}

mrmf_status mrmf_batch_create_groups(mrmf_plan plan, int32_t nvec, mrmf_batch* out) {
    if (!plan || !out) return MRMF_E_INVALID_ARG;
    *out = nullptr;
    if (plan->n_params < 1 || plan->n_params > mrmf::kBatchMaxParams) return MRMF_E_UNSUPPORTED;
    const std::vector<mrmf_plan> plans(plan->n_params, plan);
    const mrmf_status st = create(plan->n_params, plans.data(), nvec, true, out);
    return st == MRMF_OK ? mrmf_batch_share_input(*out, 1) : st;
}

void mrmf_batch_destroy(mrmf_batch batch) { delete batch; }

mrmf_status mrmf_batch_total_elems(mrmf_batch b, int64_t* elems) {
    if (!b || !elems) return MRMF_E_INVALID_ARG;
    *elems = b->total;
    return MRMF_OK;
}

mrmf_status mrmf_batch_offsets(mrmf_batch b, int64_t* out) {
    if (!b || !out) return MRMF_E_INVALID_ARG;
    std::memcpy(out, b->off.data(), sizeof(int64_t) * b->n);
    return MRMF_OK;
}

mrmf_status mrmf_batch_theta_offsets(mrmf_batch b, int32_t* out) {
    if (!b || !out) return MRMF_E_INVALID_ARG;
    std::memcpy(out, b->th_off.data(), sizeof(int32_t) * (b->n + 1));
    return MRMF_OK;
}

mrmf_status mrmf_batch_workspace_bytes(mrmf_batch b, size_t* bytes) {
    if (!b || !bytes) return MRMF_E_INVALID_ARG;
    *bytes = b->ws_bytes;
    return MRMF_OK;
}

mrmf_status mrmf_batch_upload(mrmf_batch b, void* d_ws, size_t ws_bytes, mrmf_stream stream) {
    if (!b || !d_ws || !mrmf::aligned(d_ws, 256)) return MRMF_E_INVALID_ARG;
    if (ws_bytes < b->ws_bytes) return MRMF_E_WORKSPACE;
    return mrmf::hip_status(hipMemcpyAsync(d_ws, b->image.data(), b->ws_bytes, hipMemcpyHostToDevice,
                                           static_cast<hipStream_t>(stream)));
}

mrmf_status mrmf_batch_matvec_c(mrmf_batch b, const void* d_ws, const float* d_theta_all, const void* d_X,
                                void* d_Y, mrmf_stream stream) {
    const mrmf_status st = check_call(b, d_ws, d_theta_all, d_X, d_Y);
    if (st != MRMF_OK) return st;
    return launch(b, d_ws, d_theta_all, d_X, d_Y, static_cast<hipStream_t>(stream));
}

mrmf_status mrmf_batch_graph_capture(mrmf_batch b, const void* d_ws, const float* d_theta_all, const void* d_X,
                                     void* d_Y, mrmf_stream stream) {
    mrmf_status st = check_call(b, d_ws, d_theta_all, d_X, d_Y);
    if (st != MRMF_OK) return st;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    if (b->exec) {
        hipGraphExecDestroy(b->exec);
        b->exec = nullptr;
    }
    if (b->graph) {
        hipGraphDestroy(b->graph);
        b->graph = nullptr;
    }
    if (hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal) != hipSuccess) return MRMF_E_HIP;
    st = launch(b, d_ws, d_theta_all, d_X, d_Y, s);
    hipGraph_t g = nullptr;
    const hipError_t e = hipStreamEndCapture(s, &g);
    if (st != MRMF_OK || e != hipSuccess || !g) {
        if (g) hipGraphDestroy(g);
        return st != MRMF_OK ? st : MRMF_E_HIP;
    }
    hipGraphExec_t ex = nullptr;
    if (hipGraphInstantiate(&ex, g, nullptr, nullptr, 0) != hipSuccess) {
        hipGraphDestroy(g);
        return MRMF_E_HIP;
    }
    b->graph = g;
    b->exec = ex;
    return MRMF_OK;
}

mrmf_status mrmf_batch_graph_launch(mrmf_batch b, mrmf_stream stream) {
    if (!b || !b->exec) return MRMF_E_INVALID_ARG;
    return mrmf::hip_status(hipGraphLaunch(b->exec, static_cast<hipStream_t>(stream)));
}

mrmf_status mrmf_batch_share_input(mrmf_batch b, int32_t on) {
    if (!b || (on != 0 && on != 1)) return MRMF_E_INVALID_ARG;
    if (on)
        for (const auto& d : b->dims)
            if (d != b->dims[0]) return MRMF_E_UNSUPPORTED;
    b->shared = on != 0;
    return MRMF_OK;
}

mrmf_status mrmf_sweep_combine_c(const float* d_theta, int32_t K, int32_t P, int64_t n, const void* d_G,
                                 int64_t g_stride, void* d_Y, int64_t y_stride, mrmf_stream stream) {
    using namespace mrmf;
    if (!d_theta || !d_G || !d_Y || K < 1 || P < 1 || P > kCombMaxP || n < 1 || g_stride < n || y_stride < n)
        return MRMF_E_INVALID_ARG;
    if (n >= (int64_t(1) << 31) * kCombBlock) return MRMF_E_INVALID_ARG;
    if (!aligned(d_G, 8) || !aligned(d_Y, 8) || !aligned(d_theta, 4)) return MRMF_E_INVALID_ARG;
    const size_t gb = size_t(g_stride) * (P - 1) * 8 + size_t(n) * 8, yb = size_t(y_stride) * (K - 1) * 8 + size_t(n) * 8;
    if (ranges_overlap(d_G, gb, d_Y, yb)) return MRMF_E_INVALID_ARG;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    const auto* G = static_cast<const float2*>(d_G);
    auto* Y = static_cast<float2*>(d_Y);
    switch (P) {
#define MRMF_COMB_CASE(q) \
    case q: launch_combine<q>(d_theta, K, n, G, g_stride, Y, y_stride, s); break;
        MRMF_COMB_CASE(1) MRMF_COMB_CASE(2) MRMF_COMB_CASE(3) MRMF_COMB_CASE(4) MRMF_COMB_CASE(5) MRMF_COMB_CASE(6)
        MRMF_COMB_CASE(7) MRMF_COMB_CASE(8) MRMF_COMB_CASE(9) MRMF_COMB_CASE(10) MRMF_COMB_CASE(11)
        MRMF_COMB_CASE(12) MRMF_COMB_CASE(13) MRMF_COMB_CASE(14) MRMF_COMB_CASE(15) MRMF_COMB_CASE(16)
#undef MRMF_COMB_CASE
        default: return MRMF_E_INVALID_ARG;
    }
    return launch_status();
}

mrmf_status mrmf_batch_set_shape(mrmf_batch b, int32_t tile_rows_max, int32_t block_threads) {
    if (!b || block_threads < 64 || block_threads > mrmf::kBatchMaxBlock || block_threads % 64 != 0 ||
        block_threads > mrmf::kBatchTileWords / b->nvec)
        return MRMF_E_INVALID_ARG;
    int rc = -1;
    for (int k = 0; k < mrmf::kBatchRmaxCands; ++k)
        if (mrmf::rmax_of(k, b->nvec) == tile_rows_max) rc = k;
    if (rc < 0) return MRMF_E_INVALID_ARG;
    b->rc = rc;
    b->block = block_threads;
    return MRMF_OK;
}

mrmf_status mrmf_batch_set_schedule(mrmf_batch b, int32_t sched) {
    if (!b || (sched != MRMF_BATCH_SCHED_RUNS && sched != MRMF_BATCH_SCHED_WINDOWS &&
               sched != MRMF_BATCH_SCHED_XCD_CHUNK))
        return MRMF_E_INVALID_ARG;
    b->sched = sched;
    return MRMF_OK;
}

mrmf_status mrmf_batch_get_shape(mrmf_batch b, int32_t* out) {
    if (!b || !out) return MRMF_E_INVALID_ARG;
    out[0] = mrmf::rmax_of(b->rc, b->nvec);
    out[1] = b->block;
    out[2] = b->sched;
    out[3] = batch_grid(b);
    return MRMF_OK;
}

mrmf_status mrmf_batch_autotune(mrmf_batch b, const void* d_ws, const float* d_theta_all, const void* d_X,
                                void* d_Y, mrmf_stream stream, int32_t* out) {
    mrmf_status st = check_call(b, d_ws, d_theta_all, d_X, d_Y);
    if (st != MRMF_OK) return st;
    if (!out) return MRMF_E_INVALID_ARG;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return MRMF_E_HIP;
    if (hipEventCreate(&e1) != hipSuccess) {
        hipEventDestroy(e0);
        return MRMF_E_HIP;
    }
    float best = 0.f;
    int best_i = -1;
    const int32_t R0 = b->rc, B0 = b->block, S0 = b->sched;
    // candidates: every shape with the runs schedule, then with the windows schedule, then per-XCD chunks
    for (int i = 0; i < 3 * mrmf::kNumShapes && st == MRMF_OK; ++i) {
        b->rc = mrmf::kShapes[i % mrmf::kNumShapes].rc;
        b->block = mrmf::kShapes[i % mrmf::kNumShapes].block;
        b->sched = i / mrmf::kNumShapes;
        if (b->block > mrmf::kBatchTileWords / b->nvec || b->block > 2 * mrmf::rmax_of(b->rc, b->nvec)) continue;
        st = launch(b, d_ws, d_theta_all, d_X, d_Y, s);  // warm-up
        if (st != MRMF_OK) break;
        hipEventRecord(e0, s);
        for (int r = 0; r < 3 && st == MRMF_OK; ++r) st = launch(b, d_ws, d_theta_all, d_X, d_Y, s);
        hipEventRecord(e1, s);
        if (hipEventSynchronize(e1) != hipSuccess) st = MRMF_E_HIP;
        float ms = 0.f;
        hipEventElapsedTime(&ms, e0, e1);
        if (st == MRMF_OK && (best_i < 0 || ms < best)) {
            best = ms;
            best_i = i;
        }
    }
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    if (best_i < 0) {
        b->rc = R0;
        b->block = B0;
        b->sched = S0;
        return st != MRMF_OK ? st : MRMF_E_HIP;
    }
    b->rc = mrmf::kShapes[best_i % mrmf::kNumShapes].rc;
    b->block = mrmf::kShapes[best_i % mrmf::kNumShapes].block;
    b->sched = best_i / mrmf::kNumShapes;
    out[0] = mrmf::rmax_of(b->rc, b->nvec);
    out[1] = b->block;
    out[2] = best_i;
    return st;
}

}  // extern "C"
