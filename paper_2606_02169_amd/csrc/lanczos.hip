// Device-resident Lanczos eigensolver driving the matrix-free map (the Krylov use of x -> H x, Sec. I)
// and the FP64 vector reductions it needs.  Every scalar of the recurrence (alpha_j, beta_j, the Gram-
// Schmidt coefficients, the Ritz value) stays in device memory; the host only enqueues kernels.  After a
// breakdown every later kernel of the call sees its step's halt flag and returns at once.
#include <algorithm>
#include <cmath>
#include <cstddef>
#include <type_traits>

#include "mrmf_internal.h"
#include "reduce.h"

namespace mrmf {
namespace {

constexpr int kRB = 256;            // threads per reduction block
constexpr int kMaxRedBlocks = 512;  // first-stage partials per reduction
constexpr int kGroup = 8;           // basis vectors per Gram-Schmidt block

// Rounding.  The order of every sum here is part of the result: the rows of a thread in turn, the lanes of a wave as a
// tree, the waves, then the blocks' partials one after the other.  The sign of the Ritz vector follows from the last
// bits of alpha and beta (inverse iteration with a shift that equals the eigenvalue to the last bit), so another order
// would turn it on some inputs.

// Scalars of a call.  `halt` (one flag per step, in the scratch after this struct) says whether step j runs at
// all: the kernel that ends step j writes halt[j + 1], so no kernel reads a flag that another block of the same
// launch writes.
struct LzState {
    int32_t steps;     // k: number of alpha_j computed
    int32_t breakdown;
    int32_t n_second;  // conditional Gram-Schmidt: second passes taken so far
    int32_t n_pro;     // partial reorthogonalisation: full Gram-Schmidt passes taken so far
    int32_t skip2;     // conditional Gram-Schmidt: this step's second pass is skipped
    int32_t skip_pro;  // partial reorthogonalisation: this step's pass is skipped
    int32_t force;     // partial reorthogonalisation: the next step reorthogonalises as well
    int32_t pad;
    double theta;      // lowest Ritz value
};

int red_blocks(int64_t n) {
    const int64_t b = (n + kRB - 1) / kRB;
    return static_cast<int>(b < kMaxRedBlocks ? (b < 1 ? 1 : b) : kMaxRedBlocks);
}

__device__ __forceinline__ bool halted(const int32_t* stopped) { return stopped != nullptr && *stopped != 0; }

// The sum of nb <= kMaxRedBlocks partials (stride doubles apart), one after the other, in every thread of a block.
// lds: kMaxRedBlocks + 1 doubles.  A consumer sums the partials of an earlier kernel itself, out of LDS (2 us for 512),
// where a launch of one thread that reads them from memory took 20 to 41 us.
__device__ __forceinline__ double sum_partials(const double* __restrict__ p, int nb, int stride, double* lds) {
    __syncthreads();
    for (int b = threadIdx.x; b < nb; b += blockDim.x) lds[b] = p[int64_t(b) * stride];
    __syncthreads();
    if (threadIdx.x < 64) {
        double s = 0.0;
        int b = 0;
        for (; b + 16 <= nb; b += 16) {
            double t[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) t[q] = lds[b + q];
#pragma unroll
            for (int q = 0; q < 16; ++q) s += t[q];
        }
        for (; b < nb; ++b) s += lds[b];
        if (threadIdx.x == 0) lds[kMaxRedBlocks] = s;
    }
    __syncthreads();
    return lds[kMaxRedBlocks];
}

// ---------------------------------------------------------------- first-stage reductions
__global__ __launch_bounds__(kRB) void k_norm2_partial(int64_t n, const double2* __restrict__ a,
                                                        double* __restrict__ partial) {
    __shared__ double lds[kRB / 64];
    double v[1] = {0.0};
    for (int64_t i = int64_t(blockIdx.x) * kRB + threadIdx.x; i < n; i += int64_t(gridDim.x) * kRB) {
        const double2 x = a[i];
        v[0] += x.x * x.x + x.y * x.y;
    }
    block_sum<1>(v, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = v[0];
}

// partial[b] = sum over the block's rows of conj(a) b
__global__ __launch_bounds__(kRB) void k_dot_partial(int64_t n, const double2* __restrict__ a,
                                                      const double2* __restrict__ b,
                                                      double2* __restrict__ partial) {
    __shared__ double lds[2 * kRB / 64];
    double v[2] = {0.0, 0.0};
    for (int64_t i = int64_t(blockIdx.x) * kRB + threadIdx.x; i < n; i += int64_t(gridDim.x) * kRB) {
        const double2 x = a[i], y = b[i];
        v[0] += x.x * y.x + x.y * y.y;
        v[1] += x.x * y.y - x.y * y.x;
    }
    block_sum<2>(v, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = make_double2(v[0], v[1]);
}

// partial[b] = sum over the block's rows of Re conj(v_j) H v_j; H v_j is w, or h32 for the c64 matvec's output
__global__ __launch_bounds__(kRB) void k_alpha_partial(int64_t n, const double2* __restrict__ vj,
                                                        const double2* __restrict__ w,
                                                        const float2* __restrict__ h32,
                                                        double* __restrict__ partial,
                                                        const int32_t* __restrict__ stopped) {
    if (halted(stopped)) return;
    __shared__ double lds[kRB / 64];
    double v[1] = {0.0};
    for (int64_t i = int64_t(blockIdx.x) * kRB + threadIdx.x; i < n; i += int64_t(gridDim.x) * kRB) {
        const double2 x = vj[i];
        double2 y;
        if (h32) {
            const float2 h = h32[i];
            y = make_double2(h.x, h.y);
        } else {
            y = w[i];
        }
        v[0] += x.x * y.x + x.y * y.y;
    }
    block_sum<1>(v, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = v[0];
}

// ||hu - theta u||^2 partials
__global__ __launch_bounds__(kRB) void k_resid_partial(int64_t n, const double2* __restrict__ hu,
                                                        const double2* __restrict__ u,
                                                        const LzState* __restrict__ st,
                                                        double* __restrict__ partial) {
    __shared__ double lds[kRB / 64];
    double v[1] = {0.0};
    const double th = st->theta;
    for (int64_t i = int64_t(blockIdx.x) * kRB + threadIdx.x; i < n; i += int64_t(gridDim.x) * kRB) {
        const double2 a = hu[i], b = u[i];
        const double rx = a.x - th * b.x, ry = a.y - th * b.y;
        v[0] += rx * rx + ry * ry;
    }
    block_sum<1>(v, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = v[0];
}

// ---------------------------------------------------------------- Gram-Schmidt
// partial[i * nb + block], i < k, from the threads' KM sums (the waves' trees, then in wave order); lds: 2 KM doubles a
// wave.  One barrier, and every lane ends some of the sums: 40 vectors of a small lattice took 4 us in the reduction.
template <int KM>
__device__ __forceinline__ void store_sums(double (&v)[2 * KM], int k, double2* __restrict__ partial, int nb, double* lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    wave_tree_shared<2 * KM>(v, lane);
    if ((lane & 3) == 0) {
#pragma unroll
        for (int j = 0; j < KM / 8; ++j) lds[wave * 2 * KM + wave_share(lane, 2 * KM) + j] = v[j];
    }
    __syncthreads();
    for (int t = threadIdx.x; t < 2 * k; t += kRB) {
        double s = 0.0;
        for (int w = 0; w < kRB / 64; ++w) s += lds[w * 2 * KM + t];
        reinterpret_cast<double*>(partial + int64_t(t >> 1) * nb + blockIdx.x)[t & 1] = s;
    }
}

// A pass is k_gs_dots, k_gs_finalize (large vectors) and k_gs_update; `stopped` is the step's halt flag, or the flag of a
// pass that may be skipped.  The second pass of the conditional form decides by itself, in its first kernel (pre set):
// it runs when the first one left ||w||^2 below half its value before (Daniel, Gragg, Kaufman and Stewart, 1976), and
// block (0, 0) leaves the decision in st->skip2 for the kernels after it.
//
// Coefficients c_i = <V_i|w>, i = 0..k-1: partial[i * nb + block].  Bound by the reads of the basis: the blocks of the
// other groups of kGroup vectors that read the same rows of w run at the same time on the same XCD (blockIdx.x decides
// it), so those hit its L2; 10 million rows and 20 vectors 0.65 ms, 5.1 TB/s, the GPU's copy rate.
__global__ __launch_bounds__(kRB) void k_gs_dots(int64_t n, const double2* __restrict__ V, int k,
                                                  const double2* __restrict__ w, double2* __restrict__ partial,
                                                  int nb, const double* __restrict__ pre,
                                                  const double* __restrict__ post, int nbv, LzState* __restrict__ st,
                                                  const int32_t* __restrict__ stopped) {
    __shared__ double lds[kMaxRedBlocks + 1];
    if (pre != nullptr) {
        const bool halt = halted(stopped);
        const double before = halt ? 0.0 : sum_partials(pre, nbv, 1, lds);
        const double after = halt ? 0.0 : sum_partials(post, nbv, 1, lds);
        const bool skip = halt || after >= 0.5 * before;
        if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
            st->skip2 = skip;
            if (!skip) ++st->n_second;
        }
        if (skip) return;
        __syncthreads();
    } else if (halted(stopped)) {
        return;
    }
    const int base = blockIdx.y * kGroup;
    double v[2 * kGroup];
#pragma unroll
    for (int g = 0; g < 2 * kGroup; ++g) v[g] = 0.0;
    for (int64_t i = int64_t(blockIdx.x) * kRB + threadIdx.x; i < n; i += int64_t(nb) * kRB) {
        const double2 y = w[i];
#pragma unroll
        for (int g = 0; g < kGroup; ++g) {
            if (base + g < k) {
                const double2 x = V[int64_t(base + g) * n + i];
                v[2 * g] += x.x * y.x + x.y * y.y;
                v[2 * g + 1] += x.x * y.y - x.y * y.x;
            }
        }
    }
    store_sums<kGroup>(v, k - base < kGroup ? k - base : kGroup, partial + int64_t(base) * nb, nb, lds);
}

// c_i from its partial sums, a block per coefficient (57 us -> 5 us for 512 partials: they were read by one thread each)
__global__ __launch_bounds__(kRB) void k_gs_finalize(int nb, const double2* __restrict__ partial,
                                                      double2* __restrict__ c, const int32_t* __restrict__ stopped) {
    if (halted(stopped)) return;
    __shared__ double lds[kMaxRedBlocks + 1];
    const double* p = reinterpret_cast<const double*>(partial + int64_t(blockIdx.x) * nb);
    const double re = sum_partials(p, nb, 2, lds), im = sum_partials(p + 1, nb, 2, lds);
    if (threadIdx.x == 0) c[blockIdx.x] = make_double2(re, im);
}

// w -= sum_{i<k} c_i V_i, and the partial sums of the new ||w||^2 when pn is given.  nbs > 0: c comes as nbs partial
// sums each (small vectors: summed here, which saves the launch of k_gs_finalize).  The loads of kGroup vectors are
// issued together (a loop over the vectors waited for each in turn where few blocks run).
constexpr int kCoef = 256;  // coefficients in LDS at a time
__global__ __launch_bounds__(kRB) void k_gs_update(int64_t n, const double2* __restrict__ V, int k,
                                                    const double2* __restrict__ c, int nbs, double2* __restrict__ w,
                                                    double* __restrict__ pn, const int32_t* __restrict__ stopped) {
    if (halted(stopped)) return;
    __shared__ double2 lc[kCoef];
    __shared__ double lds[kRB / 64];
    double nrm[1] = {0.0};
    const bool once = k <= kCoef;
    auto coefficients = [&](int k0) {
        const int kn = k - k0 < kCoef ? k - k0 : kCoef;
        __syncthreads();
        for (int g = threadIdx.x; g < kn; g += kRB) {
            double2 a = make_double2(0.0, 0.0);
            if (nbs > 0) {
                for (int q = 0; q < nbs; ++q) {
                    const double2 p = c[int64_t(k0 + g) * nbs + q];
                    a.x += p.x;
                    a.y += p.y;
                }
            } else {
                a = c[k0 + g];
            }
            lc[g] = a;
        }
        __syncthreads();
        return kn;
    };
    if (once) coefficients(0);
    // every thread walks the same number of rows, so that the barriers of a chunked k are met by all
    const int64_t step = int64_t(gridDim.x) * kRB;
    for (int64_t i0 = int64_t(blockIdx.x) * kRB; i0 < n; i0 += step) {
        const int64_t i = i0 + threadIdx.x;
        const bool act = i < n;
        double ar = 0.0, ai = 0.0;
        for (int k0 = 0; k0 < k; k0 += kCoef) {
            const int kn = once ? k : coefficients(k0);
            if (!act) continue;
            int g = 0;
            for (; g + kGroup <= kn; g += kGroup) {
                double2 x[kGroup];
#pragma unroll
                for (int q = 0; q < kGroup; ++q) x[q] = V[int64_t(k0 + g + q) * n + i];
#pragma unroll
                for (int q = 0; q < kGroup; ++q) {
                    const double2 cg = lc[g + q];
                    ar += cg.x * x[q].x - cg.y * x[q].y;
                    ai += cg.x * x[q].y + cg.y * x[q].x;
                }
            }
            for (; g < kn; ++g) {
                const double2 cg = lc[g], x = V[int64_t(k0 + g) * n + i];
                ar += cg.x * x.x - cg.y * x.y;
                ai += cg.x * x.y + cg.y * x.x;
            }
        }
        if (!act) continue;
        const double2 y = w[i];
        const double2 r = make_double2(y.x - ar, y.y - ai);
        w[i] = r;
        nrm[0] += r.x * r.x + r.y * r.y;
    }
    if (pn == nullptr) return;
    block_sum<1>(nrm, lds);
    if (threadIdx.x == 0) pn[blockIdx.x] = nrm[0];
}

// a basis entry: 32-bit lane offset from a uniform row
__device__ __forceinline__ double2 entry(const double2* __restrict__ row, uint32_t byte) {
    return *reinterpret_cast<const double2*>(reinterpret_cast<const char*>(row) + byte);
}

// The update of one pass and the coefficients of the next in one read of the basis: w -= sum_{i<k} c_i V_i, then
// partial[i * nb + block] = <V_i|w> of the new w.  A thread keeps the k entries of its row in registers between the two,
// and the k sums; rows, order and rounding are those of k_gs_update and k_gs_dots.  Bound by the reads of the basis (three
// instead of four for two passes): 40 steps of 10 million rows 130 -> 105 ms.
// Up to kMidMax vectors: 4 KM registers for the row and as many for the sums (beyond 256 in the accumulator half of the
// register file, whose moves the arithmetic has room for); one wave per SIMD still has KM KB of loads under way.
constexpr int kMidMax = 48;
template <int KM>
__global__ __launch_bounds__(kRB) void k_gs_middle(int64_t n, const double2* __restrict__ V, int k,
                                                    const double2* __restrict__ c, int nbs, double2* __restrict__ w,
                                                    double2* __restrict__ partial, int nb,
                                                    const int32_t* __restrict__ stopped) {
    if (halted(stopped)) return;
    __shared__ double2 lc[KM];
    __shared__ double lds[2 * KM * (kRB / 64)];
    if (threadIdx.x < KM) {  // beyond k: row k - 1 once more, with coefficient 0 and a sum that is not used
        double2 a = make_double2(0.0, 0.0);
        if (threadIdx.x >= k) {
        } else if (nbs > 0) {
            for (int q = 0; q < nbs; ++q) {
                const double2 p = c[int64_t(threadIdx.x) * nbs + q];
                a.x += p.x;
                a.y += p.y;
            }
        } else {
            a = c[threadIdx.x];
        }
        lc[threadIdx.x] = a;
    }
    __syncthreads();
    double v[2 * KM];
#pragma unroll
    for (int g = 0; g < 2 * KM; ++g) v[g] = 0.0;
    for (int64_t i = int64_t(blockIdx.x) * kRB + threadIdx.x; i < n; i += int64_t(nb) * kRB) {
        double2 x[KM];
        const uint32_t o = static_cast<uint32_t>(i) * 16u;
#pragma unroll
        for (int g = 0; g < KM; ++g) x[g] = entry(V + int64_t(g < k ? g : k - 1) * n, o);
        const double2 y = entry(w, o);
        asm volatile("" ::: "memory");  // coefficients come from LDS for each row, not from registers held across rows
        double ar = 0.0, ai = 0.0;
#pragma unroll
        for (int g = 0; g < KM; ++g) {
            const double2 cg = lc[g];
            ar += cg.x * x[g].x - cg.y * x[g].y;
            ai += cg.x * x[g].y + cg.y * x[g].x;
        }
        const double2 r = make_double2(y.x - ar, y.y - ai);
        w[i] = r;
#pragma unroll
        for (int g = 0; g < KM; ++g) {
            v[2 * g] += x[g].x * r.x + x[g].y * r.y;
            v[2 * g + 1] += x[g].x * r.y - x[g].y * r.x;
        }
    }
    store_sums<KM>(v, k, partial, nb, lds);
}

// k_three_term_norm and the coefficients <V_i|w> of the new w, i < k = j + 1, in one pass (up to kMidMax vectors): the
// row's entries of v_j and v_{j-1} are read anyway, and w and the launch are saved.  Rounding as in the two kernels.
template <int KM>
__global__ __launch_bounds__(kRB) void k_three_term_dots(int64_t n, double2* __restrict__ w,
                                                          const float2* __restrict__ h32,
                                                          const double2* __restrict__ V, int k,
                                                          const double* __restrict__ pa, int nb,
                                                          double* __restrict__ alpha, const double* __restrict__ beta,
                                                          double* __restrict__ pn, double2* __restrict__ partial,
                                                          const int32_t* __restrict__ stopped) {
    if (halted(stopped)) return;
    __shared__ double lds[kMaxRedBlocks + 1];
    const double a = sum_partials(pa, nb, 1, lds);
    if (blockIdx.x == 0 && threadIdx.x == 0) *alpha = a;
    const bool two = k > 1;
    const double b = two ? *beta : 0.0;
    double v[2 * KM], nrm[1] = {0.0};
#pragma unroll
    for (int g = 0; g < 2 * KM; ++g) v[g] = 0.0;
    for (int64_t i = int64_t(blockIdx.x) * kRB + threadIdx.x; i < n; i += int64_t(nb) * kRB) {
        double2 x[KM];
        const uint32_t o = static_cast<uint32_t>(i) * 16u;
#pragma unroll
        for (int g = 0; g < KM; ++g) x[g] = entry(V + int64_t(g < k ? g : k - 1) * n, o);
        const double2 xj = entry(V + int64_t(k - 1) * n, o), xm = entry(V + int64_t(two ? k - 2 : 0) * n, o);
        double2 y;
        if (h32) {
            const float2 h = h32[i];
            y = make_double2(h.x, h.y);
        } else {
            y = entry(w, o);
        }
        y.x -= a * xj.x;
        y.y -= a * xj.y;
        if (two) {
            y.x -= b * xm.x;
            y.y -= b * xm.y;
        }
        w[i] = y;
        nrm[0] += y.x * y.x + y.y * y.y;
#pragma unroll
        for (int g = 0; g < KM; ++g) {
            v[2 * g] += x[g].x * y.x + x[g].y * y.y;
            v[2 * g + 1] += x[g].x * y.y - x[g].y * y.x;
        }
    }
    block_sum<1>(nrm, lds);
    if (threadIdx.x == 0) pn[blockIdx.x] = nrm[0];
    store_sums<KM>(v, k, partial, nb, lds);
}

// f with the kernels' vector count for k <= kMidMax: the next multiple of a group
template <typename F>
void with_vectors(int k, F&& f) {
    switch ((k + kGroup - 1) / kGroup) {
        case 1: return f(std::integral_constant<int, kGroup>{});
        case 2: return f(std::integral_constant<int, 2 * kGroup>{});
        case 3: return f(std::integral_constant<int, 3 * kGroup>{});
        case 4: return f(std::integral_constant<int, 4 * kGroup>{});
        case 5: return f(std::integral_constant<int, 5 * kGroup>{});
        default: return f(std::integral_constant<int, 6 * kGroup>{});
    }
}
static_assert(kMidMax == 6 * kGroup, "with_vectors covers every count");

// u = sum_{i<steps} s_i V_i and the partial sums of ||u||^2
__global__ __launch_bounds__(kRB) void k_ritz_vector(int64_t n, const double2* __restrict__ V,
                                                      const LzState* __restrict__ st,
                                                      const double2* __restrict__ s, double2* __restrict__ u,
                                                      double* __restrict__ partial) {
    __shared__ double lds[kRB / 64];
    const int k = st->steps;
    double nrm[1] = {0.0};
    for (int64_t i = int64_t(blockIdx.x) * kRB + threadIdx.x; i < n; i += int64_t(gridDim.x) * kRB) {
        double ar = 0.0, ai = 0.0;
        int g = 0;
        for (; g + kGroup <= k; g += kGroup) {
            double2 x[kGroup];
#pragma unroll
            for (int q = 0; q < kGroup; ++q) x[q] = V[int64_t(g + q) * n + i];
#pragma unroll
            for (int q = 0; q < kGroup; ++q) {
                const double f = s[g + q].x;
                ar += f * x[q].x;
                ai += f * x[q].y;
            }
        }
        for (; g < k; ++g) {
            const double f = s[g].x;
            const double2 x = V[int64_t(g) * n + i];
            ar += f * x.x;
            ai += f * x.y;
        }
        u[i] = make_double2(ar, ai);
        nrm[0] += ar * ar + ai * ai;
    }
    block_sum<1>(nrm, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = nrm[0];
}

// alpha_j from its partial sums, then w = (h32 ? h32 upcast : w) - alpha_j v_j - beta_{j-1} v_{j-1} and the
// partial sums of ||w||^2 (one per block)
__global__ __launch_bounds__(kRB) void k_three_term_norm(int64_t n, double2* __restrict__ w,
                                                          const float2* __restrict__ h32,
                                                          const double2* __restrict__ vj,
                                                          const double2* __restrict__ vjm1,
                                                          const double* __restrict__ pa, int nb,
                                                          double* __restrict__ alpha,
                                                          const double* __restrict__ beta,
                                                          double* __restrict__ partial,
                                                          const int32_t* __restrict__ stopped) {
    if (halted(stopped)) return;
    __shared__ double lds[kMaxRedBlocks + 1];
    const double a = sum_partials(pa, nb, 1, lds);
    if (blockIdx.x == 0 && threadIdx.x == 0) *alpha = a;
    const double b = vjm1 ? *beta : 0.0;
    double v[1] = {0.0};
    for (int64_t i = int64_t(blockIdx.x) * kRB + threadIdx.x; i < n; i += int64_t(gridDim.x) * kRB) {
        double2 y;
        if (h32) {
            const float2 h = h32[i];
            y = make_double2(h.x, h.y);
        } else {
            y = w[i];
        }
        const double2 x = vj[i];
        y.x -= a * x.x;
        y.y -= a * x.y;
        if (vjm1) {
            const double2 z = vjm1[i];
            y.x -= b * z.x;
            y.y -= b * z.y;
        }
        w[i] = y;
        v[0] += y.x * y.x + y.y * y.y;
    }
    block_sum<1>(v, lds);
    if (threadIdx.x == 0) partial[blockIdx.x] = v[0];
}

// ---------------------------------------------------------------- the ends of a step
__device__ __forceinline__ void scale_rows(int64_t n, const double2* src, double2* dst, double s,
                                           float2* __restrict__ dst32) {
    for (int64_t i = int64_t(blockIdx.x) * kRB + threadIdx.x; i < n; i += int64_t(gridDim.x) * kRB) {
        const double2 x = src[i];
        const double2 y = make_double2(x.x / s, x.y / s);
        dst[i] = y;
        if (dst32) dst32[i] = make_float2(static_cast<float>(y.x), static_cast<float>(y.y));
    }
}

// v_0 = v0 / ||v0|| (and its c64 copy when dst32 is given); a zero or non-finite start ends the recurrence
__global__ __launch_bounds__(kRB) void k_start(int64_t n, const double2* __restrict__ v0,
                                                const double* __restrict__ partial, int nb,
                                                double2* __restrict__ dst, float2* __restrict__ dst32,
                                                LzState* __restrict__ st, int32_t* __restrict__ halt) {
    __shared__ double lds[kMaxRedBlocks + 1];
    const double nrm = sqrt(sum_partials(partial, nb, 1, lds));
    const bool ok = nrm > 0.0 && isfinite(nrm);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->steps = 0;
        st->breakdown = 0;
        st->n_second = 0;
        st->n_pro = 0;
        st->skip2 = 1;
        st->skip_pro = 1;
        st->force = 0;
        st->theta = __builtin_nan("");
        halt[0] = ok ? 0 : 1;
    }
    if (ok) scale_rows(n, v0, dst, nrm, dst32);
}

// The end of step j: beta_j = ||w|| from its partial sums, the running estimate of ||T|| (tnorm[j + 1]; tnorm[0]
// is 0), the breakdown test, and v_{j+1} = w / beta_j unless this was the last step.
__global__ __launch_bounds__(kRB) void k_next(int64_t n, double2* __restrict__ w, const double* __restrict__ partial,
                                               int nb, int j, int last, const double* __restrict__ alpha,
                                               double* __restrict__ beta, double* __restrict__ tnorm,
                                               float2* __restrict__ dst32, LzState* __restrict__ st,
                                               int32_t* __restrict__ halt) {
    __shared__ double lds[kMaxRedBlocks + 1];
    const bool first = blockIdx.x == 0 && threadIdx.x == 0;
    if (halt[j] != 0) {
        if (first) halt[j + 1] = 1;
        return;
    }
    const double bj = sqrt(sum_partials(partial, nb, 1, lds));
    const double tn = fmax(j > 0 ? tnorm[j] : 0.0, fabs(alpha[j]) + bj + (j > 0 ? beta[j - 1] : 0.0));
    const bool broke = !last && bj <= 1e-14 * tn;
    if (first) {
        beta[j] = bj;
        tnorm[j + 1] = tn;
        st->steps = j + 1;
        if (broke) st->breakdown = 1;
        halt[j + 1] = (last || broke) ? 1 : 0;
    }
    if (!last && !broke) scale_rows(n, w, w, bj, dst32);
}

// u /= ||V s|| (a basis that is only semi-orthogonal leaves it 1 + O(sqrt(eps))); a zero u is left as it is
__global__ __launch_bounds__(kRB) void k_unit(int64_t n, double2* __restrict__ u, const double* __restrict__ partial,
                                               int nb) {
    __shared__ double lds[kMaxRedBlocks + 1];
    const double nrm = sqrt(sum_partials(partial, nb, 1, lds));
    if (nrm > 0.0 && isfinite(nrm)) scale_rows(n, u, u, nrm, nullptr);
}

// Partial reorthogonalisation (H. D. Simon, "The Lanczos algorithm with partial reorthogonalization",
// Math. Comp. 42 (1984)): the inner products omega_{i,k} = <v_i|v_k> are not computed but estimated from
// the recurrence that the Lanczos relation beta_j v_{j+1} = H v_j - alpha_j v_j - beta_{j-1} v_{j-1}
// implies for them,
//     beta_j omega_{j+1,k} = beta_k omega_{j,k+1} + (alpha_k - alpha_j) omega_{j,k} + beta_{k-1} omega_{j,k-1}
//                            - beta_{j-1} omega_{j-1,k},      omega_{k,k} = 1,
// with a rounding term 2 eps ||T||, of the sign that increases |omega|, added to every new estimate, and
// omega_{j+1,j} = eps64 sqrt(D) ||T|| / beta_j (the level the FP64 three-term step leaves).  eps is the
// machine epsilon of the matvec: FP64's, or FP32's for the c64 form, whose matvec error of about
// eps32 ||H|| per step is what its basis loses orthogonality to.  (A rounding term scaled down by
// 1 / sqrt(D), as for an error vector unrelated to the basis, was measured to be unsafe: on the 20-site
// ring the c64 form's basis then drifted to |<v_i|v_k>| = 0.13.)  When some estimate exceeds sqrt(eps),
// w = beta_j v_{j+1} is orthogonalised against every earlier vector (one classical Gram-Schmidt pass, in
// FP64), and so is the next step's (the loss of orthogonality spreads to it through the recurrence); the
// estimates then restart at eps64 sqrt(D).  Semi-orthogonality (every |omega| <= sqrt(eps)) keeps the
// Ritz values as accurate as full reorthogonalisation would, to O(eps ||H||).
// One block; omega rows i at omega + (i mod 3) (m + 2); partial: the ||w||^2 partial sums of this step;
// tnorm[j]: the estimate of ||T|| before this step.
__global__ __launch_bounds__(kRB) void k_pro_estimate(const double* __restrict__ partial, int nb, int j, int m,
                                                      int64_t D, double eps, const double* __restrict__ alpha,
                                                      const double* __restrict__ beta,
                                                      const double* __restrict__ tnorm, double* __restrict__ omega,
                                                      LzState* __restrict__ st, const int32_t* __restrict__ stopped) {
    __shared__ double red[kRB], lds[kMaxRedBlocks + 1];
    const int tid = threadIdx.x;
    if (halted(stopped)) {
        if (tid == 0) st->skip_pro = 1;
        return;
    }
    const double bj = sqrt(sum_partials(partial, nb, 1, lds));
    const double eps64 = 2.220446049250313e-16;
    const double tn = fmax(j > 0 ? tnorm[j] : 0.0, fabs(alpha[j]) + bj + (j > 0 ? beta[j - 1] : 0.0));
    const double* wc = omega + (j % 3) * (m + 2);          // omega_{j, k}, k < j
    const double* wp = omega + ((j + 2) % 3) * (m + 2);    // omega_{j-1, k}, k < j - 1
    double* wn = omega + ((j + 1) % 3) * (m + 2);          // omega_{j+1, k}, k <= j
    const double level = eps64 * sqrt(static_cast<double>(D));
    const bool usable = bj > 0.0 && isfinite(bj);
    double mx = 0.0;
    if (usable) {
        auto oc = [&](int k) { return k == j ? 1.0 : wc[k]; };
        auto op = [&](int k) { return j == 0 ? 0.0 : (k == j - 1 ? 1.0 : wp[k]); };
        for (int k = tid; k <= j; k += kRB) {
            double t;
            if (k < j) {
                t = beta[k] * oc(k + 1) + (alpha[k] - alpha[j]) * oc(k) - (j > 0 ? beta[j - 1] * op(k) : 0.0);
                if (k > 0) t += beta[k - 1] * oc(k - 1);
                t += (t >= 0.0 ? 2.0 : -2.0) * eps * tn;
                t /= bj;
            } else {
                t = level * tn / bj;
            }
            wn[k] = t;
            mx = fmax(mx, fabs(t));
        }
    }
    red[tid] = mx;
    __syncthreads();
    for (int w = kRB / 2; w > 0; w >>= 1) {
        if (tid < w) red[tid] = fmax(red[tid], red[tid + w]);
        __syncthreads();
    }
    const bool over = usable && red[0] > sqrt(eps);
    const bool now = usable && (over || st->force != 0);
    __syncthreads();
    if (now)
        for (int k = tid; k <= j; k += kRB) wn[k] = level;
    if (tid == 0) {
        st->skip_pro = now ? 0 : 1;
        st->force = over ? 1 : 0;
        if (now) ++st->n_pro;
    }
}

__global__ __launch_bounds__(kRB) void k_scalar_finalize(const double* __restrict__ partial, int nb,
                                                          double* __restrict__ out, int sq) {
    __shared__ double lds[kMaxRedBlocks + 1];
    const double s = sum_partials(partial, nb, 1, lds);
    if (threadIdx.x == 0) *out = sq ? sqrt(s) : s;
}

__global__ __launch_bounds__(kRB) void k_dot_finalize(const double2* __restrict__ partial, int nb,
                                                       double* __restrict__ out) {
    __shared__ double lds[kMaxRedBlocks + 1];
    const double* p = reinterpret_cast<const double*>(partial);
    const double re = sum_partials(p, nb, 2, lds), im = sum_partials(p + 1, nb, 2, lds);
    if (threadIdx.x == 0) {
        out[0] = re;
        out[1] = im;
    }
}

// Number of eigenvalues of the k x k symmetric tridiagonal (a, b) below x: the count of negative pivots
// of the LDL^T factorisation of T - x I (Sturm sequence count, Sylvester's law of inertia), the basis of
// the bisection method of Barth, Martin and Wilkinson (1967); pivots below pivmin in magnitude are
// replaced by -pivmin so the recurrence never divides by zero.
__device__ int sturm_count(const double* a, const double* b, int k, double x, double pivmin) {
    int cnt = 0;
    double q = a[0] - x;
    if (fabs(q) < pivmin) q = -pivmin;
    if (q < 0) ++cnt;
    for (int i = 1; i < k; ++i) {
        q = a[i] - x - b[i - 1] * b[i - 1] / q;
        if (fabs(q) < pivmin) q = -pivmin;
        if (q < 0) ++cnt;
    }
    return cnt;
}

// Lowest eigenpair of T (one wave; k is small): the lowest eigenvalue by bisection on the Sturm count
// (Barth, Martin and Wilkinson), then its eigenvector by inverse iteration (Wilkinson; Peters and
// Wilkinson 1971) with T - theta I factored by Gaussian elimination with partial pivoting, which for a
// tridiagonal matrix keeps a lower band of one and an upper band of two (dl, d, du, du2).  A round takes six levels of
// the bisection: the lanes count at the 63 points it can reach, then follow the branches it takes (10 rounds of k
// divisions instead of 55 to 60).  alpha, beta and the bands sit in LDS while k <= kTriLds: in global memory a step of
// the elimination waits about a microsecond.  390 us -> 104 us at k = 50.  work: 5 * m doubles.  s_out: complex
// coefficients (s_i, 0) for the Ritz vector, zero past k.
constexpr int kTriLds = 1024;
__global__ __launch_bounds__(64) void k_tridiag_lowest(const double* __restrict__ alpha,
                                                        const double* __restrict__ beta, int m,
                                                        LzState* __restrict__ st, double* __restrict__ work,
                                                        double2* __restrict__ s_out, double* __restrict__ result) {
    __shared__ double lt[7 * kTriLds];
    const int k = st->steps, lane = threadIdx.x;
    const double qnan = __builtin_nan("");
    for (int i = lane; i < m; i += 64) s_out[i] = make_double2(0.0, 0.0);
    if (k == 0) {
        if (lane == 0) {
            result[0] = result[1] = result[2] = qnan;
            result[3] = 0.0;
            st->theta = qnan;
        }
        return;
    }
    const bool in_lds = k <= kTriLds;
    const double* a = alpha;
    const double* b = beta;
    double* band = work;  // dl, d, du, du2, x: `pitch` doubles each
    int pitch = m;
    if (in_lds) {
        for (int i = lane; i < k; i += 64) {
            lt[i] = alpha[i];
            lt[kTriLds + i] = beta[i];
        }
        a = lt;
        b = lt + kTriLds;
        band = lt + 2 * kTriLds;
        pitch = kTriLds;
    }
    __syncthreads();
    double lo = INFINITY, hi = -INFINITY, bmax2 = 0.0;
    for (int i = lane; i < k; i += 64) {
        const double r = (i > 0 ? fabs(b[i - 1]) : 0.0) + (i < k - 1 ? fabs(b[i]) : 0.0);
        lo = fmin(lo, a[i] - r);
        hi = fmax(hi, a[i] + r);
        if (i < k - 1) bmax2 = fmax(bmax2, b[i] * b[i]);
    }
    for (int w = 32; w > 0; w >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, w, 64));
        hi = fmax(hi, __shfl_xor(hi, w, 64));
        bmax2 = fmax(bmax2, __shfl_xor(bmax2, w, 64));
    }
    const double pivmin = 2.2250738585072014e-308 * fmax(1.0, bmax2);
    const double tn = fmax(fabs(lo), fabs(hi));
    lo -= 4.0 * 2.220446049250313e-16 * tn + pivmin;
    hi += 4.0 * 2.220446049250313e-16 * tn + pivmin;
    // node q of the tree of the next levels (root 1, children 2 q where the count is 0 and lo moves up, 2 q + 1 where
    // it is not and hi moves down)
    for (int it = 0; it < 400; it += 6) {
        double nlo = lo, nhi = hi;
        const int q = lane + 1;  // lane 63 idles: 63 nodes
        for (int bit = 30 - __clz(q); bit >= 0; --bit) {
            const double mid = 0.5 * (nlo + nhi);
            if ((q >> bit) & 1)
                nhi = mid;
            else
                nlo = mid;
        }
        const bool above = sturm_count(a, b, k, 0.5 * (nlo + nhi), pivmin) >= 1;
        const unsigned long long taken = __ballot(above);
        bool done = false;
        int node = 1;
        for (int level = 0; level < 6; ++level) {
            const double mid = 0.5 * (lo + hi);
            if (mid <= lo || mid >= hi) {
                done = true;
                break;
            }
            const bool up = (taken >> (node - 1)) & 1;
            if (up)
                hi = mid;
            else
                lo = mid;
            node = 2 * node + (up ? 1 : 0);
        }
        if (done) break;
    }
    const double theta = 0.5 * (lo + hi);
    // inverse iteration: LU with partial pivoting of T - theta I (rows swapped as needed), by one lane
    double* dl = band;
    double* d = band + pitch;
    double* du = band + 2 * pitch;
    double* du2 = band + 3 * pitch;
    double* x = band + 4 * pitch;
    for (int i = lane; i < k; i += 64) x[i] = 1.0;
    __syncthreads();
    const double tiny = 2.220446049250313e-16 * fmax(tn, 1e-300);
    for (int iter = 0; iter < 3; ++iter) {
        for (int i = lane; i < k; i += 64) {
            d[i] = a[i] - theta;
            if (i < k - 1) dl[i] = du[i] = b[i];
            du2[i] = 0.0;
        }
        __syncthreads();
        if (lane == 0) {
            // factor with row interchanges, applying the same eliminations to the right-hand side
            for (int i = 0; i < k - 1; ++i) {
                if (fabs(d[i]) >= fabs(dl[i])) {
                    if (d[i] == 0.0) d[i] = tiny;
                    const double f = dl[i] / d[i];
                    dl[i] = f;
                    d[i + 1] -= f * du[i];
                    du2[i] = 0.0;
                    // right-hand side forward step (no swap)
                    x[i + 1] -= f * x[i];
                } else {
                    const double f = d[i] / dl[i];
                    d[i] = dl[i];
                    dl[i] = f;
                    const double t = du[i];
                    du[i] = d[i + 1];
                    d[i + 1] = t - f * d[i + 1];
                    if (i < k - 2) {
                        du2[i] = du[i + 1];
                        du[i + 1] = -f * du[i + 1];
                    }
                    const double xt = x[i];
                    x[i] = x[i + 1];
                    x[i + 1] = xt - f * x[i + 1];
                }
            }
            if (d[k - 1] == 0.0) d[k - 1] = tiny;
            // back substitution with the upper band (d, du, du2)
            x[k - 1] /= d[k - 1];
            if (k > 1) x[k - 2] = (x[k - 2] - du[k - 2] * x[k - 1]) / d[k - 2];
            for (int i = k - 3; i >= 0; --i) x[i] = (x[i] - du[i] * x[i + 1] - du2[i] * x[i + 2]) / d[i];
        }
        __syncthreads();
        double sn = 0.0;
        for (int i = 0; i < k; ++i) sn += x[i] * x[i];
        sn = sqrt(sn);
        for (int i = lane; i < k; i += 64) x[i] /= sn;
        __syncthreads();
    }
    for (int i = lane; i < k; i += 64) s_out[i] = make_double2(x[i], 0.0);
    if (lane == 0) {
        st->theta = theta;
        result[0] = theta;
        result[1] = beta[k - 1] * fabs(x[k - 1]);
        result[3] = static_cast<double>(k);
    }
}

// result[2] = sqrt(sum partials)
__global__ __launch_bounds__(kRB) void k_resid_finalize(const double* __restrict__ partial, int nb,
                                                         const LzState* __restrict__ st,
                                                         double* __restrict__ result) {
    if (st->steps == 0) return;
    __shared__ double lds[kMaxRedBlocks + 1];
    const double s = sum_partials(partial, nb, 1, lds);
    if (threadIdx.x == 0) result[2] = sqrt(s);
}

struct LzLayout {
    size_t state, halt, tnorm, pa, pn0, pn1, pc, coef, svec, work, omega, tmp, x32, y32, total;
};

LzLayout lz_layout(int64_t D, int32_t m, int32_t precision) {
    LzLayout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = align_up(off + bytes, 256);
        return at;
    };
    L.state = take(sizeof(LzState));
    L.halt = take(sizeof(int32_t) * size_t(m + 1));
    L.tnorm = take(sizeof(double) * size_t(m + 1));
    L.pa = take(sizeof(double) * kMaxRedBlocks);   // alpha_j
    L.pn0 = take(sizeof(double) * kMaxRedBlocks);  // ||w||^2 after the three-term update
    L.pn1 = take(sizeof(double) * kMaxRedBlocks);  // ||w||^2 after a Gram-Schmidt pass
    L.pc = take(sizeof(double2) * size_t(m + 1) * kMaxRedBlocks);
    L.coef = take(sizeof(double2) * size_t(m + 1));
    L.svec = take(sizeof(double2) * size_t(m + 1));
    L.work = take(sizeof(double) * 5 * size_t(m + 1));
    L.omega = take(sizeof(double) * 3 * size_t(m + 2));
    L.tmp = take(sizeof(double2) * size_t(D));
    L.x32 = L.y32 = off;
    if (precision == MRMF_PREC_C_IN_Z) {
        L.x32 = take(sizeof(float2) * size_t(D));
        L.y32 = take(sizeof(float2) * size_t(D));
    }
    L.total = off;
    return L;
}

}  // namespace
}  // namespace mrmf

using namespace mrmf;

extern "C" {

mrmf_status mrmf_reduce_scratch_bytes(int64_t n, size_t* bytes) {
    if (n < 0 || !bytes) return MRMF_E_INVALID_ARG;
    *bytes = align_up(sizeof(double2) * kMaxRedBlocks, 256);
    return MRMF_OK;
}

mrmf_status mrmf_dot_z(int64_t n, const void* d_a, const void* d_b, double* d_out, void* d_scratch,
                       size_t scratch_bytes, mrmf_stream stream) {
    if (n < 0 || !d_a || !d_b || !d_out || !d_scratch) return MRMF_E_INVALID_ARG;
    if (scratch_bytes < sizeof(double2) * kMaxRedBlocks) return MRMF_E_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int nb = red_blocks(n);
    auto* part = static_cast<double2*>(d_scratch);
    hipLaunchKernelGGL(k_dot_partial, dim3(nb), dim3(kRB), 0, s, n, static_cast<const double2*>(d_a),
                       static_cast<const double2*>(d_b), part);
    hipLaunchKernelGGL(k_dot_finalize, dim3(1), dim3(kRB), 0, s, part, nb, d_out);
    return launch_status();
}

mrmf_status mrmf_norm_z(int64_t n, const void* d_a, double* d_out, void* d_scratch, size_t scratch_bytes,
                        mrmf_stream stream) {
    if (n < 0 || !d_a || !d_out || !d_scratch) return MRMF_E_INVALID_ARG;
    if (scratch_bytes < sizeof(double) * kMaxRedBlocks) return MRMF_E_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int nb = red_blocks(n);
    auto* part = static_cast<double*>(d_scratch);
    hipLaunchKernelGGL(k_norm2_partial, dim3(nb), dim3(kRB), 0, s, n, static_cast<const double2*>(d_a), part);
    hipLaunchKernelGGL(k_scalar_finalize, dim3(1), dim3(kRB), 0, s, part, nb, d_out, 1);
    return launch_status();
}

mrmf_status mrmf_lanczos_counts(const void* d_scratch, int32_t* d_out, mrmf_stream stream) {
    if (!d_scratch || !d_out || !aligned(d_scratch, 256) || !aligned(d_out, 4)) return MRMF_E_INVALID_ARG;
    // n_second and n_pro are adjacent in the state at the start of the scratch
    const unsigned char* st = static_cast<const unsigned char*>(d_scratch) + offsetof(LzState, n_second);
    static_assert(offsetof(LzState, n_pro) == offsetof(LzState, n_second) + sizeof(int32_t), "LzState layout");
    return hip_status(hipMemcpyAsync(d_out, st, 2 * sizeof(int32_t), hipMemcpyDeviceToDevice,
                                     static_cast<hipStream_t>(stream)));
}

mrmf_status mrmf_lanczos_scratch_bytes(mrmf_plan plan, int32_t m, int32_t precision, size_t* bytes) {
    if (!plan) return MRMF_E_INVALID_ARG;
    return lanczos_scratch_bytes(plan->D, m, precision, bytes);
}

}  // extern "C"

namespace mrmf {

mrmf_status lanczos_scratch_bytes(int64_t D, int32_t m, int32_t precision, size_t* bytes) {
    if (!bytes || m < 1 || m > 100000) return MRMF_E_INVALID_ARG;
    if (precision != MRMF_PREC_Z && precision != MRMF_PREC_C_IN_Z) return MRMF_E_INVALID_ARG;
    *bytes = lz_layout(D, m, precision).total;
    return MRMF_OK;
}

// The recurrence for any map of dimension D: mv_z applies it to a c128 vector, mv_c (C_IN_Z form) to a
// c64 one; both enqueue on the stream and honour the `stopped` flag.
mrmf_status lanczos_run(int64_t D, const MatvecOp& mv_z, const MatvecOp& mv_c, int32_t precision, int32_t m,
                        int32_t reorth, const void* d_v0, void* d_V, double* d_alpha, double* d_beta,
                        double* d_result, void* d_u, void* d_scratch, size_t scratch_bytes, mrmf_stream stream) {
    if (!d_v0 || !d_V || !d_alpha || !d_beta || !d_result || !d_u || !d_scratch) return MRMF_E_INVALID_ARG;
    if (m < 1 || m > 100000) return MRMF_E_INVALID_ARG;
    if (precision != MRMF_PREC_Z && precision != MRMF_PREC_C_IN_Z) return MRMF_E_INVALID_ARG;
    if (precision == MRMF_PREC_C_IN_Z && !mv_c) return MRMF_E_INVALID_ARG;
    if (reorth != MRMF_REORTH_CGS2 && reorth != MRMF_REORTH_NONE && reorth != MRMF_REORTH_CGS2_COND &&
        reorth != MRMF_REORTH_PARTIAL)
        return MRMF_E_INVALID_ARG;
    if (!aligned(d_scratch, 256) || !aligned(d_V, 16) || !aligned(d_u, 16) || !aligned(d_v0, 16))
        return MRMF_E_INVALID_ARG;
    const LzLayout Lo = lz_layout(D, m, precision);
    if (scratch_bytes < Lo.total) return MRMF_E_WORKSPACE;
    const size_t vb = sizeof(double2) * size_t(D);
    if (ranges_overlap(d_V, vb * size_t(m + 1), d_u, vb) || ranges_overlap(d_V, vb * size_t(m + 1), d_v0, vb))
        return MRMF_E_INVALID_ARG;

    hipStream_t s = static_cast<hipStream_t>(stream);
    unsigned char* sc = static_cast<unsigned char*>(d_scratch);
    auto at = [&](size_t off) { return reinterpret_cast<double*>(sc + off); };
    auto atz = [&](size_t off) { return reinterpret_cast<double2*>(sc + off); };
    auto* st = reinterpret_cast<LzState*>(sc + Lo.state);
    auto* halt = reinterpret_cast<int32_t*>(sc + Lo.halt);
    double *tnorm = at(Lo.tnorm), *pa = at(Lo.pa), *pn0 = at(Lo.pn0), *pn1 = at(Lo.pn1);
    double2 *pc = atz(Lo.pc), *coef = atz(Lo.coef), *svec = atz(Lo.svec);
    double *work = at(Lo.work), *omega = at(Lo.omega);
    auto* tmp = atz(Lo.tmp);
    auto* x32 = reinterpret_cast<float2*>(sc + Lo.x32);
    auto* y32 = reinterpret_cast<float2*>(sc + Lo.y32);
    auto* V = static_cast<double2*>(d_V);
    auto* u = static_cast<double2*>(d_u);
    const bool c32 = precision == MRMF_PREC_C_IN_Z;
    const int nb = red_blocks(D);
    const dim3 gv(nb), tb(kRB);
    auto row = [&](int j) { return V + int64_t(j) * D; };

    hipLaunchKernelGGL(k_norm2_partial, gv, tb, 0, s, D, static_cast<const double2*>(d_v0), pn0);
    hipLaunchKernelGGL(k_start, gv, tb, 0, s, D, static_cast<const double2*>(d_v0), pn0, nb, row(0),
                       c32 ? x32 : nullptr, st, halt);
    mrmf_status rc = launch_status();
    if (rc != MRMF_OK) return rc;

    // The kernels of Gram-Schmidt passes of w against rows 0..k-1.  Few partial sums (a small vector): the kernels that
    // use the coefficients sum them themselves.
    const bool inl = nb <= 32;
    double2* pc2 = pc + int64_t(m + 1) * (kMaxRedBlocks / 2);  // (then) the second pass's partial sums
    auto dots = [&](int k, const double2* w, bool decides, const int32_t* stop) {
        hipLaunchKernelGGL(k_gs_dots, dim3(nb, (k + kGroup - 1) / kGroup), tb, 0, s, D, V, k, w, pc, nb,
                           decides ? pn0 : nullptr, pn1, nb, st, stop);
    };
    auto finalize = [&](int k, const int32_t* stop) {
        if (!inl) hipLaunchKernelGGL(k_gs_finalize, dim3(k), tb, 0, s, nb, pc, coef, stop);
    };
    auto update = [&](int k, double2* w, const double2* part, double* pn, const int32_t* stop) {
        hipLaunchKernelGGL(k_gs_update, gv, tb, 0, s, D, V, k, inl ? part : coef, inl ? nb : 0, w, pn, stop);
    };
    // One pass.  decides: it runs only where the first one shrank w; stop: the flag that skips it otherwise; pn: where
    // the new ||w||^2 leaves its partial sums (null: not needed); dotted: the coefficients' partial sums are there.
    auto pass = [&](int k, double2* w, bool decides, const int32_t* stop, double* pn, bool dotted) {
        const int32_t* after = decides ? &st->skip2 : stop;  // the flag of the pass's later kernels
        if (!dotted) dots(k, w, decides, stop);
        finalize(k, after);
        update(k, w, pc, pn, after);
    };
    // Two passes that always run, the first one's update with the second one's dots.
    auto two_passes = [&](int k, double2* w, const int32_t* stop, double* pn) {
        finalize(k, stop);
        with_vectors(k, [&](auto KM) {
            hipLaunchKernelGGL(k_gs_middle<decltype(KM)::value>, gv, tb, 0, s, D, V, k, inl ? pc : coef, inl ? nb : 0, w,
                               inl ? pc2 : pc, nb, stop);
        });
        finalize(k, stop);
        update(k, w, pc2, pn, stop);
    };

    const bool full = reorth == MRMF_REORTH_CGS2, cond = reorth == MRMF_REORTH_CGS2_COND;
    for (int j = 0; j < m; ++j) {
        const int32_t* stopped = halt + j;
        double2* w = row(j + 1);
        // w = H v_j (the c64 form leaves H v_j in y32, read as it is by the next two kernels); alpha_j; then
        // the three-term update in one pass that also leaves the partial sums of ||w||^2 in pn0
        rc = c32 ? mv_c(x32, y32, s, stopped) : mv_z(row(j), w, s, stopped);
        if (rc != MRMF_OK) return rc;
        hipLaunchKernelGGL(k_alpha_partial, gv, tb, 0, s, D, row(j), w, c32 ? y32 : nullptr, pa, stopped);
        const double* pn = pn0;  // where the partial sums of the final ||w||^2 are
        // The kernels that hold a row of the basis in registers: up to kMidMax vectors and 32-bit lane offsets.  Up to 24
        // vectors (two waves per SIMD) they are never slower; beyond that one wave per SIMD has to be worth the read
        // that it saves.  Steps 25 to 40, with k_gs_middle against without: 2^14 rows 0.82 against 0.71 ms, 2^16 1.11
        // and 1.11, 2^18 2.49 and 2.77, 2^20 7.1 and 8.6; k_three_term_dots on top of it: 2^18 2.64, 2^20 7.30, 2^21
        // 12.2 against 12.3, 2^22 23.8 against 24.6.
        const int k = j + 1;
        const bool fits = (full || cond) && k <= kMidMax && D < (int64_t(1) << 28);
        const bool fused = fits && (k <= 24 || D >= (int64_t(1) << 21));        // three-term update with the dots
        const bool middle = full && fits && (k <= 24 || D >= (int64_t(1) << 16));  // update with the next pass's dots
        if (fused) {
            with_vectors(j + 1, [&](auto KM) {
                hipLaunchKernelGGL(k_three_term_dots<decltype(KM)::value>, gv, tb, 0, s, D, w, c32 ? y32 : nullptr, V,
                                   j + 1, pa, nb, d_alpha + j, j > 0 ? d_beta + (j - 1) : nullptr, pn0, pc, stopped);
            });
        } else {
            hipLaunchKernelGGL(k_three_term_norm, gv, tb, 0, s, D, w, c32 ? y32 : nullptr, row(j),
                               j > 0 ? row(j - 1) : nullptr, pa, nb, d_alpha + j, j > 0 ? d_beta + (j - 1) : nullptr,
                               pn0, stopped);
        }
        if (middle) {
            if (!fused) dots(k, w, false, stopped);
            two_passes(k, w, stopped, pn1);
            pn = pn1;
        } else if (full || cond) {
            pass(j + 1, w, false, stopped, cond ? pn1 : nullptr, fused);
            pass(j + 1, w, cond, stopped, pn1, false);
            pn = pn1;
        }
        if (reorth == MRMF_REORTH_PARTIAL) {
            // estimate the loss of orthogonality from ||w||; only when it calls for one, a Gram-Schmidt pass
            // against v_0 .. v_j, which also leaves the new norm's partial sums over the old ones
            const double eps = c32 ? 1.1920928955078125e-07 : 2.220446049250313e-16;  // 2^-23 or 2^-52
            hipLaunchKernelGGL(k_pro_estimate, dim3(1), tb, 0, s, pn0, nb, j, m, D, eps, d_alpha, d_beta, tnorm, omega,
                               st, stopped);
            pass(j + 1, w, false, &st->skip_pro, pn0, false);
        }
        hipLaunchKernelGGL(k_next, gv, tb, 0, s, D, w, pn, nb, j, j == m - 1 ? 1 : 0, d_alpha, d_beta, tnorm,
                           c32 ? x32 : nullptr, st, halt);
        rc = launch_status();
        if (rc != MRMF_OK) return rc;
    }
    // lowest Ritz pair of T, Ritz vector u = sum_i s_i v_i, explicit residual with the FP64 map
    hipLaunchKernelGGL(k_tridiag_lowest, dim3(1), dim3(64), 0, s, d_alpha, d_beta, m, st, work, svec, d_result);
    hipLaunchKernelGGL(k_ritz_vector, gv, tb, 0, s, D, V, st, svec, u, pn0);
    hipLaunchKernelGGL(k_unit, gv, tb, 0, s, D, u, pn0, nb);
    rc = launch_status();
    if (rc != MRMF_OK) return rc;
    rc = mv_z(u, tmp, s, nullptr);
    if (rc != MRMF_OK) return rc;
    hipLaunchKernelGGL(k_resid_partial, gv, tb, 0, s, D, tmp, u, st, pn0);
    hipLaunchKernelGGL(k_resid_finalize, dim3(1), tb, 0, s, pn0, nb, st, d_result);
    return launch_status();
}

}  // namespace mrmf

extern "C" {

mrmf_status mrmf_lanczos(mrmf_plan plan, const void* d_ws, const double* d_theta_z, const float* d_theta_c,
                         int32_t precision, int32_t m, int32_t reorth, const void* d_v0, void* d_V,
                         double* d_alpha, double* d_beta, double* d_result, void* d_u, void* d_scratch,
                         size_t scratch_bytes, mrmf_stream stream) {
    if (!plan || !d_ws || !d_theta_z) return MRMF_E_INVALID_ARG;
    if (precision == MRMF_PREC_C_IN_Z && !d_theta_c) return MRMF_E_INVALID_ARG;
    // the recurrence keeps Re<v|Hv> only and its Ritz values are eigenvalues of H only for Hermitian H
    if (!plan->hermitian) return MRMF_E_NOT_HERMITIAN;
    const MatvecOp mv_z = [&](const void* x, void* y, hipStream_t s, const int32_t* stop) {
        return matvec_lanczos_z(plan, d_ws, d_theta_z, x, y, s, stop);
    };
    const MatvecOp mv_c = [&](const void* x, void* y, hipStream_t s, const int32_t* stop) {
        return matvec_lanczos_c(plan, d_ws, d_theta_c, x, y, s, stop);
    };
    return lanczos_run(plan->D, mv_z, mv_c, precision, m, reorth, d_v0, d_V, d_alpha, d_beta, d_result, d_u,
                       d_scratch, scratch_bytes, stream);
}

}  // extern "C"
