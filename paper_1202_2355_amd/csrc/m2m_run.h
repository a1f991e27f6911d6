// The run kernel: several whole steps of one fit in one launch (its launch shape is
// run_shape in m2m_internal.h). A block has the same particles for the whole launch,
// in registers where every thread has at most one; with more they are read and
// written every step, in the 4 MB L2 of the block's XCD or, above about 10^6 FP32
// particles, the 256 MB memory-side cache. The blocks exchange only the tile sums: the
// force of change of step k + 1 needs the residuals of step k, and nothing else
// crosses blocks.
#pragma once

#include <hip/hip_ext.h>

#include <type_traits>

#include "m2m_device.h"
#include "m2m_pow10.h"
#include "m2m_smooth.h"

namespace m2m {
namespace {

// The thread index as a value that the compiler knows nothing of: what is
// addressed by it is addressed anew on every step, instead of holding address
// registers through the particle loop (the FP64 kernels spilled 50 to 75).
__device__ __forceinline__ int thread_here() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// -------------------------------------------------------------- exchange ----
// Every 64-bit word that blocks exchange carries 32 bits of data and the
// 32-bit tag of the step it belongs to, and is written and read by relaxed
// agent-scope atomics (which bypass the caches that are not shared). A reader
// waits for the tag, so no word needs an order to any other and no fence is
// taken: an agent-scope release would write back an L2 full of particles.
// The tags of a stream's area never repeat (the host counts them).
//
// Measured between 256 blocks of 1024 threads without particles: 3.6 us a
// step for 160 columns this way (owners of 16 neighbouring columns, so that a
// row's entries for one owner are four 64-byte lines), 5.4 with one column per
// owner, 4.9 with rows, a flag each and 8-byte entries, 10.5 with FP64 atomics
// into one vector; the two kernels of a step launched apart pay 7-9 us for
// the finalize, the launch gaps and the tile set-up.
using Word = uint64_t;

__device__ __forceinline__ void put_word(G<Word> p, Word v) {
    __hip_atomic_store((Word*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ Word get_word(G<const Word> p) {
    return __hip_atomic_load((const Word*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool tagged(Word w, uint32_t tag) { return (uint32_t)(w >> 32) == tag; }

// words of one value
template <typename V>
struct Words;
template <>
struct Words<float> {
    static constexpr int n = 1;
    __device__ static void put(G<Word> p, float v, uint32_t tag) {
        put_word(p, (Word)__float_as_uint(v) | ((Word)tag << 32));
    }
    __device__ static bool get(G<const Word> p, uint32_t tag, float& v) {
        const Word a = get_word(p);
        v = __uint_as_float((uint32_t)a);
        return tagged(a, tag);
    }
};
template <>
struct Words<double> {
    static constexpr int n = 2;
    __device__ static void put(G<Word> p, double v, uint32_t tag) {
        const Word b = (Word)__double_as_longlong(v);
        put_word(p, (b & 0xffffffffull) | ((Word)tag << 32));
        put_word(p + 1, (b >> 32) | ((Word)tag << 32));
    }
    __device__ static bool get(G<const Word> p, uint32_t tag, double& v) {
        const Word a = get_word(p), b = get_word(p + 1);
        v = __longlong_as_double((long long)((a & 0xffffffffull) | (b << 32)));
        return tagged(a, tag) && tagged(b, tag);
    }
};

// A wait that has ended without its value (kRunWait, which only a block that
// stopped for good can exceed): the block's later waits are skipped, so that the
// launch ends, and the fit reports the failure (error bit 1).
struct Waiter {
    uint32_t* dead;  // LDS: set by such a wait; and the longest wait
    __device__ bool expired(uint64_t t0, uint32_t most) const {
        if (wall_clock64() - t0 < most) return false;
        dead[0] = 1;
        return true;
    }
};

__device__ __forceinline__ void add_error(G<FitState> st, int32_t bits) {
    (void)__hip_atomic_fetch_or((int32_t*)&st->error, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// the value at p once it carries the tag
template <typename V>
__device__ __forceinline__ V take(const Waiter& w, G<const Word> p, uint32_t tag) {
    V v;
    if (Words<V>::get(p, tag, v) || *w.dead) return v;
    const uint64_t t0 = wall_clock64();
    const uint32_t most = w.dead[1];
    while (!Words<V>::get(p, tag, v))
        if (w.expired(t0, most)) break;
    return v;
}

// Sum over the rows r0, r0 + step, ... < n_rows of the entries at
// base + row * stride (words), in that order, U of them in flight.
template <int U>
__device__ __forceinline__ double take_rows(const Waiter& w, G<const Word> base, size_t stride, int r0,
                                            int step, int n_rows, uint32_t tag) {
    double s = 0.0;
    for (int r = r0; r < n_rows; r += U * step) {
        double v[U];
        bool ok[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            v[k] = 0.0;
            ok[k] = r + k * step >= n_rows || Words<double>::get(base + (size_t)(r + k * step) * stride, tag, v[k]);
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if (!ok[k]) v[k] = take<double>(w, base + (size_t)(r + k * step) * stride, tag);
            s += v[k];
        }
    }
    return s;
}

// The start of a launch: every block counts itself in, and the waits of the
// steps begin only once all have, i.e. are all running. A launch whose blocks
// are not all running within its patience (another kernel holds the compute
// units, or the stream owns too few of them) is called off by one of them: the
// blocks that have started by then do the run among themselves, and those that
// start later leave. So every wait of the steps ends, whatever else the GPU runs,
// and a run slows down as the compute units it gets. Blocks may start when the run
// is long done, so the counters that they read are changed by the last block to
// leave. (Had no block started, the last one to leave would do the run alone.)
constexpr uint32_t kRunOff = 0x80000000u;

// the word that counts the blocks, once all `n` have started or the launch is
// called off; v: a value of it from after this block's own count
__device__ __forceinline__ uint64_t all_running(RunSync* s, uint32_t start0, uint32_t n, uint32_t patience) {
    const uint64_t t0 = wall_clock64();
    for (;;) {
        uint64_t v = __hip_atomic_load(&s->start, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t low = (uint32_t)v, here = low - start0;
        if ((low & kRunOff) || here == n) return v;
        const uint64_t t = wall_clock64() - t0;
        if (patience ? t * here >= (uint64_t)(patience - 1) * n : t > kRunStart) {
            const uint64_t off = v | kRunOff | ((uint64_t)here << 32);
            if (__hip_atomic_compare_exchange_strong(&s->start, &v, off, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT))
                return off;
        }
    }
}

// one more block has left a launch that was called off: true for the last
__device__ __forceinline__ bool leave_run(G<RunSync> s, uint32_t n) {
    return __hip_atomic_fetch_add((uint32_t*)&s->left, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
}

// the counters after a launch of n_steps steps whose blocks have all left
__device__ __forceinline__ void ready_again(G<RunSync> s, G<FitState> st, uint32_t start0, uint32_t n,
                                            int32_t left0, int32_t n_steps) {
    const uint32_t next = run_start_after(start0, n);
    s->start = next;
    s->start0 = next;
    s->left = 0u;
    s->patience = 1u + kRunAgain;
    st->steps_left = left0 - n_steps;
}

// ------------------------------------------------------------ kept kernels ----
// The kernels K_j of a particle after its push (what the deposit of step k
// adds) are those of the force of change of step k + 1, at the same point. A
// block keeps them in LDS, one slot per particle, instead of evaluating them
// twice per step (two logarithms, the bins and the Gauss-Hermite functions:
// about 90 of 270 vector instructions in FP32).
template <typename T, int KIN>
struct Kept {
    static constexpr int KK = KIN & 7;
    static constexpr int nv = (KK == kKinGH4 || KK == kKinGHN) ? KinSlots<KIN>::n : 0;
    T* val;          // nv values per slot, slots values each
    uint32_t* code;  // jr + 1 in 13 bits, jk + 1 above
    int slots;

    __device__ static int bytes(int slots) { return slots * (nv * (int)sizeof(T) + 4); }
    __device__ void put(int at, const Kern<T, KIN>& k) const {
        code[at] = (uint32_t)(k.jr + 1) | ((uint32_t)(k.jk + 1) << 13);
#pragma unroll
        for (int m = 0; m < nv; ++m)
            if (m < k.kn) val[m * slots + at] = k.k[m];
    }
    __device__ Kern<T, KIN> get(int at, const Hot<T>& h, T vz) const {
        Kern<T, KIN> k;
        const uint32_t c = code[at];
        k.jr = (int)(c & 0x1fffu) - 1;
        k.jk = (int)(c >> 13) - 1;
        k.kn = k.jk < 0 ? 0 : (KK == kKinGHN ? h.gh_nmax : KinSlots<KIN>::n);
        if (nv == 0) k.k[0] = KK == kKinV2 ? vz * vz : T(1);
#pragma unroll
        for (int m = 0; m < nv; ++m)
            if (m < k.kn) k.k[m] = val[m * slots + at];
        return k;
    }
};

// ---------------------------------------------------------------- reduce ----
// Job q of a step: observable columns 16 q .. 16 q + 15 over all rows, then
// what the finalize kernel does for them (smoothing, Delta, force table,
// chi^2 part); one wave's 16 lanes per row group, the row groups added over
// the wave and then over the waves, in a fixed order.
template <typename T, int BLOCK, typename F, typename R>
__device__ __forceinline__ void obs_job(F fd, R ra, const Waiter& w, int q,
                                        int n_rows, int ncol, uint32_t tag, int k, bool last,
                                        double (*part)[kRunCols]) {
    constexpr int RG = BLOCK / kRunCols, NW = BLOCK / 64;
    const int t = thread_here(), lane = t & 63, wave = t >> 6;
    const int col = q * kRunCols + (t & (kRunCols - 1));
    const bool in = col < fd->J;
    double yt0 = 0.0, sg = 1.0, Yj = 0.0;
    if (t < kRunCols && in) {
        yt0 = gmem(fd->ytil)[col];
        sg = gmem(fd->sigma)[col];
        Yj = gmem(fd->Y)[col];
    }
    const G<const Word> rows = gmem<const Word>(ra->rows);
    double s = in ? take_rows<4>(w, rows + (size_t)col * 2, (size_t)ncol * 2, t / kRunCols, RG, n_rows, tag)
                  : 0.0;
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    if (lane < kRunCols) part[wave][lane] = s;
    __syncthreads();
    if (wave == 0) {
        double d2 = 0.0;
        if (lane < kRunCols && in) {
            double tot = 0.0;
            for (int v = 0; v < NW; ++v) tot += part[v][lane];
            const double yt = yt0 + fd->q * (tot - yt0);
            const double d = (yt - Yj) / sg;
            const T r = (T)(fd->foc_chi * d / sg);
            Words<T>::put(gmem<Word>(ra->res) + (size_t)col * Words<T>::n, r, tag);
            gmem(fd->ytil)[col] = yt;
            if (last) {
                gmem(fd->yv)[col] = tot;
                gmem(fd->delta)[col] = d;
                gmem<T>(fd->rp)[col] = r;
            }
            d2 = d * d;
        }
        for (int off = kRunCols / 2; off >= 1; off >>= 1) d2 += __shfl_xor(d2, off, 64);
        if (lane == 0)
            Words<double>::put(gmem<Word>(ra->parts) + ((size_t)k * ra->n_jobs + q) * 2, d2, tag);
    }
    __syncthreads();
}

// The exchange areas of the smoothing (kSmWords words): the cells' data, their
// transform and the smoothed priors (C values each), then per grid half the mean of the
// data and the scores of the three search stages.
struct SmWords {
    G<Word> data, what, prior, mean, score;
};
template <typename R>
__device__ __forceinline__ SmWords sm_words(R ra, int C, int half) {
    const G<Word> p = gmem<Word>(ra->parts) + (size_t)ra->n_jobs * kRunMaxSteps * 2;
    const G<Word> h = p + (size_t)C * 6 + (size_t)half * (2 + 3 * kSmoothMaxPoints * 2);
    return SmWords{p, p + (size_t)C * 2, p + (size_t)C * 4, h, h + 2};
}

// Cell job q of a refresh step: cells 16 q .. 16 q + 15, their weight sums
// and counts over all rows, and the means that become the priors or (SMOOTH)
// the data of their smoothing. ptag: the launch's last refresh before this one
// (0: none), whose smoothed priors another block may have written.
template <typename T, int BLOCK, bool SMOOTH, typename F, typename R>
__device__ __forceinline__ void cell_job(F fd, R ra, const Waiter& w, int q,
                                         int n_rows, int ncol, uint32_t tag, uint32_t ptag,
                                         double (*part)[kRunCols], double (*part2)[kRunCols]) {
    constexpr int RG = BLOCK / kRunCols, NW = BLOCK / 64;
    const int t = thread_here(), lane = t & 63, wave = t >> 6;
    const int c = q * kRunCols + (t & (kRunCols - 1));
    const bool in = c < fd->C;
    const G<const Word> rows = gmem<const Word>(ra->rows);
    double s = 0.0, m = 0.0;
    if (in) {
        s = take_rows<2>(w, rows + (size_t)(fd->J + c) * 2, (size_t)ncol * 2, t / kRunCols, RG, n_rows, tag);
        m = take_rows<2>(w, rows + (size_t)(fd->J + fd->C + c) * 2, (size_t)ncol * 2, t / kRunCols, RG,
                         n_rows, tag);
    }
    for (int off = 16; off <= 32; off <<= 1) {
        s += __shfl_xor(s, off, 64);
        m += __shfl_xor(m, off, 64);
    }
    if (lane < kRunCols) {
        part[wave][lane] = s;
        part2[wave][lane] = m;
    }
    __syncthreads();
    if (t < kRunCols && in) {
        double tot = 0.0, cnt = 0.0;
        for (int v = 0; v < NW; ++v) {
            tot += part[v][lane];
            cnt += part2[v][lane];
        }
        // the cell's mean weight, or the previous prior if it is empty
        if constexpr (SMOOTH) {
            const SmWords sw = sm_words(ra, fd->C, 0);
            const double d = cnt > 0.0 ? tot / cnt
                             : ptag   ? take<double>(w, sw.prior + (size_t)c * 2, ptag)
                                      : gmem(fd->gprior)[c];
            gmem(fd->cdata)[c] = d;
            Words<double>::put(sw.data + (size_t)c * 2, d, tag);
        } else {
            const double d = cnt > 0.0 ? tot / cnt : gmem(fd->gprior)[c];
            gmem(fd->cdata)[c] = d;
            gmem(fd->gprior)[c] = d;
            gmem<T>(fd->ucell)[c] = (T)d;
            Words<T>::put(gmem<Word>(ra->cell) + (size_t)c * Words<T>::n, (T)d, tag);
        }
    }
    __syncthreads();
}

// ------------------------------------------------------------- smoothing ----
// The thin-plate smoothing of one prior grid (the method and its search are
// described at the finalize kernel's smooth_priors), its n cells from `base`,
// over the blocks of a run. One block reads the basis (four matrices of (n/4)^2,
// 2 MB for 50 x 20 cells) twice at what one compute unit can have in flight and
// scores three stages of up to 65 lambdas alone: 100 us a refresh. Here
//   transform   a job of 16 outputs per block, from the tagged data,
//   search      one wave per lambda on as few blocks as hold them, the scores
//               tagged; every block that goes on finds the minimum itself,
//   back        one wave per row of the basis, the rows of the four parities of a
//               cell quadruple in four neighbouring waves, which then hold
//               everything that its cells need.
// Six exchanges, 32 us a refresh in all (200 003 FP32 particles, 50 x 20 cells: 52
// steps 959 us by the step and finalize kernels, 408 so). The areas are free again at the next refresh,
// at least two steps later: no block is past the step between them before
// all have left this one.
template <typename T, int BLOCK, typename F, typename R>
__device__ __forceinline__ void run_smooth(F fd, R ra, const Waiter& w, int half,
                                           int b, int nb, uint32_t tag, unsigned char* lds,
                                           double (*part)[kRunCols], int* pick) {
    constexpr int RG = BLOCK / kRunCols, NW = BLOCK / 64, QPB = NW / 4;
    const int t = thread_here(), lane = t & 63, wave = t >> 6;
    // as values that the compiler knows nothing of, so that nothing is derived
    // from them before the step loop and held through it
    int nE = fd->n_E, nx = fd->n_x, base = half * fd->cell_half;
    asm volatile("" : "+s"(nE), "+s"(nx), "+s"(base));
    const int n = nE * nx;
    const G<const double> basis = gmem<const double>(fd->sm_basis);
    const SmBlocks B = sm_blocks(nE, nx);
    const SmWords sw = sm_words(ra, fd->C, half);
    const G<Word> data = sw.data + (size_t)base * 2, what = sw.what + (size_t)base * 2;
    double* sa = reinterpret_cast<double*>(lds);
    double* sb = sa + n;

    // transform: w^ = Q_b^T (folded data), jobs of 16 outputs of one parity block
    const int j1 = (B.o1 + 15) / 16, j2 = j1 + (B.o2 - B.o1 + 15) / 16,
              j3 = j2 + (B.o3 - B.o2 + 15) / 16, jobs = j3 + (B.o4 - B.o3 + 15) / 16;
    if (b < jobs) {
        for (int c = t; c < n; c += BLOCK) sb[c] = take<double>(w, data + (size_t)c * 2, tag);
        __syncthreads();
        if (b == 0 && wave == 0) {
            double sm = 0.0;
            for (int c = lane; c < n; c += 64) sm += sb[c];
            for (int off = 32; off >= 1; off >>= 1) sm += __shfl_xor(sm, off, 64);
            if (lane == 0) Words<double>::put(sw.mean, sm / n, tag);
        }
        for (int c = t; c < n; c += BLOCK)
            sa[c] = fold_cell(B, nE, nx, c, [&](int q) { return sb[q]; });
        __syncthreads();
        for (int q = b; q < jobs; q += nb) {
            const int bb = q < j1 ? 0 : (q < j2 ? 1 : (q < j3 ? 2 : 3));
            const int o0 = B.off(bb), m = B.off(bb + 1) - o0;
            const int o = (q - (bb == 0 ? 0 : (bb == 1 ? j1 : (bb == 2 ? j2 : j3)))) * 16 + (t & 15);
            double s = 0.0;
            if (o < m) {
                const G<const double> Q = basis + B.qoff(bb) + o;
                int r = t >> 4;
                for (; r + 3 * RG < m; r += 4 * RG) {
                    double v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = Q[(size_t)(r + u * RG) * m];
#pragma unroll
                    for (int u = 0; u < 4; ++u) s = fma(v[u], sa[o0 + r + u * RG], s);
                }
                for (; r < m; r += RG) s = fma(Q[(size_t)r * m], sa[o0 + r], s);
            }
            s += __shfl_xor(s, 16, 64);
            s += __shfl_xor(s, 32, 64);
            if (lane < kRunCols) part[wave][lane] = s;
            __syncthreads();
            if (t < kRunCols && o < m) {
                double tot = 0.0;
                for (int v = 0; v < NW; ++v) tot += part[v][lane];
                Words<double>::put(what + (size_t)(o0 + o) * 2, tot, tag);
            }
            __syncthreads();
        }
    }

    // search, by the blocks that score lambdas and those that transform back
    const int quads = B.mE0 * B.mX0, scorers = (max(fd->sm_k1, 65) + NW - 1) / NW;
    if (b >= scorers && b * QPB >= quads) return;
    for (int c = t; c < n; c += BLOCK) {
        sa[c] = basis[c];  // eigenvalues
        sb[c] = take<double>(w, what + (size_t)c * 2, tag);
    }
    __syncthreads();
    // stage 0: sm_k1 points lo + 0.25 i; stages 1 and 2: 65 points lo + (hi - lo) i / 64
    double lo = fd->sm_plo, hi = 0.0;
    int best = 0;
#pragma unroll 1
    for (int st = 0; st < 3; ++st) {
        const int npts = st == 0 ? fd->sm_k1 : 65;
        const G<Word> sc = sw.score + (size_t)st * kSmoothMaxPoints * 2;
        for (int i = b * NW + wave; i < npts; i += nb * NW) {
            const double lam = pow10_of(st == 0 ? lo + 0.25 * i : lo + (hi - lo) * i / 64.0);
            double out;
            gcv_points<1>(sa, sb, n, lane, &lam, &out);
            if (lane == 0) Words<double>::put(sc + (size_t)i * 2, out, tag);
        }
        if (wave == 0) {
            int bi = npts;
            double bg = 0.0;
            for (int i = lane; i < npts; i += 64) {
                const double g = take<double>(w, sc + (size_t)i * 2, tag);
                if (bi == npts || g < bg) {
                    bg = g;
                    bi = i;
                }
            }
            for (int off = 32; off >= 1; off >>= 1) {
                const double og = __shfl_xor(bg, off, 64);
                const int oi = __shfl_xor(bi, off, 64);
                if (oi < npts && (bi == npts || og < bg || (og == bg && oi < bi))) {
                    bg = og;
                    bi = oi;
                }
            }
            if (lane == 0) *pick = bi < npts ? bi : 0;
        }
        __syncthreads();
        best = __builtin_amdgcn_readfirstlane(*pick);
        __syncthreads();
        if (st == 2) break;
        // the next stage: between the neighbours of the best point
        const double from = lo;
        const int i0 = best > 0 ? best - 1 : 0, i1 = best < npts - 1 ? best + 1 : npts - 1;
        lo = st == 0 ? from + 0.25 * i0 : from + (hi - from) * i0 / 64.0;
        hi = st == 0 ? from + 0.25 * i1 : from + (hi - from) * i1 / 64.0;
    }
    if (b * QPB >= quads) return;
    const double lam = pow10_of(lo + (hi - lo) * best / 64.0);
    for (int c = t; c < n; c += BLOCK) sa[c] = sb[c] / (1.0 + lam * sa[c]);
    __syncthreads();

    // back: wave 4 s + bb takes row (i, j) of parity block bb for slot s's
    // quadruple of cells (i, j), (i, nx-1-j), (nE-1-i, j), (nE-1-i, nx-1-j)
    const int bb = wave & 3, pE = bb >> 1, pX = bb & 1;
    for (int q0 = b * QPB; q0 < quads; q0 += nb * QPB) {
        const int q = q0 + (wave >> 2), i = q / B.mX0, j = q - i * B.mX0;
        double s = 0.0;
        if (q < quads && i < B.mE(pE) && j < B.mX(pX)) {
            const int o0 = B.off(bb), m = B.off(bb + 1) - o0;
            const G<const double> Q = basis + B.qoff(bb) + (size_t)(i * B.mX(pX) + j) * m;
            for (int k = lane; k < m; k += 64) s = fma(Q[k], sa[o0 + k], s);
        }
        for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
        if (lane == 0) part[wave >> 2][bb] = s;
        __syncthreads();
        if (t < 4 * QPB && q0 + (t >> 2) < quads) {
            const int qq = q0 + (t >> 2), qi = qq / B.mX0, qj = qq - qi * B.mX0;
            const int k = (t & 2) ? nE - 1 - qi : qi, l = (t & 1) ? nx - 1 - qj : qj;
            if (!((t & 2) && k == qi) && !((t & 1) && l == qj)) {
                const double floor_v = 1e-3 * take<double>(w, sw.mean, tag);
                const double v = fmax(unfold_cell(B, nE, nx, k, l, [&](int p, int, int) {
                                          return part[t >> 2][p];
                                      }), floor_v);
                const int c = base + k * nx + l;
                gmem(fd->gprior)[c] = v;
                gmem<T>(fd->ucell)[c] = (T)v;
                Words<double>::put(sw.prior + (size_t)c * 2, v, tag);
                Words<T>::put(gmem<Word>(ra->cell) + (size_t)c * Words<T>::n, (T)v, tag);
            }
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------- run ----
// memory that nothing writes during a launch (scalar loads)
template <typename V>
using Const = const __attribute__((address_space(4))) V*;

template <typename F, typename R>
struct LateArgs {
    F fd;
    R ra;
};

// the arguments of k_run
struct RunParams {
    FitDev fd;
    RunArgs ra;
    RunCall call;
};

// Steps of one fit over n_blocks blocks, by block b. Block b takes the
// particles in groups of 64 (one wave each): group (m n_blocks + b) for m = wave,
// wave + NW, ..., so that every compute unit gets the same number of waves to
// within one (blocks of 1024 consecutive particles left 300 007 FP64 particles
// on 147 compute units for two rounds, or on 37 of 256 for the second).
// KNOWN: the launch's start0 comes with the call; OWN: a fit of a
// batch, with its own steps left and setting (both at compile time: as branches
// at the start of the kernel they cost a launch of one step 0.6-0.9 of 12.4 us).
// SMOOTH: the priors are smoothed at every refresh.
// late(): where fd and ra are in memory, as addresses that the compiler knows nothing
// of: what a step needs after its particles, and the end of the launch, is read
// there. Held through the particle loop it costs the loop's scalar registers: 154
// values spilled to lanes, 100 of them read back in the loop (FP32 Gauss-Hermite,
// 1024 threads), now 92 and 48. 100 steps of 10^6 particles 1173 us so and 1124 now, one
// step of 4001 11.2 and 10.3.
template <typename T, int BLOCK, int KIN, bool KNOWN, bool OWN, bool SMOOTH, typename Late>
__device__ __forceinline__ void run_fit(const FitDev& fd, const RunArgs& ra, int b,
                                        const uint32_t n_blocks, const RunCall& call, Late late) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    constexpr int NW = BLOCK / 64;
    __shared__ double part[NW][kRunCols], part2[NW][kRunCols];
    __shared__ int flag;
    __shared__ uint32_t dead[2], group[3];
    using A = double;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = (int)fd.n;
    int nb = (int)n_blocks;
    const G<FitState> st = gmem(fd.st);
    const G<RunSync> sync = gmem(ra.sync);
    int n_steps = call.n_steps;
    if (OWN) {
        n_steps = min(n_steps, (int)st->steps_left);
        if (n_steps <= 0) return;  // uniform: the fit is idle
    }
    const uint32_t start0 = KNOWN ? call.start0 : sync->start0;
    const uint32_t tag0 = call.tag0;
    uint64_t came = 0;
    // counted in at once; the result, and what else the counters hold, is first
    // looked at when everything else has been requested (0.3-1.6 us a launch)
    if (tid == 0)
        came = __hip_atomic_fetch_add(&ra.sync->start, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    const G<T> __restrict__ X = gmem<T>(fd.x);
    const G<T> __restrict__ Y = gmem<T>(fd.y);
    const G<T> __restrict__ Z = gmem<T>(fd.z);
    const G<T> __restrict__ VX = gmem<T>(fd.vx);
    const G<T> __restrict__ VY = gmem<T>(fd.vy);
    const G<T> __restrict__ VZ = gmem<T>(fd.vz);
    const G<T> __restrict__ U = gmem<T>(fd.u);
    const G<T> __restrict__ UH = gmem<T>(fd.uh);
    const G<uint16_t> __restrict__ CI = gmem(fd.cidx);
    bool assign = st->assign_pending != 0;
    const bool correct = OWN ? st->correct != 0 : call.correct != 0;
    const bool priors = correct && fd.entropy == 0 && fd.prior_every > 0;
    // correction steps until the next refresh
    int until = priors ? fd.prior_every - (int)(st->kstep % fd.prior_every) : 0;

    // the first particles are requested before the set-up
    int i0 = (wave * nb + b) * 64 + lane, istep = NW * nb * 64;
    T nx = T(0), ny = T(0), nz = T(0), nvx = T(0), nvy = T(0), nvz = T(0), nu = T(0), nh = T(1);
    auto load = [&](int i) {
        nx = *elem<T>(X, i);
        ny = *elem<T>(Y, i);
        nz = *elem<T>(Z, i);
        nvx = *elem<T>(VX, i);
        nvy = *elem<T>(VY, i);
        nvz = *elem<T>(VZ, i);
        nu = *elem<T>(U, i);
        nh = *elem<T>(UH, i);
    };
    if (i0 < n) load(i0);

    const Hot<T> h = hot_of<T>(fd);
    const int J = h.J, C = h.C, kp = h.kp, ncol = J + 2 * C;
    Tabs<T, A> tb = carve<T, A>(lds_raw, J, kp, h.n_r, h.n_R, h.n_v, C);
    const int priv = tid & (kp - 1);
    {
        const G<const T> rp = gmem<const T>(fd.rp);
        for (int j = tid; j < J; j += BLOCK) tb.rp[j] = rp[j];
        for (int j = tid; j < J * kp; j += BLOCK) tb.sum[j] = 0.0;
        for (int j = tid; j < C; j += BLOCK) {
            tb.csum[j] = 0.0;
            tb.ccnt[j] = 0u;
        }
        const G<const T> re2 = gmem<const T>(fd.redge2);
        for (int j = tid; j <= h.n_r; j += BLOCK) tb.re2[j] = re2[j];
        const G<const T> Re2 = gmem<const T>(fd.Redge2);
        for (int j = tid; j <= h.n_R; j += BLOCK) tb.Re2[j] = Re2[j];
        const G<const T> ve = gmem<const T>(fd.vedge);
        for (int j = tid; j <= h.n_v; j += BLOCK) tb.ve[j] = ve[j];
        const G<const T> Vp = gmem<const T>(fd.Vp);
        const G<const T> isp = gmem<const T>(fd.isp);
        for (int j = tid; j < h.n_R; j += BLOCK) {
            tb.Vp[j] = Vp[j];
            tb.isp[j] = isp[j];
        }
    }
    if (tid == 0) {
        const uint32_t most = sync->wait;
        dead[0] = 0;
        dead[1] = most ? most : kRunWait;
        // the blocks that do the run (0: this one leaves) and this one's place among
        // them, and whether others had to leave
        const uint64_t v = all_running(ra.sync, start0, n_blocks, sync->patience);
        uint32_t m = n_blocks, at = (uint32_t)b, off = 0;
        if ((uint32_t)v & kRunOff) {
            off = 1;
            m = (uint32_t)(v >> 32);
            at = (uint32_t)came - start0;
            if ((uint32_t)came & kRunOff) {
                const bool end = leave_run(sync, n_blocks);
                if (end && m > 0)
                    ready_again(sync, st, start0, n_blocks, OWN ? st->steps_left : n_steps, n_steps);
                m = end && m == 0 ? 1 : 0;
                at = 0;
                off = 2;  // alone: has left already
            }
        }
        group[0] = m;
        group[1] = at;
        group[2] = off;
    }
    __syncthreads();
    const bool whole = __builtin_amdgcn_readfirstlane(group[2]) == 0;
    if (!whole) {
        nb = __builtin_amdgcn_readfirstlane(group[0]);
        if (nb == 0) return;
        b = __builtin_amdgcn_readfirstlane(group[1]);
        i0 = (wave * nb + b) * 64 + lane;
        istep = NW * nb * 64;
        if (i0 < n) load(i0);
    }
    const Waiter wt{dead};
    // at most one particle per thread: they stay in registers
    const bool resident = n <= istep;
    Kept<T, KIN> kept;
    kept.slots = (n + istep - 1) / istep * BLOCK;
    kept.val = reinterpret_cast<T*>(lds_raw + ra.keep_at);
    kept.code = reinterpret_cast<uint32_t*>(kept.val + Kept<T, KIN>::nv * kept.slots);
    const bool keep = whole && ra.keep_bytes > 0;
    bool assigned = false;  // some step of this launch wrote the priors
    uint32_t ptag = 0u;     // the last refresh of this launch

    for (int k = 0; k < n_steps; ++k) {
        const uint32_t tag = tag0 + 1u + (uint32_t)k;
        const bool last = k == n_steps - 1;
        const bool refresh = priors && --until == 0;
        if (refresh) until = fd.prior_every;
        assigned |= assign;
        // software pipeline: the loads of the next particle are in flight
        // while the current one is computed
        int at = tid;
        for (int i = i0; i < n; i += istep, at += BLOCK) {
            T x = nx, y = ny, z = nz, vx = nvx, vy = nvy, vz = nvz, u = nu, uh = nh;
            if (i + istep < n) load(i + istep);
            if (assign) {
                // the prior of the particle's cell at the last refresh: of the
                // previous step, or of an earlier launch
                const int c = min((int)*elem<uint16_t>(CI, i), C - 1);
                if (k > 0)
                    uh = take<T>(wt, gmem<const Word>(ra.cell) + (size_t)c * Words<T>::n, tag - 1u);
                else
                    uh = gmem<const T>(fd.ucell)[c];
                settle(uh);
            }
            if (correct) {
                Kern<T, KIN> kk;
                if (keep && k > 0)
                    kk = kept.get(at, h, vz);
                else
                    kk = kernels<T, A, KIN>(h, tb, x, y, z, vz);
                u = corrected_weight<T, A, KIN>(h, tb, kk, u, uh);
            }
            x += h.hdt * vx;
            y += h.hdt * vy;
            z += h.hdt * vz;
            kick<T, true>(h, x, y, z, vx, vy, vz);
            x += h.hdt * vx;
            y += h.hdt * vy;
            z += h.hdt * vz;
            const Kern<T, KIN> kk = kernels<T, A, KIN>(h, tb, x, y, z, vz);
            deposit<T, KIN>(h, tb, kk, u, priv);
            if (keep) kept.put(at, kk);
            if (refresh) {
                const int c = cell_of<T>(h, x, y, z, vx, vy, vz);
                atomicAdd(&tb.csum[c], (double)u);
                atomicAdd(&tb.ccnt[c], 1u);
                *elem<uint16_t>(CI, i) = (uint16_t)c;
            }
            settle(nx);  // the next particle, before the stores
            settle(ny);
            settle(nz);
            settle(nvx);
            settle(nvy);
            settle(nvz);
            settle(nu);
            settle(nh);
            if (resident) {
                nx = x;
                ny = y;
                nz = z;
                nvx = vx;
                nvy = vy;
                nvz = vz;
                nu = u;
                nh = uh;
            }
            if (!resident || last) {
                *elem<T>(X, i) = x;
                *elem<T>(Y, i) = y;
                *elem<T>(Z, i) = z;
                *elem<T>(VX, i) = vx;
                *elem<T>(VY, i) = vy;
                *elem<T>(VZ, i) = vz;
                if (correct) *elem<T>(U, i) = u;
                if (resident ? assigned : assign) *elem<T>(UH, i) = uh;
            }
        }
        // the first particle of the next step, requested before the exchange
        if (!resident && !last && i0 < n) load(i0);
        const auto la = late();
        __syncthreads();
        // this block's row of sums; the bins are cleared for the next step
        const int t0 = thread_here();
        const G<Word> row = gmem<Word>(la.ra->rows) + (size_t)b * ncol * 2;
        for (int j = t0; j < J; j += BLOCK) {
            double t = 0.0;
            for (int g = 0; g < kp; ++g) {
                t += tb.sum[j * kp + g];
                tb.sum[j * kp + g] = 0.0;
            }
            Words<double>::put(row + (size_t)j * 2, t, tag);
        }
        if (refresh)
            for (int j = t0; j < C; j += BLOCK) {
                Words<double>::put(row + (size_t)(J + j) * 2, tb.csum[j], tag);
                Words<double>::put(row + (size_t)(J + C + j) * 2, (double)tb.ccnt[j], tag);
                tb.csum[j] = 0.0;
                tb.ccnt[j] = 0u;
            }
        for (int q = b; q < la.ra->n_jobs; q += nb)
            obs_job<T, BLOCK>(la.fd, la.ra, wt, q, nb, ncol, tag, k, last, part);
        if (refresh)
            // cell jobs from the last block down, away from the observable jobs
            for (int q = nb - 1 - b; q < la.ra->n_cell_jobs; q += nb)
                cell_job<T, BLOCK, SMOOTH>(la.fd, la.ra, wt, q, nb, ncol, tag, ptag, part, part2);
        if (SMOOTH && refresh) {
            for (int half = 0; half <= (la.fd->cell_flags & 1); ++half)
                run_smooth<T, BLOCK>(la.fd, la.ra, wt, half, b, nb, tag,
                                     lds_raw + ((la.ra->keep_at + la.ra->keep_bytes + 7) & ~7), part, &flag);
            ptag = tag;
        }
        if (!last) {
            for (int j = t0; j < J; j += BLOCK)
                tb.rp[j] = take<T>(wt, gmem<const Word>(la.ra->res) + (size_t)j * Words<T>::n, tag);
            __syncthreads();
        }
        assign = refresh;
    }

    // every block reports its own waits: the last one may be done before
    const auto la = late();
    const G<FitState> se = gmem(la.fd->st);
    if (tid == 0) {
        if (dead[0]) add_error(se, 2);
        if (group[2]) {
            const G<RunSync> sy = gmem(la.ra->sync);
            if (group[2] == 2 || leave_run(sy, n_blocks))
                ready_again(sy, se, start0, n_blocks, OWN ? se->steps_left : n_steps, n_steps);
        }
    }
    // the last block (it has the fewest particles) ends the run: chi^2 of every
    // step from its jobs' parts in order, then the counters
    if (b != nb - 1) return;
    const int64_t kstep0 = se->kstep, tstep0 = se->tstep;
    // up to 16 lanes a step, so that the steps take one pass: one lane per step
    // read 164 parts (2610 observables) in turn, 31 us at the end of every launch
    bool bad = false;
    const int jobs = la.ra->n_jobs;
    int lanes = 16;
    while (lanes > 1 && n_steps * lanes > BLOCK) lanes >>= 1;
    const int te = thread_here(), k = te / lanes;
    double c2 = 0.0;
    if (k < n_steps)
        c2 = take_rows<4>(wt, gmem<const Word>(la.ra->parts) + (size_t)k * jobs * 2, 2, te & (lanes - 1), lanes,
                          jobs, tag0 + 1u + (uint32_t)k);
    for (int off = lanes / 2; off >= 1; off >>= 1) c2 += __shfl_xor(c2, off, 64);
    if (k < n_steps && (te & (lanes - 1)) == 0) {
        gmem(la.fd->chi2_hist)[(tstep0 + k) % kHistCap] = c2;
        if (k == n_steps - 1) se->chi2 = c2;
        bad = !isfinite(c2);
    }
    static_assert(BLOCK >= kRunMaxSteps, "one thread per step");
    const int any_bad = __syncthreads_or(bad ? 1 : 0);
    if (tid == 0) {
        if (any_bad || dead[0]) add_error(se, (any_bad ? 1 : 0) | (dead[0] ? 2 : 0));
        se->tstep = tstep0 + n_steps;
        if (correct) se->kstep = kstep0 + n_steps;
        se->correct = correct ? 1 : 0;
        se->assign_pending = assign ? 1 : 0;
        const G<RunSync> sy = gmem(la.ra->sync);
        if (group[2] == 0) {
            const uint32_t next = run_start_after(start0, n_blocks);
            if (next == 0u) sy->start = 0u;
            sy->start0 = next;
            sy->patience = 0u;
            se->steps_left = OWN ? se->steps_left - n_steps : 0;
        }
    }
}

template <typename T, int BLOCK, int KIN, bool KNOWN, bool SMOOTH>
__global__ __launch_bounds__(BLOCK) void k_run(const RunParams P) {
    run_fit<T, BLOCK, KIN, KNOWN, false, SMOOTH>(P.fd, P.ra, (int)blockIdx.x, gridDim.x, P.call, [] {
        auto p = (Const<RunParams>)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(p));
        return LateArgs<Const<FitDev>, Const<RunArgs>>{&p->fd, &p->ra};
    });
}

// the fits of a table, each over its own blocks (no fit waits for another)
template <typename T, int BLOCK, int KIN>
__global__ __launch_bounds__(BLOCK) void k_runs(const FitDev* __restrict__ fits,
                                                const RunArgs* __restrict__ ras,
                                                const RunTile* __restrict__ tiles, int32_t n_steps,
                                                uint32_t tag0) {
    const RunTile t = tiles[blockIdx.x];
    run_fit<T, BLOCK, KIN, false, true, false>(
        fits[t.fit], ras[t.fit], t.b, (uint32_t)t.nb, RunCall{n_steps, 1, 0, 0u, tag0}, [=] {
            // from the start: its loop has scalars to spare, and reading them again cost
            // 0.6-1.7 % (12 Gauss-Hermite fits of 24 000 to 120 000 10.73 us a step, 10.65 so)
            return LateArgs<const FitDev*, const RunArgs*>{fits + t.fit, ras + t.fit};
        });
}

// f(the kind of kinematic observables as a compile-time constant)
template <typename F>
hipError_t with_kin(int kin, F&& f) {
    switch (kin) {
        case kKinNone: f(std::integral_constant<int, kKinNone>()); break;
        case kKinV2: f(std::integral_constant<int, kKinV2>()); break;
        case kKinGH4: f(std::integral_constant<int, kKinGH4>()); break;
        case kKinGHN: f(std::integral_constant<int, kKinGHN>()); break;
        case kKinLOSVD: f(std::integral_constant<int, kKinLOSVD>()); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// One launch; with `done` its packet completes that event. An event recorded after
// the launch is a packet of its own: 3 us between launches of a 1 us kernel, where
// the launch's own takes 0.8, and nothing measurable behind one of 70 us.
template <typename K, typename... Args>
void launch_blocks(K kernel, int blocks, int block, size_t lds, hipStream_t s, hipEvent_t done,
                   const Args&... args) {
    if (done)
        hipExtLaunchKernelGGL(kernel, dim3(blocks), dim3(block), (uint32_t)lds, s, nullptr, done, 0, args...);
    else
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(block), lds, s, args...);
}

// SMOOTH: built without KNOWN only (a step of such a fit is rarely launched alone)
template <typename T, int BLOCK, bool SMOOTH>
hipError_t launch_run_t(int kin, const FitDev& fd, const RunArgs& ra, int blocks, size_t lds,
                        const RunCall& call, hipStream_t s, hipEvent_t done) {
    return with_kin(kin, [&](auto K) {
        constexpr int kind = decltype(K)::value;
        if constexpr (!SMOOTH)
            if (call.known) {
                launch_blocks(k_run<T, BLOCK, kind, true, false>, blocks, BLOCK, lds, s, done, RunParams{fd, ra, call});
                return;
            }
        launch_blocks(k_run<T, BLOCK, kind, false, SMOOTH>, blocks, BLOCK, lds, s, done, RunParams{fd, ra, call});
    });
}

template <typename T, int BLOCK>
hipError_t launch_runs_t(int kin, const FitDev* fits, const RunArgs* ras, const RunTile* tiles,
                         int blocks, size_t lds, int n_steps, uint32_t tag0, hipStream_t s,
                         hipEvent_t done) {
    return with_kin(kin, [&](auto K) {
        launch_blocks(k_runs<T, BLOCK, decltype(K)::value>, blocks, BLOCK, lds, s, done, fits, ras, tiles,
                      n_steps, tag0);
    });
}

}  // namespace
}  // namespace m2m
