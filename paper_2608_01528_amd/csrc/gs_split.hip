// Dense contractions with few output tiles: request-sized batches, where the
// 128 x 128 tiles of gs_gemm.hip would leave most CUs idle while a handful of
// work-groups walk the whole K range.
//
//   project, prob2vec, reconstruct, weighted sum   out = A Bop
//   bind                                           out = (A Bop) .* (A2 Bop)
//   similarity / attention scores                  out = scale A B^T / norms
//
// The output is cut into small tiles (32 x 32, 32 x 64 or 64 x 64) and the K
// range of a tile is dealt to the waves of its work-group, K-step by K-step
// (wave w takes steps w, w + WK, ...).  A wave works alone: it loads its
// step's operand slices into registers one step ahead, passes them through a
// private piece of LDS (which turns whole 128-byte row slices into matrix
// fragments; no barrier, the LDS operations of one wave stay in order), and
// accumulates the whole tile for its share of K.  The partial tiles are then
// added through LDS in wave order, so results are reproducible bit for bit,
// and the epilogue runs on the sums.
//
// What bounds it: with few tiles the matrix work of one CU (a 32 x 32 tile of
// K = 4096 fp32 is 14 us of one CU's matrix cores) and the first loads; with
// many, fp32 runs at 65-80 % of the matrix peak and bf16 at the L2 rate
// (about 15-19 TB/s over the chip: a 64 x 64 tile reads 16 KiB for 64 or 16
// MFMAs).  Per launch, before (128 x 128 tiles, one work-group walking all of
// K) and now: 777 x 203 x 4096 fp32 350 -> 26 us, bf16 86 -> 10; 1024 x 1000 x
// 4096 fp32 354 -> 77, bf16 87 -> 21; 4096 x 360 x 4096 fp32 355 -> 138; T Q
// with 64 rows, r = 1000, D = 4096 fp32 83 -> 10; the bound product of 512 rows,
// r = 360 65 -> 33.
//
// Every operand row is read in 16-byte pieces at the row's own alignment (the
// hardware takes any element-aligned address) and never past its end: the
// piece that would reach further is read as the row's last 16 bytes and moved
// down in registers.
#include <type_traits>
#include "gs_internal.h"

namespace gs {
namespace {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef short s4v __attribute__((ext_vector_type(4)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint16_t h8u __attribute__((ext_vector_type(8), aligned(2)));
#define AS_L __attribute__((address_space(3)))

constexpr int MAX_WK = 8;          // waves per work-group at most

template <typename T> struct Op;
template <> struct Op<bf16_t> {
    typedef bf8v V;
    typedef h8u U;                  // 16 bytes at any element-aligned address
    static constexpr int KS = 64, PER = 8;
};
template <> struct Op<float> {
    typedef f4v V;
    typedef f4u U;
    static constexpr int KS = 32, PER = 4;
};

// LDS hand-off between the lanes of one wave: the compiler keeps the order,
// the hardware executes a wave's LDS operations in order.
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A lane-dependent value that the compiler takes for a new one: what the rare
// edge paths derive from it is computed there, not kept live (and spilled)
// across the loop.
__device__ __forceinline__ int fresh(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// 16 bytes (PER elements) at base + off (base wave-uniform).  Every load of a
// slice is issued before the first is used, so edges are handled by clamped
// offsets, not by branches.
template <typename T>
__device__ __forceinline__ u4v load16(const char *base, uint32_t off) {
    return __builtin_bit_cast(u4v, *reinterpret_cast<const typename Op<T>::U *>(base + off));
}
// The piece moved down by e elements (0 <= e < PER, any lane its own).
template <typename T>
__device__ __forceinline__ u4v move_down(u4v v, int e) {
    if constexpr (sizeof(T) == 2) {
        const u4v h = {v[0] >> 16 | v[1] << 16, v[1] >> 16 | v[2] << 16, v[2] >> 16 | v[3] << 16, v[3] >> 16};
        v = (e & 1) ? h : v;
        e >>= 1;
    }
    v = (e & 1) ? u4v{v[1], v[2], v[3], 0} : v;
    return (e & 2) ? u4v{v[2], v[3], 0, 0} : v;
}
// Zero the elements i >= n of a piece.
template <typename T>
__device__ __forceinline__ u4v keep_first(u4v v, int n) {
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = i < n ? v[i] : 0u;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = 2 * i + 1 < n ? v[i] : (2 * i < n ? (v[i] & 0xffffu) : 0u);
    }
    return v;
}

// Row operand slice: 32 R rows x 128 bytes of a K-step, loaded by one wave.
// Piece q (0 .. 4R-1): lane l takes row 8q + l / 8, 16-byte chunk l % 8.  off[q]
// is the byte offset of that row (clamped to the last row) and chunk from the
// tile's first row.
template <typename T, int R>
struct RowSlice {
    uint32_t off[4 * R];
    u4v v[4 * R];
    __device__ __forceinline__ void init(int64_t ld, int64_t nrows, int l) {
#pragma unroll
        for (int q = 0; q < 4 * R; ++q) {
            int64_t r = 8 * q + (l >> 3);
            if (r > nrows - 1) r = nrows - 1;
            off[q] = (uint32_t)(r * ld * (int64_t)sizeof(T)) + 16 * (l & 7) + 16;
        }
    }
    // base: the tile's first row (wave-uniform).  In the K-step that reaches
    // past kend (>= PER) a chunk with n < PER elements in range is read as the
    // row's last PER elements; trim moves it down and zeroes the elements at
    // k >= kend.
    __device__ __forceinline__ void fetch(const T *base, int k0, int kend, int l) {
        const int n = kend - k0 - Op<T>::PER * (l & 7);
        const uint32_t back = n < Op<T>::PER ? (uint32_t)(Op<T>::PER - n) * (uint32_t)sizeof(T) : 0;
        // (from 16 bytes further down, so that the offsets stay positive)
        const char *p = reinterpret_cast<const char *>(base + k0) - 16;
#pragma unroll
        for (int q = 0; q < 4 * R; ++q) v[q] = load16<T>(p, off[q] - back);
    }
    __device__ __forceinline__ void trim(int k0, int kend, int l) {
        const int n = kend - k0 - Op<T>::PER * (fresh(l) & 7);
        const int back = n < Op<T>::PER ? Op<T>::PER - n : 0;
#pragma unroll
        for (int q = 0; q < 4 * R; ++q) {
            v[q] = keep_first<T>(move_down<T>(v[q], back), n);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // Sum of squares of the pieces, per row.
    __device__ __forceinline__ void add_squares(float s[4 * R]) const {
#pragma unroll
        for (int q = 0; q < 4 * R; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (sizeof(T) == 4) {
                    const float x = __uint_as_float(v[q][i]);
                    s[q] += x * x;
                } else {
                    const float x = __uint_as_float(v[q][i] << 16), y = __uint_as_float(v[q][i] & 0xffff0000u);
                    s[q] += x * x + y * y;
                }
            }
    }
    // LDS layout: chunk c of row r at c ^ ((r >> 1) & 7) of the row's eight
    // positions, so the fragment reads (one chunk of 32 rows) reach all banks
    __device__ __forceinline__ void stash(char *tile, int l) const {
#pragma unroll
        for (int q = 0; q < 4 * R; ++q)
            *reinterpret_cast<u4v *>(tile + (8 * q + (l >> 3)) * 128 + (((l & 7) ^ (4 * (q & 1) + (l >> 4))) << 4)) = v[q];
    }
};

template <typename T>
__device__ __forceinline__ typename Op<T>::V frag_rows(const char *tile, int r, int c) {
    return *reinterpret_cast<const typename Op<T>::V *>(tile + r * 128 + ((c ^ ((r >> 1) & 7)) << 4));
}

// K x N operand slice: KS k-rows x 32 NJ columns.  A k-row holds CPR chunks
// of 16 bytes; piece q: lane l takes k-row KPI q + l / CPR, chunk l % CPR.
// LDS layout: row-major, with the halves of a 256-byte bank line exchanged so
// that the rows one fragment read touches together fall on different banks
// (fp32: k and k + 4; bf16: k-rows k .. k + 3).
template <typename T, int NJ>
struct ColSlice {
    static constexpr int P = Op<T>::PER, KS = Op<T>::KS;
    static constexpr int CPR = 32 * NJ / P;         // chunks per k-row
    static constexpr int KPI = 64 / CPR;            // k-rows per piece
    static constexpr int NP = KS / KPI;             // pieces (4 NJ)
    u4v v[NP];
    static __device__ __forceinline__ int place(int k, int c) {        // byte offset of chunk c of k-row k
        if constexpr (sizeof(T) == 4) {
            if constexpr (NJ == 1) return (k ^ ((k >> 2) & 1)) * 128 + 16 * c;
            else return k * 256 + 16 * (c ^ (8 * ((k >> 2) & 1)));
        } else {
            if constexpr (NJ == 1) return k * 64 + 16 * c;
            else return k * 128 + 16 * (c ^ (4 * ((k >> 1) & 1)));
        }
    }
    // base: the operand's first row at the tile's first column; ncols columns
    // exist from there (and at least PER in the row).  In the last tile
    // column a chunk that reaches past the row's end is read as its last PER
    // elements and moved down by trim (what lands in the columns past the end
    // is not stored).  k-rows at k >= kend are read from the last one, and
    // zeroed by trim.
    __device__ __forceinline__ void fetch(const T *base, int64_t ld, int k0, int kend, int64_t ncols, int l) {
        const int n = ncols < 32 * NJ ? (int)ncols - P * (l % CPR) : P;
        const int nc = P * (l % CPR) + P - (n < P ? P - n : 0);
        // (from 16 bytes further down, so that the offsets stay positive)
        const char *p = reinterpret_cast<const char *>(base + (int64_t)k0 * ld) - 16;
        const int klast = kend - 1 - k0;
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int k = KPI * q + l / CPR;
            v[q] = load16<T>(p, (uint32_t)(((k < klast ? k : klast) * (int)ld + nc) * (int)sizeof(T)));
        }
    }
    __device__ __forceinline__ void trim(int k0, int kend, int64_t ncols, int l) {
        l = fresh(l);
        const int n = ncols < 32 * NJ ? (int)ncols - P * (l % CPR) : P;
        const int back = n < P ? P - n : 0;
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            v[q] = move_down<T>(v[q], back);
            if (KPI * q + l / CPR > kend - 1 - k0) v[q] = u4v{0, 0, 0, 0};
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __device__ __forceinline__ void stash(char *tile, int l) const {
#pragma unroll
        for (int q = 0; q < NP; ++q)
            *reinterpret_cast<u4v *>(tile + place(KPI * q + l / CPR, l % CPR)) = v[q];
    }
    // The fragment of substep q (k from 2 PER q + PER (lane / 32)) for column
    // 32 j + lane % 32.
    static __device__ __forceinline__ typename Op<T>::V frag(const char *tile, int q, int j, int l) {
        if constexpr (sizeof(T) == 4) {
            f4v r;
            const int n = 32 * j + (l & 31), k = 8 * q + 4 * (l >> 5);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                r[e] = *reinterpret_cast<const float *>(tile + place(k + e, n >> 2) + 4 * (n & 3));
            return r;
        } else {
            // two transpose reads of four k each: lane group g = l / 16 of 16
            // lanes reads k-rows k .. k + 3 and 16 columns
            const int gq = l >> 4, a = l & 15;
            const int n = 32 * j + 16 * (gq & 1) + 4 * (a & 3);
            const int k = 16 * q + 8 * (gq >> 1) + (a >> 2);
            const s4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((AS_L s4v *)(tile + place(k, n >> 3) + 2 * (n & 7)));
            const s4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((AS_L s4v *)(tile + place(k + 4, n >> 3) + 2 * (n & 7)));
            const s4v both[2] = {lo, hi};
            return *reinterpret_cast<const bf8v *>(both);
        }
    }
};

// XCD-aware tile order: consecutive logical tiles (which share their A rows)
// go to work-groups of one XCD.
__device__ __forceinline__ int64_t logical_tile(int64_t total) {
    const int64_t per = (total + 7) / 8;
    return (int64_t)(blockIdx.x & 7) * per + (blockIdx.x >> 3);
}

// Partial tiles in LDS: row-major fp32 with rows of TN + 8 floats, so the four
// rows apart that a store instruction of the accumulator layout writes fall on
// different banks.
template <int NJ> constexpr int part_row() { return 32 * NJ + 8; }
template <bool TWO, int MI, int NJ>
constexpr int wave_bytes() {        // private LDS of a wave: its operand slices, then its partial tiles
    constexpr int stage = ((TWO ? 2 : 1) * MI + NJ) * 4096, part = (TWO ? 2 : 1) * 32 * MI * part_row<NJ>() * 4;
    return stage > part ? stage : part;
}
template <bool TWO, int MI, int NJ>
constexpr size_t lds_bytes(int wk) {    // + the waves' shares of the row and column norms, + the factors
    return (size_t)wk * (wave_bytes<TWO, MI, NJ>() + (MI + NJ) * 128) + (MI + NJ) * 128;
}

// One tile of 32 MI x 32 NJ per work-group of blockDim.x / 64 waves.
template <typename T, bool BNN, bool TWO, int MI, int NJ, bool SCORES, typename TO>
__global__ void __launch_bounds__(64 * MAX_WK) split_kernel(GemmArgs g, int vec_out) {
    constexpr int TM = 32 * MI, TN = 32 * NJ, KS = Op<T>::KS;
    constexpr int NP = TWO ? 2 : 1;                 // products
    constexpr int PR = part_row<NJ>();
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int l = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wk = blockDim.x >> 6;
    const int64_t nM = (g.M + TM - 1) / TM, nN = (g.N + TN - 1) / TN;
    const int64_t L = logical_tile(nM * nN);
    if (L >= nM * nN) return;
    const int64_t m0 = (L / nN) * TM, n0 = (L % nN) * TN;

    const bool sqa = SCORES ? (g.cosine && g.qnorm2 == nullptr) : (g.rownorm2 != nullptr && n0 == 0);
    const bool sqb = SCORES && g.cosine && g.cnorm == nullptr;
    // lower-echelon R: rows j < n0 of the K x N operand are zero in this
    // tile's columns; columns k >= n0 + TN of the N x K operand are zero in
    // its rows (row norms of A need the whole range)
    int64_t k_lo = 0, k_hi = g.K;
    if (g.echelon && !sqa) {
        if (BNN) {
            if (n0 < g.K) k_lo = n0 / KS * KS;
        } else if (n0 + TN < g.K) {
            k_hi = n0 + TN;
        }
    }
    const T *A = static_cast<const T *>(g.A) + m0 * g.lda;
    const T *A2 = TWO ? static_cast<const T *>(g.A2) + m0 * g.lda2 : nullptr;
    const T *B = static_cast<const T *>(g.B) + (BNN ? n0 : n0 * g.ldb);

    RowSlice<T, MI> sa, sa2;
    typename std::conditional<BNN, ColSlice<T, NJ>, RowSlice<T, NJ>>::type sb;
    sa.init(g.lda, g.M - m0, l);
    if (TWO) sa2.init(g.lda2, g.M - m0, l);
    if constexpr (!BNN) sb.init(g.ldb, g.N - n0, l);
    char *ta = lds + w * wave_bytes<TWO, MI, NJ>();
    char *tb = ta + MI * 4096, *ta2 = tb + NJ * 4096;

    f16v acc[NP][MI][NJ];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[p][i][j] = f16v{};
    float qa[4 * MI], qb[4 * NJ];
#pragma unroll
    for (int i = 0; i < 4 * MI; ++i) qa[i] = 0.f;
#pragma unroll
    for (int j = 0; j < 4 * NJ; ++j) qb[j] = 0.f;

    const int kend = (int)k_hi, stride = wk * KS;
    auto fetch = [&](int k0) {
        sa.fetch(A, k0, kend, l);
        if (TWO) sa2.fetch(A2, k0, kend, l);
        if constexpr (BNN) sb.fetch(B, g.ldb, k0, kend, g.N - n0, l);
        else sb.fetch(B, k0, kend, l);
    };
    auto trim = [&](int k0) {
        if (k0 + KS > kend) {
            sa.trim(k0, kend, l);
            if (TWO) sa2.trim(k0, kend, l);
        }
        if constexpr (BNN) {
            if (k0 + KS > kend || g.N - n0 < TN) sb.trim(k0, kend, g.N - n0, l);
        } else {
            if (k0 + KS > kend) sb.trim(k0, kend, l);
        }
    };
    // substep q: lanes take chunk 2q + l / 32 of their rows, A and B alike, so
    // every MFMA pairs the same k
    auto substep = [&](int q) {
        const int c = 2 * q + (l >> 5);
        typename Op<T>::V fa[NP][MI], fb[NJ];
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            fa[0][i] = frag_rows<T>(ta, 32 * i + (l & 31), c);
            if constexpr (TWO) fa[1][i] = frag_rows<T>(ta2, 32 * i + (l & 31), c);
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            if constexpr (BNN) fb[j] = ColSlice<T, NJ>::frag(tb, q, j, l);
            else fb[j] = frag_rows<T>(tb, 32 * j + (l & 31), c);
        }
        if constexpr (sizeof(T) == 2) {
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
                        acc[p][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[p][i], fb[j], acc[p][i][j], 0, 0, 0);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int p = 0; p < NP; ++p)
#pragma unroll
                    for (int i = 0; i < MI; ++i)
#pragma unroll
                        for (int j = 0; j < NJ; ++j)
                            acc[p][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[p][i][e], fb[j][e], acc[p][i][j], 0, 0, 0);
        }
    };
    // the slices of one K-step are in registers (or on their way) while the
    // previous one is multiplied
    // (wave w takes the K-steps w, w + wk, ... of the whole range, so a range
    // shortened by an echelon operand leaves every sum as it is)
    int first = w * KS;
    if (k_lo > first) first += (int)((k_lo - first + stride - 1) / stride) * stride;
    for (int k0 = first - stride; k0 < kend; k0 += stride) {
        const bool have = k0 >= first;
        if (have) {
            trim(k0);
            sa.stash(ta, l);
            sb.stash(tb, l);
            if (TWO) sa2.stash(ta2, l);
            if (sqa) sa.add_squares(qa);
            if constexpr (SCORES) {
                if (sqb) sb.add_squares(qb);
            }
            wave_fence();
        }
        if (k0 + stride < kend) fetch(k0 + stride);
        if (!have) continue;
        if (k0 + KS <= kend) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                substep(q);
                if (NP * MI * NJ > 1) __builtin_amdgcn_sched_barrier(0);     // (fragments of one substep live)
            }
        } else {
            for (int q = 0; q * (KS / 4) < kend - k0; ++q) substep(q);
        }
        wave_fence();
    }

    // partial norms and tiles of this wave
    float *norms = reinterpret_cast<float *>(lds + wk * wave_bytes<TWO, MI, NJ>());
    float *fac = norms + wk * (TM + TN);            // row factors, column factors
    if (sqa || sqb) {
        float *mine = norms + w * (TM + TN);
#pragma unroll
        for (int q = 0; q < 4 * (MI + NJ); ++q) {       // piece q: row 8q + l / 8, its chunks on 8 lanes
            float s = q < 4 * MI ? qa[q < 4 * MI ? q : 0] : qb[q < 4 * MI ? 0 : q - 4 * MI];
            s += __shfl_xor(s, 1);
            s += __shfl_xor(s, 2);
            s += __shfl_xor(s, 4);
            if ((l & 7) == 0) mine[8 * q + (l >> 3)] = s;
        }
    }
    // accumulator register r of block (i, j): row 32 i + 8 (r / 4) + 4 (l / 32) + r % 4, column 32 j + l % 32
    float *part = reinterpret_cast<float *>(ta);
    const int le = fresh(l);
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    part[(p * TM + 32 * i + 8 * (r >> 2) + 4 * (le >> 5) + (r & 3)) * PR + 32 * j + (le & 31)] =
                        acc[p][i][j][r];
    __syncthreads();
    if constexpr (SCORES) {
        for (int t = threadIdx.x; t < TM + TN; t += blockDim.x) {
            float f = t < TM ? g.scale : 1.f;
            if (g.cosine) {
                float s = 0.f;
                if ((t < TM) ? sqa : sqb)
                    for (int u = 0; u < wk; ++u) s += norms[u * (TM + TN) + t];
                if (t < TM) {
                    const float n2 = g.qnorm2 ? (m0 + t < g.M ? g.qnorm2[m0 + t] : 1.f) : s;
                    f = n2 > 0.f ? g.scale / sqrtf(n2) : 0.f;
                } else {
                    const int64_t c = n0 + t - TM;
                    const float cc = g.cnorm ? (c < g.N ? g.cnorm[c] : 1.f) : sqrtf(s);
                    f = cc > 0.f ? 1.f / cc : 0.f;
                }
            }
            fac[t] = f;
        }
        __syncthreads();
    } else if (sqa) {
        for (int t = threadIdx.x; t < TM; t += blockDim.x)
            if (m0 + t < g.M) {
                float s = 0.f;
                for (int u = 0; u < wk; ++u) s += norms[u * (TM + TN) + t];
                g.rownorm2[m0 + t] = s;
            }
    }

    // four columns of a row at a time: the waves' shares in wave order
    TO *C = static_cast<TO *>(g.C);
    for (int it = threadIdx.x; it < TM * TN / 4; it += blockDim.x) {
        const int rl = it / (TN / 4), cl = 4 * (it % (TN / 4));
        const int64_t row = m0 + rl, col = n0 + cl;
        if (row >= g.M || col >= g.N) continue;
        f4v v[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const char *src = lds + ((p * TM + rl) * PR + cl) * 4;
            v[p] = *reinterpret_cast<const f4v *>(src);
            for (int u = 1; u < wk; ++u) v[p] += *reinterpret_cast<const f4v *>(src + u * wave_bytes<TWO, MI, NJ>());
        }
        f4v x = TWO ? v[0] * v[NP - 1] : v[0];
        if constexpr (SCORES) x = x * fac[rl] * *reinterpret_cast<const f4v *>(fac + TM + cl);
        TO *dst = C + row * g.ldc + col;
        if (vec_out && col + 4 <= g.N) {
            if constexpr (sizeof(TO) == 4) {
                *reinterpret_cast<f4v *>(dst) = x;
            } else {
                *reinterpret_cast<uint2 *>(dst) = uint2{(uint32_t)f32_to_bf16(x[0]) | ((uint32_t)f32_to_bf16(x[1]) << 16),
                                                        (uint32_t)f32_to_bf16(x[2]) | ((uint32_t)f32_to_bf16(x[3]) << 16)};
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + e < g.N) st_f32<TO>(dst, e, x[e]);
        }
    }
}

struct Plan {
    int cfg;        // 0: 32 x 32 tiles, 1: 64 x 64 (two products: 32 x 64)
    int wk;         // waves per tile
    double cost;
};

template <typename T, bool BNN, bool TWO, int MI, int NJ, bool SCORES, typename TO>
hipError_t launch_cfg(const GemmArgs &a, int wk, hipStream_t s) {
    const int64_t total = ((a.M + 32 * MI - 1) / (32 * MI)) * ((a.N + 32 * NJ - 1) / (32 * NJ));
    const size_t lds = lds_bytes<TWO, MI, NJ>(wk);
    auto *k = &split_kernel<T, BNN, TWO, MI, NJ, SCORES, TO>;
    if (lds > 65536) {
        hipError_t e = raise_lds_limit(reinterpret_cast<const void *>(k), lds);
        if (e != hipSuccess) return e;
    }
    // output rows whose quads of columns are aligned to their size
    const int vec_out = reinterpret_cast<uintptr_t>(a.C) % (4 * sizeof(TO)) == 0 && a.ldc % 4 == 0;
    hipLaunchKernelGGL(k, dim3((unsigned)(8 * ((total + 7) / 8))), dim3(64 * wk), lds, s, a, vec_out);
    return hipGetLastError();
}

template <typename T, bool BNN, bool TWO, bool SCORES, typename TO>
hipError_t launch_plan(const GemmArgs &a, Plan p, hipStream_t s) {
    if (p.cfg == 0) return launch_cfg<T, BNN, TWO, 1, 1, SCORES, TO>(a, p.wk, s);
    if constexpr (TWO) {
        return launch_cfg<T, BNN, TWO, 1, 2, SCORES, TO>(a, p.wk, s);
    } else {
        return launch_cfg<T, BNN, TWO, 2, 2, SCORES, TO>(a, p.wk, s);
    }
}

template <typename T>
hipError_t launch_typed(gs_dtype tout, bool b_nn, bool two, bool scores, const GemmArgs &a, Plan p, hipStream_t s) {
    if (scores) return launch_plan<T, false, false, true, float>(a, p, s);
    if (two) {
        if (!b_nn) return hipErrorInvalidValue;     // only restored vectors are bound
        return tout == GS_BF16 ? launch_plan<T, true, true, false, bf16_t>(a, p, s)
                               : launch_plan<T, true, true, false, float>(a, p, s);
    }
    if (b_nn) return tout == GS_BF16 ? launch_plan<T, true, false, false, bf16_t>(a, p, s)
                                     : launch_plan<T, true, false, false, float>(a, p, s);
    return tout == GS_BF16 ? launch_plan<T, false, false, false, bf16_t>(a, p, s)
                           : launch_plan<T, false, false, false, float>(a, p, s);
}

// Which tiles, and how many waves per tile: the cheapest by a model of the
// time in microseconds, rounds x (K-steps per wave + o) x u.  A round is 2048
// waves (two per SIMD: the matrix cores are then the limit for fp32, the
// loads for bf16); u is what a wave's K-step takes in a full round, o the
// start of a tile, the final sum and its stores in K-steps.  The constants
// reproduce measured times within about 15 % (fp32: 1024 x 1000 x 4096 on 64
// x 64 tiles 134 modelled, 135 us; 777 x 203 x 4096 on 32 x 32 tiles 24 and
// 26; bf16: 8192 x 1000 x 2048 on 64 x 64 tiles 61 and 58).
struct Model { double u, o; };
constexpr Model F32_SMALL = {1.25, 3.0}, F32_BIG = {4.0, 1.5}, BF16_SMALL = {0.7, 8.0}, BF16_BIG = {1.7, 4.0};
// The 256 x 256 tiles run one per CU; a round takes per_step x K-steps + o,
// a call c more (fp32 16384 x 1000 x 4096: 721 modelled, 747 us).
struct LargeModel { double per_step, o, c; };
constexpr LargeModel F32_LARGE = {5.5, 10.0, 7.0}, BF16_LARGE = {1.55, 6.0, 5.0};
constexpr int WAVE_SLOTS = 2048;

int64_t tiles_of(const GemmArgs &a, int tm, int tn) { return ((a.M + tm - 1) / tm) * ((a.N + tn - 1) / tn); }

bool make_plan(gs_dtype t, bool b_nn, Epi epi, const GemmArgs &a, Plan &p) {
    const int64_t es = t == GS_BF16 ? 2 : 4, ks = 128 / es;
    const bool two = epi == EPI_BIND;
    // 32-bit byte offsets inside a tile's K-step, 32-bit K indices
    const int64_t lim = (int64_t)1 << 22;
    if (a.K >= ((int64_t)1 << 30) || a.lda >= lim || a.ldb >= lim || (two && (a.lda2 >= lim || !b_nn))) return false;
    // whole 16-byte pieces within a row
    if (a.K < 16 / es || (b_nn && a.N < 16 / es)) return false;
    const int64_t steps = (a.K + ks - 1) / ks;
    p.cost = 1e300;
    for (int cfg = 0; cfg < 2; ++cfg) {
        const Model m = es == 2 ? (cfg ? BF16_BIG : BF16_SMALL) : (cfg ? F32_BIG : F32_SMALL);
        const int64_t tiles = cfg == 0 ? tiles_of(a, 32, 32) : two ? tiles_of(a, 32, 64) : tiles_of(a, 64, 64);
        const double u = (two && cfg == 0) ? 1.6 * m.u : m.u;     // (32 x 64 of two products: the blocks of 64 x 64)
        for (int wk = 1; wk <= MAX_WK && (wk == 1 || wk <= steps); wk *= 2) {
            const int64_t rounds = (tiles * wk + WAVE_SLOTS - 1) / WAVE_SLOTS;
            const double cost = (double)rounds * ((double)((steps + wk - 1) / wk) + m.o) * u;
            if (cost < p.cost) p = Plan{cfg, wk, cost};
        }
    }
    return true;
}

}  // namespace

bool split_takes(gs_dtype t, bool b_nn, Epi epi, const GemmArgs &a) {
    Plan p;
    return make_plan(t, b_nn, epi, a, p);
}

bool split_better(gs_dtype t, bool b_nn, Epi epi, const GemmArgs &a) {
    Plan p;
    if (!make_plan(t, b_nn, epi, a, p)) return false;
    const int64_t es = t == GS_BF16 ? 2 : 4;
    const LargeModel m = es == 2 ? BF16_LARGE : F32_LARGE;
    const double rounds = (double)((tiles_of(a, 256, 256) + 255) / 256), step = m.per_step * (double)((a.K * es + 127) / 128);
    // a bound product takes two launches, the second re-reading the output
    const double large = epi == EPI_BIND ? 2 * rounds * (step + m.o + 6) + m.c : rounds * (step + m.o) + m.c;
    // row results that the large tiles fold into their epilogue (whole rows
    // in a tile) cost a pass over the scores here
    const bool fused = a.N <= 256 && (epi == EPI_SOFTMAX || (epi == EPI_SIM && a.argmax));
    const double pass = fused ? 3.0 + 8.0 * (double)a.M * (double)a.N / 4e6 : 0.0;
    return p.cost + pass < large;
}

hipError_t launch_split(gs_dtype t, gs_dtype tout, bool b_nn, Epi epi, const GemmArgs &a_in, hipStream_t s) {
    if (a_in.M == 0 || a_in.N == 0) return hipSuccess;
    Plan p;
    if (!make_plan(t, b_nn, epi, a_in, p)) return hipErrorInvalidValue;
    const bool scores = epi == EPI_SIM || epi == EPI_SOFTMAX;
    GemmArgs a = a_in;
    if (epi == EPI_SOFTMAX) a.scale = a_in.scale * a_in.beta;    // the softmax acts on beta * score
    hipError_t e = (t == GS_BF16) ? launch_typed<bf16_t>(tout, b_nn, epi == EPI_BIND, scores, a, p, s)
                                  : launch_typed<float>(tout, b_nn, epi == EPI_BIND, scores, a, p, s);
    if (e != hipSuccess || !scores) return e;
    return launch_rows_pass(epi == EPI_SOFTMAX, static_cast<float *>(a.C), a.ldc, a.M, a.N,
                            epi == EPI_SOFTMAX ? nullptr : a.argmax, s);
}

}  // namespace gs
