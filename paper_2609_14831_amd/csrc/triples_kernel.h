// Contraction kernels of the Majorana bracket in triple space (see
// triples.hip for the plan and its check against the compiled records).
//
// With sigma(T, q) the sign of sorting mode q into the set T from behind and
// a4[T, q] = sigma(T, q) a[T + q], a2[w, q] = a[{w, q}] (antisymmetric), the
// action y = L(e) x of every record is
//   y[T + w]  = c sum over the 4 triples T of the string of
//               sigma(T, w) sum_q (e4[T, q] x2[w, q] - x4[T, q] e2[w, q])
//   y[{u, v}] = c sum over triples and single modes t outside {u, v} of
//               e4[t, u] x4[t, v] - x4[t, u] e4[t, v]
// (a single mode t stands for the quadratic x quadratic records).  Both are
// one matrix product per coefficient set and operand,
//   D[i][j] = sum_k R_e[i, k] S_x[j, k] - R_x[i, k] S_e[j, k],
// with i = T, j = w, k = q in the first and i = u, j = v, k = t in the second:
// the rows are read once per tile and not once per record (E / N = 235 .. 718
// times for 24 .. 64 modes), and there is no record stream.
//
// The products run on the matrix cores in FP64, v_mfma_f64_4x4x4_4b: four
// blocks of 4 x 4 x 4, one per coefficient set (77 TFLOP/s measured, as the
// 16x16x4 form; a vector FMA per record reaches the same peak but needs its
// operands from memory).  Operand lane l of an instruction is row l % 4,
// block (l / 4) % 4, k = l / 16; result lane l is column l % 4, block
// (l / 4) % 4, row l / 16.  Products of float operands are exact.
//
// Rows that do not exist (q in T, w = q, a mode past the last) are read as zero
// through an out-of-range buffer offset, so nothing is predicated; the combine
// recomputes any non-finite result from the records, which have no such terms.
#pragma once

#include "device.h"
#include "internal.h"

namespace cut {

struct TriArgs {
    // [mode][ntp]: row | sign << 31 | absent << 30, padded with absent entries: the
    // modes to a multiple of 8 plus 8, the columns by 16 past ntau
    const uint32_t* tab;
    const uint64_t* tmask;  // [nt] modes of the triple
    int32_t m, nt, ntau, ntp, nq;
    int64_t N;
    const void* A;
    const void* B;
    uint32_t bytesA, bytesB;  // from A / B to the end of the arrays
    int32_t lda, ldb;
    int32_t nsets, s0, s1;
    int32_t nred;             // operand columns summed over (A and B advance by nsets)
    const int32_t* nsteps;
    const int32_t* step;
    double* p4;               // [4][N][ldp]
    double* p2;               // [nstream][nq][ldp]
    int64_t ldp;
    int32_t nb2, nstream, nbp;  // quadratic blocks, streams (ranges of t), mode tile pairs
    int32_t nwt, ntt, per;      // quartic blocks: mode tiles, triple tiles, triple tiles per XCD
    int32_t chunks;             // blocks of sets
    const int4* tasks;          // outside-space targets: tiles (see OutTask)
    const uint32_t* bin;        // [k][64] binomials C(n, k)
    const uint32_t* pair2;      // colexicographic pairs y | z << 8
    const uint32_t* tri3;       // colexicographic triples x | y << 8 | z << 16
};

// Targets of a tile.  The two of E_L; and of E_C, for the degree-6 target Q:
//   y[Q] = c sum over its 10 cuts Q = U + V into triples
//          s(U, V) sum_q (e4[U, q] x4[V, q] - x4[U, q] e4[V, q]),
// s the sign of sorting U V.  With a the lowest and e < f the highest modes of
// Q fixed, L = {x, y, z} the rest (all between a and e), nine cuts have a
// single mode of L on one side: for each of
//   {x, a, e | y, z, f}   {x, a, f | y, z, e}   {x, e, f | y, z, a}
// the sums over q are a product of rows x and pairs yz, and the three are
// summed as one product over (cut, q): L receives it at (x; yz), (y; xz) and
// (z; xy), into partial rows 1 .. 3.  The tenth cut, L | a e f, is a product of
// the triples L and the modes f for fixed a and e, into partial row 0.
enum TriKind { TRI_QUARTIC, TRI_QUADRATIC, TRI_OUT3, TRI_OUT1 };

// A tile of outside-space targets: .x = a | e << 8 | f << 16 | (OUT1 ? 1 << 24 : 0),
// .y = first row (pair or triple), .z = first column, .w = rows of the product.
typedef int4 OutTask;

constexpr uint32_t kTriRow = 0xFFFFFFu, kTriSign = 0x80000000u, kTriAbsent = 0x40000000u;
constexpr uint32_t kTriOut = 0x80000000u;  // past every array (below 2 GiB)
constexpr int kTriW = 16;                  // modes of a tile

template <class T>
__device__ __forceinline__ T tri_signed(T v, uint32_t sgn) {
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v) ^ sgn);
    } else {
        return __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, v) ^ ((uint64_t)sgn << 32));
    }
}

typedef uint32_t tri_u4 __attribute__((ext_vector_type(4)));

// four consecutive sets of one row column
template <class T>
struct TriVec {
    tri_u4 v[sizeof(T) / 4];
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t voff, int32_t soff) {
#pragma unroll
        for (int h = 0; h < (int)sizeof(T) / 4; ++h)
            v[h] = __builtin_bit_cast(tri_u4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)(voff + 16u * h), soff, 0));
    }
    // to LDS (16-byte aligned), every element's sign flipped when sgn is set;
    // swap: a double's upper half first (see the caller)
    __device__ __forceinline__ void store(T* p, uint32_t sgn, bool swap) const {
        if constexpr (sizeof(T) == 4) {
            *reinterpret_cast<tri_u4*>(p) = v[0] ^ sgn;
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const tri_u4 f = v[h], g = v[1 - h];
                tri_u4 w;
                w.x = swap ? g.x : f.x;
                w.y = (swap ? g.y : f.y) ^ sgn;
                w.z = swap ? g.z : f.z;
                w.w = (swap ? g.w : f.w) ^ sgn;
                *reinterpret_cast<tri_u4*>(p + (swap ? 2 - 2 * h : 2 * h)) = w;
            }
        }
    }
};

__device__ __forceinline__ double tri_mfma(double a, double b, double c) {
    return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// Elements between the LDS rows of a block: SETS columns of C operands, padded
// so that the 16 rows of a fragment read start 4 (float) or 8 (double, in half
// a wavefront) banks apart.
template <int C, int SETS, class T>
constexpr int tri_stride() {
    return C * SETS + ((SETS > 4 || C % 2 == 0) ? 4 : 0);
}

// One block: 4 wavefronts are SQ set quads (4 SQ sets) x TW = 4 / SQ tiles of rows
// R; all share the 16 rows S.  Wavefront (set quad, tile) keeps the 4 TI x 16
// sums of NOPS operands for its 4 sets.  Per step of 4 k the block's rows go
// through one LDS buffer: the next step's rows are loaded into registers
// while the current step's products run, so the block holds them twice
// without a second buffer and two blocks fit a CU; the other block's products
// cover the copy between the two barriers.
// Bound by the latency of a step (about 1.6 us: two barriers, the table entries
// and then the rows from beyond L1), not by the products (0.39 of the launch).
// One stage of a flow at 40 modes, 64 sets, 5 float operands, against the
// segment kernel with shared-triple tiles: 2.78 -> 1.38 ms, of which the
// combine 0.29; 30 modes, 39 sets, 3 operands 2.4 times faster, one FP64
// action of 40 modes 180 -> 27 us (one-set kernel below).
// QUAD: the quadratic targets (R: modes u, S: modes v, k: triples and modes of
// one stream), else the quartic ones (R: triples, S: modes w, k: modes q).
struct TriTile {
    int r0, j0, kb, ke, stream;  // first row of R and S, range of k
    int set0;                    // first set of the block
    int sq, tw, u0;              // this wavefront: set quad, row tile, its first row
    int a, e, f, rows;           // outside-space tiles: fixed modes, rows of the product
};

// lexicographic rank of the triple i < j < k
__device__ __forceinline__ uint32_t tri_rank(const TriArgs& a, int i, int j, int k) {
    return (uint32_t)(a.nt - 1) - a.bin[3 * 64 + a.m - 1 - i] - a.bin[2 * 64 + a.m - 1 - j] - (uint32_t)(a.m - 1 - k);
}

// NJ: column tiles of 4 that exist (0: this wavefront has no sums and only
// stages); DIAG: only the tiles of the pairs u <= v.  Both are fixed at compile
// time: a branch around each product costs more than the product.
template <int NOPS, int SQ, int TI, class T, TriKind KIND, int NJ, bool DIAG>
__device__ __forceinline__ void tri_tile(const TriArgs& a, T* lds, const TriTile& w) {
    constexpr int C = NOPS + 1, SETS = 4 * SQ, TW = 4 / SQ, RS = TI / 4;
    constexpr int STRIDE = tri_stride<C, SETS, T>(), RROWS = TW * TI * 16;
    constexpr int NI = DIAG && NJ < TI ? NJ : TI;
    constexpr bool QUAD = KIND == TRI_QUADRATIC, OUT = KIND == TRI_OUT3 || KIND == TRI_OUT1;
    const int m = a.m, nt = a.nt, ntp = a.ntp;
    const int lane = threadIdx.x & 63;
    // staging: slot h of thread t holds the 4 sets 4 (t % SQ) .. of one (row, k)
    const int p4 = (int)threadIdx.x % SQ, rk = (int)threadIdx.x / SQ;
    const auto rsTab = row_rsrc(a.tab, 0x7FFFFFFF);
    const uint32_t lda_b = (uint32_t)a.lda * (uint32_t)sizeof(T), ldb_b = (uint32_t)a.ldb * (uint32_t)sizeof(T);
    const uint32_t lo = (uint32_t)(w.set0 + 4 * p4) * (uint32_t)sizeof(T);
    const int32_t cstep = a.nsets * (int32_t)sizeof(T);
    uint32_t ie[RS + 1];  // table index of each slot's entry at k = 0, slot RS: S
    const uint32_t kr = QUAD ? 1u : (uint32_t)ntp, ks = OUT ? (uint32_t)ntp : 1u;  // its step per k
    const bool sact = rk < 64;  // S slots: 16 rows x 4 k
    // LDS row (tile, k, row): neighbouring threads take neighbouring k, whose
    // rows lie 16 banks apart
    const int lr = rk / 16 * 16 + (rk & 3) * 4 + ((rk >> 2) & 3);
    const int rx = w.r0 + rk / 16 * 4 + ((rk >> 2) & 3);            // slot 0's row of R, slot h 16 TW further
    const int sx = w.j0 + (rk & 63) / 16 * 4 + ((rk >> 2) & 3), sk = rk & 3;
    if constexpr (!OUT) {
#pragma unroll
        for (int h = 0; h < RS; ++h) {
            const int x = rx + h * (16 * TW);
            if constexpr (QUAD) ie[h] = (uint32_t)(x < m ? x : m) * (uint32_t)ntp + (uint32_t)sk;  // row m: absent
            else ie[h] = (uint32_t)(x < nt ? x : nt - 1) + (uint32_t)sk * (uint32_t)ntp;
        }
        ie[RS] = (uint32_t)(sx < m ? sx : m) * (uint32_t)ntp + (uint32_t)(QUAD ? sk : nt + sk);
    }
    const int js = lane & 3, bs = (lane >> 2) & 3, is = lane >> 4;
    double acc[TI][NJ > 0 ? NJ : 1][NOPS];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int op = 0; op < NOPS; ++op) acc[i][j][op] = 0.0;

    // operand columns summed over; outside-space tiles: the three cuts
    const int nred = KIND == TRI_OUT3 ? 3 : KIND == TRI_OUT1 ? 1 : a.nred;
    for (int red = 0; red < nred; ++red) {
        const uint32_t ro = OUT ? 0u : (uint32_t)red * (uint32_t)cstep;
        // the first cut's sign against the others' (13, 8 and 4 + #{y, z > x}
        // inversions of V U), on its rows R
        const uint32_t flip = KIND == TRI_OUT3 && red == 0 ? kTriSign : 0u;
        if constexpr (OUT) {
            // triples of the slots' rows; past the last row the padding columns, absent
#pragma unroll
            for (int h = 0; h < RS; ++h) {
                const int x = rx + h * (16 * TW);
                uint32_t t = (uint32_t)a.ntau;
                if (x < w.rows) {
                    if constexpr (KIND == TRI_OUT1) {
                        const uint32_t l = a.tri3[x];
                        t = tri_rank(a, w.a + 1 + (int)(l & 255), w.a + 1 + (int)(l >> 8 & 255), w.a + 1 + (int)(l >> 16));
                    } else {
                        const uint32_t l = a.pair2[x];
                        const int y = w.a + 1 + (int)(l & 255), z = w.a + 1 + (int)(l >> 8);
                        t = red == 2 ? tri_rank(a, w.a, y, z) : tri_rank(a, y, z, red ? w.e : w.f);
                    }
                }
                ie[h] = (uint32_t)sk * (uint32_t)ntp + t;
            }
            uint32_t t = (uint32_t)a.ntau;
            if constexpr (KIND == TRI_OUT1) {
                if (w.e + 1 + sx < m) t = tri_rank(a, w.a, w.e, w.e + 1 + sx);
            } else {
                const int x = w.a + 1 + sx;
                if (x < w.e) t = red == 2 ? tri_rank(a, x, w.e, w.f) : tri_rank(a, w.a, x, red ? w.f : w.e);
            }
            ie[RS] = (uint32_t)sk * (uint32_t)ntp + t;
        }
        const auto rsA = row_rsrc((const char*)a.A + ro, (int64_t)(a.bytesA - ro));
        const auto rsB = row_rsrc((const char*)a.B + ro, (int64_t)(a.bytesB - ro));
        uint32_t e[RS + 1], sg[RS + 1];
        TriVec<T> st[RS + 1][C];
        auto entries = [&](int k) {
#pragma unroll
            for (int h = 0; h < RS; ++h) e[h] = buf_load<uint32_t>(rsTab, (ie[h] + (uint32_t)k * kr) * 4u, 0);
            e[RS] = buf_load<uint32_t>(rsTab, (ie[RS] + (uint32_t)k * ks) * 4u, 0);
        };
        auto load = [&]() {
#pragma unroll
            for (int h = 0; h <= RS; ++h) {
                // where the block has fewer than 256 slots of S the others load nothing
                const bool out = (e[h] & kTriAbsent) != 0 || (h == RS && SQ < 4 && !sact);
                // a2[w, q]: + for w < q, where sigma({q}, w) is -
                sg[h] = ((KIND == TRI_QUARTIC && h == RS ? ~e[h] : e[h]) & kTriSign) ^ (h < RS ? flip : 0u);
                const uint32_t va = (out ? kTriOut : (e[h] & kTriRow) * lda_b) + lo;
                const uint32_t vb = (out ? kTriOut : (e[h] & kTriRow) * ldb_b) + lo;
#pragma unroll
                for (int op = 0; op < NOPS; ++op) st[h][op].load(rsB, vb, op * cstep);
                st[h][NOPS].load(rsA, va, 0);
            }
        };
        // The two 16-byte halves of a slot's doubles in different orders in rows
        // that share banks.  Blocks of 4 and 8 sets: 40 modes x 8 sets x 3, one
        // step 748 -> 694 us; of 16 sets the selects cost more (2 %) than they save.
        const bool swap = SQ < 4 && (rk & 2) != 0;
        auto store = [&]() {
#pragma unroll
            for (int h = 0; h <= RS; ++h) {
                if (h == RS && SQ < 4 && !sact) continue;
                T* p = lds + ((h < RS ? h * (64 * TW) : RROWS) + lr) * STRIDE + 4 * p4;
#pragma unroll
                for (int c = 0; c < C; ++c) st[h][c].store(p + c * SETS, sg[h], swap);
            }
        };
        const T* fr = lds + (w.tw * TI * 16 + is * 4 + js) * STRIDE + 4 * w.sq + bs;
        const T* fs = lds + (RROWS + is * 4 + js) * STRIDE + 4 * w.sq + bs;
        // past the end the first entries again: loaded, not used
        auto at = [&](int k) { return k < w.ke ? k : w.kb; };
        entries(w.kb);
        load();
        entries(at(w.kb + 4));
        for (int k = w.kb; k < w.ke; k += 4) {
            __syncthreads();  // the previous step's reads
            store();
            __syncthreads();
            load();
            entries(at(k + 8));
            if constexpr (NJ > 0) {
                __builtin_amdgcn_sched_barrier(0);
                double er[NI], es[NJ];
#pragma unroll
                for (int i = 0; i < NI; ++i) er[i] = (double)fr[i * 16 * STRIDE + NOPS * SETS];
#pragma unroll
                for (int j = 0; j < NJ; ++j) es[j] = -(double)fs[j * 16 * STRIDE + NOPS * SETS];
#pragma unroll
                for (int op = 0; op < NOPS; ++op) {
                    double xr[NI], xs[NJ];
#pragma unroll
                    for (int i = 0; i < NI; ++i) xr[i] = (double)fr[i * 16 * STRIDE + op * SETS];
#pragma unroll
                    for (int j = 0; j < NJ; ++j) xs[j] = (double)fs[j * 16 * STRIDE + op * SETS];
                    // the two products of a sum stay apart: an instruction waits
                    // for the one whose result it adds to
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int j = 0; j < NJ; ++j)
#pragma unroll
                            for (int i = 0; i < NI; ++i) {
                                if (DIAG && i > j) continue;
                                acc[i][j][op] = tri_mfma(h ? xr[i] : er[i], h ? es[j] : xs[j], acc[i][j][op]);
                            }
                    // only LDS reads move ahead of an operand's products (its
                    // converted fragments would not fit beside the sums)
                    __builtin_amdgcn_sched_barrier(0x100);
                }
            }
        }
        __syncthreads();
    }
    if constexpr (NJ > 0) {
        const int s = w.set0 + 4 * w.sq + bs;
        if (s >= a.s1 || (a.nsteps != nullptr && a.nsteps[s] <= *a.step)) return;
        if constexpr (OUT) {
            auto bin = [&](int k, int c) { return a.bin[k * 64 + m - 1 - c]; };
            // lexicographic rank of the target, less its terms of L (OUT1: and of f)
            const uint32_t base = (uint32_t)(a.N - 1) - bin(6, w.a) - bin(2, w.e);
            uint32_t l[NI];
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int x = w.u0 + 4 * i + is;
                l[i] = x >= w.rows ? 0u : KIND == TRI_OUT1 ? a.tri3[x] : a.pair2[x];
            }
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                if (w.u0 + 4 * i + is >= w.rows) continue;
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    int c0 = w.a + 1 + (int)(l[i] & 255), c1 = w.a + 1 + (int)(l[i] >> 8 & 255), c2, f, slot;
                    uint32_t sgn = 0;
                    if constexpr (KIND == TRI_OUT1) {
                        c2 = w.a + 1 + (int)(l[i] >> 16);
                        f = w.e + 1 + w.j0 + 4 * j + js;
                        if (f >= m) continue;
                        slot = 0;
                        sgn = kTriSign;  // 3 inversions of L a e f
                    } else {
                        const int x = w.a + 1 + w.j0 + 4 * j + js;
                        if (x >= w.e || x == c0 || x == c1) continue;
                        f = w.f;
                        slot = 1 + (x < c1) + (x < c0);
                        if (slot == 2) sgn = kTriSign;
                        c2 = c1 > x ? c1 : x;
                        c1 = x < c0 ? c0 : x < c1 ? x : c1;
                        c0 = x < c0 ? x : c0;
                    }
                    const uint32_t row = base - bin(1, f) - bin(5, c0) - bin(4, c1) - bin(3, c2);
                    double* p = a.p4 + ((int64_t)slot * a.N + row) * a.ldp + s;
#pragma unroll
                    for (int op = 0; op < NOPS; ++op) p[(int64_t)op * a.nsets] = tri_signed<double>(acc[i][j][op], sgn);
                }
            }
            return;
        }
        // every target's table entry before the first store: a load behind the
        // stores would wait for them
        uint32_t et[NI][NJ];
        uint64_t tm[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int x = w.u0 + 4 * i + is;  // row of the result lane
            if constexpr (!QUAD) tm[i] = a.tmask[x < nt ? x : nt - 1];
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int y = w.j0 + 4 * j + js;
                if constexpr (QUAD) et[i][j] = a.tab[(uint32_t)(x < m ? x : m) * (uint32_t)ntp + (uint32_t)(nt + y)];
                else et[i][j] = a.tab[(uint32_t)(y < m ? y : m) * (uint32_t)ntp + (uint32_t)(x < nt ? x : nt - 1)];
            }
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int x = w.u0 + 4 * i + is;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                if (DIAG && i > j) continue;
                const int y = w.j0 + 4 * j + js;
                double* p;
                uint32_t sgn = 0;
                if constexpr (QUAD) {
                    if (x >= y || y >= m) continue;
                    p = a.p2 + ((int64_t)w.stream * a.nq + (et[i][j] & kTriRow)) * a.ldp + s;
                } else {
                    if (x >= nt || (et[i][j] & kTriAbsent)) continue;
                    const int slot = __popcll(tm[i] & ((1ull << y) - 1));  // position of w in the string
                    sgn = et[i][j] & kTriSign;
                    p = a.p4 + ((int64_t)slot * a.N + (et[i][j] & kTriRow)) * a.ldp + s;
                }
#pragma unroll
                for (int op = 0; op < NOPS; ++op) p[(int64_t)op * a.nsets] = tri_signed<double>(acc[i][j][op], sgn);
            }
        }
    }
}

template <int NOPS, int SQ, int TI, class T, bool QUAD>
__device__ __forceinline__ void tri_block(const TriArgs& a, T* lds, int b) {
    constexpr int TW = 4 / SQ;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    TriTile w;
    w.sq = wave % SQ;
    w.tw = wave / SQ;
    w.stream = 0;
    // block b runs on XCD b % 8; there the set blocks of one tile follow each
    // other: two of them share the rows' cache lines
    const int i = (b >> 3) / a.chunks;
    w.set0 = a.s0 + (b >> 3) % a.chunks * (4 * SQ);
    if constexpr (QUAD) {
        // the tile pairs of one stream read the same rows: they run on one XCD
        const int sx = (a.nstream + 7) / 8;
        int bp = i % a.nbp;
        w.stream = (b & 7) * sx + i / a.nbp;
        if (w.stream >= a.nstream) return;
        int vt = 0;
        while (bp > vt / TW) bp -= vt++ / TW + 1;
        w.r0 = bp * (TW * 4 * TI);
        w.j0 = vt * kTriW;
        const int n4 = (a.ntau + 3) / 4;
        w.kb = (int)((int64_t)w.stream * n4 / a.nstream) * 4;
        w.ke = (int)((int64_t)(w.stream + 1) * n4 / a.nstream) * 4;
    } else {
        // so do the mode tiles of one triple tile
        const int tt = (b & 7) * a.per + i / a.nwt;
        if (tt >= a.ntt) return;
        w.r0 = tt * (TW * 4 * TI);
        w.j0 = (i % a.nwt) * kTriW;
        w.kb = 0;
        w.ke = a.m;
    }
    w.u0 = w.r0 + w.tw * (4 * TI);
    const bool half = a.m - w.j0 <= 8;  // no more than two column tiles exist
    const bool work = w.set0 + 4 * w.sq < a.s1 && (QUAD ? (w.u0 <= w.j0 && w.u0 < a.m) : w.u0 < a.nt);
    constexpr TriKind KIND = QUAD ? TRI_QUADRATIC : TRI_QUARTIC;
    if (!work) tri_tile<NOPS, SQ, TI, T, KIND, 0, false>(a, lds, w);
    else if (QUAD && w.u0 == w.j0) {
        if (half) tri_tile<NOPS, SQ, TI, T, KIND, 2, QUAD>(a, lds, w);
        else tri_tile<NOPS, SQ, TI, T, KIND, 4, QUAD>(a, lds, w);
    } else {
        if (half) tri_tile<NOPS, SQ, TI, T, KIND, 2, false>(a, lds, w);
        else tri_tile<NOPS, SQ, TI, T, KIND, 4, false>(a, lds, w);
    }
}

// one tile of outside-space targets, for the set block b % chunks
template <int NOPS, int SQ, class T, TriKind KIND>
__device__ __forceinline__ void tri_outside(const TriArgs& a, T* lds, const OutTask& t, int chunk) {
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    TriTile w;
    w.sq = wave % SQ;
    w.tw = wave / SQ;
    w.stream = 0;
    w.set0 = a.s0 + chunk * (4 * SQ);
    w.a = t.x & 255;
    w.e = t.x >> 8 & 255;
    w.f = t.x >> 16 & 255;
    w.rows = t.w;
    w.r0 = t.y;
    w.j0 = t.z;
    w.kb = 0;
    w.ke = a.m;
    w.u0 = w.r0 + w.tw * 16;
    const int cols = (KIND == TRI_OUT1 ? a.m : w.e) - (KIND == TRI_OUT1 ? w.e : w.a) - 1;
    if (w.set0 + 4 * w.sq >= a.s1 || w.u0 >= w.rows) tri_tile<NOPS, SQ, 4, T, KIND, 0, false>(a, lds, w);
    else if (cols - w.j0 <= 8) tri_tile<NOPS, SQ, 4, T, KIND, 2, false>(a, lds, w);
    else tri_tile<NOPS, SQ, 4, T, KIND, 4, false>(a, lds, w);
}

// Bound like the tiles of E_L by the latency of a step, and by padding: 0.54 of
// the 16 x 16 tiles' elements are targets at 24 modes, 0.65 at 32.  24 modes, 8
// sets x 3 FP64 operands: 0.30 ms, the products alone 0.10; the combine 0.02.
template <int NOPS, int SQ, class T>
__global__ __launch_bounds__(256, 2) void k_outside(TriArgs a) {
    extern __shared__ __align__(16) unsigned char tri_lds[];
    const int chunk = (int)blockIdx.x % a.chunks;
    const OutTask t = a.tasks[blockIdx.x / a.chunks];
    if (t.x >> 24) tri_outside<NOPS, SQ, T, TRI_OUT1>(a, reinterpret_cast<T*>(tri_lds), t, chunk);
    else tri_outside<NOPS, SQ, T, TRI_OUT3>(a, reinterpret_cast<T*>(tri_lds), t, chunk);
}

template <int NOPS, int SQ, int TI, class T>
__global__ __launch_bounds__(256, 2) void k_triples(TriArgs a) {
    extern __shared__ __align__(16) unsigned char tri_lds[];
    const int b = (int)blockIdx.x;
    if (b < a.nb2) tri_block<NOPS, SQ, 4, T, true>(a, reinterpret_cast<T*>(tri_lds), b);
    else tri_block<NOPS, SQ, TI, T, false>(a, reinterpret_cast<T*>(tri_lds), b - a.nb2);
}

// One coefficient set: the four blocks of an instruction are four slices of k
// (16 per step), added at the end; every wavefront owns a 16 x 8 tile of its
// own and loads its operands straight into registers (no LDS, no barriers:
// the sizes are small and latency counts).
template <int NOPS, class T, bool QUAD>
__device__ __forceinline__ void tri_wave(const TriArgs& a, int wv) {
    constexpr int C = NOPS + 1, NJ = 2, NF = 4 + NJ;  // fragments per operand
    const int m = a.m, nt = a.nt, ntp = a.ntp;
    const int lane = threadIdx.x & 63;
    const int i0 = lane & 3, b = (lane >> 2) & 3, kk = lane >> 4;
    int r0, j0, kb, ke, stream = 0;
    if constexpr (QUAD) {
        int bp = wv % a.nbp;
        stream = wv / a.nbp;
        int vt = 0;
        while (bp > vt / 2) bp -= vt++ / 2 + 1;
        r0 = bp * 16;
        j0 = vt * 8;
        const int n16 = (a.ntau + 15) / 16;
        kb = (int)((int64_t)stream * n16 / a.nstream) * 16;
        ke = (int)((int64_t)(stream + 1) * n16 / a.nstream) * 16;
    } else {
        r0 = (wv / a.nwt) * 16;
        j0 = (wv % a.nwt) * 8;
        kb = 0;
        ke = m;
    }
    const auto rsTab = row_rsrc(a.tab, 0x7FFFFFFF);
    const uint32_t lda_b = (uint32_t)a.lda * (uint32_t)sizeof(T), ldb_b = (uint32_t)a.ldb * (uint32_t)sizeof(T);
    const uint32_t kr = QUAD ? 1u : (uint32_t)ntp;
    uint32_t ie[NF];  // table index of each fragment's entry at k = 0: rows of R, then of S
#pragma unroll
    for (int t = 0; t < NF; ++t) {
        const int x = r0 + 4 * t + i0, y = j0 + 4 * (t - 4) + i0, k = 4 * b + kk;
        if (t >= 4) ie[t] = (uint32_t)(y < m ? y : m) * (uint32_t)ntp + (uint32_t)(QUAD ? k : nt + k);
        else if (QUAD) ie[t] = (uint32_t)(x < m ? x : m) * (uint32_t)ntp + (uint32_t)k;
        else ie[t] = (uint32_t)(x < nt ? x : nt - 1) + (uint32_t)k * (uint32_t)ntp;
    }
    double acc[4][NJ][NOPS];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int op = 0; op < NOPS; ++op) acc[i][j][op] = 0.0;
    for (int red = 0; red < a.nred; ++red) {
        const uint32_t ro = (uint32_t)red * (uint32_t)sizeof(T);
        const auto rsA = row_rsrc((const char*)a.A + ro, (int64_t)(a.bytesA - ro));
        const auto rsB = row_rsrc((const char*)a.B + ro, (int64_t)(a.bytesB - ro));
        uint32_t e[NF], sg[NF];
        T v[NF][C];
        auto entries = [&](int k) {
#pragma unroll
            for (int t = 0; t < NF; ++t)
                e[t] = buf_load<uint32_t>(rsTab, (ie[t] + (uint32_t)k * (t < 4 ? kr : 1u)) * 4u, 0);
        };
        auto load = [&]() {
#pragma unroll
            for (int t = 0; t < NF; ++t) {
                const bool out = (e[t] & kTriAbsent) != 0;
                sg[t] = (!QUAD && t >= 4 ? ~e[t] : e[t]) & kTriSign;
                const uint32_t va = out ? kTriOut : (e[t] & kTriRow) * lda_b;
                const uint32_t vb = out ? kTriOut : (e[t] & kTriRow) * ldb_b;
#pragma unroll
                for (int op = 0; op < NOPS; ++op) v[t][op] = buf_load<T>(rsB, vb, op * (int32_t)sizeof(T));
                v[t][NOPS] = buf_load<T>(rsA, va, 0);
            }
        };
        entries(kb);
        load();
        entries(kb + 16 < ke ? kb + 16 : kb);
        for (int k = kb; k < ke; k += 16) {
            double f[NF][C];
#pragma unroll
            for (int t = 0; t < NF; ++t)
#pragma unroll
                for (int c = 0; c < C; ++c)
                    f[t][c] = (double)tri_signed<T>(v[t][c], t >= 4 && c == NOPS ? sg[t] ^ kTriSign : sg[t]);
            load();
            entries(k + 32 < ke ? k + 32 : kb);
#pragma unroll
            for (int op = 0; op < NOPS; ++op)
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int j = 0; j < NJ; ++j)
                            acc[i][j][op] = tri_mfma(f[i][h ? op : NOPS], f[4 + j][h ? NOPS : op], acc[i][j][op]);
        }
    }
    // the four slices: block pairs 2 apart, then 1 apart, each keeping the row
    // tiles of its block number
    const int x = r0 + 4 * b + kk;  // row of the result lane: tile b
    uint32_t et[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int y = j0 + 4 * j + i0;
        if constexpr (QUAD) et[j] = a.tab[(uint32_t)(x < m ? x : m) * (uint32_t)ntp + (uint32_t)(nt + y)];
        else et[j] = a.tab[(uint32_t)(y < m ? y : m) * (uint32_t)ntp + (uint32_t)(x < nt ? x : nt - 1)];
    }
    const uint64_t tm = QUAD ? 0 : a.tmask[x < nt ? x : nt - 1];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int y = j0 + 4 * j + i0;  // column of the result lane
        double r[NOPS];
#pragma unroll
        for (int op = 0; op < NOPS; ++op) {
            const bool hi = (b & 2) != 0, odd = (b & 1) != 0;
            double k0 = hi ? acc[2][j][op] : acc[0][j][op], k1 = hi ? acc[3][j][op] : acc[1][j][op];
            k0 += __shfl_xor(hi ? acc[0][j][op] : acc[2][j][op], 8);
            k1 += __shfl_xor(hi ? acc[1][j][op] : acc[3][j][op], 8);
            r[op] = (odd ? k1 : k0) + __shfl_xor(odd ? k0 : k1, 4);
        }
        double* p;
        uint32_t sgn = 0;
        if constexpr (QUAD) {
            if (x >= y || y >= m) continue;
            p = a.p2 + ((int64_t)stream * a.nq + (et[j] & kTriRow)) * a.ldp;
        } else {
            if (x >= nt || (et[j] & kTriAbsent)) continue;
            const int slot = __popcll(tm & ((1ull << y) - 1));
            sgn = et[j] & kTriSign;
            p = a.p4 + ((int64_t)slot * a.N + (et[j] & kTriRow)) * a.ldp;
        }
#pragma unroll
        for (int op = 0; op < NOPS; ++op) p[op] = tri_signed<double>(r[op], sgn);
    }
}

template <int NOPS, class T>
__global__ __launch_bounds__(256, 2) void k_triples1(TriArgs a) {
    if (a.nsteps != nullptr && a.nsteps[0] <= *a.step) return;
    const int wv = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    if (wv < a.nb2) tri_wave<NOPS, T, true>(a, wv);
    else if (wv - a.nb2 < a.ntt * a.nwt) tri_wave<NOPS, T, false>(a, wv - a.nb2);
}

// operand columns of one launch: the most whose sums and staged rows stay in
// registers; row tiles of 4 per wavefront: 8 where they do
template <class T>
constexpr int tri_ops() { return sizeof(T) == 4 ? 5 : 3; }
constexpr int tri_rows(int nops, int esz) { return nops * esz <= 8 ? 8 : 4; }

template <int NOPS, int SQ, int TI, class T>
static void launch_triples_k(const TriArgs& a, dim3 grid, hipStream_t s) {
    constexpr int TW = 4 / SQ;
    constexpr size_t lds = (size_t)(TW * TI * 16 + 64) * tri_stride<NOPS + 1, 4 * SQ, T>() * sizeof(T);
    hipLaunchKernelGGL((k_triples<NOPS, SQ, TI, T>), grid, dim3(256), lds, s, a);
}

template <int NOPS, class T>
static void launch_triples_n(const TriArgs& a, int sq, int ti, dim3 grid, hipStream_t s) {
    if (sq == 0) {
        hipLaunchKernelGGL((k_triples1<NOPS, T>), grid, dim3(256), 0, s, a);
    } else if (sq == 4) {
        if constexpr (tri_rows(NOPS, sizeof(T)) == 8) {
            if (ti == 8) {
                launch_triples_k<NOPS, 4, 8, T>(a, grid, s);
                return;
            }
        }
        launch_triples_k<NOPS, 4, 4, T>(a, grid, s);
    } else if (sq == 2) {
        launch_triples_k<NOPS, 2, 4, T>(a, grid, s);
    } else {
        launch_triples_k<NOPS, 1, 4, T>(a, grid, s);
    }
}

// one launch over `nops` operand columns; sq: set quads per block (0: one set),
// ti: row tiles of 4 per wavefront of the quartic blocks
template <class T>
void launch_triples_t(const TriArgs& a, int nops, int sq, int ti, dim3 grid, hipStream_t s);

// one launch over `nops` operand columns of the outside-space tiles
template <int NOPS, class T>
static void launch_outside_n(const TriArgs& a, int sq, dim3 grid, hipStream_t s) {
    auto lds = [](int q) -> size_t {
        const int stride = q == 4 ? tri_stride<NOPS + 1, 16, T>() : q == 2 ? tri_stride<NOPS + 1, 8, T>() : tri_stride<NOPS + 1, 4, T>();
        return (size_t)(4 / q * 64 + 64) * stride * sizeof(T);
    };
    if (sq == 4) hipLaunchKernelGGL((k_outside<NOPS, 4, T>), grid, dim3(256), lds(4), s, a);
    else if (sq == 2) hipLaunchKernelGGL((k_outside<NOPS, 2, T>), grid, dim3(256), lds(2), s, a);
    else hipLaunchKernelGGL((k_outside<NOPS, 1, T>), grid, dim3(256), lds(1), s, a);
}
template <class T>
void launch_outside_t(const TriArgs& a, int nops, int sq, dim3 grid, hipStream_t s);

}  // namespace cut
