// Whole flow of a small graph in one launch (Sec. 2.2, classic RK4 on the
// stage right-hand side L(eta(Z_h)) Z): the sets of a batch are independent, so
// one workgroup per set keeps its state, stage operands, accumulator and
// generator in LDS over all the steps and needs no other workgroup.
//
// A step of the general path is eight dependent launches of at least 3.5 us
// each (4 generator evaluations, 4 actions); a small graph's records take less
// than that.  Here a stage costs two barriers and a chain of dependent reads of
// offsets, records and rows, all in LDS where they fit (else records come from
// L2, four per lane in flight).  200 steps of the 8 x 8 one-body flow: 8.4 ->
// 0.98 ms (1.2 us a stage; 1.9 with the records in L2 and shuffles through LDS).
#include <algorithm>
#include <type_traits>

#include "device.h"
#include "internal.h"

namespace cut {

struct SmallFlow {
    const int64_t* off;   // E_L by target
    const uint2* rec;
    const int64_t* goff;  // E_eta by target (Wegner generator)
    const uint2* grec;
    const int4* stencil;  // G2 (null: Wegner)
    const int32_t* pairs;
    const double* ftab;
    double gsign, d2, ds;
    int32_t N, NG, nsets, f32, nrec, ngrec;
    const int32_t* nsteps;
    int64_t t0, t1, ckpt_every;
    double* z;     // [N][nops][nsets]
    double* ckpt;  // slot t / ckpt_every of every multiple t in [t0, t1) (null: none)
};

constexpr int kSmallThreads = 1024, kSmallLanes = 16;  // lanes of one target's records

__device__ __forceinline__ double rec_factor(uint2 r) {
    return (double)__builtin_bit_cast(float, (r.x & 0xFF000000u) | ((r.y >> 24) << 16));
}

// sum over the 16 lanes of a row of the wavefront, in every one of them
__device__ __forceinline__ double lanes_sum(double v) {
    auto ror = [](double x, auto n) {
        const uint64_t u = __builtin_bit_cast(uint64_t, x);
        constexpr int ctrl = 0x120 + decltype(n)::value;  // row_ror
        const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, ctrl, 0xF, 0xF, false);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), ctrl, 0xF, 0xF, false);
        return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
    };
    v += ror(v, std::integral_constant<int, 8>());
    v += ror(v, std::integral_constant<int, 4>());
    v += ror(v, std::integral_constant<int, 2>());
    v += ror(v, std::integral_constant<int, 1>());
    return v;
}

// sum over the records [beg, end) of factor x a[i] x b[j][op], in each of the 16
// lanes; BATCH records per lane are loaded before the first is used
template <int NOPS, int BATCH>
__device__ __forceinline__ void small_sum(int beg, int end, const uint2* rec, int l, const double* a,
                                          const double* b, double* v) {
#pragma unroll
    for (int op = 0; op < NOPS; ++op) v[op] = 0.0;
    for (int e = beg + l; e < end; e += BATCH * kSmallLanes) {
        uint2 r[BATCH];
#pragma unroll
        for (int t = 0; t < BATCH; ++t) r[t] = rec[e + t * kSmallLanes < end ? e + t * kSmallLanes : e];
#pragma unroll
        for (int t = 0; t < BATCH; ++t) {
            const bool in = e + t * kSmallLanes < end;
            const double fa = rec_factor(r[t]) * a[r[t].x & 0xFFFFFFu];
            const double* x = b + (int)(r[t].y & 0xFFFFFFu) * NOPS;
#pragma unroll
            for (int op = 0; op < NOPS; ++op) {
                const double w = __builtin_fma(fa, x[op], v[op]);
                v[op] = in ? w : v[op];
            }
        }
    }
#pragma unroll
    for (int op = 0; op < NOPS; ++op) v[op] = lanes_sum(v[op]);
}

// INLDS: the records are copied into LDS behind the state once per launch.
template <int NOPS, bool INLDS>
__global__ __launch_bounds__(kSmallThreads) void k_flow_small(SmallFlow a) {
    extern __shared__ double small_lds[];
    const int s = (int)blockIdx.x, tid = (int)threadIdx.x;
    const int M = a.N * NOPS;
    double *z = small_lds, *acc = z + M, *xa = acc + M, *xb = xa + M, *h = xb + M, *eta = h + a.N;
    int32_t* off = (int32_t*)(eta + a.NG);  // both record sets' offsets
    int32_t* goff = off + a.N + 1;
    uint2* lrec = (uint2*)(eta + a.NG + (a.N + a.NG + 3) / 2);
    uint2* lgrec = lrec + a.nrec;
    for (int q = tid; q <= a.N; q += kSmallThreads) off[q] = (int32_t)a.off[q];
    if (!a.stencil)
        for (int q = tid; q <= a.NG; q += kSmallThreads) goff[q] = (int32_t)a.goff[q];
    if constexpr (INLDS) {
        for (int q = tid; q < a.nrec; q += kSmallThreads) lrec[q] = a.rec[q];
        for (int q = tid; q < a.ngrec; q += kSmallThreads) lgrec[q] = a.grec[q];
    }
    const uint2* rec = INLDS ? lrec : a.rec;
    const uint2* grec = INLDS ? lgrec : a.grec;
    auto shadow = [&](double v) { return a.f32 ? (double)(float)v : v; };
    double* zg = a.z + s;
    for (int q = tid; q < M; q += kSmallThreads) {
        const double v = zg[(int64_t)q * a.nsets];
        z[q] = v;
        xa[q] = shadow(v);
        if (q % NOPS == 0) h[q / NOPS] = v;
    }
    __syncthreads();
    const int l = tid % kSmallLanes, grp = tid / kSmallLanes;
    constexpr int kBatch = INLDS ? 2 : 4;
    constexpr int kGroups = kSmallThreads / kSmallLanes;
    const int64_t last = a.nsteps[s];
    for (int64_t t = a.t0; t < a.t1; ++t) {
        if (a.ckpt && t % a.ckpt_every == 0) {
            double* c = a.ckpt + (t / a.ckpt_every) * ((int64_t)M * a.nsets) + s;
            for (int q = tid; q < M; q += kSmallThreads) c[(int64_t)q * a.nsets] = z[q];
        }
        if (t >= last) {
            if (a.ckpt) continue;  // the later checkpoints hold the finished state
            break;
        }
        for (int st = 0; st < 4; ++st) {
            if (a.stencil) {
                for (int S = tid; S < a.N; S += kSmallThreads) {
                    double num = 0.0, q = 0.0;
                    bool has = false;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const int4 e = a.stencil[(int64_t)S * 4 + k];
                        if (e.x < 0) continue;
                        has = true;
                        const double ce = a.ftab[e.z] * h[a.pairs[e.y]];
                        num = __builtin_fma(ce, h[e.x], num);
                        q = __builtin_fma(ce, ce, q);
                    }
                    eta[S] = has ? shadow(a.gsign * num / (q + a.d2)) : 0.0;
                }
            } else {
                for (int row = grp; row < a.NG; row += kGroups) {
                    double v[1];
                    small_sum<1, kBatch>(goff[row], goff[row + 1], grec, l, h, h, v);
                    if (l == 0) eta[row] = shadow(a.gsign * v[0]);
                }
            }
            __syncthreads();
            const double* x = (st & 1) ? xb : xa;
            double* xn = (st & 1) ? xa : xb;
            for (int row = grp; row < a.N; row += kGroups) {
                double v[NOPS];
                small_sum<NOPS, kBatch>(off[row], off[row + 1], rec, l, eta, x, v);
                double f = v[0];
#pragma unroll
                for (int op = 1; op < NOPS; ++op) f = l == op ? v[op] : f;
                if (l < NOPS) {
                    const int q = row * NOPS + l;
                    const double zk = z[q];
                    double nxt;
                    if (st == 0) {
                        acc[q] = zk + (a.ds / 6.0) * f;
                        nxt = zk + 0.5 * a.ds * f;
                    } else if (st < 3) {
                        acc[q] += (a.ds / 3.0) * f;
                        nxt = zk + (st == 1 ? 0.5 * a.ds : a.ds) * f;
                    } else {
                        nxt = acc[q] + (a.ds / 6.0) * f;
                        z[q] = nxt;
                    }
                    xn[q] = shadow(nxt);
                    if (l == 0) h[row] = nxt;
                }
            }
            __syncthreads();
        }
    }
    for (int q = tid; q < M; q += kSmallThreads) zg[(int64_t)q * a.nsets] = z[q];
}

// Records up to which one workgroup per set is faster than launches over the
// whole card, for any batch and for one whose launches take 64-lane groups (more
// than 32 sets).  Per step of an 8-step call, us, launches -> here:
//   8 modes (E = 3696), 1 set 48 -> 14, 4 sets x 3 operands 51 -> 17
//   10 modes (15840), 4 x 5 FP64 58 -> 39, 1 x 5 float 56 -> 39
//   12 modes (48840), 64 x 1 117 -> 54, 64 x 5 float 151 -> 97; but 1 x 1 48 -> 53, 4 x 5 68 -> 95
constexpr int64_t kSmallRecords = 20000, kSmallRecordsWide = 60000;

// Sets up to which it is: two workgroups are resident per CU, so past 512 sets its
// time grows with their number, while a launch over the card is not yet full.  An
// 8-step call, ms, launches -> here (G2; 12 modes in float have the wide graphs' line):
//   up to it   8 modes, 2048 sets float 0.82 -> 0.78, FP64 0.98 -> 0.79; 6 modes, 2048 float 0.58 -> 0.51
//              12 modes, 1536 sets x 2 operands float 3.18 -> 3.06; 8 x 8 one-body, 2048 sets 0.62 -> 0.47
//   past it    8 modes, 4096 sets float 1.27 -> 1.52; 12 modes, 4096 float 5.57 -> 6.57, 2048 x 2 3.82 -> 4.06
//              16 x 16 one-body, 4096 sets 2.25 -> 2.43
// FP64 record passes have half the rate: there the longer graphs of G2 have no such
// line (12,000 sets: 10 modes 10.2 -> 7.3, 12 modes 21.0 -> 19.1 and x 5 81.5 -> 35.3).
constexpr int64_t kSmallSets = 2048, kSmallSetsWide = 1536, kSmallLongRecords = 10000;

static int64_t small_lds_bytes(const Graph& g, int gen, int64_t nops, bool records) {
    int64_t b = (g.N * (4 * nops + 1) + g.NG) * 8 + (g.N + g.NG + 3) / 2 * 8;
    if (records) b += (g.csr[0][0].nrec + (gen == CUT_GEN_G2 ? 0 : g.csr[1][0].nrec)) * 8;
    return b;
}

// Real record graphs whose flow state of one set fits in LDS, with no
// outside-space records (the diagnostic runs on the general path, and its flow
// has to be bitwise the flow without it).
bool small_flow_usable(const Graph& g, int gen, int prec, int64_t nsets, int64_t nops) {
    if (prec == CUT_F32 || (gen != CUT_GEN_WEGNER_GRAPH && gen != CUT_GEN_G2) || nops > 8) return false;
    if (g.have_outside || g.csr[0][0].cx || g.NG != g.N) return false;
    const int64_t nrec = g.csr[0][0].nrec;
    const bool any = prec == CUT_F64 && gen == CUT_GEN_G2 && nrec > kSmallLongRecords;
    if (!any && nsets > (nrec > kSmallRecords ? kSmallSetsWide : kSmallSets)) return false;
    return nrec <= (nsets > 32 ? kSmallRecordsWide : kSmallRecords) &&
           small_lds_bytes(g, gen, nops, false) <= g.max_lds;
}

template <int NOPS>
static void launch_small_n(const SmallFlow& a, bool in, dim3 grid, size_t lds, hipStream_t s) {
    if (in) hipLaunchKernelGGL((k_flow_small<NOPS, true>), grid, dim3(kSmallThreads), lds, s, a);
    else hipLaunchKernelGGL((k_flow_small<NOPS, false>), grid, dim3(kSmallThreads), lds, s, a);
}

void launch_flow_small(const Graph& g, int gen, int prec, double ds, double delta, int64_t nsets, int64_t nops,
                       const int32_t* nsteps, int64_t t0, int64_t t1, double* z, double* ckpt, int64_t ckpt_every,
                       hipStream_t s) {
    SmallFlow a{};
    a.off = g.csr[0][0].off;
    a.rec = g.csr[0][0].rec;
    a.goff = g.csr[1][0].off;
    a.grec = g.csr[1][0].rec;
    a.stencil = gen == CUT_GEN_G2 ? g.stencil : nullptr;
    a.pairs = g.pairs;
    a.ftab = g.ftab;
    a.gsign = g.gen_sign;
    a.d2 = delta * delta;
    a.ds = ds;
    a.N = (int32_t)g.N;
    a.NG = (int32_t)g.NG;
    a.nsets = (int32_t)nsets;
    a.f32 = prec != CUT_F64;
    a.nsteps = nsteps;
    a.z = z;
    a.ckpt = ckpt;
    a.ckpt_every = ckpt_every;
    a.nrec = (int32_t)g.csr[0][0].nrec;
    a.ngrec = gen == CUT_GEN_G2 ? 0 : (int32_t)g.csr[1][0].nrec;
    const bool in = small_lds_bytes(g, gen, nops, true) <= g.max_lds;
    const size_t lds = (size_t)small_lds_bytes(g, gen, nops, in);
    const dim3 grid((unsigned)nsets);
    // bounded launches: the state is in z between them
    constexpr int64_t kSteps = 1024;
    for (int64_t t = t0; t < t1; t += kSteps) {
        a.t0 = t;
        a.t1 = std::min(t1, t + kSteps);
        switch (nops) {
            case 1: launch_small_n<1>(a, in, grid, lds, s); break;
            case 2: launch_small_n<2>(a, in, grid, lds, s); break;
            case 3: launch_small_n<3>(a, in, grid, lds, s); break;
            case 4: launch_small_n<4>(a, in, grid, lds, s); break;
            case 5: launch_small_n<5>(a, in, grid, lds, s); break;
            case 6: launch_small_n<6>(a, in, grid, lds, s); break;
            case 7: launch_small_n<7>(a, in, grid, lds, s); break;
            default: launch_small_n<8>(a, in, grid, lds, s); break;
        }
    }
}

}  // namespace cut
