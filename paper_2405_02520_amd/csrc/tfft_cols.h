#pragma once
// Column kernels: the strided and last passes of multi-pass plans whose checksum
// groups have 64 members.
#include "tfft_kernels.h"

namespace tfft {

// A wavefront's lanes run along MB members of a checksum group (all 64 of them
// for sub-transforms of M <= 128 points), so that it works on PW = 64 / MB
// positions j = 0..T - 1 (T = M / 8) of each: LDS addresses are a lane constant
// plus an immediate, without swizzle, and the batch weight b + 1 is the lane's.
// With PW = 1 the stage twiddles, the checksum vector and the classes of e are
// the same for every lane and live in scalar registers, and d2 = sum of
// (lane + 1) d1(lane) needs no sums of its own; with more, the tables are read
// from LDS (a few addresses per wavefront).  A tile is MB members; a group is
// 64 / MB of them in turn.
//
// The last pass reads rows, so its first stage has the lanes along the
// positions; its exchange turns the tile, and the outputs leave with the lanes
// along the members, which is the transposed store.
//
// Bound by HBM (16 bytes per element and pass) and, with the checksum, close to
// it by instruction issue.  128 registers, so that 16 wavefronts per CU hide
// each other's exchanges with the next tile's loads in flight, where the pass
// kernels hold 190-240 and 8.  (The checksummed strided kernel of 256 points needs
// 8 more: 16 bytes a lane go to scratch and back once per group, outside the tile
// loop; with offset tables 2 registers do in every tile.)  Measured at 1 GiB, FT CORRECT, us of the first and
// the last pass, pass kernels then columns: N = 2^13 531 + 535 -> 432 + 464 (4.0
// -> 4.8 TB/s), 2^17 605 + 540 -> 541 + 490; N = 2^19 first pass (M = 512) 670 ->
// 545; N = 2^19 with the checksum off 629 -> 509 in all.
template <typename R, int M, int KIND, int FT>
struct ColCfg {
    static constexpr bool BLK = FT == FT_BLOCK;
    static constexpr int E = 8;
    static constexpr int T = M / E;
    static constexpr int WV = T < 16 ? T : 16;
    static constexpr int NT = WV * 64;
    static constexpr int PW = T / WV;
    static constexpr int MB = 64 / PW;
    static constexpr int ROUNDS = PW;
    static constexpr int C = cfg_wide_C(M);
    static constexpr int NSTAGE = n_stages(M, E);
    static constexpr bool UNIF = PW == 1;
    static constexpr bool W2SUM = !(KIND == KIND_STRIDED && UNIF);  // d2 has sums of its own
    static constexpr int NSUM = W2SUM ? 5 : 3;                      // partial sums per thread
    static constexpr size_t TILE = sizeof(cx<R>) * M * MB;
    static constexpr size_t RED = BLK ? sizeof(double) * NSUM * NT : 16;
    static constexpr bool LCV = BLK && !(KIND == KIND_STRIDED && UNIF);  // checksum vector in LDS
    static constexpr bool LTW = !UNIF;                                   // stage twiddles in LDS
    static constexpr size_t TAB = (LCV ? 16 * M : 16) + (LTW ? sizeof(cx<R>) * M : 16);
    // a second exchange buffer saves the barrier after each exchange's reads
    // (with two exchanges per tile, so that the sums are ordered as well)
    static constexpr int NBUF = NSTAGE == 3 && 2 * TILE + RED + TAB <= 158 * 1024 ? 2 : 1;
};

// v with its sign bit flipped by the mask 0 or 0x80000000.
__device__ __forceinline__ float flip_sign(float v, uint32_t mask) { return __uint_as_float(__float_as_uint(v) ^ mask); }
__device__ __forceinline__ double flip_sign(double v, uint32_t mask) {
    return __longlong_as_double(__double_as_longlong(v) ^ (long long)((unsigned long long)mask << 32));
}

// Scalar load of a uniform table entry.
template <typename T>
__device__ __forceinline__ cx<T> uload(const cx<T> *p, int i) {
    const auto *q = (const __attribute__((address_space(4))) nvec2<T> *)(p);
    const nvec2<T> v = q[i];
    return {v.x, v.y};
}

// HOOK: the fault hook is compiled in (launched when faults are installed).
// RAG: the signals lie where the offset tables say (ragged classes).
template <typename R, int M, int KIND, int FT, bool HOOK, bool RAG>
__global__ void __launch_bounds__(cfg_col_threads(M)) col_kernel(PassArgs args) {
    using Cf = ColCfg<R, M, KIND, FT>;
    constexpr bool BLK = Cf::BLK;
    constexpr int E = Cf::E, T = Cf::T, WV = Cf::WV, C = Cf::C, NSTAGE = Cf::NSTAGE, MB = Cf::MB, PW = Cf::PW;
    // the next tile's loads ahead; not where the fault hook leaves no registers for
    // them (the strided passes of 256 and 512 points would spill in every tile; as
    // they are, they and the hooked last passes spill 8 registers once per group)
    constexpr bool AHEAD = !(HOOK && KIND == KIND_STRIDED && M >= 256);
    using St = Stages<M, E>;
    __shared__ __align__(16) cx<R> lds[Cf::NBUF][M * MB];
    __shared__ double red[BLK ? Cf::NSUM : 1][BLK ? WV : 1][64];
    __shared__ __align__(16) cx<double> lcv[Cf::LCV ? M : 1];
    __shared__ __align__(16) cx<R> ltw[Cf::LTW ? M : 1];
    __shared__ double fin[BLK ? 2 : 1][5];
    __shared__ DevFault f0;
    int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // The arguments (args) in place: read from the scalar cache where they are
    // used, through a pointer made opaque per tile, instead of held over the
    // loop in more scalar registers than there are.
    const auto *k = (const __attribute__((address_space(4))) PassArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    int mem, j;   // member within the tile and position of this thread (j uniform if PW == 1)
    int mb0, j0;  // the same in the first stage of the last pass
    auto place = [&]() {
        mem = PW == 1 ? lane : lane % MB;
        j = PW == 1 ? wv : wv * PW + lane / MB;
        mb0 = KIND == KIND_LAST ? (wv * 64 + lane) / T : mem;
        j0 = KIND == KIND_LAST ? (wv * 64 + lane) % T : j;
    };
    place();
    if constexpr (Cf::LCV) {
        for (int t = threadIdx.x; t < M; t += Cf::NT) lcv[t] = ldg(reinterpret_cast<const cx<double> *>(k->cvec) + t);
    }
    if constexpr (Cf::LTW) {
        for (int t = threadIdx.x; t < M; t += Cf::NT) ltw[t] = ldg(reinterpret_cast<const cx<R> *>(k->stw) + t);
    }
    if constexpr (Cf::LCV || Cf::LTW) __syncthreads();

    // Addresses: a uniform base per tile and element plus a byte offset of the
    // lane (below 2^32: at most 64 / C units of 2^24 elements).  Members of a
    // partial last group that do not exist work on the last unit's data; they
    // are neither stored nor summed.
    auto unit = [&]() { return KIND == KIND_STRIDED ? k->L : k->n; };  // elements per outer unit
    // opaque, so that the lane's offset stays the 32-bit part of the address
    typedef __attribute__((address_space(1))) nvec2<R> G;
    auto at = [](const cx<R> *p, uint32_t vo) -> G * {
        if constexpr (!RAG) asm volatile("" : "+s"(p));
        return (G *)((__attribute__((address_space(1))) char *)p + vo);
    };
    auto load = [](const G *p) -> cx<R> {
        const nvec2<R> v = __builtin_nontemporal_load(p);
        return {v.x, v.y};
    };
    struct Loc {
        int64_t u0;  // the group's first outer unit
        int first;   // its first member's column or row
        int last;    // last outer unit of the group that exists
    };
    // (group and unit numbers are below 2^31, checked by the host: compared in
    // 32 bits, which the scalar unit can)
    auto locate = [&](int g) -> Loc {
        Loc l;
        const int u0 = (g >> k->ns_log2) * k->rb;
        l.u0 = u0;
        l.first = (g & ((int)k->n_strips - 1)) * C;
        const int left = (int)k->n_outer - 1 - u0;
        l.last = left < k->rb - 1 ? left : k->rb - 1;
        return l;
    };
    auto voff = [&](const Loc &l, int b, int64_t step) -> uint32_t {
        const int u = b / C < l.last ? b / C : l.last;
        const uint32_t first = RAG ? 0u : (uint32_t)u * (uint32_t)unit();
        return (uint32_t)sizeof(cx<R>) * (first + (uint32_t)(b % C) * (uint32_t)step);
    };
    // First element of the unit of member b (of round r) in a buffer: for back
    // to back signals the group's first unit (voff adds the rest), else the
    // unit's own, one of the at most two units of a tile, whose table entries
    // are scalar loads.
    auto ubase = [&](const Loc &l, int r, int b, bool input) -> int64_t {
        if constexpr (!RAG) {
            return l.u0 * unit();
        } else {
            const int64_t *sig = input ? k->in_sig : k->out_sig;
            auto one = [&](int i) -> int64_t {
                const int64_t u = l.u0 + (i < l.last ? i : l.last);
                if (!sig) return u * unit();
                const int64_t s = ((const __attribute__((address_space(4))) int64_t *)sig)[u >> k->o_log2];
                return s + (KIND == KIND_STRIDED ? (u & (k->O - 1)) * k->L : 0);
            };
            const int i0 = r * MB / C;
            const int64_t a0 = one(i0);
            if constexpr (MB <= C) return a0;
            const int64_t a1 = one(i0 + 1);
            return b / C > i0 ? a1 : a0;
        }
    };
    cx<R> nx[E];
    // (past the last group the same first elements are read over and over, so
    // that the number of loads in flight is the same on every path)
    auto load_tile = [&](int g, int r) {
        const bool past = g >= (int)k->n_groups;
        const Loc l = locate(past ? 0 : g);
        const cx<R> *in = reinterpret_cast<const cx<R> *>(k->in);
        if constexpr (KIND == KIND_STRIDED) {
            const uint32_t st = past ? 0u : (uint32_t)k->S;
            const int64_t ub = ubase(l, r, r * MB + mem, true);
            const cx<R> *s = in + (past ? 0 : ub + l.first) + (uint32_t)(wv * PW) * st;
            const uint32_t vo = voff(l, r * MB + mem, 1) +
                                (PW == 1 ? 0u : (uint32_t)sizeof(cx<R>) * (uint32_t)(lane / MB) * st);
#pragma unroll
            for (int m = 0; m < E; ++m) nx[m] = load(at(s + (uint32_t)(T * m) * st, vo));
        } else {
            const int64_t o = (int64_t)(l.first & (k->m1 - 1)) * k->m2 + (l.first >> k->m1_log2);
            const int64_t ub = ubase(l, r, r * MB + mb0, true);
            const cx<R> *s = in + (past ? 0 : ub + o * M);
            const uint32_t vo =
                voff(l, r * MB + mb0, (int64_t)k->m2 * M) + (uint32_t)sizeof(cx<R>) * (uint32_t)j0;
#pragma unroll
            for (int m = 0; m < E; ++m) nx[m] = load(at(s, vo) + T * m);
        }
    };
    // LDS slot of (position, member): the first exchange of the last pass is
    // written with lanes along positions 8 j0 + q, read with lanes along members
    auto slot = [](int pos, int mm, bool turned) -> int {
        const int l = pos * MB + mm;
        if (KIND == KIND_LAST && turned) return l ^ (((pos >> 3) * (64 / T > 1 ? 64 / T : 1)) & 31);
        return l;
    };
    // A group is settled while the next one is transformed, by wavefronts in
    // turn, so that no barrier waits for more than one step of it: a wavefront
    // per partial sum adds it up over the wavefronts and lanes, between the
    // first barrier after the sums were written and the next; one thread
    // decides at the end, where the fewest registers are in use.
    auto add_up = [&](int i) {
        i = __builtin_amdgcn_readfirstlane(i);
        asm volatile("" : "+s"(i));  // its LDS addresses are formed here
        const int q = (wv - i) & (WV - 1);
        if (q >= Cf::NSUM) return;
        double x = 0.0;
#pragma unroll 4
        for (int w = 0; w < WV; ++w) x += red[q][w][lane];
        if constexpr (!Cf::W2SUM) {
            // q: d1 (re), d1 (im), S; d2 is d1 weighted by the member's number
            if (q < 2) {
                const double y = wave_sum_dpp(double(lane + 1) * x, Dpp64{});
                if (lane == 63) fin[i & 1][2 + q] = y;
            }
            x = wave_sum_dpp(x, Dpp64{});
            if (lane == 63) fin[i & 1][q < 2 ? q : 4] = x;
        } else {
            x = wave_sum_dpp(x, Dpp64{});
            if (lane == 63) fin[i & 1][q] = x;
        }
    };
    auto settle = [&](int i, int g) {
        i = __builtin_amdgcn_readfirstlane(i);
        asm volatile("" : "+s"(i));  // its LDS addresses are formed here
        if (wv != ((i + 8) & (WV - 1)) || lane != 0) return;
        // the threshold test in squares (sums of binary32 data: no overflow, and
        // the host bounds the factor); the record's member is located by whoever
        // reads it
        const double *s = fin[i & 1];
        if (!(s[0] * s[0] + s[1] * s[1] <= k->tau_sq * s[4])) {
            const double tc = k->tau_coef;
            const unsigned long long n = atomicAdd(&k->rep->n_flag, 1ULL);
            if ((int64_t)n < k->rec_cap) {
                DevRecord *rc = k->recs + n;
                rc->group = k->g_base + g;
                rc->pass = k->pass;
                rc->task = k->task;
                rc->action = 1;  // detected
                rc->member = kUnlocated;
                rc->method = 0;
                rc->d1r = s[0];
                rc->d1i = s[1];
                rc->d2r = s[2];
                rc->d2i = s[3];
                rc->tau = tc * sqrt(s[4]);
                rc->s = s[4];
            }
        }
    };

    const int nwg = gridDim.x;
    int g = blockIdx.x;
    if (nwg % 8 == 0) g = (int)(blockIdx.x % 8) * (nwg / 8) + (int)(blockIdx.x / 8);
    int it = 0;
    if constexpr (AHEAD) load_tile(g, 0);
    const int n_groups = (int)k->n_groups;
    for (; g < n_groups; g += nwg) {
        asm volatile("" : "+s"(k));
        const int32_t *fhp = k->fault_head ? k->fault_head + k->g_base + g : &kNoFault;
        const int fh = HOOK ? *fhp : -1;
        bool fmulti = true;
        if (fh >= 0) {
            __syncthreads();
            if (threadIdx.x == 0) f0 = k->faults[fh];
            __syncthreads();
            fmulti = f0.next >= 0;
        }
        const Loc L = locate(g);
        double D1r = 0.0, D1i = 0.0, D2r = 0.0, D2i = 0.0, S = 0.0;
        for (int r = 0; r < Cf::ROUNDS; ++r) {
            // opaque per tile, like the arguments: tables in LDS are read again
            // and offsets formed again instead of held in registers
            asm volatile("" : "+s"(k));
            asm volatile("" : "+v"(lane));
            place();
            const auto *stw = reinterpret_cast<const cx<R> *>(k->stw);
            const auto *cv = reinterpret_cast<const cx<double> *>(k->cvec);
            const int b = r * MB + mem;  // member of the stages from the second on (strided: of all)
            const bool ok = b / C <= L.last;
            const int bl = r * MB + mb0;  // member whose inputs the thread holds
            const bool okl = KIND == KIND_STRIDED ? ok : bl / C <= L.last;
            cx<double> twA{1.0, 0.0}, twB{1.0, 0.0};
            if constexpr (KIND == KIND_STRIDED) {
                // w_N^{k i N/L}, exponents below 2^31 before the reduction mod N
                const uint32_t i = ((uint32_t)L.first + b % C) * (uint32_t)k->tw_scale, mask = (uint32_t)k->n - 1;
                twA = itw(*k, ((uint32_t)j * i) & mask);
                twB = itw(*k, ((uint32_t)T * i) & mask);
            }
            if constexpr (!AHEAD) load_tile(g, r);
            cx<R> d[E];
#pragma unroll
            for (int m = 0; m < E; ++m) {
                d[m] = nx[m];
                // in registers before the next tile's loads are issued
                asm volatile("" : "+v"(d[m].re), "+v"(d[m].im));
            }
            asm volatile("" ::: "memory");
            if constexpr (AHEAD) load_tile(r + 1 < Cf::ROUNDS ? g : g + nwg, r + 1 < Cf::ROUNDS ? r + 1 : 0);

            if constexpr (BLK) {
                double lr = 0.0, li = 0.0, sv = 0.0;
                int jc = j0;
#pragma unroll
                for (int m = 0; m < E; ++m) {
                    const double xr = double(d[m].re), xi = double(d[m].im);
                    cx<double> cm;
                    // a quarter of the table entries in registers at a time:
                    // the next reads wait for the sums so far
                    if (Cf::LCV && m % 2 == 0) asm volatile("" : "+v"(jc), "+v"(lr), "+v"(li));
                    if constexpr (Cf::LCV) cm = lcv[jc + T * m];
                    else cm = uload(cv, j + T * m);
                    lr = __builtin_fma(cm.re, xr, lr);
                    lr = __builtin_fma(-cm.im, xi, lr);
                    li = __builtin_fma(cm.re, xi, li);
                    li = __builtin_fma(cm.im, xr, li);
                    sv = __builtin_fma(xr, xr, sv);
                    sv = __builtin_fma(xi, xi, sv);
                }
                lr = okl ? lr : 0.0;
                li = okl ? li : 0.0;
                S += okl ? sv : 0.0;
                D1r -= lr;
                D1i -= li;
                if constexpr (Cf::W2SUM) {
                    const double w2 = double(bl + 1);
                    D2r -= w2 * lr;
                    D2i -= w2 * li;
                }
            }
            const uint32_t flip_in = k->conj_in ? 0x80000000u : 0u;
#pragma unroll
            for (int m = 0; m < E; ++m) d[m].im = flip_sign(d[m].im, flip_in);

            static_for<0, NSTAGE>([&](auto Sx) {
                constexpr int s = Sx;
                constexpr int RAD = St::radix(s), NS = St::ns(s), NB = St::nb(s);
                constexpr bool rows = KIND == KIND_LAST && s == 0;  // lanes along positions
                cx<R> *buf = lds[(s & 1) % Cf::NBUF];
                if constexpr (s > 0) {
                    cx<R> *pbuf = lds[((s - 1) & 1) % Cf::NBUF];
#pragma unroll
                    for (int m = 0; m < E; ++m) d[m] = pbuf[slot(j + T * m, mem, s == 1)];
                    if constexpr (Cf::NBUF == 1) __syncthreads();
                    if constexpr (s == 1 && BLK && Cf::NBUF == 2) {
                        if (r == 0 && it > 0) add_up(it - 1);
                    }
                    static_for<0, NB>([&](auto p) {
                        static_for<1, RAD>([&](auto q) {
                            const int t = (((j + p * T) % NS) * q) * (M / (NS * RAD));
                            const cx<R> w = Cf::LTW ? ltw[t] : uload(stw, t);
                            d[p + q * NB] = cmul(d[p + q * NB], w);
                        });
                    });
                }
                static_for<0, NB>([&](auto p) {
                    cx<R> x[RAD];
                    static_for<0, RAD>([&](auto q) { x[q] = d[p + q * NB]; });
                    dft_small<R, RAD>(x);
                    static_for<0, RAD>([&](auto q) { d[p + q * NB] = x[q]; });
                });
                if (fh >= 0) apply_faults_g<R, E>(d, f0, fmulti, k->faults, fh, s, rows ? bl : b, rows ? j0 : j);
                if constexpr (s < NSTAGE - 1) {
                    static_for<0, NB>([&](auto p) {
                        const int i = (rows ? j0 : j) + p * T;
                        const int base = (i / NS) * NS * RAD + (i % NS);
                        static_for<0, RAD>(
                            [&](auto q) { buf[slot(base + q * NS, rows ? mb0 : mem, s == 0)] = d[p + q * NB]; });
                    });
                    __syncthreads();
                }
                if constexpr (s == 0 && BLK && Cf::NBUF == 1) {
                    if (r == 0 && it > 0) add_up(it - 1);
                }
            });

            // final values: register m holds output k = j + T m
            FaultHit hf{-1, 0.0, 0.0, 0ull, 0ull};
            if (fh >= 0) hf = fault_hit_g(f0, fmulti, k->faults, fh, -1, b, j);
            const uint32_t flip_out = k->conj_out ? 0x80000000u : 0u;
            const R sc = R(k->out_scale);
            double Ar[3] = {0.0, 0.0, 0.0}, Ai[3] = {0.0, 0.0, 0.0};  // sums of e-class 0, 1, 2
            cx<double> P = twA;
#pragma unroll
            for (int m = 0; m < E; ++m) {
                cx<R> y = d[m];
                if constexpr (KIND == KIND_STRIDED) {
                    y = cmul(y, cx<R>{R(P.re), R(P.im)});
                } else {
                    y.re *= sc;  // exact where the scale is 1
                    y.im *= sc;
                }
                y.im = flip_sign(y.im, flip_out);
                if (fh >= 0) y = hit_one(y, hf, m);
                d[m] = y;
                if constexpr (BLK) {
                    const int cls = ((T % 3) * m) % 3;
                    const double yr = double(y.re), yi = double(y.im);
                    if constexpr (KIND == KIND_STRIDED) {
                        // e' = e conj(applied twiddle): the twiddle product is
                        // inside the check
                        const double pr = P.re, pi = flip_sign(P.im, flip_out);
                        Ar[cls] = __builtin_fma(yr, pr, Ar[cls]);
                        Ar[cls] = __builtin_fma(yi, pi, Ar[cls]);
                        Ai[cls] = __builtin_fma(yi, pr, Ai[cls]);
                        Ai[cls] = __builtin_fma(-yr, pi, Ai[cls]);
                    } else {
                        Ar[cls] += yr;
                        Ai[cls] += yi;
                    }
                }
                if constexpr (KIND == KIND_STRIDED) {
                    if (m + 1 < E) P = cmul(P, twB);
                }
            }
            if (ok) {
                const uint32_t ostr = KIND == KIND_STRIDED ? (uint32_t)k->S : (uint32_t)k->rows;
                const cx<R> *dst = reinterpret_cast<const cx<R> *>(k->out) + ubase(L, r, b, false) + L.first +
                                   (uint32_t)(wv * PW) * ostr;
                const uint32_t vo =
                    voff(L, b, 1) + (PW == 1 ? 0u : (uint32_t)sizeof(cx<R>) * (uint32_t)(lane / MB) * ostr);
#pragma unroll
                for (int m = 0; m < E; ++m)
                    __builtin_nontemporal_store(nvec2<R>{d[m].re, d[m].im}, at(dst + (uint32_t)(T * m) * ostr, vo));
            }
            if constexpr (BLK) {
                const double sr = Ar[0] + kW3r * (Ar[1] + Ar[2]) - kW3i * (Ai[1] - Ai[2]);
                const double si = Ai[0] + kW3r * (Ai[1] + Ai[2]) + kW3i * (Ar[1] - Ar[2]);
                const int jr = j % 3;  // e_k = w_3^(k mod 3), k = j + T m
                const double rotr = jr == 0 ? 1.0 : kW3r;
                const double roti = jr == 0 ? 0.0 : (jr == 1 ? kW3i : -kW3i);
                double rr = sr * rotr - si * roti, ri = sr * roti + si * rotr;
                rr = ok ? rr : 0.0;
                ri = ok ? ri : 0.0;
                D1r += rr;
                D1i += ri;
                if constexpr (Cf::W2SUM) {
                    const double w2 = double(b + 1);
                    D2r += w2 * rr;
                    D2i += w2 * ri;
                }
            }
        }
        if constexpr (BLK) {
            if (it > 0) settle(it - 1, g - nwg);
            red[0][wv][lane] = D1r;
            red[1][wv][lane] = D1i;
            if constexpr (Cf::W2SUM) {
                red[2][wv][lane] = D2r;
                red[3][wv][lane] = D2i;
                red[4][wv][lane] = S;
            } else {
                red[2][wv][lane] = S;
            }
        }
        ++it;
    }
    if constexpr (BLK) {
        // the last group; g is past it
        __syncthreads();
        if (it > 0) add_up(it - 1);
        __syncthreads();
        if (it > 0) settle(it - 1, g - nwg);
    }
}

template <typename R, int M, int KIND, int FT, bool RAG>
static hipError_t launch_cols_hook(const PassArgs &a, int grid, hipStream_t st) {
    const dim3 n(cfg_col_threads(M));
    if (a.fault_head) hipLaunchKernelGGL((col_kernel<R, M, KIND, FT, true, RAG>), dim3(grid), n, 0, st, a);
    else hipLaunchKernelGGL((col_kernel<R, M, KIND, FT, false, RAG>), dim3(grid), n, 0, st, a);
    return hipGetLastError();
}
template <typename R, int M, int KIND, int FT>
static hipError_t launch_cols_one(const PassArgs &a, int grid, hipStream_t st) {
    return a.in_sig || a.out_sig ? launch_cols_hook<R, M, KIND, FT, true>(a, grid, st)
                                 : launch_cols_hook<R, M, KIND, FT, false>(a, grid, st);
}

template <typename R, int M>
hipError_t cols_m(int kind, int ft, const PassArgs &a, int grid, hipStream_t st) {
    static_assert(cfg_cols(sizeof(R) == 8, M, KIND_STRIDED) && cfg_cols(sizeof(R) == 8, M, KIND_LAST), "column kernel shape");
    if (kind == KIND_STRIDED)
        return ft ? launch_cols_one<R, M, KIND_STRIDED, FT_BLOCK>(a, grid, st)
                  : launch_cols_one<R, M, KIND_STRIDED, FT_NONE>(a, grid, st);
    if (kind == KIND_LAST)
        return ft ? launch_cols_one<R, M, KIND_LAST, FT_BLOCK>(a, grid, st)
                  : launch_cols_one<R, M, KIND_LAST, FT_NONE>(a, grid, st);
    return hipErrorInvalidValue;
}

#define TFFT_INSTANTIATE_COLS(R, M) template hipError_t cols_m<R, M>(int, int, const PassArgs &, int, hipStream_t);
#define TFFT_EXTERN_COLS(R, M) extern template hipError_t cols_m<R, M>(int, int, const PassArgs &, int, hipStream_t);

}  // namespace tfft
