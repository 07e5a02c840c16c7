// Chains of contractions with their intermediates in LDS, and the launch
// that runs them beside a level's small nodes.  Included by HIP translation
// units only.
//
// What bounds it: a node-by-node launch list moves every intermediate
// through memory twice.  A chain reads F_0 and the G_i once and writes F_L
// once; its tiles pass from stage to stage through LDS.  A tile is a
// contiguous piece of F_1's storage order (every operand stores its summed
// variables lowest), so F_0 is read in whole rows.
//
// Numerics: a stage forms every sum in double, in the order of the summed
// index, and rounds once to the storage type, as the other node kernels do;
// only the power of two a tensor is stored with differs.  The launch list
// brings every operand's largest entry to [0.5, 1) as it reads it; the tiles
// of an intermediate exist one after another, so here stage i reads F_{i-1}
// as it was stored.  Instead the whole chain, F_L included, is stored
// 2^lift larger (chain word CS_LIFT; the published exponent takes it back).
//
// Range: let S_i be F_i as stored here and R_i as the launch list stores it,
// S_i = 2^c_i R_i.  The list reads R_i scaled by the power of two that S_i is
// 2^e_i away from, e_i the exponent of S_i's largest entry, so c_1 = lift
// and c_{i+1} = e_i.  As long as every intermediate has an entry of at least
// chain_tiny = 2^-1 (e_i >= 0), no c_i is negative: nothing the launch list
// can represent is lost here, neither in an intermediate nor in F_L.  Each
// stage but the last reports whether its unrounded sums reached chain_tiny
// and whether one was nonzero; a chain with an intermediate that was nonzero
// but below chain_tiny everywhere is run again on the general launch list.
#pragma once
#include "wmc_kernels.h"

// Descriptors are read through the constant address space, so that
// wave-uniform reads are scalar loads.
typedef const __attribute__((address_space(4))) unsigned *chain_words;
__device__ __forceinline__ chain_words const_words(const unsigned *p) {
    return (chain_words)(unsigned long long)p;
}

// Smallest largest entry of an intermediate (see Range above).
constexpr double chain_tiny = 0.5;

// LDS entry e sits at slot chain_slot(e): 16-byte units XOR-ed with the
// three address bits above a 128-byte bank row, so that lanes reading rows
// of 2 to 16 units at a power-of-two stride spread over all banks.  Linear
// over XOR, and a permutation within aligned runs of 256 entries.
template <typename T>
__device__ __forceinline__ unsigned chain_slot(unsigned e) {
    return e ^ ((e >> 3) & (sizeof(T) == 8 ? 0xEu : 0x1Cu));
}

// N consecutive entries of an LDS row whose first slot is `slot` (rows are
// aligned to N entries).
template <typename T, int N>
__device__ __forceinline__ void chain_row(const T *lds, unsigned slot, double *v) {
    if constexpr (sizeof(T) == 8 && N >= 2) {
#pragma unroll
        for (int h = 0; h < N / 2; ++h) {
            const double2 x = *(const double2 *)(lds + (slot ^ (unsigned)(2 * h)));
            v[2 * h] = x.x;
            v[2 * h + 1] = x.y;
        }
    } else if constexpr (sizeof(T) == 4 && N >= 4) {
#pragma unroll
        for (int h = 0; h < N / 4; ++h) {
            const float4 x = *(const float4 *)(lds + (slot ^ (unsigned)(4 * h)));
            v[4 * h] = x.x;
            v[4 * h + 1] = x.y;
            v[4 * h + 2] = x.z;
            v[4 * h + 3] = x.w;
        }
    } else if constexpr (N == 2) {
        const float2 x = *(const float2 *)(lds + slot);
        v[0] = x.x;
        v[1] = x.y;
    } else {
        v[0] = (double)lds[slot];
    }
}

// Copies the part of an operand that a tile reads into LDS, where entry q
// goes to slot q: memory to LDS directly, without a register in between, so
// that all copies of a tile are in flight together (the caller waits for
// them).  ch: the chain's words; x: the operand's; src: its first entry for
// the tile; the calling waves take runs wave, wave + WAVES, ... of 64 pieces.
template <typename T, int WAVES>
__device__ __forceinline__ void chain_copy(const unsigned *ch, const unsigned *x, const T *src, T *lds, unsigned wave) {
    typedef const __attribute__((address_space(1))) unsigned *gp;
    typedef __attribute__((address_space(3))) unsigned *lp;
    constexpr unsigned EW = sizeof(T) / 4, VE = 16 / sizeof(T);  // words per entry, entries per 16 bytes
    const uint4 xv = *(const uint4 *)x;
    const unsigned nb = __builtin_amdgcn_readfirstlane(xv.x), low = __builtin_amdgcn_readfirstlane(xv.y);
    T *dst = lds + __builtin_amdgcn_readfirstlane(xv.z);
    const unsigned *list = ch + __builtin_amdgcn_readfirstlane(xv.w);
    const unsigned lane = threadIdx.x & 63u;
    auto offset = [&](unsigned q) {
        unsigned o = q & ((1u << low) - 1u);
        for (unsigned b = low; b < nb; ++b) o |= (0u - ((q >> b) & 1u)) & list[b - low];
        return o;
    };
    if ((1u << low) >= VE) {  // runs of 16 bytes
        for (unsigned u0 = wave * 64u; (u0 * VE) >> nb == 0u; u0 += WAVES * 64u) {
            const unsigned p = (u0 + lane) * VE;
            if (p >> nb) continue;
            __builtin_amdgcn_global_load_lds((gp)(const unsigned *)(src + offset(chain_slot<T>(p))),
                                             (lp)(unsigned *)(dst + u0 * VE), 16, 0, 0);
        }
    } else {
        for (unsigned u0 = wave * 64u; (u0 / EW) >> nb == 0u; u0 += WAVES * 64u) {
            const unsigned p = (u0 + lane) / EW;
            if (p >> nb) continue;
            __builtin_amdgcn_global_load_lds((gp)((const unsigned *)(src + offset(chain_slot<T>(p))) + lane % EW),
                                             (lp)((unsigned *)dst + u0), 4, 0, 0);
        }
    }
}

// Short chains, one stage: one output per thread and entry index.  lds is
// the tiles' and copies' memory, w the stage's words (in LDS, 16-byte
// aligned).  Without register bits the entry index of an LDS output is the
// thread and entry index itself.
template <typename T, int LB, int NK, bool SG, bool DG>
__device__ __forceinline__ void chain_stage_short(const unsigned *ch, const unsigned *w, unsigned tb,
                                                  const T *__restrict__ S,
                                                  T *__restrict__ C, T *lds, const unsigned *mask, int se,
                                                  double &vmax) {
    constexpr int K = 1 << NK;
    const uint4 head = *(const uint4 *)(w + 4);  // CS_TG, CS_SRC, CS_DST
    const unsigned sbase = __builtin_amdgcn_readfirstlane(head.y), dbase = __builtin_amdgcn_readfirstlane(head.z);
    const unsigned gbase = __builtin_amdgcn_readfirstlane(w[CS_X + CX_LDS]);
    auto map = [&](const unsigned *x) {
        unsigned v[12];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const uint4 t = *(const uint4 *)(x + 4 * q);
            v[4 * q] = t.x;
            v[4 * q + 1] = t.y;
            v[4 * q + 2] = t.z;
            v[4 * q + 3] = t.w;
        }
        unsigned r = 0;
#pragma unroll
        for (int b = 0; b < LB; ++b) r |= mask[b] & v[b];
        return r;
    };
    // source and G together: their indices fit half words, and slots, starts
    // and bit steps act on both halves at once
    unsigned sg = map(w + CS_BIT_SG), src = 0, out = threadIdx.x;
    if constexpr (SG) src = map(ch + CH_SRC);
    if constexpr (DG) out = map(ch + CH_OUT);
    const unsigned bases = sbase | (gbase << 16);
    constexpr unsigned swz = sizeof(T) == 8 ? 0x000E000Eu : 0x001C001Cu;
    if (tb < LB && threadIdx.x >> tb) return;
    const unsigned nh = tb > LB ? 1u << (tb - LB) : 1u;
#pragma clang loop unroll(disable)
    for (unsigned h = 0;;) {
        double sv[K], gv[K];
        const unsigned slots = sg ^ ((sg >> 3) & swz) ^ bases;
        chain_row<T, K>(lds, slots >> 16, gv);
        if constexpr (SG) {
            constexpr int KC = K < 4 ? K : 4;
#pragma unroll
            for (int kc = 0; kc < K; kc += KC) load_chunk<T, KC>(S + src + kc, sv + kc);
        } else {
            chain_row<T, K>(lds, slots & 0xFFFFu, sv);
        }
        double acc = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) acc = fma(sv[k], gv[k], acc);
        const double a = ldexp(acc, se);
        const T v = (T)a;
        if constexpr (DG) {
            C[out] = v;
            vmax = fmax(vmax, fabs((double)v));
        } else {
            lds[chain_slot<T>(out) ^ dbase] = v;
            vmax = fmax(vmax, fabs(a));
        }
        if (++h == nh) break;
        // entry index in Gray order: one bit changes
        const unsigned b = LB + __builtin_ctz(h);
        sg ^= w[CS_BIT_SG + b];
        if constexpr (SG) src ^= ch[CH_SRC + b];
        if constexpr (DG) out ^= ch[CH_OUT + b];
        else out ^= 1u << b;
    }
}

template <typename T, int LB, bool SG, bool DG>
__device__ __forceinline__ void chain_stage_short_any(const unsigned *ch, const unsigned *w, unsigned wave, const T *S,
                                                      T *C, T *lds, const unsigned *mask, int se, double &vmax) {
    const uint2 head = *(const uint2 *)w;  // CS_SHAPE, CS_TBITS
    const unsigned nk = __builtin_amdgcn_readfirstlane(head.x), tb = __builtin_amdgcn_readfirstlane(head.y);
    // waves past a small tile's last entry have nothing to do
    if (tb < LB && (wave << 6) >> tb) return;
    switch (nk) {
    case 0: chain_stage_short<T, LB, 0, SG, DG>(ch, w, tb, S, C, lds, mask, se, vmax); break;
    case 1: chain_stage_short<T, LB, 1, SG, DG>(ch, w, tb, S, C, lds, mask, se, vmax); break;
    case 2: chain_stage_short<T, LB, 2, SG, DG>(ch, w, tb, S, C, lds, mask, se, vmax); break;
    default: chain_stage_short<T, LB, 3, SG, DG>(ch, w, tb, S, C, lds, mask, se, vmax); break;
    }
}

// A stage's maps for one thread of a chain of many tiles: the offsets of its
// index bits, a lane part and a part uniform in the wave.
struct ChainMaps {
    unsigned src, g, out;  // lane
    unsigned us, ug, uo;   // wave
};

__device__ __forceinline__ ChainMaps chain_maps(chain_words st, const unsigned *mask, unsigned wave) {
    ChainMaps m{0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int b = 0; b < 6; ++b) {
        m.src |= mask[b] & st[CS_BIT_S + b];
        m.g |= mask[b] & st[CS_BIT_G + b];
        m.out |= mask[b] & st[CS_BIT_O + b];
    }
#pragma unroll
    for (int b = 6; b < WMC_CHAIN_LANE_BIG; ++b) {
        const unsigned on = 0u - ((wave >> (b - 6)) & 1u);
        m.us |= on & st[CS_BIT_S + b];
        m.ug |= on & st[CS_BIT_G + b];
        m.uo |= on & st[CS_BIT_O + b];
    }
    return m;
}

// Chains of many tiles: the thread's 2^(NP + NQ) outputs of every entry
// index.  Bound by instruction issue (about 100 vector and 100 scalar
// instructions per wave and stage beside the products) and the L2 latency of
// G: 4 waves per workgroup and 2 x 2 outputs per thread took the min-fill
// lattice from 57 (8 waves) to 42 ms; copying each tile's part of G to LDS
// leaves room for smaller tiles only (59 ms), and fetching the next stage's G
// ahead costs registers (50 ms).  SG: the source rows are in memory (stage 1), else in LDS; DG: the
// outputs go to memory (last stage), else to LDS.
template <typename T, int NK, int NP, int NQ, bool SG, bool DG>
__device__ __forceinline__ void chain_stage(chain_words st, const T *__restrict__ S, const T *__restrict__ G,
                                            T *__restrict__ C, T *lds, const unsigned *mask, unsigned wave, int se,
                                            bool nt, double &vmax) {
    constexpr int K = 1 << NK, KC = K < 4 ? K : 4;
    constexpr int P = 1 << NP, Q = 1 << NQ, LB = WMC_CHAIN_LANE_BIG;
    const unsigned tb = st[CS_TBITS];
    // waves past a small tile's last entry have nothing to do
    if (tb < LB && (wave << 6) >= (1u << tb)) return;
    const unsigned sbase = st[CS_SRC], dbase = st[CS_DST];
    ChainMaps m = chain_maps(st, mask, wave);
    unsigned ps[P], po[P], qg[Q], qo[Q];
#pragma unroll
    for (int i = 0; i < P; ++i) {
        ps[i] = po[i] = 0;
#pragma unroll
        for (int t = 0; t < NP; ++t)
            if ((i >> t) & 1) {
                ps[i] |= st[CS_PS + t];
                po[i] |= st[CS_PO + t];
            }
        if constexpr (!SG) ps[i] = chain_slot<T>(ps[i]);
        if constexpr (!DG) po[i] = chain_slot<T>(po[i]);
    }
#pragma unroll
    for (int j = 0; j < Q; ++j) {
        qg[j] = qo[j] = 0;
#pragma unroll
        for (int t = 0; t < NQ; ++t)
            if ((j >> t) & 1) {
                qg[j] |= st[CS_QG + t];
                qo[j] |= st[CS_QO + t];
            }
        if constexpr (!DG) qo[j] = chain_slot<T>(qo[j]);
    }
    const bool live = tb >= LB || threadIdx.x < (1u << tb);
    const unsigned nh = tb > LB ? 1u << (tb - LB) : 1u;
    for (unsigned h = 0; h < nh; ++h) {
        if (h) {  // entry index in Gray order: one bit changes, so one XOR per map
            chain_words x = st + LB + __builtin_ctz(h);
            m.us ^= x[CS_BIT_S];
            m.ug ^= x[CS_BIT_G];
            m.uo ^= x[CS_BIT_O];
        }
        if (!live) continue;
        const unsigned s0 = SG ? (m.src ^ m.us) : (chain_slot<T>(m.src ^ m.us) ^ sbase);
        const unsigned g0 = m.g ^ m.ug;
        const unsigned o0 = DG ? (m.out ^ m.uo) : (chain_slot<T>(m.out ^ m.uo) ^ dbase);
        double acc[P][Q];
#pragma unroll
        for (int i = 0; i < P; ++i)
#pragma unroll
            for (int j = 0; j < Q; ++j) acc[i][j] = 0.0;
#pragma unroll
        for (int kc = 0; kc < K; kc += KC) {
            double sv[P][KC], gv[Q][KC];
#pragma unroll
            for (int i = 0; i < P; ++i) {
                if constexpr (SG) load_chunk<T, KC>(S + (s0 ^ ps[i]) + kc, sv[i]);
                else chain_row<T, KC>(lds, s0 ^ ps[i] ^ (unsigned)kc, sv[i]);
            }
#pragma unroll
            for (int j = 0; j < Q; ++j) load_chunk<T, KC>(G + (g0 ^ qg[j]) + kc, gv[j]);
#pragma unroll
            for (int i = 0; i < P; ++i)
#pragma unroll
                for (int j = 0; j < Q; ++j)
#pragma unroll
                    for (int k = 0; k < KC; ++k) acc[i][j] = fma(sv[i][k], gv[j][k], acc[i][j]);
        }
#pragma unroll
        for (int i = 0; i < P; ++i)
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                const double a = ldexp(acc[i][j], se);
                const T v = (T)a;
                if constexpr (DG) {
                    if (nt) store_nt(C + (o0 ^ po[i] ^ qo[j]), v);
                    else C[o0 ^ po[i] ^ qo[j]] = v;
                    vmax = fmax(vmax, fabs((double)v));
                } else {
                    lds[o0 ^ po[i] ^ qo[j]] = v;
                    vmax = fmax(vmax, fabs(a));
                }
            }
    }
}

template <typename T, bool SG, bool DG>
__device__ __forceinline__ void chain_stage_any(chain_words st, const T *S, const T *G, T *C, T *lds,
                                                const unsigned *mask, unsigned wave, int se, bool nt, double &vmax) {
#define WMC_CHAIN_CASE(NKV, NPV, NQV)                                                            \
    case (NKV) | ((NPV) << 8) | ((NQV) << 16):                                                   \
        chain_stage<T, NKV, NPV, NQV, SG, DG>(st, S, G, C, lds, mask, wave, se, nt, vmax);       \
        break;
#define WMC_CHAIN_NK_CASES(NKV)                                                                        \
    WMC_CHAIN_CASE(NKV, 0, 0) WMC_CHAIN_CASE(NKV, 1, 0) WMC_CHAIN_CASE(NKV, 0, 1)                       \
    WMC_CHAIN_CASE(NKV, 1, 1) WMC_CHAIN_CASE(NKV, 2, 0) WMC_CHAIN_CASE(NKV, 0, 2)
    switch (st[CS_SHAPE]) {
        WMC_CHAIN_NK_CASES(0) WMC_CHAIN_NK_CASES(1) WMC_CHAIN_NK_CASES(2) WMC_CHAIN_NK_CASES(3)
    default: break;
    }
#undef WMC_CHAIN_NK_CASES
#undef WMC_CHAIN_CASE
}

// Block barrier that orders LDS only: the waves exchange nothing else, and
// loads of G for the next stage stay in flight across it.
__device__ __forceinline__ void chain_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Kept across the lanes of every wave: in lane 0 F_0's offset in the tile, in
// lane 1 C's, in lane 2 + i G_i's; in lane i the scale data of stage i's G
// (lane L: of F_0).
struct ChainLanes {
    unsigned off;
    unsigned long long maxbits;
    long long exp;
};

// The loads of the scale data are not waited for here.
template <int STRIDE, typename WP>
__device__ __forceinline__ ChainLanes chain_lanes(WP ch, unsigned L, unsigned ob, unsigned tile, const wmc_meta *meta) {
    const unsigned lane = threadIdx.x & 63u;
    ChainLanes c{0, 0, 0};
    if (lane <= L) {
        const wmc_meta *m = meta + ch[lane < L ? CH_WORDS + lane * STRIDE + CS_TG : CH_TF];
        c.maxbits = m->maxbits;
        c.exp = m->exp;
    }
    if (lane < L + 2) {
        const unsigned tab = CH_WORDS + L * STRIDE + lane * ob;
        for (unsigned b = 0; b < ob; ++b) c.off ^= (0u - ((tile >> b) & 1u)) & ch[tab + b];
    }
    return c;
}

// In lane i, the power of two stage i's products are scaled by; the first
// workgroup also publishes the chain's exponent.  lift: CS_LIFT.
__device__ __forceinline__ int chain_shifts(const ChainLanes &c, unsigned L, wmc_meta *meta, unsigned tc, bool first,
                                            int lift) {
    const unsigned lane = threadIdx.x & 63u;
    const int own = lane <= L ? scale_exp(c.maxbits) : 0;
    if (first && threadIdx.x < 64) {
        long long e = lane <= L ? c.exp + own : 0;
        for (int o = 8; o > 0; o >>= 1) e += __shfl_xor(e, o, WMC_WAVE);
        if (lane == 0) meta[tc].exp = e - lift;
    }
    const int f = __builtin_amdgcn_readlane(own, L);
    return lane == 0 ? lift - own - f : -own;
}

// Range bits of stage s's intermediate, whose largest unrounded magnitude in
// this thread is v: an ordinary entry, a nonzero entry.
__device__ __forceinline__ unsigned chain_range(double v, unsigned s) {
    return ((v >= chain_tiny ? 1u : 0u) | (v > 0.0 ? 2u : 0u)) << (2 * s);
}

__device__ __forceinline__ void chain_end(wmc_meta *meta, unsigned tmask, unsigned tc, unsigned range, double vmax) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) range |= __shfl_xor(range, o, WMC_WAVE);
    if ((threadIdx.x & 63u) == 0u) {
        unsigned long long *mask = &meta[tmask].maxbits;
        if (range & ~(unsigned)__atomic_load_n(mask, __ATOMIC_RELAXED)) atomicOr(mask, (unsigned long long)range);
    }
    publish_max_block(meta, (int)tc, vmax);
}

__device__ __forceinline__ long long chain_base(unsigned lo, unsigned hi) {
    return (long long)(((unsigned long long)hi << 32) | lo);
}

// One tile of a short chain.  What bounds it is waiting: read where they are
// first needed, a stage's words, its G and its sources are a cold miss each
// (2 to 3 us a stage); fetched together before the first stage, a stage takes
// 0.4 to 0.7 us and the start 3 us.  A workgroup of 2^LB threads: 2^9 where a call
// waits for it, 2^8 where many chains share the device and each wave's fixed
// instructions count (512-instance batch FP64 4.18 -> 3.72 ms).  smem: the chain's words, then (from the next
// 1024-byte boundary) its LDS entries.
template <typename T, int LB>
__device__ __forceinline__ void chain_run_short(const unsigned *__restrict__ words, unsigned nwords, unsigned tile,
                                                T *__restrict__ arena, wmc_meta *meta, char *smem) {
    const unsigned tid = threadIdx.x;
    unsigned *ch = (unsigned *)smem;
    T *lds = (T *)(smem + ((nwords * 4u + 1023u) & ~1023u));
    {
        constexpr unsigned NV = (3u << WMC_CHAIN_LANE) >> LB;  // words are at most 3 << WMC_CHAIN_LANE
        unsigned v[NV];
#pragma unroll
        for (unsigned j = 0; j < NV; ++j)
            if (tid + (j << LB) < nwords) v[j] = words[tid + (j << LB)];
#pragma unroll
        for (unsigned j = 0; j < NV; ++j)
            if (tid + (j << LB) < nwords) ch[tid + (j << LB)] = v[j];
    }
    __syncthreads();
    auto uni = [](unsigned x) { return (unsigned)__builtin_amdgcn_readfirstlane(x); };
    const unsigned L = uni(ch[CH_STAGES]), ob = uni(ch[CH_TILE_BITS]), wave = uni(tid >> 6);
    const ChainLanes cl = chain_lanes<CS_WORDS>(ch, L, ob, tile, meta);
    const T *F0 = arena + chain_base(uni(ch[CH_F]), uni(ch[CH_F_HI])) + (unsigned)__builtin_amdgcn_readlane(cl.off, 0);
    T *C = arena + chain_base(uni(ch[CH_C]), uni(ch[CH_C_HI])) + (unsigned)__builtin_amdgcn_readlane(cl.off, 1);
    const bool fcopy = uni(ch[CH_FCOPY]) != 0u;
    constexpr int WAVES = 1 << (LB - 6);
    if (fcopy) chain_copy<T, WAVES>(ch, ch + CH_X, F0, lds, wave);
    // the G_i are small: one wave copies each
#pragma clang loop unroll(disable)
    for (unsigned s = wave; s < L; s += WAVES) {
        const unsigned *w = ch + CH_WORDS + s * CS_WORDS;
        chain_copy<T, 1>(ch, w + CS_X,
                         arena + chain_base(uni(w[CS_G]), uni(w[CS_G_HI])) +
                             (unsigned)__builtin_amdgcn_readlane(cl.off, 2 + s),
                         lds, 0u);
    }
    unsigned mask[LB];
#pragma unroll
    for (int b = 0; b < LB; ++b) mask[b] = 0u - ((tid >> b) & 1u);
    const unsigned tc = uni(ch[CH_TC]);
    const int shift = chain_shifts(cl, L, meta, tc, tile == 0u, (int)uni(ch[CH_WORDS + CS_LIFT]));
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    unsigned range = 0;
    double vmax = 0.0;
#pragma clang loop unroll(disable)
    for (unsigned s = 0; s < L; ++s) {
        const unsigned *w = ch + CH_WORDS + s * CS_WORDS;
        const int se = __builtin_amdgcn_readlane(shift, s);
        double v = 0.0;
        if (s + 1 == L) {
            chain_stage_short_any<T, LB, false, true>(ch, w, wave, F0, C, lds, mask, se, vmax);
        } else {
            if (s == 0 && !fcopy) chain_stage_short_any<T, LB, true, false>(ch, w, wave, F0, C, lds, mask, se, v);
            else chain_stage_short_any<T, LB, false, false>(ch, w, wave, F0, C, lds, mask, se, v);
            range |= chain_range(v, s);
            chain_barrier();
        }
    }
    chain_end(meta, uni(ch[CH_MASK]), tc, range, vmax);
}

// Tiles [blk << jb, (blk + 1) << jb) of a chain of many tiles, in Gray order:
// consecutive tiles differ in one index bit, so each offset changes by one
// XOR.
template <typename T>
__device__ __forceinline__ void chain_run_big(chain_words ch, unsigned blk, unsigned jb, T *__restrict__ arena,
                                              wmc_meta *meta, T *lds) {
    const unsigned tid = threadIdx.x, lane = tid & 63u;
    const unsigned L = ch[CH_STAGES], ob = ch[CH_TILE_BITS];
    const ChainLanes cl = chain_lanes<CS_WORDS_BIG>(ch, L, ob, blk << jb, meta);
    unsigned cur = cl.off;
    const int shift = chain_shifts(cl, L, meta, ch[CH_TC], blk == 0u, (int)ch[CH_WORDS + CS_LIFT]);
    const unsigned tab = CH_WORDS + L * CS_WORDS_BIG + lane * ob;
    unsigned mask[6];
#pragma unroll
    for (int b = 0; b < 6; ++b) mask[b] = 0u - ((tid >> b) & 1u);
    const unsigned wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const T *F0 = arena + chain_base(ch[CH_F], ch[CH_F_HI]);
    T *C0 = arena + chain_base(ch[CH_C], ch[CH_C_HI]);
    const bool nt = ch[CH_NT] != 0u;
    unsigned range = 0;
    double vmax = 0.0;
    const unsigned ntile = 1u << jb;
#pragma clang loop unroll(disable)
    for (unsigned i = 0; i < ntile; ++i) {
        const T *S = F0 + (unsigned)__builtin_amdgcn_readlane(cur, 0);
        T *C = C0 + (unsigned)__builtin_amdgcn_readlane(cur, 1);
        unsigned flip = 0;
        if (i + 1 < ntile && lane < L + 2) flip = ch[tab + __builtin_ctz(i + 1)];
#pragma clang loop unroll(disable)
        for (unsigned s = 0; s < L; ++s) {
            chain_words st = ch + CH_WORDS + s * CS_WORDS_BIG;
            const T *G = arena + chain_base(st[CS_G], st[CS_G_HI]) + (unsigned)__builtin_amdgcn_readlane(cur, 2 + s);
            const int se = __builtin_amdgcn_readlane(shift, s);
            double v = 0.0;
            if (s + 1 == L) {
                chain_stage_any<T, false, true>(st, S, G, C, lds, mask, wave, se, nt, v);
                vmax = fmax(vmax, v);
            } else {
                if (s == 0) chain_stage_any<T, true, false>(st, S, G, C, lds, mask, wave, se, nt, v);
                else chain_stage_any<T, false, false>(st, S, G, C, lds, mask, wave, se, nt, v);
                range |= chain_range(v, s);
            }
            chain_barrier();
        }
        cur ^= flip;
    }
    chain_end(meta, ch[CH_MASK], ch[CH_TC], range, vmax);
}

// One level: workgroups [0, cblocks) run chain records, the rest the
// level's small nodes.
struct FusedStepArgs {
    const ChainRec *recs;
    const unsigned *words;
    const NodeDesc *nodes;
    const int *wave_node;
    long long node_work;
    unsigned cblocks, nblocks;
    int nnodes, pad;
};

#define WMC_CHAIN_THREADS_BIG (1 << WMC_CHAIN_LANE_BIG)

template <typename T, int LB>
__global__ void __launch_bounds__(1 << LB) k_chain(const FusedStepArgs a, T *__restrict__ arena, wmc_meta *meta,
                                                   const SliceGroup sg) {
    WMC_ENTER_SLICE(arena, meta, sg);
    extern __shared__ char smem_raw[];
    if (blockIdx.x < a.cblocks) {
        chain_words r = const_words((const unsigned *)(a.recs + blockIdx.x));
        chain_run_short<T, LB>(a.words + r[0], r[3], r[1], arena, meta, smem_raw);
    } else {
        nodes_body<T>(a.nodes, a.nnodes, a.node_work, arena, meta, a.wave_node, blockIdx.x - a.cblocks, a.nblocks);
    }
}

// One chain of many tiles.
template <typename T>
__global__ void __launch_bounds__(WMC_CHAIN_THREADS_BIG) k_chain_big(const ChainRec *recs, const unsigned *words,
                                                                     T *__restrict__ arena, wmc_meta *meta,
                                                                     const SliceGroup sg) {
    WMC_ENTER_SLICE(arena, meta, sg);
    extern __shared__ char smem_raw[];
    chain_words r = const_words((const unsigned *)(recs + blockIdx.x));
    chain_run_big<T>(const_words(words) + r[0], r[1], r[2], arena, meta, (T *)smem_raw);
}

// Workgroups of 2^LB threads for a step's small nodes.
template <int LB>
static inline unsigned chain_node_blocks(long long work) {
    const long long b = (work + (1 << LB) - 1) >> LB;
    return (unsigned)(b > (1ll << 20) ? 1ll << 20 : b);
}

template <typename T, int LB>
static inline void launch_fused_step(const FusedStepArgs &a, int lds, T *arena, wmc_meta *meta, hipStream_t st,
                                     const SliceGroup sg = SliceGroup{0, 0, 0}, unsigned nz = 1) {
    const unsigned g = a.cblocks + a.nblocks;
    if (g)
        hipLaunchKernelGGL((k_chain<T, LB>), dim3(g, 1, nz), dim3(1 << LB), (size_t)lds * sizeof(T), st, a, arena, meta,
                           sg);
}

template <typename T>
static inline void launch_chain_big(const FusedStepArgs &a, int lds, T *arena, wmc_meta *meta, hipStream_t st,
                                    const SliceGroup sg = SliceGroup{0, 0, 0}, unsigned nz = 1) {
    hipLaunchKernelGGL(k_chain_big<T>, dim3(a.cblocks, 1, nz), dim3(WMC_CHAIN_THREADS_BIG), (size_t)lds * sizeof(T), st,
                       a.recs, a.words, arena, meta, sg);
}
