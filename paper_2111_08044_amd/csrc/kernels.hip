// HIP kernels of the Floquet brickwork engine (gfx950, wave64).
//
//  k_sweep_tiles / k_sweep_lanes / k_sweep_quads / k_sweep_one
//             fused gate sweep: one HBM read + write of the state applies
//             every gate of a pass (Sec. II Eq. (2), fused as in Sec. II).
//  k_rdm_windows / k_rdm
//             two-site reduced density matrices of the bonds of a pass (plus
//             the norm): exact products of the stored amplitudes, FP64 sums
//             (Sec. II Eq. (1); Sec. IV Eq. (10)).
//  k_apply_h_tiles / k_apply_h
//             lambda = H0 psi, out of place (Sec. IV Eq. (11), Sec. V).
//  k_adjoint_tiles / k_adjoint_quads / k_adjoint_one / k_adjoint_win4
//             reverse replay with G^dagger and the overlap terms of the
//             gradient of <H0>.
//  k_dense6 / k_dense4
//             pre-multiplied 6-qubit (FP32 or split BF16x3) and 4-qubit (FP32)
//             windows on the matrix cores (Sec. II on half-precision matrix
//             units).
//  k_init     product initial state (Sec. IV Eq. (9) form; product of spinors).
//  k_overlap  <phi|psi> and both norms across precisions (Sec. V echo measure).
//  k_finalize deterministic sum of per-workgroup partials.
//
// Tile kernels hold a tile of 2^K amplitudes (see fl_common.h for the
// geometry); each thread keeps 2^R amplitudes of one register group in VGPRs,
// applies the group's 4x4 gates there, and the tile changes register layout
// between groups through LDS.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fl_common.h"
#include "kernels.h"

namespace fl {

template <typename T> struct CT;
template <> struct CT<float> { typedef float2 c; };
template <> struct CT<double> { typedef double2 c; };

typedef float fl_f32x4 __attribute__((ext_vector_type(4)));
typedef double fl_f64x2 __attribute__((ext_vector_type(2)));
typedef float fl_f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 fl_bf16x8 __attribute__((ext_vector_type(8)));

// ---------------------------------------------------------------------------
// register-level gate application
// ---------------------------------------------------------------------------

// out_i = sum_j G_ij a_j on the four amplitudes whose register index has bits
// (I, I+1) = local index (2*bit(I+1) + bit(I)), for every value of the other
// R-2 register bits.  G holds 16 complex entries, row-major, (re, im) pairs, in
// registers; the amplitudes are updated in place.
// Every output first sums the seven terms that do not hold its own input
// amplitude; the last FMA of output (re|im)_i then adds the diagonal term
// Re(G_ii) (re|im)_i.  That FMA is the last read of its input, so it can
// write the result into the input's own register: each variant ends with
// every amplitude in the register it started in, and the variants for
// different I rejoin without register copies.
// The empty asm markers carry the bit position as an immediate: they keep the
// optimizer from merging the variants for different I into one body with
// run-time register indices (which would force the arrays into scratch).
template <typename T, int R, int I>
__device__ __forceinline__ void apply_pair_g(T (&vr)[1 << R], T (&vi)[1 << R], const T (&g)[32]) {
    __asm__ volatile("; gate on register bits %0" ::"i"(I));
#pragma unroll
    for (int c = 0; c < (1 << (R - 2)); ++c) {
        const int b = (c & ((1 << I) - 1)) | ((c >> I) << (I + 2));
        T sr[4], si[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = b | (i << I);
            sr[i] = -g[8 * i + 2 * i + 1] * vi[e];
            si[i] = g[8 * i + 2 * i + 1] * vr[e];
#pragma unroll
            for (int jj = 1; jj < 4; ++jj) {
                const int j = (i + jj) & 3;
                const int f = b | (j << I);
                sr[i] = fma(g[8 * i + 2 * j], vr[f], sr[i]);
                sr[i] = fma(-g[8 * i + 2 * j + 1], vi[f], sr[i]);
                si[i] = fma(g[8 * i + 2 * j], vi[f], si[i]);
                si[i] = fma(g[8 * i + 2 * j + 1], vr[f], si[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = b | (i << I);
            vr[e] = fma(g[8 * i + 2 * i], vr[e], sr[i]);
            vi[e] = fma(g[8 * i + 2 * i], vi[e], si[i]);
        }
    }
    __asm__ volatile("; end gate on register bits %0" ::"i"(I));
}

// Calls f(std::integral_constant<int, I>) for the run-time bit position
// i in [0, R-2].  The last position is the switch default, so every path of
// the switch applies a gate: a path that did nothing would rejoin the others
// with the untouched values and cost register copies at the join.
template <int R, typename F>
__device__ __forceinline__ void with_bit(int i, F&& f) {
    static_assert(R == 3 || R == 4, "register group size");
    if constexpr (R == 3) {
        switch (i) {
            case 0: f(std::integral_constant<int, 0>{}); break;
            default: f(std::integral_constant<int, 1>{}); break;
        }
    } else {
        switch (i) {
            case 0: f(std::integral_constant<int, 0>{}); break;
            case 1: f(std::integral_constant<int, 1>{}); break;
            default: f(std::integral_constant<int, 2>{}); break;
        }
    }
}

template <typename T, int R>
__device__ __forceinline__ void apply_op_g(T (&vr)[1 << R], T (&vi)[1 << R], int i, const T (&g)[32]) {
    with_bit<R>(i, [&](auto I) { apply_pair_g<T, R, decltype(I)::value>(vr, vi, g); });
}

// ---------------------------------------------------------------------------
// tile load / store (global <-> LDS), 16-byte global accesses
// ---------------------------------------------------------------------------

// LDS slot of tile element j: fl_swz (SW = 0) or fl_swz12 (SW = 1)
template <int SW>
__device__ __forceinline__ uint32_t tile_swz(uint32_t j) {
    return SW ? fl_swz12(j) : fl_swz(j);
}

template <typename T, int KT, int NT = FL_NT, int SW = 0>
__device__ __forceinline__ void tile_load(const typename CT<T>::c* __restrict__ psi, uint64_t base, int K, int C,
                                          int h, typename CT<T>::c* lds) {
    typedef typename CT<T>::c cplx;
    if constexpr (sizeof(T) == 4) {
        const int n2 = 1 << (K - 1);  // pairs of amplitudes
        if constexpr (KT > 0) {
            constexpr int ITER = (1 << (KT - 1)) / NT;
            float4 v[ITER];
#pragma unroll
            for (int s = 0; s < ITER; ++s) {
                const uint32_t j = 2u * (threadIdx.x + s * NT);
                // streaming: each amplitude is read once per pass
                const fl_f32x4 t =
                    __builtin_nontemporal_load(reinterpret_cast<const fl_f32x4*>(psi + base + fl_tile_offset(j, C, h)));
                v[s] = make_float4(t[0], t[1], t[2], t[3]);
            }
#pragma unroll
            for (int s = 0; s < ITER; ++s) {
                const uint32_t j = 2u * (threadIdx.x + s * NT);
                lds[tile_swz<SW>(j)] = make_float2(v[s].x, v[s].y);
                lds[tile_swz<SW>(j + 1)] = make_float2(v[s].z, v[s].w);
            }
        } else {
            for (int p = threadIdx.x; p < n2; p += NT) {
                const uint32_t j = 2u * p;
                const float4 v = *reinterpret_cast<const float4*>(psi + base + fl_tile_offset(j, C, h));
                lds[tile_swz<SW>(j)] = make_float2(v.x, v.y);
                lds[tile_swz<SW>(j + 1)] = make_float2(v.z, v.w);
            }
        }
    } else {
        const int n = 1 << K;
        if constexpr (KT > 0) {
            constexpr int ITER = (1 << KT) / NT;
            cplx v[ITER];
#pragma unroll
            for (int s = 0; s < ITER; ++s) {
                const uint32_t j = threadIdx.x + s * NT;
                v[s] = psi[base + fl_tile_offset(j, C, h)];
            }
#pragma unroll
            for (int s = 0; s < ITER; ++s) lds[tile_swz<SW>(threadIdx.x + s * NT)] = v[s];
        } else {
            for (int j = threadIdx.x; j < n; j += NT) lds[tile_swz<SW>(j)] = psi[base + fl_tile_offset(j, C, h)];
        }
    }
}

template <typename T, int KT, int NT = FL_NT, int SW = 0>
__device__ __forceinline__ void tile_store(typename CT<T>::c* __restrict__ psi, uint64_t base, int K, int C, int h,
                                           const typename CT<T>::c* lds) {
    if constexpr (sizeof(T) == 4) {
        const int n2 = 1 << (K - 1);
        if constexpr (KT > 0) {
            constexpr int ITER = (1 << (KT - 1)) / NT;
#pragma unroll
            for (int s = 0; s < ITER; ++s) {
                const uint32_t j = 2u * (threadIdx.x + s * NT);
                const float2 a = lds[tile_swz<SW>(j)], b = lds[tile_swz<SW>(j + 1)];
                const fl_f32x4 t = {a.x, a.y, b.x, b.y};
                __builtin_nontemporal_store(t, reinterpret_cast<fl_f32x4*>(psi + base + fl_tile_offset(j, C, h)));
            }
        } else {
            for (int p = threadIdx.x; p < n2; p += NT) {
                const uint32_t j = 2u * p;
                const float2 a = lds[tile_swz<SW>(j)], b = lds[tile_swz<SW>(j + 1)];
                *reinterpret_cast<float4*>(psi + base + fl_tile_offset(j, C, h)) = make_float4(a.x, a.y, b.x, b.y);
            }
        }
    } else {
        const int n = 1 << K;
        for (int j = threadIdx.x; j < n; j += NT) psi[base + fl_tile_offset(j, C, h)] = lds[tile_swz<SW>(j)];
    }
}

// ---------------------------------------------------------------------------
// fused sweep
// ---------------------------------------------------------------------------

// Reads one gate (32 reals, one address for the whole wave: broadcasts) from
// the workgroup's LDS copy of the gate table.
template <typename T>
__device__ __forceinline__ void load_gate_lds(const T* src, T (&gv)[32]) {
    typedef typename std::conditional<sizeof(T) == 4, fl_f32x4, fl_f64x2>::type v16;
    constexpr int PER = 16 / sizeof(T);
#pragma unroll
    for (int k = 0; k < 32 / PER; ++k) {
        const v16 v = reinterpret_cast<const v16*>(src)[k];
#pragma unroll
        for (int e = 0; e < PER; ++e) gv[PER * k + e] = v[e];
    }
}

// The first NO outputs of a gate on one quad (v holds the quad, g the NO rows),
// their chains side by side: a wave alone on its SIMD would wait for each FMA's
// result on two chains.  Each output is the same sum in the same order as in
// apply_pair_g: own imaginary term, the others in cyclic order, own real term.
template <typename T, int NO>
__device__ __forceinline__ void apply_rows(T (&vr)[4], T (&vi)[4], const T (&g)[8 * NO]) {
    T sr[NO], si[NO];
#pragma unroll
    for (int i = 0; i < NO; ++i) {
        sr[i] = -g[10 * i + 1] * vi[i];
        si[i] = g[10 * i + 1] * vr[i];
    }
#pragma unroll
    for (int jj = 1; jj < 4; ++jj) {
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            const int j = (i + jj) & 3;
            sr[i] = fma(g[8 * i + 2 * j], vr[j], sr[i]);
            si[i] = fma(g[8 * i + 2 * j], vi[j], si[i]);
        }
#pragma unroll
        for (int i = 0; i < NO; ++i) {
            const int j = (i + jj) & 3;
            sr[i] = fma(-g[8 * i + 2 * j + 1], vi[j], sr[i]);
            si[i] = fma(g[8 * i + 2 * j + 1], vr[j], si[i]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < NO; ++i) {
        vr[i] = fma(g[10 * i], vr[i], sr[i]);
        vi[i] = fma(g[10 * i], vi[i], si[i]);
    }
}

// A thread's place in a quad chain with S threads per quad: the quad, and the
// first of the 4 / S outputs that it computes.  The threads of a quad are lanes
// of one wave, so all of them have read the quad before any writes to it.
template <int S>
struct fl_quad_lane {
    static constexpr int QPW = 64 / S;   // quads per wave
    uint32_t quad, rot;
    __device__ __forceinline__ fl_quad_lane()
        : quad((threadIdx.x >> 6) * QPW + (threadIdx.x & (QPW - 1))), rot(((threadIdx.x & 63) / QPW) * (4 / S)) {}
};

// LDS byte offsets of the thread's quad on tile bits (u0, u0 + 1): la[m] is
// amplitude (m + rot) & 3.
template <typename T, int S>
__device__ __forceinline__ void quad_addr(const fl_quad_lane<S>& me, int u0, uint32_t (&la)[4]) {
    constexpr uint32_t SZ = sizeof(typename CT<T>::c);
    const uint32_t s0 = fl_swz(1u << u0) * SZ, s1 = fl_swz(2u << u0) * SZ;
    const uint32_t b = fl_swz(fl_spread(me.quad, u0, 2)) * SZ;
    if constexpr (S == 4) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const uint32_t x = m + me.rot;
            la[m] = b ^ ((x & 1) ? s0 : 0u) ^ ((x & 2) ? s1 : 0u);
        }
    } else {
        la[0] = S == 2 ? b ^ (me.rot ? s1 : 0u) : b;
        la[1] = la[0] ^ s0;
        la[2] = la[0] ^ s1;
        la[3] = la[1] ^ s1;
    }
}

// Rows rot .. rot + 4 / S - 1 of the gate at src, their columns from rot on.
template <typename T, int S>
__device__ __forceinline__ void load_gate_rows(const fl_quad_lane<S>& me, const T* src, T (&g)[32 / S]) {
    typedef typename CT<T>::c cplx;
    constexpr int NO = 4 / S;
    src += 8 * me.rot;
    if constexpr (S == 1) {
        load_gate_lds<T>(src, g);
    } else if constexpr (S == 2 && sizeof(T) == 4) {
#pragma unroll
        for (int i = 0; i < NO; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const fl_f32x4 v = *reinterpret_cast<const fl_f32x4*>(src + 8 * i + ((4 * h) ^ (2 * me.rot)));
#pragma unroll
                for (int x = 0; x < 4; ++x) g[8 * i + 4 * h + x] = v[x];
            }
    } else {
#pragma unroll
        for (int i = 0; i < NO; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const cplx v = *reinterpret_cast<const cplx*>(src + 8 * i + 2 * ((j + me.rot) & 3));
                g[8 * i + 2 * j] = v.x;
                g[8 * i + 2 * j + 1] = v.y;
            }
    }
}

// Applies the pass's gates to a tile (or a whole short chain) in LDS, one quad
// of amplitudes per S threads and gate, a barrier between gates.  A serial
// chain: only its latency matters, so the next gate's descriptor word, its
// address and its entries (from lg) are fetched while the current one's FMAs
// run, and between two barriers a thread only reads its quad, applies 64 / S
// FMAs and writes its outputs back.  Each thread holds the quad and its gate
// rows rotated, so that its first output stands first; the sums do not depend
// on S.  The nops gates run over and over, total gates in all.  About 0.33 us a
// gate (0.39 with one thread per quad, of which 0.13 are the 64 FMAs of a wave
// alone on its SIMD).  meta holds a pass in words form with one op per group:
// first bits, then gates << 8.
template <typename T, int S>
__device__ __forceinline__ void quad_chain(typename CT<T>::c* lds, const T* lg, const uint32_t* meta, int nops, int total,
                                           const fl_quad_lane<S>& me, bool active) {
    typedef typename CT<T>::c cplx;
    constexpr int NO = 4 / S;
    char* const lb = reinterpret_cast<char*>(lds);
    // word k: head (first bit) and op of gate k
    auto word = [&](int k) {
        return (uint32_t)__builtin_amdgcn_readfirstlane(meta[k] & 255u) |
               (uint32_t)__builtin_amdgcn_readfirstlane(meta[nops + k]) << 8;
    };
    if (nops == 0) return;
    T ga[8 * NO], gb[8 * NO];
    uint32_t w = word(0), la[4];
    load_gate_rows<T, S>(me, lg + 32 * (w >> 16), ga);
    quad_addr<T, S>(me, w & 255, la);
    auto after = [&](int k) { return k + 1 < nops ? k + 1 : 0; };
    int kn = after(0);   // the gate after the current one
    uint32_t wn = word(kn);
    // one gate with its entries in g; the next one's go to gn
    auto step = [&](const T (&g)[8 * NO], T (&gn)[8 * NO]) {
        T vr[4], vi[4];
        if (active) {
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const cplx a = *reinterpret_cast<const cplx*>(lb + la[m]);
                vr[m] = a.x;
                vi[m] = a.y;
            }
        }
        __builtin_amdgcn_sched_barrier(0);   // the quad's reads lead the LDS queue
        // the next gate: its word was read one gate ago
        uint32_t ln[4];
        quad_addr<T, S>(me, wn & 255, ln);
        load_gate_rows<T, S>(me, lg + 32 * (wn >> 16), gn);
        kn = after(kn);
        const uint32_t h2 = meta[kn], o2 = meta[nops + kn];
#pragma unroll
        for (int m = 0; m < 4; ++m) __asm__ volatile("" : "+v"(ln[m]));
        __builtin_amdgcn_sched_barrier(0);
        if (active) {
            apply_rows<T, NO>(vr, vi, g);
#pragma unroll
            for (int m = 0; m < NO; ++m) {
                cplx a;
                a.x = vr[m];
                a.y = vi[m];
                *reinterpret_cast<cplx*>(lb + la[m]) = a;
            }
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) la[m] = ln[m];
        wn = (uint32_t)__builtin_amdgcn_readfirstlane(h2 & 255u) | (uint32_t)__builtin_amdgcn_readfirstlane(o2) << 8;
        __syncthreads();
    };
    for (int q = 0; q < total; q += 2) {
        step(ga, gb);
        if (q + 1 < total) step(gb, ga);
    }
}

// Chains of at most FL_KMAX_ONE sites: one workgroup holds the whole state in
// LDS for reps runs of the pass.
template <typename T, int S, int NT>
__global__ __launch_bounds__(NT) void k_sweep_one(typename CT<T>::c* __restrict__ psi, const T* __restrict__ gates,
                                                  int L, fl_sweep_words pd, int reps) {
    typedef typename CT<T>::c cplx;
    __shared__ __attribute__((aligned(16))) T lg[FL_KMAX_ONE * 32];
    __shared__ uint32_t meta[FL_SWEEP_WORDS];
    __shared__ __attribute__((aligned(16))) cplx lds[1 << FL_KMAX_ONE];
    for (uint32_t j = threadIdx.x; j < (1u << L); j += NT) lds[fl_swz(j)] = psi[j];
    for (int t = threadIdx.x; t < (L - 1) * 32; t += NT) lg[t] = gates[t];
    for (int t = threadIdx.x; t < pd.nwords; t += NT) meta[t] = pd.w[t];
    __syncthreads();
    const fl_quad_lane<S> me;
    quad_chain<T, S>(lds, lg, meta, pd.ngroups, pd.ngroups * reps, me, me.quad < (1u << (L - 2)));
    for (uint32_t j = threadIdx.x; j < (1u << L); j += NT) psi[j] = lds[fl_swz(j)];
}

// Tiles of 2^KT amplitudes (KT = 11), one per workgroup: eight waves of one
// thread per quad (16 periods at L = 19: 190 us, 193 with two per quad).
template <typename T, int KT, int CL>
__global__ __launch_bounds__(1 << (KT - 2)) void k_sweep_quads(typename CT<T>::c* __restrict__ psi,
                                                              const T* __restrict__ gates, int W, fl_sweep_words pd,
                                                              int ngates) {
    typedef typename CT<T>::c cplx;
    constexpr int K = KT, C = CL, NT = 1 << (K - 2);
    constexpr int APL = sizeof(T) == 4 ? 2 : 1;   // amplitudes per 16 bytes
    constexpr int ITER = (1 << K) / (APL * NT);
    static_assert(ITER >= 1, "a whole access per thread");
    static_assert((APL * NT) % (1 << C) == 0, "tile access stride");
    typedef typename std::conditional<sizeof(T) == 4, fl_f32x4, fl_f64x2>::type v16;
    __shared__ __attribute__((aligned(16))) cplx lds[1 << K];
    __shared__ __attribute__((aligned(16))) T lg[FL_MAX_GATE_TABLE * 32];
    __shared__ uint32_t meta[FL_SWEEP_WORDS];
    const int h = pd.h;
    cplx* const src = psi + fl_tile_base(blockIdx.x, C, W, h) + fl_tile_offset(APL * threadIdx.x, C, h);
    const uint64_t tstride = (uint64_t)((APL * NT) >> C) << h;
    const uint32_t l0 = fl_swz(APL * threadIdx.x);
    v16 a[ITER];
#pragma unroll
    for (int s = 0; s < ITER; ++s) a[s] = *reinterpret_cast<const v16*>(src + s * tstride);
    const fl_f32x4* gsrc = reinterpret_cast<const fl_f32x4*>(gates);
    for (int t = threadIdx.x; t < ngates * (int)(32 * sizeof(T) / 16); t += NT) reinterpret_cast<fl_f32x4*>(lg)[t] = gsrc[t];
    for (int t = threadIdx.x; t < pd.nwords; t += NT) meta[t] = pd.w[t];
#pragma unroll
    for (int s = 0; s < ITER; ++s) {
        const uint32_t l = l0 ^ fl_swz((uint32_t)(s * APL * NT));
        if constexpr (sizeof(T) == 4) {
            lds[l] = make_float2(a[s][0], a[s][1]);
            lds[l ^ 1] = make_float2(a[s][2], a[s][3]);
        } else {
            lds[l] = make_double2(a[s][0], a[s][1]);
        }
    }
    __syncthreads();
    quad_chain<T, 1>(lds, lg, meta, pd.ngroups, pd.ngroups, fl_quad_lane<1>(), true);
#pragma unroll
    for (int s = 0; s < ITER; ++s) {
        const uint32_t l = l0 ^ fl_swz((uint32_t)(s * APL * NT));
        v16 x;
        if constexpr (sizeof(T) == 4) {
            const float2 p = lds[l], q = lds[l ^ 1];
            x = v16{p.x, p.y, q.x, q.y};
        } else {
            const double2 p = lds[l];
            x = v16{p.x, p.y};
        }
        *reinterpret_cast<v16*>(src + s * tstride) = x;
    }
}

// Op q of group g as (gate-table index, register bit), read as aligned 32-bit
// words of the pass descriptor so that the loads stay scalar (sub-dword
// loads of the kernel arguments would go through the vector memory path).
typedef int32_t __attribute__((may_alias)) fl_i32a;
__device__ __forceinline__ int pass_gate(const fl_pass& pd, int g, int q) {
    const int32_t w = reinterpret_cast<const fl_i32a*>(&pd.opg[g][0])[q >> 1];
    return (q & 1) ? (w >> 16) : (int)(int16_t)(w & 0xffff);
}
__device__ __forceinline__ int pass_slot(const fl_pass& pd, int g, int q) {
    const int32_t w = reinterpret_cast<const fl_i32a*>(&pd.ops[g][0])[q >> 1];
    return (q & 1) ? (w >> 16) : (int)(int16_t)(w & 0xffff);
}
__device__ __forceinline__ int pass_byte(const int8_t* row, int i) {
    const int32_t w = reinterpret_cast<const fl_i32a*>(row)[i >> 2];
    return (int)(int8_t)((w >> (8 * (i & 3))) & 0xff);
}
__device__ __forceinline__ int pass_u0(const fl_pass& pd, int g) { return pass_byte(pd.u0, g); }
__device__ __forceinline__ int pass_nops(const fl_pass& pd, int g) { return pass_byte(pd.nops, g); }
__device__ __forceinline__ int pass_bit(const fl_pass& pd, int g, int q) {
    const int32_t w = reinterpret_cast<const fl_i32a*>(&pd.opi[g][0])[q >> 2];
    return (w >> (8 * (q & 3))) & 0xff;
}

// lgkmcnt(0) with no wait on the vector-memory and export counters.
#define FL_WAIT_LGKM0 0xc07f

// The ops of register group g applied to the thread's register group, the
// gates read from the workgroup's LDS copy of the table (lg, 32 reals per
// gate) into vector registers: FP32 FMAs whose operands all sit in vector
// registers can issue two per cycle per SIMD on gfx950 when two waves have one
// ready, where an FMA that reads a scalar register issues alone.  (complex128:
// two 64-register gates do not fit the scalar registers; fetched one ahead
// they spilled 231 of them, 2970 us for 16 periods at L = 23 against 2420.)
// Ops run two per iteration: the register copies that LLVM places on a loop
// back edge after the choice of gate bits are then not needed at all.
template <typename T, int R>
__device__ __forceinline__ void sweep_group_ops(T (&vr)[1 << R], T (&vi)[1 << R], const fl_pass& pd, int g,
                                                const T* lg, int gofs) {
    const int nops = pass_nops(pd, g);
    // op metadata (bit, gate index) is read with scalar loads one op ahead;
    // LDS and scalar loads share one wait counter, so the next op's scalar
    // loads are issued only after this op's gate has arrived from LDS, and
    // they complete under the op's FMAs.
    int bit = pass_bit(pd, g, 0), idx = pass_gate(pd, g, 0) - gofs;
    auto run = [&](int q) {
        __builtin_amdgcn_s_waitcnt(FL_WAIT_LGKM0);
        T gv[32];
        load_gate_lds<T>(lg + 32 * idx, gv);
        __builtin_amdgcn_s_waitcnt(FL_WAIT_LGKM0);
        const int i = bit;
        const int qn = q + 1 < nops ? q + 1 : q;
        bit = pass_bit(pd, g, qn);
        idx = pass_gate(pd, g, qn) - gofs;
        apply_op_g<T, R>(vr, vi, i, gv);
    };
    for (int q = 0; q < nops; q += 2) {
        run(q);
        if (q + 1 < nops) run(q + 1);
    }
}

// Tiles of 2^KT amplitudes, one per workgroup; every thread holds one register
// group of 2^R amplitudes.  D is the descriptor: fl_pass, read with scalar
// loads (many workgroups per CU: the loads hit the scalar cache and other
// waves fill the wait), or fl_sweep_words, copied to LDS (short chains with at
// most one workgroup per CU, where a scalar-cache miss per group or op would
// add to a serial chain: 16 periods at L = 17 on 10-bit tiles with 3-bit groups
// took 170 us against 192 with scalar loads).
//
// The first group is loaded straight from HBM into its register layout, and
// the last group stored straight back, when the group's lowest bit u0 is at
// least FL_DIRECT_MIN_U0: the lanes then still cover runs of >= 2^4
// contiguous amplitudes (>= 128 bytes), so every access coalesces.  This
// saves one LDS round trip and one barrier at each end of the pass.  Groups
// starting lower go through the LDS transpose, as every middle group does.
template <typename T, int R, int KT, int NT, int CL, int WPE, typename D>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WPE))) void k_sweep_tiles(
    typename CT<T>::c* __restrict__ psi, const T* __restrict__ gates, int W, D pd, int ngates, int gofs) {
    typedef typename CT<T>::c cplx;
    constexpr bool LM = std::is_same<D, fl_sweep_words>::value;
    __shared__ __attribute__((aligned(16))) T lg[FL_MAX_GATE_TABLE * 32];
    __shared__ uint32_t meta[LM ? FL_SWEEP_WORDS : 1];
    // gates of the pass's direction: table entries gofs .. gofs + ngates - 1
    auto copy_tables = [&]() {
        const fl_f32x4* src = reinterpret_cast<const fl_f32x4*>(gates + 32 * gofs);
        for (int t = threadIdx.x; t < ngates * (int)(32 * sizeof(T) / 16); t += NT)
            reinterpret_cast<fl_f32x4*>(lg)[t] = src[t];
        if constexpr (LM)
            for (int t = threadIdx.x; t < pd.nwords; t += NT) meta[t] = pd.w[t];
    };
    constexpr int C = CL;
    constexpr int DMIN = C < FL_DIRECT_MIN_U0 ? C : FL_DIRECT_MIN_U0;   // lowest group bit for direct transfers
    constexpr int K = KT;
    static_assert((1 << (K - R)) == NT, "one register group per thread");
    constexpr int APL = (sizeof(T) == 4) ? 2 : 1;           // amplitudes per 16-byte access
    constexpr int ITER = (1 << K) / (APL * NT);
    typedef typename std::conditional<sizeof(T) == 4, float4, double2>::type v16;
    __shared__ cplx lds[1 << K];
    const int h = pd.h;
    const int ng = pd.ngroups;
    cplx* const base = psi + fl_tile_base(blockIdx.x, C, W, h);
    // Element j = APL (tid + s NT) of a tile sits at toff + s * tstride: APL NT
    // is a multiple of 2^C, so s only moves the window part of the offset.
    static_assert((APL * NT) % (1 << C) == 0, "tile access stride");
    const uint64_t toff = fl_tile_offset(APL * threadIdx.x, C, h);
    const uint64_t tstride = (uint64_t)((APL * NT) >> C) << h;
    // LDS slot of element j + s APL NT is fl_swz(j) ^ fl_swz(s APL NT) (the
    // swizzle is linear over XOR, the two have disjoint bits), and
    // fl_swz(j + 1) = fl_swz(j) ^ 1 for even j.
    const uint32_t l0 = fl_swz(APL * threadIdx.x);
    int ufirst = -1, ulast = -1;   // first bits of the first and the last group
    if constexpr (LM) {
        ufirst = pd.ufirst;
        ulast = pd.ulast;
    } else if (ng > 0) {
        ufirst = pass_u0(pd, 0);
        ulast = pass_u0(pd, ng - 1);
    }
    const bool din = ufirst >= DMIN;
    const bool dout = ulast >= DMIN;

    T vr[1 << R], vi[1 << R];
    // HBM offsets of a register group: element b0 | (m << u0) of the tile sits
    // at off(b0) + sum over the set bits k of m of d[k].
    auto group_offsets = [&](int u0, uint64_t& o, uint64_t (&d)[R]) {
#pragma unroll
        for (int k = 0; k < R; ++k) {
            const int q = u0 + k;
            d[k] = q < C ? (1ull << q) : (1ull << (h + q - C));
        }
        o = fl_tile_offset(fl_spread(threadIdx.x, u0, R), C, h);
    };
    auto moff = [&](const uint64_t (&d)[R], int m) {
        uint64_t r = 0;
#pragma unroll
        for (int k = 0; k < R; ++k)
            if ((m >> k) & 1) r += d[k];
        return r;
    };
    // LDS byte offsets of the current register group.  The swizzle is linear
    // over XOR and b0 and m << u0 have disjoint bits, so
    // slot(b0 | m << u0) = slot(b0) ^ slot(m << u0), and slot(m << u0) is the
    // XOR of the (uniform) slots of m's set bits: one VALU XOR per element.
    // Kept for the group's write-back.
    uint32_t la[1 << R];
    auto lds_addrs = [&](int u0) {
        uint32_t bk[R];
#pragma unroll
        for (int k = 0; k < R; ++k) bk[k] = fl_swz(1u << (u0 + k)) * (uint32_t)sizeof(cplx);
        la[0] = fl_swz(fl_spread(threadIdx.x, u0, R)) * (uint32_t)sizeof(cplx);
#pragma unroll
        for (int m = 1; m < (1 << R); ++m) la[m] = la[m & (m - 1)] ^ bk[__builtin_ctz(m)];
    };
    char* const lbytes = reinterpret_cast<char*>(lds);
    auto lds_to_regs = [&]() {
#pragma unroll
        for (int m = 0; m < (1 << R); ++m) {
            const cplx a = *reinterpret_cast<const cplx*>(lbytes + la[m]);
            vr[m] = a.x;
            vi[m] = a.y;
        }
    };
    auto regs_to_lds = [&]() {
#pragma unroll
        for (int m = 0; m < (1 << R); ++m) {
            cplx a;
            a.x = vr[m];
            a.y = vi[m];
            *reinterpret_cast<cplx*>(lbytes + la[m]) = a;
        }
    };

    // The tile's loads are issued before those of the tables, so that their
    // latencies overlap.
    if (din) {
        uint64_t o, d[R];
        group_offsets(ufirst, o, d);
#pragma unroll
        for (int m = 0; m < (1 << R); ++m) {
            const cplx a = base[o + moff(d, m)];
            vr[m] = a.x;
            vi[m] = a.y;
        }
        copy_tables();
    } else {
        v16 nxt[ITER];
#pragma unroll
        for (int s = 0; s < ITER; ++s) nxt[s] = *reinterpret_cast<const v16*>(base + toff + s * tstride);
        copy_tables();
#pragma unroll
        for (int s = 0; s < ITER; ++s) {
            const uint32_t l = l0 ^ fl_swz((uint32_t)(s * APL * NT));
            if constexpr (sizeof(T) == 4) {
                lds[l] = make_float2(nxt[s].x, nxt[s].y);
                lds[l ^ 1] = make_float2(nxt[s].z, nxt[s].w);
            } else {
                lds[l] = nxt[s];
            }
        }
        __syncthreads();
        if (ng > 0) {
            lds_addrs(ufirst);
            lds_to_regs();
        }
    }

    if (din) __syncthreads();   // the tables (the other path passed a barrier after the tile load)
    if constexpr (LM) {
        auto word_at = [&](int k) { return (uint32_t)__builtin_amdgcn_readfirstlane(meta[k]); };
        int pos = ng;   // the ops' words follow the groups' heads
        uint32_t head = word_at(0);
        if (din) lds_addrs(head & 255);
        for (int g = 0; g < ng; ++g) {
            const int nops = head >> 8;
            uint32_t word = word_at(pos);
            head = word_at(g + 1);   // past the last group: the first op's word, unused
            auto run = [&]() {
                T gv[32];
                load_gate_lds<T>(lg + 32 * (word >> 8), gv);
                const int i = word & 255;
                const uint32_t next = meta[++pos];
                apply_op_g<T, R>(vr, vi, i, gv);
                word = __builtin_amdgcn_readfirstlane(next);
            };
            for (int q = 0; q < nops; q += 2) {
                run();
                if (q + 1 < nops) run();
            }
            if (g == ng - 1 && dout) break;
            regs_to_lds();
            if (g + 1 < ng) lds_addrs(head & 255);
            __syncthreads();
            if (g + 1 < ng) lds_to_regs();
        }
    } else {
        for (int g = 0; g < ng; ++g) {
            if (g > 0 || din) lds_addrs(pass_u0(pd, g));
            if (g > 0) lds_to_regs();
            sweep_group_ops<T, R>(vr, vi, pd, g, lg, gofs);
            if (g == ng - 1 && dout) break;
            regs_to_lds();
            __syncthreads();
        }
    }

    if (dout) {
        uint64_t o, d[R];
        group_offsets(ulast, o, d);
#pragma unroll
        for (int m = 0; m < (1 << R); ++m) {
            cplx a;
            a.x = vr[m];
            a.y = vi[m];
            base[o + moff(d, m)] = a;
        }
    } else {
#pragma unroll
        for (int s = 0; s < ITER; ++s) {
            const uint32_t l = l0 ^ fl_swz((uint32_t)(s * APL * NT));
            if constexpr (sizeof(T) == 4) {
                const float2 a = lds[l], b = lds[l ^ 1];
                *reinterpret_cast<float4*>(base + toff + s * tstride) = make_float4(a.x, a.y, b.x, b.y);
            } else {
                *reinterpret_cast<v16*>(base + toff + s * tstride) = lds[l];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// wave-level reductions
// ---------------------------------------------------------------------------

// NV values per lane -> lane l returns the wave-wide sum of value index
// l >> (6 - log2 NV).  Each step keeps one half of the values and trades the
// other half with the partner lane, so the whole reduction costs
// NV/2 + NV/4 + ... shuffles instead of NV * 6.  Written as a template
// recursion so that every array index is a compile-time constant.
// FP32 form on gfx950: the first two steps are one v_permlane32_swap /
// v_permlane16_swap per value pair (the swap trades exactly the half that the
// partner keeps, so x' + y' is the step's result without any select), the
// distance-8 step moves the sent half by DPP row_ror:8 (= lane ^ 8 inside a
// row of 16), and the final in-quad steps use DPP quad_perm.
template <int CTRL>
__device__ __forceinline__ float fl_dpp_f(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xf, 0xf, false));
}

template <int N, int D>
__device__ __forceinline__ void tr_steps_f32(float (&v)[N], int lane) {
    if constexpr (N > 1) {
        constexpr int H = N / 2;
#pragma unroll
        for (int k = 0; k < H; ++k) {
            if constexpr (D == 32 || D == 16) {
                const auto r = (D == 32) ? __builtin_amdgcn_permlane32_swap(__float_as_uint(v[k]),
                                                                            __float_as_uint(v[k + H]), false, false)
                                         : __builtin_amdgcn_permlane16_swap(__float_as_uint(v[k]),
                                                                            __float_as_uint(v[k + H]), false, false);
                v[k] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
            } else {
                const bool upper = (lane & D) != 0;
                const float keep = upper ? v[k + H] : v[k];
                const float send = upper ? v[k] : v[k + H];
                // D = 8: row_ror:8 pairs lane i with i ^ 8.  D = 4:
                // row_half_mirror pairs lane i with 7 - i in its run of 8; any
                // pairing of the lanes with bit 2 clear to those with it set
                // serves, the later steps sum over the whole run.
                float got;
                if constexpr (D == 8)
                    got = fl_dpp_f<0x128>(send);
                else if constexpr (D == 4)
                    got = fl_dpp_f<0x141>(send);
                else
                    got = __shfl_xor(send, D);
                v[k] = keep + got;
            }
        }
        tr_steps_f32<H, D / 2>(*reinterpret_cast<float(*)[H]>(&v[0]), lane);
    } else {
        if constexpr (D >= 32) v[0] += __shfl_xor(v[0], 32);
        if constexpr (D >= 16) v[0] += __shfl_xor(v[0], 16);
        if constexpr (D >= 8) v[0] += fl_dpp_f<0x128>(v[0]);
        if constexpr (D >= 4) v[0] += fl_dpp_f<0x141>(v[0]);  // row_half_mirror: lane 7 - i of the run of 8
        if constexpr (D >= 2) v[0] += fl_dpp_f<0x4E>(v[0]);   // quad_perm(2,3,0,1): lane ^ 2
        if constexpr (D >= 1) v[0] += fl_dpp_f<0xB1>(v[0]);   // quad_perm(1,0,3,2): lane ^ 1
    }
}

// FP64 form: the same lane pattern as tr_steps_f32, moving each double as its
// two 32-bit halves (two permlane swaps or two DPP moves per value); the adds
// are FP64.
template <int CTRL>
__device__ __forceinline__ double fl_dpp_d(double x) {
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

template <int N, int D>
__device__ __forceinline__ void tr_steps_f64(double (&v)[N], int lane) {
    if constexpr (N > 1) {
        constexpr int H = N / 2;
#pragma unroll
        for (int k = 0; k < H; ++k) {
            if constexpr (D == 32 || D == 16) {
                const uint64_t a = (uint64_t)__double_as_longlong(v[k]), b = (uint64_t)__double_as_longlong(v[k + H]);
                const auto rl = (D == 32) ? __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false)
                                          : __builtin_amdgcn_permlane16_swap((uint32_t)a, (uint32_t)b, false, false);
                const auto rh = (D == 32)
                                    ? __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false)
                                    : __builtin_amdgcn_permlane16_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
                const double x = __longlong_as_double((long long)(((uint64_t)rh[0] << 32) | rl[0]));
                const double y = __longlong_as_double((long long)(((uint64_t)rh[1] << 32) | rl[1]));
                v[k] = x + y;
            } else {
                const bool upper = (lane & D) != 0;
                const double keep = upper ? v[k + H] : v[k];
                const double send = upper ? v[k] : v[k + H];
                double got;
                if constexpr (D == 8)
                    got = fl_dpp_d<0x128>(send);
                else if constexpr (D == 4)
                    got = fl_dpp_d<0x141>(send);
                else
                    got = __shfl_xor(send, D);
                v[k] = keep + got;
            }
        }
        tr_steps_f64<H, D / 2>(*reinterpret_cast<double(*)[H]>(&v[0]), lane);
    } else {
        if constexpr (D >= 32) v[0] += __shfl_xor(v[0], 32);
        if constexpr (D >= 16) v[0] += __shfl_xor(v[0], 16);
        if constexpr (D >= 8) v[0] += fl_dpp_d<0x128>(v[0]);
        if constexpr (D >= 4) v[0] += fl_dpp_d<0x141>(v[0]);
        if constexpr (D >= 2) v[0] += fl_dpp_d<0x4E>(v[0]);
        if constexpr (D >= 1) v[0] += fl_dpp_d<0xB1>(v[0]);
    }
}

template <typename T, int NV>
__device__ __forceinline__ T wave_transpose_reduce(T (&v)[NV]) {
    static_assert(NV >= 1 && NV <= 64 && (NV & (NV - 1)) == 0, "NV must be a power of two <= 64");
    if constexpr (sizeof(T) == 4)
        tr_steps_f32<NV, 32>(v, threadIdx.x & 63);
    else
        tr_steps_f64<NV, 32>(v, threadIdx.x & 63);
    return v[0];
}

// ---------------------------------------------------------------------------
// short chains: gates between the lanes of a wave
// ---------------------------------------------------------------------------
// lane ^ X of x for the distances of the quads on 4 lane bits
template <int X>
__device__ __forceinline__ float lane_xor(float x) {
    if constexpr (X == 1) return fl_dpp_f<0xB1>(x);                      // quad_perm(1,0,3,2)
    else if constexpr (X == 2) return fl_dpp_f<0x4E>(x);                 // quad_perm(2,3,0,1)
    else if constexpr (X == 3) return fl_dpp_f<0x1B>(x);                 // quad_perm(3,2,1,0)
    else if constexpr (X == 8) return fl_dpp_f<0x128>(x);                // row_ror:8
    else if constexpr (X == 4) return fl_dpp_f<0x141>(lane_xor<3>(x));   // row_half_mirror: ^ 7
    else if constexpr (X == 6) return fl_dpp_f<0x141>(lane_xor<1>(x));
    else {
        static_assert(X == 12, "distance");
        return fl_dpp_f<0x140>(lane_xor<3>(x));                          // row_mirror: ^ 15
    }
}
template <int X>
__device__ __forceinline__ double lane_xor(double x) {
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = __float_as_uint(lane_xor<X>(__uint_as_float((uint32_t)u)));
    const uint32_t hi = __float_as_uint(lane_xor<X>(__uint_as_float((uint32_t)(u >> 32))));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// A gate on lane bits (I, I + 1), one amplitude per lane: c holds the lane's
// row, entry d for the amplitude of the lane whose two bits differ by d.  The
// own real term comes last, as in apply_pair_g.
template <typename T, int I>
__device__ __forceinline__ void apply_lanes(T& vr, T& vi, const T (&c)[8]) {
    const T ar = lane_xor<(1 << I)>(vr), ai = lane_xor<(1 << I)>(vi);
    const T br = lane_xor<(2 << I)>(vr), bi = lane_xor<(2 << I)>(vi);
    const T dr = lane_xor<(3 << I)>(vr), di = lane_xor<(3 << I)>(vi);
    T sr = -c[1] * vi, si = c[1] * vr;
    sr = fma(c[2], ar, sr);
    si = fma(c[2], ai, si);
    sr = fma(-c[3], ai, sr);
    si = fma(c[3], ar, si);
    sr = fma(c[4], br, sr);
    si = fma(c[4], bi, si);
    sr = fma(-c[5], bi, sr);
    si = fma(c[5], br, si);
    sr = fma(c[6], dr, sr);
    si = fma(c[6], di, si);
    sr = fma(-c[7], di, sr);
    si = fma(c[7], dr, si);
    vr = fma(c[0], vr, sr);
    vi = fma(c[0], vi, si);
}

// The gate table as k_sweep_lanes reads it: entry d of row i is column i ^ d.
template <typename T>
__device__ __forceinline__ void lane_table(typename CT<T>::c* lg, const T* gates, int ngates, int nt) {
    const typename CT<T>::c* const src = reinterpret_cast<const typename CT<T>::c*>(gates);
    for (int t = threadIdx.x; t < ngates * 16; t += nt) lg[t] = src[(t & ~3) | ((t ^ (t >> 2)) & 3)];
}

// Tiles of 2^KT amplitudes (KT <= 10), one per workgroup and one amplitude per
// thread.  A register group's 4 tile bits are the low 4 lane bits: its gates
// exchange amplitudes between lanes of a row of 16 (DPP), with no LDS round
// trip and no barrier between them; only a change of group goes through LDS.
// The next gate's row, and the word of the one after, are fetched under the
// current one's FMAs.  Against the quad chain with two threads per quad (a
// barrier per gate), 16 periods (us): complex128 on 9 bits L = 12 80 / 92, 17
// 138 / 153, on 10 bits 18 169 / 181; complex64 on 10 bits L = 11 61 / 65, 12 70 /
// 73, 17 123 / 126, 18 140 / 144.  Bound by latency: of 0.3 us a gate the 16 FMAs,
// 6 to 8 lane moves and the waits between them, and a third of an LDS exchange.
// Two amplitudes per thread (half the waves) are slower: complex64 L = 12 72,
// complex128 L = 12 85.  In one workgroup (L <= 10) this form is within 5% of the
// quads, either way.
template <typename T, int KT, int CL>
__global__ __launch_bounds__(1 << KT) void k_sweep_lanes(typename CT<T>::c* __restrict__ psi,
                                                        const T* __restrict__ gates, int W, fl_sweep_words pd,
                                                        int ngates) {
    typedef typename CT<T>::c cplx;
    typedef typename std::conditional<sizeof(T) == 4, fl_f32x4, fl_f64x2>::type v16;
    constexpr int NT = 1 << KT, PER = 16 / sizeof(T);
    __shared__ __attribute__((aligned(16))) cplx lds[NT];
    __shared__ __attribute__((aligned(16))) cplx lgt[FL_MAX_GATE_TABLE * 16];
    __shared__ uint32_t meta[FL_SWEEP_WORDS];
    cplx* const p = psi + fl_tile_base(blockIdx.x, CL, W, pd.h) + fl_tile_offset(threadIdx.x, CL, pd.h);
    const cplx first = *p;
    lane_table<T>(lgt, gates, ngates, NT);
    for (int t = threadIdx.x; t < pd.nwords; t += NT) meta[t] = pd.w[t];
    lds[fl_swz(threadIdx.x)] = first;
    __syncthreads();
    const T* const lg = reinterpret_cast<const T*>(lgt);
    char* const lb = reinterpret_cast<char*>(lds);
    const int ng = pd.ngroups, nt = pd.nwords - 1 - ng;   // groups, gates
    const uint32_t m = threadIdx.x & 15;
    auto uni = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane(x); };
    auto addr = [&](uint32_t head) {
        const int u0 = head & 255;
        return fl_swz(fl_spread(threadIdx.x >> 4, u0, 4) | (m << u0)) * (uint32_t)sizeof(cplx);
    };
    auto row = [&](uint32_t w, T (&c)[8]) {
        const T* const src = lg + 32 * (w >> 8) + 8 * ((m >> (w & 255)) & 3);
#pragma unroll
        for (int k = 0; k < 8 / PER; ++k) {
            const v16 v = reinterpret_cast<const v16*>(src)[k];
#pragma unroll
            for (int e = 0; e < PER; ++e) c[PER * k + e] = v[e];
        }
    };
    if (nt > 0) {
        T ca[8], cb[8], vr, vi;
        uint32_t w = uni(meta[ng]), head = uni(meta[0]);
        row(w, ca);
        int pos = nt > 1 ? 1 : 0;
        uint32_t wn = uni(meta[ng + pos]);
        auto op = [&](const T (&c)[8], T (&cn)[8]) {
            row(wn, cn);
            if (pos + 1 < nt) ++pos;
            const uint32_t w2 = meta[ng + pos];
            with_bit<4>(w & 255, [&](auto I) { apply_lanes<T, decltype(I)::value>(vr, vi, c); });
            w = wn;
            wn = uni(w2);
        };
        for (int g = 0; g < ng; ++g) {
            const int nops = head >> 8;
            cplx* const at = reinterpret_cast<cplx*>(lb + addr(head));
            const cplx a = *at;
            vr = a.x;
            vi = a.y;
            const uint32_t next = meta[g + 1];   // past the last group: the first gate's word, unused
            for (int q = 0; q < nops; q += 2) {
                op(ca, cb);
                if (q + 1 < nops) {
                    op(cb, ca);
                } else {
#pragma unroll
                    for (int k = 0; k < 8; ++k) ca[k] = cb[k];
                }
            }
            cplx b;
            b.x = vr;
            b.y = vi;
            *at = b;
            head = uni(next);
            __syncthreads();
        }
    }
    *p = lds[fl_swz(threadIdx.x)];
}

// ---------------------------------------------------------------------------
// reduced density matrices of the bonds of a cover pass (+ norm)
// ---------------------------------------------------------------------------
// Per bond: rho[i][j] = sum_r psi_{r,i} conj(psi_{r,j}); stored as 16 reals:
// [0..3] = rho_ii, then (re, im) of rho_01, rho_02, rho_03, rho_12, rho_13, rho_23.
// partials layout: [gridDim.x][nslot][16] doubles, slot = bond, slot L-1 = norm.

#define FL_RDM_MAXG (FL_KMAX_RDM - 1)

// Chains below FL_RDM_MIN_WINDOWS sites, in one workgroup: bond by bond.
template <typename T>
__global__ __launch_bounds__(FL_NT) void k_rdm(const typename CT<T>::c* __restrict__ psi, int K, fl_pass pd,
                                               double* __restrict__ partials, int nslot) {
    typedef typename CT<T>::c cplx;
    __shared__ cplx lds[1 << FL_KMAX_RDM];
    __shared__ double wacc[FL_NT / 64][FL_RDM_MAXG + 1][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double acc[FL_RDM_MAXG];
#pragma unroll
    for (int g = 0; g < FL_RDM_MAXG; ++g) acc[g] = 0.0;
    double nrm = 0.0;
    const uint32_t ngrp = 1u << (K - 2);
    for (uint32_t j = threadIdx.x; j < (1u << K); j += FL_NT) {
        const cplx a = psi[j];
        lds[fl_swz(j)] = a;
        nrm += (double)a.x * (double)a.x + (double)a.y * (double)a.y;
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < FL_RDM_MAXG; ++g) {
        if (g < pd.ngroups) {
            const int u = pd.u0[g];
            double r[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) r[k] = 0.0;
            for (uint32_t o = threadIdx.x; o < ngrp; o += FL_NT) {
                const uint32_t b0 = fl_spread(o, u, 2);
                double ar[4], ai[4];
#pragma unroll
                for (int l = 0; l < 4; ++l) {
                    const cplx a = lds[fl_swz(b0 | ((uint32_t)l << u))];
                    ar[l] = a.x;
                    ai[l] = a.y;
                }
#pragma unroll
                for (int l = 0; l < 4; ++l) r[l] = fma(ar[l], ar[l], fma(ai[l], ai[l], r[l]));
                int k = 4;
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = i + 1; j < 4; ++j) {
                        r[k] = fma(ar[i], ar[j], fma(ai[i], ai[j], r[k]));
                        r[k + 1] = fma(ai[i], ar[j], fma(-ar[i], ai[j], r[k + 1]));
                        k += 2;
                    }
            }
            acc[g] += wave_transpose_reduce<double, 16>(r);
        }
    }
    // per-wave accumulators -> LDS -> the sums
    double nv[1] = {nrm};
    const double ntot = wave_transpose_reduce<double, 1>(nv);
    if ((lane & 3) == 0) {
#pragma unroll
        for (int g = 0; g < FL_RDM_MAXG; ++g) wacc[wave][g][lane >> 2] = acc[g];
    }
    if (lane == 0) wacc[wave][FL_RDM_MAXG][0] = ntot;
    __syncthreads();
    for (int t = threadIdx.x; t < (pd.ngroups + 1) * 16; t += FL_NT) {
        const int g = t >> 4, v = t & 15;
        const int gg = (g < pd.ngroups) ? g : FL_RDM_MAXG;
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < FL_NT / 64; ++w) s += wacc[w][gg][v];
        if (g < pd.ngroups)
            partials[(size_t)pd.ops[g][0] * 16 + v] = s;
        else if (v == 0)
            partials[(size_t)(nslot - 1) * 16] = s;
    }
}

// Chains from FL_RDM_MIN_WINDOWS sites on, in tiles of 2^K amplitudes.  The bonds of a
// pass come in 1, 2 or 4 windows of 4 consecutive tile bits (up to 3 bonds
// each); wave w sums window w mod nwin over all tiles of its workgroup, so a
// lane keeps a window's sums in registers from tile to tile and the wave trees
// run once every FL_RDM_FLUSH tiles instead of once per tile and bond.
//
// A window's bonds share their products.  The 16 |a_m|^2 give every diagonal
// entry (and the norm); the products of amplitude pairs that differ in bit k
// are summed by the values of the bits beside k, and give the entries 01, 23
// of the bond above and 02, 13 of the bond below; pairs that differ in both
// bits of a bond give 03 and 12.  That is 16 FMA an amplitude for three bonds
// (8 each when every bond forms its own 16 sums).
//
// All sums are FP64: complex64 amplitudes are widened first, so every product
// of two of them is exact and only the FP64 additions round, in chains of at
// most FL_RDM_FLUSH tiles and trees above them.
//
// Bound by the vector ALUs: at L = 27 the three passes issue 1.69e8, 1.35e8
// and 0.86e8 instructions, 87%, 79% and 61% of their 435, 383 and 316 us (medians
// of 20 under a kernel trace, which runs them 4% longer than the untraced whole)
// at the 2.3 ns a wave instruction takes here; the last pass, 6 bonds, waits for
// its reads the rest.  Readout at L = 27: 1.09 ms (1.54 with 16 sums per bond
// reduced per tile, on four passes of 7-bit windows), L = 30: 11.9 ms (13.4),
// complex128 L = 26: 0.70 ms (1.21).  3 low bits (64-byte runs) would save a
// pass at L = 30 but read slower: 11.8 ms there, 1.25 ms at L = 27.
// partials as in k_rdm.
#define FL_RDM_FLUSH 16

template <typename T, int K, int CL, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2))) void k_rdm_windows(
    const typename CT<T>::c* __restrict__ psi, int W, uint32_t ntiles, rdm_desc pd, double* __restrict__ partials,
    int nslot) {
    typedef typename CT<T>::c cplx;
    constexpr int C = CL, NW = NT / 64;
    constexpr int APL = sizeof(T) == 4 ? 2 : 1;
    constexpr int ITER = (1 << K) / (APL * NT);
    constexpr int UNITS = (1 << (K - 4)) / 64;   // wave-sized parts of a window's register groups
    static_assert(NW == 4 && UNITS >= 1, "1, 2 or 4 windows share the waves evenly (4 below 12 tile bits)");
    constexpr bool PREF = sizeof(T) == 4;   // complex128 has no registers left for the next tile
    typedef typename std::conditional<sizeof(T) == 4, fl_f32x4, fl_f64x2>::type v16;
    __shared__ __attribute__((aligned(16))) cplx lds[1 << K];
    __shared__ double wacc[NW][4][16];   // per wave: the window's three bonds, and the norm
    const int h = pd.h, nwin = pd.nwin;
    // readfirstlane: everything that hangs on the window is uniform
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int win = wave & (nwin - 1), part = wave / nwin, nunit = UNITS * nwin / NW;
    const int u0 = pd.u0[win], mask = pd.mask[win];   // bit j of mask: a bond on window bits (j, j + 1)
    for (int t = threadIdx.x; t < NW * 4 * 16; t += NT) (&wacc[0][0][0])[t] = 0.0;
    __syncthreads();
    static_assert((APL * NT) % (1 << C) == 0 && (APL * NT) % 256 == 0, "tile access stride");
    const uint64_t toff = fl_tile_offset(APL * threadIdx.x, C, h);
    const uint64_t tstride = (uint64_t)((APL * NT) >> C) << h;
    const uint32_t l0 = fl_swz(APL * threadIdx.x);
    uint32_t bk[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) bk[k] = fl_swz(1u << (u0 + k)) * (uint32_t)sizeof(cplx);

    double P[16], S[24], D[12];   // S: bit k's sums at 0, 4, 12, 20, (re, im) by its neighbours; D: 03, 12 of each bond
    auto clear = [&]() {
#pragma unroll
        for (int m = 0; m < 16; ++m) P[m] = 0.0;
#pragma unroll
        for (int m = 0; m < 24; ++m) S[m] = 0.0;
#pragma unroll
        for (int m = 0; m < 12; ++m) D[m] = 0.0;
    };
    clear();
    // the lanes' sums to the wave's accumulators, as the 16 reals of each bond
    auto flush = [&]() {
        auto add = [&](int row, double (&r)[16]) {
            const double red = wave_transpose_reduce<double, 16>(r);   // lane l: the sum of value l >> 2
            if ((lane & 3) == 0) wacc[wave][row][lane >> 2] += red;
        };
#pragma unroll
        for (int j = 0; j < 3; ++j)
            if ((mask >> j) & 1) {
                double r[16];
#pragma unroll
                for (int l = 0; l < 4; ++l) {
                    r[l] = 0.0;
#pragma unroll
                    for (int m = 0; m < 16; ++m)
                        if (((m >> j) & 3) == l) r[l] += P[m];
                }
                // bit k's sum at neighbour values (lo, hi); entries 01, 23: bit j by
                // its upper neighbour; 02, 13: bit j + 1 by its lower neighbour
                auto single = [&](int k, int lo, int hi, int c) {
                    const int off = k == 0 ? 0 : k == 1 ? 4 : k == 2 ? 12 : 20;
                    return S[off + 2 * (k == 0 ? hi : k == 3 ? lo : lo + 2 * hi) + c];
                };
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    r[4 + c] = j == 0 ? single(0, 0, 0, c) : single(j, 0, 0, c) + single(j, 1, 0, c);
                    r[14 + c] = j == 0 ? single(0, 0, 1, c) : single(j, 0, 1, c) + single(j, 1, 1, c);
                    r[6 + c] = j == 2 ? single(3, 0, 0, c) : single(j + 1, 0, 0, c) + single(j + 1, 0, 1, c);
                    r[12 + c] = j == 2 ? single(3, 1, 0, c) : single(j + 1, 1, 0, c) + single(j + 1, 1, 1, c);
                    r[8 + c] = D[4 * j + c];
                    r[10 + c] = D[4 * j + 2 + c];
                }
                add(j, r);
            }
        if (win == 0 && (pd.flags & 1)) {
            double n[1] = {0.0};
#pragma unroll
            for (int m = 0; m < 16; ++m) n[0] += P[m];
            const double red = wave_transpose_reduce<double, 1>(n);
            if (lane == 0) wacc[wave][3][0] += red;
        }
        clear();
    };
    v16 v[ITER];
    auto fetch = [&](uint32_t tile) {
        const cplx* src = psi + fl_tile_base(tile, C, W, h) + toff;
        // streaming: each amplitude is read once per pass
#pragma unroll
        for (int s = 0; s < ITER; ++s) v[s] = __builtin_nontemporal_load(reinterpret_cast<const v16*>(src + s * tstride));
    };
    if (PREF && blockIdx.x < ntiles) fetch(blockIdx.x);
    int held = 0;
    for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        if (!PREF) fetch(tile);
        __syncthreads();   // the previous tile's LDS reads are done
#pragma unroll
        for (int s = 0; s < ITER; ++s) {
            const uint32_t l = l0 + s * (APL * NT);
            if constexpr (sizeof(T) == 4) {
                lds[l] = make_float2(v[s][0], v[s][1]);
                lds[l ^ 1] = make_float2(v[s][2], v[s][3]);
            } else {
                lds[l] = make_double2(v[s][0], v[s][1]);
            }
        }
        __syncthreads();
        if (PREF && tile + gridDim.x < ntiles) fetch(tile + gridDim.x);
        for (int q = 0; q < nunit; ++q) {
            const uint32_t o = (uint32_t)(part * nunit + q) * 64 + lane;
            uint32_t la[16];
            la[0] = fl_swz(fl_spread(o, u0, 4)) * (uint32_t)sizeof(cplx);
#pragma unroll
            for (int m = 1; m < 16; ++m) la[m] = la[m & (m - 1)] ^ bk[__builtin_ctz(m)];
            double ar[16], ai[16];
#pragma unroll
            for (int m = 0; m < 16; ++m) {
                const cplx a = *reinterpret_cast<const cplx*>(reinterpret_cast<const char*>(lds) + la[m]);
                ar[m] = (double)a.x;
                ai[m] = (double)a.y;
            }
#pragma unroll
            for (int m = 0; m < 16; ++m) P[m] = fma(ar[m], ar[m], fma(ai[m], ai[m], P[m]));
            // (re, im) of a_x conj(a_y)
            auto pair_sum = [&](int x, int y, double& re, double& im) {
                re = fma(ar[x], ar[y], fma(ai[x], ai[y], re));
                im = fma(ai[x], ar[y], fma(-ar[x], ai[y], im));
            };
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (mask & (k == 0 ? 1 : k == 1 ? 3 : k == 2 ? 6 : 4)) {
                    const int off = k == 0 ? 0 : k == 1 ? 4 : k == 2 ? 12 : 20;
#pragma unroll
                    for (int m = 0; m < 16; ++m) {
                        if ((m >> k) & 1) continue;
                        const int lo = k > 0 ? (m >> (k - 1)) & 1 : 0, hi = k < 3 ? (m >> (k + 1)) & 1 : 0;
                        const int e = off + 2 * (k == 0 ? hi : k == 3 ? lo : lo + 2 * hi);
                        pair_sum(m, m | (1 << k), S[e], S[e + 1]);
                    }
                }
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if ((mask >> j) & 1) {
#pragma unroll
                    for (int m = 0; m < 16; ++m) {
                        if ((m >> (j + 1)) & 1) continue;
                        const int e = 4 * j + (((m >> j) & 1) ? 2 : 0);
                        pair_sum(m, m ^ (3 << j), D[e], D[e + 1]);
                    }
                }
        }
        if (++held == FL_RDM_FLUSH) {
            flush();
            held = 0;
        }
    }
    flush();
    __syncthreads();
    // the waves of a window in order -> partials[block][bond][16]
    for (int t = threadIdx.x; t < nwin * 64; t += NT) {
        const int w = t >> 6, row = (t >> 4) & 3, x = t & 15;
        double sum = 0.0;
        for (int k = w; k < NW; k += nwin) sum += wacc[k][row][x];
        if (row < 3 && ((pd.mask[w] >> row) & 1))
            partials[((size_t)blockIdx.x * nslot + pd.bond[w][row]) * 16 + x] = sum;
        else if (row == 3 && w == 0 && x == 0 && (pd.flags & 1))
            partials[((size_t)blockIdx.x * nslot + (nslot - 1)) * 16] = sum;
    }
}

// ---------------------------------------------------------------------------
// product state, overlap, finalize
// ---------------------------------------------------------------------------

template <typename T>
__global__ __launch_bounds__(256) void k_init(typename CT<T>::c* __restrict__ psi, const double2* __restrict__ tlo,
                                              const double2* __restrict__ tmid, const double2* __restrict__ thi,
                                              int a, int b, uint64_t n) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t x = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += stride) {
        const double2 p = thi[x >> (a + b)], q = tmid[(x >> a) & ((1ull << b) - 1ull)], r = tlo[x & ((1ull << a) - 1ull)];
        const double pr = p.x * q.x - p.y * q.y, pi = p.x * q.y + p.y * q.x;
        typename CT<T>::c o;
        o.x = (T)(pr * r.x - pi * r.y);
        o.y = (T)(pr * r.y + pi * r.x);
        psi[x] = o;
    }
}

// complex64 form: a thread writes amplitudes x, x + 1 (x even, one 16-byte
// store); they share the two high factors because the low table covers at
// least one bit.  Same FP64 arithmetic per amplitude as k_init.
__global__ __launch_bounds__(256) void k_init_pairs_c64(float4* __restrict__ psi2, const double2* __restrict__ tlo,
                                                       const double2* __restrict__ tmid,
                                                       const double2* __restrict__ thi, int a, int b, uint64_t n2) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n2; k += stride) {
        const uint64_t x = 2 * k;
        const double2 p = thi[x >> (a + b)], q = tmid[(x >> a) & ((1ull << b) - 1ull)];
        const double2 r0 = tlo[x & ((1ull << a) - 1ull)], r1 = tlo[(x + 1) & ((1ull << a) - 1ull)];
        const double pr = p.x * q.x - p.y * q.y, pi = p.x * q.y + p.y * q.x;
        float4 o;
        o.x = (float)(pr * r0.x - pi * r0.y);
        o.y = (float)(pr * r0.y + pi * r0.x);
        o.z = (float)(pr * r1.x - pi * r1.y);
        o.w = (float)(pr * r1.y + pi * r1.x);
        psi2[k] = o;
    }
}

template <typename TA, typename TB>
__global__ __launch_bounds__(256) void k_overlap(const typename CT<TA>::c* __restrict__ a,
                                                 const typename CT<TB>::c* __restrict__ b, uint64_t n,
                                                 double* __restrict__ partials) {
    __shared__ double wacc[4][4];
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t x = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += stride) {
        const double ar = a[x].x, ai = a[x].y, br = b[x].x, bi = b[x].y;
        v[0] = fma(ar, br, fma(ai, bi, v[0]));     // Re conj(a) b
        v[1] = fma(ar, bi, fma(-ai, br, v[1]));    // Im conj(a) b
        v[2] = fma(ar, ar, fma(ai, ai, v[2]));
        v[3] = fma(br, br, fma(bi, bi, v[3]));
    }
    const double r = wave_transpose_reduce<double, 4>(v);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if ((lane & 15) == 0) wacc[wave][lane >> 4] = r;
    __syncthreads();
    if (threadIdx.x < 4) {
        double s = 0.0;
        for (int w = 0; w < 4; ++w) s += wacc[w][threadIdx.x];
        partials[(size_t)blockIdx.x * 4 + threadIdx.x] = s;
    }
}

// One workgroup per output value: thread t sums partial rows t, t + 256, ...
// in order, then a fixed LDS tree adds the 256 thread sums, so the result
// does not depend on timing.
__global__ __launch_bounds__(256) void k_finalize(const double* __restrict__ partials, int nblocks, int nvals,
                                                  double* __restrict__ out) {
    __shared__ double red[256];
    const int v = blockIdx.x;
    double s = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += 256) s += partials[(size_t)b * nvals + v];
    red[threadIdx.x] = s;
    __syncthreads();
#pragma unroll
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[v] = red[0];
}

// <H0> = sum_b Re tr(h_b rho_b) from the finalized bond sums (Sec. IV,
// Eq. (10)), in FP64 on the device: thread b expands rho_b from its 16 reals
// and contracts it with h_b (FP64, row-major complex); thread 0 adds the bond
// terms in bond order.  out[0] = <H0>, out[1] = <psi|psi>; rdm (optional)
// receives every rho_b as 4x4 complex.  One workgroup of 64 threads, L <= 65.
__global__ __launch_bounds__(64) void k_energy_contract(const double* __restrict__ red, const double* __restrict__ h64,
                                                        int L, double* __restrict__ out, double* __restrict__ rdm) {
    __shared__ double trs[64];
    const int b = threadIdx.x;
    if (b < L - 1) {
        const double* v = red + (size_t)b * 16;
        double rr[16], ri[16];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            rr[5 * i] = v[i];
            ri[5 * i] = 0.0;
        }
        int k = 4;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = i + 1; j < 4; ++j) {
                rr[4 * i + j] = v[k];
                ri[4 * i + j] = v[k + 1];
                rr[4 * j + i] = v[k];
                ri[4 * j + i] = -v[k + 1];
                k += 2;
            }
        const double* hb = h64 + (size_t)b * 32;
        double tr = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) tr += hb[2 * (4 * i + j)] * rr[4 * j + i] - hb[2 * (4 * i + j) + 1] * ri[4 * j + i];
        trs[b] = tr;
        if (rdm) {
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                rdm[(size_t)b * 32 + 2 * q] = rr[q];
                rdm[(size_t)b * 32 + 2 * q + 1] = ri[q];
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double E = 0.0;
        for (int q = 0; q < L - 1; ++q) E += trs[q];
        out[0] = E;
        out[1] = red[(size_t)(L - 1) * 16];
    }
}

// ---------------------------------------------------------------------------
// lambda = H0 psi, out of place (the Hamiltonian application of Sec. V)
// ---------------------------------------------------------------------------
// One cover pass per launch; the first pass writes lambda, later passes add.
// Bond by bond, with all 16 entries of each term as given: chains of one tile,
// and longer ones whose terms are not Hermitian to rounding.

template <typename T, int KMAX>
__global__ __launch_bounds__(FL_NT) void k_apply_h(const typename CT<T>::c* __restrict__ psi,
                                                   typename CT<T>::c* __restrict__ lam, const T* __restrict__ hmat,
                                                   int C, int W, fl_pass pd, int first) {
    typedef typename CT<T>::c cplx;
    __shared__ cplx lp[1 << KMAX];
    __shared__ cplx ll[1 << KMAX];
    const int K = C + W;
    const int h = pd.h;
    const uint64_t base = fl_tile_base(blockIdx.x, C, W, h);
    tile_load<T, 0>(psi, base, K, C, h, lp);
    if (first) {
        for (uint32_t j = threadIdx.x; j < (1u << K); j += FL_NT) {
            cplx z;
            z.x = 0;
            z.y = 0;
            ll[j] = z;
        }
    } else {
        tile_load<T, 0>(lam, base, K, C, h, ll);
    }
    __syncthreads();
    const uint32_t ngrp = 1u << (K - 2);
    for (int g = 0; g < pd.ngroups; ++g) {
        const int u = pd.u0[g];
        const T* H = hmat + 32 * pd.ops[g][0];
        for (uint32_t o = threadIdx.x; o < ngrp; o += FL_NT) {
            const uint32_t b0 = fl_spread(o, u, 2);
            T ar[4], ai[4];
#pragma unroll
            for (int l = 0; l < 4; ++l) {
                const cplx a = lp[fl_swz(b0 | ((uint32_t)l << u))];
                ar[l] = a.x;
                ai[l] = a.y;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t idx = fl_swz(b0 | ((uint32_t)i << u));
                cplx acc = ll[idx];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const T hr = H[8 * i + 2 * j], hi = H[8 * i + 2 * j + 1];
                    acc.x = fma(hr, ar[j], fma(-hi, ai[j], acc.x));
                    acc.y = fma(hr, ai[j], fma(hi, ar[j], acc.y));
                }
                ll[idx] = acc;
            }
        }
        __syncthreads();
    }
    tile_store<T, 0>(lam, base, K, C, h, ll);
}

// Full tiles (W > 0), Hermitian terms.  The bonds of a pass come packed into windows of 4
// consecutive tile bits (up to 3 bonds each), and every thread applies a
// window's summed Hamiltonian to 2^4 amplitudes at once.  A row of that sum
// has one real diagonal entry, one entry per flipped bit (the bonds on both
// sides of the bit share it) and one per flipped neighbour pair, so three
// bonds cost 30 FMA an amplitude instead of 48; by Hermiticity 52 reals hold
// them all (layout: apply_h_window), read as scalars.
//
// psi sits in LDS for the whole tile; lambda changes layout between windows
// through a second LDS tile (a thread reads the 16 elements it owns in this
// window and writes the same ones: one barrier per window).  The last window
// adds the lambda of earlier passes, loaded straight from HBM in that window's
// layout, and stores the result the same way.  The two tiles leave room for
// one workgroup per CU, so the kernel is bound by how well one workgroup hides
// its HBM phases: persistent workgroups fetch the next tile's psi and lambda
// into registers before the windows of the current one.
//
// DOT: the last pass also sums <psi|lambda>, <lambda|lambda> and <psi|psi>
// (FP64, of the stored values) into dots[block][4].
//
// complex64, L = 25 (3 passes, 256 MiB state), H0 psi and its sums: 0.57 ms,
// 180 - 206 us a pass (the adding passes move 0.8 GB: 4.5 TB/s).  One bond at
// a time with a read-modify-write of lambda and a barrier per bond took 513 us
// a pass, and the sums another 90 us pass over both states: 1.63 ms.
// lambda += H_w psi on the 16 amplitudes of a window; bit k of m is window bit
// k.  w: [0..15] diagonal entries of row m; then the single flips of bit k
// (rows with bit k clear; the set ones take the conjugate), as (re, im) for
// (bit k-1, bit k+1) = 00, 10, 01, 11 where those bits are in the window
// (k = 0 and k = 3 have one neighbour, hence two entries); then the flips
// 00 -> 11 (entry h_03) and 01 -> 10 (h_12) of each bond.
template <typename T>
__device__ __forceinline__ void apply_h_window(const T (&pr)[16], const T (&pi)[16], T (&lr)[16], T (&li)[16],
                                               const T* __restrict__ w) {
    auto pair_term = [&](int x, int y, T re, T im) {
        lr[x] = fma(re, pr[y], lr[x]);
        lr[x] = fma(-im, pi[y], lr[x]);
        li[x] = fma(re, pi[y], li[x]);
        li[x] = fma(im, pr[y], li[x]);
        lr[y] = fma(re, pr[x], lr[y]);
        lr[y] = fma(im, pi[x], lr[y]);
        li[y] = fma(re, pi[x], li[y]);
        li[y] = fma(-im, pr[x], li[y]);
    };
#pragma unroll
    for (int m = 0; m < 16; ++m) {
        lr[m] = fma(w[m], pr[m], lr[m]);
        li[m] = fma(w[m], pi[m], li[m]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int off = k == 0 ? 16 : k == 1 ? 20 : k == 2 ? 28 : 36;
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            if ((m >> k) & 1) continue;
            const int lo = k > 0 ? (m >> (k - 1)) & 1 : 0, hi = k < 3 ? (m >> (k + 1)) & 1 : 0;
            const int e = off + 2 * (k == 0 ? hi : lo + 2 * hi);
            pair_term(m, m | (1 << k), w[e], w[e + 1]);
        }
    }
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int m = 0; m < 16; ++m) {
            if ((m >> (j + 1)) & 1) continue;
            const int e = 40 + 4 * j + (((m >> j) & 1) ? 2 : 0);   // rows 00 and 01 of the bond (row 01 flips to 10)
            pair_term(m, m ^ (3 << j), w[e], w[e + 1]);
        }
}

template <typename T, int KT, int NT, int CL, bool DOT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT / 256))) void k_apply_h_tiles(
    const typename CT<T>::c* __restrict__ psi, typename CT<T>::c* __restrict__ lam, const T* __restrict__ tab, int W,
    uint32_t ntiles, apply_h_desc pd, double* __restrict__ dots) {
    typedef typename CT<T>::c cplx;
    constexpr int R = 4, C = CL, K = KT;
    static_assert((1 << (K - R)) == NT, "one window of 16 amplitudes per thread");
    constexpr int APL = sizeof(T) == 4 ? 2 : 1;
    constexpr int ITER = (1 << K) / (APL * NT);
    typedef typename std::conditional<sizeof(T) == 4, fl_f32x4, fl_f64x2>::type v16;
    __shared__ __attribute__((aligned(16))) cplx lp[1 << K];
    __shared__ __attribute__((aligned(16))) cplx ll[1 << K];
    const int h = pd.h, nw = pd.nwin;
    static_assert((APL * NT) % (1 << C) == 0 && (APL * NT) % 256 == 0, "tile access stride");
    const uint64_t toff = fl_tile_offset(APL * threadIdx.x, C, h);
    const uint64_t tstride = (uint64_t)((APL * NT) >> C) << h;
    const uint32_t l0 = fl_swz(APL * threadIdx.x);
    // offsets of the last window's elements, relative to the tile base
    const int ul = pd.u0[nw - 1];
    const uint64_t ob = fl_tile_offset(fl_spread(threadIdx.x, ul, R), C, h);
    uint64_t od[R];
#pragma unroll
    for (int k = 0; k < R; ++k) od[k] = fl_tile_offset(1u << (ul + k), C, h);
    auto moff = [&](int m) {
        uint64_t r = 0;
#pragma unroll
        for (int k = 0; k < R; ++k)
            if ((m >> k) & 1) r += od[k];
        return r;
    };
    v16 np[ITER];       // psi of the next tile
    cplx nl[1 << R];    // lambda of the current tile, in the last window's layout
    auto fetch_psi = [&](uint32_t tile) {
        const cplx* src = psi + fl_tile_base(tile, C, W, h) + toff;
#pragma unroll
        for (int s = 0; s < ITER; ++s) np[s] = *reinterpret_cast<const v16*>(src + s * tstride);
    };
    double dE = 0.0, dL = 0.0, dN = 0.0;
    // complex128 has no registers left for the next tile's psi
    constexpr bool PREF = sizeof(T) == 4;
    if (PREF && blockIdx.x < ntiles) fetch_psi(blockIdx.x);
    for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        if (!PREF) fetch_psi(tile);
        cplx* const lbase = lam + fl_tile_base(tile, C, W, h) + ob;
        if (tile != blockIdx.x) __syncthreads();   // the previous tile's LDS reads are done
#pragma unroll
        for (int s = 0; s < ITER; ++s) {
            const uint32_t l = l0 + s * (APL * NT);
            if constexpr (sizeof(T) == 4) {
                lp[l] = make_float2(np[s][0], np[s][1]);
                lp[l ^ 1] = make_float2(np[s][2], np[s][3]);
            } else {
                lp[l] = make_double2(np[s][0], np[s][1]);
            }
        }
        __syncthreads();
        if (!pd.first) {
#pragma unroll
            for (int m = 0; m < (1 << R); ++m) nl[m] = lbase[moff(m)];
        }
        if (PREF && tile + gridDim.x < ntiles) fetch_psi(tile + gridDim.x);
        for (int g = 0; g < nw; ++g) {
            const int u0 = pd.u0[g];
            uint32_t la[1 << R];
            la[0] = fl_swz(fl_spread(threadIdx.x, u0, R)) * (uint32_t)sizeof(cplx);
#pragma unroll
            for (int m = 1; m < (1 << R); ++m)
                la[m] = la[m & (m - 1)] ^ (fl_swz(1u << (u0 + __builtin_ctz(m))) * (uint32_t)sizeof(cplx));
            char* const pb = reinterpret_cast<char*>(lp);
            char* const lb = reinterpret_cast<char*>(ll);
            T pr[16], pi[16], lr[16], li[16];
#pragma unroll
            for (int m = 0; m < 16; ++m) {
                const cplx a = *reinterpret_cast<const cplx*>(pb + la[m]);
                pr[m] = a.x;
                pi[m] = a.y;
                lr[m] = 0;
                li[m] = 0;
            }
            if (g > 0) {
#pragma unroll
                for (int m = 0; m < 16; ++m) {
                    const cplx a = *reinterpret_cast<const cplx*>(lb + la[m]);
                    lr[m] = a.x;
                    li[m] = a.y;
                }
            }
            apply_h_window<T>(pr, pi, lr, li, tab + FL_HWIN_REALS * g);
            if (g + 1 < nw) {
#pragma unroll
                for (int m = 0; m < 16; ++m) {
                    cplx a;
                    a.x = lr[m];
                    a.y = li[m];
                    *reinterpret_cast<cplx*>(lb + la[m]) = a;
                }
                __syncthreads();
            } else {
#pragma unroll
                for (int m = 0; m < 16; ++m) {
                    cplx a;
                    a.x = lr[m];
                    a.y = li[m];
                    if (!pd.first) {
                        a.x += nl[m].x;
                        a.y += nl[m].y;
                    }
                    lbase[moff(m)] = a;
                    if constexpr (DOT) {
                        const double xr = pr[m], xi = pi[m], yr = a.x, yi = a.y;
                        dE = fma(xr, yr, fma(xi, yi, dE));
                        dL = fma(yr, yr, fma(yi, yi, dL));
                        dN = fma(xr, xr, fma(xi, xi, dN));
                    }
                }
            }
        }
    }
    if constexpr (DOT) {
        double v[4] = {dE, 0.0, dN, dL};   // the order of k_overlap's sums
        const double r = wave_transpose_reduce<double, 4>(v);
        double* const wacc = reinterpret_cast<double*>(lp);
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        __syncthreads();
        if ((lane & 15) == 0) wacc[wave * 4 + (lane >> 4)] = r;
        __syncthreads();
        if (threadIdx.x < 4) {
            double s = 0.0;
            for (int k = 0; k < NT / 64; ++k) s += wacc[k * 4 + threadIdx.x];
            dots[(size_t)blockIdx.x * 4 + threadIdx.x] = s;
        }
    }
}

// ---------------------------------------------------------------------------
// reverse pass of the gradient: undo gates on psi and lambda together
// ---------------------------------------------------------------------------
// Every op with a slot first accumulates, for its bond b on register bits
// (i, i+1), the anti-Hermitian overlap
//   D_b[i][j] += sum_r conj(lambda_{r,i}) psi_{r,j} - conj(psi_{r,i}) lambda_{r,j}
// (the only part of M_b = sum_r conj(lambda_{r,i}) psi_{r,j} that an
// anti-Hermitian gate derivative A = (dG) G^dagger sees), then applies the
// gate (G_b^dagger) to both states.  16 reals per bond:
// [0..3] = Im(conj(lambda_i) psi_i) summed, then (re, im) of D_01, D_02,
// D_03, D_12, D_13, D_23.
// Mpart layout: [gridDim.x][nbonds][16] doubles, accumulated across launches.

template <typename T, int R, int I>
__device__ __forceinline__ void adj_overlap(const T (&pr)[1 << R], const T (&pi)[1 << R], const T (&lr)[1 << R],
                                            const T (&li)[1 << R], T (&d)[16]) {
#pragma unroll
    for (int c = 0; c < (1 << (R - 2)); ++c) {
        const int b = (c & ((1 << I) - 1)) | ((c >> I) << (I + 2));
        T ar[4], ai[4], br[4], bi[4];   // a = lambda, b = psi
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            ar[l] = lr[b | (l << I)];
            ai[l] = li[b | (l << I)];
            br[l] = pr[b | (l << I)];
            bi[l] = pi[b | (l << I)];
        }
#pragma unroll
        for (int l = 0; l < 4; ++l) d[l] = fma(ar[l], bi[l], fma(-ai[l], br[l], d[l]));
        int k = 4;
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int y = x + 1; y < 4; ++y) {
                T re = d[k], im = d[k + 1];
                re = fma(ar[x], br[y], re);
                re = fma(ai[x], bi[y], re);
                re = fma(-br[x], ar[y], re);
                re = fma(-bi[x], ai[y], re);
                im = fma(ar[x], bi[y], im);
                im = fma(-ai[x], br[y], im);
                im = fma(-br[x], ai[y], im);
                im = fma(bi[x], ar[y], im);
                d[k] = re;
                d[k + 1] = im;
                k += 2;
            }
    }
}

// One reverse op on a register group: the overlap terms of the op's slot
// (before the gate), summed over the wave into acc[16], then the gate (read
// from LDS at lgate) on both states.  Every op of a reverse plan has both a
// slot and a gate.  The overlap is reduced before the gate is read, which
// keeps the registers of the two apart.
template <typename T, int R, typename F>
__device__ __forceinline__ void adj_op(T (&pr)[1 << R], T (&pi)[1 << R], T (&lr)[1 << R], T (&li)[1 << R], int i,
                                       const T* lgate, double (&acc)[16], int lane, F&& next_op) {
    {
        T d[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) d[k] = 0;
        with_bit<R>(i, [&](auto I) {
            __asm__ volatile("; overlap on register bits %0" ::"i"(decltype(I)::value));
            adj_overlap<T, R, decltype(I)::value>(pr, pi, lr, li, d);
        });
        // lane l holds the sum of value l >> 2; one lane of each four adds it and
        // the other three add zero, as an LDS atomic with every lane active (no
        // divergent branch in the op loop)
        const T r = wave_transpose_reduce<T, 16>(d);
        __hip_atomic_fetch_add(&acc[lane >> 2], (lane & 3) == 0 ? (double)r : 0.0, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    T gv[32];
    load_gate_lds<T>(lgate, gv);
    next_op();   // the next op's descriptor, under this op's FMAs
    with_bit<R>(i, [&](auto I) {
        apply_pair_g<T, R, decltype(I)::value>(pr, pi, gv);
        apply_pair_g<T, R, decltype(I)::value>(lr, li, gv);
    });
}

// Sums a and b over the lanes l and l ^ 32: a's sum in the lower half of the
// wave, b's in the upper half.
template <typename T>
__device__ __forceinline__ T fold32(T a, T b) {
    if constexpr (sizeof(T) == 4) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    } else {
        const uint64_t x = (uint64_t)__double_as_longlong(a), y = (uint64_t)__double_as_longlong(b);
        const auto rl = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
        const auto rh = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
        return __longlong_as_double((long long)(((uint64_t)rh[0] << 32) | rl[0])) +
               __longlong_as_double((long long)(((uint64_t)rh[1] << 32) | rl[1]));
    }
}

// The reverse pass's quad chain: as quad_chain with two threads per quad, on
// both states, the overlap terms of the op's slot taken before its gate.  The
// thread with rot = 0 (lower half of the wave) and the one with rot = 2 (upper
// half) run the same instructions on the quad as they hold it, v_m = amplitude
// (m + rot) & 3: the terms of D_00, D_11, D_01, D_12 become those of D_22,
// D_33, D_23 and D_30 = -conj(D_03), and each has one half of D_02 and D_13
// (the other half with the amplitudes exchanged, real parts negated).  So the
// first of the wave sum's steps is done for 12 of the 16 values.  The quads'
// reads and the next gate's stand first, the wave sum after the write-back.
// meta: first bits, then slot << 8 | gate << 16.  A serial chain like the
// sweep's.  fl_grad over 50 periods, against one thread per quad with the gate
// read behind the sums (us): complex64 L = 12 657 / 812, 14 794 / 977, 17 1054 /
// 1280, 18 1228 / 1463; complex128 L = 14 882 / 1058, 18 1608 / 1694.
template <typename T>
__device__ __forceinline__ void adj_quad_chain(typename CT<T>::c* lp, typename CT<T>::c* ll, const T* lg,
                                               const uint32_t* meta, int nops, int total, double (*acc)[16],
                                               const fl_quad_lane<2>& me, bool active) {
    typedef typename CT<T>::c cplx;
    char* const pb = reinterpret_cast<char*>(lp);
    char* const lb = reinterpret_cast<char*>(ll);
    const int lane = threadIdx.x & 63;
    const T sg = me.rot ? T(-1) : T(1);
    // after the sum lane l holds value (l >> 2) & 7 of its half's list
    const int vi8 = (lane >> 2) & 7;
    const int at = me.rot ? (vi8 < 2 ? vi8 + 2 : vi8 < 4 ? vi8 + 12 : vi8 < 6 ? vi8 + 4 : vi8 + 6)
                          : (vi8 < 2 ? vi8 : vi8 < 4 ? vi8 + 2 : vi8 < 6 ? vi8 + 6 : vi8);
    const bool adds = (lane & 3) == 0;
    auto uni = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane(x); };
    if (nops == 0) return;
    T ga[16], gb[16];
    uint32_t u = uni(meta[0]), w = uni(meta[nops]), la[4];
    load_gate_rows<T, 2>(me, lg + 32 * (w >> 16), ga);
    quad_addr<T, 2>(me, u, la);
    auto after = [&](int k) { return k + 1 < nops ? k + 1 : 0; };
    int kn = after(0);
    uint32_t un = uni(meta[kn]), wn = uni(meta[nops + kn]);
    auto step = [&](const T (&g)[16], T (&gn)[16]) {
        T pr[4], pi[4], lr[4], li[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            pr[m] = pi[m] = lr[m] = li[m] = 0;   // an idle thread has no part in the sums
            if (active) {
                const cplx a = *reinterpret_cast<const cplx*>(pb + la[m]), b = *reinterpret_cast<const cplx*>(lb + la[m]);
                pr[m] = a.x;
                pi[m] = a.y;
                lr[m] = b.x;
                li[m] = b.y;
            }
        }
        __builtin_amdgcn_sched_barrier(0);   // the quads' reads lead the LDS queue
        uint32_t ln[4];
        quad_addr<T, 2>(me, un, ln);
        load_gate_rows<T, 2>(me, lg + 32 * (wn >> 16), gn);
        kn = after(kn);
        const uint32_t u2 = meta[kn], w2 = meta[nops + kn];
#pragma unroll
        for (int m = 0; m < 4; ++m) __asm__ volatile("" : "+v"(ln[m]));
        __builtin_amdgcn_sched_barrier(0);
        // first halves of conj(lambda_x) psi_y - conj(psi_x) lambda_y, then the second
        auto half = [&](int x, int y, T& re, T& im) {
            re = fma(lr[x], pr[y], li[x] * pi[y]);
            im = fma(lr[x], pi[y], -li[x] * pr[y]);
        };
        auto whole = [&](int x, int y, T& re, T& im) {
            half(x, y, re, im);
            re = fma(-pr[x], lr[y], re);
            re = fma(-pi[x], li[y], re);
            im = fma(-pr[x], li[y], im);
            im = fma(pi[x], lr[y], im);
        };
        T v[8], r02, i02, r13, i13;
        v[0] = fma(lr[0], pi[0], -li[0] * pr[0]);
        v[1] = fma(lr[1], pi[1], -li[1] * pr[1]);
        whole(0, 1, v[2], v[3]);
        whole(1, 2, v[4], v[5]);
        half(0, 2, r02, i02);
        half(1, 3, r13, i13);
        v[4] *= sg;
        apply_rows<T, 2>(pr, pi, g);
        apply_rows<T, 2>(lr, li, g);
        if (active) {
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                cplx a, b;
                a.x = pr[m];
                a.y = pi[m];
                b.x = lr[m];
                b.y = li[m];
                *reinterpret_cast<cplx*>(pb + la[m]) = a;
                *reinterpret_cast<cplx*>(lb + la[m]) = b;
            }
        }
        v[6] = fold32<T>(r02 * sg, r13 * sg);
        v[7] = fold32<T>(i02, i13);
        T r;
        if constexpr (sizeof(T) == 4) tr_steps_f32<8, 16>(v, lane);
        else tr_steps_f64<8, 16>(v, lane);
        r = v[0];
        __hip_atomic_fetch_add(&acc[(w >> 8) & 255][at], adds ? (double)r : 0.0, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
        for (int m = 0; m < 4; ++m) la[m] = ln[m];
        w = wn;
        un = uni(u2);
        wn = uni(w2);
        __syncthreads();
    };
    for (int q = 0; q < total; q += 2) {
        step(ga, gb);
        if (q + 1 < total) step(gb, ga);
    }
}

// The workgroup's sums of every slot, added to its row of Mpart.
template <int NT>
__device__ __forceinline__ void adj_flush(const double (*wacc)[FL_MAX_SLOTS][16], const fl_adj_words& pd, double* row) {
    for (int t = threadIdx.x; t < pd.nslots * 16; t += NT) {
        const int sl = t >> 4, v = t & 15;
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) s += wacc[w][sl][v];
        row[(size_t)pd.sbond[sl] * 16 + v] += s;
    }
}

// Chains of at most FL_KMAX_ONE sites: one workgroup, as k_sweep_one.
template <typename T, int NT>
__global__ __launch_bounds__(NT) void k_adjoint_one(typename CT<T>::c* __restrict__ psi,
                                                    typename CT<T>::c* __restrict__ lam, const T* __restrict__ gates,
                                                    int L, fl_adj_words pd, int reps, double* __restrict__ Mpart) {
    typedef typename CT<T>::c cplx;
    constexpr int NW = NT / 64;
    __shared__ __attribute__((aligned(16))) cplx lp[1 << FL_KMAX_ONE];
    __shared__ __attribute__((aligned(16))) cplx ll[1 << FL_KMAX_ONE];
    __shared__ __attribute__((aligned(16))) T lg[FL_KMAX_ONE * 32];
    __shared__ double wacc[NW][FL_MAX_SLOTS][16];
    __shared__ uint32_t meta[FL_SWEEP_WORDS];
    for (uint32_t j = threadIdx.x; j < (1u << L); j += NT) {
        lp[fl_swz(j)] = psi[j];
        ll[fl_swz(j)] = lam[j];
    }
    for (int t = threadIdx.x; t < (L - 1) * 32; t += NT) lg[t] = gates[t];
    for (int t = threadIdx.x; t < pd.nwords; t += NT) meta[t] = pd.w[t];
    for (int t = threadIdx.x; t < NW * FL_MAX_SLOTS * 16; t += NT) (&wacc[0][0][0])[t] = 0.0;
    __syncthreads();
    const fl_quad_lane<2> me;
    adj_quad_chain<T>(lp, ll, lg, meta, pd.ngroups, pd.ngroups * reps, wacc[threadIdx.x >> 6], me,
                      me.quad < (1u << (L - 2)));
    for (uint32_t j = threadIdx.x; j < (1u << L); j += NT) {
        psi[j] = lp[fl_swz(j)];
        lam[j] = ll[fl_swz(j)];
    }
    adj_flush<NT>(wacc, pd, Mpart);
}

// Tiles of 2^KT amplitudes (KT <= 11) of both states, one per workgroup, as
// k_sweep_quads.
template <typename T, int KT, int CL>
__global__ __launch_bounds__(2 << (KT - 2)) void k_adjoint_quads(typename CT<T>::c* __restrict__ psi,
                                                                typename CT<T>::c* __restrict__ lam,
                                                                const T* __restrict__ gates, int W, fl_adj_words pd,
                                                                double* __restrict__ Mpart, int nbonds) {
    typedef typename CT<T>::c cplx;
    constexpr int K = KT, C = CL, NT = 2 << (K - 2), NW = NT / 64;
    constexpr int APL = sizeof(T) == 4 ? 2 : 1;   // amplitudes per 16 bytes
    constexpr int ITER = (1 << K) / (APL * NT);
    static_assert(ITER >= 1, "a whole access per thread");
    static_assert((APL * NT) % (1 << C) == 0, "tile access stride");
    typedef typename std::conditional<sizeof(T) == 4, fl_f32x4, fl_f64x2>::type v16;
    __shared__ __attribute__((aligned(16))) cplx lp[1 << K];
    __shared__ __attribute__((aligned(16))) cplx ll[1 << K];
    __shared__ __attribute__((aligned(16))) T lg[FL_MAX_GATE_TABLE * 32];
    __shared__ double wacc[NW][FL_MAX_SLOTS][16];
    __shared__ uint32_t meta[FL_SWEEP_WORDS];
    const uint64_t at = fl_tile_base(blockIdx.x, C, W, pd.h) + fl_tile_offset(APL * threadIdx.x, C, pd.h);
    const uint64_t tstride = (uint64_t)((APL * NT) >> C) << pd.h;
    const uint32_t l0 = fl_swz(APL * threadIdx.x);
    v16 a[ITER], b[ITER];
#pragma unroll
    for (int s = 0; s < ITER; ++s) {
        a[s] = *reinterpret_cast<const v16*>(psi + at + s * tstride);
        b[s] = *reinterpret_cast<const v16*>(lam + at + s * tstride);
    }
    const fl_f32x4* gsrc = reinterpret_cast<const fl_f32x4*>(gates);
    for (int t = threadIdx.x; t < nbonds * (int)(32 * sizeof(T) / 16); t += NT) reinterpret_cast<fl_f32x4*>(lg)[t] = gsrc[t];
    for (int t = threadIdx.x; t < pd.nwords; t += NT) meta[t] = pd.w[t];
    for (int t = threadIdx.x; t < NW * FL_MAX_SLOTS * 16; t += NT) (&wacc[0][0][0])[t] = 0.0;
#pragma unroll
    for (int s = 0; s < ITER; ++s) {
        const uint32_t l = l0 ^ fl_swz((uint32_t)(s * APL * NT));
        if constexpr (sizeof(T) == 4) {
            lp[l] = make_float2(a[s][0], a[s][1]);
            lp[l ^ 1] = make_float2(a[s][2], a[s][3]);
            ll[l] = make_float2(b[s][0], b[s][1]);
            ll[l ^ 1] = make_float2(b[s][2], b[s][3]);
        } else {
            lp[l] = make_double2(a[s][0], a[s][1]);
            ll[l] = make_double2(b[s][0], b[s][1]);
        }
    }
    __syncthreads();
    adj_quad_chain<T>(lp, ll, lg, meta, pd.ngroups, pd.ngroups, wacc[threadIdx.x >> 6], fl_quad_lane<2>(), true);
#pragma unroll
    for (int s = 0; s < ITER; ++s) {
        const uint32_t l = l0 ^ fl_swz((uint32_t)(s * APL * NT));
        v16 x, y;
        if constexpr (sizeof(T) == 4) {
            const float2 p0 = lp[l], p1 = lp[l ^ 1], q0 = ll[l], q1 = ll[l ^ 1];
            x = v16{p0.x, p0.y, p1.x, p1.y};
            y = v16{q0.x, q0.y, q1.x, q1.y};
        } else {
            const double2 p0 = lp[l], q0 = ll[l];
            x = v16{p0.x, p0.y};
            y = v16{q0.x, q0.y};
        }
        *reinterpret_cast<v16*>(psi + at + s * tstride) = x;
        *reinterpret_cast<v16*>(lam + at + s * tstride) = y;
    }
    adj_flush<NT>(wacc, pd, Mpart + (size_t)blockIdx.x * nbonds * 16);
}

// Tiles of both states, persistent workgroups (the sums stay in LDS from tile
// to tile).  Descriptors as in k_sweep_tiles.  The gates come from the
// workgroup's LDS copy of G^dagger into vector registers, so that the FMAs of
// two waves can issue together (two waves per SIMD on 12-bit tiles: two
// workgroups' tiles fill the LDS).  Bound by the vector ALUs: 736 FMA-type
// instructions per op and 16 amplitudes, and about 100 of the wave sums, which
// do not pair.  complex64 L = 24, 50 periods: 26.1 ms (28.5 with the gates in
// scalar registers); c128 L = 22: 13.7 ms (14.1).
template <typename T, int R, int KT, int NT, int CL, int WPE, typename D>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WPE))) void k_adjoint_tiles(
    typename CT<T>::c* __restrict__ psi, typename CT<T>::c* __restrict__ lam, const T* __restrict__ gates, int W,
    uint32_t ntiles, D pd, double* __restrict__ Mpart, int nbonds) {
    typedef typename CT<T>::c cplx;
    constexpr bool LM = std::is_same<D, fl_adj_words>::value;
    constexpr int C = CL, K = KT, NW = NT / 64;
    static_assert((1 << (K - R)) == NT, "one register group per thread");
    constexpr int APL = sizeof(T) == 4 ? 2 : 1;
    constexpr int ITER = (1 << K) / (APL * NT);
    typedef typename std::conditional<sizeof(T) == 4, fl_f32x4, fl_f64x2>::type v16;
    __shared__ __attribute__((aligned(16))) cplx lp[1 << K];
    __shared__ __attribute__((aligned(16))) cplx ll[1 << K];
    __shared__ __attribute__((aligned(16))) T lg[FL_MAX_GATE_TABLE * 32];
    __shared__ double wacc[NW][FL_MAX_SLOTS][16];
    __shared__ uint32_t meta[LM ? FL_SWEEP_WORDS : 1];
    const int h = pd.h, ng = pd.ngroups;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    char* const pb = reinterpret_cast<char*>(lp);
    char* const lb = reinterpret_cast<char*>(ll);
    static_assert((APL * NT) % (1 << C) == 0, "tile access stride");
    // full-size tiles stream through; the states of short chains stay in cache
    auto load = [](const cplx* p) {
        const v16* q = reinterpret_cast<const v16*>(p);
        return LM ? *q : __builtin_nontemporal_load(q);
    };
    auto store = [](const v16& x, cplx* p) {
        v16* q = reinterpret_cast<v16*>(p);
        if (LM) *q = x;
        else __builtin_nontemporal_store(x, q);
    };
    for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        // opaque per tile: addresses are formed anew, not kept across the ops
        uint32_t tid = threadIdx.x;
        __asm__ volatile("" : "+v"(tid));
        const uint64_t base = fl_tile_base(tile, C, W, h);
        const uint64_t toff = fl_tile_offset(APL * tid, C, h);
        const uint64_t tstride = (uint64_t)((APL * NT) >> C) << h;
        const uint32_t l0 = fl_swz(APL * tid);
        {
            const cplx* sp = psi + base + toff;
            const cplx* sl = lam + base + toff;
            v16 a[ITER], b[ITER];
#pragma unroll
            for (int s = 0; s < ITER; ++s) a[s] = load(sp + s * tstride);
#pragma unroll
            for (int s = 0; s < ITER; ++s) b[s] = load(sl + s * tstride);
            if (tile == blockIdx.x) {
                const fl_f32x4* src = reinterpret_cast<const fl_f32x4*>(gates);
                for (int t = threadIdx.x; t < nbonds * (int)(32 * sizeof(T) / 16); t += NT)
                    reinterpret_cast<fl_f32x4*>(lg)[t] = src[t];
                if constexpr (LM)
                    for (int t = threadIdx.x; t < pd.nwords; t += NT) meta[t] = pd.w[t];
                for (int t = threadIdx.x; t < NW * FL_MAX_SLOTS * 16; t += NT) (&wacc[0][0][0])[t] = 0.0;
            } else {
                __syncthreads();   // the previous tile's stores have read LDS
            }
#pragma unroll
            for (int s = 0; s < ITER; ++s) {
                const uint32_t l = l0 ^ fl_swz((uint32_t)(s * APL * NT));
                if constexpr (sizeof(T) == 4) {
                    lp[l] = make_float2(a[s][0], a[s][1]);
                    lp[l ^ 1] = make_float2(a[s][2], a[s][3]);
                    ll[l] = make_float2(b[s][0], b[s][1]);
                    ll[l ^ 1] = make_float2(b[s][2], b[s][3]);
                } else {
                    lp[l] = make_double2(a[s][0], a[s][1]);
                    ll[l] = make_double2(b[s][0], b[s][1]);
                }
            }
        }
        __syncthreads();
        int pos = ng;
        for (int g = 0; g < ng; ++g) {
            int u0, nops;
            if constexpr (LM) {
                const uint32_t head = __builtin_amdgcn_readfirstlane(meta[g]);
                u0 = head & 255;
                nops = head >> 8;
            } else {
                u0 = pass_u0(pd, g);
                nops = pass_nops(pd, g);
            }
            uint32_t bk[R];
#pragma unroll
            for (int k = 0; k < R; ++k) bk[k] = fl_swz(1u << (u0 + k)) * (uint32_t)sizeof(cplx);
            const uint32_t vb = fl_swz(fl_spread(tid, u0, R)) * (uint32_t)sizeof(cplx);
            auto loff = [&](int m) {
                uint32_t r = vb;
#pragma unroll
                for (int k = 0; k < R; ++k)
                    if ((m >> k) & 1) r ^= bk[k];
                return r;
            };
            T pr[1 << R], pi[1 << R], lr[1 << R], li[1 << R];
#pragma unroll
            for (int m = 0; m < (1 << R); ++m) {
                const uint32_t o = loff(m);
                const cplx a = *reinterpret_cast<const cplx*>(pb + o), b = *reinterpret_cast<const cplx*>(lb + o);
                pr[m] = a.x;
                pi[m] = a.y;
                lr[m] = b.x;
                li[m] = b.y;
            }
            // op metadata one op ahead, as in the sweep
            int bit, slot, idx;
            auto fetch = [&](int q) {
                if constexpr (LM) {
                    const uint32_t w = __builtin_amdgcn_readfirstlane(meta[pos + q]);
                    bit = w & 255;
                    slot = (w >> 8) & 255;
                    idx = w >> 16;
                } else {
                    bit = pass_bit(pd, g, q);
                    slot = pass_slot(pd, g, q);
                    idx = pass_gate(pd, g, q) - nbonds;
                }
            };
            fetch(0);
            auto run = [&](int q) {
                adj_op<T, R>(pr, pi, lr, li, bit, lg + 32 * idx, wacc[wave][slot], lane,
                             [&] { fetch(q + 1 < nops ? q + 1 : q); });
            };
            for (int q = 0; q < nops; q += 2) {
                run(q);
                if (q + 1 < nops) run(q + 1);
            }
            pos += nops;
#pragma unroll
            for (int m = 0; m < (1 << R); ++m) {
                const uint32_t o = loff(m);
                cplx a, b;
                a.x = pr[m];
                a.y = pi[m];
                b.x = lr[m];
                b.y = li[m];
                *reinterpret_cast<cplx*>(pb + o) = a;
                *reinterpret_cast<cplx*>(lb + o) = b;
            }
            __syncthreads();
        }
        {
            cplx* dp = psi + base + toff;
            cplx* dl = lam + base + toff;
#pragma unroll
            for (int s = 0; s < ITER; ++s) {
                const uint32_t l = l0 ^ fl_swz((uint32_t)(s * APL * NT));
                v16 a, b;
                if constexpr (sizeof(T) == 4) {
                    const float2 a0 = lp[l], a1 = lp[l ^ 1], b0 = ll[l], b1 = ll[l ^ 1];
                    a = v16{a0.x, a0.y, a1.x, a1.y};
                    b = v16{b0.x, b0.y, b1.x, b1.y};
                } else {
                    const double2 a0 = lp[l], b0 = ll[l];
                    a = v16{a0.x, a0.y};
                    b = v16{b0.x, b0.y};
                }
                store(a, dp + s * tstride);
                store(b, dl + s * tstride);
            }
        }
    }
    __syncthreads();
    const int nslots = pd.nslots;
    for (int t = threadIdx.x; t < nslots * 16; t += NT) {
        const int sl = t >> 4, v = t & 15;
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += wacc[w][sl][v];
        double* dst = Mpart + ((size_t)blockIdx.x * nbonds + pd.sbond[sl]) * 16 + v;
        *dst += s;
    }
}

// The reverse pass of the gradient for the 4-qubit-window form (complex64,
// full 13-bit tiles), on the matrix cores.  The forward pass of that form
// applies, per register group (a 4-bit window whose ops q = 0 .. n-1 apply
// G_q inside the window), the FP32 real form of U = G_{n-1} ... G_0.  This
// kernel replays the same passes backwards, groups in reverse order, with the
// transposes of those FP32 matrices, i.e. the exact adjoints U^dagger of what
// the forward applied, so psi retraces the forward's states up to arithmetic
// rounding (as the plain form's replay with the adjoints of its FP32 gates
// does) and a reset from a checkpoint does not jump.  Per group:
//  - the window overlap Q[x][y] = sum_r psi_{r,x} conj(lambda_{r,y}) of the
//    state after the forward group, as the real 32 x 32 product
//    D[2x + a][2y + b] = sum_c psi_{x,a}(c) lambda_{y,b}(c) over the wave's
//    64 columns c (a, b = re, im) on v_mfma_f32_32x32x2f32: lane l supplies
//    row i = l % 32 of psi and column j = l % 32 of lambda at column k = l / 32
//    of the step, the same LDS position in both tiles.  Then
//    Re Q = D[2x][2y] + D[2x+1][2y+1] and Im Q = D[2x+1][2y] - D[2x][2y+1],
//    formed between neighbouring lanes and summed over the workgroup's tiles
//    in LDS (FP32, one 2 KiB row per group of the pass).  Every forward op's
//    bond overlap follows from Q: with the reverse ops r = 0 .. n-1 applying
//    G_{n-1-r}^dagger, the state before reverse op r is P_r Q P_r^dagger
//    (P_r the product of the reverse ops before it), traced over the two
//    window bits off the bond; the host forms these terms in FP64;
//  - U^dagger on psi and on lambda as in k_dense4 (mats: 4 KiB of A fragments
//    per group of the reverse pass, B = a 32-column block of the state).
// Wave w owns columns 64 w .. 64 w + 63 of the group (column = the tile bits
// off the window, in order) for both parts, so a barrier is needed only where
// the next group assigns the tile's elements to the waves differently.  The
// tiles use the slots of fl_swz12, under which the Q reads (lanes along the
// window's amplitudes) and the column reads meet at most two distinct
// addresses per bank.  At the end Qpart[blockIdx][g][0..255] = Re Q[x][y] at
// 16 x + y, [256..511] = Im Q (FP64 copies of the FP32 sums).
__global__ __launch_bounds__(FL_WIN4_NT) __attribute__((amdgpu_waves_per_eu(2))) void k_adjoint_win4(
    float2* __restrict__ psi, float2* __restrict__ lam, const float4* __restrict__ mats, int W, uint32_t ntiles,
    fl_pass pd, double* __restrict__ Qpart) {
    constexpr int K = FL_KMAX_C64;
    constexpr int C = FL_DENSE4_LOWBITS;
    constexpr int NT = FL_WIN4_NT;
    constexpr int NW = NT / 64;
    constexpr int KC = K - 4;                   // column bits of a group
    constexpr int NB = (1 << KC) / (32 * NW);   // 32-column blocks per wave
    constexpr int WB = __builtin_ctz(NW);       // column bits that name the wave
    constexpr int NG = FL_WIN4_MAX_GROUPS;
    constexpr int IT = (1 << (K - 1)) / NT;     // 16-byte tile accesses per thread and state
    static_assert(NB == 2 && (1 << KC) == 64 * NW, "a wave owns 64 columns");
    __shared__ __attribute__((aligned(16))) float2 lp[1 << K];
    __shared__ __attribute__((aligned(16))) float2 ll[1 << K];
    __shared__ float qacc[NG][512];
    const int h = pd.h;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int lc = lane & 31, lk = lane >> 5;
    for (int t = threadIdx.x; t < NG * 512; t += NT) (&qacc[0][0])[t] = 0.f;
    char* const pb = reinterpret_cast<char*>(lp);
    char* const lb = reinterpret_cast<char*>(ll);
    auto load_a = [&](int g, float (&dst)[16]) {
        const float4* M = mats + (size_t)g * 256 + (size_t)lane * 4;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 t = M[q];
            dst[4 * q] = t.x;
            dst[4 * q + 1] = t.y;
            dst[4 * q + 2] = t.z;
            dst[4 * q + 3] = t.w;
        }
    };
    // tile element pairs (2 (tid + s NT), + 1) of both states, through
    // registers, so that the next tile's psi loads run under the current
    // tile's last group
    float4 tp[IT], tl[IT];
    auto fetch = [&](uint32_t tile, const float2* __restrict__ src, float4 (&dst)[IT]) {
        const uint64_t base = fl_tile_base(tile, C, W, h);
#pragma unroll
        for (int s = 0; s < IT; ++s)
            dst[s] = *reinterpret_cast<const float4*>(src + base + fl_tile_offset(2u * (threadIdx.x + s * NT), C, h));
    };
    auto put = [&]() {
#pragma unroll
        for (int s = 0; s < IT; ++s) {
            const uint32_t j = 2u * (threadIdx.x + s * NT);
            lp[fl_swz12(j)] = make_float2(tp[s].x, tp[s].y);
            lp[fl_swz12(j + 1)] = make_float2(tp[s].z, tp[s].w);
            ll[fl_swz12(j)] = make_float2(tl[s].x, tl[s].y);
            ll[fl_swz12(j + 1)] = make_float2(tl[s].z, tl[s].w);
        }
    };
    // the wave's columns are 64 w + (0 .. 63); which tile bits name the wave
    // depends only on how many of column bits KC - WB .. KC - 1 lie below u0
    auto part = [](int u) { return u <= KC - WB ? 0 : u - (KC - WB); };
    const float qsgn = (lc & 1) ? -1.0f : 1.0f;
    if (blockIdx.x < ntiles) {
        fetch(blockIdx.x, psi, tp);
        fetch(blockIdx.x, lam, tl);
        put();
    }
    for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const uint32_t next = tile + gridDim.x;
        bool fetched = false;
        __syncthreads();
        float a[16], an[16];
        if (pd.ngroups > 0) load_a(0, a);
        for (int g = 0; g < pd.ngroups; ++g) {
            const int u0 = pass_u0(pd, g);
            load_a(g + 1 < pd.ngroups ? g + 1 : g, an);
            // (1) window overlap.  Step s takes columns 64 w + 2 s + k;
            // element spread(64 w + lk) | (lc >> 1) << u0 | spread(2 s)
            // (disjoint bits), component lc & 1: a per-lane byte offset XOR a
            // uniform one.
            const uint32_t ql = (fl_swz12(fl_spread((uint32_t)(64 * w + lk), u0, 4) | ((uint32_t)(lc >> 1) << u0)) * 8u) |
                                (4u * (uint32_t)(lc & 1));
            auto read_q = [&](int h0, float (&qx)[16], float (&qy)[16]) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int st = h0 + i;
                    const uint32_t o =
                        ql ^ __builtin_amdgcn_readfirstlane(fl_swz12(fl_spread((uint32_t)(2 * st), u0, 4)) * 8u);
                    qx[i] = *reinterpret_cast<const float*>(pb + o);
                    qy[i] = *reinterpret_cast<const float*>(lb + o);
                }
            };
            // (2) B operands of U^dagger on psi: amplitude 2t + lk of the
            // lane's column in block cb
            uint32_t vb[NB];
#pragma unroll
            for (int cb = 0; cb < NB; ++cb) vb[cb] = fl_swz12(fl_spread((uint32_t)(64 * w + 32 * cb + lc), u0, 4)) * 8u;
            const uint32_t lkoff = fl_swz12((uint32_t)lk << u0) * 8u;
            auto read_b = [&](const char* sb, float (&bq)[16][NB]) {
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const uint32_t ss = fl_swz12((uint32_t)(2 * t) << u0) * 8u;
#pragma unroll
                    for (int cb = 0; cb < NB; ++cb) {
                        const float2 x = *reinterpret_cast<const float2*>(sb + ((vb[cb] ^ lkoff) ^ ss));
                        bq[t][cb] = x.x;
                        bq[t + 8][cb] = x.y;
                    }
                }
            };
            auto mfma_u = [&](const float (&bq)[16][NB], fl_f32x16 (&acc)[NB]) {
#pragma unroll
                for (int cb = 0; cb < NB; ++cb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[cb][r] = 0.0f;
#pragma unroll
                for (int st = 0; st < 16; ++st)
#pragma unroll
                    for (int cb = 0; cb < NB; ++cb)
                        acc[cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[st], bq[st][cb], acc[cb], 0, 0, 0);
            };
            // register r of block cb holds row 8 (r / 4) + 4 lk + r % 4 = 2 m + c
            auto write_u = [&](char* sb, const fl_f32x16 (&acc)[NB]) {
#pragma unroll
                for (int cb = 0; cb < NB; ++cb)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            const uint32_t m = 4 * q + 2 * lk + p;
                            float2 v;
                            v.x = acc[cb][4 * q + 2 * p];
                            v.y = acc[cb][4 * q + 2 * p + 1];
                            *reinterpret_cast<float2*>(sb + (vb[cb] ^ (fl_swz12(m << u0) * 8u))) = v;
                        }
            };
            // The phases in order, each one's LDS traffic placed between the
            // previous one's MFMAs (the scheduler pins 2 MFMAs : 1 LDS access):
            // Q reads A | Q MFMAs A + Q reads B | Q MFMAs B + psi reads |
            // Q sums | psi MFMAs + lambda reads | lambda MFMAs + psi writes |
            // lambda writes.  Each wave touches only its own columns, and its
            // LDS accesses run in program order.
            float bp[16][NB], bl[16][NB];
            fl_f32x16 ap[NB], al[NB];
            {
                fl_f32x16 dq;
#pragma unroll
                for (int r = 0; r < 16; ++r) dq[r] = 0.0f;
                float qa[16], qb[16], qc[16], qd[16];
                read_q(0, qa, qb);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 16; ++i) dq = __builtin_amdgcn_mfma_f32_32x32x2f32(qa[i], qb[i], dq, 0, 0, 0);
                read_q(16, qc, qd);
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
                    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);   // DS read
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 16; ++i) dq = __builtin_amdgcn_mfma_f32_32x32x2f32(qc[i], qd[i], dq, 0, 0, 0);
                read_b(pb, bp);
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);   // MFMA
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 1);   // DS read
                }
                __builtin_amdgcn_sched_barrier(0);
                // register r of dq is row 8 (r / 4) + 4 lk + r % 4 of D; rows
                // (r, r + 1), r even, are window amplitude x = 4 (r / 4) + 2 lk +
                // (r % 4) / 2, components re, im, and this lane's column is
                // (y, b) = (lc >> 1, lc & 1).  With t = register r + 1 of the
                // neighbouring lane, b = 0 forms Re Q = D[2x][2y] + t and b = 1
                // forms Im Q = t - D[2x][2y+1].
#pragma unroll
                for (int pr = 0; pr < 8; ++pr) {
                    const int r = 2 * pr;
                    const float t = fl_dpp_f<0xB1>(dq[r + 1]);   // quad_perm(1,0,3,2): lane ^ 1
                    const float v = fmaf(qsgn, dq[r], t);
                    const int x = 4 * (pr >> 1) + 2 * lk + (pr & 1);
                    __hip_atomic_fetch_add(&qacc[g][(lc & 1) * 256 + 16 * x + (lc >> 1)], v, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
            // the next tile's psi loads run under the last group's MFMAs
            if (g + 1 == pd.ngroups && next < ntiles) {
                fetch(next, psi, tp);
                fetched = true;
            }
            __builtin_amdgcn_sched_barrier(0);
            // (2) U^dagger on psi, with lambda's reads in between
            mfma_u(bp, ap);
            read_b(lb, bl);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 2, 2);   // MFMA
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 2);   // DS read
            }
            __builtin_amdgcn_sched_barrier(0);
            // (3) U^dagger on lambda, with psi's writes in between
            mfma_u(bl, al);
            write_u(pb, ap);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 2, 3);   // MFMA
                __builtin_amdgcn_sched_group_barrier(0x200, 1, 3);   // DS write
            }
            __builtin_amdgcn_sched_barrier(0);
            write_u(lb, al);
            if (g + 1 == pd.ngroups || part(pass_u0(pd, g + 1)) != part(u0))
                __syncthreads();
            else
                __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int k = 0; k < 16; ++k) a[k] = an[k];
        }
        const uint64_t base = fl_tile_base(tile, C, W, h);
        tile_store<float, K, NT, 1>(psi, base, K, C, h, lp);
        tile_store<float, K, NT, 1>(lam, base, K, C, h, ll);
        if (next < ntiles) {
            if (!fetched) fetch(next, psi, tp);
            fetch(next, lam, tl);
            __syncthreads();   // every wave has read the tile out of LDS
            put();
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < pd.ngroups * 512; t += NT)
        Qpart[(size_t)blockIdx.x * NG * 512 + t] = (double)(&qacc[0][0])[t];
}

// Qsum[t] += sum over the workgroups of Qpart[b][t] (t < nvals).  A block
// takes 32 consecutive values; its thread (v, j) sums rows b = j, j + 8, ...
// of value v (coalesced 256-byte rows), then the 8 partial sums of each value
// are added in j order, so the result does not depend on timing.
__global__ __launch_bounds__(256) void k_qsum(const double* __restrict__ Qpart, int nblocks, int nvals,
                                              double* __restrict__ Qsum) {
    __shared__ double part[8][32];
    const int v = threadIdx.x & 31, j = threadIdx.x >> 5;
    const int t = blockIdx.x * 32 + v;
    double s = 0.0;
    if (t < nvals) {
#pragma unroll 8
        for (int b = j; b < nblocks; b += 8) s += Qpart[(size_t)b * FL_WIN4_MAX_GROUPS * 512 + t];
    }
    part[j][v] = s;
    __syncthreads();
    if (j == 0 && t < nvals) {
        double r = part[0][v];
#pragma unroll
        for (int k = 1; k < 8; ++k) r += part[k][v];
        Qsum[t] += r;
    }
}

__global__ void k_zero(double* __restrict__ p, uint64_t n) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0.0;
}

// ---------------------------------------------------------------------------
// dense 6-qubit windows on the matrix cores (complex64 states)
// ---------------------------------------------------------------------------
// Every register group of a dense plan is one window of 6 consecutive tile
// bits [u0, u0+6); its gates were multiplied on the host (FP64) into a 64x64
// complex matrix U, applied here as the real 128x128 contraction
//   Y = A X,  A[2m'+c'][2m+c] = (Re U, -Im U; Im U, Re U)[c'][c] at (m', m),
// on the 128-column matrix X whose column v is the 64-vector of amplitudes
// sharing the other 7 tile bits, real index k = 2m + (0: re, 1: im).
// Wave w owns output rows [32w, 32w+32) and keeps its A rows in VGPRs.
//   MODE 0: FP32 MFMA v_mfma_f32_32x32x2f32 (k = 2 per step).
//   MODE 1: split BF16x3: X = Xh + Xl, A = Ah + Al (round-to-nearest-even
//           bf16 splits), Y = Ah Xh + Ah Xl + Al Xh with
//           v_mfma_f32_32x32x16_bf16 and FP32 accumulation.
// A fragments arrive pre-arranged per (wave, lane): MODE 0 as 64 floats
// (step kk = k/2), MODE 1 as 8 steps x 8 bf16 for hi, then the same for lo.


#define FL_DENSE_PLANE_STRIDE 136   // bf16 per column of a split plane (128 + 8 pad)

// FULL: the tile has the full KMAXD = 13 bits (every chain with L >= 13), so
// the column-block and element counts are compile-time constants.  The FP32
// tile uses the slots of fl_swz12: the 32 columns of a block read at one
// window position then meet at most two addresses per bank even for windows
// starting at bit 0, where fl_swz left them on 4 distinct slots.
template <int MODE, bool FULL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_dense6(float2* __restrict__ psi, const float4* __restrict__ mats,
                                                uint32_t ntiles, int C, int W, fl_pass pd) {
    constexpr int KMAXD = 13;
    constexpr int TILE_BYTES = (1 << KMAXD) * 8;
    constexpr int PLANE_BYTES = 128 * FL_DENSE_PLANE_STRIDE * 2;
    constexpr int LDS_BYTES = (MODE == 1 && 2 * PLANE_BYTES > TILE_BYTES) ? 2 * PLANE_BYTES : TILE_BYTES;
    __shared__ __attribute__((aligned(16))) unsigned char smem[LDS_BYTES];
    float2* lds = reinterpret_cast<float2*>(smem);
    const int K = FULL ? KMAXD : C + W;
    const int h = pd.h;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int lc = lane & 31, lk = lane >> 5;
    const int ncb = FULL ? 4 : 1 << (K - 6 - 5);   // 32-column blocks (1, 2 or 4)
    const int ng = pd.ngroups;
    const uint64_t base = fl_tile_base(blockIdx.x, C, W, h);
    // full tiles: the unrolled form, every thread's 16 loads in flight at once
    if constexpr (FULL)
        tile_load<float, KMAXD, 256, 1>(psi, base, K, C, h, lds);
    else
        tile_load<float, 0, 256, 1>(psi, base, K, C, h, lds);
    __syncthreads();
    // write Y (registers of one window) back to the FP32 tile: register r of
    // block cb holds row 32w + 8(r/4) + 4 lk + r%4 (= 2m' + c'), column
    // 32 cb + lc; slot(cbase | m << u0) = slot(cbase) ^ slot(m << u0), the
    // second part uniform
    auto store_fp32 = [&](const fl_f32x16 (&acc)[4], const uint32_t (&cbase)[4], int u0) {
        const uint32_t mrow = 16 * w + 2 * lk;   // m of register 0 (rows 32w + 4lk, +1)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            if (cb < ncb) {
                const uint32_t vb = fl_swz12(cbase[cb]) * 8u;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        const uint32_t m = mrow + 4 * q + p;   // rows 32w + 8q + 4lk + 2p, +1
                        float2 v;
                        v.x = acc[cb][4 * q + 2 * p];
                        v.y = acc[cb][4 * q + 2 * p + 1];
                        *reinterpret_cast<float2*>(smem + (vb ^ (fl_swz12(m << u0) * 8u))) = v;
                    }
                }
            }
        }
    };
    auto column_bases = [&](int u0, uint32_t (&cbase)[4]) {
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) cbase[cb] = fl_spread((32 * cb + lc) & ((1 << (K - 6)) - 1), u0, 6);
    };
    if constexpr (MODE == 0) {
        for (int g = 0; g < ng; ++g) {
            const int u0 = pass_u0(pd, g);
            // 4096 float4 (64 KiB) per window
            const float4* M = mats + (size_t)pass_gate(pd, g, 0) * 4096 + (size_t)(w * 64 + lane) * 16;
            uint32_t cbase[4];
            column_bases(u0, cbase);
            fl_f32x16 acc[4];
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[cb][r] = 0.0f;
            float a[64];
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const float4 t = M[q];
                a[4 * q] = t.x;
                a[4 * q + 1] = t.y;
                a[4 * q + 2] = t.z;
                a[4 * q + 3] = t.w;
            }
            // element (column, m) of the tile sits at slot(cbase | m << u0) =
            // slot(cbase) ^ slot(m << u0) (the swizzle is linear over XOR); the
            // lane's half (re for lk = 0, im for lk = 1) is 4 lk bytes further
            uint32_t bb[4];
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) bb[cb] = fl_swz12(cbase[cb]) * 8u + 4u * (uint32_t)lk;
            // B operands of step kk + 2 are read while step kk multiplies
            constexpr int PF = 2;
            float bq[PF + 1][4];
            auto fetch = [&](int kk, float (&dst)[4]) {
                const uint32_t sk = fl_swz12((uint32_t)kk << u0) * 8u;
#pragma unroll
                for (int cb = 0; cb < 4; ++cb)
                    if (cb < ncb) dst[cb] = *reinterpret_cast<const float*>(smem + (bb[cb] ^ sk));
            };
#pragma unroll
            for (int kk = 0; kk < PF; ++kk) fetch(kk, bq[kk]);
#pragma unroll
            for (int kk = 0; kk < 64; ++kk) {
                if (kk + PF < 64) fetch(kk + PF, bq[(kk + PF) % (PF + 1)]);
#pragma unroll
                for (int cb = 0; cb < 4; ++cb)
                    if (cb < ncb)
                        acc[cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[kk], bq[kk % (PF + 1)][cb], acc[cb], 0, 0, 0);
            }
            __syncthreads();
            store_fp32(acc, cbase, u0);
            __syncthreads();
        }
    } else {
        // The B operand of a window lives in LDS as two bf16 planes (hi, lo)
        // laid out [column][k]; element j of the tile (window bits from u) sits
        // at plane offset o_u(j) = col_u(j) STRIDE + 2 m_u(j) (+1 for the
        // imaginary part).  col_u and m_u are bit fields of j, so o_u is
        // additive over indices with disjoint bits.  The planes of the first
        // window come from the FP32 tile; those of every later window straight
        // from the previous window's accumulators (split once, when written),
        // and only the last window writes FP32 again, for the store.
        __bf16* ph = reinterpret_cast<__bf16*>(smem);
        __bf16* pl = ph + 128 * FL_DENSE_PLANE_STRIDE;
        typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
        auto plane_off = [](uint32_t j, int u) {
            const uint32_t m = (j >> u) & 63;
            const uint32_t col = (j & ((1u << u) - 1)) | ((j >> (u + 6)) << u);
            return col * FL_DENSE_PLANE_STRIDE + 2 * m;
        };
        // (re, im) of one amplitude are adjacent in a plane: one 32-bit LDS
        // store per plane; hi = RNE_bf16(x), lo = RNE_bf16(x - hi)
        auto split_store = [&](float re, float im, uint32_t o) {
            bf2 hv, lv;
            hv.x = (__bf16)re;
            hv.y = (__bf16)im;
            lv.x = (__bf16)(re - (float)hv.x);
            lv.y = (__bf16)(im - (float)hv.y);
            *reinterpret_cast<bf2*>(ph + o) = hv;
            *reinterpret_cast<bf2*>(pl + o) = lv;
        };
        if (ng > 0) {
            // first window: every thread reads its amplitudes of the FP32
            // tile, the workgroup syncs, then the planes overwrite the tile
            constexpr int PER = (1 << KMAXD) / 256;
            float2 mine[PER];
            const int nper = FULL ? PER : (1 << K) / 256;
            const uint32_t l0 = fl_swz12(threadIdx.x);   // slot(tid + 256 t) = l0 ^ slot(256 t)
#pragma unroll
            for (int t = 0; t < PER; ++t)
                if (t < nper) mine[t] = lds[l0 ^ fl_swz12(256u * (uint32_t)t)];
            __syncthreads();
            const int u0 = pass_u0(pd, 0);
            const uint32_t otid = plane_off(threadIdx.x, u0);
#pragma unroll
            for (int t = 0; t < PER; ++t)
                if (t < nper)
                    // readfirstlane: keep the uniform term a scalar
                    split_store(mine[t].x, mine[t].y,
                                otid + __builtin_amdgcn_readfirstlane(plane_off(256u * (uint32_t)t, u0)));
            __syncthreads();
        }
        // A fragments of a window: 8 steps x 8 bf16 for hi, then for lo.  The
        // window stores each (Re, Im) pair of U once (32 KiB): lanes 2m' and
        // 2m'+1 of a half-wave load the same 16 bytes, and row 2m' takes them
        // as (Re, -Im), row 2m'+1 as (Im, Re): a rotation by 16 bits per lane
        // parity, then a sign flip of the high half for the even rows.
        fl_bf16x8 ah[8], al[8];
        const uint32_t rot = 16u * (uint32_t)(lane & 1);
        const uint32_t neg = (lane & 1) ? 0u : 0x80000000u;
        auto fix = [&](const float4& t) {
            uint4 u = *reinterpret_cast<const uint4*>(&t);
            u.x = __builtin_amdgcn_alignbit(u.x, u.x, rot) ^ neg;
            u.y = __builtin_amdgcn_alignbit(u.y, u.y, rot) ^ neg;
            u.z = __builtin_amdgcn_alignbit(u.z, u.z, rot) ^ neg;
            u.w = __builtin_amdgcn_alignbit(u.w, u.w, rot) ^ neg;
            return *reinterpret_cast<const fl_bf16x8*>(&u);
        };
        auto load_a = [&](int g) {
            const float4* M = mats + (size_t)pass_gate(pd, g, 0) * 2048 + (size_t)(w * 16 * 16 + lk * 16 + (lc >> 1));
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const float4 th = M[q * 32], tl = M[1024 + q * 32];
                ah[q] = fix(th);
                al[q] = fix(tl);
            }
        };
        if (ng > 0) load_a(0);
        for (int g = 0; g < ng; ++g) {
            const int u0 = pass_u0(pd, g);
            uint32_t cbase[4];
            column_bases(u0, cbase);
            fl_f32x16 acc[4];
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[cb][r] = 0.0f;
#pragma unroll
            for (int st = 0; st < 8; ++st) {
                const int k0 = 16 * st + 8 * lk;
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) {
                    if (cb < ncb) {
                        const uint32_t col = 32 * cb + lc;
                        const uint32_t o = col * FL_DENSE_PLANE_STRIDE + k0;
                        const fl_bf16x8 bh = *reinterpret_cast<const fl_bf16x8*>(ph + o);
                        const fl_bf16x8 bl = *reinterpret_cast<const fl_bf16x8*>(pl + o);
                        acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[st], bh, acc[cb], 0, 0, 0);
                        acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[st], bl, acc[cb], 0, 0, 0);
                        acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[st], bh, acc[cb], 0, 0, 0);
                    }
                }
            }
            // the next window's fragments go into the registers just freed,
            // so that their latency overlaps the barrier and the split
            if (g + 1 < ng) load_a(g + 1);
            __syncthreads();   // every wave has read this window's planes
            if (g + 1 < ng) {
                // element of register (cb, q, p): j = cbase[cb] | (mrow + 4q + p) << u0,
                // three parts with disjoint bits: o(j) = o(cbase | mrow << u0) + o((4q + p) << u0)
                const int un = pass_u0(pd, g + 1);
                const uint32_t mrow = 16 * w + 2 * lk;
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) {
                    if (cb < ncb) {
                        const uint32_t ob = plane_off(cbase[cb] | (mrow << u0), un);
#pragma unroll
                        for (int q = 0; q < 4; ++q)
#pragma unroll
                            for (int p = 0; p < 2; ++p)
                                split_store(acc[cb][4 * q + 2 * p], acc[cb][4 * q + 2 * p + 1],
                                            ob + __builtin_amdgcn_readfirstlane(
                                                     plane_off((uint32_t)(4 * q + p) << u0, un)));
                    }
                }
            } else {
                store_fp32(acc, cbase, u0);
            }
            __syncthreads();
        }
    }
    if constexpr (FULL)
        tile_store<float, KMAXD, 256, 1>(psi, base, K, C, h, lds);
    else
        tile_store<float, 0, 256, 1>(psi, base, K, C, h, lds);
}

// ---------------------------------------------------------------------------
// dense 4-qubit windows on the FP32 matrix cores (complex64 states)
// ---------------------------------------------------------------------------
// Every register group of a dense-4 plan is one window of 4 consecutive tile
// bits [u0, u0+4); its gates were multiplied on the host (FP64) into a 16x16
// complex matrix U, applied as the real 32x32 contraction Y = A X with
// A[2m'+c'][2m+c] = (Re U, -Im U; Im U, Re U)[c'][c] at (m', m): exactly one
// v_mfma_f32_32x32x2f32 output tile, K = 32 in 16 steps of 2.  Column v of X
// is the 16-vector of amplitudes sharing the other 9 tile bits; a tile has
// 512 columns, 512 / NW per wave (blocks of 32).  The contraction index runs
// component-major, k' = 16 c + m: step s takes k' = 2s + l/32, so lane l
// supplies A[l%32][k'] (16 VGPRs, the same for every wave) and, per block,
// component s/8 of amplitude 2(s mod 8) + l/32 of its column; steps s and
// s + 8 use the two halves of one 8-byte LDS read.  A wave reads and writes
// only its own columns: the columns of wave w are those whose log2(NW)
// highest bits outside the window equal w, so consecutive windows that leave
// the same tile bits to the wave index (with NW = 8 all windows below bit 7
// leave bits 10, 11 and 12) need no barrier between them, only this wave's
// own LDS order.
template <int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW / 2))) void k_dense4(
    float2* __restrict__ psi, const float4* __restrict__ mats, int W, fl_pass pd) {
    constexpr int K = 13;
    constexpr int C = FL_DENSE4_LOWBITS;
    constexpr int NB = 16 / NW;                  // 32-column blocks per wave (512 columns per tile)
    constexpr int WB = __builtin_ctz(NW);        // column bits that name the wave
    __shared__ __attribute__((aligned(16))) float2 lds[1 << K];
    const char* const lbytes = reinterpret_cast<const char*>(lds);
    const int h = pd.h;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int lc = lane & 31, lk = lane >> 5;
    const uint64_t base = fl_tile_base(blockIdx.x, C, W, h);
    tile_load<float, K, 64 * NW>(psi, base, K, C, h, lds);
    __syncthreads();
    // A fragments of a window: 64 lanes x 16 floats (4 KiB).  The next
    // window's fragments are fetched while the current window is applied; the
    // last window fetches its own again, so that no branch lets the loads
    // drift down to their use.
    auto load_a = [&](int g, float (&dst)[16]) {
        const float4* M = mats + (size_t)pass_gate(pd, g, 0) * 256 + (size_t)lane * 4;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 t = M[q];
            dst[4 * q] = t.x;
            dst[4 * q + 1] = t.y;
            dst[4 * q + 2] = t.z;
            dst[4 * q + 3] = t.w;
        }
    };
    float a[16], an[16];
    if (pd.ngroups > 0) load_a(0, a);
    for (int g = 0; g < pd.ngroups; ++g) {
        const int u0 = pass_u0(pd, g);
        load_a(g + 1 < pd.ngroups ? g + 1 : g, an);
        __builtin_amdgcn_sched_barrier(0);
        // slot(spread(col) | s << u0) = slot(spread(col)) ^ slot(s << u0): the
        // second part is uniform (the swizzle is linear over XOR)
        uint32_t vb[NB];
#pragma unroll
        for (int cb = 0; cb < NB; ++cb)
            vb[cb] = fl_swz(fl_spread((uint32_t)(32 * NB * w + 32 * cb + lc), u0, 4)) * 8u;
        fl_f32x16 acc[NB];
#pragma unroll
        for (int cb = 0; cb < NB; ++cb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[cb][r] = 0.0f;
        float bq[16][NB];
        // amplitude 2t + lk of the column: slot(spread(col)) ^ slot(lk << u0) ^ slot(2t << u0)
        const uint32_t lkoff = fl_swz((uint32_t)lk << u0) * 8u;
        auto read_b = [&](int cb) {
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const uint32_t ss = fl_swz((uint32_t)(2 * t) << u0) * 8u;
                const float2 x = *reinterpret_cast<const float2*>(lbytes + ((vb[cb] ^ lkoff) ^ ss));
                bq[t][cb] = x.x;
                bq[t + 8][cb] = x.y;
            }
        };
        auto mfma_b = [&](int cb) {
#pragma unroll
            for (int st = 0; st < 16; ++st)
                acc[cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[st], bq[st][cb], acc[cb], 0, 0, 0);
        };
        // register r of block cb holds row 8(r/4) + 4 lk + r%4 = 2m' + c'
        auto write_b = [&](int cb) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    const uint32_t m = 4 * q + 2 * lk + p;
                    float2 v;
                    v.x = acc[cb][4 * q + 2 * p];
                    v.y = acc[cb][4 * q + 2 * p + 1];
                    *reinterpret_cast<float2*>(reinterpret_cast<char*>(lds) + (vb[cb] ^ (fl_swz(m << u0) * 8u))) = v;
                }
        };
        // Blocks in two halves, so that the LDS traffic of one half runs
        // under the MFMAs of the other: read the first half, then its MFMAs
        // with the second half's reads in between, then the second half's
        // MFMAs with the first half's writes in between, then those writes.
        // (Each block reads and writes only its own columns.)
        constexpr int HB = NB / 2;
#pragma unroll
        for (int cb = 0; cb < HB; ++cb) read_b(cb);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int cb = 0; cb < HB; ++cb) mfma_b(cb);
#pragma unroll
        for (int cb = HB; cb < NB; ++cb) read_b(cb);
#pragma unroll
        for (int i = 0; i < 8 * HB; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);   // MFMA
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // DS read
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int cb = HB; cb < NB; ++cb) mfma_b(cb);
#pragma unroll
        for (int cb = 0; cb < HB; ++cb) write_b(cb);
#pragma unroll
        for (int i = 0; i < 8 * HB; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 1);   // MFMA
            __builtin_amdgcn_sched_group_barrier(0x200, 1, 1);   // DS write
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int cb = HB; cb < NB; ++cb) write_b(cb);
        // the WB tile bits that select a wave's columns: column bits 9 - WB .. 8,
        // which sit 4 higher when at or above the window, so the set depends
        // only on how many of them lie below u0
        auto part = [](int u) { return u <= 9 - WB ? 0 : u - (9 - WB); };
        if (g + 1 == pd.ngroups || part(pass_u0(pd, g + 1)) != part(u0))
            __syncthreads();
        else
            __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int k = 0; k < 16; ++k) a[k] = an[k];
    }
    tile_store<float, K, 64 * NW>(psi, base, K, C, h, lds);
}

// ---------------------------------------------------------------------------
// launch wrappers
// ---------------------------------------------------------------------------

static inline uint32_t ntiles_of(const fl_geom& g) { return 1u << (g.L - g.K); }

// The words form of a pass's descriptor, gates relative to table entry gofs.
static bool sweep_words(const fl_pass& pd, int gofs, fl_sweep_words& w) {
    int n = pd.ngroups;
    for (int g = 0; g < pd.ngroups; ++g) n += pd.nops[g];
    if (n + 1 > FL_SWEEP_WORDS) return false;
    w.h = pd.h;
    w.ngroups = pd.ngroups;
    w.ufirst = pd.ngroups > 0 ? pd.u0[0] : -1;
    w.ulast = pd.ngroups > 0 ? pd.u0[pd.ngroups - 1] : -1;
    n = 0;
    for (int g = 0; g < pd.ngroups; ++g) w.w[n++] = (uint32_t)pd.u0[g] | (uint32_t)pd.nops[g] << 8;
    for (int g = 0; g < pd.ngroups; ++g)
        for (int k = 0; k < pd.nops[g]; ++k)
            w.w[n++] = (uint32_t)pd.opi[g][k] | (uint32_t)(pd.opg[g][k] - gofs) << 8;
    w.w[n++] = 0;   // read one op ahead
    w.nwords = n;
    return true;
}

template <typename T, int R, int K, int C, int WPE, typename D>
static hipError_t launch_tiles(const fl_geom& g, void* psi, const void* gates, const fl_pass& pd, int gofs,
                               hipStream_t s) {
    typedef typename CT<T>::c cplx;
    constexpr int NT = 1 << (K - R);
    const dim3 grid(ntiles_of(g)), block(NT);
    if constexpr (std::is_same<D, fl_sweep_words>::value) {
        fl_sweep_words w;
        if (!sweep_words(pd, gofs, w)) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_sweep_tiles<T, R, K, NT, C, WPE, D>), grid, block, 0, s, (cplx*)psi, (const T*)gates, g.W,
                           w, g.L - 1, gofs);
    } else {
        hipLaunchKernelGGL((k_sweep_tiles<T, R, K, NT, C, WPE, D>), grid, block, 0, s, (cplx*)psi, (const T*)gates, g.W,
                           pd, g.L - 1, gofs);
    }
    return hipGetLastError();
}

// The words form with one op per group (2-bit groups): a bond's gates never
// follow each other without its neighbours' between them, unless it has none.
static bool quad_words(const fl_pass& pd, int gofs, fl_sweep_words& w) {
    if (!sweep_words(pd, gofs, w)) return false;
    int n = 0;
    for (int g = 0; g < pd.ngroups; ++g) n += pd.nops[g];
    if (2 * n + 1 > FL_SWEEP_WORDS) return false;
    int k = 0;
    for (int g = 0; g < pd.ngroups; ++g)
        for (int q = 0; q < pd.nops[g]; ++q, ++k) {
            w.w[k] = (uint32_t)pd.u0[g];
            w.w[n + k] = (uint32_t)(pd.opg[g][q] - gofs) << 8;
        }
    w.w[2 * n] = 0;
    w.ngroups = n;
    w.nwords = 2 * n + 1;
    return true;
}

template <typename T, int K, int C>
static hipError_t launch_quads(const fl_geom& g, void* psi, const void* gates, const fl_pass& pd, int gofs,
                               hipStream_t s) {
    typedef typename CT<T>::c cplx;
    fl_sweep_words w;
    if (!quad_words(pd, gofs, w)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_sweep_quads<T, K, C>), dim3(ntiles_of(g)), dim3(1 << (K - 2)), 0, s, (cplx*)psi,
                       (const T*)gates + 32 * gofs, g.W, w, g.L - 1);
    return hipGetLastError();
}

template <typename T, int K, int C>
static hipError_t launch_lanes(const fl_geom& g, void* psi, const void* gates, const fl_pass& pd, int gofs,
                               hipStream_t s) {
    typedef typename CT<T>::c cplx;
    fl_sweep_words w;
    if (!sweep_words(pd, gofs, w)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_sweep_lanes<T, K, C>), dim3(ntiles_of(g)), dim3(1 << K), 0, s, (cplx*)psi,
                       (const T*)gates + 32 * gofs, g.W, w, g.L - 1);
    return hipGetLastError();
}

template <typename T, int S, int NT>
static hipError_t launch_one_s(int L, void* psi, const void* gates, const fl_sweep_words& w, int gofs, int reps,
                               hipStream_t s) {
    typedef typename CT<T>::c cplx;
    hipLaunchKernelGGL((k_sweep_one<T, S, NT>), dim3(1), dim3(NT), 0, s, (cplx*)psi, (const T*)gates + 32 * gofs, L, w,
                       reps);
    return hipGetLastError();
}

// Threads per quad: as many as give every SIMD a wave (L = 8: 64 quads in four
// waves instead of one), two at most where the quads alone do; up to L = 6 one
// wave holds all and no barrier waits for another.  16 periods, with one thread
// per quad in 256-thread workgroups before, on plans of 16 periods (us):
// complex64 L = 4 20.1 -> 14.0, 8 44.0 -> 36.2, 9 54.3 -> 42.5, 10 62.9 -> 54.3;
// complex128 L = 6 34.8 -> 20.9, 8 50.2 -> 40.0, 10 77.2 -> 72.1.  Four per quad
// are slower at L = 9 (45.8) and 10 (66.3): each reads the whole quad.  L = 2 has nothing to share.
template <typename T>
static hipError_t launch_one(int L, void* psi, const void* gates, const fl_sweep_words& w, int gofs, int reps,
                             hipStream_t s) {
    if (L == 2) return launch_one_s<T, 1, 64>(L, psi, gates, w, gofs, reps, s);
    if (L <= 6) return launch_one_s<T, 4, 64>(L, psi, gates, w, gofs, reps, s);
    if (L <= 8) return launch_one_s<T, 4, 256>(L, psi, gates, w, gofs, reps, s);
    if (L == 9) return launch_one_s<T, 2, 256>(L, psi, gates, w, gofs, reps, s);
    return launch_one_s<T, 2, 512>(L, psi, gates, w, gofs, reps, s);
}

hipError_t launch_sweep(int dtype, const fl_geom& g, void* psi, const void* gates, const fl_pass& pd, int reps,
                        hipStream_t s) {
    if (reps < 1 || (reps > 1 && g.W != 0)) return hipErrorInvalidValue;
    // a pass applies gates of one direction: G_b (table entries 0 .. L-2) or G_b^dagger
    const int nb = g.L - 1;
    if (nb > FL_MAX_GATE_TABLE) return hipErrorInvalidValue;
    int gofs = 0;
    for (int q = 0; q < pd.ngroups; ++q)
        if (pd.nops[q] > 0) gofs = pd.opg[q][0] >= nb ? nb : 0;
    for (int q = 0; q < pd.ngroups; ++q)
        for (int k = 0; k < pd.nops[q]; ++k)
            if (pd.opg[q][k] < gofs || pd.opg[q][k] >= gofs + nb) return hipErrorInvalidValue;
    if (g.W == 0) {
        if (g.L < 2 || g.L > FL_KMAX_ONE || g.R != 2) return hipErrorInvalidValue;
        fl_sweep_words w;
        if (!quad_words(pd, gofs, w)) return hipErrorInvalidValue;
        return dtype == 0 ? launch_one<float>(g.L, psi, gates, w, gofs, reps, s)
                          : launch_one<double>(g.L, psi, gates, w, gofs, reps, s);
    }
    // the geometries of sweep_geom
    const int key = (dtype << 12) | (g.K << 8) | (g.C << 4) | g.R;
    auto code = [](int dt, int K, int C, int R) { return (dt << 12) | (K << 8) | (C << 4) | R; };
    if (key == code(0, 13, 4, 4)) return launch_tiles<float, 4, 13, 4, 4, fl_pass>(g, psi, gates, pd, gofs, s);
    if (key == code(0, 12, 4, 3)) return launch_tiles<float, 3, 12, 4, 4, fl_sweep_words>(g, psi, gates, pd, gofs, s);
    if (key == code(0, 11, 3, 2)) return launch_quads<float, 11, 3>(g, psi, gates, pd, gofs, s);
    if (key == code(0, 10, 3, 4)) return launch_lanes<float, 10, 3>(g, psi, gates, pd, gofs, s);
    if (key == code(1, 12, 6, 4)) return launch_tiles<double, 4, 12, 6, 2, fl_pass>(g, psi, gates, pd, gofs, s);
    if (key == code(1, 12, 3, 4)) return launch_tiles<double, 4, 12, 3, 2, fl_pass>(g, psi, gates, pd, gofs, s);
    if (key == code(1, 11, 3, 3)) return launch_tiles<double, 3, 11, 3, 2, fl_sweep_words>(g, psi, gates, pd, gofs, s);
    if (key == code(1, 10, 3, 4)) return launch_lanes<double, 10, 3>(g, psi, gates, pd, gofs, s);
    if (key == code(1, 9, 3, 4)) return launch_lanes<double, 9, 3>(g, psi, gates, pd, gofs, s);
    return hipErrorInvalidValue;
}

hipError_t launch_rdm(int dtype, const fl_geom& g, const void* psi, const fl_pass& pd, double* partials, int nslot,
                      hipStream_t s) {
    if (g.W != 0 || g.K > FL_KMAX_RDM || pd.ngroups > FL_RDM_MAXG) return hipErrorInvalidValue;
    if (dtype == 0)
        hipLaunchKernelGGL(k_rdm<float>, dim3(1), dim3(FL_NT), 0, s, (const float2*)psi, g.K, pd, partials, nslot);
    else
        hipLaunchKernelGGL(k_rdm<double>, dim3(1), dim3(FL_NT), 0, s, (const double2*)psi, g.K, pd, partials, nslot);
    return hipGetLastError();
}

template <typename T, int K>
static void launch_windows(const fl_geom& g, const void* psi, const rdm_desc& pd, double* partials, int grid, int nslot,
                           hipStream_t s) {
    hipLaunchKernelGGL((k_rdm_windows<T, K, FL_RDM_LOWBITS, 256>), dim3(grid), dim3(256), 0, s,
                       (const typename CT<T>::c*)psi, g.W, ntiles_of(g), pd, partials, nslot);
}

hipError_t launch_rdm_windows(int dtype, const fl_geom& g, const void* psi, const rdm_desc& pd, double* partials,
                              int grid, int nslot, hipStream_t s) {
    if (g.C != FL_RDM_LOWBITS || g.C + g.W != g.K || (pd.nwin != 1 && pd.nwin != 2 && pd.nwin != 4) || grid < 1)
        return hipErrorInvalidValue;
    if (g.K < 12 && pd.nwin != 4) return hipErrorInvalidValue;   // fewer windows would leave waves without a part
    for (int w = 0; w < pd.nwin; ++w)
        if (pd.u0[w] < 0 || pd.u0[w] + 4 > g.K) return hipErrorInvalidValue;
    switch (g.K | dtype << 8) {
        case 10: launch_windows<float, 10>(g, psi, pd, partials, grid, nslot, s); break;
        case 11: launch_windows<float, 11>(g, psi, pd, partials, grid, nslot, s); break;
        case 12: launch_windows<float, 12>(g, psi, pd, partials, grid, nslot, s); break;
        case 13: launch_windows<float, 13>(g, psi, pd, partials, grid, nslot, s); break;
        case 10 | 256: launch_windows<double, 10>(g, psi, pd, partials, grid, nslot, s); break;
        case 11 | 256: launch_windows<double, 11>(g, psi, pd, partials, grid, nslot, s); break;
        case 12 | 256: launch_windows<double, 12>(g, psi, pd, partials, grid, nslot, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_energy_contract(const double* red, const double* h64, int L, double* out, double* rdm, hipStream_t s) {
    if (L < 2 || L > 65) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_energy_contract, dim3(1), dim3(64), 0, s, red, h64, L, out, rdm);
    return hipGetLastError();
}

hipError_t launch_finalize(const double* partials, int nblocks, int nvals, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_finalize, dim3(nvals), dim3(256), 0, s, partials, nblocks, nvals, out);
    return hipGetLastError();
}

hipError_t launch_init(int dtype, void* psi, int L, const void* tabs, int a, int b, hipStream_t s) {
    const uint64_t n = 1ull << L;
    const double2* t = (const double2*)tabs;
    const double2* tlo = t;
    const double2* tmid = t + (1 << a);
    const double2* thi = tmid + (1 << b);
    const uint64_t want = (n + 255) / 256;
    const unsigned grid = (unsigned)(want < 65536 ? want : 65536);
    if (dtype == 0 && a >= 1) {
        const uint64_t want2 = (n / 2 + 255) / 256;
        hipLaunchKernelGGL(k_init_pairs_c64, dim3((unsigned)(want2 < 65536 ? want2 : 65536)), dim3(256), 0, s,
                           (float4*)psi, tlo, tmid, thi, a, b, n / 2);
    } else if (dtype == 0)
        hipLaunchKernelGGL(k_init<float>, dim3(grid), dim3(256), 0, s, (float2*)psi, tlo, tmid, thi, a, b, n);
    else
        hipLaunchKernelGGL(k_init<double>, dim3(grid), dim3(256), 0, s, (double2*)psi, tlo, tmid, thi, a, b, n);
    return hipGetLastError();
}

hipError_t launch_overlap(int dta, const void* a, int dtb, const void* b, uint64_t n, double* partials, int grid,
                          hipStream_t s) {
    if (dta == 1 && dtb == 0)
        hipLaunchKernelGGL((k_overlap<double, float>), dim3(grid), dim3(256), 0, s, (const double2*)a, (const float2*)b,
                           n, partials);
    else if (dta == 1 && dtb == 1)
        hipLaunchKernelGGL((k_overlap<double, double>), dim3(grid), dim3(256), 0, s, (const double2*)a,
                           (const double2*)b, n, partials);
    else if (dta == 0 && dtb == 1)
        hipLaunchKernelGGL((k_overlap<float, double>), dim3(grid), dim3(256), 0, s, (const float2*)a,
                           (const double2*)b, n, partials);
    else
        hipLaunchKernelGGL((k_overlap<float, float>), dim3(grid), dim3(256), 0, s, (const float2*)a, (const float2*)b,
                           n, partials);
    return hipGetLastError();
}

hipError_t launch_apply_h(int dtype, const fl_geom& g, const void* psi, void* lam, const void* hmat, const fl_pass& pd,
                          int first, hipStream_t s) {
    const dim3 grid(ntiles_of(g)), block(FL_NT);
    if (dtype == 0)
        hipLaunchKernelGGL((k_apply_h<float, FL_KMAX_C64>), grid, block, 0, s, (const float2*)psi, (float2*)lam,
                           (const float*)hmat, g.C, g.W, pd, first);
    else
        hipLaunchKernelGGL((k_apply_h<double, FL_KMAX_C128>), grid, block, 0, s, (const double2*)psi,
                           (double2*)lam, (const double*)hmat, g.C, g.W, pd, first);
    return hipGetLastError();
}

hipError_t launch_apply_h_tiles(int dtype, const fl_geom& g, const void* psi, void* lam, const void* tab,
                                const apply_h_desc& pd, double* dots, int grid, hipStream_t s) {
    if (g.W == 0 || pd.nwin < 1 || pd.nwin > FL_HWIN_MAX || pd.u0[pd.nwin - 1] < 4 || grid < 1)
        return hipErrorInvalidValue;
    for (int k = 0; k < pd.nwin; ++k)
        if (pd.u0[k] < 0 || pd.u0[k] + 4 > g.K) return hipErrorInvalidValue;
    const uint32_t nt = ntiles_of(g);
    if (dtype == 0) {
        if (g.K != FL_KMAX_C64 || g.C != FL_SWEEP_LOWBITS_C64) return hipErrorInvalidValue;
        constexpr int K = FL_KMAX_C64, C = FL_SWEEP_LOWBITS_C64;
        auto* p = (const float2*)psi;
        auto* l = (float2*)lam;
        auto* t = (const float*)tab;
        if (dots)
            hipLaunchKernelGGL((k_apply_h_tiles<float, K, 512, C, true>), dim3(grid), dim3(512), 0, s, p, l, t, g.W, nt, pd, dots);
        else
            hipLaunchKernelGGL((k_apply_h_tiles<float, K, 512, C, false>), dim3(grid), dim3(512), 0, s, p, l, t, g.W, nt, pd, dots);
    } else {
        if (g.K != FL_KMAX_C128 || g.C != FL_LOWBITS) return hipErrorInvalidValue;
        constexpr int K = FL_KMAX_C128, C = FL_LOWBITS;
        auto* p = (const double2*)psi;
        auto* l = (double2*)lam;
        auto* t = (const double*)tab;
        if (dots)
            hipLaunchKernelGGL((k_apply_h_tiles<double, K, 256, C, true>), dim3(grid), dim3(256), 0, s, p, l, t, g.W, nt, pd, dots);
        else
            hipLaunchKernelGGL((k_apply_h_tiles<double, K, 256, C, false>), dim3(grid), dim3(256), 0, s, p, l, t, g.W, nt, pd, dots);
    }
    return hipGetLastError();
}

static bool adj_words(const fl_pass& pd, int gofs, fl_adj_words& w) {
    int n = pd.ngroups;
    for (int g = 0; g < pd.ngroups; ++g) n += pd.nops[g];
    if (n + 1 > FL_SWEEP_WORDS) return false;
    w.h = pd.h;
    w.ngroups = pd.ngroups;
    w.nslots = pd.nslots;
    for (int k = 0; k < FL_MAX_SLOTS; ++k) w.sbond[k] = pd.sbond[k];
    n = 0;
    for (int g = 0; g < pd.ngroups; ++g) w.w[n++] = (uint32_t)pd.u0[g] | (uint32_t)pd.nops[g] << 8;
    for (int g = 0; g < pd.ngroups; ++g)
        for (int k = 0; k < pd.nops[g]; ++k)
            w.w[n++] = (uint32_t)pd.opi[g][k] | (uint32_t)pd.ops[g][k] << 8 | (uint32_t)(pd.opg[g][k] - gofs) << 16;
    w.w[n++] = 0;
    w.nwords = n;
    return true;
}

// The words form with one op per group, as quad_words.
static bool adj_quad_words(const fl_pass& pd, int gofs, fl_adj_words& w) {
    if (!adj_words(pd, gofs, w)) return false;
    int n = 0;
    for (int g = 0; g < pd.ngroups; ++g) n += pd.nops[g];
    if (2 * n > FL_SWEEP_WORDS) return false;
    int k = 0;
    for (int g = 0; g < pd.ngroups; ++g)
        for (int q = 0; q < pd.nops[g]; ++q, ++k) {
            w.w[k] = (uint32_t)pd.u0[g];
            w.w[n + k] = (uint32_t)pd.ops[g][q] << 8 | (uint32_t)(pd.opg[g][q] - gofs) << 16;
        }
    w.ngroups = n;
    w.nwords = 2 * n;
    return true;
}

template <typename T, int K, int C>
static hipError_t launch_adj_quads(const fl_geom& g, void* psi, void* lam, const void* gates, const fl_pass& pd,
                                   double* Mpart, int grid, hipStream_t s) {
    typedef typename CT<T>::c cplx;
    const int nb = g.L - 1;
    fl_adj_words w;
    if ((uint32_t)grid != ntiles_of(g) || !adj_quad_words(pd, nb, w)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_adjoint_quads<T, K, C>), dim3(grid), dim3(2 << (K - 2)), 0, s, (cplx*)psi, (cplx*)lam,
                       (const T*)gates + 32 * nb, g.W, w, Mpart, nb);
    return hipGetLastError();
}

template <typename T, int NT>
static hipError_t launch_adj_one(int L, void* psi, void* lam, const void* gates, const fl_adj_words& w, int reps,
                                 double* Mpart, hipStream_t s) {
    typedef typename CT<T>::c cplx;
    hipLaunchKernelGGL((k_adjoint_one<T, NT>), dim3(1), dim3(NT), 0, s, (cplx*)psi, (cplx*)lam,
                       (const T*)gates + 32 * (L - 1), L, w, reps, Mpart);
    return hipGetLastError();
}

template <typename T, int R, int K, int C, int WPE, typename D>
static hipError_t launch_adj_tiles(const fl_geom& g, void* psi, void* lam, const void* gates, const fl_pass& pd,
                                   double* Mpart, int grid, hipStream_t s) {
    typedef typename CT<T>::c cplx;
    constexpr int NT = 1 << (K - R);
    const int nb = g.L - 1;
    const T* G = (const T*)gates + 32 * nb;   // G^dagger
    if constexpr (std::is_same<D, fl_adj_words>::value) {
        fl_adj_words w;
        if (!adj_words(pd, nb, w)) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_adjoint_tiles<T, R, K, NT, C, WPE, D>), dim3(grid), dim3(NT), 0, s, (cplx*)psi, (cplx*)lam,
                           G, g.W, ntiles_of(g), w, Mpart, nb);
    } else {
        hipLaunchKernelGGL((k_adjoint_tiles<T, R, K, NT, C, WPE, D>), dim3(grid), dim3(NT), 0, s, (cplx*)psi, (cplx*)lam,
                           G, g.W, ntiles_of(g), pd, Mpart, nb);
    }
    return hipGetLastError();
}

hipError_t launch_adjoint(int dtype, const fl_geom& g, void* psi, void* lam, const void* gates, const fl_pass& pd,
                          int reps, double* Mpart, int grid, hipStream_t s) {
    const int nb = g.L - 1;
    if (reps < 1 || (reps > 1 && g.W != 0)) return hipErrorInvalidValue;
    if (nb > FL_MAX_GATE_TABLE || grid < 1 || pd.nslots > FL_MAX_SLOTS) return hipErrorInvalidValue;
    for (int q = 0; q < pd.ngroups; ++q) {
        if (pd.nops[q] < 1) return hipErrorInvalidValue;
        for (int k = 0; k < pd.nops[q]; ++k)
            if (pd.opg[q][k] < nb || pd.opg[q][k] >= 2 * nb || pd.ops[q][k] < 0 || pd.ops[q][k] >= pd.nslots)
                return hipErrorInvalidValue;
    }
    if (g.W == 0) {
        fl_adj_words w;
        if (g.L < 2 || g.L > FL_KMAX_ONE || g.R != 2 || !adj_quad_words(pd, nb, w)) return hipErrorInvalidValue;
        if (dtype == 0)
            return g.L <= 7   ? launch_adj_one<float, 64>(g.L, psi, lam, gates, w, reps, Mpart, s)
                   : g.L <= 9 ? launch_adj_one<float, 256>(g.L, psi, lam, gates, w, reps, Mpart, s)
                              : launch_adj_one<float, 512>(g.L, psi, lam, gates, w, reps, Mpart, s);
        return g.L <= 7   ? launch_adj_one<double, 64>(g.L, psi, lam, gates, w, reps, Mpart, s)
               : g.L <= 9 ? launch_adj_one<double, 256>(g.L, psi, lam, gates, w, reps, Mpart, s)
                          : launch_adj_one<double, 512>(g.L, psi, lam, gates, w, reps, Mpart, s);
    }
    // the geometries of adjoint_geom
    const int key = (dtype << 12) | (g.K << 8) | (g.C << 4) | g.R;
    auto code = [](int dt, int K, int C, int R) { return (dt << 12) | (K << 8) | (C << 4) | R; };
    if (key == code(0, 12, 4, 4)) return launch_adj_tiles<float, 4, 12, 4, 2, fl_pass>(g, psi, lam, gates, pd, Mpart, grid, s);
    if (key == code(0, 12, 4, 3)) return launch_adj_tiles<float, 3, 12, 4, 2, fl_adj_words>(g, psi, lam, gates, pd, Mpart, grid, s);
    if (key == code(0, 11, 3, 2)) return launch_adj_quads<float, 11, 3>(g, psi, lam, gates, pd, Mpart, grid, s);
    if (key == code(0, 10, 3, 2)) return launch_adj_quads<float, 10, 3>(g, psi, lam, gates, pd, Mpart, grid, s);
    if (key == code(0, 9, 3, 2)) return launch_adj_quads<float, 9, 3>(g, psi, lam, gates, pd, Mpart, grid, s);
    if (key == code(1, 12, 4, 4)) return launch_adj_tiles<double, 4, 12, 4, 1, fl_pass>(g, psi, lam, gates, pd, Mpart, grid, s);
    if (key == code(1, 11, 3, 3)) return launch_adj_tiles<double, 3, 11, 3, 1, fl_adj_words>(g, psi, lam, gates, pd, Mpart, grid, s);
    if (key == code(1, 10, 3, 2)) return launch_adj_quads<double, 10, 3>(g, psi, lam, gates, pd, Mpart, grid, s);
    if (key == code(1, 9, 3, 2)) return launch_adj_quads<double, 9, 3>(g, psi, lam, gates, pd, Mpart, grid, s);
    return hipErrorInvalidValue;
}

hipError_t launch_adjoint_win4(const fl_geom& g, void* psi, void* lam, const void* mats, const fl_pass& pd,
                               double* Qpart, int grid, double* Qsum, hipStream_t s) {
    if (g.K != FL_KMAX_C64 || g.R != 4 || g.C != FL_DENSE4_LOWBITS || g.C + g.W != FL_KMAX_C64 ||
        pd.ngroups > FL_WIN4_MAX_GROUPS || grid < 1)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_adjoint_win4, dim3(grid), dim3(FL_WIN4_NT), 0, s, (float2*)psi, (float2*)lam,
                       (const float4*)mats, g.W, ntiles_of(g), pd, Qpart);
    const int nvals = pd.ngroups * 512;
    if (nvals > 0) hipLaunchKernelGGL(k_qsum, dim3((nvals + 31) / 32), dim3(256), 0, s, Qpart, grid, nvals, Qsum);
    return hipGetLastError();
}

hipError_t launch_zero(double* p, uint64_t n, hipStream_t s) {
    const uint64_t want = (n + 255) / 256;
    const unsigned grid = (unsigned)(want < 4096 ? (want ? want : 1) : 4096);
    hipLaunchKernelGGL(k_zero, dim3(grid), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_dense4(const fl_geom& g, void* psi, const void* mats, const fl_pass& pd, hipStream_t s) {
    if (g.C + g.W != 13) return hipErrorInvalidValue;
    if (g.W == 0) {
        // a single 13-bit tile (L = 13): the same amplitudes as low bits
        // [0, C) plus the window [C, 13), the kernel's fixed geometry
        fl_pass p = pd;
        p.h = FL_DENSE4_LOWBITS;
        hipLaunchKernelGGL(k_dense4<FL_DENSE4_NW>, dim3(1), dim3(64 * FL_DENSE4_NW), 0, s, (float2*)psi,
                           (const float4*)mats, 13 - FL_DENSE4_LOWBITS, p);
        return hipGetLastError();
    }
    if (g.C != FL_DENSE4_LOWBITS) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_dense4<FL_DENSE4_NW>, dim3(ntiles_of(g)), dim3(64 * FL_DENSE4_NW), 0, s, (float2*)psi,
                       (const float4*)mats, g.W, pd);
    return hipGetLastError();
}

hipError_t launch_dense6(int mode, const fl_geom& g, void* psi, const void* mats, const fl_pass& pd, hipStream_t s) {
    const uint32_t nt = ntiles_of(g);
    const bool full = g.C + g.W == 13;
    if (mode == 0 && full)
        hipLaunchKernelGGL((k_dense6<0, true>), dim3(nt), dim3(256), 0, s, (float2*)psi, (const float4*)mats, nt, g.C,
                           g.W, pd);
    else if (mode == 0)
        hipLaunchKernelGGL((k_dense6<0, false>), dim3(nt), dim3(256), 0, s, (float2*)psi, (const float4*)mats, nt, g.C,
                           g.W, pd);
    else if (full)
        hipLaunchKernelGGL((k_dense6<1, true>), dim3(nt), dim3(256), 0, s, (float2*)psi, (const float4*)mats, nt, g.C,
                           g.W, pd);
    else
        hipLaunchKernelGGL((k_dense6<1, false>), dim3(nt), dim3(256), 0, s, (float2*)psi, (const float4*)mats, nt, g.C,
                           g.W, pd);
    return hipGetLastError();
}

}  // namespace fl
