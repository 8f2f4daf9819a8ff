// Device code shared by the kernel files of libadasum: storage types and granules, streaming loads and
// stores, wave sums, the tile split, and the walk of the tree's scalars over a Gram matrix.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "adasum_host.h"

// Whether streaming loads / stores carry the non-temporal hint (compile-time knobs).
#ifndef ADASUM_NT_LOAD
#define ADASUM_NT_LOAD 1
#endif
#ifndef ADASUM_NT_STORE
#define ADASUM_NT_STORE 1
#endif

namespace adasum {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

struct bf16_t { unsigned short v; };
struct f16_t { unsigned short v; };   // IEEE binary16
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));

// VEC: elements per 16-byte granule; acc_t: the type lanes compute in (fp64 storage is
// reduced in fp64 throughout, everything else in fp32 lanes with fp64 above the wave)
template <typename T> struct Traits;
template <> struct Traits<float>  { static constexpr int VEC = 4; typedef float acc_t; };
template <> struct Traits<bf16_t> { static constexpr int VEC = 8; typedef float acc_t; };
template <> struct Traits<f16_t>  { static constexpr int VEC = 8; typedef float acc_t; };
template <> struct Traits<double> { static constexpr int VEC = 2; typedef double acc_t; };

__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

// round to nearest even; NaN stays NaN (quiet), overflow rounds to infinity
__device__ __forceinline__ unsigned int f32_to_bf16_rne(float f) {
    unsigned int u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x0040u;
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}

// G consecutive elements of T held as raw 32-bit words (8, 16 or 32 bytes)
template <typename T, int G>
struct Granule {
    static constexpr int NW = G * (int)sizeof(T) / 4;
    static_assert(NW == 2 || NW == 4 || NW == 8, "granule must be 8, 16 or 32 bytes");
    unsigned int w[NW];
};

template <typename V>
__device__ __forceinline__ V stream_load(const V* p) {
#if ADASUM_NT_LOAD
    return __builtin_nontemporal_load(p);
#else
    return *p;
#endif
}

template <bool NT, typename V>
__device__ __forceinline__ void stream_store(V v, V* p) {
    if constexpr (NT && ADASUM_NT_STORE) {
        __builtin_nontemporal_store(v, p);
    } else {
        *p = v;
    }
}

// p must be aligned to the granule size (to 16 bytes for a 32-byte granule)
template <typename T, int G>
__device__ __forceinline__ void load_raw(Granule<T, G>& r, const T* p) {
    constexpr int NW = Granule<T, G>::NW;
    if constexpr (NW == 2) {
        const u32x2 q = stream_load(reinterpret_cast<const u32x2*>(p));
        r.w[0] = q.x;
        r.w[1] = q.y;
    } else {
#pragma unroll
        for (int i = 0; i < NW / 4; ++i) {
            const u32x4 q = stream_load(reinterpret_cast<const u32x4*>(p) + i);
            r.w[4 * i + 0] = q.x;
            r.w[4 * i + 1] = q.y;
            r.w[4 * i + 2] = q.z;
            r.w[4 * i + 3] = q.w;
        }
    }
}

template <int G>
__device__ __forceinline__ void unpack(const Granule<float, G>& r, float (&v)[G]) {
#pragma unroll
    for (int i = 0; i < G; ++i) v[i] = __uint_as_float(r.w[i]);
}

template <int G>
__device__ __forceinline__ void unpack(const Granule<bf16_t, G>& r, float (&v)[G]) {
#pragma unroll
    for (int i = 0; i < G / 2; ++i) {
        v[2 * i + 0] = __uint_as_float(r.w[i] << 16);
        v[2 * i + 1] = __uint_as_float(r.w[i] & 0xffff0000u);
    }
}

template <int G>
__device__ __forceinline__ void unpack(const Granule<f16_t, G>& r, float (&v)[G]) {
#pragma unroll
    for (int i = 0; i < G / 2; ++i) {
        const f16x2_t h = __builtin_bit_cast(f16x2_t, r.w[i]);
        v[2 * i + 0] = static_cast<float>(h.x);
        v[2 * i + 1] = static_cast<float>(h.y);
    }
}

template <int G>
__device__ __forceinline__ void unpack(const Granule<double, G>& r, double (&v)[G]) {
#pragma unroll
    for (int i = 0; i < G; ++i)
        v[i] = __longlong_as_double((static_cast<long long>(r.w[2 * i + 1]) << 32) |
                                    static_cast<long long>(r.w[2 * i]));
}

// fp32 -> binary16, round to nearest even (the conversion instruction's default mode)
__device__ __forceinline__ unsigned int f32_to_f16_bits(float f) {
    const _Float16 h = static_cast<_Float16>(f);
    return static_cast<unsigned int>(__builtin_bit_cast(unsigned short, h));
}

template <bool NT, int NW>
__device__ __forceinline__ void store_words(void* p, const unsigned int (&w)[NW]) {
    if constexpr (NW == 2) {
        u32x2 q;
        q.x = w[0];
        q.y = w[1];
        stream_store<NT>(q, reinterpret_cast<u32x2*>(p));
    } else {
#pragma unroll
        for (int i = 0; i < NW / 4; ++i) {
            u32x4 q;
            q.x = w[4 * i + 0];
            q.y = w[4 * i + 1];
            q.z = w[4 * i + 2];
            q.w = w[4 * i + 3];
            stream_store<NT>(q, reinterpret_cast<u32x4*>(p) + i);
        }
    }
}

template <bool NT, int G>
__device__ __forceinline__ void store_granule(float* p, const float (&v)[G]) {
    unsigned int w[G];
#pragma unroll
    for (int i = 0; i < G; ++i) w[i] = __float_as_uint(v[i]);
    store_words<NT>(p, w);
}

template <bool NT, int G>
__device__ __forceinline__ void store_granule(bf16_t* p, const float (&v)[G]) {
    unsigned int w[G / 2];
#pragma unroll
    for (int i = 0; i < G / 2; ++i) w[i] = f32_to_bf16_rne(v[2 * i]) | (f32_to_bf16_rne(v[2 * i + 1]) << 16);
    store_words<NT>(p, w);
}

template <bool NT, int G>
__device__ __forceinline__ void store_granule(f16_t* p, const float (&v)[G]) {
    unsigned int w[G / 2];
#pragma unroll
    for (int i = 0; i < G / 2; ++i) w[i] = f32_to_f16_bits(v[2 * i]) | (f32_to_f16_bits(v[2 * i + 1]) << 16);
    store_words<NT>(p, w);
}

template <bool NT, int G>
__device__ __forceinline__ void store_granule(double* p, const double (&v)[G]) {
    unsigned int w[2 * G];
#pragma unroll
    for (int i = 0; i < G; ++i) {
        const long long b = __double_as_longlong(v[i]);
        w[2 * i] = static_cast<unsigned int>(b);
        w[2 * i + 1] = static_cast<unsigned int>(b >> 32);
    }
    store_words<NT>(p, w);
}

__device__ __forceinline__ double load_elem(const double* p) { return *p; }
__device__ __forceinline__ void store_elem(double* p, double v) { *p = v; }
__device__ __forceinline__ float load_elem(const float* p) { return *p; }
__device__ __forceinline__ float load_elem(const f16_t* p) {
    return static_cast<float>(__builtin_bit_cast(_Float16, p->v));
}
__device__ __forceinline__ void store_elem(f16_t* p, float v) {
    p->v = static_cast<unsigned short>(f32_to_f16_bits(v));
}
__device__ __forceinline__ float load_elem(const bf16_t* p) {
    return __uint_as_float(static_cast<unsigned int>(p->v) << 16);
}
__device__ __forceinline__ void store_elem(float* p, float v) { *p = v; }
__device__ __forceinline__ void store_elem(bf16_t* p, float v) {
    p->v = static_cast<unsigned short>(f32_to_bf16_rne(v));
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

// x of the lane N places on in the same row of 16 lanes, round the row.  (Adding what is turned by 8, 4, 2 and 1 in this order
// gives every lane the row's sum, with the bits of __shfl_xor by 8, 4, 2 and 1, without a trip through LDS for each.)
template <int N>
__device__ __forceinline__ double turned(double x) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(b), 0x120 + N, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(b >> 32), 0x120 + N, 0xf, 0xf, true);
    return __longlong_as_double(static_cast<long long>(hi) << 32 | static_cast<long long>(static_cast<unsigned>(lo)));
}
// x of the lane whose number differs in bit N (1 or 2).
template <int N>
__device__ __forceinline__ double swapped(double x) {
    constexpr int kOrder = N == 1 ? 0xb1 : 0x4e;   // 1 0 3 2 and 2 3 0 1 of every four lanes
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(b), kOrder, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(b >> 32), kOrder, 0xf, 0xf, true);
    return __longlong_as_double(static_cast<long long>(hi) << 32 | static_cast<long long>(static_cast<unsigned>(lo)));
}
// The sum over each run of N = 1, 4, 16 or 64 lanes, in every lane of it, with the bits of __shfl_xor by N / 2 .. 1.
template <int N>
__device__ __forceinline__ double run_of_lanes_sum(double v) {
    static_assert(N == 1 || N == 4 || N == 16 || N == 64, "");
    if constexpr (N == 64) {
        v += __shfl_xor(v, 32, 64);
        v += __shfl_xor(v, 16, 64);
    }
    if constexpr (N >= 16) {
        v += turned<8>(v);
        v += turned<4>(v);
    }
    if constexpr (N >= 4) {
        v += swapped<2>(v);
        v += swapped<1>(v);
    }
    return v;
}
__device__ __forceinline__ double of_lane(double x, int lane) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane(static_cast<int>(b), lane), hi = __builtin_amdgcn_readlane(static_cast<int>(b >> 32), lane);
    return __longlong_as_double(static_cast<long long>(hi) << 32 | static_cast<long long>(static_cast<unsigned>(lo)));
}

// Sums every one of N per-lane values over the 64 lanes of a wave with N + N/2 + ... shuffles
// instead of 6 N: at the step with mask m a lane whose bit m is clear keeps the even-indexed
// values and hands the odd-indexed ones to its partner (and the other way round), so each step
// halves the number of values a lane carries.  On return lane l holds in v[i] the complete sum
// of value number l + 64 i (values past N are padding).  Fixed order: bit-identical reruns.
template <typename A, int N>
__device__ __forceinline__ void wave_sum_scatter(A (&v)[N], int lane) {
    static_assert(N >= 1, "");
    int n = N;
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        const bool upper = (lane & m) != 0;
        const int half = (n + 1) / 2;
#pragma unroll
        for (int i = 0; i < (N + 1) / 2; ++i) {
            if (i < half) {
                const A a = v[2 * i];
                const A b = (2 * i + 1 < n) ? v[2 * i + 1] : static_cast<A>(0);
                const A keep = upper ? b : a, send = upper ? a : b;
                v[i] = keep + __shfl_xor(send, m, 64);
            }
        }
        n = half;
    }
}

template <int R>
__device__ __forceinline__ const void* operand_ptr(const Operands& ops, int g, int r) {
    return ops.pack[g * R + r];
}

// The tile split every kernel uses: [start, hs) scalar head, [bs, be) whole
// granules aligned to G elements of the global index, [ts, end) scalar tail.
struct Split {
    long long start, end, bs, hs, ts;
    int ng, nh, nt;
};

template <int G>
__device__ __forceinline__ Split split_tile(const adasum_tile& t) {
    Split s;
    s.start = t.start;
    s.end = t.start + t.len;
    s.bs = (s.start + (G - 1)) / G * G;
    const long long be = s.end / G * G;
    s.hs = s.bs < s.end ? s.bs : s.end;
    s.ts = be > s.hs ? be : s.hs;
    s.ng = be > s.bs ? static_cast<int>((be - s.bs) / G) : 0;
    s.nh = static_cast<int>(s.hs - s.start);
    s.nt = static_cast<int>(s.end - s.ts);
    return s;
}

// Entry e of the Gram kernel's order -> (i, j).
template <int R, bool DIAG>
__device__ __forceinline__ void entry_to_ij(int e, int& i, int& j) {
    i = 0;
    int rowlen = DIAG ? R : R - 1;
    while (e >= rowlen) {
        e -= rowlen;
        ++i;
        --rowlen;
    }
    j = (DIAG ? i : i + 1) + e;
}

// The tree's weights from one Gram matrix, computed by one wave (64 lanes): every node of
// the tree is a combination of its leaves, node = sum_p w_p x_p; for two sibling nodes A and
// B the operator of Section 3 needs d = A.B = sum_{p in A, q in B} w_p w_q G_pq, n1 = |A|^2,
// n2 = |B|^2 (quadratic forms whose terms are spread over the lanes and summed in a fixed
// order) and scales A's weights by 1 - d/(2 n1), B's by 1 - d/(2 n2); a zero squared norm
// gives coefficient 1.  G and w live in LDS; r leaves are real, the rest get weight 0.
template <int R>
__device__ __forceinline__ double wave_quadratic(const double* G, const double* w, int a0, int a1, int b0, int b1,
                                                 int lane) {
    const int nb = b1 - b0, n = (a1 - a0) * nb;
    double v = 0.0;
    for (int i = lane; i < n; i += 64) {
        const int p = a0 + i / nb, q = b0 + i % nb;
        v += w[p] * w[q] * G[p * R + q];
    }
    return wave_sum(v);
}

template <int R>
__device__ __forceinline__ void wave_merge(const double* G, double* w, int a0, int a1, int b0, int b1, int lane) {
    const double n1 = wave_quadratic<R>(G, w, a0, a1, a0, a1, lane);
    const double n2 = wave_quadratic<R>(G, w, b0, b1, b0, b1, lane);
    const double d = wave_quadratic<R>(G, w, a0, a1, b0, b1, lane);
    const double ca = n1 > 0.0 ? 1.0 - d / (2.0 * n1) : 1.0;
    const double cb = n2 > 0.0 ? 1.0 - d / (2.0 * n2) : 1.0;
    if (lane >= a0 && lane < a1) w[lane] *= ca;
    if (lane >= b0 && lane < b1) w[lane] *= cb;
}

template <int R>
__device__ __forceinline__ void wave_tree_weights(const double* G, double* w, int r, int order, int lane) {
    if (lane < R) w[lane] = lane < r ? 1.0 : 0.0;
    if (order == ADASUM_ORDER_LINEAR) {
        for (int k = 1; k < r; ++k) wave_merge<R>(G, w, 0, k, k, k + 1, lane);
        return;
    }
    // the halving tree over r leaves, deepest nodes first: children before parents
    int levels = 0;
    while ((1 << levels) < r) ++levels;
    for (int d = levels - 1; d >= 0; --d) {
        for (int j = 0; j < (1 << d); ++j) {
            int lo, hi;
            leaf_range(r, d, j, lo, hi);
            if (hi - lo >= 2) {
                const int mid = lo + (hi - lo) / 2;
                wave_merge<R>(G, w, lo, mid, mid, hi, lane);
            }
        }
    }
}

// The same walk for the balanced tree over R = 2, 4, 8 or 16 leaves, a whole depth at a time: the terms of all
// quadratic forms of a depth are spread over the lanes (4 s^2 slots per node with s leaves a side: the left
// norm, the right norm, the dot product, an empty quarter) and summed in the order wave_merge sums them.
// q: LDS scratch of 2 R doubles.  (A sum over up to 16 lanes takes no trips through LDS: K = 16 bf16, ResNet-50 sizes, 237 us
// instead of 241, K = 8 fp32 190.5 instead of 192.)
template <int R, int S = 1>
__device__ __forceinline__ void wave_balanced_weights(const double* G, double* w, double* q, int lane) {
    if constexpr (S == 1) {
        if (lane < R) w[lane] = 1.0;
    }
    if constexpr (S < R) {
        constexpr int sq = S * S;
        // (the last of the four is empty: where a run of 64 lanes is one form's, there is none for it)
        constexpr int kSlots = sq == 64 ? 3 * 64 * (R / (2 * S)) : 2 * R * S;
#pragma unroll
        for (int base = 0; base < kSlots; base += 64) {
            const int slot = base + lane;
            const int what = slot / sq % 4, node = slot / (4 * sq), term = slot % sq;
            const int left = node * 2 * S;
            const int a = (what == 1 ? left + S : left) + term / S, b = (what == 0 ? left : left + S) + term % S;
            double v = 0.0;
            if (slot < kSlots && what < 3) v = w[a] * w[b] * G[a * R + b];
            v = run_of_lanes_sum<sq < 64 ? sq : 64>(v);
            if (slot < kSlots && term == 0) q[slot / sq] = v;
        }
        if (lane < R) {
            const int node = lane / (2 * S);
            const double n1 = q[4 * node], n2 = q[4 * node + 1], d = q[4 * node + 2];
            const double ca = n1 > 0.0 ? 1.0 - d / (2.0 * n1) : 1.0;
            const double cb = n2 > 0.0 ? 1.0 - d / (2.0 * n2) : 1.0;
            w[lane] *= lane % (2 * S) < S ? ca : cb;
        }
        wave_balanced_weights<R, 2 * S>(G, w, q, lane);
    }
}

// The same for the halving tree over any r leaves, R - 1 <= r <= R <= 16 and r > 8 if R > 8: the three forms of a
// depth's nodes are worked out side by side by equal runs of lanes, each summed in a fixed order.  About 0.4 us a
// depth, where wave_tree_weights takes 0.5 us a node.  q: LDS scratch of 4 R doubles.
template <int R>
__device__ __forceinline__ void wave_level_weights(const double* G, double* w, double* q, int r, int lane) {
    static_assert(R >= 2 && R <= 16, "");
    constexpr int LEVELS = R > 8 ? 4 : R > 4 ? 3 : R > 2 ? 2 : 1;
    static_assert((4 << (LEVELS - 1)) <= 4 * R, "a slot of q per form");
    if (lane < R) w[lane] = lane < r ? 1.0 : 0.0;
    for (int d = LEVELS - 1; d >= 0; --d) {
        const int run = 16 >> d;                    // lanes per form: 64 / (4 * 2^d)
        const int slot = lane / run, i = lane % run;
        const int node = slot / 4, what = slot % 4;
        int lo, hi;
        leaf_range(r, d, node, lo, hi);
        const int mid = lo + (hi - lo) / 2;
        const int a0 = what == 1 ? mid : lo, a1 = what == 1 ? hi : mid;
        const int b0 = what == 0 ? lo : mid, b1 = what == 0 ? mid : hi;
        const int side = (R + (2 << d) - 1) / (2 << d);   // leaves a side has at most
        const bool real = what < 3 && hi - lo >= 2;
        double v = 0.0;
        int a = a0 + i / side, b = i % side;              // (term i, then every run-th one)
        for (int k = i; k < side * side; k += run) {
            if (real && a < a1 && b0 + b < b1) v += w[a] * w[b0 + b] * G[a * R + b0 + b];
            for (b += run; b >= side; b -= side) ++a;
        }
        for (int m = run / 2; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
        if (i == 0) q[slot] = v;
        if (lane < r) {
            // the node of this depth that holds leaf `lane`
            int l0 = 0, l1 = r, j = 0;
            for (int b = 0; b < d; ++b) {
                const int m = l0 + (l1 - l0) / 2;
                j = 2 * j + (lane >= m ? 1 : 0);
                if (lane >= m) l0 = m; else l1 = m;
            }
            if (l1 - l0 >= 2) {
                const int m = l0 + (l1 - l0) / 2;
                const double n1 = q[4 * j], n2 = q[4 * j + 1], dd = q[4 * j + 2];
                const double ca = n1 > 0.0 ? 1.0 - dd / (2.0 * n1) : 1.0;
                const double cb = n2 > 0.0 ? 1.0 - dd / (2.0 * n2) : 1.0;
                w[lane] *= lane < m ? ca : cb;
            }
        }
    }
}

}  // namespace
}  // namespace adasum
