// The resident pass (gfx950): a pass whose layers fit on the chip reads its operands ONCE.  A workgroup loads a unit
// (a run of consecutive elements of one layer, all operands), keeps it in registers and LDS, sends its
// partial Gram entries to the other workgroups of the layer, gets the layer's whole Gram matrix back, walks the tree's
// scalars and combines from what it kept.  One launch takes the place of gram_kernel, gram_finish_kernel and
// combine_kernel, and operands that those read twice cross the fabric between the memory and the compute dies once.
//
// Its layers of some waves of units need the chip for themselves: beside other kernels units wait longer for each other,
// and some give up (see redo_units).  Measured beside 8192^3 bf16 matrix products, copies of 1 GB and small
// products (512 x 4096 x 4096) on another stream, us per reduction, three kernels in brackets: ResNet-50 sizes, K = 2 bf16 1200
// (1580), 67 (95), 55 (66); K = 8 fp32 1009 (2436), 333 (500), 441 (320); K = 16 bf16 1126 (2221), 890 (507), 337 (352); a
// quarter of them, K = 8 bf16, 842 (3002), 74 (128), 56 (96).  So programs that reduce large models of 8 and more workers
// beside small or streaming kernels are better off with separate_passes.
//
// What bounds it.  Re-reading is what the three kernels lose: the Infinity Cache gives a compute die no more bandwidth
// than memory does (7.1 TB/s, measured on 64 .. 256 MB re-read in a loop against 7.0 TB/s fresh), so bytes have to stay
// in registers and LDS to be saved.  The chip holds some 110 MB there, about 15 us of memory traffic; a unit lives
// through its loads (5 .. 16 us: a compute unit alone loads some 33 GB/s, 229 KB in 7 us, so memory is full only while nearly
// all of them load), the exchange (4 .. 10 us: two trips through memory under load, and waiting for the layer's slowest
// unit), the scalars (1 us) and its stores.  So the pass is bound by how much is kept over how long:
// hence as much as the register file takes per unit, LDS filled straight from memory beside it, an exchange without
// atomics, flags or fences (a fence of agent scope cost 1.4 x the whole pass), and launch order (order_units).
// Measured against the three kernels, us per reduction: ResNet-50 sizes, K = 8 fp32 298 -> 190, K = 2 bf16 51 -> 36,
// K = 6 binary16 152 -> 88, K = 16 bf16 with statistics 316 -> 215; 400 odd tensors, K = 12 bf16, 182 -> 83.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "adasum_host.h"
#include "adasum_device.h"
#include "adasum_outcome.h"

namespace adasum {
namespace {

template <typename T> struct DtypeOf;
template <> struct DtypeOf<float> { enum { value = ADASUM_F32 }; };
template <> struct DtypeOf<bf16_t> { enum { value = ADASUM_BF16 }; };
template <> struct DtypeOf<f16_t> { enum { value = ADASUM_F16 }; };
template <> struct DtypeOf<double> { enum { value = ADASUM_F64 }; };

// element k of some 32-bit words of T, widened to the type lanes compute in
template <typename T> __device__ __forceinline__ typename Traits<T>::acc_t element(const unsigned int* w, int k) {
    if constexpr (std::is_same<T, float>::value) return __uint_as_float(w[k]);
    else if constexpr (std::is_same<T, bf16_t>::value)
        return __uint_as_float((k & 1) ? (w[k / 2] & 0xffff0000u) : (w[k / 2] << 16));
    else if constexpr (std::is_same<T, f16_t>::value) {
        const f16x2_t h = __builtin_bit_cast(f16x2_t, w[k / 2]);
        return static_cast<float>((k & 1) ? h.y : h.x);
    } else {
        return __longlong_as_double((static_cast<long long>(w[2 * k + 1]) << 32) | static_cast<long long>(w[2 * k]));
    }
}

// The rows and columns of the Gram entries (i <= j), row by row.
template <int R>
struct Entries {
    int row[R * (R + 1) / 2], col[R * (R + 1) / 2];
    constexpr Entries() : row(), col() {
        int e = 0;
        for (int i = 0; i < R; ++i)
            for (int j = i; j < R; ++j) {
                row[e] = i;
                col[e] = j;
                ++e;
            }
    }
};
template <int R> constexpr Entries<R> kEntries{};

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
// X X^T of 16 rows of 32 elements, added to c
template <typename T>
__device__ __forceinline__ f32x4_t mfma_square(const u32x4& x, const f32x4_t& c) {
    if constexpr (std::is_same<T, bf16_t>::value) {
        const bf16x8_t v = __builtin_bit_cast(bf16x8_t, x);
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, v, c, 0, 0, 0);
    } else {
        const f16x8_t v = __builtin_bit_cast(f16x8_t, x);
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(v, v, c, 0, 0, 0);
    }
}

// ---- values that one workgroup of a launch writes and others read ----
// A double travels as two 8-byte words, each with half of its bits and the call's tag: a reader knows from the word
// itself whether it was written in this call, so there are no flags, no counters and nothing to wait for between a
// value and its announcement.  Both words go in one 16-byte access (a tag for each half, so it need not be atomic), past
// the compute dies' own caches.
constexpr int kPastCaches = 16;   // (the sc1 bit: agent scope)
typedef __amdgpu_buffer_rsrc_t buffer_t;
__device__ __forceinline__ buffer_t buffer_of(const void* base, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}
__device__ __forceinline__ void send(buffer_t b, int offset, double v, unsigned tag) {
    const unsigned long long bits = static_cast<unsigned long long>(__double_as_longlong(v));
    u32x4 w;
    w.x = static_cast<unsigned>(bits);
    w.y = tag;
    w.z = static_cast<unsigned>(bits >> 32);
    w.w = tag;
    __builtin_amdgcn_raw_buffer_store_b128(w, b, offset, 0, kPastCaches);
}
__device__ __forceinline__ u32x4 peek(buffer_t b, int offset) { return __builtin_amdgcn_raw_buffer_load_b128(b, offset, 0, kPastCaches); }
__device__ __forceinline__ bool tagged(const u32x4& w, unsigned tag) { return w.y == tag && w.w == tag; }
__device__ __forceinline__ double value(const u32x4& w) {
    return __longlong_as_double(static_cast<long long>(w.z) << 32 | static_cast<long long>(w.x));
}
// Looks at N values side by side, and at all of them again until they are there or `more` says no (false).  (One after another,
// each that was late would take a trip through memory of its own.)
template <int N, typename More>
__device__ __forceinline__ bool await(buffer_t b, const int (&offset)[N], u32x4 (&w)[N], unsigned tag, More&& more) {
    for (;;) {
        bool there = true;
#pragma unroll
        for (int k = 0; k < N; ++k) w[k] = peek(b, offset[k]);
#pragma unroll
        for (int k = 0; k < N; ++k) there = there && tagged(w[k], tag);
        if (there) return true;
        if (!more()) return false;
        __builtin_amdgcn_s_sleep(2);
        asm volatile("" ::: "memory");   // (the next look is another)
    }
}
// The tag of a call: calls before it, and one, in the low bits of the word that counts them.  Above those bits the launch's last workgroups
// count themselves while it runs.
constexpr int kTagMask = 0xffffff, kArrival = kTagMask + 1;
__device__ __forceinline__ unsigned tag_of(int epoch) { return static_cast<unsigned>(epoch & kTagMask) + 1u; }

// Where entry e of the layer's unit number u lies (of W units, NP entries), in bytes: runs of kRun entries of every unit follow each
// other, so that the lanes that sum a run over the units read whole memory sectors.  (With the NP entries of a unit in one
// piece each lane's 16 bytes are a sector of their own, again with every look, and 136 waves of a layer look at 384 units:
// K = 16 bf16, ResNet-50 sizes, 271 us instead of 242, K = 8 fp32 207 instead of 190.)
constexpr int kRun = 4;
template <int NP>
__device__ __forceinline__ int partial_at(int u, int e, int W) {
    const int run = e / kRun * kRun;
    return (run * W + u * (NP - run < kRun ? NP - run : kRun) + (e - run)) * 16;
}
// A workgroup sums a run: kRun lanes side by side per unit, kRunUnits units at a time.
constexpr int kRunUnits = kThreads / kRun;
// Units of a layer up to which every workgroup reads all partial sums itself.  (K = 2 bf16, ResNet-50 sizes: 37.4 us with 4,
// 38.4 with 16, 40.7 with 170; K = 8 fp32 and K = 16 bf16 take the same with 4 to 32, 1.5 % longer with 2.  K = 2 of four types on 13
// tables, 10 to 109 us: 16 takes 0.95 to 1.06 times what 4 takes, 0.999 in the mean; small calls of one side differ by as much.
// ResNet-50 sizes: bf16 33.5 with 4 and 33.8 with 16, binary16 31.7 and 32.7, fp32 57.1 and 58.1, fp64 109.1 and 108.7.)
constexpr int direct_units(int R) { return R == 2 ? 4 : kDirectUnits; }
// the sum over the units of a wave; lanes 0 .. kRun - 1 hold the entries'
__device__ __forceinline__ double run_sum(double v) {
#pragma unroll
    for (int m = 32; m >= kRun; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

// Units a workgroup looks at that sees to those which gave up: 4, and more where the chip would not hold all such workgroups of a
// launch of their own at once (K = 16 bf16, ResNet-50 sizes, with nothing to do: 1080 of them 8.2 us, 512 4.8), or
// kArrival's place in its word has no room for them at the end of the launch itself.
constexpr int kRedoScan = 4, kRedoBlocks = 96;
constexpr int redo_per_cu(int R) { return R > 8 ? 2 : 4; }
// form 1, whose units are small
template <int SV, int SL> constexpr bool kRedoInLaunch = SV == 1 && SL == 0;
constexpr int kTicksPerUs = 100;         // of wall_clock64
// Looks that the last workgroups of a launch take at something that is on its way, more than a microsecond each.  Nothing that runs as
// it should comes near it.  (Counted in looks, not in time: while the chip is another process's they do not run out.)
constexpr int kMostLooks = 1 << 21;

// 16 bytes per lane straight from memory into LDS (lane l's at dst + 16 l; base: the same for all lanes): no registers are
// held meanwhile.  A buffer load: after a global_load_lds, which counts as a flat access, the compiler waits for every
// load in flight before it uses any.
[[maybe_unused]] __device__ __forceinline__ void load_to_lds(const void* base, unsigned offset, void* dst) {
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0x7fffffff, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)dst, 16, offset, 0, 0, 2 /* non-temporal */);
}

__device__ __forceinline__ unsigned long long same_for_all(unsigned long long v) {
    const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(v)));
    const unsigned hi = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(v >> 32)));
    return static_cast<unsigned long long>(hi) << 32 | lo;
}

// f(0), f(1), ... f(N - 1), each argument a constant of its own type
template <int N, typename F>
__device__ __forceinline__ void each(F&& f) {
    if constexpr (N > 0) {
        each<N - 1>(f);
        f(std::integral_constant<int, N - 1>());
    }
}

// ---- what is done with a layer's Gram matrix, by a unit and by those that redo it ----
// the weights (by one wave; the workgroup waits for these few instructions)
template <int R>
__device__ __forceinline__ void unit_weights(const double* shG, double* shW, double* shQ, int order, int leaves, int lane) {
    __builtin_amdgcn_s_setprio(3);
    if (order == ADASUM_ORDER_LINEAR) wave_tree_weights<R>(shG, shW, leaves, order, lane);
    else if ((R & (R - 1)) == 0 && leaves == R) wave_balanced_weights<R>(shG, shW, shQ, lane);
    else wave_level_weights<R>(shG, shW, shQ, leaves, lane);
    __builtin_amdgcn_s_setprio(0);
}

// the combine of one granule of every row (DELTA: the last row is `start`).  More than 8 rows of a 16-bit type are summed in
// two chains, the even-numbered and the odd-numbered ones, as the 16-operand combine of those types does: one chain puts a
// tenth more error on an fp32 result (K = 16, one layer of 2 million elements: 6.5e-8 against 5.7e-8).
template <typename TI, typename TO, int R, bool DELTA, bool NTS>
__device__ __forceinline__ void combine_granule(const Granule<TI, Traits<TI>::VEC> (&q)[R + (DELTA ? 1 : 0)],
                                                const typename Traits<TI>::acc_t (&w)[R], TO* out,
                                                typename Traits<TI>::acc_t& nacc) {
    constexpr int G = Traits<TI>::VEC;
    typedef typename Traits<TI>::acc_t acc_t;
    acc_t z[G];
#pragma unroll
    for (int k = 0; k < G; ++k) {
        acc_t sv = 0;
        if constexpr (DELTA) sv = element<TI>(q[R].w, k);
        z[k] = w[0] * (DELTA ? element<TI>(q[0].w, k) - sv : element<TI>(q[0].w, k));
        if constexpr (resident_matrix(DtypeOf<TI>::value, R)) {
            acc_t odd = w[1] * element<TI>(q[1].w, k);
#pragma unroll
            for (int r = 2; r < R; r += 2) {
                z[k] = fma_t(w[r], element<TI>(q[r].w, k), z[k]);
                odd = fma_t(w[r + 1], element<TI>(q[r + 1].w, k), odd);
            }
            z[k] += odd;
        } else {
#pragma unroll
            for (int r = 1; r < R; ++r)
                z[k] = fma_t(w[r], DELTA ? element<TI>(q[r].w, k) - sv : element<TI>(q[r].w, k), z[k]);
        }
        nacc = fma_t(z[k], z[k], nacc);
        if constexpr (DELTA) z[k] += sv;
    }
    store_granule<NTS>(out, z);
}

// one ragged head/tail element: fp64 arithmetic, one rounding at the store; its square is returned
template <typename TI, typename TO, int R, bool DELTA>
__device__ __forceinline__ double combine_ragged(const Operands& ops, const TI* start, const double* shW, TO* out, long long idx) {
    typedef typename Traits<TO>::acc_t out_acc_t;
    double sd = 0.0;
    if constexpr (DELTA) sd = static_cast<double>(load_elem(start + idx));
    double z = shW[0] * (static_cast<double>(load_elem(static_cast<const TI*>(ops.pack[0]) + idx)) - sd);
#pragma unroll
    for (int r = 1; r < R; ++r)
        z = __builtin_fma(shW[r], static_cast<double>(load_elem(static_cast<const TI*>(ops.pack[r]) + idx)) - sd, z);
    const out_acc_t zs = static_cast<out_acc_t>(z);
    if constexpr (DELTA) z += sd;
    store_elem(out + idx, static_cast<out_acc_t>(z));
    return static_cast<double>(zs) * static_cast<double>(zs);
}

// A layer of at most kSmallLayer elements, by the definition itself (as small_reduce_kernel, and with its bits): one wave, pair by
// pair in fp64 in the order of the recursion, nothing stored in between.  Lanes 16 j .. 16 j + 15 hold the layer's elements
// four times over, so that one sum over 16 lanes gives the dot product and both squared norms.  In launches of their own,
// one before the pass that copies these layers and one after it, they cost 18 us of 98 (400 odd tensors, K = 12 bf16), here 4.
// v: LDS, R x 16.  norm: where the squared norm of the result goes; gram: a matrix whose trace is the operands' squared norms
// summed (either or both null).
template <typename TI, typename TO, int R, bool DELTA>
__device__ __forceinline__ void small_unit(const Operands& ops, const TI* start, TO* out, long long first, int len, int order,
                                           int leaves, double (*v)[16], int lane, double* norm, double* gram) {
    const int e = lane & 15, what = lane >> 4;
    const bool live = e < len;
    const long long idx = first + (live ? e : 0);
    double base = 0.0;
    if constexpr (DELTA) base = static_cast<double>(load_elem(start + idx));
    double leafsq = 0.0;
#pragma unroll 8
    for (int k = 0; k < R; ++k) {
        double x = static_cast<double>(load_elem(static_cast<const TI*>(ops.pack[k]) + idx)) - base;
        x = live && k < leaves ? x : 0.0;
        leafsq = __builtin_fma(x, x, leafsq);
        if (what == 0) v[k][e] = x;
    }
    __builtin_amdgcn_wave_barrier();
    auto sum16 = [](double x) {
        x += turned<8>(x);
        x += turned<4>(x);
        x += turned<2>(x);
        return x + turned<1>(x);
    };
    auto pair = [&](double a, double b) {
        const double s = sum16(what == 0 ? a * b : what == 1 ? a * a : b * b);
        const double d = of_lane(s, 0), n1 = of_lane(s, 16), n2 = of_lane(s, 32);
        const double ca = n1 > 0.0 ? 1.0 - d / (2.0 * n1) : 1.0;
        const double cb = n2 > 0.0 ? 1.0 - d / (2.0 * n2) : 1.0;
        return ca * a + cb * b;
    };
    double r = v[0][e];
    int depth = 0;   // of the stack of finished sub-trees, kept where the leaves were
    for (int k = 1; k < leaves; ++k) {
        const double x = v[k][e];
        if (order == ADASUM_ORDER_LINEAR) {
            r = pair(r, x);
            continue;
        }
        v[depth++][e] = r;
        r = x;
        // as many merges as nodes of the halving tree end with leaf k
        for (int a = 0, b = leaves, merges = 0;;) {
            if (b - a < 2) {
                for (; merges > 0; --merges) r = pair(v[--depth][e], r);
                break;
            }
            if (b == k + 1) ++merges;
            const int mid = a + (b - a) / 2;
            if (k < mid) b = mid;
            else a = mid;
        }
    }
    const double rsq = sum16(r * r);
    leafsq = sum16(leafsq);
    if (lane == 0 && norm != nullptr) *norm = rsq;
    if (gram != nullptr && lane < R) gram[lane * (R + 1)] = lane == 0 ? leafsq : 0.0;   // (its trace is what is asked for)
    if (live && what == 0) store_elem(out + idx, static_cast<typename Traits<TO>::acc_t>(DELTA ? r + base : r));
}

// The block-th four of a table's small layers, a wave each.
template <typename TI, typename TO, int R, bool DELTA>
__device__ __forceinline__ void small_layers(const Operands& ops, TO* out, SmallTable small, int block, double* __restrict__ gram,
                                             double* __restrict__ normparts, const TI* start, int order, int leaves,
                                             double (*shSmall)[kSmallLayer]) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int i = block * (kThreads / 64) + wave;
    if (i >= small.n) return;
    const SmallLayer l = small.layers[i];
    double* norm = nullptr;
    if (normparts != nullptr) {   // (a layer may be cut into two units)
        norm = normparts + small.unit_begin[l.layer];
        if (small.unit_begin[l.layer + 1] - small.unit_begin[l.layer] > 1 && lane == 0) norm[1] = 0.0;
    }
    small_unit<TI, TO, R, DELTA>(ops, start, out, l.start, l.len, order, leaves, shSmall + wave * R, lane, norm,
                                 gram != nullptr ? gram + static_cast<long long>(l.layer) * (R * R) : nullptr);
}

// Units that gave up waiting, from memory, with the same arithmetic in the same order; and the tag moves on.  A workgroup
// (`first` of `step`) looks at every step-th unit: a layer's units follow each other and tend to give up together.
// SAME_LAUNCH: by the last workgroups of the launch itself, for reductions that the chip holds all at once in small units: a
// second launch costs 4 us of 19 there.  They wait for every unit's outcome: units are dispatched before them and end within their
// own limit whatever these do.  Where that does not hold -- calls that overlap in one memory, against the rule, clear each other's
// words -- they still end after kMostLooks, and units whose outcome or whose layer's sums are not there are made NaN.
template <typename TI, typename TO, int R, bool DELTA, bool SAME_LAUNCH>
__device__ __forceinline__ void redo_units(const Operands& ops, TO* out, const ResidentUnit* __restrict__ units, int n_units, int first,
                                           int step, const ResidentState& st, double* __restrict__ gram,
                                           double* __restrict__ normparts, const TI* start, int order, int leaves, double* shR,
                                           double* shG, double* shW, double* shQ, double* shNorm, unsigned long long* shTodo,
                                           int* shLate) {
    constexpr int G = Traits<TI>::VEC;
    constexpr int NP = R * (R + 1) / 2;
    constexpr int NW = kThreads / 64;
    constexpr int ROWS = kThreads / NP;
    constexpr int kDirect = direct_units(R);
    constexpr int RL = R + (DELTA ? 1 : 0);
    typedef typename Traits<TI>::acc_t acc_t;
    constexpr bool NTS = !(sizeof(TI) == 2 && sizeof(TO) == 4 && R <= 2);   // as combine_kernel
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned tag = SAME_LAUNCH ? tag_of(__hip_atomic_load(st.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) : 0u;
    int looks = kMostLooks;
    auto outcome = [&](int i) __attribute__((always_inline)) {
        if constexpr (!SAME_LAUNCH) return st.outcome[i] & 7;
        return await_outcome([&]() __attribute__((always_inline)) { return __hip_atomic_load(st.outcome + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); },
                             tag,
                             [&]() __attribute__((always_inline)) {
                                 __builtin_amdgcn_s_sleep(8);
                                 return --looks > 0;
                             });
    };
    if (SAME_LAUNCH && tid == 0) *shLate = 0;   // (long before anybody has looked in vain for the last time)
    int layer = -1;
    for (int i0 = first; i0 < n_units; i0 += step * kThreads) {
        const int mine = i0 + tid * step;
        const int what = mine < n_units ? outcome(mine) : static_cast<int>(kDone);
        const unsigned long long some = __ballot(SAME_LAUNCH ? what != kDone : what == kGaveUp);
        if (lane == 0) shTodo[wave] = some;
        if (SAME_LAUNCH && what == kOverdue) *shLate = 1;
        __syncthreads();
        if (tid == 0 && i0 + step * kThreads >= n_units) {
            if constexpr (!SAME_LAUNCH) {
                if (first == 0) *st.epoch = static_cast<int>(tag_of(*st.epoch) & kTagMask);
            } else if (*shLate || __hip_atomic_fetch_add(st.epoch, kArrival, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) / kArrival == step - 1) {
                // (the last of them to have seen its units' outcomes: all that read the tag have done so.  Late ones leave no arrivals
                // for the next call.)
                __hip_atomic_store(st.epoch, static_cast<int>(tag & kTagMask), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        for (int w0 = 0; w0 < NW; ++w0) for (unsigned long long todo = same_for_all(shTodo[w0]); todo != 0; todo &= todo - 1) {
            const int b = w0 * 64 + __builtin_ctzll(todo);
            const int at = i0 + b * step;
            const ResidentUnit t = units[at];
            adasum_tile tile;
            tile.start = t.start;
            tile.len = t.len;
            tile.layer = t.layer;
            const Split s = split_tile<G>(tile);
            const int W = t.layer_end - t.layer_first;
            bool late = false;
            if constexpr (SAME_LAUNCH)
                late = same_answer([&]() __attribute__((always_inline)) { return *shLate != 0; },
                                   []() __attribute__((always_inline)) { __syncthreads(); });
            if (t.layer != layer && !late) {   // (else its weights are there from the unit before)
                layer = t.layer;
                const buffer_t partials = buffer_of(st.partials + static_cast<long long>(t.layer_first) * (NP * 2), W * NP * 16);
                // the sum of entry e over the units u0, u0 + step, ... of the layer (which have all been sent, or will be)
                auto sum_units = [&](int e, int u0, int step) __attribute__((always_inline)) {
                    constexpr int kAhead = 4;
                    double v = 0.0;
                    for (; u0 < W; u0 += step * kAhead) {
                        int offset[kAhead];
                        u32x4 x[kAhead];
#pragma unroll
                        for (int k = 0; k < kAhead; ++k) offset[k] = partial_at<NP>(u0 + k * step < W ? u0 + k * step : W - 1, e, W);
                        if constexpr (SAME_LAUNCH) {
                            if (!await(partials, offset, x, tag, [&]() __attribute__((always_inline)) { return --looks > 0; })) *shLate = 1;
                        } else {
#pragma unroll
                            for (int k = 0; k < kAhead; ++k) x[k] = __builtin_amdgcn_raw_buffer_load_b128(partials, offset[k], 0, 0);
                        }
#pragma unroll
                        for (int k = 0; k < kAhead; ++k)
                            if (u0 + k * step < W) v += value(x[k]);
                    }
                    return v;
                };
                if (W <= kDirect) {
                    const int row = tid / NP, e = tid % NP;
                    if (row < ROWS) shR[row * NP + e] = sum_units(e, row, ROWS);
                    __syncthreads();
                    if (tid < NP) {
                        double tot = shR[tid];
#pragma unroll
                        for (int k = 1; k < ROWS; ++k) tot += shR[k * NP + tid];
                        int i, j;
                        entry_to_ij<R, true>(tid, i, j);
                        shG[i * R + j] = shG[j * R + i] = tot;
                    }
                } else {
                    for (int run = 0; run < NP; run += kRun) {
                        const int e = run + tid % kRun;
                        const double v = run_sum(sum_units(e < NP ? e : NP - 1, tid / kRun, kRunUnits));
                        if (lane < kRun) shR[wave * kRun + lane] = v;
                        __syncthreads();
                        if (tid < kRun && e < NP) {
                            double tot = shR[tid];
#pragma unroll
                            for (int w = 1; w < NW; ++w) tot += shR[w * kRun + tid];
                            int i, j;
                            entry_to_ij<R, true>(e, i, j);
                            shG[i * R + j] = shG[j * R + i] = tot;
                        }
                        __syncthreads();
                    }
                }
                __syncthreads();
                if (wave == 0) unit_weights<R>(shG, shW, shQ, order, leaves, lane);
                if (gram != nullptr && t.unit == t.layer_first)
                    for (int i = tid; i < R * R; i += kThreads) gram[static_cast<long long>(t.layer) * (R * R) + i] = shG[i];
                __syncthreads();
                if constexpr (SAME_LAUNCH) late = *shLate != 0;   // (no wave writes to it before all are at the next unit)
            }
            if (late) {
                const double nan = __builtin_nan("");
                for (int j = tid; j < t.len; j += kThreads) store_elem(out + t.start + j, static_cast<typename Traits<TO>::acc_t>(nan));
                if (tid == 0 && normparts != nullptr) normparts[t.unit] = nan;
                if (tid == 0 && gram != nullptr) gram[static_cast<long long>(t.layer) * (R * R)] = nan;
                continue;
            }
            acc_t w[R];
#pragma unroll
            for (int r = 0; r < R; ++r) w[r] = static_cast<acc_t>(shW[r]);
            acc_t nacc = 0;
            for (int j = tid; j < s.ng; j += kThreads) {
                const long long idx = s.bs + static_cast<long long>(j) * G;
                Granule<TI, G> q[RL];
#pragma unroll
                for (int r = 0; r < R; ++r) load_raw(q[r], static_cast<const TI*>(ops.pack[r]) + idx);
                if constexpr (DELTA) load_raw(q[R], start + idx);
                combine_granule<TI, TO, R, DELTA, NTS>(q, w, out + idx, nacc);
            }
            const int nedge = s.nh + s.nt;
            double enorm = 0.0;
            if (nedge > 0 && wave == 0) {
                if (lane < nedge)
                    enorm = combine_ragged<TI, TO, R, DELTA>(ops, start, shW, out, lane < s.nh ? s.start + lane : s.ts + (lane - s.nh));
                if (normparts != nullptr) enorm = wave_sum(enorm);
            }
            if (normparts != nullptr) {
                const acc_t ws = wave_sum(nacc);
                if (lane == 0) shNorm[wave] = static_cast<double>(ws);
                __syncthreads();
                if (tid == 0) {
                    double tot = shNorm[0];
#pragma unroll
                    for (int k = 1; k < NW; ++k) tot += shNorm[k];
                    if (nedge > 0) tot += enorm;
                    normparts[t.unit] = tot;
                }
            }
            if (tid == 0) st.outcome[at] += kRedone - kGaveUp;
            __syncthreads();   // (the next unit's sums go through the same memory)
        }
        __syncthreads();
    }
}

struct ResidentArgs {
    Operands ops;
    void* out;
    const ResidentUnit* units;
    ResidentState state;
    SmallTable small;
    double* gram;
    double* normparts;
    const void* start;
    int n_units, n_redo, wait_us, order, leaves;
};

// One workgroup per unit.  SV steps of 256 granules (16 bytes) of every operand stay in registers, SL in LDS; WPS
// waves per SIMD are resident, i.e. WPS workgroups per compute unit.
//
// A layer of W units gets its Gram matrix in one trip when W is small (every workgroup reads the W partial matrices)
// and in two otherwise (the q-th workgroup sums the q-th run of entries over the units; everybody reads the sums).
// The order of the sums depends on W alone: identical inputs give bit-identical outputs.
//
// Waiting is bounded, because nothing promises that a layer's workgroups run side by side (another stream's kernels
// may hold part of the chip): after wait_us a workgroup marks its unit and ends; redo_units does it then.
// The layers of at most kSmallLayer elements are left to small_layers.
// DELTA: operands are x - start, the result is start + z (the single pass of the after-optimizer form).
template <typename TI, typename TO, int R, bool DELTA, int SV, int SL, int WPS>
__global__ void __launch_bounds__(kThreads, WPS)
resident_kernel(const ResidentArgs args) {
    constexpr int G = Traits<TI>::VEC;
    constexpr int NP = R * (R + 1) / 2;
    constexpr int NW = kThreads / 64;
    constexpr int ROWS = kThreads / NP;
    constexpr int kDirect = direct_units(R);
    constexpr int kEdge = 2 * (G - 1);
    constexpr int RL = R + (DELTA ? 1 : 0);   // rows kept: the operands, and `start`
    // entries accumulated side by side: more than some 60 do not fit beside what is kept, and take more sweeps over it
    constexpr int SWEEPS = (NP + 59) / 60;
    constexpr int NA = (NP + SWEEPS - 1) / SWEEPS;
    // more than 8 operands of a 16-bit type: the Gram matrix on the matrix cores (multiply_staged below)
    constexpr bool MFMA = resident_matrix(DtypeOf<TI>::value, R);
    typedef typename Traits<TI>::acc_t acc_t;
    typedef typename Traits<TO>::acc_t out_acc_t;
    constexpr bool NTS = !(sizeof(TI) == 2 && sizeof(TO) == 4 && R <= 2);   // as combine_kernel
    static_assert(ROWS >= 1 && SV >= 1 && R <= 16 && !(MFMA && SL > 1), "");

    __shared__ double shP[NW * (MFMA ? 256 : NP)];
    __shared__ double shR[ROWS * NP > NW * kRun ? ROWS * NP : NW * kRun];
    __shared__ double shEdge[R][kEdge > 0 ? kEdge : 1];
    __shared__ double shG[R * R];
    __shared__ double shW[R];
    __shared__ double shQ[4 * R];
    __shared__ double shNorm[NW];
    __shared__ int shSkip;
    __shared__ unsigned long long shTodo[NW];
    __shared__ double shSmall[kRedoInLaunch<SV, SL> && !MFMA ? NW * R : 1][kSmallLayer];
    __shared__ __align__(16) unsigned char shStage[MFMA ? NW * 16 * 1024 : 16];
    __shared__ __align__(16) unsigned char shKeep[SL > 0 && !MFMA ? SL * RL * kThreads * 16 : 16];

    // (WPS workgroups of the planner's count fit a compute unit: registers by the launch bounds, LDS here)
    static_assert(WPS * (sizeof(shP) + sizeof(shR) + sizeof(shEdge) + sizeof(shG) + sizeof(shW) + sizeof(shQ) + sizeof(shNorm) +
                         sizeof(shSkip) + sizeof(shTodo) + sizeof(shSmall) + sizeof(shStage) + sizeof(shKeep) + 1280) <= 160 * 1024, "");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int at = static_cast<int>(blockIdx.x);
    if constexpr (kRedoInLaunch<SV, SL>) {
        const int n_units = args.n_units, n_redo = args.n_redo;
        if (at >= n_units + n_redo) {
            small_layers<TI, TO, R, DELTA>(args.ops, static_cast<TO*>(args.out), args.small, at - n_units - n_redo, args.gram, args.normparts,
                                           static_cast<const TI*>(args.start), args.order, args.leaves,
                                           MFMA ? reinterpret_cast<double(*)[kSmallLayer]>(shStage) : shSmall);
            return;
        }
        if (at >= n_units) {
            redo_units<TI, TO, R, DELTA, true>(args.ops, static_cast<TO*>(args.out), args.units, n_units, at - n_units, n_redo, args.state,
                                               args.gram, args.normparts, static_cast<const TI*>(args.start), args.order, args.leaves, shR,
                                               shG, shW, shQ, shNorm, shTodo, &shSkip);
            return;
        }
    }
    const Operands& ops = args.ops;
    const ResidentUnit* __restrict__ const units = args.units;
    const ResidentState st = args.state;
    const TI* const start = static_cast<const TI*>(args.start);
    const ResidentUnit t = units[at];   // (before any atomic access: scalar loads)
    // (while it runs, only the last workgroups of this launch itself write to that word)
    const unsigned tag = tag_of(kRedoInLaunch<SV, SL> ? __hip_atomic_load(st.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *st.epoch);
    auto decide = [&](int what) __attribute__((always_inline)) {
        if constexpr (!kRedoInLaunch<SV, SL>) {
            if (what == kGaveUp && tid == 0) st.outcome[at] = kGaveUp;
        } else if (tid == 0) __hip_atomic_store(st.outcome + at, outcome_word(tag, what), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    const int W = t.layer_end - t.layer_first;
    const buffer_t partials = buffer_of(st.partials + static_cast<long long>(t.layer_first) * (NP * 2), W * NP * 16);
    adasum_tile tile;
    tile.start = t.start;
    tile.len = t.len;
    tile.layer = t.layer;
    const Split s = split_tile<G>(tile);
    auto operand = [&](int r) { return static_cast<const TI*>(ops.pack[r]); };

    const int nedge = s.nh + s.nt;
    auto edge_at = [&]() { return lane < s.nh ? s.start + lane : s.ts + (lane - s.nh); };
    if (tid == 0) shSkip = 0;
    // the ragged head and tail are multiplied and summed in fp64
    if (wave == 0 && lane < nedge) {
        const long long eidx = edge_at();
        double sd = 0.0;
        if constexpr (DELTA) sd = static_cast<double>(load_elem(start + eidx));
#pragma unroll
        for (int r = 0; r < R; ++r) shEdge[r][lane] = static_cast<double>(load_elem(operand(r) + eidx)) - sd;
    }

    // Every load of the unit is issued before anything is consumed, and there is no branch around a step's loads: a lane
    // past the last granule re-reads that one, and so does a whole step past it.  So the compiler knows how many
    // loads are in flight behind each step, and the first step is multiplied while the others are still on their way.  (With
    // a branch around every step's loads it can only wait for all of them: K = 8 fp32, ResNet-50 sizes, 215 us instead of
    // 207, K = 8 bf16 in the after-optimizer form 149 instead of 143.)
    auto granule_at = [&](int i) {
        const int j = i * kThreads + tid;
        return static_cast<unsigned>((j < s.ng ? j : s.ng - 1) * 16);
    };
    auto row_at = [&](int r) { return (!DELTA || r < R ? operand(r) : start) + s.bs; };
    Granule<TI, G> raw[SV][RL];
    // step SV + i, row r: this wave's 1 KB
    auto keep = [&](int i, int r) { return shKeep + ((i * RL + r) * NW + wave) * 1024; };
    // (Where units have many steps, one that has a single step does not load the rest for nothing, and waits here, so that the
    // steps of the others can still be told apart: ResNet-50 sizes, K = 2 bf16 33.5 us instead of 34.8, binary16 31.7 instead of 33.1, a
    // sixteenth of BERT-Large, bf16, 31.4 instead of 32.6.  K = 2 fp32 and fp64 and K = 3 and 4 take the same either way:
    // without it 0.99 to 1.01 times on tables of more than 30 us, 0.95 to 1.08 on smaller ones, whose runs differ by as much, 0.988
    // (K = 2 fp32) to 1.004 in the mean of 13 tables.  With 7 steps of 8 rows it is K = 8 fp32 192 instead of 191.)
    if (SV >= 10 && s.ng <= kThreads) {
        if (s.ng > 0) {
            const unsigned off = granule_at(0);
#pragma unroll
            for (int r = 0; r < RL; ++r) load_raw(raw[0][r], reinterpret_cast<const TI*>(reinterpret_cast<const char*>(row_at(r)) + off));
            __builtin_amdgcn_s_waitcnt(0x0f70);   // (no vector loads in flight)
        }
    } else if (s.ng > 0) {
#pragma unroll
        for (int i = 0; i < SV + (MFMA ? 0 : SL); ++i) {
            __builtin_amdgcn_sched_barrier(0);
            const unsigned off = granule_at(i);
#pragma unroll
            for (int r = 0; r < RL; ++r) {
                if (i < SV) load_raw(raw[i < SV ? i : 0][r], reinterpret_cast<const TI*>(reinterpret_cast<const char*>(row_at(r)) + off));
                else load_to_lds(row_at(r), off, keep(i - SV, r));
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    {
        if constexpr (MFMA) {
            // G = X X^T with v_mfma_f32_16x16x32: per lane, eight consecutive elements (a granule) of row lane % 16, for
            // either operand.  What is kept has a row's granules along the lanes, so a step goes through LDS (a wave's own
            // 16 KB, no barrier): granule c of row r lies at place c ^ r, conflict-free both ways.  Four accumulators
            // where the vector units would need R (R + 1) / 2: 136 of them took three sweeps over what is kept (K = 16 bf16
            // on a sixteenth of ResNet-50: 82 us with spills, 30 this way).  The products are exact; four instructions in a row accumulate 128 of them in fp32, and those
            // sums are added up in fp64, so that a unit of more steps is no less exact.
            unsigned char* stage = shStage + wave * (16 * 1024);
            const int m = lane & 15, kg = lane >> 4;
            double sum[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int r = R; r < 16; ++r) *reinterpret_cast<u32x4*>(stage + r * 1024 + lane * 16) = u32x4{0u, 0u, 0u, 0u};
            auto multiply_staged = [&]() __attribute__((always_inline)) {
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int b0 = 0; b0 < 16; b0 += 4) {
                    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int b = b0; b < b0 + 4; ++b) {
                        const u32x4 x = *reinterpret_cast<const u32x4*>(stage + m * 1024 + ((4 * b + kg) ^ m) * 16);
                        acc = mfma_square<TI>(x, acc);
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) sum[v] += static_cast<double>(acc[v]);
                }
                __builtin_amdgcn_wave_barrier();
            };
#pragma unroll
            for (int i = 0; i < SV; ++i)
                if (i * kThreads < s.ng) {
                    const bool live = i * kThreads + tid < s.ng;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        u32x4 v;
                        v.x = live ? raw[i][r].w[0] : 0u;
                        v.y = live ? raw[i][r].w[1] : 0u;
                        v.z = live ? raw[i][r].w[2] : 0u;
                        v.w = live ? raw[i][r].w[3] : 0u;
                        *reinterpret_cast<u32x4*>(stage + r * 1024 + (lane ^ r) * 16) = v;
                    }
                    multiply_staged();
                }
            if constexpr (SL > 0) {
                // One more step stays where the others pass through, loaded straight there once they have: lane l takes granule
                // l ^ r of row r, so that it lies as above.  (A third more is kept:
                // K = 16 bf16, ResNet-50 sizes, 214 us instead of 237.)
                if (SV * kThreads < s.ng) {
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const int j = SV * kThreads + wave * 64 + (lane ^ r);
                        load_to_lds(row_at(r), static_cast<unsigned>((j < s.ng ? j : s.ng - 1) * 16), stage + r * 1024);
                    }
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    if (SV * kThreads + tid >= s.ng) {
#pragma unroll
                        for (int r = 0; r < R; ++r) *reinterpret_cast<u32x4*>(stage + r * 1024 + (lane ^ r) * 16) = u32x4{0u, 0u, 0u, 0u};
                    }
                    multiply_staged();
                }
            }
            // (accumulator v of a lane: row 4 (lane / 16) + v, column lane % 16)
#pragma unroll
            for (int v = 0; v < 4; ++v) shP[wave * 256 + (4 * kg + v) * 16 + m] = sum[v];
        } else {
#pragma unroll
        for (int sweep = 0; sweep < SWEEPS; ++sweep) {
            // (opaque: what a sweep derives from the kept operands is derived again by the next, not held in registers)
            int n_live = s.ng;
            if constexpr (SWEEPS > 1) asm volatile("" : "+s"(n_live)::"memory");
            acc_t acc[NA];
#pragma unroll
            for (int e = 0; e < NA; ++e) acc[e] = 0;
            // eight bytes of every row
            auto multiply = [&](const unsigned int (&q)[RL][2], bool live) {
#pragma unroll
                    for (int k = 0; k < G / 2; ++k) {
                        acc_t v[R];
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            v[r] = element<TI>(q[r], k);
                            if constexpr (DELTA) v[r] -= element<TI>(q[R], k);
                            v[r] = live ? v[r] : static_cast<acc_t>(0);
                        }
#pragma unroll
                        for (int e = 0; e < NA; ++e)
                            if (sweep * NA + e < NP) {
                                const int a = kEntries<R>.row[sweep * NA + e], b = kEntries<R>.col[sweep * NA + e];
                                acc[e] = fma_t(v[a], v[b], acc[e]);
                            }
                    }
            };
#pragma unroll
            for (int i = 0; i < SV; ++i)
                if (i * kThreads < s.ng) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        unsigned int q[RL][2];
#pragma unroll
                        for (int r = 0; r < RL; ++r) {
                            q[r][0] = raw[i][r].w[2 * h];
                            q[r][1] = raw[i][r].w[2 * h + 1];
                        }
                        multiply(q, i * kThreads + tid < n_live);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            each<SL>([&](auto step) {
                constexpr int i = decltype(step)::value;
                if ((SV + i) * kThreads < s.ng) {
                    // what this wave sent to LDS is there, but for the steps behind (a lane reads only what it loaded itself)
                    asm volatile("s_waitcnt vmcnt(%0)" ::"i"((SL - 1 - i) * RL) : "memory");
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        unsigned int q[RL][2];
#pragma unroll
                        for (int r = 0; r < RL; ++r) {
                            const u32x2 v = *reinterpret_cast<const u32x2*>(keep(i, r) + lane * 16 + 8 * h);
                            q[r][0] = v.x;
                            q[r][1] = v.y;
                        }
                        multiply(q, (SV + i) * kThreads + tid < n_live);
                    }
                }
            });
            wave_sum_scatter(acc, lane);
#pragma unroll
            for (int i = 0; i < (NA + 63) / 64; ++i) {
                const int e = lane + 64 * i;
                if (e < NA && sweep * NA + e < NP) shP[wave * NP + sweep * NA + e] = static_cast<double>(acc[i]);
            }
        }
        }
        __syncthreads();
        if (tid < NP) {
            int a, b;
            entry_to_ij<R, true>(tid, a, b);
            const int cell = MFMA ? a * 16 + b : tid;
            double tot = shP[cell];
#pragma unroll
            for (int w = 1; w < NW; ++w) tot += shP[w * (MFMA ? 256 : NP) + cell];
            for (int k = 0; k < nedge; ++k) tot += shEdge[a][k] * shEdge[b][k];
            if (W > 1) send(partials, partial_at<NP>(t.unit - t.layer_first, tid, W), tot, tag);
            else shG[a * R + b] = shG[b * R + a] = tot;
        }
    }

    if (t.small > 0) {   // (small_layers does it; a branch on it further up would cut the load of `t` in two)
        decide(kDone);
        return;
    }
    // The other arguments are read here: fetched at the start with the rest, they do not fit the scalar registers beside the
    // operands' addresses, and a kernel that has to put some away elsewhere starts its waves later (K = 16 bf16, ResNet-50
    // sizes, 246 us instead of 241).
    typedef const __attribute__((address_space(4))) ResidentArgs* arguments_t;
    arguments_t late = (arguments_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(late));
    TO* const out = static_cast<TO*>(late->out);
    double* const gram = late->gram;
    double* const normparts = late->normparts;
    const int order = late->order, leaves = late->leaves, wait_us = late->wait_us;
    if (W > 1) {
        const long long deadline = static_cast<long long>(wall_clock64()) + static_cast<long long>(wait_us) * kTicksPerUs;
        auto in_time = [&]() __attribute__((always_inline)) { return static_cast<long long>(wall_clock64()) <= deadline; };
        bool ok = wait_us >= 0;
        // the sum of entry e over the units u0, u0 + step, ... of the layer, kAhead of them looked at side by side
        auto sum_ahead = [&](auto ahead, int e, int u0, int step) __attribute__((always_inline)) {
            constexpr int kAhead = decltype(ahead)::value;
            double v = 0.0;
            for (; u0 < W; u0 += step * kAhead) {
                int offset[kAhead];
                u32x4 x[kAhead];
#pragma unroll
                for (int k = 0; k < kAhead; ++k) offset[k] = partial_at<NP>(u0 + step * k < W ? u0 + step * k : W - 1, e, W);
                ok = await(partials, offset, x, tag, in_time) && ok;
#pragma unroll
                for (int k = 0; k < kAhead; ++k)
                    if (u0 + step * k < W) v += value(x[k]);
            }
            return v;
        };
        auto sum_units = [&](int e, int u0, int step) __attribute__((always_inline)) {
            if (W <= step) return sum_ahead(std::integral_constant<int, 1>(), e, u0, step);
            return W <= 2 * step ? sum_ahead(std::integral_constant<int, 2>(), e, u0, step) : sum_ahead(std::integral_constant<int, 4>(), e, u0, step);
        };
        if (W <= kDirect) {
            const int row = tid / NP, e = tid % NP;
            if (row < ROWS) shR[row * NP + e] = sum_units(e, row, ROWS);
            __syncthreads();
            if (tid < NP) {
                double tot = shR[tid];
#pragma unroll
                for (int k = 1; k < ROWS; ++k) tot += shR[k * NP + tid];
                int a, b;
                entry_to_ij<R, true>(tid, a, b);
                shG[a * R + b] = shG[b * R + a] = tot;
            }
        } else {
            const buffer_t sums = buffer_of(st.sums + static_cast<long long>(t.layer) * (NP * 2), NP * 16);
            for (int run = (t.unit - t.layer_first) * kRun; run < NP; run += W * kRun) {
                const int e = run + tid % kRun;
                const double v = run_sum(sum_units(e < NP ? e : NP - 1, tid / kRun, kRunUnits));
                if (__ballot(!ok) != 0 && lane == 0) shSkip = 1;
                if (lane < kRun) shR[wave * kRun + lane] = v;
                __syncthreads();
                if (tid < kRun && e < NP && !shSkip) {
                    double tot = shR[tid];
#pragma unroll
                    for (int w = 1; w < NW; ++w) tot += shR[w * kRun + tid];
                    send(sums, e * 16, tot, tag);
                }
                __syncthreads();   // (the next run's sums go through the same memory)
            }
            if (tid < NP) {
                const int offset[1] = {tid * 16};
                u32x4 x[1];
                if (lane == 0) ok = await(sums, offset, x, tag, in_time) && ok;   // (one lane's looks are enough until then)
                ok = await(sums, offset, x, tag, in_time) && ok;
                int a, b;
                entry_to_ij<R, true>(tid, a, b);
                shG[a * R + b] = shG[b * R + a] = value(x[0]);
            }
        }
        if (!ok) shSkip = 1;
    }
    __syncthreads();
    if (shSkip) {
        decide(kGaveUp);
        return;
    }
    decide(kDone);
    if (wave == 0) unit_weights<R>(shG, shW, shQ, order, leaves, lane);
    if (gram != nullptr && t.unit == t.layer_first)   // (for the statistics)
        for (int i = tid; i < R * R; i += kThreads) gram[static_cast<long long>(t.layer) * (R * R) + i] = shG[i];
    __syncthreads();
    acc_t w[R];
#pragma unroll
    for (int r = 0; r < R; ++r) w[r] = static_cast<acc_t>(shW[r]);
    acc_t nacc = 0;
    auto combine = [&](const Granule<TI, G> (&q)[RL], int i) {
        const int j = i * kThreads + tid;
        if (j < s.ng) combine_granule<TI, TO, R, DELTA, NTS>(q, w, out + s.bs + static_cast<long long>(j) * G, nacc);
    };
#pragma unroll
    for (int i = 0; i < SV; ++i)
        if (i * kThreads < s.ng) combine(raw[i], i);
    if constexpr (SL > 0) {
#pragma unroll
        for (int i = 0; i < SL; ++i)
            if ((SV + i) * kThreads < s.ng) {
                Granule<TI, G> q[RL];
#pragma unroll
                for (int r = 0; r < RL; ++r) {
                    const u32x4 v = *reinterpret_cast<const u32x4*>(
                        MFMA ? shStage + wave * (16 * 1024) + r * 1024 + (lane ^ r) * 16 : keep(i, r) + lane * 16);
                    q[r].w[0] = v.x;
                    q[r].w[1] = v.y;
                    q[r].w[2] = v.z;
                    q[r].w[3] = v.w;
                }
                combine(q, SV + i);
            }
    }
    double enorm = 0.0;
    if (nedge > 0 && wave == 0) {
        if (lane < nedge) enorm = combine_ragged<TI, TO, R, DELTA>(ops, start, shW, out, edge_at());
        if (normparts != nullptr) enorm = wave_sum(enorm);
    }
    if (normparts != nullptr) {
        const acc_t ws = wave_sum(nacc);
        if (lane == 0) shNorm[wave] = static_cast<double>(ws);
        __syncthreads();
        if (tid == 0) {
            double tot = shNorm[0];
#pragma unroll
            for (int k = 1; k < NW; ++k) tot += shNorm[k];
            if (nedge > 0) tot += enorm;
            normparts[t.unit] = tot;
        }
    }
}

// The second launch of the other forms.  Usually there is nothing to do, and it costs 4 us at 3726 units.  Where every unit gave
// up it streams like a combine pass: ResNet-50 sizes, K = 8 fp32 316 us in all, K = 16 bf16 482, K = 2 bf16 95.
template <typename TI, typename TO, int R, bool DELTA>
__global__ void __launch_bounds__(kThreads, redo_per_cu(R))
resident_redo_kernel(const Operands ops, TO* out, const ResidentUnit* __restrict__ units, int n_units, const ResidentState st,
                     double* __restrict__ gram, double* __restrict__ normparts, const TI* start, int order, int leaves, int n_redo,
                     const SmallTable small) {
    constexpr int NP = R * (R + 1) / 2;
    constexpr int NW = kThreads / 64;
    constexpr int ROWS = kThreads / NP;
    const int at = static_cast<int>(blockIdx.x);
    __shared__ double shR[ROWS * NP > NW * kRun ? ROWS * NP : NW * kRun];
    __shared__ double shG[R * R];
    __shared__ double shW[R];
    __shared__ double shQ[4 * R];
    __shared__ double shNorm[NW];
    __shared__ unsigned long long shTodo[NW];
    __shared__ double shSmall[NW * R][kSmallLayer];
    if (at >= n_redo)
        small_layers<TI, TO, R, DELTA>(ops, out, small, at - n_redo, gram, normparts, start, order, leaves, shSmall);
    else
        redo_units<TI, TO, R, DELTA, false>(ops, out, units, n_units, at, n_redo, st, gram, normparts, start, order, leaves, shR, shG,
                                            shW, shQ, shNorm, shTodo, nullptr);
}

// One launch, and what became of this one: the thread's last error may be an older one, of a call that is not ours, and the second
// launch of a pass must not fall out for that once the first is on its way.
template <typename... P>
int enqueue(void (*kernel)(P...), int blocks, hipStream_t stream, P... args) {
    void* at[] = {const_cast<void*>(static_cast<const void*>(&args))...};
    return static_cast<int>(hipLaunchKernel(reinterpret_cast<const void*>(kernel), dim3(static_cast<unsigned>(blocks)), dim3(kThreads), at, 0, stream));
}

template <typename TI, typename TO, int R, bool DELTA, int SV, int SL, int WPS>
int launch_s(const ResidentCall& c, hipStream_t stream) {
    const bool same = kRedoInLaunch<SV, SL> && c.n_units <= WPS * kResidentCus;
    const int redo = std::min((c.n_units + kRedoScan - 1) / kRedoScan, same ? kRedoBlocks : redo_per_cu(R) * kResidentCus);
    const int small = (c.small.n + kThreads / 64 - 1) / (kThreads / 64);
    ResidentArgs args;
    args.ops = c.ops;
    args.out = c.out;
    args.units = c.units;
    args.state = c.state;
    args.small = c.small;
    args.gram = c.gram;
    args.normparts = c.normparts;
    args.start = c.start;
    args.n_units = c.n_units;
    args.n_redo = redo;
    args.wait_us = c.wait_us;
    args.order = c.order;
    args.leaves = c.leaves;
    const int e = enqueue(resident_kernel<TI, TO, R, DELTA, SV, SL, WPS>, c.n_units + (same ? redo + small : 0), stream, args);
    if (same || e != 0) return e;
    return enqueue(resident_redo_kernel<TI, TO, R, DELTA>, redo + small, stream, c.ops, static_cast<TO*>(c.out), c.units, c.n_units, c.state,
                   c.gram, c.normparts, static_cast<const TI*>(c.start), c.order, c.leaves, redo, c.small);
}

template <typename TI, typename TO, int R, bool DELTA>
int launch_r(const ResidentCall& c, hipStream_t stream) {
    constexpr int D = DtypeOf<TI>::value;
    int e = static_cast<int>(hipErrorInvalidValue);
    if (c.form == 1) e = launch_s<TI, TO, R, DELTA, 1, 0, resident_per_cu(D, R, 1)>(c, stream);
    if constexpr (R <= 8) {
        if (c.form == 2)
            e = launch_s<TI, TO, R, DELTA, resident_register_steps(D, R, DELTA, 2), resident_lds_steps(D, R, DELTA, 2), resident_per_cu(D, R, 2)>(c, stream);
    }
    if (c.form == 3)
        e = launch_s<TI, TO, R, DELTA, resident_register_steps(D, R, DELTA, 3), resident_lds_steps(D, R, DELTA, 3), resident_per_cu(D, R, 3)>(c, stream);
    return e;
}

template <typename TI, typename TO, bool DELTA>
int launch_t(const ResidentCall& c, hipStream_t stream) {
#define ADASUM_RESIDENT(RR) \
    case RR: return launch_r<TI, TO, RR, DELTA>(c, stream)
    switch (c.R) {
#if ADASUM_WIDE_GROUPS
        ADASUM_RESIDENT(10);
        ADASUM_RESIDENT(12);
        ADASUM_RESIDENT(14);
        ADASUM_RESIDENT(16);
#else
        ADASUM_RESIDENT(2);
        ADASUM_RESIDENT(3);
        ADASUM_RESIDENT(4);
        ADASUM_RESIDENT(5);
        ADASUM_RESIDENT(6);
        ADASUM_RESIDENT(7);
        ADASUM_RESIDENT(8);
#endif
        default: return static_cast<int>(hipErrorInvalidValue);
    }
#undef ADASUM_RESIDENT
}

}  // namespace

// This file is compiled once per storage type of the operands (ADASUM_LEAF_TYPE) and range of group sizes
// (ADASUM_WIDE_GROUPS: 10 .. 16 operands, else 2 .. 8).
#if ADASUM_LEAF_TYPE == 0
typedef float leaf_t;
#define ADASUM_ENTRY_NAME(x) x##_f32
#elif ADASUM_LEAF_TYPE == 1
typedef bf16_t leaf_t;
#define ADASUM_ENTRY_NAME(x) x##_bf16
#elif ADASUM_LEAF_TYPE == 2
typedef f16_t leaf_t;
#define ADASUM_ENTRY_NAME(x) x##_f16
#else
typedef double leaf_t;
#define ADASUM_ENTRY_NAME(x) x##_f64
#endif
#if ADASUM_WIDE_GROUPS
int ADASUM_ENTRY_NAME(launch_resident_wide)(const ResidentCall& c, void* stream) {
#else
int ADASUM_ENTRY_NAME(launch_resident)(const ResidentCall& c, void* stream) {
#endif
    hipStream_t s = static_cast<hipStream_t>(stream);
    constexpr int D = DtypeOf<leaf_t>::value;
    if (c.n_units < 1) return static_cast<int>(hipErrorInvalidConfiguration);
#if !ADASUM_WIDE_GROUPS
    if (c.start != nullptr) return c.out_dtype == D ? launch_t<leaf_t, leaf_t, true>(c, s) : static_cast<int>(hipErrorInvalidValue);
#else
    if (c.start != nullptr) return static_cast<int>(hipErrorInvalidValue);
#endif
    if (c.out_dtype == D) return launch_t<leaf_t, leaf_t, false>(c, s);
#if ADASUM_LEAF_TYPE == 1 || ADASUM_LEAF_TYPE == 2
    if (c.out_dtype == ADASUM_F32) return launch_t<leaf_t, float, false>(c, s);
#elif ADASUM_LEAF_TYPE == 0
    if (c.out_dtype == ADASUM_BF16) return launch_t<float, bf16_t, false>(c, s);
    if (c.out_dtype == ADASUM_F16) return launch_t<float, f16_t, false>(c, s);
#endif
    return static_cast<int>(hipErrorInvalidValue);
}

}  // namespace adasum
