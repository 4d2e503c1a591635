// cpes_kernels.hip -- gfx950 kernels of the CoPES parameter-space hot path.
//
// Streaming kernels (perturb, restore, master staging, update) work on
// "units" of consecutive subspace positions: 8 for bf16 weights (one 16-byte
// vector, two Philox blocks) and 4 for fp32 weights (one 16-byte vector, one
// Philox block), one unit per thread at a time.  A wave therefore moves 1 KiB
// per vector access, fully coalesced.  The ragged tail takes an
// element-by-element path with the same arithmetic.  Subspaces are ranges,
// int64 or uint32 element maps, or chunk lists.  Noise never leaves registers.
#include <algorithm>
#include <type_traits>

#include "cpes_device.hpp"
#include "cpes_launch.hpp"

namespace cpes {

namespace {

template <typename T> struct UnitOf;
template <> struct UnitOf<uint16_t> { static constexpr int n = 8; };
template <> struct UnitOf<float> { static constexpr int n = 4; };

template <typename T> __device__ __forceinline__ float to_f32(T v);
template <> __device__ __forceinline__ float to_f32<uint16_t>(uint16_t v) { return bf16_to_f32(v); }
template <> __device__ __forceinline__ float to_f32<float>(float v) { return v; }

template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ uint16_t from_f32<uint16_t>(float v) { return f32_to_bf16(v); }
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }

template <int N, typename Q>
__device__ __forceinline__ void unit_normals(uint32_t k0, uint32_t k1, Q q, const Bm& tb, float z[N])
{
    if constexpr (N == 8) normals8<Q>(k0, k1, q, tb, z);
    else normals4<Q>(k0, k1, q, tb, z);
}

// 16-byte vector loads / stores of one unit.  NT marks the accesses
// non-temporal: a copy far larger than the caches (a subspace of 10^8
// parameters and up) then streams past them instead of evicting lines that
// are never reused, which measured 3-5 % faster on such copies; copies of a
// few tens of MB keep the default policy, since they run from cache.
//
// The vectors need no more than their elements' alignment: an even split of a
// model whose size is no multiple of 8 K starts its subspaces at any element,
// and gfx950 takes 16-byte accesses at any address (a wave's 1 KiB then spans
// nine 128-byte lines instead of eight).  33,333,335 bf16 weights from an odd
// element on: restore 54 -> 17.6 us, perturbation 69 -> 38 us against an
// element path, 17.3 and 37.5 us from an aligned one.
typedef unsigned int V4u __attribute__((ext_vector_type(4)));
typedef float V4f __attribute__((ext_vector_type(4)));
typedef V4f V4fAnywhere __attribute__((aligned(4)));
typedef unsigned int V2u __attribute__((ext_vector_type(2)));
typedef V2u V2uAnywhere __attribute__((aligned(2)));
template <typename T> struct Vec16;
template <> struct Vec16<uint16_t> { typedef V4u type __attribute__((aligned(2))); };
template <> struct Vec16<float> { typedef V4u type __attribute__((aligned(4))); };

template <typename T, bool NT = false>
__device__ __forceinline__ void load_vec(const T* p, T v[UnitOf<T>::n])
{
    typedef typename Vec16<T>::type V;
    const V* q = reinterpret_cast<const V*>(p);
    *reinterpret_cast<V4u*>(v) = NT ? __builtin_nontemporal_load(q) : *q;
}
template <typename T, bool NT = false>
__device__ __forceinline__ void store_vec(T* p, const T v[UnitOf<T>::n])
{
    typedef typename Vec16<T>::type V;
    const V4u x = *reinterpret_cast<const V4u*>(v);
    if (NT)
        __builtin_nontemporal_store(x, reinterpret_cast<V*>(p));
    else
        *reinterpret_cast<V*>(p) = x;
}
template <int N, bool NT = false>
__device__ __forceinline__ void load_f32s(const float* p, float v[N])
{
#pragma unroll
    for (int h = 0; h < N / 4; ++h) {
        const V4fAnywhere* q = reinterpret_cast<const V4fAnywhere*>(p) + h;
        const V4f x = NT ? __builtin_nontemporal_load(q) : *q;
        v[4 * h + 0] = x[0]; v[4 * h + 1] = x[1]; v[4 * h + 2] = x[2]; v[4 * h + 3] = x[3];
    }
}
template <int N, bool NT = false>
__device__ __forceinline__ void store_f32s(float* p, const float v[N])
{
#pragma unroll
    for (int h = 0; h < N / 4; ++h) {
        const V4f x = {v[4 * h + 0], v[4 * h + 1], v[4 * h + 2], v[4 * h + 3]};
        if (NT)
            __builtin_nontemporal_store(x, reinterpret_cast<V4fAnywhere*>(p) + h);
        else
            reinterpret_cast<V4fAnywhere*>(p)[h] = x;
    }
}
__device__ __forceinline__ int64_t grid_stride() { return (int64_t)gridDim.x * blockDim.x; }
__device__ __forceinline__ int64_t global_tid() { return (int64_t)blockIdx.x * blockDim.x + threadIdx.x; }

// Subspace addressing: position j is parameter offset + j (kContig),
// index[offset + j] (kGather), or, with chunks of 2^s parameters,
// index[offset + (j >> s)] * 2^s + (j mod 2^s) (kChunk).
constexpr int kContig = kAddrContig, kGather = kAddrGather, kChunk = kAddrChunk, kGather32 = kAddrGather32;

// An element-level map (int64 or uint32 entries).
template <int ADDR>
constexpr bool kMap = ADDR == kGather || ADDR == kGather32;

// Resolve the parameter index of position j; returns false for a map entry
// outside [0, numel) (skipped, never dereferenced).
template <int ADDR>
__device__ __forceinline__ bool param_at(const int64_t* index, int64_t offset, int64_t numel, int shift, int64_t j,
                                         int64_t& i)
{
    if (ADDR == kContig) {
        i = offset + j;
        return true;
    }
    if (ADDR == kGather) {
        i = index[offset + j];
        return i >= 0 && i < numel;
    }
    if (ADDR == kGather32) {
        i = reinterpret_cast<const uint32_t*>(index)[offset + j];
        return i < numel;
    }
    const int64_t c = index[offset + (j >> shift)];
    if (c < 0 || c > (numel >> shift)) return false;
    i = (c << shift) + (j & ((1ll << shift) - 1));
    return i < numel;
}

template <int ADDR>
__device__ __forceinline__ bool param_of(const StreamArgs& a, int64_t j, int64_t& i)
{
    return param_at<ADDR>(a.index, a.offset, a.numel, a.chunk_shift, j, i);
}

// First parameter of the unit starting at position j0 for contiguous and
// chunked subspaces (a unit never crosses a chunk); false if the unit would
// leave [0, numel), in which case the caller takes the element path.
//
// The 64 lanes of a wave always hold 64 consecutive units whose first
// position is a multiple of 64 n.  When a chunk holds at least 64 n positions
// the whole wave therefore lies in one chunk, and its chunk id is read once,
// by a scalar load from the wave's first active lane: the chunk list is
// read-only here, so it is addressed as constant memory.
typedef const int64_t __attribute__((address_space(4)))* ConstI64;

__device__ __forceinline__ int64_t wave_uniform(int64_t x)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

template <int ADDR>
__device__ __forceinline__ bool unit_base(const int64_t* index, int64_t offset, int64_t numel, int shift, int64_t j0,
                                          int n, int64_t& base)
{
    if (ADDR == kContig) {
        base = offset + j0;
        return true;
    }
    int64_t c;
    if ((int64_t)64 * n <= (1ll << shift))
        c = ((ConstI64)(uintptr_t)index)[offset + (wave_uniform(j0) >> shift)];
    else
        c = index[offset + (j0 >> shift)];
    if (c < 0 || c > (numel >> shift)) return false;
    base = (c << shift) + (j0 & ((1ll << shift) - 1));
    return base + n <= numel;
}

// Drive a streaming kernel: every full unit goes through `vec_body` (16-byte
// accesses) in a branch-free grid-stride loop, so that per-launch invariants
// (polynomial constants, key schedule) stay hoisted; the ragged last unit, if
// any, is done once by thread 0 with `scalar_body` (element accesses).
template <int N, typename VecBody, typename ScalarBody>
__device__ __forceinline__ void for_each_unit(int64_t length, VecBody&& vec_body, ScalarBody&& scalar_body)
{
    const int64_t full = length / N;
    for (int64_t u = global_tid(); u < full; u += grid_stride()) vec_body(u);
    if (full * N < length && global_tid() == 0) scalar_body(full);
}

// ---------------------------------------------------------------- perturb --
// w[p(j)] = cast(fmaf(scale, eps_j, src_j)); src = w (optionally backed up to
// the snapshot first), the fp32 master, or an existing backup.  Also serves
// replay restore with scale = -sign * sigma.  Contiguous and chunked
// subspaces; index maps take k_perturb_map below.
template <typename T, int AUX, typename Q, int ADDR>
__global__ __launch_bounds__(kBlock) void k_perturb(StreamArgs a)
{
    constexpr int N = UnitOf<T>::n;
    const Bm tb = stage_bm_tables<kBlock>();
    T* w = static_cast<T*>(a.w);
    auto scalar_body = [&](int64_t u) {
        const int64_t j0 = u * N;
        float z[N];
        unit_normals<N, Q>(a.k0, a.k1, (Q)((uint64_t)(a.noise0 + j0) >> 2), tb, z);
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const int64_t j = j0 + e;
            int64_t i;
            if (j >= a.length || !param_of<ADDR>(a, j, i)) continue;
            float src;
            if (AUX == kAuxMaster) {
                src = static_cast<const float*>(a.aux)[j];
            } else if (AUX == kAuxBackup) {
                src = to_f32<T>(static_cast<const T*>(a.aux)[j]);
            } else {
                const T old = w[i];
                if (AUX == kAuxSnapshot) static_cast<T*>(a.aux)[j] = old;
                src = to_f32<T>(old);
            }
            w[i] = from_f32<T>(__builtin_fmaf(a.scale, z[e], src));
        }
    };
    auto vec_body = [&](int64_t u) {
        const int64_t j0 = u * N;
        int64_t base = 0;
        if (!unit_base<ADDR>(a.index, a.offset, a.numel, a.chunk_shift, j0, N, base)) {
            scalar_body(u);
            return;
        }
        float src[N];
        T old[N];
        if (AUX != kAuxMaster && AUX != kAuxBackup) load_vec<T>(w + base, old);
        if (AUX == kAuxMaster) {
            load_f32s<N>(static_cast<const float*>(a.aux) + j0, src);
        } else if (AUX == kAuxBackup) {
            T b[N];
            load_vec<T>(static_cast<const T*>(a.aux) + j0, b);
#pragma unroll
            for (int e = 0; e < N; ++e) src[e] = to_f32<T>(b[e]);
        } else {
#pragma unroll
            for (int e = 0; e < N; ++e) src[e] = to_f32<T>(old[e]);
            if (AUX == kAuxSnapshot) store_vec<T>(static_cast<T*>(a.aux) + j0, old);
        }
        float z[N];
        unit_normals<N, Q>(a.k0, a.k1, (Q)((uint64_t)(a.noise0 + j0) >> 2), tb, z);
        T out[N];
#pragma unroll
        for (int e = 0; e < N; ++e) out[e] = from_f32<T>(__builtin_fmaf(a.scale, z[e], src[e]));
        store_vec<T>(w + base, out);
    };
    for_each_unit<N>(a.length, vec_body, scalar_body);
}

// --------------------------------------------------------------- restores --
// Snapshot restore: w[p(j)] = snap[j], a bit copy.
template <typename T, bool NT, int ADDR>
__global__ __launch_bounds__(kBlock) void k_restore_copy(StreamArgs a)
{
    constexpr int N = UnitOf<T>::n;
    T* w = static_cast<T*>(a.w);
    const T* snap = static_cast<const T*>(a.aux);
    auto scalar_body = [&](int64_t u) {
        const int64_t j0 = u * N;
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const int64_t j = j0 + e;
            int64_t i;
            if (j < a.length && param_of<ADDR>(a, j, i)) w[i] = snap[j];
        }
    };
    auto vec_body = [&](int64_t u) {
        const int64_t j0 = u * N;
        int64_t base;
        if (!unit_base<ADDR>(a.index, a.offset, a.numel, a.chunk_shift, j0, N, base)) {
            scalar_body(u);
            return;
        }
        T v[N];
        load_vec<T, NT>(snap + j0, v);
        store_vec<T, NT>(w + base, v);
    };
    for_each_unit<N>(a.length, vec_body, scalar_body);
}

// Backup copy: backup[j] = w[p(j)] (bit copy), for backups taken apart from a
// perturbation, in device memory or in pinned host memory.
template <typename T, bool NT, int ADDR>
__global__ __launch_bounds__(kBlock) void k_backup_copy(StreamArgs a)
{
    constexpr int N = UnitOf<T>::n;
    const T* w = static_cast<const T*>(a.w);
    T* backup = static_cast<T*>(a.aux);
    auto scalar_body = [&](int64_t u) {
        const int64_t j0 = u * N;
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const int64_t j = j0 + e;
            int64_t i;
            if (j < a.length) backup[j] = param_of<ADDR>(a, j, i) ? w[i] : T(0);
        }
    };
    auto vec_body = [&](int64_t u) {
        const int64_t j0 = u * N;
        int64_t base;
        if (!unit_base<ADDR>(a.index, a.offset, a.numel, a.chunk_shift, j0, N, base)) {
            scalar_body(u);
            return;
        }
        T v[N];
        load_vec<T, NT>(w + base, v);
        store_vec<T, NT>(backup + j0, v);
    };
    for_each_unit<N>(a.length, vec_body, scalar_body);
}

// Master restore (bf16 weights): w[p(j)] = rne_bf16(master[j]).
template <bool NT, int ADDR>
__global__ __launch_bounds__(kBlock) void k_restore_master(StreamArgs a)
{
    constexpr int N = 8;
    uint16_t* w = static_cast<uint16_t*>(a.w);
    const float* master = static_cast<const float*>(a.aux);
    auto scalar_body = [&](int64_t u) {
        const int64_t j0 = u * N;
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const int64_t j = j0 + e;
            int64_t i;
            if (j < a.length && param_of<ADDR>(a, j, i)) w[i] = f32_to_bf16(master[j]);
        }
    };
    auto vec_body = [&](int64_t u) {
        const int64_t j0 = u * N;
        int64_t base;
        if (!unit_base<ADDR>(a.index, a.offset, a.numel, a.chunk_shift, j0, N, base)) {
            scalar_body(u);
            return;
        }
        float m[N];
        load_f32s<N, NT>(master + j0, m);
        uint16_t v[N];
#pragma unroll
        for (int e = 0; e < N; ++e) v[e] = f32_to_bf16(m[e]);
        store_vec<uint16_t, NT>(w + base, v);
    };
    for_each_unit<N>(a.length, vec_body, scalar_body);
}

// Master staging: master[j] = f32(w[p(j)]).
template <typename T, bool NT, int ADDR>
__global__ __launch_bounds__(kBlock) void k_stage_master(StreamArgs a)
{
    constexpr int N = UnitOf<T>::n;
    const T* w = static_cast<const T*>(a.w);
    float* master = static_cast<float*>(a.aux);
    auto scalar_body = [&](int64_t u) {
        const int64_t j0 = u * N;
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const int64_t j = j0 + e;
            int64_t i;
            if (j < a.length && param_of<ADDR>(a, j, i)) master[j] = to_f32<T>(w[i]);
        }
    };
    auto vec_body = [&](int64_t u) {
        const int64_t j0 = u * N;
        int64_t base;
        if (!unit_base<ADDR>(a.index, a.offset, a.numel, a.chunk_shift, j0, N, base)) {
            scalar_body(u);
            return;
        }
        T v[N];
        load_vec<T, NT>(w + base, v);
        float m[N];
#pragma unroll
        for (int e = 0; e < N; ++e) m[e] = to_f32<T>(v[e]);
        store_f32s<N, NT>(master + j0, m);
    };
    for_each_unit<N>(a.length, vec_body, scalar_body);
}

// ----------------------------------------------------------------- update --
// theta_S += step * sum_u c_u eps_u, c_u = sum over members of stream u of
// sign * rnorm.  Each thread reads its unit of weights once, regenerates every
// stream's noise for it in registers, accumulates in fp64 and writes once.
//
// Bound by the VALU.  fp64 runs at the rate of fp32 here, so the sums stay in
// fp64 from the Box-Muller products on: c rho cos and c rho sin are one product
// for the pair and one fma for each sum, where normals rounded to fp32 take a
// product, a conversion and an fma each.  504,654,080 bf16 positions,
// 30 streams: 226 instead of 242 VALU instructions per 8 normals, 11.92 instead
// of 12.27 ms; 64 mirrored pairs on 251 M with a master, 10.46 and 10.75 ms.

// Stream coefficients, and a bit for each stream that contributes: those with
// a coefficient other than zero.  A mirrored pair with equal rewards cancels to
// exactly zero (half of the pairs under success / failure rewards), and so does
// every member when all rewards are equal; c = 0 would add c eps = +-0 to a sum
// that is never -0, so leaving the stream's noise ungenerated changes no bit.
// 16 mirrored pairs with success / failure rewards on 9.4 M bf16 weights: 71 us
// against 143 us; 64 pairs with rewards averaged over 8 rollouts, 251 M weights
// with a master: 10.5 against 13.2 ms.
struct Streams {
    double coef[kMaxMembers];
    uint64_t some[kMaxMembers / 64 + 1];   // a range may start behind the last word
};

// Fold members into stream coefficients, in member order, in fp64; every
// thread of the workgroup must call it (it ends with a barrier).  The members'
// values are gathered into LDS in one round trip, so a workgroup starts after
// two memory latencies whatever the number of members.
__device__ __forceinline__ const Streams* fold_members(const MemberTable& t, int n_members, int n_streams,
                                                       const float* rnorm)
{
    __shared__ Streams st;
    __shared__ float value[kMaxMembers];
    static_assert(kBlock == kMaxMembers, "one thread per member and per stream");
    const int u = threadIdx.x;
    if (u < n_members) {
        const uint32_t m = t.member[u];
        const float r = rnorm[m & (kNegative - 1u)];
        value[u] = (m & kNegative) ? -r : r;
    }
    const int i0 = u < n_streams ? t.first_member[u] : 0, i1 = u < n_streams ? t.first_member[u + 1] : 0;
    __syncthreads();
    double c = 0.0;
    for (int i = i0; i < i1; ++i) c += (double)value[i];
    st.coef[u] = c;
    const uint64_t some = __builtin_amdgcn_ballot_w64(u < n_streams && !(c == 0.0));       // a NaN counts
    if ((u & 63) == 0) st.some[u / 64] = some;
    __syncthreads();
    return &st;
}

// acc[e] = sum over the contributing streams s0 <= s < s1 of c_s eps_s (q-th
// block pair), in stream order.  The bits are tested by the scalar unit, which
// also reads the seeds and runs the key schedule.
template <int N, typename Q>
__device__ __forceinline__ void accumulate_streams(const MemberTable& t, const Streams* st, int s0, int s1, Q q,
                                                   const Bm& tb, float acc[N])
{
    double sum[N];
#pragma unroll
    for (int e = 0; e < N; ++e) sum[e] = 0.0;
    uint64_t bits = (uint64_t)wave_uniform((int64_t)st->some[s0 / 64]) >> (s0 & 63);   // from stream s on
    for (int s = s0; s < s1; ++s) {
        const bool some = bits & 1u;
        bits >>= 1;
        if (((s + 1) & 63) == 0 && s + 1 < s1) bits = (uint64_t)wave_uniform((int64_t)st->some[(s + 1) / 64]);
        if (!some) continue;
        add_normals<N, Q>(t.seed_lo[s], t.seed_hi[s], q, tb, st->coef[s], sum);
    }
#pragma unroll
    for (int e = 0; e < N; ++e) acc[e] = (float)sum[e];
}

template <typename T, bool MASTER, typename Q, int ADDR>
__global__ __launch_bounds__(kBlock) void k_update(UpdateArgs a)
{
    constexpr int N = MASTER ? 8 : UnitOf<T>::n;
    const Bm tb = stage_bm_tables<kBlock>();
    const Streams* st = fold_members(a.members, a.n_members, a.n_streams, a.rnorm);

    T* w = static_cast<T*>(a.w);
    auto accumulate = [&](int64_t j0, float acc[N]) {
        accumulate_streams<N, Q>(a.members, st, 0, a.n_streams, (Q)((uint64_t)(a.noise0 + j0) >> 2), tb, acc);
    };
    auto scalar_finish = [&](int64_t j0, const float acc[N]) {
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const int64_t j = j0 + e;
            int64_t i;
            if (j >= a.length || !param_at<ADDR>(a.index, a.offset, a.numel, a.chunk_shift, j, i)) continue;
            if (MASTER) {
                const float m = __builtin_fmaf(a.step, acc[e], a.master[j]);
                a.master[j] = m;
                w[i] = from_f32<T>(m);
            } else {
                w[i] = from_f32<T>(__builtin_fmaf(a.step, acc[e], to_f32<T>(w[i])));
            }
        }
    };
    auto scalar_body = [&](int64_t u) {
        float acc[N];
        accumulate(u * N, acc);
        scalar_finish(u * N, acc);
    };
    auto vec_body = [&](int64_t u) {
        const int64_t j0 = u * N;
        float acc[N];
        accumulate(j0, acc);
        int64_t base = 0;
        T v[N];
        if (!unit_base<ADDR>(a.index, a.offset, a.numel, a.chunk_shift, j0, N, base)) {
            scalar_finish(j0, acc);
            return;
        }
        if (!MASTER) load_vec<T>(w + base, v);
        T out[N];
        if (MASTER) {
            float m[N];
            load_f32s<N>(a.master + j0, m);
#pragma unroll
            for (int e = 0; e < N; ++e) {
                m[e] = __builtin_fmaf(a.step, acc[e], m[e]);
                out[e] = from_f32<T>(m[e]);
            }
            store_f32s<N>(a.master + j0, m);
        } else {
#pragma unroll
            for (int e = 0; e < N; ++e) out[e] = from_f32<T>(__builtin_fmaf(a.step, acc[e], to_f32<T>(v[e])));
        }
        store_vec<T>(w + base, out);
    };
    for_each_unit<N>(a.length, vec_body, scalar_body);
}

// ------------------------------------------------------- index-map kernels --
// Subspaces given by an element map (int64 or uint32 entries; a partition's
// maps are ascending, at density d_k / d across the weights).  A wave owns
// tiles of 64 N consecutive positions.  Map entries, and the weights they
// address, are taken lane-interleaved: lane l handles positions t0 + l + 64 e,
// e < N.  Each memory instruction then covers 64 consecutive map entries, a
// window of about 64 d / d_k consecutive weights (a few 128-byte lines), where
// a unit per lane would touch 64 windows that far apart.  Noise comes in
// units of N consecutive positions per lane, and so do contiguous side
// buffers (backup, master); a per-wave LDS buffer of one tile converts
// between the two layouts.

template <int ADDR>
__device__ __forceinline__ int64_t map_entry(const int64_t* index, int64_t p)
{
    if (ADDR == kGather) return index[p];
    return (int64_t)reinterpret_cast<const uint32_t*>(index)[p];
}

// The wave's index and the number of waves in the grid (uniform in a wave).
__device__ __forceinline__ int64_t wave_id()
{
    return (int64_t)blockIdx.x * (kBlock / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
}
__device__ __forceinline__ int64_t wave_count() { return (int64_t)gridDim.x * (kBlock / 64); }

// Parameters of lane `lane`'s positions in the tile at t0:
// idx[e] = map[offset + t0 + lane + 64 e], or -1 beyond the subspace or for
// an entry outside [0, numel) (skipped, never dereferenced).  Returns true
// when every entry of the wave is valid (a full tile of a partition's map).
template <int ADDR, int N>
__device__ __forceinline__ bool tile_entries(const int64_t* index, int64_t offset, int64_t length, int64_t numel,
                                             int64_t t0, int lane, int64_t idx[N])
{
    bool ok = true;
    if (t0 + 64 * N <= length) {
#pragma unroll
        for (int e = 0; e < N; ++e) idx[e] = map_entry<ADDR>(index, offset + t0 + lane + 64 * e);
    } else {
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const int64_t j = t0 + lane + 64 * e;
            idx[e] = j < length ? map_entry<ADDR>(index, offset + j) : -1;
        }
        ok = false;
    }
#pragma unroll
    for (int e = 0; e < N; ++e)
        if ((uint64_t)idx[e] >= (uint64_t)numel) {
            idx[e] = -1;
            ok = false;
        }
    return __builtin_amdgcn_ballot_w64(!ok) == 0;
}

// Gather w at the tile's entries (lane-interleaved); skipped entries read 0.
template <typename T, int N>
__device__ __forceinline__ void gather_lanes(const T* w, const int64_t idx[N], bool all_valid, T v[N])
{
    if (all_valid) {
#pragma unroll
        for (int e = 0; e < N; ++e) v[e] = w[idx[e]];
    } else {
#pragma unroll
        for (int e = 0; e < N; ++e) v[e] = idx[e] >= 0 ? w[idx[e]] : T(0);
    }
}

// Scatter lane-interleaved values.  With every entry valid the stores carry
// no branch and issue back to back; a branch around each store would make the
// compiler wait for the loaded data before every one of them.
template <typename T, int N>
__device__ __forceinline__ void scatter_lanes(T* w, const int64_t idx[N], bool all_valid, const T v[N])
{
    if (all_valid) {
#pragma unroll
        for (int e = 0; e < N; ++e) w[idx[e]] = v[e];
    } else {
#pragma unroll
        for (int e = 0; e < N; ++e)
            if (idx[e] >= 0) w[idx[e]] = v[e];
    }
}

// Lane-level ordering of the exchange buffer: LDS accesses of one wave take
// effect in program order, so the compiler only has to keep them in order.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// Units (lane l holds positions N l .. N l + N - 1 of the tile) to lanes
// (lane l holds l + 64 e), and back, through the wave's tile buffer `buf`
// (64 N elements, 16-byte aligned).
template <int BYTES> struct UnitVec;
template <> struct UnitVec<16> { typedef V4u type; };
template <> struct UnitVec<8> { typedef uint2 type; };

template <typename T, int N>
__device__ __forceinline__ void units_to_lanes(T* buf, int lane, const T in[N], T out[N])
{
    typedef typename UnitVec<N * sizeof(T)>::type U;
    *reinterpret_cast<U*>(buf + N * lane) = *reinterpret_cast<const U*>(in);
    wave_lds_sync();
#pragma unroll
    for (int e = 0; e < N; ++e) out[e] = buf[lane + 64 * e];
    wave_lds_sync();
}
template <typename T, int N>
__device__ __forceinline__ void lanes_to_units(T* buf, int lane, const T in[N], T out[N])
{
    typedef typename UnitVec<N * sizeof(T)>::type U;
#pragma unroll
    for (int e = 0; e < N; ++e) buf[lane + 64 * e] = in[e];
    wave_lds_sync();
    *reinterpret_cast<U*>(out) = *reinterpret_cast<const U*>(buf + N * lane);
    wave_lds_sync();
}

// Unit-wise side buffer access at positions j0 .. j0 + N - 1, bounded by
// `length` (a tile may end inside a unit); 16-byte vectors when the unit is
// whole.
template <typename T, int N>
__device__ __forceinline__ void load_unit(const T* p, int64_t j0, int64_t length, T v[N])
{
    if (j0 + N <= length) {
        if (sizeof(T) * N == 16) {
            load_vec<T>(p + j0, v);
        } else {
            load_f32s<N>(reinterpret_cast<const float*>(p) + j0, reinterpret_cast<float*>(v));
        }
    } else {
#pragma unroll
        for (int e = 0; e < N; ++e) v[e] = j0 + e < length ? p[j0 + e] : T(0);
    }
}
template <typename T, int N>
__device__ __forceinline__ void store_unit(T* p, int64_t j0, int64_t length, const T v[N])
{
    if (j0 + N <= length) {
        if (sizeof(T) * N == 16) {
            store_vec<T>(p + j0, v);
        } else {
            store_f32s<N>(reinterpret_cast<float*>(p) + j0, reinterpret_cast<const float*>(v));
        }
    } else {
#pragma unroll
        for (int e = 0; e < N; ++e)
            if (j0 + e < length) p[j0 + e] = v[e];
    }
}

// Perturbation through a map (see k_perturb for the arithmetic).
template <typename T, int AUX, typename Q, int ADDR>
__global__ __launch_bounds__(kBlock) void k_perturb_map(StreamArgs a)
{
    constexpr int N = UnitOf<T>::n;
    const Bm tb = stage_bm_tables<kBlock>();
    __shared__ __attribute__((aligned(16))) T xch[kBlock / 64][64 * N];
    const int lane = threadIdx.x & 63;
    T* buf = xch[threadIdx.x / 64];
    T* w = static_cast<T*>(a.w);
    const int64_t tiles = (a.length + 64 * N - 1) / (64 * N);
    for (int64_t t = wave_id(); t < tiles; t += wave_count()) {
        const int64_t t0 = t * 64 * N, j0 = t0 + (int64_t)N * lane;
        int64_t idx[N];
        const bool all_valid = tile_entries<ADDR, N>(a.index, a.offset, a.length, a.numel, t0, lane, idx);
        float src[N];
        if (AUX == kAuxMaster) {
            load_unit<float, N>(static_cast<const float*>(a.aux), j0, a.length, src);
        } else {
            T old[N];
            if (AUX == kAuxBackup) {
                load_unit<T, N>(static_cast<const T*>(a.aux), j0, a.length, old);
            } else {
                T g[N];
                gather_lanes<T, N>(w, idx, all_valid, g);
                lanes_to_units<T, N>(buf, lane, g, old);
                if (AUX == kAuxSnapshot) store_unit<T, N>(static_cast<T*>(a.aux), j0, a.length, old);
            }
#pragma unroll
            for (int e = 0; e < N; ++e) src[e] = to_f32<T>(old[e]);
        }
        float z[N];
        unit_normals<N, Q>(a.k0, a.k1, (Q)((uint64_t)(a.noise0 + j0) >> 2), tb, z);
        T out[N], v[N];
#pragma unroll
        for (int e = 0; e < N; ++e) out[e] = from_f32<T>(__builtin_fmaf(a.scale, z[e], src[e]));
        units_to_lanes<T, N>(buf, lane, out, v);
        scatter_lanes<T, N>(w, idx, all_valid, v);
    }
}

// Copies through a map, all lane-interleaved (no noise, no exchange):
// KIND 0: w[p(j)] = aux[j] (restore from the backup);
// KIND 1: aux[j] = w[p(j)] (backup; skipped entries give 0);
// KIND 2: w[p(j)] = rne_bf16(master[j]) (restore from a master);
// KIND 3: master[j] = f32(w[p(j)]) (master staging).
constexpr int kCopyRestore = 0, kCopyBackup = 1, kCopyRestoreMaster = 2, kCopyStageMaster = 3;

template <typename T, int KIND, bool NT, int ADDR>
__global__ __launch_bounds__(kBlock) void k_copy_map(StreamArgs a)
{
    constexpr int N = UnitOf<T>::n;
    const int lane = threadIdx.x & 63;
    T* w = static_cast<T*>(a.w);
    const int64_t tiles = (a.length + 64 * N - 1) / (64 * N);
    for (int64_t t = wave_id(); t < tiles; t += wave_count()) {
        const int64_t t0 = t * 64 * N;
        int64_t idx[N];
        const bool all_valid = tile_entries<ADDR, N>(a.index, a.offset, a.length, a.numel, t0, lane, idx);
        const bool full = t0 + 64 * N <= a.length;
        if (KIND == kCopyRestore || KIND == kCopyRestoreMaster) {
            T v[N];
#pragma unroll
            for (int e = 0; e < N; ++e) {
                const int64_t j = t0 + lane + 64 * e;
                if (KIND == kCopyRestore) {
                    const T* snap = static_cast<const T*>(a.aux);
                    v[e] = full || j < a.length ? (NT ? __builtin_nontemporal_load(snap + j) : snap[j]) : T(0);
                } else {
                    const float* master = static_cast<const float*>(a.aux);
                    const float m = full || j < a.length ? (NT ? __builtin_nontemporal_load(master + j) : master[j])
                                                        : 0.0f;
                    v[e] = from_f32<T>(m);
                }
            }
            scatter_lanes<T, N>(w, idx, all_valid, v);
        } else {
            T v[N];
            gather_lanes<T, N>(w, idx, all_valid, v);
#pragma unroll
            for (int e = 0; e < N; ++e) {
                const int64_t j = t0 + lane + 64 * e;
                if (!full && j >= a.length) continue;
                if (KIND == kCopyBackup) {
                    T* backup = static_cast<T*>(a.aux);
                    if (NT) __builtin_nontemporal_store(v[e], backup + j);
                    else backup[j] = v[e];
                } else {
                    float* master = static_cast<float*>(a.aux);
                    if (NT) __builtin_nontemporal_store(to_f32<T>(v[e]), master + j);
                    else master[j] = to_f32<T>(v[e]);
                }
            }
        }
    }
}

// ------------------------------------------ dense windows on ascending maps --
// Restores through a strictly ascending element map (a partition's own maps,
// flagged CPES_SUB_ASCENDING).  The weights a wave tile of kDenseTile entries
// touches lie in a narrow window of 128-byte lines.  Each line belongs to the
// tile holding the line's first entry of the subspace; that tile's wave reads
// its lines whole into LDS, overlays its entries -- and those of the next
// tile that fall in its last line (at most 63, the "spill") -- and writes the
// lines back whole.  Each line is then written once and in full, where
// scattered 2-byte stores leave a partial write in nearly every 32-byte
// sector at density 1/8, which the memory system completes by reading the
// sector first.  The other parameters in those lines are written back with
// the values just read.  A tile whose lines do not fit the window (a
// subspace sparser than about 1/10) stores its entries one by one, keeping
// line ownership: it still takes its spill and leaves the entries in a shared
// first line to the previous tile.  bf16 weights only; any map entry outside
// [0, numel) is skipped.  (Perturbations tile without a spill, below, so
// that a wave generates the noise of its own tile's positions only.)
constexpr int kDenseTile = 256;      // entries per wave tile: 4 per lane
constexpr int kDensePer = kDenseTile / 64;
constexpr int kLineElems = 64;       // bf16 elements per 128-byte line
constexpr int kDenseLines = 40;      // LDS window per wave: 5 KiB

struct DenseTile {
    int64_t t0, t1;     // the tile's entries [t0, t1)
    int64_t lo, hi;     // lines [lo, hi] it owns
    bool window;        // the owned lines fit the LDS window (and the tile's ends are in range)
};

template <int ADDR>
__device__ __forceinline__ DenseTile dense_tile(const int64_t* index, int64_t offset, int64_t length, int64_t numel,
                                                int64_t t, int64_t tile)
{
    DenseTile d;
    d.t0 = t * tile;
    d.t1 = d.t0 + tile < length ? d.t0 + tile : length;
    const int64_t first = wave_uniform(map_entry<ADDR>(index, offset + d.t0));
    const int64_t last = wave_uniform(map_entry<ADDR>(index, offset + d.t1 - 1));
    const int64_t A = first >> 6, B = last >> 6;      // floor division by kLineElems
    bool shared = false;
    if (d.t0 > 0) shared = (wave_uniform(map_entry<ADDR>(index, offset + d.t0 - 1)) >> 6) == A;
    d.lo = shared ? A + 1 : A;
    d.hi = B;
    d.window = first >= 0 && last < numel && first <= last && d.hi - d.lo + 1 <= kDenseLines;
    return d;
}

// The tile's own entries (lane-interleaved: position t0 + lane + 64 e) with
// the entries of a shared first line dropped, and this lane's spill entry
// (position t1 + lane, kept if it falls in line hi); -1 where there is none.
template <int ADDR>
__device__ __forceinline__ void dense_entries(const int64_t* index, int64_t offset, int64_t length, int64_t numel,
                                              const DenseTile& d, int lane, int64_t idx[kDensePer], int64_t& sidx)
{
#pragma unroll
    for (int e = 0; e < kDensePer; ++e) {
        const int64_t j = d.t0 + lane + 64 * e;
        int64_t i = j < d.t1 ? map_entry<ADDR>(index, offset + j) : -1;
        if ((uint64_t)i >= (uint64_t)numel || (i >> 6) < d.lo) i = -1;
        idx[e] = i;
    }
    sidx = -1;
    const int64_t j = d.t1 + lane;
    if (j < length) {
        const int64_t i = map_entry<ADDR>(index, offset + j);
        if ((uint64_t)i < (uint64_t)numel && (i >> 6) == d.hi) sidx = i;
    }
}

// Window transfers: lines [lo, hi] of w to and from the wave's LDS buffer,
// one 16-byte vector per lane per step, non-temporal (the weights far exceed
// the caches); the element path covers a window running past numel.  Lines
// count from the first weight, which may lie at any element's address.
__device__ __forceinline__ void window_load(const uint16_t* w, int64_t numel, const DenseTile& d, uint16_t* buf,
                                            int lane)
{
    const int64_t base = d.lo * kLineElems, nvec = (d.hi - d.lo + 1) * (kLineElems / 8);
    const bool whole = base + nvec * 8 <= numel;
    typedef Vec16<uint16_t>::type V;
    for (int64_t v = lane; v < nvec; v += 64) {
        if (whole) {
            *reinterpret_cast<V4u*>(buf + 8 * v) =
                __builtin_nontemporal_load(reinterpret_cast<const V*>(w + base) + v);
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int64_t i = base + 8 * v + k;
                buf[8 * v + k] = i < numel ? w[i] : (uint16_t)0;
            }
        }
    }
}
__device__ __forceinline__ void window_store(uint16_t* w, int64_t numel, const DenseTile& d, const uint16_t* buf,
                                             int lane)
{
    const int64_t base = d.lo * kLineElems, nvec = (d.hi - d.lo + 1) * (kLineElems / 8);
    const bool whole = base + nvec * 8 <= numel;
    typedef Vec16<uint16_t>::type V;
    for (int64_t v = lane; v < nvec; v += 64) {
        if (whole) {
            __builtin_nontemporal_store(*reinterpret_cast<const V4u*>(buf + 8 * v),
                                        reinterpret_cast<V*>(w + base) + v);
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int64_t i = base + 8 * v + k;
                if (i < numel) w[i] = buf[8 * v + k];
            }
        }
    }
}

// Write the tile's new values: overlaid on the window and stored whole, or
// (no window) stored one by one.
__device__ __forceinline__ void dense_write(uint16_t* w, int64_t numel, const DenseTile& d, uint16_t* buf, int lane,
                                            const int64_t idx[kDensePer], const uint16_t v[kDensePer], int64_t sidx,
                                            uint16_t sv)
{
    if (d.window) {
        const int64_t base = d.lo * kLineElems, nelem = (d.hi - d.lo + 1) * kLineElems;
#pragma unroll
        for (int e = 0; e < kDensePer; ++e)
            if (idx[e] >= base && idx[e] < base + nelem) buf[idx[e] - base] = v[e];
        if (sidx >= base && sidx < base + nelem) buf[sidx - base] = sv;
        wave_lds_sync();
        window_store(w, numel, d, buf, lane);
        wave_lds_sync();
    } else {
#pragma unroll
        for (int e = 0; e < kDensePer; ++e)
            if (idx[e] >= 0) w[idx[e]] = v[e];
        if (sidx >= 0) w[sidx] = sv;
    }
}

// Restore through an ascending map: w[p(j)] = aux[j] (bf16 backup, KIND
// kCopyRestore) or rne_bf16(aux[j]) (fp32 master, KIND kCopyRestoreMaster).
template <int KIND, int ADDR>
__global__ __launch_bounds__(kBlock) void k_restore_dense(StreamArgs a)
{
    __shared__ __attribute__((aligned(16))) uint16_t win[kBlock / 64][kDenseLines * kLineElems];
    const int lane = threadIdx.x & 63;
    uint16_t* buf = win[threadIdx.x / 64];
    uint16_t* w = static_cast<uint16_t*>(a.w);
    auto source = [&](int64_t j) -> uint16_t {
        if (KIND == kCopyRestore) return __builtin_nontemporal_load(static_cast<const uint16_t*>(a.aux) + j);
        return f32_to_bf16(__builtin_nontemporal_load(static_cast<const float*>(a.aux) + j));
    };
    const int64_t tiles = (a.length + kDenseTile - 1) / kDenseTile;
    for (int64_t t = wave_id(); t < tiles; t += wave_count()) {
        const DenseTile d = dense_tile<ADDR>(a.index, a.offset, a.length, a.numel, t, kDenseTile);
        int64_t idx[kDensePer], sidx;
        dense_entries<ADDR>(a.index, a.offset, a.length, a.numel, d, lane, idx, sidx);
        uint16_t v[kDensePer], sv = 0;
#pragma unroll
        for (int e = 0; e < kDensePer; ++e) v[e] = idx[e] >= 0 ? source(d.t0 + lane + 64 * e) : (uint16_t)0;
        if (sidx >= 0) sv = source(d.t1 + lane);
        if (d.window) {
            window_load(w, a.numel, d, buf, lane);
            wave_lds_sync();
        }
        dense_write(w, a.numel, d, buf, lane, idx, v, sidx, sv);
    }
}

// ----------------------------------- whole-line perturbations (ascending) --
// A perturbation through an ascending map writes whole lines too, on fixed
// tiles of kDenseTile entries but without a spill: the lines strictly inside
// a tile's span hold no entry of another tile and go through the tile's LDS
// window; its entries in a first or last line shared with a neighbouring tile
// are stored one by one, as the neighbour stores its own entries there, so a
// line written whole has no other writer.  Lane l takes the tile's positions
// t0 + 4 l .. t0 + 4 l + 3, which are one Philox block of noise, and moves
// the map and the side buffers as 8- or 16-byte vectors.  The
// perturbation is that of Eq. (8) on a subspace of the partition of Eq. (7).
// (Restores tiled this way, with no noise to generate, measured a few per
// cent slower than the spill kernel above, which they therefore keep.)
template <int ADDR>
__device__ __forceinline__ DenseTile edge_tile(const int64_t* index, int64_t offset, int64_t length, int64_t numel,
                                               int64_t t)
{
    DenseTile d;
    d.t0 = t * kDenseTile;
    d.t1 = d.t0 + kDenseTile < length ? d.t0 + kDenseTile : length;
    const int64_t first = wave_uniform(map_entry<ADDR>(index, offset + d.t0));
    const int64_t last = wave_uniform(map_entry<ADDR>(index, offset + d.t1 - 1));
    const int64_t A = first >> 6, B = last >> 6;
    const bool prev = d.t0 > 0 && (wave_uniform(map_entry<ADDR>(index, offset + d.t0 - 1)) >> 6) == A;
    const bool next = d.t1 < length && (wave_uniform(map_entry<ADDR>(index, offset + d.t1)) >> 6) == B;
    d.lo = prev ? A + 1 : A;
    d.hi = next ? B - 1 : B;
    if (d.hi < d.lo) d.hi = d.lo - 1;   // every entry lies in a shared line: an empty window
    d.window = first >= 0 && last < numel && first <= last && d.hi - d.lo + 1 <= kDenseLines;
    return d;
}

// Entries p .. p + 3 of the map (n of them exist; -1 for the others and for
// entries outside [0, numel)).
template <int ADDR>
__device__ __forceinline__ void map_entries4(const int64_t* index, int64_t p, int64_t n, int64_t numel,
                                             int64_t idx[4])
{
    if (n >= 4) {
        typedef Vec16<float>::type V;
        if (ADDR == kGather) {
            const V4u x = *reinterpret_cast<const V*>(index + p);
            const V4u y = *reinterpret_cast<const V*>(index + p + 2);
            idx[0] = (int64_t)(((uint64_t)x[1] << 32) | x[0]);
            idx[1] = (int64_t)(((uint64_t)x[3] << 32) | x[2]);
            idx[2] = (int64_t)(((uint64_t)y[1] << 32) | y[0]);
            idx[3] = (int64_t)(((uint64_t)y[3] << 32) | y[2]);
        } else {
            const V4u x = *reinterpret_cast<const V*>(reinterpret_cast<const uint32_t*>(index) + p);
#pragma unroll
            for (int e = 0; e < 4; ++e) idx[e] = (int64_t)x[e];
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) idx[e] = e < n ? map_entry<ADDR>(index, p + e) : -1;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if ((uint64_t)idx[e] >= (uint64_t)numel) idx[e] = -1;
}

// The tile's new values: those in the window (in[e]) overlaid on it and its
// lines stored whole, the others (in a shared line, or all of them when the
// tile has no window) stored one by one.
__device__ __forceinline__ void edge_write(uint16_t* w, int64_t numel, const DenseTile& d, uint16_t* buf, int lane,
                                           const int64_t idx[4], const bool in[4], int64_t base, const uint16_t v[4])
{
    if (d.window) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (in[e]) buf[idx[e] - base] = v[e];
        wave_lds_sync();
        window_store(w, numel, d, buf, lane);
        wave_lds_sync();
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (!in[e] && idx[e] >= 0) w[idx[e]] = v[e];
}

// Workgroups of kDenseBlock threads share one copy of the noise tables; with
// at most 80 VGPRs, three of them (52 KiB of LDS each) give 6 waves per SIMD,
// where 256-thread workgroups (32 KiB each) give 5.  Measured on 0.5 G-entry
// maps: 6-20 % faster, except the perturbation from the backup through an
// int64 map (3 % slower).
constexpr int kDenseBlock = 512;

template <int AUX, typename Q, int ADDR>
__global__ __launch_bounds__(kDenseBlock, 6) void k_perturb_dense(StreamArgs a)
{
    const Bm tb = stage_bm_tables<kDenseBlock>();
    __shared__ __attribute__((aligned(16))) uint16_t win[kDenseBlock / 64][kDenseLines * kLineElems];
    const int lane = threadIdx.x & 63;
    uint16_t* buf = win[threadIdx.x / 64];
    uint16_t* w = static_cast<uint16_t*>(a.w);
    const int64_t tiles = (a.length + kDenseTile - 1) / kDenseTile;
    const int64_t waves = (int64_t)gridDim.x * (kDenseBlock / 64);
    for (int64_t t = (int64_t)blockIdx.x * (kDenseBlock / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x / 64); t < tiles;
         t += waves) {
        const DenseTile d = edge_tile<ADDR>(a.index, a.offset, a.length, a.numel, t);
        const int64_t j0 = d.t0 + 4 * lane;
        const bool whole = j0 + 4 <= a.length;
        int64_t idx[4];
        map_entries4<ADDR>(a.index, a.offset + j0, a.length - j0, a.numel, idx);
        float src[4];
        if (AUX == kAuxBackup) {
            const uint16_t* b = static_cast<const uint16_t*>(a.aux) + j0;
            uint16_t o[4];
            if (whole) {
                *reinterpret_cast<V2u*>(o) = *reinterpret_cast<const V2uAnywhere*>(b);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = j0 + e < a.length ? b[e] : (uint16_t)0;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) src[e] = bf16_to_f32(o[e]);
        } else if (AUX == kAuxMaster) {
            const float* m = static_cast<const float*>(a.aux) + j0;
            if (whole) {
                load_f32s<4>(m, src);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) src[e] = j0 + e < a.length ? m[e] : 0.0f;
            }
        }
        float z[4];
        normals4<Q>(a.k0, a.k1, (Q)((uint64_t)(a.noise0 + j0) >> 2), tb, z);
        int64_t base = 0, nelem = 0;
        if (d.window) {
            base = d.lo * kLineElems;
            nelem = (d.hi - d.lo + 1) * kLineElems;
            window_load(w, a.numel, d, buf, lane);
            wave_lds_sync();
        }
        bool in[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) in[e] = idx[e] >= base && idx[e] < base + nelem;
        if (AUX == kAuxNone || AUX == kAuxSnapshot) {
            uint16_t o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = in[e] ? buf[idx[e] - base] : idx[e] >= 0 ? w[idx[e]] : (uint16_t)0;
            if (AUX == kAuxSnapshot) {
                uint16_t* snap = static_cast<uint16_t*>(a.aux) + j0;
                if (whole) {
                    *reinterpret_cast<V2uAnywhere*>(snap) = *reinterpret_cast<const V2u*>(o);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (j0 + e < a.length) snap[e] = o[e];
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) src[e] = bf16_to_f32(o[e]);
        }
        uint16_t v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = f32_to_bf16(__builtin_fmaf(a.scale, z[e], src[e]));
        edge_write(w, a.numel, d, buf, lane, idx, in, base, v);
    }
}

// Update through a map (see k_update for the arithmetic).
template <typename T, bool MASTER, typename Q, int ADDR>
__global__ __launch_bounds__(kBlock) void k_update_map(UpdateArgs a)
{
    constexpr int N = UnitOf<T>::n;   // a master update has bf16 weights: N = 8
    const Bm tb = stage_bm_tables<kBlock>();
    __shared__ __attribute__((aligned(16))) T xch[kBlock / 64][64 * N];
    const Streams* st = fold_members(a.members, a.n_members, a.n_streams, a.rnorm);
    const int lane = threadIdx.x & 63;
    T* buf = xch[threadIdx.x / 64];
    T* w = static_cast<T*>(a.w);
    const int64_t tiles = (a.length + 64 * N - 1) / (64 * N);
    for (int64_t t = wave_id(); t < tiles; t += wave_count()) {
        const int64_t t0 = t * 64 * N, j0 = t0 + (int64_t)N * lane;
        int64_t idx[N];
        const bool all_valid = tile_entries<ADDR, N>(a.index, a.offset, a.length, a.numel, t0, lane, idx);
        T g[N];
        if (!MASTER) gather_lanes<T, N>(w, idx, all_valid, g);   // in flight while the noise is generated
        float acc[N];
        accumulate_streams<N, Q>(a.members, st, 0, a.n_streams, (Q)((uint64_t)(a.noise0 + j0) >> 2), tb, acc);
        T out[N], v[N];
        if (MASTER) {
            float m[N];
            load_unit<float, N>(a.master, j0, a.length, m);
#pragma unroll
            for (int e = 0; e < N; ++e) {
                m[e] = __builtin_fmaf(a.step, acc[e], m[e]);
                out[e] = from_f32<T>(m[e]);
            }
            store_unit<float, N>(a.master, j0, a.length, m);
        } else {
            T old[N];
            lanes_to_units<T, N>(buf, lane, g, old);
#pragma unroll
            for (int e = 0; e < N; ++e) out[e] = from_f32<T>(__builtin_fmaf(a.step, acc[e], to_f32<T>(old[e])));
        }
        units_to_lanes<T, N>(buf, lane, out, v);
        scatter_lanes<T, N>(w, idx, all_valid, v);
    }
}

// ------------------------------------------------------------ step update --
// theta += sum_k P_k step_k sum_{u in streams of k} c_u eps_u (Eq. 13, Alg. 1):
// every subspace of the partition with its own members, in one launch.  Units
// restart at each subspace's first position, so noise position j is always
// relative to the subspace; each wave works on 64 units of one subspace (one
// tile, taken lane-interleaved on an element map as in the map kernels).
template <typename T, typename Q, int ADDR>
__global__ __launch_bounds__(kBlock) void k_update_step(StepArgs a)
{
    constexpr int N = UnitOf<T>::n;
    const Bm tb = stage_bm_tables<kBlock>();
    __shared__ __attribute__((aligned(16))) T xch[kBlock / 64][64 * N];
    const Streams* st = fold_members(a.members, a.n_members, a.n_streams, a.rnorm);
    T* w = static_cast<T*>(a.w);
    const int lane = threadIdx.x & 63;
    T* buf = xch[threadIdx.x / 64];
    const int64_t tiles = a.tile_begin[a.K];
    for (int64_t t = wave_id(); t < tiles; t += wave_count()) {
        // t is the same for the whole wave; so are k and the stream range, which
        // keeps the seed and coefficient reads scalar
        int k = 0;
        while (k + 1 < a.K && a.tile_begin[k + 1] <= t) ++k;
        k = __builtin_amdgcn_readfirstlane(k);
        const int st0 = __builtin_amdgcn_readfirstlane(a.stream_begin[k]);
        const int st1 = __builtin_amdgcn_readfirstlane(a.stream_begin[k + 1]);
        const int64_t off = a.offset[k];
        const int64_t len = a.length[k];
        const float step = a.step[k];
        const int64_t t0 = (t - a.tile_begin[k]) * 64 * N;
        const int64_t j0 = t0 + (int64_t)N * lane;
        if (kMap<ADDR>) {
            int64_t idx[N];
            const bool all_valid = tile_entries<ADDR, N>(a.index, off, len, a.numel, t0, lane, idx);
            T g[N], old[N], out[N], v[N];
            gather_lanes<T, N>(w, idx, all_valid, g);
            float acc[N];
            accumulate_streams<N, Q>(a.members, st, st0, st1, (Q)((uint64_t)j0 >> 2), tb, acc);
            lanes_to_units<T, N>(buf, lane, g, old);
#pragma unroll
            for (int e = 0; e < N; ++e) out[e] = from_f32<T>(__builtin_fmaf(step, acc[e], to_f32<T>(old[e])));
            units_to_lanes<T, N>(buf, lane, out, v);
            scatter_lanes<T, N>(w, idx, all_valid, v);
            continue;
        }
        if (j0 >= len) continue;
        int64_t base = 0;
        const bool vec = j0 + N <= len &&
                         unit_base<ADDR>(a.index, off, a.numel, a.chunk_shift, j0, N, base);
        float acc[N];
        accumulate_streams<N, Q>(a.members, st, st0, st1, (Q)((uint64_t)j0 >> 2), tb, acc);
        if (vec) {
            T v[N], out[N];
            load_vec<T>(w + base, v);
#pragma unroll
            for (int e = 0; e < N; ++e) out[e] = from_f32<T>(__builtin_fmaf(step, acc[e], to_f32<T>(v[e])));
            store_vec<T>(w + base, out);
        } else {
#pragma unroll
            for (int e = 0; e < N; ++e) {
                const int64_t j = j0 + e;
                int64_t i;
                if (j >= len || !param_at<ADDR>(a.index, off, a.numel, a.chunk_shift, j, i)) continue;
                w[i] = from_f32<T>(__builtin_fmaf(step, acc[e], to_f32<T>(w[i])));
            }
        }
    }
}

// -------------------------------------------------------------- normalise --
// Bound by latency: at most 4,096 rewards, 16 KiB.  Three kernels share the
// work by what has to be known of the other rewards:
//  * k_normalize_z, joint z-scores: one workgroup holds all rewards in
//    registers and needs two sums;
//  * k_normalize_z_groups: a workgroup per group, which reads all rewards and
//    sums its own;
//  * k_normalize_rank: a workgroup per 16 rewards, which counts, for each of
//    them, the smaller and the equal ones among all;
// and k_normalize (sorted, one workgroup) takes the last two where the output
// overlaps the inputs, since there another workgroup's result could be read
// for a reward.  Per call, launch included, of 4,096 rewards: joint z-scores
// 75 -> 5.2 us, ranks 64 -> 8.8 us, z-scores in 64 groups 63 -> 7.8 us (first
// figure: sorted); of 30 rewards 5.6 -> 5.1 us.
//
// The fp64 sums are taken in a fixed order (a thread's entries in index order,
// an xor-shuffle butterfly over the wave, the waves in order), so results are
// the same from run to run.
constexpr int kNormMaxN = 4096;
constexpr int kNormMaxGroups = 1024;

__device__ __forceinline__ uint32_t order_bits(float v)
{
    uint32_t u = __float_as_uint(v == 0.0f ? 0.0f : v);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float from_order_bits(uint32_t o)
{
    return __uint_as_float((o & 0x80000000u) ? (o & 0x7FFFFFFFu) : ~o);
}

__device__ __forceinline__ double wave_sum(double x)
{
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) x += __shfl_xor(x, m, 64);
    return x;
}

// Sum over the workgroup, the same in every thread; `part` is written once per call.
template <int WAVES>
__device__ __forceinline__ double block_sum(double x, double* part)
{
    x = wave_sum(x);
    if (WAVES == 1) return x;
    if ((threadIdx.x & 63) == 0) part[threadIdx.x / 64] = x;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) s += part[w];
    return s;
}

// Whether `x` is set in any thread of the workgroup.
template <int WAVES>
__device__ __forceinline__ int block_or(int x, int* part)
{
    const int any = (__builtin_amdgcn_ballot_w64(x & 1) != 0 ? 1 : 0) | (__builtin_amdgcn_ballot_w64(x & 2) != 0 ? 2 : 0);
    if (WAVES == 1) return any;
    if ((threadIdx.x & 63) == 0) part[threadIdx.x / 64] = any;
    __syncthreads();
    int s = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) s |= part[w];
    return s;
}

// Joint z-scores, four rewards per thread: one wave up to 256 rewards (no
// barrier), 4 and 16 waves above.
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_normalize_z(NormalizeArgs a)
{
#pragma clang fp contract(off)
    constexpr int kPer = 4;
    __shared__ double part[2][WAVES];
    __shared__ int flag[WAVES];
    float r[kPer];
    int bad = 0;
    double sum = 0.0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int i = (int)threadIdx.x + 64 * WAVES * k;
        r[k] = i < a.n ? a.r[i] : 0.0f;
        if (!__builtin_isfinite(r[k])) bad = 1;
        sum += (double)r[k];
    }
    bad = block_or<WAVES>(bad, flag);
    const double mu = block_sum<WAVES>(sum, part[0]) / (double)a.n;
    double dev2 = 0.0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const double dev = (int)threadIdx.x + 64 * WAVES * k < a.n ? (double)r[k] - mu : 0.0;
        dev2 += dev * dev;
    }
    const double sd = __builtin_sqrt(block_sum<WAVES>(dev2, part[1]) / (double)a.n);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int i = (int)threadIdx.x + 64 * WAVES * k;
        if (i < a.n) a.out[i] = bad == 0 && sd > 0.0 ? (float)(((double)r[k] - mu) / sd) : 0.0f;
    }
    if (a.status && threadIdx.x == 0) *a.status = bad;
}

// Failures of a grouped or ranked call: every output 0, written by the first
// workgroup alone.  Returns whether the call failed.
__device__ __forceinline__ bool normalize_failed(const NormalizeArgs& a, int bad)
{
    const int status = (bad & 2) ? 2 : (bad & 1);
    if (blockIdx.x == 0) {
        if (status != 0)
            for (int i = threadIdx.x; i < a.n; i += blockDim.x) a.out[i] = 0.0f;
        if (a.status && threadIdx.x == 0) *a.status = status;
    }
    return status != 0;
}

// Z-scores by group: workgroup g sums the rewards of group g.
__global__ __launch_bounds__(kBlock) void k_normalize_z_groups(NormalizeArgs a)
{
#pragma clang fp contract(off)
    constexpr int kWaves = kBlock / 64, kPer = kNormMaxN / kBlock;
    __shared__ double part[3][kWaves];
    __shared__ int flag[kWaves];
    float r[kPer];
    uint32_t mine = 0;
    int bad = 0;
    double sum = 0.0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int i = (int)threadIdx.x + kBlock * k;
        const int32_t g = i < a.n ? a.group[i] : 0;
        r[k] = i < a.n ? a.r[i] : 0.0f;
        if (!__builtin_isfinite(r[k])) bad |= 1;
        if (g < 0 || g >= a.n_groups) bad |= 2;
        if (i < a.n && g == (int32_t)blockIdx.x) {
            mine |= 1u << k;
            sum += (double)r[k];
        }
    }
    if (normalize_failed(a, block_or<kWaves>(bad, flag))) return;
    const double c = block_sum<kWaves>((double)__builtin_popcount(mine), part[0]);
    const double mu = block_sum<kWaves>(sum, part[1]) / c;
    double dev2 = 0.0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const double dev = (mine >> k) & 1u ? (double)r[k] - mu : 0.0;
        dev2 += dev * dev;
    }
    const double sd = __builtin_sqrt(block_sum<kWaves>(dev2, part[2]) / c);
#pragma unroll
    for (int k = 0; k < kPer; ++k)
        if ((mine >> k) & 1u)
            a.out[threadIdx.x + kBlock * k] = sd > 0.0 ? (float)(((double)r[k] - mu) / sd) : 0.0f;
}

// Centred ranks: 16 rewards per workgroup, 16 threads count for each of them,
// every sixteenth entry of all rewards in LDS.
constexpr int kRankPer = 16;

template <bool GROUPS>
__global__ __launch_bounds__(kBlock) void k_normalize_rank(NormalizeArgs a)
{
#pragma clang fp contract(off)
    constexpr int kWaves = kBlock / 64, kThreads = kBlock / kRankPer;
    __shared__ uint32_t value[kNormMaxN];
    __shared__ uint16_t group[GROUPS ? kNormMaxN : 1];
    __shared__ int flag[kWaves];
    int bad = 0;
    for (int i = threadIdx.x; i < a.n; i += kBlock) {
        const float r = a.r[i];
        if (!__builtin_isfinite(r)) bad |= 1;
        value[i] = order_bits(r);
        if (GROUPS) {
            const int32_t g = a.group[i];
            if (g < 0 || g >= a.n_groups) bad |= 2;
            group[i] = (uint16_t)g;
        }
    }
    if (normalize_failed(a, block_or<kWaves>(bad, flag))) return;
    const int i = (int)blockIdx.x * kRankPer + (int)threadIdx.x / kThreads;
    const uint32_t v = i < a.n ? value[i] : 0u;
    const uint32_t g = GROUPS && i < a.n ? group[i] : 0u;
    int less = 0, equal = 0, count = 0;
#pragma unroll 8
    for (int j = threadIdx.x % kThreads; j < a.n; j += kThreads) {
        const uint32_t vj = value[j];
        const bool same = GROUPS ? group[j] == g : true;       // no branches: every read is in flight at once
        less += (int)(same & (vj < v));
        equal += (int)(same & (vj == v));
        if (GROUPS) count += (int)same;
    }
#pragma unroll
    for (int m = kThreads / 2; m > 0; m >>= 1) {
        less += __shfl_xor(less, m, 64);
        equal += __shfl_xor(equal, m, 64);
        if (GROUPS) count += __shfl_xor(count, m, 64);
    }
    if (!GROUPS) count = a.n;
    if (i < a.n && threadIdx.x % kThreads == 0) {
        const double rank = (double)less + 0.5 * (double)(equal - 1);
        a.out[i] = count > 1 ? (float)(rank / (double)(count - 1) - 0.5) : 0.0f;
    }
}

// Z-scores of groups and ranks in place, one workgroup.  The rewards are sorted in LDS by
// the 64-bit key (group, value, index) -- the value as an order-preserving
// 32-bit image of the fp32 bits, -0 taken as +0 -- with a bitonic network.
// Each group is then one run of the sorted keys.  Z: one wave per group sums
// the run in fp64 (lane l takes run entries l, l + 64, ... in order, then the
// butterfly), for the mean and then for the squared deviations.  RANK: the
// rank of an entry is the start of its run of equal values within its group,
// the number of ties the run's length, both found by binary search.
constexpr int kNormThreads = 1024;
constexpr int kNormIdxBits = 12;                 // index < kNormMaxN
constexpr int kNormValShift = kNormIdxBits;      // value bits 12 .. 43
constexpr int kNormGroupShift = kNormIdxBits + 32;   // group bits 44 .. 53
static_assert((1 << kNormIdxBits) >= kNormMaxN && kNormMaxGroups <= (1 << (64 - kNormGroupShift - 1)),
              "index, value and group fit the sort key");

// First position p in [0, n) with keys[p] >= x (keys ascending).
__device__ __forceinline__ int lower_bound_u64(const uint64_t* keys, int n, uint64_t x)
{
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (keys[mid] < x)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

__global__ __launch_bounds__(kNormThreads) void k_normalize(NormalizeArgs a)
{
#pragma clang fp contract(off)
    __shared__ uint64_t keys[kNormMaxN];
    __shared__ int32_t start[kNormMaxGroups + 1];
    __shared__ int bad;
    if (threadIdx.x == 0) bad = 0;
    __syncthreads();
    int n2 = 1;
    while (n2 < a.n) n2 <<= 1;
    int my_bad = 0;
    for (int i = threadIdx.x; i < n2; i += blockDim.x) {
        uint64_t key = ~0ull;                              // padding sorts last
        if (i < a.n) {
            const float v = a.r[i];
            const int32_t gi = a.group ? a.group[i] : 0;
            if (!__builtin_isfinite(v)) my_bad |= 1;
            if (gi < 0 || gi >= a.n_groups) my_bad |= 2;
            key = ((uint64_t)(uint32_t)gi << kNormGroupShift) | ((uint64_t)order_bits(v) << kNormValShift) |
                  (uint64_t)i;
        }
        keys[i] = key;
    }
    if (my_bad) atomicOr(&bad, my_bad);
    __syncthreads();
    const int status = (bad & 2) ? 2 : (bad & 1) ? 1 : 0;
    if (status != 0) {
        for (int i = threadIdx.x; i < a.n; i += blockDim.x) a.out[i] = 0.0f;
        if (a.status && threadIdx.x == 0) *a.status = status;
        return;
    }
    // bitonic sort, ascending
    for (int k = 2; k <= n2; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < n2; i += blockDim.x) {
                const int p = i ^ j;
                if (p > i) {
                    const uint64_t x = keys[i], y = keys[p];
                    if ((x > y) == ((i & k) == 0)) {
                        keys[i] = y;
                        keys[p] = x;
                    }
                }
            }
            __syncthreads();
        }
    }
    // group g is the run [start[g], start[g + 1])
    for (int g = threadIdx.x; g <= a.n_groups; g += blockDim.x)
        start[g] = lower_bound_u64(keys, a.n, (uint64_t)g << kNormGroupShift);
    __syncthreads();
    constexpr uint64_t kIdxMask = (1ull << kNormIdxBits) - 1ull;
    if (a.mode == 0) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
        for (int g = wave; g < a.n_groups; g += waves) {
            const int s0 = start[g], s1 = start[g + 1], c = s1 - s0;
            if (c == 0) continue;
            double part = 0.0;
            for (int p = s0 + lane; p < s1; p += 64)
                part += (double)from_order_bits((uint32_t)(keys[p] >> kNormValShift));
            const double mu = wave_sum(part) / (double)c;
            part = 0.0;
            for (int p = s0 + lane; p < s1; p += 64) {
                const double dev = (double)from_order_bits((uint32_t)(keys[p] >> kNormValShift)) - mu;
                part += dev * dev;
            }
            const double sd = __builtin_sqrt(wave_sum(part) / (double)c);
            for (int p = s0 + lane; p < s1; p += 64) {
                const int i = (int)(keys[p] & kIdxMask);
                a.out[i] = sd > 0.0 ? (float)(((double)a.r[i] - mu) / sd) : 0.0f;
            }
        }
    } else {
        for (int p = threadIdx.x; p < a.n; p += blockDim.x) {
            const uint64_t key = keys[p];
            const int g = (int)(key >> kNormGroupShift);
            const uint64_t first = key & ~kIdxMask;           // (group, value, index 0)
            const int lo = lower_bound_u64(keys, a.n, first);
            const int hi = lower_bound_u64(keys, a.n, first + (kIdxMask + 1));
            const int c = start[g + 1] - start[g];
            float o = 0.0f;
            if (c > 1) {
                const double rank = (double)(lo - start[g]) + 0.5 * (double)(hi - lo - 1);
                o = (float)(rank / (double)(c - 1) - 0.5);
            }
            a.out[(int)(key & kIdxMask)] = o;
        }
    }
    if (a.status && threadIdx.x == 0) *a.status = 0;
}

// -------------------------------------------------------------- partition --
// Keyed Feistel permutation of [0, 2^(2h)), eight rounds, round function =
// word 0 of Philox block (counter (R, r, 3, 0), key seed); cycle-walked into
// [0, d).  h <= 28 (d < 2^55), so each half fits one 32-bit word.
constexpr int kFeistelRounds = 8;
constexpr int kMaxWalk = 1 << 16;
constexpr int kMaxTablePasses = 1 << 20;

// X: uint32_t where 2h <= 32 (d <= 2^32), uint64_t otherwise.
template <typename X>
__device__ __forceinline__ X feistel(uint32_t k0, uint32_t k1, int h, X x)
{
    const uint32_t mask = (1u << h) - 1u;
    uint32_t L = (uint32_t)(x >> h), R = (uint32_t)x & mask;
#pragma unroll
    for (int r = 0; r < kFeistelRounds; ++r) {
        const Words4 y = philox4x32_10(R, (uint32_t)r, 3u, 0u, k0, k1);
        const uint32_t nr = __builtin_amdgcn_bitop3_b32(L, y.x, mask, 0x78);   // L ^ (y & mask)
        L = R;
        R = nr;
    }
    return ((X)L << h) | (X)R;
}

__device__ __forceinline__ uint64_t prp(uint32_t k0, uint32_t k1, int h, uint64_t d, uint64_t x, bool& overflow)
{
    uint64_t y = feistel<uint64_t>(k0, k1, h, x);
    int walk = 0;
    while (y >= d) {
        y = feistel<uint64_t>(k0, k1, h, y);
        if (++walk >= kMaxWalk) {
            overflow = true;
            y = 0;
            break;
        }
    }
    return y;
}

// floor(y K / d) for y < d.  For d <= 2^32 (X = uint32_t) in fp64: y (K / d)
// is within 2^-43 of the quotient, whose fractional part is 0 or lies in
// [2^-32, 1 - 2^-32], so 2^-36 above it truncates to the quotient exactly; a
// 64-bit integer division by a run-time d costs about a hundred instructions
// instead of three.
template <typename X>
__device__ __forceinline__ uint32_t bucket_of(X y, const PartitionArgs& a)
{
    if (sizeof(X) == 4) return (uint32_t)__builtin_fma((double)y, a.k_over_d, 0x1p-36);
    return (uint32_t)(((uint64_t)y * (uint64_t)a.K) / (uint64_t)a.d);
}

__global__ void k_status_zero(int32_t* status)
{
    *status = 0;
}

// A workgroup of these passes is four waves.  A large partition gives each
// wave a tile of kTile elements of its own (WPT = 1 wave per tile).  Below
// kPartTableMin elements a workgroup shares one tile (WPT = 4): a partition of
// a chunk list has a few thousand ids, and one wave per tile would leave
// almost every CU idle behind a few waves that take 2,048 elements one after
// the other (2,304 ids: 62 us with one wave per tile, 27 us with four, 29 us
// with sixteen; 2^22: 71, 66 and 72 us).
constexpr int kPartWaves = 4;
template <int WPT> constexpr int kPartTiles = kPartWaves / WPT;          // tiles per workgroup
template <int WPT> constexpr int kPartSub = (int)kTile / WPT;            // elements per wave

// Partitions of at least this many elements take the table path below: 2^22
// elements take 47 us there and 66 us in k_part_bucket, but 2^22 + 5 (three
// of four walks leave the range) 296 and 223 us; 2^23: 166 and 214 us,
// 2^26: 341 and 720 us, 2^26 + 1: 1,790 and 2,590 us, measured when the line
// was drawn (the table path now takes 160, 285 and 1,330 us at the last three).
constexpr int64_t kPartTableMin = 1ll << 23;

// Pass 1: bucket of every element, and per-tile bucket counts.  Bound by the
// VALU: eight Philox blocks (about 290 instructions) per step of a walk.  The
// number of steps differs from element to element (1 to 4 on average, with a
// geometric tail), so the lanes of a wave don't wait for each other: a lane
// whose element has arrived in [0, d) takes the next one of the wave's range
// at once, ranked among the lanes that finish with it.  Buckets are collected
// in LDS (the elements of a lane are not consecutive) and written as 16-byte
// vectors.  It serves partitions below kPartTableMin (X = uint32_t, WPT = 4)
// and above 2^32 elements (X = uint64_t, WPT = 1), this pass alone: 2^22
// elements 43 us and 2^22 + 5 (three of four walks leave the range) 238 us,
// where lanes walking in step, a wave per tile and a 64-bit division per
// element took 50 and 682 us; 2^32 + 5 elements 167 ms against 556 ms.
template <typename X, int WPT>
__global__ __launch_bounds__(64 * kPartWaves) void k_part_bucket(PartitionArgs a)
{
    constexpr int kWaves = kPartWaves, kTiles = kPartTiles<WPT>, kSub = kPartSub<WPT>;
    __shared__ uint32_t hist[kTiles][256];
    __shared__ __attribute__((aligned(16))) uint8_t stage[kWaves][kSub];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x & 63;
    const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
    for (int k = threadIdx.x; k < kTiles * 256; k += 64 * kWaves) hist[0][k] = 0;
    __syncthreads();
    const int64_t tile = (int64_t)blockIdx.x * kTiles + wave / WPT;
    const int64_t first = tile * kTile + (wave % WPT) * kSub;
    const int n = first >= a.d ? 0 : a.d - first < kSub ? (int)(a.d - first) : kSub;
    uint32_t* counts = hist[wave / WPT];
    bool overflow = false;
    int e = lane, next = 64, walk = 0;
    X y = (X)(first + e);
    while (__builtin_amdgcn_ballot_w64(e < n) != 0) {
        y = feistel<X>(k0, k1, a.half_bits, y);
        bool done = (uint64_t)y < (uint64_t)a.d;
        if (!done && ++walk >= kMaxWalk) {
            overflow |= e < n;
            y = 0;
            done = true;
        }
        if (done && e < n) {
            const uint32_t b = bucket_of<X>(y, a);
            stage[wave][e] = (uint8_t)b;
            atomicAdd(&counts[b], 1u);
        }
        const uint64_t m = __builtin_amdgcn_ballot_w64(done);
        if (done) {
            e = next + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
            y = (X)(first + e);
            walk = 0;
        }
        next += __popcll(m);
    }
    if (overflow && a.status) atomicOr(a.status, 1);
    __syncthreads();
    for (int v = lane; v < n / 16; v += 64)
        reinterpret_cast<V4u*>(a.bucket + first)[v] = reinterpret_cast<const V4u*>(stage[wave])[v];
    for (int v = (n & ~15) + lane; v < n; v += 64) a.bucket[first + v] = stage[wave][v];
    if (tile < a.n_tiles)
        for (int k = lane + 64 * (wave % WPT); k < a.K; k += 64 * WPT)
            a.counts[(int64_t)k * a.n_tiles + tile] = counts[k];
}

// Pass 1 of a large partition, by table.  The round function has only 2^h
// arguments (h <= 16 for d <= 2^32) and 8 rounds: k_part_tables evaluates all
// of them once, 8 * 2^h uint16 values (at most 1 MiB), and a step of a walk
// becomes eight LDS look-ups instead of eight Philox blocks.  The tables lie
// in the map that the scatter writes afterwards.  Below h = 16 the values are
// kept doubled: a half of a walk is then the byte offset of its look-up.
__global__ __launch_bounds__(kBlock) void k_part_tables(PartitionArgs a)
{
    const uint32_t t = blockIdx.x * kBlock + threadIdx.x;
    if (t >= (uint32_t)kFeistelRounds << a.half_bits) return;
    const uint32_t mask = (1u << a.half_bits) - 1u;
    const Words4 y = philox4x32_10(t & mask, t >> a.half_bits, 3u, 0u, (uint32_t)a.seed, (uint32_t)(a.seed >> 32));
    a.tables[t] = (uint16_t)((y.x & mask) << (a.half_bits < 16 ? 1 : 0));
}

// One workgroup of 16 waves per CU, 128 KiB of its LDS filled with tables,
// each wave walking a contiguous range of elements in kPartSlots slots per
// lane.  Every pass takes each slot one step further, G rounds per stage; slots
// that have arrived in [0, d) give their bucket and take the next element of
// the range.  h <= 13: all 8 rounds fit (G = 8).  h = 14, 15: a stage's tables
// take half of the space (G = 2, 1), and the next stage's are loaded straight
// into the other half during the look-ups, with one barrier a stage.  h = 16:
// one round fills it (G = 1), and the waves wait for each refill.  Bound by the
// LDS (random 2-byte reads); the more slots a pass moves, the less the refills
// from L2 count.  1,009,308,160 elements (h = 15): 8.8 ms with Philox evaluated
// in each step, 3.2 ms with two rounds per refill and the waves waiting for it,
// 2.52 ms so (without the refills it is no faster: they are hidden).
template <int H> constexpr int kPartRounds = H == 13 ? 8 : H == 14 ? 2 : 1;
template <int H> constexpr int kPartSlots = H == 13 ? 16 : H == 14 ? 24 : 32;
constexpr int kTableWaves = 16;
constexpr int kTableGroups = 256;         // workgroups: one per CU
constexpr int kTableElems = 1 << 16;      // uint16 entries in LDS

// Half of the LDS (64 KiB) from `src`, 64 bytes per thread, without a register
// in between: a wave's 64 lanes write 1 KiB at m0 and the offset.  The caller
// waits with lds_half_wait before the data is read, the buffer reused, or the
// kernel ends.  Written out because the compiler would wait for the transfer
// before any other LDS read.
__device__ __forceinline__ void lds_half_load(const uint16_t* src, uint16_t* half)
{
    static_assert(kTableElems / 2 * 2 == 64 * kTableWaves * 64, "64 bytes per thread");
    typedef __attribute__((address_space(3))) uint16_t Lds;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x & 63;
    const uint32_t to = (uint32_t)(uintptr_t)(Lds*)(half + wave * 2048);
    const uint16_t* from = src + wave * 2048 + lane * 8;
    asm volatile("s_mov_b32 m0, %0\n\t"
                 "s_nop 0\n\t"
                 "global_load_lds_dwordx4 %1, off\n\t"
                 "global_load_lds_dwordx4 %1, off offset:1024\n\t"
                 "global_load_lds_dwordx4 %1, off offset:2048\n\t"
                 "global_load_lds_dwordx4 %1, off offset:3072"
                 :: "s"(to), "v"(from) : "memory", "m0");
}
__device__ __forceinline__ void lds_half_wait()
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// H: the tables' 2^h arguments, 13 for all h <= 13.
template <int H>
__global__ __launch_bounds__(64 * kTableWaves) void k_part_bucket_table(PartitionArgs a)
{
    __shared__ __attribute__((aligned(16))) uint16_t tab[kTableElems];
    constexpr int kSlots = kPartSlots<H>, G = kPartRounds<H>, kStages = kFeistelRounds / G;
    constexpr bool kHalves = H == 14 || H == 15;
    static_assert(!kHalves || (G << H == kTableElems / 2 && kStages % 2 == 0), "a stage fills half of the LDS");
    const int lane = threadIdx.x & 63;
    const int64_t wave = (int64_t)blockIdx.x * kTableWaves + __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    constexpr int64_t kWaves = (int64_t)kTableGroups * kTableWaves;
    const int64_t range = (a.d + kWaves - 1) / kWaves;             // at most 2^20 elements
    const int64_t first = wave * range;
    const int n = first >= a.d ? 0 : a.d - first < range ? (int)(a.d - first) : (int)range;
    constexpr int kDouble = H < 16 ? 1 : 0;
    const int h = H == 13 ? a.half_bits : H;
    const uint32_t mask = (1u << h) - 1u;
    uint8_t* bucket = a.bucket + first;
    // A slot holds the halves (L, R) of its walk, doubled like the tables, as
    // L << 16 | R: a round is then a rotation by 16 and an xor with the
    // looked-up value, and R the offset to look up.
    // (Elements behind the range, which a slot without work holds, are masked into the tables too.)
    auto split = [&](uint32_t i) -> uint32_t {
        return (((i >> h) & mask) << (16 + kDouble)) | ((i & mask) << kDouble);
    };
    auto halves = [&](int v) -> uint32_t { return split((uint32_t)first + (uint32_t)v); };
    const uint32_t x_last = split((uint32_t)(a.d - 1));
    auto look_up = [&](const uint16_t* t, uint32_t x) -> uint32_t {
        return *reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(t) + ((x & 0xFFFFu) << (1 - kDouble)));
    };
    uint32_t x[kSlots];
    int e[kSlots];
    int next = 64 * kSlots, missing = n;                           // buckets not written yet
#pragma unroll
    for (int i = 0; i < kSlots; ++i) {
        e[i] = 64 * i + lane;
        x[i] = halves(e[i]);
    }
    if (kHalves) lds_half_load(a.tables, tab);
    for (int pass = 0;; ++pass) {
#pragma unroll 1
        for (int g = 0; g < kStages; ++g) {
            const uint16_t* stage = tab;
            if (kHalves) {
                lds_half_wait();                                   // this stage's tables, as far as this wave loads them
                __syncthreads();                                   // all of them, and no wave reads the other half any more
                stage = tab + (g & 1) * (kTableElems / 2);
                lds_half_load(a.tables + ((size_t)((g + 1) % kStages * G) << h), tab + (~g & 1) * (kTableElems / 2));
            } else if (G < kFeistelRounds || pass == 0) {
                if (G < kFeistelRounds) __syncthreads();           // every wave is done with the last tables
                const V4u* src = reinterpret_cast<const V4u*>(a.tables + ((size_t)(g * G) << h));
                for (uint32_t v = threadIdx.x; v < (uint32_t)(G << h) / 8u; v += 64 * kTableWaves)
                    reinterpret_cast<V4u*>(tab)[v] = src[v];
                __syncthreads();
            }
#pragma unroll
            for (int r = 0; r < G; ++r) {
                const uint16_t* t = stage + ((uint32_t)r << h);
#pragma unroll
                for (int i0 = 0; i0 < kSlots; i0 += 8) {
                    uint32_t f[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) f[i] = look_up(t, x[i0 + i]);
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        x[i0 + i] = __builtin_amdgcn_alignbit(x[i0 + i], x[i0 + i], 16) ^ f[i];
                    __builtin_amdgcn_sched_barrier(0);             // eight look-ups in flight: enough, and no spills
                }
            }
        }
        const bool stuck = pass >= kMaxTablePasses;                // cannot happen for a bijection
        if (stuck) {
            for (int v = lane; v < n; v += 64) bucket[v] = 0;
            if (a.status && lane == 0) atomicOr(a.status, 1);
        }
#pragma unroll
        for (int i = 0; i < kSlots; ++i) {
            const bool done = x[i] <= x_last;                      // slots compare like the elements they hold
            const uint64_t m = __builtin_amdgcn_ballot_w64(done);
            const bool mine = e[i] < n;
            missing -= __popcll(m & __builtin_amdgcn_ballot_w64(mine));
            if (done && mine && !stuck) {
                const uint32_t y = ((x[i] >> (16 + kDouble)) << h) | ((x[i] & 0xFFFFu) >> kDouble);
                bucket[(uint32_t)e[i]] = (uint8_t)bucket_of<uint32_t>(y, a);
            }
            if (done) {
                e[i] = next + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
                x[i] = halves(e[i]);
            }
            next += __popcll(m);
            __builtin_amdgcn_sched_barrier(0);
        }
        const bool left = missing > 0 && !stuck;
        if (G < kFeistelRounds ? !__syncthreads_or(left) : __builtin_amdgcn_ballot_w64(left) == 0) break;
    }
    if (kHalves) lds_half_wait();                                  // for the load that no stage reads
}

// Bucket counts of every tile for the table path, one wave per tile.  Up to 8
// buckets (NB = 3) are counted in registers, one byte of a 64-bit word each (a
// lane sees 32 elements); more of them in LDS, in four copies by lane so that
// the lanes of an atomic seldom meet in one.
template <int NB>
__global__ __launch_bounds__(kBlock) void k_part_count(PartitionArgs a)
{
    constexpr int kCopies = NB > 3 ? 4 : 1, kBuckets = 1 << NB;
    __shared__ uint32_t hist[kBlock / 64][kCopies * kBuckets];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x & 63;
    const int64_t tile = (int64_t)blockIdx.x * (kBlock / 64) + wave;
    if (tile >= a.n_tiles) return;
    const int64_t first = tile * kTile;
    const int n = a.d - first < kTile ? (int)(a.d - first) : (int)kTile;
    uint32_t* h = hist[wave];
    for (int k = lane; k < kCopies * kBuckets; k += 64) h[k] = 0;
    wave_lds_sync();
    uint32_t* mine = h + (lane % kCopies) * kBuckets;
    uint64_t packed = 0;
    auto count = [&](uint32_t b) {
        if (NB <= 3) packed += 1ull << (8u * b);
        else atomicAdd(&mine[b], 1u);
    };
    for (int v = lane; v < n / 16; v += 64) {
        const V4u x = reinterpret_cast<const V4u*>(a.bucket + first)[v];
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
            for (int b = 0; b < 4; ++b) count((x[w] >> (8 * b)) & 255u);
    }
    for (int v = (n & ~15) + lane; v < n; v += 64) count(a.bucket[first + v]);
    if (NB <= 3) {
        // 16-bit fields of two words hold the wave's sums (at most 2,048)
        uint64_t even = packed & 0x00FF00FF00FF00FFull, odd = (packed >> 8) & 0x00FF00FF00FF00FFull;
#pragma unroll
        for (int m = 32; m > 0; m >>= 1) {
            even += __shfl_xor(even, m, 64);
            odd += __shfl_xor(odd, m, 64);
        }
        if (lane < a.K)
            a.counts[(int64_t)lane * a.n_tiles + tile] = (uint32_t)(((lane & 1) ? odd : even) >> (16 * (lane >> 1))) & 0xFFFFu;
        return;
    }
    wave_lds_sync();
    for (int k = lane; k < a.K; k += 64) {
        uint32_t c = 0;
#pragma unroll
        for (int q = 0; q < kCopies; ++q) c += h[q * kBuckets + k];
        a.counts[(int64_t)k * a.n_tiles + tile] = c;
    }
}

// Scan pass A: sum of each chunk of kScanChunk counts.
__global__ __launch_bounds__(kBlock) void k_scan_reduce(const uint32_t* counts, int64_t n, int64_t* block_sums)
{
    __shared__ int64_t part[kBlock];
    const int64_t base = (int64_t)blockIdx.x * kScanChunk;
    int64_t s = 0;
    for (int k = threadIdx.x; k < kScanChunk; k += kBlock)
        if (base + k < n) s += counts[base + k];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int off = kBlock / 2; off > 0; off >>= 1) {
        if (threadIdx.x < off) part[threadIdx.x] += part[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) block_sums[blockIdx.x] = part[0];
}

// Block-wide exclusive scan of kBlock values held one per thread.
__device__ __forceinline__ int64_t block_exclusive_scan(int64_t v, int64_t* tmp, int64_t& total)
{
    tmp[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < kBlock; off <<= 1) {
        const int64_t add = threadIdx.x >= (unsigned)off ? tmp[threadIdx.x - off] : 0;
        __syncthreads();
        tmp[threadIdx.x] += add;
        __syncthreads();
    }
    total = tmp[kBlock - 1];
    const int64_t incl = tmp[threadIdx.x];
    __syncthreads();
    return incl - v;
}

// Scan pass B: exclusive scan of the chunk sums, in place (one workgroup).
__global__ __launch_bounds__(kBlock) void k_scan_blocks(int64_t* block_sums, int64_t nb)
{
    __shared__ int64_t tmp[kBlock];
    int64_t carry = 0;
    for (int64_t base = 0; base < nb; base += kBlock) {
        const int64_t i = base + threadIdx.x;
        const int64_t v = i < nb ? block_sums[i] : 0;
        int64_t total;
        const int64_t ex = block_exclusive_scan(v, tmp, total);
        if (i < nb) block_sums[i] = carry + ex;
        carry += total;
    }
}

// Scan pass C: exclusive positions of every count (block_sums: null when one
// workgroup covers them all).
__global__ __launch_bounds__(kBlock) void k_scan_down(const uint32_t* counts, int64_t n, const int64_t* block_sums,
                                                      int64_t* pos)
{
    __shared__ int64_t tmp[kBlock];
    constexpr int per = kScanChunk / kBlock;   // consecutive entries per thread
    const int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * per;
    int64_t v[per];
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < per; ++k) {
        v[k] = base + k < n ? counts[base + k] : 0;
        s += v[k];
    }
    int64_t total;
    int64_t run = (block_sums ? block_sums[blockIdx.x] : 0) + block_exclusive_scan(s, tmp, total);
#pragma unroll
    for (int k = 0; k < per; ++k) {
        if (base + k < n) pos[base + k] = run;
        run += v[k];
    }
}

// Pass 3: stable scatter.  A tile's entries are ordered by bucket in LDS
// first: each wave walks its part of the tile in element order, ranks the 64
// elements of a step among equal buckets with ballots and appends them to
// each bucket's run.  The runs are then written from consecutive lanes to
// consecutive map entries, as whole lines but for a run's two ends, where a
// store per step would write 64 / K entries to each of K places.  16-bit
// entries (K <= 32) leave room for six workgroups per CU.  1,009,308,160
// elements, K = 8, int64 map: 1.82 ms (5 TB/s), against 3.0 ms with stores per
// step.
// NB: bits of a bucket number (K <= 2^NB).
template <int NB, int WPT>
__global__ __launch_bounds__(64 * kPartWaves) void k_part_scatter(PartitionArgs a)
{
    constexpr int kWaves = kPartWaves, kTiles = kPartTiles<WPT>, kSub = kPartSub<WPT>;
    constexpr int kThreads = 64 * WPT;                       // threads of one tile
    typedef typename std::conditional<NB <= 5, uint16_t, uint32_t>::type Entry;
    constexpr int kElemBits = 11, kBuckets = 1 << NB;
    static_assert(kTile == 1 << kElemBits, "an entry holds an element of the tile and its bucket");
    __shared__ Entry order[kTiles][kTile];                   // element | bucket << kElemBits, by bucket
    __shared__ int64_t delta[kTiles][kBuckets];              // map position - place in the tile, of each bucket
    __shared__ uint32_t cur[kWaves][kBuckets];               // next place of each bucket, by wave
    __shared__ __attribute__((aligned(16))) uint8_t stage[kWaves][kSub];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x & 63;
    const int slot = wave / WPT, sub = wave % WPT;
    const int64_t tile = (int64_t)blockIdx.x * kTiles + slot;
    const int64_t first = tile * kTile + sub * kSub;
    const int n = first >= a.d ? 0 : a.d - first < kSub ? (int)(a.d - first) : kSub;
    for (int v = lane; v < n / 16; v += 64)
        reinterpret_cast<V4u*>(stage[wave])[v] = reinterpret_cast<const V4u*>(a.bucket + first)[v];
    for (int v = (n & ~15) + lane; v < n; v += 64) stage[wave][v] = a.bucket[first + v];
    // places of the tile's runs: an exclusive scan of its bucket counts
    if (sub == 0 && tile < a.n_tiles) {
        uint32_t before = 0;
        for (int k = lane; k < ((a.K + 63) & ~63); k += 64) {
            const uint32_t c = k < a.K ? a.counts[(int64_t)k * a.n_tiles + tile] : 0u;
            uint32_t incl = c;
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) {
                const uint32_t up = __shfl_up(incl, m, 64);
                if (lane >= m) incl += up;
            }
            const uint32_t place = before + incl - c;
            if (k < a.K) {
                cur[wave][k] = place;
                delta[slot][k] = a.pos[(int64_t)k * a.n_tiles + tile] - (int64_t)place;
            }
            before += __shfl(incl, 63, 64);
        }
    }
    if (WPT > 1) {
        // several waves per tile: each starts behind the waves before it
        for (int k = lane; k < a.K && sub > 0; k += 64) cur[wave][k] = 0;
        __syncthreads();
        for (int v = lane; v < n && sub + 1 < WPT; v += 64) atomicAdd(&cur[wave + 1][stage[wave][v]], 1u);
    }
    __syncthreads();
    if (WPT > 1) {
        for (int k = threadIdx.x % kThreads; k < a.K; k += kThreads) {
            uint32_t run = cur[slot * WPT][k];
            for (int s = 1; s < WPT; ++s) cur[slot * WPT + s][k] = run += cur[slot * WPT + s][k];
        }
        __syncthreads();
    }
    for (int v0 = 0; v0 < n; v0 += 64) {
        const int v = v0 + lane;
        const bool valid = v < n;
        const uint32_t b = valid ? stage[wave][v] : 0u;
        const uint64_t any = __builtin_amdgcn_ballot_w64(valid);
        uint32_t lo = (uint32_t)any, hi = (uint32_t)(any >> 32);
#pragma unroll
        for (int bit = 0; bit < NB; ++bit) {
            const uint32_t set = (uint32_t)((int32_t)(b << (31 - bit)) >> 31);       // all ones if the bit is set
            const uint64_t m = __builtin_amdgcn_ballot_w64(set != 0);
            lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)m, set, 0x90);            // lo & ~(m ^ set)
            hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(m >> 32), set, 0x90);
        }
        const int rank = (int)__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
        if (valid) {
            const uint32_t place = cur[wave][b];
            order[slot][place + rank] = (Entry)((uint32_t)(sub * kSub + v) | (b << kElemBits));
            wave_lds_sync();
            if (rank == 0) cur[wave][b] = place + (uint32_t)(__builtin_popcount(lo) + __builtin_popcount(hi));
        }
        wave_lds_sync();
    }
    __syncthreads();
    const int64_t t0 = tile * kTile;
    const int total = t0 >= a.d ? 0 : a.d - t0 < kTile ? (int)(a.d - t0) : (int)kTile;
    for (int p = threadIdx.x % kThreads; p < total; p += kThreads) {
        const uint32_t v = order[slot][p];
        const int64_t at = delta[slot][v >> kElemBits] + p;
        const int64_t e = t0 + (v & (uint32_t)(kTile - 1));
        if (a.index32)
            a.index32[at] = (uint32_t)e;
        else
            a.index[at] = e;
    }
}

// ------------------------------------------------------------------ debug --
__global__ __launch_bounds__(kBlock) void k_debug_philox(uint64_t seed, uint32_t domain, uint64_t q0, int64_t nblocks,
                                                         uint32_t* out)
{
    for (int64_t b = global_tid(); b < nblocks; b += grid_stride()) {
        const Words4 x = stream_block((uint32_t)seed, (uint32_t)(seed >> 32), domain, q0 + (uint64_t)b);
        reinterpret_cast<uint4*>(out)[b] = make_uint4(x.x, x.y, x.z, x.w);
    }
}

__global__ __launch_bounds__(kBlock) void k_debug_normals(uint64_t seed, int64_t j0, int64_t n, float* out)
{
    const Bm tb = stage_bm_tables<kBlock>();
    const int64_t qa = j0 >> 2;                      // first block touched
    const int64_t qb = (j0 + n + 3) >> 2;            // one past the last
    for (int64_t q = qa + global_tid(); q < qb; q += grid_stride()) {
        float z[4];
        normals4((uint32_t)seed, (uint32_t)(seed >> 32), (uint64_t)q, tb, z);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int64_t j = 4 * q + t;
            if (j >= j0 && j < j0 + n) out[j - j0] = z[t];
        }
    }
}

// Seeded normal fill: w[j] = cast(stddev * z_j), z_j the normal of position
// j in stream (seed, domain).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_fill_normal(T* w, int64_t n, uint64_t seed, uint32_t domain, float stddev)
{
    constexpr int N = UnitOf<T>::n;
    const Bm tb = stage_bm_tables<kBlock>();
    const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    auto body = [&](int64_t u, bool vec) {
        const int64_t j0 = u * N;
        float z[N];
        if (N == 8)
            normals8(k0, k1, (uint64_t)j0 >> 2, tb, z, domain);
        else
            normals4(k0, k1, (uint64_t)j0 >> 2, tb, z, domain);
        T v[N];
#pragma unroll
        for (int e = 0; e < N; ++e) v[e] = from_f32<T>(stddev * z[e]);
        if (vec) {
            store_vec<T>(w + j0, v);
        } else {
#pragma unroll
            for (int e = 0; e < N; ++e)
                if (j0 + e < n) w[j0 + e] = v[e];
        }
    };
    const int64_t full = n / N;
    for (int64_t u = global_tid(); u < full; u += grid_stride()) body(u, true);
    if (full * N < n && global_tid() == 0) body(full, false);
}

__global__ __launch_bounds__(kBlock) void k_debug_bm_grid(uint32_t m0, int64_t n, double* rho, double* c, double* s)
{
    const Bm tb = stage_bm_tables<kBlock>();
    for (int64_t k = global_tid(); k < n; k += grid_stride()) {
        const uint32_t word = (m0 + (uint32_t)k - 1u) << 8;
        if (rho) rho[k] = 0.5 * bm_radius2(word, tb);
        double cc, ss;
        bm_half_angle(word, tb, cc, ss);
        if (c) c[k] = 2.0 * cc;
        if (s) s[k] = 2.0 * ss;
    }
}

__global__ __launch_bounds__(kBlock) void k_debug_prp(uint64_t seed, int64_t d, int32_t K, int32_t h, int64_t i0,
                                                      int64_t n, int64_t* perm, int32_t* bucket)
{
    for (int64_t k = global_tid(); k < n; k += grid_stride()) {
        bool overflow = false;
        const uint64_t y = prp((uint32_t)seed, (uint32_t)(seed >> 32), h, (uint64_t)d, (uint64_t)(i0 + k), overflow);
        if (perm) perm[k] = (int64_t)y;
        if (bucket) bucket[k] = (int32_t)((y * (uint64_t)K) / (uint64_t)d);
    }
}

__global__ void k_zero_u32(uint32_t* p)
{
    *p = 0u;
}

// RNG-only probe: each thread takes units of 8 positions and, like the update,
// adds the scaled noise of kRngProbeStreams consecutive seeds for each unit to
// 8 independent fp64 sums (a perturbation rounds each normal to fp32 first, a
// few instructions more); the sums' bits are folded into one word at the end.
// No memory traffic but one atomic per wave.
constexpr int kRngProbeStreams = 16;

template <typename Q>
__global__ __launch_bounds__(kBlock) void k_rng_probe(uint64_t seed, int64_t units, uint32_t* sink)
{
    const Bm tb = stage_bm_tables<kBlock>();
    double acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.0;
    for (int64_t u = global_tid(); u < units; u += grid_stride()) {
        for (int st = 0; st < kRngProbeStreams; ++st) {
            const uint64_t key = seed + (uint64_t)st;
            add_normals<8, Q>((uint32_t)key, (uint32_t)(key >> 32), (Q)(u * 2), tb, 0.5, acc);
        }
    }
    uint32_t x = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) x ^= (uint32_t)__double2loint(acc[e]) ^ (uint32_t)__double2hiint(acc[e]);
    for (int off = 32; off > 0; off >>= 1) x ^= __shfl_xor(x, off);
    if ((threadIdx.x & 63) == 0) atomicXor(sink, x);
}

// Measurement references with nothing but the memory traffic.  The plainest
// gather (DIR 0: buf[j] = w[p(j)]) or scatter (DIR 1: w[p(j)] = buf[j])
// through an element map, one position per thread.
template <typename T, int DIR, int ADDR>
__global__ __launch_bounds__(kBlock) void k_probe_map_copy(StreamArgs a)
{
    T* w = static_cast<T*>(a.w);
    T* buf = static_cast<T*>(a.aux);
    for (int64_t j = global_tid(); j < a.length; j += grid_stride()) {
        const int64_t i = map_entry<ADDR>(a.index, a.offset + j);
        if ((uint64_t)i >= (uint64_t)a.numel) continue;
        if (DIR == 0)
            buf[j] = w[i];
        else
            w[i] = buf[j];
    }
}

// A plain copy of n16 16-byte vectors, one per thread per iteration; NT
// takes non-temporal loads and stores.
template <bool NT>
__global__ __launch_bounds__(kBlock) void k_probe_copy(const V4u* src, V4u* dst, int64_t n16)
{
    for (int64_t i = global_tid(); i < n16; i += grid_stride()) {
        if (NT)
            __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
        else
            dst[i] = src[i];
    }
}

int64_t grid_for(int64_t work_items, int64_t cap = kMaxGrid)
{
    int64_t blocks = (work_items + kBlock - 1) / kBlock;
    if (blocks < 1) blocks = 1;
    return blocks < cap ? blocks : cap;
}

// Workgroups of a noise kernel on `items` units of a contiguous or chunked
// subspace (threads of kBlock).  Up to 8,192 of them take one unit per thread.
// Larger launches loop: the tables are staged once per workgroup, so a
// workgroup wants several units, but with few, long workgroups the launch ends
// on the slowest CU (504,654,080 positions, 16 streams: 8,192 workgroups 6.64
// ms, one workgroup per four units of a thread 6.50 ms, per three 6.46 ms, per
// two 6.51 ms; one perturbation 566, 558, 548 and 553 us).  Between 8,193 and
// 24,576 workgroups' worth of units the grid stays at 8,192 and some threads
// take a unit more than others; the same number of units for each is at most
// 3 % faster and often slower (one bf16 perturbation in place, this rule, and
// one, two, three units a thread: 9.4 M positions 13.0, 12.9, 12.8, 12.8 us;
// 17 M 20.5, 20.6, 20.3, 19.8; 33.3 M 35.2, 36.1, 35.5, 36.6; 37.7 M 39.8,
// 40.8, 40.0, 40.5; 50.4 M 52.1, 52.6, 53.5, 54.1; an update with 10 streams on
// 17 M 143, 143, 148, 146, on 37.7 M 305, 302, 304, 304).  The same rule serves
// perturbations through ascending maps, in workgroups of two (126,163,520
// positions, int64 map, from the backup, with its restore: 1,811 us with 4,096
// workgroups of 512 threads, 1,755 us with one per three tiles of a wave, 1,774
// us per eight).
int64_t noise_grid_cap(int64_t items)
{
    const int64_t blocks = (items + kBlock - 1) / kBlock;
    return std::max(kRngMaxGrid, std::min((blocks + 2) / 3, kMaxGrid));
}

template <typename K, typename A>
hipError_t launch1d(K kernel, int64_t items, const A& args, hipStream_t s, int64_t cap)
{
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid_for(items, cap)), dim3(kBlock), 0, s, args);
    return hipGetLastError();
}

template <typename T>
int64_t units_of(int64_t length)
{
    return (length + UnitOf<T>::n - 1) / UnitOf<T>::n;
}

// Map kernels: one wave per tile of 64 N positions, up to the grid cap; the
// waves of a launch then start in position order, which keeps the scattered
// accesses in flight within a narrow window of the weights.
template <typename T>
int64_t map_threads(int64_t length)
{
    const int64_t tile = 64 * UnitOf<T>::n;
    return (length + tile - 1) / tile * 64;
}

// Instantiate a streaming kernel for the addressing mode; element maps go to
// the map kernel MAPK instantiated with MARGS.
#define CPES_DISPATCH(KERNEL, KARGS, MAPK, MARGS)                                                     \
    switch (addr) {                                                                                  \
    case kGather: return launch1d(MAPK<MARGS, kGather>, map_threads<T>(a.length), a, s, kMaxGrid); \
    case kGather32: return launch1d(MAPK<MARGS, kGather32>, map_threads<T>(a.length), a, s, kMaxGrid); \
    case kChunk: return launch1d(KERNEL<KARGS, kChunk>, u, a, s, cap);                               \
    default: return launch1d(KERNEL<KARGS, kContig>, u, a, s, cap);                                  \
    }
#define CPES_COMMA ,

// Every noise block of positions [0, length) is below 2^32.
inline bool short_blocks(int64_t noise0, int64_t length)
{
    return noise0 + length <= (1ll << 34);
}

// Dense-window kernels (ascending maps, bf16): one wave per tile of kDenseTile entries.
int64_t dense_threads(int64_t length)
{
    return (length + kDenseTile - 1) / kDenseTile * 64;
}

template <typename T, int AUX, typename Q>
hipError_t perturb_t(int addr, const StreamArgs& a, hipStream_t s)
{
    if (std::is_same<T, uint16_t>::value && a.dense) {
        const int64_t threads = dense_threads(a.length);
        const dim3 grid((unsigned)std::min((threads + kDenseBlock - 1) / kDenseBlock, noise_grid_cap(threads) / (kDenseBlock / kBlock)));
        if (addr == kGather) hipLaunchKernelGGL((k_perturb_dense<AUX, Q, kGather>), grid, dim3(kDenseBlock), 0, s, a);
        else if (addr == kGather32) hipLaunchKernelGGL((k_perturb_dense<AUX, Q, kGather32>), grid, dim3(kDenseBlock), 0, s, a);
        if (addr == kGather || addr == kGather32) return hipGetLastError();
    }
    const int64_t u = units_of<T>(a.length), cap = noise_grid_cap(u);
    CPES_DISPATCH(k_perturb, T CPES_COMMA AUX CPES_COMMA Q, k_perturb_map, T CPES_COMMA AUX CPES_COMMA Q)
}

template <typename T, bool MASTER, typename Q>
hipError_t update_t(int addr, const UpdateArgs& a, hipStream_t s)
{
    constexpr int N = MASTER ? 8 : UnitOf<T>::n;
    const int64_t u = (a.length + N - 1) / N, cap = noise_grid_cap(u);
    CPES_DISPATCH(k_update, T CPES_COMMA MASTER CPES_COMMA Q, k_update_map, T CPES_COMMA MASTER CPES_COMMA Q)
}

// Copies whose source and destination together exceed the 256 MB last-level
// cache take the non-temporal loads and stores.
constexpr int64_t kStreamingBytes = 256ll << 20;

inline bool streaming(int64_t length, int bytes_per_position)
{
    return length * bytes_per_position > kStreamingBytes;
}

template <typename T>
hipError_t restore_copy_t(int addr, const StreamArgs& a, hipStream_t s)
{
    if (std::is_same<T, uint16_t>::value && a.dense) {
        if (addr == kGather) return launch1d(k_restore_dense<kCopyRestore, kGather>, dense_threads(a.length), a, s, kMaxGrid);
        if (addr == kGather32) return launch1d(k_restore_dense<kCopyRestore, kGather32>, dense_threads(a.length), a, s, kMaxGrid);
    }
    const int64_t u = units_of<T>(a.length), cap = kMaxGrid;
    if (streaming(a.length, 2 * sizeof(T))) {
        CPES_DISPATCH(k_restore_copy, T CPES_COMMA true, k_copy_map, T CPES_COMMA kCopyRestore CPES_COMMA true)
    }
    CPES_DISPATCH(k_restore_copy, T CPES_COMMA false, k_copy_map, T CPES_COMMA kCopyRestore CPES_COMMA false)
}

template <typename T>
hipError_t backup_copy_t(int addr, const StreamArgs& a, hipStream_t s)
{
    const int64_t u = units_of<T>(a.length), cap = kMaxGrid;
    if (streaming(a.length, 2 * sizeof(T))) {
        CPES_DISPATCH(k_backup_copy, T CPES_COMMA true, k_copy_map, T CPES_COMMA kCopyBackup CPES_COMMA true)
    }
    CPES_DISPATCH(k_backup_copy, T CPES_COMMA false, k_copy_map, T CPES_COMMA kCopyBackup CPES_COMMA false)
}

template <typename T>
hipError_t stage_master_t(int addr, const StreamArgs& a, hipStream_t s)
{
    const int64_t u = units_of<T>(a.length), cap = kMaxGrid;
    if (streaming(a.length, sizeof(T) + 4)) {
        CPES_DISPATCH(k_stage_master, T CPES_COMMA true, k_copy_map, T CPES_COMMA kCopyStageMaster CPES_COMMA true)
    }
    CPES_DISPATCH(k_stage_master, T CPES_COMMA false, k_copy_map, T CPES_COMMA kCopyStageMaster CPES_COMMA false)
}

hipError_t restore_master_t(int addr, const StreamArgs& a, hipStream_t s)
{
    using T = uint16_t;
    if (a.dense) {
        if (addr == kGather) return launch1d(k_restore_dense<kCopyRestoreMaster, kGather>, dense_threads(a.length), a, s, kMaxGrid);
        if (addr == kGather32) return launch1d(k_restore_dense<kCopyRestoreMaster, kGather32>, dense_threads(a.length), a, s, kMaxGrid);
    }
    const int64_t u = (a.length + 7) / 8, cap = kMaxGrid;
    if (streaming(a.length, 6)) {
        CPES_DISPATCH(k_restore_master, true, k_copy_map, T CPES_COMMA kCopyRestoreMaster CPES_COMMA true)
    }
    CPES_DISPATCH(k_restore_master, false, k_copy_map, T CPES_COMMA kCopyRestoreMaster CPES_COMMA false)
}

template <typename T, typename Q>
hipError_t update_step_t(int addr, const StepArgs& a, hipStream_t s)
{
    const bool map = addr == kGather || addr == kGather32;
    const int64_t units = a.tile_begin[a.K] * 64;
    const int64_t blocks = grid_for(units, map ? kMaxGrid : noise_grid_cap(units));
    switch (addr) {
    case kGather: hipLaunchKernelGGL((k_update_step<T, Q, kGather>), dim3((unsigned)blocks), dim3(kBlock), 0, s, a); break;
    case kGather32: hipLaunchKernelGGL((k_update_step<T, Q, kGather32>), dim3((unsigned)blocks), dim3(kBlock), 0, s, a); break;
    case kChunk: hipLaunchKernelGGL((k_update_step<T, Q, kChunk>), dim3((unsigned)blocks), dim3(kBlock), 0, s, a); break;
    default: hipLaunchKernelGGL((k_update_step<T, Q, kContig>), dim3((unsigned)blocks), dim3(kBlock), 0, s, a); break;
    }
    return hipGetLastError();
}

}  // namespace

namespace {

template <typename T, typename Q>
hipError_t perturb_aux(int aux, int addr, const StreamArgs& a, hipStream_t s)
{
    if (aux == kAuxSnapshot) return perturb_t<T, kAuxSnapshot, Q>(addr, a, s);
    if constexpr (std::is_same<T, uint16_t>::value)
        if (aux == kAuxMaster) return perturb_t<T, kAuxMaster, Q>(addr, a, s);
    if (aux == kAuxBackup) return perturb_t<T, kAuxBackup, Q>(addr, a, s);
    return perturb_t<T, kAuxNone, Q>(addr, a, s);
}

template <typename Q>
hipError_t update_any(int dtype, bool master, int addr, const UpdateArgs& a, hipStream_t s)
{
    if (dtype != 0) return update_t<float, false, Q>(addr, a, s);
    return master ? update_t<uint16_t, true, Q>(addr, a, s) : update_t<uint16_t, false, Q>(addr, a, s);
}

}  // namespace

hipError_t launch_perturb(int dtype, int aux, int addr, const StreamArgs& a, hipStream_t s)
{
    if (short_blocks(a.noise0, a.length))
        return dtype == 0 ? perturb_aux<uint16_t, uint32_t>(aux, addr, a, s) : perturb_aux<float, uint32_t>(aux, addr, a, s);
    return dtype == 0 ? perturb_aux<uint16_t, uint64_t>(aux, addr, a, s) : perturb_aux<float, uint64_t>(aux, addr, a, s);
}

hipError_t launch_restore_copy(int dtype, int addr, const StreamArgs& a, hipStream_t s)
{
    return dtype == 0 ? restore_copy_t<uint16_t>(addr, a, s) : restore_copy_t<float>(addr, a, s);
}

hipError_t launch_backup_copy(int dtype, int addr, const StreamArgs& a, hipStream_t s)
{
    return dtype == 0 ? backup_copy_t<uint16_t>(addr, a, s) : backup_copy_t<float>(addr, a, s);
}

hipError_t launch_restore_master(int addr, const StreamArgs& a, hipStream_t s)
{
    return restore_master_t(addr, a, s);
}

hipError_t launch_stage_master(int dtype, int addr, const StreamArgs& a, hipStream_t s)
{
    return dtype == 0 ? stage_master_t<uint16_t>(addr, a, s) : stage_master_t<float>(addr, a, s);
}

hipError_t launch_update(int dtype, bool master, int addr, const UpdateArgs& a, hipStream_t s)
{
    return short_blocks(a.noise0, a.length) ? update_any<uint32_t>(dtype, master, addr, a, s)
                                            : update_any<uint64_t>(dtype, master, addr, a, s);
}

hipError_t launch_update_step(int dtype, int addr, const StepArgs& a, hipStream_t s)
{
    bool is_short = true;
    for (int k = 0; k < a.K; ++k) is_short = is_short && short_blocks(0, a.length[k]);
    if (is_short) return dtype == 0 ? update_step_t<uint16_t, uint32_t>(addr, a, s) : update_step_t<float, uint32_t>(addr, a, s);
    return dtype == 0 ? update_step_t<uint16_t, uint64_t>(addr, a, s) : update_step_t<float, uint64_t>(addr, a, s);
}

hipError_t launch_fill_normal(int dtype, void* w, int64_t n, uint64_t seed, uint32_t domain, float stddev,
                              hipStream_t s)
{
    const dim3 grid((unsigned)grid_for(n / (dtype == 0 ? 8 : 4) + 1, kRngMaxGrid)), block(kBlock);
    if (dtype == 0)
        hipLaunchKernelGGL(k_fill_normal<uint16_t>, grid, block, 0, s, static_cast<uint16_t*>(w), n, seed, domain, stddev);
    else
        hipLaunchKernelGGL(k_fill_normal<float>, grid, block, 0, s, static_cast<float*>(w), n, seed, domain, stddev);
    return hipGetLastError();
}

namespace {

bool overlap(const void* a, const void* b, int n)      // of n 4-byte entries
{
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b, len = 4 * (uintptr_t)n;
    return a && b && x < y + len && y < x + len;
}

}  // namespace

hipError_t launch_normalize(const NormalizeArgs& a, hipStream_t s)
{
    const dim3 rank_grid((unsigned)((a.n + kRankPer - 1) / kRankPer));
    if (a.mode == 0 && !a.group) {
        if (a.n <= 256) hipLaunchKernelGGL(k_normalize_z<1>, dim3(1), dim3(64), 0, s, a);
        else if (a.n <= 1024) hipLaunchKernelGGL(k_normalize_z<4>, dim3(1), dim3(256), 0, s, a);
        else hipLaunchKernelGGL(k_normalize_z<16>, dim3(1), dim3(1024), 0, s, a);
    } else if (overlap(a.out, a.r, a.n) || overlap(a.out, a.group, a.n)) {
        hipLaunchKernelGGL(k_normalize, dim3(1), dim3(kNormThreads), 0, s, a);
    } else if (a.mode == 0) {
        hipLaunchKernelGGL(k_normalize_z_groups, dim3((unsigned)a.n_groups), dim3(kBlock), 0, s, a);
    } else if (a.group) {
        hipLaunchKernelGGL(k_normalize_rank<true>, rank_grid, dim3(kBlock), 0, s, a);
    } else {
        hipLaunchKernelGGL(k_normalize_rank<false>, rank_grid, dim3(kBlock), 0, s, a);
    }
    return hipGetLastError();
}

namespace {

template <int WPT>
void partition_scatter(const PartitionArgs& a, dim3 grid, dim3 block, hipStream_t s)
{
    if (a.K <= 8) hipLaunchKernelGGL((k_part_scatter<3, WPT>), grid, block, 0, s, a);
    else if (a.K <= 32) hipLaunchKernelGGL((k_part_scatter<5, WPT>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_part_scatter<8, WPT>), grid, block, 0, s, a);
}

void partition_tables(const PartitionArgs& a, hipStream_t s)
{
    const dim3 grid(kTableGroups), block(64 * kTableWaves);
    const unsigned entries = (unsigned)kFeistelRounds << a.half_bits;
    hipLaunchKernelGGL(k_part_tables, dim3((entries + kBlock - 1) / kBlock), dim3(kBlock), 0, s, a);
    if (a.half_bits <= 13) hipLaunchKernelGGL((k_part_bucket_table<13>), grid, block, 0, s, a);
    else if (a.half_bits == 14) hipLaunchKernelGGL((k_part_bucket_table<14>), grid, block, 0, s, a);
    else if (a.half_bits == 15) hipLaunchKernelGGL((k_part_bucket_table<15>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_part_bucket_table<16>), grid, block, 0, s, a);
    const dim3 tiles((unsigned)((a.n_tiles + kBlock / 64 - 1) / (kBlock / 64)));
    if (a.K <= 8) hipLaunchKernelGGL((k_part_count<3>), tiles, dim3(kBlock), 0, s, a);
    else hipLaunchKernelGGL((k_part_count<8>), tiles, dim3(kBlock), 0, s, a);
}

// WPT: kPartTableMin draws the line between shared tiles (4) and large partitions (1).
template <int WPT>
void partition_passes(const PartitionArgs& a, hipStream_t s)
{
    const dim3 grid((unsigned)((a.n_tiles + kPartTiles<WPT> - 1) / kPartTiles<WPT>)), block(64 * kPartWaves);
    const int64_t n_counts = (int64_t)a.K * a.n_tiles;
    const unsigned scan_blocks = (unsigned)((n_counts + kScanChunk - 1) / kScanChunk);
    if constexpr (WPT == 4) hipLaunchKernelGGL((k_part_bucket<uint32_t, WPT>), grid, block, 0, s, a);
    else if (a.tables) partition_tables(a, s);
    else hipLaunchKernelGGL((k_part_bucket<uint64_t, WPT>), grid, block, 0, s, a);
    if (scan_blocks > 1) {
        hipLaunchKernelGGL(k_scan_reduce, dim3(scan_blocks), dim3(kBlock), 0, s, a.counts, n_counts, a.block_sums);
        hipLaunchKernelGGL(k_scan_blocks, dim3(1), dim3(kBlock), 0, s, a.block_sums, (int64_t)scan_blocks);
    }
    hipLaunchKernelGGL(k_scan_down, dim3(scan_blocks), dim3(kBlock), 0, s, a.counts, n_counts,
                       scan_blocks > 1 ? a.block_sums : nullptr, a.pos);
    partition_scatter<WPT>(a, grid, block, s);
}

}  // namespace

hipError_t launch_partition(const PartitionArgs& args, hipStream_t s)
{
    PartitionArgs a = args;
    if (a.status) hipLaunchKernelGGL(k_status_zero, dim3(1), dim3(1), 0, s, a.status);
    a.tables = nullptr;
    if (a.d >= kPartTableMin && a.d <= (1ll << 32)) {
        // the first 16-byte boundary of the output map: 8 * 2^h uint16 entries
        // and 15 bytes fit its d > 2^(2h - 2) entries of at least 4 bytes
        const uintptr_t out = a.index32 ? (uintptr_t)a.index32 : (uintptr_t)a.index;
        a.tables = reinterpret_cast<uint16_t*>((out + 15) & ~(uintptr_t)15);
    }
    if (a.d < kPartTableMin) partition_passes<4>(a, s);
    else partition_passes<1>(a, s);
    return hipGetLastError();
}

hipError_t launch_debug_philox(uint64_t seed, uint32_t domain, uint64_t q0, int64_t nblocks, uint32_t* out, hipStream_t s)
{
    hipLaunchKernelGGL(k_debug_philox, dim3((unsigned)grid_for(nblocks)), dim3(kBlock), 0, s, seed, domain, q0, nblocks, out);
    return hipGetLastError();
}

hipError_t launch_debug_normals(uint64_t seed, int64_t j0, int64_t n, float* out, hipStream_t s)
{
    const int64_t blocks = ((j0 + n + 3) >> 2) - (j0 >> 2);
    hipLaunchKernelGGL(k_debug_normals, dim3((unsigned)grid_for(blocks, kRngMaxGrid)), dim3(kBlock), 0, s, seed, j0, n, out);
    return hipGetLastError();
}

hipError_t launch_debug_bm_grid(uint32_t m0, int64_t n, double* rho, double* c, double* sn, hipStream_t s)
{
    hipLaunchKernelGGL(k_debug_bm_grid, dim3((unsigned)grid_for(n, kRngMaxGrid)), dim3(kBlock), 0, s, m0, n, rho, c, sn);
    return hipGetLastError();
}

hipError_t launch_debug_prp(uint64_t seed, int64_t d, int32_t K, int32_t half_bits, int64_t i0, int64_t n,
                            int64_t* perm, int32_t* bucket, hipStream_t s)
{
    hipLaunchKernelGGL(k_debug_prp, dim3((unsigned)grid_for(n)), dim3(kBlock), 0, s, seed, d, K, half_bits, i0, n,
                       perm, bucket);
    return hipGetLastError();
}

hipError_t launch_rng_probe(uint64_t seed, int64_t n, uint32_t* sink, hipStream_t s)
{
    // a few workgroups per CU looping over the units: one atomic per wave
    const int64_t units = (n + 8 * kRngProbeStreams - 1) / (8 * kRngProbeStreams);
    const int64_t blocks = grid_for(units, kRngMaxGrid);
    hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(1), 0, s, sink);
    if (short_blocks(0, 8 * units))
        hipLaunchKernelGGL(k_rng_probe<uint32_t>, dim3((unsigned)blocks), dim3(kBlock), 0, s, seed, units, sink);
    else
        hipLaunchKernelGGL(k_rng_probe<uint64_t>, dim3((unsigned)blocks), dim3(kBlock), 0, s, seed, units, sink);
    return hipGetLastError();
}

hipError_t launch_probe_map_copy(int dtype, int addr, int direction, const StreamArgs& a, hipStream_t s)
{
    const int64_t g = grid_for(a.length);
#define CPES_PROBE(T, D, A) hipLaunchKernelGGL((k_probe_map_copy<T, D, A>), dim3((unsigned)g), dim3(kBlock), 0, s, a)
    if (dtype == 0) {
        if (addr == kGather32) {
            if (direction == 0) CPES_PROBE(uint16_t, 0, kGather32); else CPES_PROBE(uint16_t, 1, kGather32);
        } else {
            if (direction == 0) CPES_PROBE(uint16_t, 0, kGather); else CPES_PROBE(uint16_t, 1, kGather);
        }
    } else {
        if (addr == kGather32) {
            if (direction == 0) CPES_PROBE(float, 0, kGather32); else CPES_PROBE(float, 1, kGather32);
        } else {
            if (direction == 0) CPES_PROBE(float, 0, kGather); else CPES_PROBE(float, 1, kGather);
        }
    }
#undef CPES_PROBE
    return hipGetLastError();
}

hipError_t launch_probe_copy(const void* src, void* dst, int64_t bytes, bool nontemporal, hipStream_t s)
{
    const int64_t n16 = bytes / 16;
    const dim3 grid((unsigned)grid_for(n16)), block(kBlock);
    if (nontemporal)
        hipLaunchKernelGGL(k_probe_copy<true>, grid, block, 0, s, static_cast<const V4u*>(src), static_cast<V4u*>(dst), n16);
    else
        hipLaunchKernelGGL(k_probe_copy<false>, grid, block, 0, s, static_cast<const V4u*>(src), static_cast<V4u*>(dst), n16);
    return hipGetLastError();
}

}  // namespace cpes
