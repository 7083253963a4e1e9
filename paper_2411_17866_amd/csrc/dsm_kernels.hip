// gfx950 kernels of distributed sign momentum with local steps
// (arXiv 2411.17866, Algorithm 1).
//
// Every kernel streams fp32 arenas: a wave takes one strip (64 lanes x one
// float4 = 256 elements, 1 KiB per stream) of one chunk of one tensor, with
// 128-bit loads and stores, nontemporal where nothing reads the line again soon
// (Policy, below), consecutive lanes on consecutive 16-byte groups, and every
// element is read and written once per pass.
// Nothing here is a dense contraction, so there is no MFMA; the bound is HBM
// bandwidth, and what is left to gain is how close the mix of read and write
// streams comes to it (see "Launch shape" below).
//
// Arithmetic: fp32, one IEEE round-to-nearest operation per written
// operation, in the order the formulas are written; no contraction into FMA
// (-ffp-contract=off and the pragma below), correctly rounded division and
// square root, denormals kept.
#include <hip/hip_runtime.h>

#include <mutex>

#include "dsm_internal.h"
#include "philox_device.h"

#pragma clang fp contract(off)

namespace dsm {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

// Cache policy of a launch's streams.
// kStream: nontemporal loads and stores, for arenas that have left every cache
// before they are read again.
// kShared: the same, but for a local step's starting point, which in the
// interleaved order the n workers read one soon after the other: a plain load
// leaves it in the caches for the others, and x comes from HBM once.
// kCached: plain loads and stores, for problems whose arenas are still in the
// 256 MB last-level cache at the next call (RepLayout::cached()): rounds of 1.1M
// elements, n = 2, 27.8 us against 36.6 us with nontemporal ones; 8 x 128K,
// n = 4 (75 MB), 74.4 us against 84.0 us; but 161 MB 167.9 against 165.2 us and
// 510 MB 344 against 317 us.  It pays for as long as the program's other kernels
// leave room: 8 x 128K, n = 4, H = 4, the gradients written and a copy made
// before each call, the round with all of that 101 us against 106 us without a
// copy, 121 against 132 us where it moves 32 MB, 176 against 186 us with 128 MB.  It costs once they fill the cache themselves, whose lines plain
// accesses then displace and whose stores they wait for: 312 against 268 us with
// 256 MB; after a 512 MB fill, local steps of 2M to 5M elements of all workers
// take 16-20% longer.
enum Policy { kStream, kShared, kCached };

template <int POLICY>
__device__ __forceinline__ f4 load(const f4* p) {
    if constexpr (POLICY == kCached)
        return *p;
    else
        return __builtin_nontemporal_load(p);
}
template <int POLICY>
__device__ __forceinline__ void store(f4 v, f4* p) {
    if constexpr (POLICY == kCached)
        *p = v;
    else
        __builtin_nontemporal_store(v, p);
}

// Stores the first k (1..3) lanes of v: the ragged end of a tensor.
__device__ __forceinline__ void store_head(f4 v, float* p, int k) {
    p[0] = v.x;
    if (k > 1) p[1] = v.y;
    if (k > 2) p[2] = v.z;
}

// Stores v at p: the whole group when its four lanes are inside the chunk
// (valid >= 4), else only the valid lanes.
template <int POLICY>
__device__ __forceinline__ void store_vec(f4 v, f4* p, int valid) {
    if (valid >= 4)
        store<POLICY>(v, p);
    else
        store_head(v, reinterpret_cast<float*>(p), valid);
}

// Where copy i of a replica buffer keeps arena element e (RepLayout):
// (e >> shift) * block_stride + i * copy_stride + (e & (2^shift - 1)).
// Contiguous copies use shift 62 (the block term vanishes) and copy_stride =
// d_pad; 64 KiB blocks interleaved by copy use shift 14, block_stride =
// n * 16384 and copy_stride = 16384; "every copy is x" uses shift 62 and
// copy_stride 0.  A strip never crosses a block, so one base per strip and
// copy serves the whole wave.
__device__ __forceinline__ int64_t rep_index(const RepLayout& L, int64_t i, int64_t e) {
    const int64_t mask = (int64_t(1) << L.shift) - 1;
    return (e >> L.shift) * L.block_stride + i * L.copy_stride + (e & mask);
}

// ---------------------------------------------------------------- strips

// A strip of a chunk: 64 consecutive float4 groups, one per lane of a wave
// (fewer at the chunk's end, none past it).  Wave-uniform.
struct Strip {
    Chunk c;
    int nq;          // float4 groups in the strip
    int valid0;      // lanes of the chunk from the strip's first group on
    int64_t e0;      // arena element of the strip's first group
    uint32_t j4;     // in-tensor index of the first group, divided by 4
    uint32_t piece;  // the 1024-element piece the strip lies in
};

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }
__device__ __forceinline__ int wave_id() {
    return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

// The chunk that holds strip group g (Chunk.group0 ascends over the chunks):
// a 64-ary search by the whole wave, one gather per factor of 64 in the
// number of chunks.  Fetching whole chunks at the last level, to spare the load
// of the one found, gains 0.6% with 13 tensors and loses 2% with 400, and two
// strips per search lose 1% (rounds of 17.4 and 78.4 us).
__device__ __forceinline__ uint32_t find_chunk(const Chunk* __restrict__ chunks, uint32_t n_chunks,
                                               uint32_t g) {
    ChunkRange r{0, n_chunks};
    while (r.size > 1) {
        const uint32_t at = probe_of(r, static_cast<uint32_t>(lane_id()));
        const bool at_or_below = at < r.size && chunks[r.lo + min(at, r.size - 1)].group0 <= g;
        r = narrowed(r, static_cast<uint32_t>(__popcll(__ballot(at_or_below))));
    }
    return __builtin_amdgcn_readfirstlane(r.lo);
}

// Strip si of a launch: of all chunks' kStrips each, or (rows.sparse_chunks
// > 0) of the strip groups that hold elements.
__device__ __forceinline__ Strip strip_at(const Chunk* __restrict__ chunks, const Rows& rows,
                                          uint32_t si) {
    uint32_t ci = si / kStrips, s = si % kStrips;
    if (rows.sparse_chunks > 0) {
        ci = find_chunk(chunks, rows.sparse_chunks, si / kGroupStrips);
        s = si - chunks[ci].group0 * kGroupStrips;
    }
    Strip st;
    st.c = chunks[ci];
    const int nvec = (st.c.len + 3) >> 2;
    const int q_lo = static_cast<int>(s) * kStripVec;
    st.nq = max(0, min(nvec - q_lo, kStripVec));
    st.valid0 = st.c.len - 4 * q_lo;
    st.e0 = st.c.off + 4 * static_cast<int64_t>(q_lo);
    st.j4 = static_cast<uint32_t>(st.c.j0 >> 2) + static_cast<uint32_t>(q_lo);
    st.piece = ci * kSplit + s / kQuadWaves;
    return st;
}

// Strip k (0..3) of work-group b of a launch over pieces (quads): strip
// b % 8 + 8 k of the 32 strips of work-groups 8 (b / 8) to 8 (b / 8) + 7, so
// that the XCDs, which get the work-groups in turn, interleave at 1 KiB as
// with one-strip work-groups; over sparse chunks, whose neighbouring strip
// groups may lie in different tensors, four consecutive strips.
__device__ __forceinline__ Strip quad_strip(const Chunk* __restrict__ chunks, const Rows& rows,
                                            int k) {
    const uint32_t b = blockIdx.x, uk = static_cast<uint32_t>(k);
    if (rows.sparse_chunks > 0) return strip_at(chunks, rows, b * kQuadWaves + uk);
    return strip_at(chunks, rows, b / kXcds * (kXcds * kQuadWaves) + uk * kXcds + b % kXcds);
}

// The strip of this wave: of a one-wave work-group, or of a quad of four.
__device__ __forceinline__ Strip strip_of(const Chunk* __restrict__ chunks, const Rows& rows) {
    if (rows.map & kQuads) return quad_strip(chunks, rows, wave_id());
    return strip_at(chunks, rows, blockIdx.x);
}

// The bound word of work-group b of a quad launch.
__device__ __forceinline__ uint32_t quad_word(const Strip& st, const Rows& rows) {
    return rows.sparse_chunks > 0 ? st.piece : blockIdx.x;
}

// The strip and worker of a local step's wave.  Without kInterleaveWorkers in
// the map the grid is (work-groups, workers) and runs worker by worker; with it
// the grid is one row of strips x workers in which a turn of one worker is
// followed by the same turn of the next: a strip group (eight strips, one per
// XCD), or (WIDE, kWideTurns) kTurnGroups of them, the last turn maybe fewer.
template <bool WIDE>
__device__ __forceinline__ Strip local_strip(const Chunk* __restrict__ chunks, const Rows& rows,
                                             int worker0, int n_workers, int64_t& w) {
    const uint32_t b = blockIdx.x;
    if (rows.map & kInterleaveWorkers) {
        const uint32_t g = b / kGroupStrips, n = static_cast<uint32_t>(n_workers);
        uint32_t worker = g % n, group = g / n;
        if (WIDE && (rows.map & kWideTurns)) {
            const uint32_t turn = g / (kTurnGroups * n), r = g % (kTurnGroups * n);
            const uint32_t size =
                min(kTurnGroups, gridDim.x / kGroupStrips / n - turn * kTurnGroups);
            worker = r / size;
            group = turn * kTurnGroups + r % size;
        }
        w = worker0 + static_cast<int64_t>(worker);
        return strip_at(chunks, rows, group * kGroupStrips + b % kGroupStrips);
    }
    w = worker0 + static_cast<int64_t>(blockIdx.y);
    return strip_of(chunks, rows);
}

// ---------------------------------------------------------------- AdamW

// Correctly rounded square root (the build asks for correctly rounded fp32
// division and square root).
__device__ __forceinline__ f4 sqrt_rn(f4 a) {
    return f4{__builtin_sqrtf(a.x), __builtin_sqrtf(a.y), __builtin_sqrtf(a.z), __builtin_sqrtf(a.w)};
}

// Algorithm 2 on four elements (lane-wise); x, m, v updated in place.
__device__ __forceinline__ void adamw4(f4& x, f4 g, f4& m, f4& v, float lam, const AdamScalars& s) {
    const f4 m1 = s.beta1 * m;
    const f4 m2 = s.one_minus_beta1 * g;
    m = m1 + m2;
    const f4 gg = g * g;
    const f4 v1 = s.beta2 * v;
    const f4 v2 = s.one_minus_beta2 * gg;
    v = v1 + v2;
    const f4 m_hat = m / s.bc1;
    const f4 v_hat = v / s.bc2;
    const f4 den = sqrt_rn(v_hat) + s.eps;
    const f4 r = m_hat / den;
    const f4 wx = lam * x;
    const f4 d = r + wx;
    const f4 st = s.lr * d;
    x = x - st;
}

// Worker w reads its step's starting point at x_src + rep_index(sl, w, e)
// (its own replica, or with a zero copy stride the global model x when the
// replicas are stale after a global step without broadcast) and writes the
// result to its replica, x_rep + rep_index(rl, w, e); its gradient and
// moments sit at rep_index(ml.g / ml.s1 / ml.s2, w, e) of their buffers.  The two may be the
// same memory, so neither pointer is __restrict__; each lane loads every
// stream of its group before it stores.
template <int POLICY>
__global__ __launch_bounds__(kBlockThreads) void k_local_adamw(
    const Chunk* __restrict__ chunks, Rows rows, float* x_rep, RepLayout rl, const float* x_src,
    RepLayout sl, const float* __restrict__ g_rep, float* __restrict__ s1,
    float* __restrict__ s2, StateLayout ml, int worker0, int n_workers, AdamScalars sc) {
    int64_t w;
    const Strip st = local_strip<POLICY == kShared>(chunks, rows, worker0, n_workers, w);
    const int q = lane_id();
    if (q >= st.nq) return;
    f4* xp = reinterpret_cast<f4*>(x_rep + rep_index(rl, w, st.e0)) + q;
    f4* mp = reinterpret_cast<f4*>(s1 + rep_index(ml.s1, w, st.e0)) + q;
    f4* vp = reinterpret_cast<f4*>(s2 + rep_index(ml.s2, w, st.e0)) + q;
    f4 x = load<POLICY == kShared ? kCached : POLICY>(
        reinterpret_cast<const f4*>(x_src + rep_index(sl, w, st.e0)) + q);
    const f4 g = load<POLICY>(reinterpret_cast<const f4*>(g_rep + rep_index(ml.g, w, st.e0)) + q);
    f4 m = load<POLICY>(mp), v = load<POLICY>(vp);
    adamw4(x, g, m, v, st.c.decay ? sc.wd : 0.0f, sc);
    const int valid = st.valid0 - 4 * q;
    store_vec<POLICY>(x, xp, valid);
    store_vec<POLICY>(m, mp, valid);
    store_vec<POLICY>(v, vp, valid);
}

// ---------------------------------------------------------------- SGD + momentum

// Algorithm 3 on four elements (lane-wise).
__device__ __forceinline__ void sgdm4(f4& x, f4 g, f4& m, const SgdScalars& s) {
    const f4 m1 = s.mu * m;
    m = m1 + g;
    const f4 st = s.lr * m;
    x = x - st;
}

template <int POLICY>
__global__ __launch_bounds__(kBlockThreads) void k_local_sgdm(
    const Chunk* __restrict__ chunks, Rows rows, float* x_rep, RepLayout rl, const float* x_src,
    RepLayout sl, const float* __restrict__ g_rep, float* __restrict__ s1, StateLayout ml,
    int worker0, int n_workers, SgdScalars sc) {
    int64_t w;
    const Strip st = local_strip<POLICY == kShared>(chunks, rows, worker0, n_workers, w);
    const int q = lane_id();
    if (q >= st.nq) return;
    f4* xp = reinterpret_cast<f4*>(x_rep + rep_index(rl, w, st.e0)) + q;
    f4* mp = reinterpret_cast<f4*>(s1 + rep_index(ml.s1, w, st.e0)) + q;
    f4 x = load<POLICY == kShared ? kCached : POLICY>(
        reinterpret_cast<const f4*>(x_src + rep_index(sl, w, st.e0)) + q);
    const f4 g = load<POLICY>(reinterpret_cast<const f4*>(g_rep + rep_index(ml.g, w, st.e0)) + q);
    f4 m = load<POLICY>(mp);
    sgdm4(x, g, m, sc);
    const int valid = st.valid0 - 4 * q;
    store_vec<POLICY>(x, xp, valid);
    store_vec<POLICY>(m, mp, valid);
}

// ---------------------------------------------------------------- global step

// sign with sign(+-0) = +0 and sign(NaN) = NaN.
__device__ __forceinline__ float sign_of(float u) {
    return u > 0.0f ? 1.0f : (u < 0.0f ? -1.0f : (u == u ? 0.0f : u));
}

// Worker sum of (x - x_i) over the n replicas of group q of the strip that
// starts at arena element e0, in worker order, divided by n.  N > 0:
// compile-time worker count (a power of two, so the division is the exact
// multiplication by 1/n), every replica's load in flight together; N == 0:
// runtime count, kReplicaBatch loads in flight at a time.
constexpr int kReplicaBatch = 4;
template <int N, int POLICY>
__device__ __forceinline__ f4 worker_mean_diff(f4 xv, const float* __restrict__ x_rep,
                                               const RepLayout& rl, int64_t e0, int q,
                                               const GlobalScalars& s) {
    if constexpr (N > 0) {
        f4 r[N];
#pragma unroll
        for (int i = 0; i < N; ++i)
            r[i] = load<POLICY>(reinterpret_cast<const f4*>(x_rep + rep_index(rl, i, e0)) + q);
        f4 acc = xv - r[0];
#pragma unroll
        for (int i = 1; i < N; ++i) acc = acc + (xv - r[i]);
        return acc * s.inv_n;
    } else {
        f4 acc;
        for (int i0 = 0; i0 < s.n; i0 += kReplicaBatch) {
            f4 r[kReplicaBatch];
#pragma unroll
            for (int k = 0; k < kReplicaBatch; ++k)
                if (i0 + k < s.n)
                    r[k] = load<POLICY>(reinterpret_cast<const f4*>(x_rep + rep_index(rl, i0 + k, e0)) + q);
#pragma unroll
            for (int k = 0; k < kReplicaBatch; ++k)
                if (i0 + k < s.n) {
                    const f4 d = xv - r[k];
                    acc = (i0 + k == 0) ? d : acc + d;
                }
        }
        if (s.n_pow2) return acc * s.inv_n;
        return acc / s.n_f;
    }
}

__device__ __forceinline__ f4 sign4(f4 u) {
    return f4{sign_of(u.x), sign_of(u.y), sign_of(u.z), sign_of(u.w)};
}

// Eqs. (6) and (8) from the old m, lane-wise; returns u, updates m.
__device__ __forceinline__ f4 momentum4(f4& m, f4 delta, const GlobalScalars& s) {
    const f4 u1 = s.beta1 * m;
    const f4 u2 = s.c1 * delta;
    const f4 u = u1 + u2;
    const f4 m1 = s.beta2 * m;
    const f4 m2 = s.c2 * delta;
    m = m1 + m2;
    return u;
}

// Eq. (7) with the applied sign S, lane-wise.
__device__ __forceinline__ f4 model4(f4 x, f4 S, float lam, const GlobalScalars& s) {
    const f4 wx = lam * x;
    const f4 a = S + wx;
    const f4 st = s.step * a;
    return x - st;
}

// Global-step rules (dsm_global_rule).
constexpr int kRuleSignMomentum = 0;  // Eqs. (6)-(8)
constexpr int kRuleLookahead = 1;     // Section 4.1: x - eta gamma (u + lambda x)
constexpr int kRuleSignedSlowMo = 2;  // Section 4.1: sign on the averaged difference
constexpr int kRuleGlobalAdamW = 3;   // Algorithm 7

// Algorithm 7 on four elements: AdamW on the pseudo-gradient
// g = (1/gamma) delta; m and v updated in place; returns the new x.
__device__ __forceinline__ f4 global_adamw4(f4 x, f4 delta, f4& m, f4& v, float lam,
                                           const GlobalScalars& s) {
    const f4 g = s.inv_gamma * delta;
    const f4 m1 = s.beta1 * m;
    const f4 m2 = s.one_minus_beta1 * g;
    m = m1 + m2;
    const f4 gg = g * g;
    const f4 v1 = s.beta2 * v;
    const f4 v2 = s.one_minus_beta2 * gg;
    v = v1 + v2;
    const f4 m_hat = m / s.bc1;
    const f4 v_hat = v / s.bc2;
    const f4 den = sqrt_rn(v_hat) + s.eps;
    const f4 r = m_hat / den;
    const f4 wx = lam * x;
    const f4 d = r + wx;
    const f4 st = s.eta * d;
    return x - st;
}

template <int N, int RULE, bool BCAST, int POLICY>
__global__ __launch_bounds__(kBlockThreads) void k_global_det(
    const Chunk* __restrict__ chunks, Rows rows, float* __restrict__ x, float* __restrict__ m,
    float* __restrict__ v, float* __restrict__ x_rep, RepLayout rl, GlobalScalars sc) {
    const Strip st = strip_of(chunks, rows);
    const int q = lane_id();
    if (q >= st.nq) return;
    const int n = N > 0 ? N : sc.n;
    f4* __restrict__ xp = reinterpret_cast<f4*>(x + st.e0) + q;
    f4* __restrict__ mp = reinterpret_cast<f4*>(m + st.e0) + q;
    f4* __restrict__ vp = reinterpret_cast<f4*>(v + st.e0) + q;
    const float lam = st.c.decay ? sc.lam : 0.0f;
    const int valid = st.valid0 - 4 * q;
    const f4 xv = load<POLICY>(xp);
    f4 mv = load<POLICY>(mp), vv;
    if (RULE == kRuleGlobalAdamW) vv = load<POLICY>(vp);
    const f4 delta = worker_mean_diff<N, POLICY>(xv, x_rep, rl, st.e0, q, sc);
    f4 xn;
    if constexpr (RULE == kRuleSignMomentum) {
        const f4 u = momentum4(mv, delta, sc);
        xn = model4(xv, sign4(u), lam, sc);
    } else if constexpr (RULE == kRuleLookahead) {
        const f4 u = momentum4(mv, delta, sc);
        xn = model4(xv, u, lam, sc);
    } else if constexpr (RULE == kRuleSignedSlowMo) {
        // u from the old m and the sign of the difference; m by Eq. (8).
        const f4 u1 = sc.beta1 * mv;
        const f4 u2 = sc.c1 * sign4(delta);
        const f4 u = u1 + u2;
        const f4 m1 = sc.beta2 * mv;
        const f4 m2 = sc.c2 * delta;
        mv = m1 + m2;
        xn = model4(xv, u, lam, sc);
    } else {
        xn = global_adamw4(xv, delta, mv, vv, lam, sc);
        store_vec<POLICY>(vv, vp, valid);
    }
    store_vec<POLICY>(xn, xp, valid);
    store_vec<POLICY>(mv, mp, valid);
    if (BCAST) {
        for (int i = 0; i < n; ++i)
            store_vec<POLICY>(xn, reinterpret_cast<f4*>(x_rep + rep_index(rl, i, st.e0)) + q, valid);
    }
}

// Largest of a wave's values, in every lane.
__device__ __forceinline__ uint32_t wave_max(uint32_t bits) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t o = __shfl_xor(bits, off, 64);
        bits = o > bits ? o : bits;
    }
    return bits;
}

// Largest of the values of a work-group of THREADS threads, valid in thread
// 0.  lds holds THREADS / 64 words of LDS.
template <int THREADS>
__device__ __forceinline__ uint32_t block_max(uint32_t bits, uint32_t* lds) {
    bits = wave_max(bits);
    if (lane_id() == 0) lds[threadIdx.x >> 6] = bits;
    __syncthreads();
    uint32_t b = lds[0];
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < THREADS / 64; ++w) b = lds[w] > b ? lds[w] : b;
    }
    return b;
}

// Largest |u| of the first `valid` lanes, as a bit pattern (for non-negative
// IEEE floats the unsigned order of the bit patterns is the numeric order).
__device__ __forceinline__ uint32_t abs_max(f4 u, int valid) {
    uint32_t b = __float_as_uint(fabsf(u.x));
    if (valid > 1) b = max(b, __float_as_uint(fabsf(u.y)));
    if (valid > 2) b = max(b, __float_as_uint(fabsf(u.z)));
    if (valid > 3) b = max(b, __float_as_uint(fabsf(u.w)));
    return b;
}

// Randomized sign, pass 1: the all-reduce difference, u_{t+1} (staged to u)
// and m_{t+1} (Eqs. (6), (8)), and the tensor bound B_p = max |u|, reduced in
// two levels with plain loads and stores and no atomics.  Level one: each
// work-group (a quad) stores its largest |u| in its own word.  Level two is
// k_bound_reduce.
template <int N, int POLICY>
__global__ __launch_bounds__(kBlockThreads) void k_global_rand_pass1(
    const Chunk* __restrict__ chunks, Rows rows, const float* __restrict__ x,
    float* __restrict__ m, const float* __restrict__ x_rep, RepLayout rl,
    float* __restrict__ u_out, uint32_t* __restrict__ piece_max, GlobalScalars sc) {
    __shared__ uint32_t lds[kBlockThreads / 64];
    const Strip st = strip_of(chunks, rows);
    const int q = lane_id();
    uint32_t maxbits = 0;
    if (q < st.nq) {
        f4* __restrict__ mp = reinterpret_cast<f4*>(m + st.e0) + q;
        const f4 xv = load<POLICY>(reinterpret_cast<const f4*>(x + st.e0) + q);
        f4 mv = load<POLICY>(mp);
        const f4 delta = worker_mean_diff<N, POLICY>(xv, x_rep, rl, st.e0, q, sc);
        const int valid = st.valid0 - 4 * q;  // lanes inside the tensor
        const f4 u = momentum4(mv, delta, sc);
        store_vec<POLICY>(u, reinterpret_cast<f4*>(u_out + st.e0) + q, valid);
        store_vec<POLICY>(mv, mp, valid);
        maxbits = abs_max(u, valid);
    }
    maxbits = block_max<kBlockThreads>(maxbits, lds);
    if (threadIdx.x == 0) piece_max[quad_word(st, rows)] = maxbits;
}

// The level-one words of tensor p: kSplit for each of its chunks.  Over sparse
// chunks only the words of the strip groups that hold elements have been
// written: a prefix, since all chunks of a tensor but the last are full.
struct BoundRange {
    int64_t lo, n;  // lo a multiple of 4 words, which start 256-byte aligned
};
__device__ __forceinline__ BoundRange bound_range(const Chunk* __restrict__ chunks,
                                                  const int32_t* __restrict__ chunk0, uint32_t p,
                                                  bool sparse) {
    const int32_t c_lo = chunk0[p], c_hi = chunk0[p + 1];
    BoundRange r{static_cast<int64_t>(c_lo) * kSplit, static_cast<int64_t>(c_hi - c_lo) * kSplit};
    if (sparse && r.n > 0)
        r.n -= kSplit - (chunks[c_hi - 1].len + kGroupElems - 1) / kGroupElems * kGroupPieces;
    return r;
}

// Largest of every THREADS-th four of r's words from thread t's on.
template <int THREADS>
__device__ __forceinline__ uint32_t max_words(const uint32_t* __restrict__ piece_max,
                                              const BoundRange& r, int t) {
    uint32_t b = 0;
    const uint4* __restrict__ v = reinterpret_cast<const uint4*>(piece_max + r.lo);
#pragma unroll 4
    for (int64_t i = t; i < r.n / 4; i += THREADS) {
        const uint4 w = v[i];
        b = max(b, max(max(w.x, w.y), max(w.z, w.w)));
    }
    const int64_t i = r.n / 4 * 4 + t;
    return i < r.n ? max(b, piece_max[r.lo + i]) : b;
}

// Level two of the tensor bound: work-group p stores the largest level-one
// word of tensor p in bound_bits[p]; an empty tensor has none and gets 0.
constexpr int kReduceThreads = 1024;
__global__ __launch_bounds__(kReduceThreads) void k_bound_reduce(
    const Chunk* __restrict__ chunks, const uint32_t* __restrict__ piece_max,
    const int32_t* __restrict__ chunk0, uint32_t* __restrict__ bound_bits, bool sparse) {
    __shared__ uint32_t lds[kReduceThreads / 64];
    const BoundRange r = bound_range(chunks, chunk0, blockIdx.x, sparse);
    const uint32_t b = block_max<kReduceThreads>(
        max_words<kReduceThreads>(piece_max, r, static_cast<int>(threadIdx.x)), lds);
    if (threadIdx.x == 0) bound_bits[blockIdx.x] = b;
}

// S_r(u) of Eq. (9) (MODE 1) or Eq. (10) (MODE 2) for one element, given the
// Philox word w (U = (w >> 8) 2^-24) and the bound B (as double).  "sign(u)
// with probability p" is decided by the exact comparison U < p, evaluated in
// fp64 where both sides are exact: (2k - 2^24) B < |u| 2^24 for Eq. (9),
// k B < |u| 2^24 for Eq. (10).
template <int MODE>
__device__ __forceinline__ float rand_sign(float u, uint32_t w, double B) {
    const float sgn = sign_of(u);
    const double au = static_cast<double>(fabsf(u)) * 16777216.0;
    const int32_t k = static_cast<int32_t>(w >> 8);
    if constexpr (MODE == 1) {
        const double a = static_cast<double>(2 * k - (1 << 24));
        return (a * B < au) ? sgn : 0.0f - sgn;
    } else {
        return (static_cast<double>(k) * B < au) ? sgn : 0.0f;
    }
}

// Randomized sign, pass 2: S_r, Eq. (7) and the synchronisation step.
// Section 3.1 defines S_r only for a finite bound: a tensor whose bound is
// NaN or infinite (it holds a non-finite u) gets S = NaN at every element,
// so its step is NaN rather than a step of a reversed or zero sign.
//
// FOLD: level two of the bound as well.  Each wave takes the maximum of its
// tensor's words itself, and the wave of the tensor's first strip stores it.
template <int MODE, bool BCAST, int POLICY, bool FOLD>
__global__ __launch_bounds__(kBlockThreads) void k_global_rand_pass2(
    const Chunk* __restrict__ chunks, Rows rows, float* __restrict__ x, float* __restrict__ x_rep,
    RepLayout rl, const float* __restrict__ u_in, BoundWords bw, GlobalScalars sc) {
    const Strip st = strip_of(chunks, rows);
    const int q = lane_id();
    if (st.nq == 0) return;
    const bool on = q < st.nq;
    f4* __restrict__ xp = reinterpret_cast<f4*>(x + st.e0) + q;
    f4 xv, u;
    if (on) {
        xv = load<POLICY>(xp);
        u = load<POLICY>(reinterpret_cast<const f4*>(u_in + st.e0) + q);
    }
    uint32_t bbits;
    if constexpr (FOLD) {
        const BoundRange r = bound_range(chunks, bw.chunk0, st.c.tensor, rows.sparse_chunks > 0);
        bbits = wave_max(max_words<kWave>(bw.piece_max, r, q));
        if (st.j4 == 0 && q == 0) bw.bits[st.c.tensor] = bbits;
    } else {
        bbits = bw.bits[st.c.tensor];
    }
    if (!on) return;
    const float lam = st.c.decay ? sc.lam : 0.0f;
    const bool bound_finite = bbits < 0x7f800000u;   // B >= 0: below the +inf pattern
    const double B = static_cast<double>(__uint_as_float(bbits));
    const float undefined = __builtin_nanf("");
    uint32_t w0 = st.j4 + static_cast<uint32_t>(q), w1 = st.c.tensor, w2 = sc.t, w3 = kSignStream;
    philox4x32_10(w0, w1, w2, w3, sc.key0, sc.key1);
    f4 S = {rand_sign<MODE>(u.x, w0, B), rand_sign<MODE>(u.y, w1, B),
            rand_sign<MODE>(u.z, w2, B), rand_sign<MODE>(u.w, w3, B)};
    if (!bound_finite) S = f4{undefined, undefined, undefined, undefined};
    const f4 xn = model4(xv, S, lam, sc);
    const int valid = st.valid0 - 4 * q;
    store_vec<POLICY>(xn, xp, valid);
    if (BCAST) {
        for (int i = 0; i < sc.n; ++i)
            store_vec<POLICY>(xn, reinterpret_cast<f4*>(x_rep + rep_index(rl, i, st.e0)) + q, valid);
    }
}

// ---------------------------------------------------------------- fused round end

// Base optimizer of the fused round end.
constexpr int kBaseAdamW = 0;
constexpr int kBaseSgd = 1;

// The last local step of every worker (Algorithm 2 or 3, Eq. (4)) fused with
// the global step (all-reduce, Eqs. (6)-(8)): each worker's step-H replica
// value stays on the CU and is folded into the worker-order sum
// sum_i (x - x_i), so the replicas are neither stored after step H nor read
// back.  Per element the operations and their order are those of k_local_*
// followed by k_global_det / k_global_rand_pass1, so the results are
// bit-identical.  KIND: 0 deterministic sign, 1 deterministic sign with
// broadcast, 2 randomized pass 1 (u, m and the bound; pass 2 follows).
//
// A strip's workers are spread over `workers` waves of a work-group, which
// leave their step-H values in LDS for the first of them to do the global
// step.  PIECE false: a work-group takes one strip (KIND 2: and raises its
// bound word by an atomic max).  PIECE true (KIND 2): it takes the four strips
// of a bound word side by side and stores the word.
template <int BASE, int KIND, bool PIECE, int POLICY>
__global__ __launch_bounds__(kMaxRoundEndWaves * kWave) void k_round_end(
    const Chunk* __restrict__ chunks, Rows rows, float* x, float* __restrict__ m, float* x_rep,
    RepLayout rl, const float* x_src, RepLayout sl, const float* __restrict__ g_rep,
    float* __restrict__ s1, float* __restrict__ s2, float* __restrict__ u_out,
    uint32_t* __restrict__ piece_max, StateLayout ml, int workers, AdamScalars as, SgdScalars ss,
    GlobalScalars gs) {
    // x_src is the replicas or, when they are stale, x itself: it may alias
    // x and x_rep, so none of the three is __restrict__.  Every load of a
    // group precedes its stores.
    extern __shared__ f4 x_end[];  // [strips][n][64]: step-H values
    const int q = lane_id();
    const int k = PIECE ? wave_id() / workers : 0;  // which of the strips
    const int w0 = PIECE ? wave_id() % workers : wave_id();
    f4* const ends = x_end + k * gs.n * kWave + q;
    const Strip st = PIECE ? quad_strip(chunks, rows, k) : strip_at(chunks, rows, blockIdx.x);
    uint32_t maxbits = 0;
    const bool on = q < st.nq;
    const int valid = st.valid0 - 4 * q;
    f4* xp = reinterpret_cast<f4*>(x + st.e0) + q;
    f4* __restrict__ mp = reinterpret_cast<f4*>(m + st.e0) + q;
    f4 xv, mv;
    if (w0 == 0 && on) {
        xv = load<POLICY>(xp);
        mv = load<POLICY>(mp);
    }
    const float lam_local = st.c.decay ? as.wd : 0.0f;
    for (int i = w0; i < gs.n && on; i += workers) {
        f4* __restrict__ s1p = reinterpret_cast<f4*>(s1 + rep_index(ml.s1, i, st.e0)) + q;
        f4 xi = load<POLICY>(reinterpret_cast<const f4*>(x_src + rep_index(sl, i, st.e0)) + q);
        const f4 g = load<POLICY>(reinterpret_cast<const f4*>(g_rep + rep_index(ml.g, i, st.e0)) + q);
        f4 mi = load<POLICY>(s1p);
        if (BASE == kBaseAdamW) {
            f4* __restrict__ s2p = reinterpret_cast<f4*>(s2 + rep_index(ml.s2, i, st.e0)) + q;
            f4 vi = load<POLICY>(s2p);
            adamw4(xi, g, mi, vi, lam_local, as);
            store_vec<POLICY>(vi, s2p, valid);
        } else {
            sgdm4(xi, g, mi, ss);
        }
        store_vec<POLICY>(mi, s1p, valid);
        ends[i * kWave] = xi;
    }
    __syncthreads();
    if (w0 == 0 && on) {
        f4 acc = xv - ends[0];
        for (int i = 1; i < gs.n; ++i) acc = acc + (xv - ends[i * kWave]);
        const f4 delta = gs.n_pow2 ? acc * gs.inv_n : acc / gs.n_f;
        const f4 u = momentum4(mv, delta, gs);
        store_vec<POLICY>(mv, mp, valid);
        if (KIND == 2) {
            store_vec<POLICY>(u, reinterpret_cast<f4*>(u_out + st.e0) + q, valid);
            maxbits = max(maxbits, abs_max(u, valid));
        } else {
            const f4 xn = model4(xv, sign4(u), st.c.decay ? gs.lam : 0.0f, gs);
            store_vec<POLICY>(xn, xp, valid);
            if (KIND == 1) {
                for (int i = 0; i < gs.n; ++i)
                    store_vec<POLICY>(xn, reinterpret_cast<f4*>(x_rep + rep_index(rl, i, st.e0)) + q,
                              valid);
            }
        }
    }
    if constexpr (KIND == 2 && !PIECE) {
        if (w0 == 0) {
            maxbits = wave_max(maxbits);
            if (q == 0) atomicMax(piece_max + st.piece, maxbits);
        }
    }
    if constexpr (PIECE) {
        uint32_t* const strip_max = reinterpret_cast<uint32_t*>(x_end);
        maxbits = wave_max(maxbits);
        __syncthreads();  // the step-H values have been read
        if (w0 == 0 && q == 0) strip_max[k] = maxbits;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int j = 1; j < kQuadWaves; ++j) maxbits = max(maxbits, strip_max[j]);
            piece_max[quad_word(st, rows)] = maxbits;
        }
    }
}

// Zeroes the bound words that atomic maxima will raise.
__global__ __launch_bounds__(kBlockThreads) void k_clear_words(uint4* __restrict__ words,
                                                              int64_t n4) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kBlockThreads + threadIdx.x;
    if (i < n4) words[i] = uint4{0, 0, 0, 0};
}

// ---------------------------------------------------------------- sync / init

// Synchronisation step: x_rep[i] <- x for every replica.
template <int POLICY>
__global__ __launch_bounds__(kBlockThreads) void k_broadcast(
    const Chunk* __restrict__ chunks, Rows rows, const float* __restrict__ x, float* __restrict__ x_rep,
    RepLayout rl, int n) {
    const Strip st = strip_of(chunks, rows);
    const int q = lane_id();
    if (q >= st.nq) return;
    const f4 v = load<POLICY>(reinterpret_cast<const f4*>(x + st.e0) + q);
    const int valid = st.valid0 - 4 * q;
    for (int i = 0; i < n; ++i)
        store_vec<POLICY>(v, reinterpret_cast<f4*>(x_rep + rep_index(rl, i, st.e0)) + q, valid);
}

// Algorithm 1 initialisation: m = 0, replicas = x, base state = 0.
__global__ __launch_bounds__(kBlockThreads) void k_init(
    const Chunk* __restrict__ chunks, Rows rows, const float* __restrict__ x, float* __restrict__ m,
    float* __restrict__ v, float* __restrict__ x_rep, RepLayout rl, float* __restrict__ s1,
    float* __restrict__ s2, StateLayout ml, int n) {
    const Strip st = strip_of(chunks, rows);
    const int q = lane_id();
    if (q >= st.nq) return;
    const f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    const f4 xv = load<kStream>(reinterpret_cast<const f4*>(x + st.e0) + q);
    const int valid = st.valid0 - 4 * q;
    store_vec<kStream>(zero, reinterpret_cast<f4*>(m + st.e0) + q, valid);
    if (v != nullptr) store_vec<kStream>(zero, reinterpret_cast<f4*>(v + st.e0) + q, valid);
    for (int i = 0; i < n; ++i) {
        store_vec<kStream>(xv, reinterpret_cast<f4*>(x_rep + rep_index(rl, i, st.e0)) + q, valid);
        store_vec<kStream>(zero, reinterpret_cast<f4*>(s1 + rep_index(ml.s1, i, st.e0)) + q, valid);
        if (s2 != nullptr)
            store_vec<kStream>(zero, reinterpret_cast<f4*>(s2 + rep_index(ml.s2, i, st.e0)) + q, valid);
    }
}

__global__ __launch_bounds__(kBlockThreads) void k_test_philox(uint32_t key0, uint32_t key1,
                                                              uint32_t tensor, uint32_t t,
                                                              uint32_t q0, int64_t count,
                                                              uint32_t* __restrict__ out) {
    const int64_t b = static_cast<int64_t>(blockIdx.x) * kBlockThreads + threadIdx.x;
    if (b >= count) return;
    uint32_t w0 = q0 + static_cast<uint32_t>(b), w1 = tensor, w2 = t, w3 = kSignStream;
    philox4x32_10(w0, w1, w2, w3, key0, key1);
    out[4 * b + 0] = w0;
    out[4 * b + 1] = w1;
    out[4 * b + 2] = w2;
    out[4 * b + 3] = w3;
}

// Streaming diagnostics with the 16-byte nontemporal accesses of the kernels
// above, consecutive lanes on consecutive groups, in a shape of their own: one
// piece of kPieceVec float4 groups per work-group, XCD k on the k-th eighth of
// the buffer, every wave resident.  The rates are a yardstick, not an upper
// bound of the kernels' shape.  The read
// kernel folds its piece into one word (the XOR of its 32-bit patterns) and
// writes only where that word equals `pattern`, so with a pattern no piece
// matches it issues no write at all: even one 4-byte store per piece,
// interleaved with the loads, costs the read stream a measurable share of
// its rate.  The write kernel stores the float with bit pattern `pattern`.
__device__ __forceinline__ uint32_t stream_piece() {
    const uint32_t b = blockIdx.x, per = gridDim.x / kXcds;
    if (b >= per * kXcds) return b;
    return (b % kXcds) * per + b / kXcds;
}

__global__ __launch_bounds__(kBlockThreads) void k_stream_read(const float* __restrict__ buf,
                                                              uint32_t* __restrict__ words,
                                                              uint32_t pattern) {
    __shared__ uint32_t wave_acc[kBlockThreads / 64];
    const uint32_t wi = stream_piece();
    const f4* __restrict__ p = reinterpret_cast<const f4*>(buf) + static_cast<int64_t>(wi) * kPieceVec;
    uint32_t acc = 0;
    for (int q = threadIdx.x; q < kPieceVec; q += kBlockThreads) {
        const f4 v = load<kStream>(p + q);
        acc ^= __float_as_uint(v.x) ^ __float_as_uint(v.y) ^ __float_as_uint(v.z) ^
               __float_as_uint(v.w);
    }
    for (int off = 32; off > 0; off >>= 1) acc ^= __shfl_xor(acc, off, 64);
    if ((threadIdx.x & 63) == 0) wave_acc[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t total = 0;
        for (int k = 0; k < kBlockThreads / 64; ++k) total ^= wave_acc[k];
        if (total == pattern) words[wi] = 1u;
    }
}

__global__ __launch_bounds__(kBlockThreads) void k_stream_write(float* __restrict__ buf,
                                                               uint32_t pattern) {
    const uint32_t wi = stream_piece();
    f4* __restrict__ p = reinterpret_cast<f4*>(buf) + static_cast<int64_t>(wi) * kPieceVec;
    const float value = __uint_as_float(pattern);
    const f4 v = {value, value, value, value};
    for (int q = threadIdx.x; q < kPieceVec; q += kBlockThreads) store<kStream>(v, p + q);
}

// Launch shape.  All kernels are bound by HBM, and what decides how much of
// it they get is how many DRAM rows their reads and writes fight over.  Three
// things keep that number down:
// * Strips of 1 KiB per stream in grid order: the hardware deals consecutive
//   work-groups to the 8 XCDs in turn, so all XCDs sweep the same few MB of
//   every stream instead of eight regions far apart, and a row is used up
//   while it is open.
// * Few waves per CU: just enough requests in flight (about 48 KiB of reads
//   per CU) to cover the latency.  Dynamic LDS that nothing uses holds the
//   number of resident work-groups down.
// * One wave per work-group where the kernel allows it, so a finished strip
//   is replaced at once.
// Local AdamW, GPT-2 small, n = 4, contiguous (% of 8 TB/s): 4 KiB pieces, an
// eighth of the arena per XCD, all waves resident 70.6-73.1; 4 KiB pieces in
// grid order, 12 waves per CU 79.8; 1 KiB strips 76.9 with all waves resident,
// 79.4 with 16 per CU, 82.7 with 12, below 77 with 8.  With 12 waves per CU and
// the XCDs taking 512 B or 256 B of a stream in turn 77.1 and 64.5, 2 KiB or
// 4 KiB 79.7 and 80.2.  State-blocked, n = 8: 75.8 before, 84.6 now.
//
// Dynamic LDS that lets `groups` work-groups live on a CU.  A CU's 160 KiB come
// in steps of 1280 bytes, so not every count can be had: asked for 13, 19 or 20,
// 14 and 21 (twice) fit.
constexpr unsigned kLdsBytes = 160 * 1024, kLdsStep = 1280;
constexpr unsigned lds_for(int groups) {
    return groups >= kAllWaves ? 0u : kLdsBytes / static_cast<unsigned>(groups) / kLdsStep * kLdsStep;
}
// Work-groups that fit a CU with that much LDS each.
constexpr int groups_with(unsigned lds) {
    return lds == 0 ? kAllWaves : static_cast<int>(kLdsBytes / ((lds + kLdsStep - 1) / kLdsStep * kLdsStep));
}
constexpr bool attainable(int groups) { return groups_with(lds_for(groups)) == groups; }
// The same for work-groups of four waves, the whole number of them nearest to
// `waves` waves per CU (10 gives 12), beside up to 256 bytes of LDS that the
// kernel itself holds: a step more, and one work-group fewer would fit.
constexpr unsigned quad_lds(int waves) {
    return waves >= kAllWaves ? 0u : lds_for((waves + kQuadWaves / 2) / kQuadWaves) - 256;
}
static_assert(groups_with(quad_lds(8)) == 2 && groups_with(quad_lds(10)) == 3 &&
                  groups_with(quad_lds(12)) == 3 && groups_with(quad_lds(16)) == 4 &&
                  groups_with(quad_lds(20)) == 5,
              "work-groups of four waves");

// Waves per CU by kernel, swept from 6 to 32 at GPT-2 small to xl.  Local
// steps: AdamW (four loads) 12, SGD (three, and little arithmetic) 21: medium,
// n = 8, 84.0% against 83.2% with 16 and 78% with 14.  From the shared x one
// load of most waves hits the L2, so a few more.
constexpr int kAdamWWaves = 12, kAdamWSharedWaves = 14;
constexpr int kSgdWaves = 21, kSgdSharedWaves = 18;
static_assert(attainable(kAdamWWaves) && attainable(kAdamWSharedWaves) && attainable(kSgdWaves) &&
                  attainable(kSgdSharedWaves),
              "waves of the local steps");
// The global step loads n + 2 streams at once: n = 4, 80.3% with 8, 77% with
// 12; n = 1, 81.0% with 12, 76% with 8.  n = 2 has 10 in one-wave work-groups
// and 12 in those of four.  Where n has no kernel of its own, four loads are in
// flight at a time, and without the broadcast's stores 8 waves are too few: 100M
// elements of all workers, n = 5, contiguous 140 us with 8, 119 us with 12 (the
// kernel before 121 us), state-blocked 145 and 119 us; n = 3 165 and 141 us, n =
// 9 105 and 94 us; n = 12 91 us with 8, 86 us with 10, 400M 338 us with 10, 349
// us with 12.  From 16 workers on 8 again (n = 16, 400M, state-blocked 312 us
// with 8, 323 us with 10), and with the broadcast at every n.
constexpr int global_waves(int n, bool broadcast) {
    if (n <= 2) return n == 1 ? 12 : 10;
    if (broadcast || n == 4 || n == 8 || n >= 16) return 8;
    return n < 10 ? 12 : 10;
}
static_assert(attainable(8) && attainable(10) && attainable(12), "waves of the global step");
// The randomized first pass has no replica to write and lasts well with a few
// more: n = 4 and 8, 80.7-81.8% with 12; n = 1 and 2, 79.6 and 83.3% with 16.
constexpr int pass1_waves(int n) { return n <= 2 ? 16 : 12; }
// The second pass and the synchronisation load two streams and one; their
// stores count: with one worker 21 (20 in work-groups of four) and all of them
// (sync, n = 1: 81.5%, 71% with 12), down to 12 and 8 with many (sync, n = 8:
// 82-86%, 74% with 32).
constexpr int pass2_waves(int stores) { return stores <= 2 ? 21 : stores == 3 ? 16 : 12; }
static_assert(attainable(pass2_waves(2)) && attainable(pass2_waves(3)) && attainable(pass2_waves(4)),
              "waves of the second pass");
constexpr int copy_waves(int n) {
    return n == 1 ? kAllWaves : n == 2 ? 20 : n == 3 ? 16 : n <= 5 ? 12 : 8;
}
constexpr int init_waves(int n) { return n == 1 ? 16 : 8; }

// A launch that touches less than half the 256 MB last-level cache is over
// before its rows fight: it is bound by latency, and takes all the waves that
// fit (a local step's working set of 67 MB: round 83.4 us against 85.5 us).
// Local steps of 40 to 130 MB of loads, all waves against as many as beyond:
// SGD the same within 2% throughout; AdamW, contiguous, 14.2 and 14.9 us at 40
// MB, 31.2 and 31.5 us at 100 MB, 36.2 and 35.6 us at 115 MB (one worker a
// launch), 12.9 and 13.7, 30.5 and 30.7, 35.3 and 35.2 us (four workers).
constexpr int64_t kSmallBytes = int64_t(128) << 20;

// Strip groups of a launch, and the Rows its kernel finds them by.
int64_t groups_of(int64_t n_chunks, const RepLayout& rl) {
    return rl.groups() > 0 ? rl.groups() : n_chunks * (kStrips / kGroupStrips);
}
Rows rows_of(int64_t n_chunks, const RepLayout& rl, int map) {
    return Rows{map, rl.groups() > 0 ? static_cast<uint32_t>(n_chunks) : 0u};
}
dim3 strip_grid(int64_t n_chunks, const RepLayout& rl) {
    return dim3(static_cast<unsigned>(groups_of(n_chunks, rl) * kGroupStrips));
}
dim3 quad_grid(int64_t n_chunks, const RepLayout& rl) {
    return dim3(static_cast<unsigned>(groups_of(n_chunks, rl) * kGroupPieces));
}
// Grid of a local step: one row of strips x workers when the map interleaves
// the workers, else (strips or quads, workers).
dim3 local_grid(int64_t n_chunks, const RepLayout& rl, int n_workers, int map) {
    const unsigned n = static_cast<unsigned>(n_workers);
    const dim3 row = map & kQuads ? quad_grid(n_chunks, rl) : strip_grid(n_chunks, rl);
    return map & kInterleaveWorkers ? dim3(row.x * n) : dim3(row.x, n);
}

// Whether a launch over `streams` arenas is small.
bool small_launch(int64_t n_chunks, const RepLayout& rl, int streams) {
    return groups_of(n_chunks, rl) * streams * (4 * kGroupElems) <= kSmallBytes;
}
int waves_for(int64_t n_chunks, const RepLayout& rl, int streams, int waves) {
    return small_launch(n_chunks, rl, streams) ? kAllWaves : waves;
}

// Launches a kernel that touches `streams` arenas over every strip, at most
// `waves` waves per CU unless it is small, in the map's work-group shape.
template <typename K, typename... Args>
void launch_strips(K kernel, const Chunk* chunks, int64_t n_chunks, const RepLayout& rl, int map,
                   int streams, int waves, hipStream_t stream, Args... args) {
    const Rows rows = rows_of(n_chunks, rl, map);
    waves = waves_for(n_chunks, rl, streams, waves);
    if (map & kQuads)
        hipLaunchKernelGGL(kernel, quad_grid(n_chunks, rl), dim3(kBlockThreads), quad_lds(waves),
                           stream, chunks, rows, args...);
    else
        hipLaunchKernelGGL(kernel, strip_grid(n_chunks, rl), dim3(kWave), lds_for(waves), stream,
                           chunks, rows, args...);
}

}  // namespace

// ---------------------------------------------------------------- launchers

hipError_t launch_init(const Chunk* chunks, int64_t n_chunks, float* x, float* m, float* v,
                       float* x_rep, RepLayout rl, float* s1, float* s2, StateLayout ml, int n,
                       int map, hipStream_t st) {
    if (n_chunks == 0) return hipSuccess;
    launch_strips(k_init, chunks, n_chunks, rl, map, 3 * n + 2, init_waves(n), st, x, m, v, x_rep, rl,
                  s1, s2, ml, n);
    return hipGetLastError();
}

// Launches a local step's kernel, which loads `streams` arenas of each worker,
// over n_workers workers.
template <typename K, typename... Args>
static void launch_local(K kernel, const Chunk* chunks, int64_t n_chunks, const RepLayout& rl,
                         int map, int streams, int waves, int n_workers, hipStream_t st,
                         Args... args) {
    const bool small = small_launch(n_chunks, rl, streams * n_workers);
    // Small launches over sparse chunks are bound by the dispatch of their
    // work-groups and the search: four waves to a group (125 tensors of 64K
    // elements in all, n = 16: round 57 us against 66 us; 400 tensors of 3M,
    // n = 2, 80.5 us against 81.4 us; with full chunks it is the other way
    // round, 75.8 us against 74.4 us for 8 tensors of 128K, n = 4).
    if (small && rl.groups() > 0) map = kQuads;
    if (small) map &= ~kWideTurns;  // 2% of a round of 350K elements, n = 16
    const int group_waves = map & kQuads ? kQuadWaves : 1;
    hipLaunchKernelGGL(kernel, local_grid(n_chunks, rl, n_workers, map), dim3(group_waves * kWave),
                       lds_for(small ? kAllWaves : waves), st, chunks, rows_of(n_chunks, rl, map),
                       args...);
}

hipError_t launch_local_adamw(const Chunk* chunks, int64_t n_chunks, float* x_rep, RepLayout rl,
                              const float* x_src, RepLayout sl, const float* g_rep, float* s1,
                              float* s2, StateLayout ml, int worker0, int n_workers,
                              const AdamScalars& sc, int map, hipStream_t st) {
    if (n_chunks == 0) return hipSuccess;
    map = local_map(n_chunks, n_workers, map);
    launch_local(rl.cached() ? k_local_adamw<kCached> : k_local_adamw<kStream>, chunks, n_chunks, rl,
                 map, 4, kAdamWWaves, n_workers, st, x_rep, rl, x_src, sl, g_rep, s1, s2, ml,
                 worker0, n_workers, sc);
    return hipGetLastError();
}

hipError_t launch_local_sgdm(const Chunk* chunks, int64_t n_chunks, float* x_rep, RepLayout rl,
                             const float* x_src, RepLayout sl, const float* g_rep, float* s1,
                             StateLayout ml, int worker0, int n_workers, const SgdScalars& sc,
                             int map, hipStream_t st) {
    if (n_chunks == 0) return hipSuccess;
    map = local_map(n_chunks, n_workers, map);
    launch_local(rl.cached() ? k_local_sgdm<kCached> : k_local_sgdm<kStream>, chunks, n_chunks, rl,
                 map, 3, kSgdWaves, n_workers, st, x_rep, rl, x_src, sl, g_rep, s1, ml, worker0,
                 n_workers, sc);
    return hipGetLastError();
}

// Local step of every worker when every replica is stale (after a global step
// without broadcast): each worker starts from the global model.  The workers
// are interleaved, so that x is read from HBM once for all of them, or for as
// many as fit a row (12 workers of 1.45G elements, SGD: two launches of six take
// 44.2 ms, one launch with x read for each worker 54.0 ms).  One wave
// taking all n steps of a strip, with its 3 n + 1 streams at a time, ran at
// 66.1% (small, n = 8, state-blocked) and 67.5% (n = 4, contiguous) of 8 TB/s
// over the same bytes; this at 83.1% and 80%.
hipError_t launch_local_from_x(const Chunk* chunks, int64_t n_chunks, const float* x,
                               float* x_rep, RepLayout rl, const float* g_rep, float* s1,
                               float* s2, StateLayout ml, int n, bool adamw,
                               const AdamScalars& as, const SgdScalars& ss, int map,
                               hipStream_t st) {
    if (n_chunks == 0) return hipSuccess;
    const int per = workers_per_row(n_chunks, n, map);
    map = local_map(n_chunks, per, map);
    for (int w0 = 0; w0 < n; w0 += per) {
        const int nw = per < n - w0 ? per : n - w0;
        if (adamw)
            launch_local(rl.cached() ? k_local_adamw<kCached> : k_local_adamw<kShared>, chunks,
                         n_chunks, rl, map, 4, kAdamWSharedWaves, nw, st, x_rep, rl, x,
                         single_copy(), g_rep, s1, s2, ml, w0, nw, as);
        else
            launch_local(rl.cached() ? k_local_sgdm<kCached> : k_local_sgdm<kShared>, chunks,
                         n_chunks, rl, map, 3, kSgdSharedWaves, nw, st, x_rep, rl, x,
                         single_copy(), g_rep, s1, ml, w0, nw, ss);
    }
    return hipGetLastError();
}

// Work-groups of the round end per CU, by waves per work-group.  Many waves
// of a group wait for its last, so more waves are resident than in a local
// step, and fewer groups the larger they are.  AdamW: swept 2 to 24 at GPT-2
// small to xl; deterministic, one worker 77.4% with 10-12, 72% with 8, 74% with
// 14; the randomized one has one more, or two with one worker.  SGD loads fewer
// streams a wave and has little arithmetic: swept 4 to 32 at 8M to 400M elements
// of all workers, deterministic, both from x and from replicas; 25M, contiguous,
// from x, with AdamW's counts and with its own: one worker 125 and 117 us, two 92
// and 84 us, three 86 and 74 us, four 76 and 67 us, five 76 and 67 us; eight at
// 2.8G from replicas 8.4 and 7.8 ms with 4 and 5.  From eight waves a group on,
// the 32 waves that a CU holds are the limit, but not the LDS: waves that are
// done make room for the next group's while the first of theirs takes the global
// step.  16 waves again 4 (2.8G, contiguous, 8.0 ms, 8.2 ms with 5).
constexpr int round_end_groups(int waves, bool randomized, bool adamw) {
    if (!adamw) {
        constexpr int sgd[] = {16, 12, 10, 8, 6, 5, 5, 5};
        return waves <= 8 ? sgd[waves - 1] : randomized ? 5 : 4;
    }
    const int groups = waves == 1 ? 12 : waves == 2 ? 8 : waves == 3 ? 6 : waves == 4 ? 5 : 4;
    return groups + (randomized ? (waves == 1 ? 2 : 1) : 0);
}
constexpr bool round_end_groups_attainable() {
    for (int waves = 1; waves <= kMaxRoundEndWaves; ++waves)
        for (int which = 0; which < 4; ++which)
            if (!attainable(round_end_groups(waves, which & 1, which & 2))) return false;
    return true;
}
static_assert(round_end_groups_attainable(), "work-groups of the round end");

template <int BASE, int KIND, bool PIECE>
static void launch_round_end_shape(const Chunk* chunks, int64_t n_chunks, const RoundEndArgs& a,
                                   hipStream_t st) {
    constexpr int strips = PIECE ? kQuadWaves : 1;
    const dim3 grid = PIECE ? quad_grid(n_chunks, a.rl) : strip_grid(n_chunks, a.rl);
    constexpr bool adamw = BASE == kBaseAdamW;
    int workers = PIECE ? quad_strip_waves(a.gs.n, adamw) : strip_waves(a.gs.n, adamw);
    // A grid dimension holds fewer than 2^32 threads.
    while (static_cast<int64_t>(grid.x) * workers * strips * kWave >= (int64_t(1) << 32))
        workers /= 2;
    // Four strips of one worker are as many waves as four work-groups of one, and
    // held to 16 (AdamW) or 20 (SGD): 25M elements, state-blocked, randomized
    // round end from x with its second pass 207 and 180 us with all waves, 200
    // and 175 us; from replicas at 100M, contiguous, 867 and 723 us, 830 and 691
    // us.  With more workers the barriers hold them back enough.
    const int groups = waves_for(
        n_chunks, a.rl, 4 * a.gs.n + 2,
        !PIECE ? round_end_groups(workers, KIND == 2, adamw) : a.gs.n > 1 ? kAllWaves : adamw ? 4 : 5);
    const unsigned ends = static_cast<unsigned>(strips * a.gs.n * kWave * sizeof(f4));
    const unsigned lds = ends > lds_for(groups) ? ends : lds_for(groups);
    const auto kernel = a.rl.cached() ? k_round_end<BASE, KIND, PIECE, kCached>
                                    : k_round_end<BASE, KIND, PIECE, kStream>;
    hipLaunchKernelGGL(kernel, grid, dim3(workers * strips * kWave), lds, st, chunks,
                       rows_of(n_chunks, a.rl, 0), a.x, a.m, a.x_rep, a.rl, a.x_src, a.sl,
                       a.g_rep, a.s1, a.s2, a.u, a.bound.piece_max, a.ml, workers, a.as, a.ss,
                       a.gs);
}

template <int BASE, int KIND>
static void launch_round_end_kind(const Chunk* chunks, int64_t n_chunks, const RoundEndArgs& a,
                                  hipStream_t st) {
    if constexpr (KIND == 2) {
        // A word's four strips keep 4 n KiB of step-H values in LDS.
        if (takes_quads(groups_of(n_chunks, a.rl), a.gs.n, BASE == kBaseAdamW)) {
            launch_round_end_shape<BASE, KIND, true>(chunks, n_chunks, a, st);
            return;
        }
        const int64_t n4 = n_chunks * kSplit / 4;
        hipLaunchKernelGGL(k_clear_words,
                           dim3(static_cast<unsigned>((n4 + kBlockThreads - 1) / kBlockThreads)),
                           dim3(kBlockThreads), 0, st,
                           reinterpret_cast<uint4*>(a.bound.piece_max), n4);
    }
    launch_round_end_shape<BASE, KIND, false>(chunks, n_chunks, a, st);
}

template <int BASE>
static void launch_round_end_base(const Chunk* chunks, int64_t n_chunks, const RoundEndArgs& a,
                                  int kind, hipStream_t st) {
    if (kind == 0)
        launch_round_end_kind<BASE, 0>(chunks, n_chunks, a, st);
    else if (kind == 1)
        launch_round_end_kind<BASE, 1>(chunks, n_chunks, a, st);
    else
        launch_round_end_kind<BASE, 2>(chunks, n_chunks, a, st);
}

// Whether the second pass takes the tensor bounds itself.  Every wave then
// reads its tensor's words, through the L2: worth it for as long as that is
// less time than a launch, ~4.5 us.  At 14 MB of such reads a round of 2M
// elements takes 40.0 us against 42.1 us, at 31 MB the two are equal, at 66 MB
// the reads cost 2% of a 40 us round.
static bool fold_bound(int64_t n_chunks, const RepLayout& rl, const BoundWords& bw) {
    constexpr int64_t kMaxFoldBytes = int64_t(32) << 20;
    return groups_of(n_chunks, rl) * kGroupStrips * bw.max_words * 4 <= kMaxFoldBytes;
}

// The randomized sign after its first pass: level two of the tensor bound
// (also with no chunks at all, so that every bound is written) and the second
// pass.
static void launch_rand_rest(const Chunk* chunks, int64_t n_chunks, int n_tensors, float* x,
                             float* x_rep, const RepLayout& rl, const float* u,
                             const BoundWords& bw, const GlobalScalars& sc, bool broadcast, int map,
                             hipStream_t st) {
    const bool fold = n_chunks > 0 && fold_bound(n_chunks, rl, bw);
    if (n_tensors > 0 && !fold)
        hipLaunchKernelGGL(k_bound_reduce, dim3(static_cast<unsigned>(n_tensors)),
                           dim3(kReduceThreads), 0, st, chunks, bw.piece_max, bw.chunk0, bw.bits,
                           rl.groups() > 0);
    if (n_chunks == 0) return;
    const int stores = broadcast ? sc.n + 1 : 1;
#define DSM_PASS2(MODE, B, POLICY, FOLD)                                                        \
    launch_strips(k_global_rand_pass2<MODE, B, POLICY, FOLD>, chunks, n_chunks, rl, map,        \
                  stores + 1, pass2_waves(stores), st, x, x_rep, rl, u, bw, sc)
#define DSM_PASS2_POLICY(MODE, B)                                                               \
    do {                                                                                        \
        if (!fold && !rl.cached()) DSM_PASS2(MODE, B, kStream, false);                            \
        else if (!fold) DSM_PASS2(MODE, B, kCached, false);                                     \
        else if (!rl.cached()) DSM_PASS2(MODE, B, kStream, true);                                 \
        else DSM_PASS2(MODE, B, kCached, true);                                                 \
    } while (0)
    if (sc.mode == 1) {
        if (broadcast) DSM_PASS2_POLICY(1, true); else DSM_PASS2_POLICY(1, false);
    } else {
        if (broadcast) DSM_PASS2_POLICY(2, true); else DSM_PASS2_POLICY(2, false);
    }
#undef DSM_PASS2_POLICY
#undef DSM_PASS2
}

hipError_t launch_round_end(const Chunk* chunks, int64_t n_chunks, int n_tensors, bool adamw,
                            const RoundEndArgs& a, bool broadcast, hipStream_t st) {
    const bool randomized = a.gs.mode != 0;
    const int kind = randomized ? 2 : (broadcast ? 1 : 0);
    if (n_chunks > 0) {
        if (adamw)
            launch_round_end_base<kBaseAdamW>(chunks, n_chunks, a, kind, st);
        else
            launch_round_end_base<kBaseSgd>(chunks, n_chunks, a, kind, st);
    }
    if (randomized)
        launch_rand_rest(chunks, n_chunks, n_tensors, a.x, a.x_rep, a.rl, a.u, a.bound, a.gs,
                         broadcast, a.map_pass2, st);
    return hipGetLastError();
}

template <int RULE, bool BCAST>
static void launch_global_det_n(const Chunk* chunks, int64_t n_chunks, float* x, float* m,
                                float* v, float* x_rep, RepLayout rl, const GlobalScalars& sc,
                                int map, hipStream_t st) {
    if (rl.cached()) {
        launch_strips(k_global_det<0, RULE, BCAST, kCached>, chunks, n_chunks, rl, map, sc.n + 2,
                      global_waves(sc.n, BCAST), st, x, m, v, x_rep, rl, sc);
        return;
    }
#define DSM_GLOBAL_DET(NW)                                                                       \
    launch_strips(k_global_det<NW, RULE, BCAST, kStream>, chunks, n_chunks, rl, map, sc.n + 2,            \
                  global_waves(sc.n, BCAST), st, x, m, v, x_rep, rl, sc)
    switch (sc.n) {
        case 1: DSM_GLOBAL_DET(1); break;
        case 2: DSM_GLOBAL_DET(2); break;
        case 4: DSM_GLOBAL_DET(4); break;
        case 8: DSM_GLOBAL_DET(8); break;
        default: DSM_GLOBAL_DET(0); break;
    }
#undef DSM_GLOBAL_DET
}

template <int RULE>
static void launch_global_det_rule(const Chunk* chunks, int64_t n_chunks, float* x, float* m,
                                   float* v, float* x_rep, RepLayout rl, const GlobalScalars& sc,
                                   bool broadcast, int map, hipStream_t st) {
    if (broadcast)
        launch_global_det_n<RULE, true>(chunks, n_chunks, x, m, v, x_rep, rl, sc, map, st);
    else
        launch_global_det_n<RULE, false>(chunks, n_chunks, x, m, v, x_rep, rl, sc, map, st);
}

hipError_t launch_global_det(const Chunk* chunks, int64_t n_chunks, float* x, float* m,
                             float* v, float* x_rep, RepLayout rl, const GlobalScalars& sc,
                             bool broadcast, int map, hipStream_t st) {
    if (n_chunks == 0) return hipSuccess;
    switch (sc.rule) {
        case kRuleLookahead:
            launch_global_det_rule<kRuleLookahead>(chunks, n_chunks, x, m, v, x_rep, rl, sc,
                                                   broadcast, map, st);
            break;
        case kRuleSignedSlowMo:
            launch_global_det_rule<kRuleSignedSlowMo>(chunks, n_chunks, x, m, v, x_rep, rl, sc,
                                                      broadcast, map, st);
            break;
        case kRuleGlobalAdamW:
            launch_global_det_rule<kRuleGlobalAdamW>(chunks, n_chunks, x, m, v, x_rep, rl, sc,
                                                     broadcast, map, st);
            break;
        default:
            launch_global_det_rule<kRuleSignMomentum>(chunks, n_chunks, x, m, v, x_rep, rl, sc,
                                                      broadcast, map, st);
            break;
    }
    return hipGetLastError();
}

hipError_t launch_global_rand(const Chunk* chunks, int64_t n_chunks, int n_tensors, float* x,
                              float* m, float* x_rep, RepLayout rl, float* u,
                              const BoundWords& bw, const GlobalScalars& sc, bool broadcast,
                              int map, hipStream_t st) {
    if (n_chunks > 0) {
#define DSM_PASS1(NW, POLICY)                                                                    \
    launch_strips(k_global_rand_pass1<NW, POLICY>, chunks, n_chunks, rl, kQuads, sc.n + 3,       \
                  pass1_waves(sc.n), st, x, m, x_rep, rl, u, bw.piece_max, sc)
        if (rl.cached())
            DSM_PASS1(0, kCached);
        else switch (sc.n) {
            case 1: DSM_PASS1(1, kStream); break;
            case 2: DSM_PASS1(2, kStream); break;
            case 4: DSM_PASS1(4, kStream); break;
            case 8: DSM_PASS1(8, kStream); break;
            default: DSM_PASS1(0, kStream); break;
        }
#undef DSM_PASS1
    }
    launch_rand_rest(chunks, n_chunks, n_tensors, x, x_rep, rl, u, bw, sc, broadcast, map, st);
    return hipGetLastError();
}

hipError_t launch_broadcast(const Chunk* chunks, int64_t n_chunks, const float* x, float* x_rep,
                            RepLayout rl, int n, int map, hipStream_t st) {
    if (n_chunks == 0) return hipSuccess;
    launch_strips(rl.cached() ? k_broadcast<kCached> : k_broadcast<kStream>, chunks, n_chunks, rl,
                  map, n + 1, copy_waves(n), st, x, x_rep, rl, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------- static scratch

// Workspace and u staging of the contexts made by dsm_init_static, for
// callers that cannot allocate device memory.  Host code never passes this
// name to a kernel: it stands for a device address only through
// hipGetSymbolAddress, below.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

hipError_t static_scratch(void** ptr) {
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (addr[dev] == nullptr) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

hipError_t launch_test_stream(int kind, float* buf, int64_t n_pieces, uint32_t* words,
                              uint32_t pattern, hipStream_t st) {
    if (n_pieces == 0) return hipSuccess;
    const dim3 grid(static_cast<unsigned>(n_pieces)), block(kBlockThreads);
    if (kind == 0)
        hipLaunchKernelGGL(k_stream_read, grid, block, 0, st, buf, words, pattern);
    else
        hipLaunchKernelGGL(k_stream_write, grid, block, 0, st, buf, pattern);
    return hipGetLastError();
}

hipError_t launch_test_philox(uint32_t key0, uint32_t key1, uint32_t tensor, uint32_t t,
                              uint32_t q0, int64_t count, uint32_t* out, hipStream_t st) {
    if (count == 0) return hipSuccess;
    const int64_t blocks = (count + kBlockThreads - 1) / kBlockThreads;
    hipLaunchKernelGGL(k_test_philox, dim3(static_cast<unsigned>(blocks)), dim3(kBlockThreads), 0,
                       st, key0, key1, tensor, t, q0, count, out);
    return hipGetLastError();
}

}  // namespace dsm
