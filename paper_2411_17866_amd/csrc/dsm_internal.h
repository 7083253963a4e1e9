// Internal interface between the host runtime (dsm_runtime.cpp) and the
// gfx950 kernels (dsm_kernels.hip).  Not part of the public C ABI.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

namespace dsm {

// Elements per chunk.  A chunk never crosses a tensor boundary, so the
// per-tensor facts a kernel needs (decay flag, tensor index for the randomized
// sign's bound and Philox counter) are uniform per wave and read once.
constexpr int kChunkElems = 16384;
// A wave takes one strip of a chunk per stream: 64 lanes x one float4.  Eight
// strips, one per XCD, are a strip group.
constexpr int kWave = 64;
constexpr int kAllWaves = 32;  // waves a CU holds
constexpr int kXcds = 8;       // MI355X: work-groups go to its 8 XCDs round-robin
constexpr int kStripVec = kWave;
constexpr int kStrips = kChunkElems / 4 / kStripVec;  // strips per chunk
constexpr int kGroupStrips = kXcds;
constexpr int kGroupElems = 4 * kStripVec * kGroupStrips;
static_assert(kChunkElems % kGroupElems == 0, "a chunk must split into whole strip groups");
// Work-groups of four waves (quads), and the 1024-element pieces of a chunk.
// The randomized sign's bound has as many words as a chunk has pieces, one for
// each four strips.
constexpr int kQuadWaves = 4;
constexpr int kBlockThreads = kQuadWaves * kWave;
constexpr int kPieceVec = kBlockThreads;
constexpr int kSplit = kChunkElems / 4 / kPieceVec;  // pieces per chunk
constexpr int kGroupPieces = kGroupStrips / kQuadWaves;
static_assert(kSplit % kXcds == 0, "the strips of a quad must lie in one chunk");
// Most waves of a work-group of the fused round end (more workers share them).
constexpr int kMaxRoundEndWaves = 16;
// Waves for n workers where at most `most` fit: no more than it takes for the
// same number of turns, so that the last turn is as full as can be.
constexpr int even_waves(int n, int most) {
    const int turns = (n + most - 1) / most;
    return (n + turns - 1) / turns;
}
// Waves a strip of the round end that takes four strips in a work-group.  SGD:
// 4.  AdamW's waves take longer and less evenly, and a barrier over 16 of them
// waits longer than more turns of 12 do: 25M elements of all workers,
// contiguous, randomized round end with its second pass, 4 workers 152 us with
// 16 waves, 122 us with 8; 7 workers 136 us, 116 us with 12; 8 workers 122 us,
// 112 us.  Past 15 workers 3 waves would take six turns against four, and 3M
// elements of 16 workers 19.7 us against 19.2 us (state-blocked 20.1 and 18.2
// us).  Even turns: 5 AdamW workers 169 us with 4 waves of which one takes two,
// 120 us with 3; 9 SGD workers 79 us and 76 us.
constexpr int quad_strip_waves(int n, bool adamw) {
    return even_waves(n, adamw && n < kMaxRoundEndWaves ? 3 : 4);
}
// Whether the randomized round end over so many strip groups takes the four
// strips of a bound word in a work-group, or clears the words (a launch of its
// own, ~4 us) and raises them by atomic maxima, one strip per work-group.  The
// round end from replicas with its second pass, one strip and four, us, at 8M,
// 32M, 128M and 400M elements of all workers:
//   SGD,   2 workers, contiguous    50  44 | 161 150 | 591 578 | 1819 1843
//   SGD,   8 workers, contiguous    35  32 | 110 110 | 411 415 | 1244 1315
//   SGD,   8 workers, state-blocked 35  33 | 105 110 | 377 404 | 1165 1251
//   AdamW, 2 workers, contiguous    61  57 | 206 198 | 774 756 | 2373 2398
//   AdamW, 8 workers, contiguous    50  45 | 162 158 | 614 610 | 1870 1922
//   AdamW, 8 workers, state-blocked 51  46 | 162 157 | 585 581 | 1802 1796
// The sides cross from 16M (SGD, state-blocked, five workers and more: up to 8%
// from there on) to beyond 400M; the line is at 134M, 65536 strip groups times
// workers.  SGD with three waves a strip (12 in a work-group, of which a CU
// holds two and 8 waves stay idle) crosses at 16M: three workers, contiguous,
// 45 45 | 137 148 | 499 571, five, state-blocked, 38 38 | 114 122 | 424 442, six
// 37 35 | 111 115 | 407 422.  So does AdamW with 10 workers and more, whose
// three waves a strip then take four turns and more: 14 workers at 16M, 24M, 64M
// and 130M, contiguous, 84 84 | 119 123 | 293 308 | 581 621, state-blocked 84 84 |
// 112 122 | 277 301 | 547 596.
constexpr bool takes_quads(int64_t groups, int n, bool adamw) {
    const bool crosses_early = adamw ? n >= 10 : n == 3 || n == 5 || n == 6;
    return n <= kMaxRoundEndWaves && groups * n < (crosses_early ? 8192 : 65536);
}
// Waves of the round end that takes one strip in a work-group.  SGD: 16; AdamW:
// 8 (16 workers of 30M parameters: AdamW 65.3% (contiguous) and 72.6%
// (state-blocked) of 8 TB/s with 16 waves, 68.0% and 75.4% with 8; SGD 73.9% and
// 83.8% with 16, 70.0% and 78.9% with 8).  Where a second turn would leave three
// quarters of them or more idle, even turns: deterministic, 25M elements of all
// workers, contiguous, SGD with 17 workers 69.2 us with 16 waves, 62.7 us with 9;
// with 20 workers 64.1 and 61.2 us; AdamW with 9 workers 104 us with 8 waves, 100
// us with 5.  Beyond, all waves: SGD with 24 workers 59.0 us with 16, 59.6 us
// with 12 (state-blocked 55.8 and 58.6 us).
constexpr int strip_waves(int n, bool adamw) {
    const int most = adamw ? kMaxRoundEndWaves / 2 : kMaxRoundEndWaves;
    return n <= most + most / 4 ? even_waves(n, most) : most;
}
// Arena alignment of every tensor, in elements (256 bytes).
constexpr int64_t kTensorAlign = 64;
constexpr int kMaxWorkers = 64;

// Replica buffers in 64 KiB blocks (dsm_problem.replica_layout =
// DSM_REPLICAS_BLOCKED): copy i of block b sits at element (b * n + i) *
// kRepBlockElems.  Tensors then start on a multiple of the piece size (and of
// 1024 elements), so a wave's strip never crosses a block, and the
// arena length is a whole number of blocks.
constexpr int kRepBlockShift = 14;
constexpr int64_t kRepBlockElems = int64_t(1) << kRepBlockShift;
constexpr int64_t kPieceElems = int64_t(kPieceVec) * 4;
static_assert(kRepBlockElems % kPieceElems == 0, "a block must hold whole pieces");
constexpr int64_t kBlockedTensorAlign = kPieceElems > 1024 ? kPieceElems : 1024;

// Where copy i of a replica buffer keeps arena element e:
// (e >> shift) * block_stride + i * copy_stride + (e & (2^shift - 1)).
struct RepLayout {
    int64_t block_stride;
    int64_t copy_stride;
    int32_t shift;
    // Of the problem, not of the buffer, set by problem_facts().  groups: 0, or
    // where most strip groups of its chunks hold no elements (many tensors far
    // shorter than a chunk), the number of those that do; its launches then go
    // over these only.  cached: its arenas are small enough to stay in the
    // caches between calls.
    uint32_t facts;
    int64_t groups() const { return facts & 0x7fffffffu; }
    bool cached() const { return facts >> 31 != 0; }
};
// Sparse from half the groups empty on.  A wave of a sparse launch searches for
// its chunk, ~1 us; the waves it saves cost their dispatch (125 tensors of 64K
// elements in all, n = 16, 25 times as many empty groups as full ones: a fused
// round takes 72 us, 142 us before; 400 tensors, 43% of the groups hold
// elements: 81 us, 86 us before).
constexpr bool sparse_chunks(int64_t groups, int64_t n_chunks) {
    return 2 * groups <= n_chunks * (kStrips / kGroupStrips);
}
// Three eighths of the 256 MB last-level cache: problems of 106 MB taking turns
// already lose 2% to plain accesses.
constexpr int64_t kCachedBytes = int64_t(96) << 20;
// RepLayout::facts of a problem with `groups` strip groups that hold elements,
// n_chunks chunks and `bytes` of arenas.
constexpr uint32_t problem_facts(int64_t groups, int64_t n_chunks, int64_t bytes) {
    return (sparse_chunks(groups, n_chunks) ? static_cast<uint32_t>(groups) : 0u) |
           (bytes <= kCachedBytes ? 0x80000000u : 0u);
}
// n contiguous copies of d_pad elements.
inline RepLayout contiguous_copies(int64_t d_pad) { return RepLayout{0, d_pad, 62, 0}; }
// n copies interleaved in 64 KiB blocks.
inline RepLayout blocked_copies(int n) {
    return RepLayout{int64_t(n) * kRepBlockElems, kRepBlockElems, kRepBlockShift, 0};
}
// Every copy is the same single buffer (stale replicas read the global x).
inline RepLayout single_copy() { return RepLayout{0, 0, 62, 0}; }

// The replicas and their state in one allocation (dsm_problem.replica_layout =
// DSM_REPLICAS_STATE_BLOCKED): 16 KiB blocks, and block b holds the n x_rep
// copies, then the n g_rep copies, the n s1_rep copies and (AdamW) the n
// s2_rep copies of elements [4096 b, 4096 b + 4096).  Buffer j of the
// kStateBuffers starts j * n blocks into the allocation.
constexpr int kStateBlockShift = 12;
constexpr int64_t kStateBlockElems = int64_t(1) << kStateBlockShift;
static_assert(kStateBlockElems % kPieceElems == 0, "a state block must hold whole pieces");
inline RepLayout state_blocked_copies(int n, int buffers) {
    return RepLayout{int64_t(buffers) * n * kStateBlockElems, kStateBlockElems, kStateBlockShift,
                     0};
}

// Where the gradient and the base-optimizer moments of worker i keep their
// elements (the same RepLayout addressing as the replicas).
struct StateLayout {
    RepLayout g, s1, s2;
};

// One chunk of one tensor inside an arena copy.  32 bytes.
struct Chunk {
    int64_t off;      // element offset of the chunk in the arena
    int64_t j0;       // index of the chunk's first element inside its tensor
    int32_t len;      // elements in the chunk, 1..kChunkElems
    uint32_t tensor;  // tensor index p
    uint32_t decay;   // 1 if weight decay applies to the tensor
    uint32_t group0;  // strip groups of the chunks before this one that hold elements
};
static_assert(sizeof(Chunk) == 32, "chunk descriptor is 32 bytes");

// One level of the search for the chunk that holds a strip group, over the
// ascending Chunk.group0: a wave's 64 lanes probe the range at equal steps, and
// the number of lanes that find a group0 at or below the group (a prefix with
// lane 0 in it) narrows the range to one step.
struct ChunkRange {
    uint32_t lo, size;
};
constexpr uint32_t probe_step(const ChunkRange& r) { return (r.size + kWave - 1) / kWave; }
// Offset into the range that a lane probes; past the range when not below size.
constexpr uint32_t probe_of(const ChunkRange& r, uint32_t lane) { return lane * probe_step(r); }
constexpr ChunkRange narrowed(const ChunkRange& r, uint32_t below) {
    const uint32_t step = probe_step(r), skip = (below - 1) * step;
    return ChunkRange{r.lo + skip, step < r.size - skip ? step : r.size - skip};
}

// fp32 coefficients of one AdamW local step, formed on the host in fp64 and
// rounded once.
struct AdamScalars {
    float beta1, one_minus_beta1, beta2, one_minus_beta2;
    float bc1, bc2;   // 1 - beta1^s, 1 - beta2^s
    float lr, eps, wd;
};

struct SgdScalars {
    float mu, lr;
};

// fp32 coefficients of one global step.
struct GlobalScalars {
    float beta1, beta2;
    float c1, c2;      // (1 - beta1)/gamma, (1 - beta2)/gamma
    float step;        // eta * gamma
    float lam;         // lambda (decayed tensors)
    float inv_n;       // 1/n, used only when n is a power of two (then exact)
    float n_f;         // n as float
    int32_t n;
    int32_t n_pow2;    // 1 if n is a power of two
    uint32_t key0, key1;  // Philox key (seed low, seed high)
    uint32_t t;           // outer iteration (Philox counter word 2)
    int32_t mode;         // dsm_sign
    int32_t rule;         // dsm_global_rule
    // Global AdamW (Algorithm 7) only.
    float inv_gamma;      // 1/gamma
    float one_minus_beta1, one_minus_beta2;
    float bc1, bc2;       // 1 - beta^(t+1)
    float eta, eps;
};

// How a launch goes over the strips (its map), by kernel kind and replica
// layout.
// Without flags, one-wave work-groups take the strips in order.
//
// kInterleaveWorkers (local steps): the grid is one row of strips x workers in
// which a strip group of one worker is followed by the same group of the next.
// With the state blocked, consecutive work-groups then sweep whole blocks (xl,
// n = 4: 85.4% of 8 TB/s; a strip instead of a group at a time 83.2%).  For the
// step from x (from_x), in every layout, it also brings the n reads of an x
// line together.
//
// kWideTurns (with kInterleaveWorkers): turns of 1024 strip groups, 8 MiB per
// stream.  Where the workers' buffers lie far apart, one group at a time has
// the streams of all n workers open at once; in wide turns the step from x has
// one worker's, as the other local steps do, and finds x in the last-level
// cache: six workers, 51M, contiguous 80.5% of 8 TB/s against 76.8%; small,
// n = 4, 80.1% against 78.6%; large, n = 2, blocked, 81.4% against 80.1%.
// Turns of 256 groups 79.8, 80.1 and 80.0%; of 4096 70.7% where 1024 has 76.3%
// (8.5M, n = 4).  With the state blocked one group at a time is ahead (82.7%
// against 81.6% and less).
//
// kQuads (the other kinds): work-groups of four waves.  Ahead where a kernel
// writes every replica from blocks (global step, state-blocked, n = 8: 79.2%
// against 78.4%; sync 82-88% in all layouts, 79-81% with one wave), behind
// elsewhere (global step, contiguous, n = 4: 78.0% against 78.7%).
// global: the global steps and the randomized second pass of the round end;
// copy: the broadcast of dsm_sync and the initial copy of dsm_init.  The round
// end has shapes of its own.
constexpr int kInterleaveWorkers = 4;
constexpr int kQuads = 8;
constexpr int kWideTurns = 16;
constexpr uint32_t kTurnGroups = 1024;
struct LaunchMaps {
    int local, from_x, global, copy;
};
constexpr LaunchMaps kMapsByLayout[3] = {
    {0, kInterleaveWorkers | kWideTurns, 0, kQuads},            // contiguous
    {0, kInterleaveWorkers | kWideTurns, 0, kQuads},            // blocked
    {kInterleaveWorkers, kInterleaveWorkers, kQuads, kQuads}};  // state-blocked

// How a kernel finds its strips: the launch map, and the number of chunks when
// it goes over the strip groups that hold elements (RepLayout::groups()), else 0.
struct Rows {
    int32_t map;
    uint32_t sparse_chunks;
};

// The map a local step over n_workers workers launches with: the interleaved
// order needs the whole pieces x workers row in one grid dimension, which
// holds fewer than 2^32 threads; past that the step runs worker by worker.
inline int local_map(int64_t n_chunks, int n_workers, int map) {
    const int64_t row = n_chunks * kSplit * n_workers;
    if ((map & kInterleaveWorkers) && row * kBlockThreads >= (int64_t(1) << 32))
        return map & ~kInterleaveWorkers;
    return map;
}

// The workers that one launch of the step from x takes: all n, or where their
// row is too long for the map, a half, a quarter and so on of them.
inline int workers_per_row(int64_t n_chunks, int n, int map) {
    int per = n;
    while (per > 1 && local_map(n_chunks, per, map) != map) per = (per + 1) / 2;
    return per;
}

// Kernel launchers (dsm_kernels.hip).  All return the launch status.  The
// replica buffer x_rep is addressed through its RepLayout rl, and g_rep, s1
// and s2 through the layouts of ml; map is the launch's map.
hipError_t launch_init(const Chunk* chunks, int64_t n_chunks, float* x, float* m, float* v,
                       float* x_rep, RepLayout rl, float* s1, float* s2, StateLayout ml, int n,
                       int map, hipStream_t st);
// Local steps: worker w reads its starting point from x_src through sl (its
// replica, or the shared global model with single_copy()) and writes its
// replica through rl.
hipError_t launch_local_adamw(const Chunk* chunks, int64_t n_chunks, float* x_rep, RepLayout rl,
                              const float* x_src, RepLayout sl, const float* g_rep, float* s1,
                              float* s2, StateLayout ml, int worker0, int n_workers,
                              const AdamScalars& sc, int map, hipStream_t st);
hipError_t launch_local_sgdm(const Chunk* chunks, int64_t n_chunks, float* x_rep, RepLayout rl,
                             const float* x_src, RepLayout sl, const float* g_rep, float* s1,
                             StateLayout ml, int worker0, int n_workers, const SgdScalars& sc,
                             int map, hipStream_t st);

// Local step of all n workers from the global model x (every replica stale):
// x is read once per element and each worker's result goes to its replica.
hipError_t launch_local_from_x(const Chunk* chunks, int64_t n_chunks, const float* x,
                               float* x_rep, RepLayout rl, const float* g_rep, float* s1,
                               float* s2, StateLayout ml, int n, bool adamw,
                               const AdamScalars& as, const SgdScalars& ss, int map,
                               hipStream_t st);

// Workspace words of the randomized sign's per-tensor bound B_p = max |u|,
// reduced in two levels.  A level-one word is the largest |u| of four strips of
// one chunk: stored by the work-group that takes the four (strips 8 apart, or
// four in a row over sparse chunks), or raised by atomic maxima of the four
// strips of a 1024-element piece (a large round end).  Which four share a word
// does not matter: level two takes all words of a tensor.
struct BoundWords {
    uint32_t* bits;         // [n_tensors] B_p, fp32 bit patterns
    uint32_t* piece_max;    // [n_chunks * kSplit] level one: max |u| of four strips each
    const int32_t* chunk0;  // [n_tensors + 1] first chunk of each tensor; last = n_chunks
    int64_t max_words;      // most level-one words of a tensor
};

// Arguments of the fused last-local-step + global-step launch.
struct RoundEndArgs {
    float *x, *m, *x_rep;
    RepLayout rl;           // the replicas
    const float* x_src;     // where step H starts: the replicas, or x when they are stale
    RepLayout sl;
    const float* g_rep;
    float *s1, *s2, *u;
    BoundWords bound;
    StateLayout ml;
    AdamScalars as;
    SgdScalars ss;
    GlobalScalars gs;
    int map_pass2;  // launch map of the randomized sign's second pass
};
hipError_t launch_round_end(const Chunk* chunks, int64_t n_chunks, int n_tensors, bool adamw,
                            const RoundEndArgs& a, bool broadcast, hipStream_t st);
// Deterministic global step of any rule; v is the Global AdamW second moment.
hipError_t launch_global_det(const Chunk* chunks, int64_t n_chunks, float* x, float* m,
                             float* v, float* x_rep, RepLayout rl, const GlobalScalars& sc,
                             bool broadcast, int map, hipStream_t st);
hipError_t launch_global_rand(const Chunk* chunks, int64_t n_chunks, int n_tensors, float* x,
                              float* m, float* x_rep, RepLayout rl, float* u,
                              const BoundWords& bw, const GlobalScalars& sc, bool broadcast,
                              int map, hipStream_t st);
hipError_t launch_broadcast(const Chunk* chunks, int64_t n_chunks, const float* x, float* x_rep,
                            RepLayout rl, int n, int map, hipStream_t st);
// Streaming diagnostic over n_pieces pieces of kPieceElems floats: kind 0
// reads buf and writes 1 to words[k] for each piece k whose 32-bit patterns
// XOR to pattern; kind 1 writes the float with bit pattern `pattern`.
hipError_t launch_test_stream(int kind, float* buf, int64_t n_pieces, uint32_t* words,
                              uint32_t pattern, hipStream_t st);
hipError_t launch_test_philox(uint32_t key0, uint32_t key1, uint32_t tensor, uint32_t t,
                              uint32_t q0, int64_t count, uint32_t* out, hipStream_t st);

// The static device scratch of dsm_init_static: a file-scope array of
// kStaticScratchBytes in dsm_kernels.hip, one copy per GPU.
constexpr int64_t kStaticScratchBytes = int64_t(64) << 20;
constexpr int kMaxDevices = 64;
// Device address of the scratch on the current device, looked up once per
// device (hipGetSymbolAddress) and kept.
hipError_t static_scratch(void** ptr);

}  // namespace dsm
