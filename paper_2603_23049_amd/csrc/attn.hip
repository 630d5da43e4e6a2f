// Paged prefix-reuse prefill attention for gfx950 (bf16 in, fp32 accumulate, bf16 out).
//
// For sequence b with p cached and s new tokens, query head h and suffix row i
// (absolute position p+i): out = softmax_j(sm_scale <q, k_j>) v_j over keys
// j = 0 .. p+i, with K/V read from the paged pool through the block table
// (exact prefix reuse, Sec. 2.2; paged blocks, Sec. 5).
//
// Work decomposition. The s*G query rows of one (sequence, kv head) pair,
// G = Hq/Hkv, are packed token-major (row r = token r/G, head-in-group r%G)
// so that all rows of a workgroup share one K/V stream. A workgroup has 8 waves in
// two groups (waves 0-3 and 4-7, 32 rows per wave), so each SIMD runs one wave of
// each group: one wave's softmax overlaps the other's matrix work. Three schedules:
//   key halves: the workgroup takes 128 packed rows; both groups hold the same rows
//     and walk the two halves of the key range, merged through LDS at the end;
//   row halves: the workgroup takes 256 packed rows, 128 per group, and both groups
//     walk the whole key range, group 1 one phase behind, through one copy of each
//     tile that group 0 loads; no merge;
//   key split: key halves with each row tile's keys cut into chunks, one workgroup each,
//     whose partial results (O, max, sum) a second kernel merges; for launches that
//     leave compute units idle.
// Row halves give each workgroup twice the work for one start-up and no merge; the
// host takes them when they are estimated to be faster (schedule_time).
//
// Per wave and 64-key tile (4 pool blocks), with v_mfma_f32_32x32x16_bf16:
//   S^T[key][q] = K Q^T   A = K rows from LDS, B = this wave's Q (registers)
//   O^T[d][q]  += V^T P^T A = V^T from LDS,  B = P (registers)
// Each lane holds one query column q = lane%32 of both accumulators, so the
// online softmax is in-lane; the two half-waves holding the same query trade
// only their tile max (one shuffle) and their partial sums at the end. K rows
// are fed to the first product in a permuted key order chosen so that the S^T
// accumulator registers of a lane are, in order, the P^T operand registers of
// the second product. V is stored d-major inside each pool block, so a V^T
// operand (8 consecutive keys of one dim) is one 16-byte LDS read.
//
// Softmax runs in the log2 domain. The first product of a tile starts from
// -m_ref, so the raw scores <q, k> come out already shifted, and one fp32
// multiply by c = sm_scale * log2(e) precedes each exp2. (Folding c into Q
// instead would round q*c to bf16: a relative error of 2^-9 on every score,
// which for sharp rows of large |<q, k>| moves the output by far more than the
// bf16 inputs themselves do.) The reference max m_ref is only raised (and O
// rescaled) when a tile's scaled max exceeds it by more than 8, i.e. a factor
// of 2^8; otherwise the stale value stays, which keeps probabilities below 256
// and skips the rescale of 64 accumulators per lane.
//
// Tiles move global -> LDS with global_load_lds_dwordx4 (no staging
// registers), double-buffered with one barrier per tile. LDS chunks are
// XOR-swizzled so that lanes reading 32 different key rows (K) or dims (V)
// hit distinct banks; the swizzle is applied through the source address of
// each lane, since a direct load writes lane l's 16 bytes at base + 16*l.
#include <algorithm>
#include <atomic>
#include <mutex>
#include <type_traits>
#include <vector>

#include "decode_wave.h"
#include "pcr_internal.h"

namespace pcr {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16;

constexpr int kGroupWaves = 4;
constexpr int kRowsPerWave = 32;
constexpr int kRowsPerWG = kGroupWaves * kRowsPerWave;   // 128 rows (key halves: both groups)
constexpr int kThreads = 2 * kGroupWaves * 64;           // 512
constexpr int kTileKeys = 64;
constexpr int kTileBlocks = kTileKeys / kBlockSize;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kRescaleThreshold = 8.0f;                // log2 units: P <= 2^8
// LDS fragment reads kept in flight ahead of the MFMAs in the matrix cluster. With the
// shared row-halves tiles 3 and 4 measured 0.4-0.8% faster than 5 and 1-2% faster than 6
// or 7 on the 70B and RAG-mix shapes: the reads are bound by the LDS's throughput, not
// its latency.
#ifndef KAHEAD
#define KAHEAD 4
#endif
constexpr int kXcds = 8;                                 // MI355X: 8 XCDs, workgroups dealt round-robin

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// Key (within a 32-key half tile) whose K row is fed as A-operand row i of the
// first product. With this order, accumulator register r of lane (q, half)
// holds key 16*(r/8) + 8*half + r%8 of the half tile, i.e. registers 8t..8t+7
// are the 8 keys P^T needs in the second product's k-step t.
__device__ __forceinline__ constexpr int key_of_row(int i)
{
    return 16 * (i >> 4) + 8 * ((i >> 2) & 1) + 4 * ((i >> 3) & 1) + (i & 3);
}

// LDS chunk swizzle of a K tile row (chunks of 16 B; CPR chunks per row).
template <int CPR>
__device__ __forceinline__ constexpr int k_swizzle(int key) { return key % CPR; }

template <int D>
struct TileGeom {
    static constexpr int CPR = D / 8;                          // 16-B chunks per K row
    static constexpr int KBYTES = kTileKeys * D * 2;           // K tile bytes
    static constexpr int VBYTES = kTileKeys * D * 2;           // V tile bytes
    static constexpr int KLOADS = KBYTES / 1024 / kGroupWaves; // 1 KB direct loads per thread, K tile
    static constexpr int VLOADS = VBYTES / 1024 / kGroupWaves; // same, V tile
};

__device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// s_waitcnt immediate that waits for LDS, scalar-memory and message counters only
// (lgkmcnt = 0; vmcnt and expcnt at their maxima, so they do not wait).
constexpr int kWaitLgkm0 = 0xC07F;

// Workgroup barrier without a memory fence. The phase schedule orders its memory
// traffic explicitly: every direct load is waited for (vmcnt) by the wave that
// issued it before the barrier that precedes its first reader, and every LDS read
// is consumed before its wave reaches the next barrier. The empty asm statements
// keep the compiler from moving memory operations across the barrier.
__device__ __forceinline__ void phase_barrier()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// One wave-wide direct load global -> LDS: lane l's 16 bytes at src land at
// lds_dst + 16*l (lds_dst wave-uniform). Issued as inline assembly because the
// compiler counts a global-to-LDS load as a pending LDS access of unknown order and
// then drains every outstanding LDS read (lgkmcnt(0)) at the next operand wait,
// which would empty the fragment pipeline after each load. The hardware signals
// completion of these loads on vmcnt only; the kernel waits for them explicitly
// before the barrier that precedes their first reader.
// The source is a wave-uniform base (SGPR pair) plus a 32-bit per-lane byte offset.
// lds_dst is an LDS byte address (M0 form). M0 is a register the compiler reserves:
// it does not honour the clobber, and relies on M0 only for instructions that read
// it, of which this file has none besides these loads (each sets it first).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma16(const char *base, uint32_t lane_off, uint32_t lds_dst)
{
    const unsigned m0 = __builtin_amdgcn_readfirstlane(lds_dst);
    // The base is wave-uniform; reading it through readfirstlane states that to the
    // register allocator (free when it already sits in SGPRs), which otherwise may keep
    // it in VGPRs under SGPR pressure and then cannot meet the "s" constraint.
    // (readfirstlane returns int: each half goes through uint32_t before widening, or a
    // low word with bit 31 set would sign-extend into the high half of the address)
    const uint64_t b64 = reinterpret_cast<uint64_t>(base);
    const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b64 >> 32));
    const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b64);
    const uint64_t sb = (hi << 32) | lo;
    asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_off),
                 "s"(reinterpret_cast<const char *>(sb)), "s"(m0)
                 : "memory", "m0");
}
// The same with a full address per lane.
__device__ __forceinline__ void dma16_at(const char *src, uint32_t lds_dst)
{
    const unsigned m0 = __builtin_amdgcn_readfirstlane(lds_dst);
    asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(m0) : "memory", "m0");
}
#pragma clang diagnostic pop

// Wait until at most N vector-memory operations of this wave are outstanding
// (the N most recent may still be in flight).
template <int N>
__device__ __forceinline__ void wait_vmem_keep()
{
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Order of one launch's work items (row tile of a sequence, kv head), built on the
// host from the sequence lengths and passed by value in the kernel arguments.
// Sequences are taken heaviest first (longest key range), and inside a sequence the
// last row tiles (the most keys) first, so the long items start early and the
// short ones fill the tail. Each slot also carries its sequence's lengths, so a
// workgroup finds everything it needs about its sequence in one parallel read of
// the map (the kernel arguments) instead of a chain of dependent loads.
constexpr int kMaxMapSeqs = 128;
struct AttnWorkMap {
    int32_t n_seq;                      // slots in use (sequences with new tokens)
    int32_t per_head;                   // work items of all sequences, one kv head
    int32_t chunk;                      // key split: 64-key tiles per item (else unused)
    uint64_t launch;                    // key split: the launch's number (else unused)
    int32_t seq[kMaxMapSeqs];           // sequence in each slot
    int32_t tiles_end[kMaxMapSeqs];     // items of the slots up to and including this one
    int32_t prefix[kMaxMapSeqs];        // the slot's cached tokens p
    int32_t first[kMaxMapSeqs];         // the slot's first new token (row of q and out)
    int32_t count[kMaxMapSeqs];         // the slot's new tokens s
};

// How a launch divides its work among workgroups (see the head of this file).
enum AttnMode { kKeyHalves = 0, kRowHalves = 1, kKeySplit = 2 };

// Scratch of key-split launches: kSplitSlots slots of kSplitParts partial results per
// device, held until the process ends. A launch owns one slot from its claim kernel until
// every workgroup of its combine kernel has counted itself out. The slot's owner word
// holds the launch's number, which the host gives every enqueued launch: the workgroups
// find their slot by looking for it, and which one it is is not fixed on the host
// (launches on any streams and threads, and replays of captured graphs, claim theirs when
// they run). The number and not the output pointer names the launch, since calls that
// overlap may share an output (equal calls on two streams, say). With every slot taken a
// launch runs unsplit.
// Replays of one captured launch have one number, and HIP lets them overlap. They take
// turns to claim (replay_lock), and one that finds its number in use joins: both write the
// same partial results, and the entry is free when both are through. One that finds no
// slot takes one of the entries past the slots, which have no scratch, so that a replay
// that starts beside it runs unsplit too.
constexpr int kSplitSlots = 8;
constexpr int kSplitEntries = 64;                        // the slots, then entries without scratch
constexpr int kSplitMinChunk = 4;                        // key tiles of an item, at least
constexpr int kSplitParts = 256;                         // items of one launch, at most
constexpr int kSplitPartO = kRowsPerWG * 128 * 4;        // bytes: O of 128 rows x 128 dims, fp32
constexpr int kSplitPartML = kRowsPerWG * 2 * 8;         // bytes: (max, sum) per lane of 4 waves
struct SplitControl {
    // Number of the entry's last launch (48 bits) and, below it, the counts at which that
    // launch is through (16 bits). A claim exchanges the word as a whole.
    unsigned long long owner[kSplitEntries];
    // Combine workgroups that are through, of all launches so far, per XCD. Each count has
    // a line to itself: 256 workgroups counting at one address took 2-3 us, and the end of
    // a launch does not wait for a count to come back.
    unsigned int done[kSplitEntries][kXcds][32];
    unsigned int replay_lock;
};
__device__ SplitControl split_control;
__device__ __attribute__((aligned(1024))) char split_o[kSplitSlots][kSplitParts][kSplitPartO];
__device__ __attribute__((aligned(1024))) char split_ml[kSplitSlots][kSplitParts][kSplitPartML];

// The entry owned by the launch with this number (wave-uniform), or -1. From kSplitSlots on
// it has no scratch.
__device__ __forceinline__ int split_entry(uint64_t launch)
{
    const int lane = threadIdx.x & 63;
    static_assert(kSplitEntries == 64, "one lane per entry");
    const unsigned long long own =
        __hip_atomic_load(&split_control.owner[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t mine = __builtin_amdgcn_ballot_w64(own >> 16 == launch);
    return mine ? (int)__builtin_ctzll(mine) : -1;
}

// 64-key tiles of the keys [0, last].
__device__ __host__ __forceinline__ int key_tiles(int last) { return last / kTileKeys + 1; }

// A sequence with one new token in a prefill launch (a decode row, Sec. 2.2; prefill
// and decode rows in one pass, Sec. 4.3): its G rows would fill G columns of the
// 128- or 256-row tiles, and the workgroup would spend the matrix time of the whole
// tile on them while its loads sit idle. Its workgroup instead runs the decode
// kernel's wave routine (decode_wave.h): the 8 waves each take one chunk of the keys
// (with two register sets, which the prefill kernel's register budget allows) and
// merge their (O, max, sum) through LDS. The work is then bound by reading K/V, and
// it overlaps the matrix-bound workgroups of the prefill rows on the other compute
// units.
// Keys [n0, n_keys) of the row; with part_o they leave the unnormalised O, max and sum
// there (a chunk of a key-split launch), otherwise the row is written.
template <int D>
__device__ __forceinline__ void decode_workgroup(const u16 *__restrict__ q, const u16 *__restrict__ pool_k,
                                                 const u16 *__restrict__ pool_v, int32_t num_blocks, int32_t Hkv,
                                                 const int32_t *__restrict__ bt_row, int32_t max_blocks, int g, int G,
                                                 int32_t Hq, int n0, int n_keys, int64_t t0, float scale_log2,
                                                 u16 *__restrict__ out, char *lds, f32x4 *part_out,
                                                 float *part_out_ml)
{
    constexpr int MT = D / 16;
    constexpr int kWaves = kThreads / 64;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int chunk = ((n_keys - n0 + kWaves - 1) / kWaves + decode_wave::kStepKeys - 1) / decode_wave::kStepKeys *
                      decode_wave::kStepKeys;
    const int kbeg = n0 + wave * chunk;
    const int kend = min(n_keys, kbeg + chunk);
    const int last_blk = max(0, min((n_keys - 1) >> 4, max_blocks - 1));
    const int c = lane & 15, q4 = lane >> 4;
    const bool col = c < G;
    const int h = g * G + c;
    f32x4 o[MT];
    float m_run = decode_wave::kNoMax, l_run = 0.f;
    if (kbeg < n_keys) {
        const u16 *qrow = q + (t0 * Hq + (col ? h : g * G)) * D + 8 * q4;
        decode_wave::chunk<D, 2, true>(qrow, col, pool_k, pool_v, num_blocks, Hkv, g, bt_row, last_blk, kbeg, kend,
                                 scale_log2, o, m_run, l_run);
    } else {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) o[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    float l_tot = l_run + __shfl_xor(l_run, 16);
    l_tot += __shfl_xor(l_tot, 32);
    // Waves 1.. leave O (lane layout), max and sum in LDS; wave 0 merges and writes. A
    // chunk past the end, or without a finite score, contributes max kNoMax, sum 0, O 0.
    f32x4 *part_o = reinterpret_cast<f32x4 *>(lds);                         // [wave][MT][64 lanes]
    float *part_ml = reinterpret_cast<float *>(part_o + kWaves * MT * 64);   // [wave][64 lanes][2]
    if (wave > 0) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) part_o[(wave * MT + mt) * 64 + lane] = o[mt];
        part_ml[2 * (wave * 64 + lane)] = m_run;
        part_ml[2 * (wave * 64 + lane) + 1] = l_tot;
    }
    __syncthreads();
    // (no early return here: a return on a lane condition inside this inlined function
    // made the compiler treat the prefill path's block offsets as divergent)
    if (wave == 0) {
        float M = m_run;
        for (int w = 1; w < kWaves; ++w) M = fmaxf(M, part_ml[2 * (w * 64 + lane)]);
        const float a0 = __builtin_amdgcn_exp2f(m_run - M);
        l_tot *= a0;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) o[mt] *= a0;
        for (int w = 1; w < kWaves; ++w) {
            const float a = __builtin_amdgcn_exp2f(part_ml[2 * (w * 64 + lane)] - M);
            l_tot += a * part_ml[2 * (w * 64 + lane) + 1];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) o[mt] += a * part_o[(w * MT + mt) * 64 + lane];
        }
        if (part_out) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) part_out[mt * 64 + lane] = o[mt];
            part_out_ml[2 * lane] = M;
            part_out_ml[2 * lane + 1] = l_tot;
        } else if (col) {
            const float inv = 1.f / l_tot;
            u16 *orow = out + (t0 * Hq + h) * D + 4 * q4;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const bf16x4 v = __builtin_convertvector(o[mt] * inv, bf16x4);
                *reinterpret_cast<u32x2 *>(orow + 16 * mt) = __builtin_bit_cast(u32x2, v);
            }
        }
    }
}

// One work item of a launch.
struct Item {
    int g, j;             // kv head and the item's index in the work map (g >= Hkv: none)
    int b, p, t0, s;      // sequence, cached tokens, first new token, new tokens
    int local;            // item within the sequence, counted from the sequence's last
};

// XCD-aware order: workgroup L runs on XCD L % 8. The row tiles of one (sequence,
// kv head), which read the same K/V, go to workgroups of one XCD and share its L2.
// With Hkv a multiple of 8, XCD x takes kv heads x, x+8, ... of every sequence, so the
// eight XCDs get equal work.
__device__ __forceinline__ Item locate_item(const AttnWorkMap &wm, int32_t Hkv)
{
    const int lane = threadIdx.x & 63;
    Item it;
    const int x = (int)(blockIdx.x % kXcds), i = (int)(blockIdx.x / kXcds);
    const int per_xcd = (int)(gridDim.x / kXcds);
    if (Hkv % kXcds == 0) {
        const int hh = i / wm.per_head;
        it.g = x + kXcds * hh;
        it.j = i - hh * wm.per_head;
    } else {
        const int w = x * per_xcd + i;
        it.g = w / wm.per_head;
        it.j = w - it.g * wm.per_head;
    }
    // Slot of item j: the number of slots whose items end at or before j. Lane l
    // reads slots l and l + 64 (all fields at once); the slot's fields are then taken
    // from the lane that holds them.
    int e[2], fs[2], fp[2], ft[2], fc[2];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
        const int k = lane + 64 * hf;
        const bool in = k < wm.n_seq;
        e[hf] = in ? wm.tiles_end[k] : INT32_MAX;
        fs[hf] = in ? wm.seq[k] : 0;
        fp[hf] = in ? wm.prefix[k] : 0;
        ft[hf] = in ? wm.first[k] : 0;
        fc[hf] = in ? wm.count[k] : 0;
    }
    const int slot = __builtin_popcountll(__builtin_amdgcn_ballot_w64(e[0] <= it.j)) +
                     __builtin_popcountll(__builtin_amdgcn_ballot_w64(e[1] <= it.j));
    const int hf = slot >> 6, sl = slot & 63;
    it.b = __builtin_amdgcn_readlane(hf ? fs[1] : fs[0], sl);
    it.p = __builtin_amdgcn_readlane(hf ? fp[1] : fp[0], sl);
    it.t0 = __builtin_amdgcn_readlane(hf ? ft[1] : ft[0], sl);
    it.s = __builtin_amdgcn_readlane(hf ? fc[1] : fc[0], sl);
    it.local = __builtin_amdgcn_readlane(hf ? e[1] : e[0], sl) - 1 - it.j;
    return it;
}

// Output of one wave's 32 rows x W dims through LDS, so that whole lines leave it 16
// bytes a lane. In the accumulator layout a lane holds 4 consecutive dims of its row at
// a time: stored directly (8 bytes a lane, 32 rows in one instruction) the rows' lines
// went out in 32-byte pieces, and a workgroup's end waited for them: from the first wave's
// last store to the next workgroup's start on the compute unit 4.0 us, 1.6 us with whole
// lines (row halves, a ragged batch of 23 rounds; 3.9 and 1.1 us at the 70B layer).
// Rows of W bf16 lie back to back in the wave's own LDS area; 16-byte chunk c of row q is
// at chunk c ^ (q % (W/8)), and its two 8-byte halves change places in rows 16.., so that the
// 32 lanes of a half wave write every bank once and 16 lanes read every bank once. (The
// conflict counter still shows 64 cycles a wave with row halves, 32 with key halves.)
template <int W>
__device__ __forceinline__ void stage_row(char *stage, int lane, int chunk, f32x4 v)
{
    const int q = lane & 31, half = lane >> 5;
    const bf16x4 bv = __builtin_convertvector(v, bf16x4);   // dims 8 chunk + 4 half ..
    *reinterpret_cast<u32x2 *>(stage + q * (W * 2) + ((chunk ^ (q % (W / 8))) * 16) + ((half ^ (q >> 4)) * 8)) =
        __builtin_bit_cast(u32x2, bv);
}

// orow: the output row of lane q's row (-1: none); the W dims go to column col of rows of D.
template <int W, int D = W>
__device__ __forceinline__ void store_rows(const char *stage, int lane, int orow, u16 *__restrict__ out, int col)
{
    constexpr int CH = W / 8;             // chunks per row
    asm volatile("" ::: "memory");        // after the wave's stage_row writes (LDS runs them in order)
#pragma unroll
    for (int i = 0; i < 32 * CH / 64; ++i) {
        const int id = i * 64 + lane, q = id / CH, c = id % CH;
        const int row = __shfl(orow, q);
        u32x4 v = *reinterpret_cast<const u32x4 *>(stage + q * (W * 2) + ((c ^ (q % CH)) * 16));
        if (q >> 4) v = u32x4{v[2], v[3], v[0], v[1]};
        if (row >= 0) *reinterpret_cast<u32x4 *>(out + (int64_t)row * D + col + c * 8) = v;
    }
}

template <int D, int MODE>
__global__ __launch_bounds__(kThreads) void prefill_attn_kernel(
    const u16 *__restrict__ q, const u16 *__restrict__ pool_k, const u16 *__restrict__ pool_v,
    int32_t num_blocks, int32_t Hkv, const int32_t *__restrict__ block_tables, int32_t max_blocks, int32_t Hq,
    int32_t T, float scale_log2, float rescale_thr, u16 *__restrict__ out, const AttnWorkMap wm)
{
    using Geo = TileGeom<D>;
    constexpr int CPR = Geo::CPR;
    constexpr int KSTEPS = D / 16;
    constexpr int MT = D / 32;
    constexpr int64_t kPayloadBytes = kBlockSize * D * 2;   // one (block, kv head) of K or V
    constexpr int kSlabs = (int)(kPayloadBytes / 1024);       // 1 KB slabs per payload
    static_assert(kGroupWaves % kSlabs == 0, "slab-to-wave mapping");
    constexpr int kKLoads = Geo::KLOADS, kVLoads = Geo::VLOADS;
    constexpr bool ROWS = MODE == kRowHalves;
    constexpr int RPW = ROWS ? 2 * kRowsPerWG : kRowsPerWG;   // packed rows per workgroup

    // Per group: K buffers 0/1 then V buffers 0/1 (double-buffered, tile j in buffer j&1);
    // with row halves both groups use group 0's. The whole array is reused for the merge
    // at the end of key halves.
    __shared__ __attribute__((aligned(1024))) char lds[2][2 * (Geo::KBYTES + Geo::VBYTES)];

    const int tid = threadIdx.x, lane = tid & 63;
    const Item it = locate_item(wm, Hkv);
    const int g = it.g;
    if (g >= Hkv) return;
    const int b = it.b, p = it.p, t0 = it.t0, s = it.s;
    // Key split: item `local` of the sequence is chunk sp of row tile rt.
    int rt = it.local, sp = 0, part = -1;
    if constexpr (MODE == kKeySplit) {
        const int ns = (key_tiles(p + s - 1) + wm.chunk - 1) / wm.chunk;
        rt = it.local / ns;
        sp = it.local - rt * ns;
        const int slot = split_entry(wm.launch);
        const bool whole = slot < 0 || slot >= kSplitSlots;
        if (whole && sp > 0) return;                 // unsplit: chunk 0 takes every key
        if (!whole) part = slot * kSplitParts + g * wm.per_head + it.j;
    }
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave >> 2;              // key halves: which half of the keys; row halves: of the rows
    const int wg = wave & 3;                // wave within the group (selects the rows)
    const int qc = lane & 31, half = lane >> 5;

    const int G = Hq / Hkv;
    const int rows_total = s * G;
    const int row0 = rt * RPW;
    if (s <= 0 || row0 >= rows_total || T <= 0) return;   // uniform over the workgroup
    if (s == 1 && G <= decode_wave::kMaxCols) {           // a decode row (uniform too)
        static_assert(kThreads / 64 * (D / 16) * 64 * 16 + kThreads / 64 * 64 * 8 <= (int)sizeof(lds), "merge area");
        if (t0 >= T) return;
        int n0 = 0, n_keys = p + 1;                  // keys 0 .. p: the row's causal range
        f32x4 *po = nullptr;
        float *pml = nullptr;
        if constexpr (MODE == kKeySplit) {
            if (part >= 0 && n_keys > wm.chunk * kTileKeys) {
                n0 = sp * wm.chunk * kTileKeys;
                n_keys = min(n_keys, n0 + wm.chunk * kTileKeys);
                po = reinterpret_cast<f32x4 *>(&split_o[0][0][0] + (int64_t)part * kSplitPartO);
                pml = reinterpret_cast<float *>(&split_ml[0][0][0] + (int64_t)part * kSplitPartML);
            }
        }
        decode_workgroup<D>(q, pool_k, pool_v, num_blocks, Hkv, block_tables + (int64_t)b * max_blocks, max_blocks,
                            g, G, Hq, n0, n_keys, t0, scale_log2, out, &lds[0][0], po, pml);
        return;
    }
    const int total = p + s;

    // This lane's packed query row (rows past the end compute a copy of the last row).
    const int wrow0 = row0 + (ROWS ? grp * kRowsPerWG : 0) + wg * kRowsPerWave;   // this wave's first row
    const int R = wrow0 + qc;
    const bool row_valid = R < rows_total;
    const int Rc = row_valid ? R : rows_total - 1;
    const int i = Rc / G, hl = Rc - i * G;
    const int limit = p + i;                         // last key this row attends to
    const int tq = min(t0 + i, T - 1);               // (T * Hq fits 31 bits)
    const int qrow = tq * Hq + g * G + hl;           // its row of q and out
    // Its output row, -1 past the end; held in one register over the loop.
    int orow = row_valid ? qrow : -1;
    asm volatile("" : "+v"(orow));

    const int wg_last = min(rows_total - 1, row0 + RPW - 1);
    const int all_tiles = key_tiles(p + wg_last / G);
    // This workgroup's tiles [t_lo, t_lo + ntiles): all, or a chunk of a key split.
    int t_lo = 0, ntiles = all_tiles;
    if constexpr (MODE == kKeySplit) {
        if (part >= 0) {
            t_lo = sp * wm.chunk;
            ntiles = min(all_tiles - t_lo, wm.chunk);
            if (ntiles <= 0) return;                 // (an earlier row tile ends before this chunk)
            if (all_tiles <= wm.chunk) part = -1;    // the only chunk of its row tile: written directly
        }
    }
    // key halves: group 0 takes the first `split` tiles, group 1 the rest; row halves:
    // both take every tile
    const int split = ROWS ? ntiles : (ntiles + 1) >> 1;
    const int tile_begin = t_lo + ((!ROWS && grp) ? split : 0);
    const int n = (ROWS || !grp) ? split : ntiles - split;        // this group's tiles
    const int w_first = min(rows_total - 1, wrow0);
    const int w_min_limit = p + w_first / G;
    const int valid_blocks = min((total + kBlockSize - 1) / kBlockSize, max_blocks);

    bf16x8 qf[KSTEPS];    // the Q^T operand (k-step ks: dims 16ks + 8half .. +7 of this lane's row)

    f32x16 o_acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o_acc[mt][r] = 0.f;
    // Scores are kept relative to a reference m_ref (raw units of <q,k>): the first
    // product starts from -m_ref, so S^T holds <q,k> - m_ref and P = exp2(c * S^T) with
    // c = scale_log2.
    float m_ref = 0.f;
    // The reference moves when a tile's max (relative to it) exceeds thr: -inf until the
    // first real score of the row, then rescale_thr = 8 / c, so P stays <= 2^8 and O is
    // rescaled rarely.
    float thr = -INFINITY;
    // Row sums of the bf16 P on the matrix pipe (64 fewer VALU instructions per tile in
    // the softmax than adding the rounded values there, for 4 short MFMAs that fill idle
    // matrix-pipe cycles): v_mfma_f32_16x16x32_bf16 with B = a P^T
    // operand of the second product (read in that instruction's layout: column c = lane%16
    // takes the 8-key runs of lanes c, c+16, c+32, c+48, i.e. queries c and c+16, each over
    // both key halves) and a constant A whose row m is 1 on the runs of query c when m is
    // even and of query c+16 when m is odd. Per tile, four such products (one per P^T
    // operand) start from zero; lane l then holds the tile's sum of query l%16 in
    // tsum[0] and of query l%16+16 in tsum[1], i.e. of its own query (l%32) in
    // tsum[(l >> 4) & 1]. The next softmax adds it to the running sum before any
    // rescale, so the running sum stays one fp32 per lane.
    f32x4 tsum = {0.f, 0.f, 0.f, 0.f};   // the last PV'd tile's sums (zero before the first)
    float l_run = 0.f;                     // this lane's query: sum over the earlier tiles
    bf16x8 sum_pat;
    {
        const __bf16 one = (((lane & 15) ^ (lane >> 4)) & 1) ? (__bf16)0.f : (__bf16)1.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) sum_pat[e] = one;
    }
    f32x16 nbias;
#pragma unroll
    for (int r = 0; r < 16; ++r) nbias[r] = 0.f;

    const int32_t *bt = block_tables + (int64_t)b * max_blocks;
    const int lgrp = ROWS ? 0 : grp;        // whose tile buffers this group reads
    auto kbuf = [&](int j) __attribute__((always_inline)) { return &lds[lgrp][(j & 1) * Geo::KBYTES]; };
    auto vbuf = [&](int j) __attribute__((always_inline)) { return &lds[lgrp][2 * Geo::KBYTES + (j & 1) * Geo::VBYTES]; };
    // The same buffers as LDS byte addresses, for the direct loads (no generic-pointer casts).
    const uint32_t lds_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)&lds[lgrp][0];
    auto kbuf_off = [&](int j) __attribute__((always_inline)) { return (uint32_t)((j & 1) * Geo::KBYTES); };
    auto vbuf_off = [&](int j) __attribute__((always_inline)) { return (uint32_t)(2 * Geo::KBYTES + (j & 1) * Geo::VBYTES); };

    // Pool block ids of this group's tile j, read raw (as scalars) one phase before
    // use. Logical blocks past the sequence read the last valid entry, so the four loads
    // are independent and nothing consumes their values until the range check at use:
    // every key past the sequence is masked and the V entries past it are cleared in
    // the last tile, so any in-pool block can stand in there; an id outside the pool
    // becomes block 0, so no load ever leaves the pool.
    const char *bt_bytes = reinterpret_cast<const char *>(bt);
    auto tile_ids = [&](int j, int32_t (&ids)[kTileBlocks]) __attribute__((always_inline)) {
#pragma unroll
        for (int jb = 0; jb < kTileBlocks; ++jb) {
            const uint32_t lb = (uint32_t)min((tile_begin + j) * kTileBlocks + jb, valid_blocks - 1);
            ids[jb] = *reinterpret_cast<const int32_t *>(bt_bytes + lb * 4u);   // 32-bit offset form
        }
    };
    // Byte offset of the (pool block, kv head g) payload of a raw block id; an id outside
    // the pool becomes block 0. (blk * Hkv + g fits in 32 bits for any pool that fits in
    // memory: 2^32 payloads would be 8 TB.)
    auto payload_off = [&](int32_t blk) __attribute__((always_inline)) -> int64_t {
        const uint32_t b = (uint32_t)blk < (uint32_t)num_blocks ? (uint32_t)blk : 0u;
        return (int64_t)(b * (uint32_t)Hkv + (uint32_t)g) * kPayloadBytes;
    };
    auto to_offs = [&](const int32_t (&ids)[kTileBlocks], int64_t (&offs)[kTileBlocks]) __attribute__((always_inline)) {
#pragma unroll
        for (int jb = 0; jb < kTileBlocks; ++jb) offs[jb] = payload_off(ids[jb]);
    };
    int32_t ids_raw[kTileBlocks];   // ids of the tile two ahead, read in a vector cluster
    // Direct-load addressing. A tile's K (or V) is 4 pool blocks of one kv head, each a
    // contiguous payload of kSlabs 1 KB slabs; wave wg loads slabs u*4 + wg. Because 4
    // is a multiple of kSlabs, a lane's byte offset inside the payload is the same for
    // every u, so it is computed once here; the LDS swizzle is applied through it.
    const char *pool_k_bytes = reinterpret_cast<const char *>(pool_k);
    const char *pool_v_bytes = reinterpret_cast<const char *>(pool_v);
    uint32_t k_off, v_off;
    {
        const int chunk = (wg % kSlabs) * 64 + lane;          // 16-B chunk within the payload
        const int key = chunk / CPR, pc = chunk % CPR;        // K: row (slot) and chunk of the row
        k_off = (uint32_t)(key * 2 * D + ((pc ^ k_swizzle<CPR>(key)) * 16));
        const int d = chunk >> 1, pch = chunk & 1;            // V: dim and half of its 16 slots
        v_off = (uint32_t)(d * 2 * kBlockSize + ((pch ^ ((d >> 3) & 1)) * 16));
    }

    // Direct loads of this group's tile j (K or V) into its buffer; 1 KB slab per
    // wave-wide load; the LDS swizzle is applied through each lane's source.
    // One direct load (load u of the tile's K or V) of this group's tile j into its buffer:
    // a 1 KB slab per wave-wide load; the LDS swizzle is applied through each lane's source.
    auto load_k = [&](int j, const int64_t (&offs)[kTileBlocks], int u) __attribute__((always_inline)) {
        const int slab = u * kGroupWaves + wg;                             // wave-uniform
        dma16(pool_k_bytes + offs[slab / kSlabs], k_off, lds_addr + kbuf_off(j) + slab * 1024);
    };
    auto load_v = [&](int j, const int64_t (&offs)[kTileBlocks], int u) __attribute__((always_inline)) {
        const int slab = u * kGroupWaves + wg;
        dma16(pool_v_bytes + offs[slab / kSlabs], v_off, lds_addr + vbuf_off(j) + slab * 1024);
    };
    auto issue_k = [&](int j, const int64_t (&offs)[kTileBlocks]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kKLoads; ++u) load_k(j, offs, u);
    };

    // ---- matrix work: O^T += V^T(j) P^T(j), k-step t = pool block t of the tile.
    // In the tile holding the sequence end, V entries of keys >= total are cleared
    // in the operand (their slots may hold anything; 0 * NaN would poison O).
    auto pv = [&](int j, const bf16x8 (&pf)[kTileBlocks], auto clear_tag) __attribute__((always_inline)) {
        constexpr bool CLEAR = decltype(clear_tag)::value;
        const char *tv = vbuf(j);
        const int vlim = total - (tile_begin + j) * kTileKeys;     // valid keys in the tile
#pragma unroll
        for (int t = 0; t < kTileBlocks; ++t) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const int d = 32 * mt + qc;
                const int pch = half ^ ((d >> 3) & 1);
                u32x4 raw = *reinterpret_cast<const u32x4 *>(tv + ((t * D + d) * 2 + pch) * 16);
                if constexpr (CLEAR) {
                    const int nvalid = vlim - 16 * t - 8 * half;   // valid keys among this lane's 8
#pragma unroll
                    for (int wd = 0; wd < 4; ++wd)
                        raw[wd] &= (2 * wd < nvalid ? 0x0000FFFFu : 0u) | (2 * wd + 1 < nvalid ? 0xFFFF0000u : 0u);
                }
                o_acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(raw), pf[t], o_acc[mt], 0, 0, 0);
            }
            tsum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sum_pat, pf[t], t == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : tsum,
                                                           0, 0, 0);
        }
    };

    // ---- matrix cluster: PV(j) (optional) then QK(j+1) (optional) as one stream of
    // (LDS fragment, MFMA) pairs, the fragment reads running kAhead pairs ahead (a single
    // wave gets about one 1 KB LDS read per MFMA time, so reads must stay in flight
    // behind the MFMAs). When QK runs, the cluster also issues the direct loads of
    // V(j+1) and K(j+2), one per few MFMAs, so the texture path never backs up a wave.
    auto matrix_cluster = [&](auto pv_tag, auto qk_tag, int j, const bf16x8 (&pf)[kTileBlocks],
                              f32x16 (&st)[2], int64_t (&idv)[kTileBlocks], int64_t (&idk)[kTileBlocks],
                              auto convert_tag, auto load_tag) __attribute__((always_inline)) {
        constexpr bool DO_PV = decltype(pv_tag)::value, DO_QK = decltype(qk_tag)::value;
        constexpr bool LOADS = decltype(load_tag)::value;

        constexpr int NPV = DO_PV ? kTileBlocks * MT : 0, NQK = DO_QK ? 2 * KSTEPS : 0, NALL = NPV + NQK;
        constexpr int NLD = DO_QK && LOADS ? kVLoads + kKLoads : 0;
        constexpr int NLD1 = NLD > 0 ? NLD : 1;
        constexpr int EVERY = NALL / NLD1 > 0 ? NALL / NLD1 : 1;
        constexpr int kAhead = KAHEAD;
        const char *tv = vbuf(j);
        const char *tk = kbuf(j + 1);
        auto frag = [&](int i) __attribute__((always_inline)) -> u32x4 {
            if (i < NPV) {
                const int t = i / MT, mt = i % MT;
                const int d = 32 * mt + qc;
                const int pch = half ^ ((d >> 3) & 1);
                return *reinterpret_cast<const u32x4 *>(tv + ((t * D + d) * 2 + pch) * 16);
            }
            const int m = (i - NPV) / KSTEPS, ks = (i - NPV) % KSTEPS;
            const int krow = 32 * m + key_of_row(qc);
            const int pc = (2 * ks + half) ^ k_swizzle<CPR>(krow);
            return *reinterpret_cast<const u32x4 *>(tk + (krow * CPR + pc) * 16);
        };
        // The wave in its matrix cluster takes issue priority over the other wave of its
        // SIMD (in its vector cluster): otherwise the older wave of each SIMD always wins
        // arbitration and the younger group is late in every phase.
        __builtin_amdgcn_s_setprio(1);
        u32x4 fr[NALL];
#pragma unroll
        for (int i = 0; i < kAhead && i < NALL; ++i) fr[i] = frag(i);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(convert_tag)::value && LOADS) {
            // Block ids read in the preceding vector cluster (and waited for at its end)
            // become payload offsets here, while the first fragment reads are in flight.
#pragma unroll
            for (int jb = 0; jb < kTileBlocks; ++jb) {
                idv[jb] = idk[jb];
                idk[jb] = payload_off(ids_raw[jb]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        int ld = 0;
#pragma unroll
        for (int i = 0; i < NALL; ++i) {
            if (i + kAhead < NALL) fr[i + kAhead] = frag(i + kAhead);
            if (i < NPV) {
                const int t = i / MT, mt = i % MT;
                o_acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(fr[i]), pf[t], o_acc[mt], 0, 0, 0);
                if (mt == MT - 1)
                    tsum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sum_pat, pf[t],
                                                                   t == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : tsum, 0, 0, 0);
            } else {
                const int m = (i - NPV) / KSTEPS, ks = (i - NPV) % KSTEPS;
                st[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(fr[i]), qf[ks], ks == 0 ? nbias : st[m],
                                                                0, 0, 0);
            }
            if (NLD && i % EVERY == EVERY - 1 && ld < NLD) {
                if (ld < kVLoads) load_v(j + 1, idv, ld);
                else load_k(j + 2, idk, ld - kVLoads);
                ++ld;
            }
        }
        // keep that schedule: (read, MFMA[, load]) groups, then the last MFMAs
#pragma unroll
        for (int i = 0; i < NALL; ++i) {
            if (i + kAhead < NALL) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            if (i < NPV && i % MT == MT - 1)   // PV MFMA, then the row-sum MFMA
                __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
            else
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(0);
    };

    // ---- vector work: online softmax of S^T(j) into bf16 P(j) (lazy rescale) ----
    auto softmax = [&](int j, f32x16 (&st)[2], bf16x8 (&pf)[kTileBlocks]) __attribute__((always_inline)) {
        l_run += (lane & 16) ? tsum[1] : tsum[0];   // tile j-1 (zero before the first tile)
        const int kbase = (tile_begin + j) * kTileKeys;
        if (kbase + kTileKeys - 1 > w_min_limit) {
            // register r of half tile m holds key kbase + 32m + 16(r/8) + 8half + r%8
            const int lim = limit - kbase - 8 * half;
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    st[m][r] = (32 * m + 16 * (r >> 3) + (r & 7)) > lim ? -INFINITY : st[m][r];
        }
        // NaN-propagating maximum (v_maximum3_f32): unlike fmaxf it needs no
        // canonicalisation of the MFMA results. Written as two chains of
        // max(max(m, a), b), one three-operand instruction per two scores; a pairwise
        // tree would spend a three-operand instruction on every pair.
        float mc[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            mc[m] = __builtin_elementwise_maximum(st[m][0], st[m][1]);
#pragma unroll
            for (int r = 2; r < 16; r += 2)
                mc[m] = __builtin_elementwise_maximum(__builtin_elementwise_maximum(mc[m], st[m][r]), st[m][r + 1]);
        }
        float mx = __builtin_elementwise_maximum(mc[0], mc[1]);
        {   // The other half-wave holds the other 32 keys of the same query: swap halves and
            // take the larger. The two swap results are copied out of the returned vector
            // before the bit casts: a bit cast applied to an element of it directly reads
            // element 0 for both, which drops the half-wave's own keys from its max.
            const unsigned mine = __builtin_bit_cast(unsigned, mx);
            const auto sw = __builtin_amdgcn_permlane32_swap(mine, mine, false, false);
            const unsigned lo = sw[0], hi = sw[1];
            mx = __builtin_elementwise_maximum(__builtin_bit_cast(float, lo), __builtin_bit_cast(float, hi));
        }
        const bool need = mx > thr;
        if (__builtin_amdgcn_ballot_w64(need)) {
            const float delta = need ? mx : 0.f;
            // Before a row's first real score nothing has accumulated, and that first max
            // may lie far below the initial reference (2^-delta would overflow to +inf
            // and turn the zero accumulators into NaN): scale by 0 then.
            const float alpha = thr == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(-delta * scale_log2);
            thr = need ? rescale_thr : thr;
            m_ref += delta;
            l_run *= alpha;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 16; ++r) o_acc[mt][r] *= alpha;
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int r = 0; r < 16; ++r) st[m][r] -= delta;
#pragma unroll
            for (int r = 0; r < 16; ++r) nbias[r] = -m_ref;
        }
        // P rounded to bf16 is both the second product's operand and what the row sums
        // add (on the matrix pipe, see tsum): the weights then sum to one however P
        // rounds (a one-hot row returns its V row exactly), where a sum of the fp32
        // values would leave up to 2^-8 of relative error on a dominant term.
#pragma unroll
        for (int t = 0; t < kTileBlocks; ++t) {
            f32x8 pv8;
#pragma unroll
            for (int e = 0; e < 8; ++e)
                pv8[e] = __builtin_amdgcn_exp2f(st[t >> 1][8 * (t & 1) + e] * scale_log2);
            pf[t] = __builtin_convertvector(pv8, bf16x8);
        }
    };

    // Ping-pong schedule. Each group runs the cluster sequence
    //   C(-1), M(0), C(0), M(1), C(1), ..., M(n-1), C(n-1)
    // with C(j) = [PV(j), QK(j+1), direct loads of V(j+1) and K(j+2)] (matrix) and
    // M(j) = [softmax(j)] (vector). Group 1 runs one phase behind group 0, so in every
    // phase each SIMD has one wave in a matrix cluster and one in a vector cluster.
    // Every phase ends with a workgroup barrier (both groups pass the same number);
    // the loads issued in C(j) are waited for at the end of M(j+1), one phase before
    // C(j+1) reads them. Rows whose causal limit ends before a tile get P = 0 there.
    // Block offsets travel one phase ahead: at C(j), ids_v holds tile j+1's (for
    // V(j+1)) and ids_k tile j+2's (for K(j+2)).
    // With row halves both groups walk the same tiles, and only group 0 loads them:
    // group 1 reads group 0's buffers one phase later. Two buffers per operand still
    // suffice: group 0's C(j) (phase 2j+2 counted from the first barrier) overwrites the
    // buffers of V(j-1) and K(j), whose last reader is group 1's C(j-1) in phase 2j+1,
    // and the barrier between phases orders the two. The LDS then takes one tile's
    // direct-load writes per two phases instead of two, on a path whose fragment reads
    // already run near its bandwidth.
    const bool loader = !ROWS || grp == 0;
    int64_t ids_v[kTileBlocks], ids_k[kTileBlocks];   // payload byte offsets
    int32_t ids_next[kTileBlocks];
    tile_ids(0, ids_raw);
    tile_ids(1, ids_next);
    to_offs(ids_raw, ids_v);
    if (n > 0 && loader) issue_k(0, ids_v);            // K(0) for C(-1)
    // Q^T operand fragments (k-step ks: dims 16ks + 8half .. +7 of this lane's row), the
    // bf16 input as it is, requested after K(0): eight loads in the operand layout touch 32
    // rows for 32 bytes each, and K(0) waited behind them (8B layer: 1.2 us from the item's
    // lookup to K(0)'s request, 0.6 us now). Key halves take whole rows through LDS, each
    // wave's 32 rows by direct loads into this group's V buffers, free until after the
    // barrier below, swizzled as a K tile (8B layer 65.1 -> 64.5 us with both changes; row
    // halves read the operand layout, as the way through LDS cost them 6 spilled registers
    // and the 70B layer 1%).
    if constexpr (ROWS) {
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks)
            qf[ks] = *reinterpret_cast<const bf16x8 *>(q + (int64_t)qrow * D + 16 * ks + 8 * half);
        to_offs(ids_next, ids_k);
        wait_vmem();
    } else {
        constexpr int kQBytes = kRowsPerWave * D * 2;
        static_assert(kGroupWaves * kQBytes <= 2 * Geo::VBYTES, "Q in the V buffers");
        const uint32_t q_off = (uint32_t)(2 * Geo::KBYTES + wg * kQBytes);
#pragma unroll
        for (int u = 0; u < kQBytes / 1024; ++u) {
            const int id = u * 64 + lane, r = id / CPR, pc = id % CPR;
            const int64_t row = __shfl(qrow, r);
            dma16_at(reinterpret_cast<const char *>(q + row * D) + ((pc ^ (r % CPR)) * 16), lds_addr + q_off + u * 1024);
        }
        to_offs(ids_next, ids_k);
        wait_vmem();
        const char *q_tile = &lds[lgrp][0] + q_off;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks)
            qf[ks] = *reinterpret_cast<const bf16x8 *>(q_tile + qc * (2 * D) + (((2 * ks + half) ^ (qc % CPR)) * 16));
        // read before another wave of the group loads V(0) over it
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    }
    __syncthreads();

    const int n0 = split, n1 = ROWS ? ntiles : ntiles - split;
    const int phases = max(2 * n0 + 1, 2 * n1 + 2);
    int ph = 0;
    auto phase_end = [&]() __attribute__((always_inline)) {
        phase_barrier();
        ++ph;
    };
    // M(j): softmax of tile j; block ids of tile j+2 (read now, range-checked and
    // converted at the start of C(j)) when this group loads; then wait for the loads
    // C(j-1) issued.
    auto vector_cluster = [&](int j, f32x16 (&st)[2], bf16x8 (&pf)[kTileBlocks], auto load_tag) __attribute__((always_inline)) {
        // The scalar loads of the ids go out before the softmax, whose length covers
        // their latency (left to itself the scheduler sinks them next to their use).
        if constexpr (decltype(load_tag)::value) tile_ids(j + 2, ids_raw);
        __builtin_amdgcn_sched_barrier(0);
        softmax(j, st, pf);
        wait_vmem();
        // The id loads landed long ago; an explicit wait here (seen by the compiler) keeps
        // it from placing one among the next matrix cluster's fragment reads.
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    };

    f32x16 st[2];
    bf16x8 pf[kTileBlocks];
    if (grp == 1) phase_end();
    // The tile loop, instantiated once for a group that loads and once for one that
    // only reads (row halves, group 1), so that no branch splits a matrix cluster.
    auto run_tiles = [&](auto load_tag) __attribute__((always_inline)) {
        constexpr std::true_type T_{};
        constexpr std::false_type F_{};
        // C(-1): QK(0), loads of V(0) and K(1) (K(1) lands in an unused buffer if n == 1)
        matrix_cluster(F_, T_, -1, pf, st, ids_v, ids_k, F_, load_tag);
        phase_end();
        // Four (M, C) pairs per iteration: the scores made in one pair's matrix cluster
        // feed the next pair's softmax in the same registers, and the register copies
        // that the loop-carried scores and the softmax shift cost at the iteration
        // boundary are paid once per four tiles (about 0.7% faster than two pairs).
        // C(j): PV(j), QK(j+1), loads of V(j+1) and K(j+2) (the last K lands unused).
        int j = 0;
        for (; j + 4 < n; j += 4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                vector_cluster(j + u, st, pf, load_tag);
                phase_end();
                matrix_cluster(T_, T_, j + u, pf, st, ids_v, ids_k, T_, load_tag);
                phase_end();
            }
        }
        for (; j + 2 < n; j += 2) {
            vector_cluster(j, st, pf, load_tag);
            phase_end();
            matrix_cluster(T_, T_, j, pf, st, ids_v, ids_k, T_, load_tag);
            phase_end();
            vector_cluster(j + 1, st, pf, load_tag);
            phase_end();
            matrix_cluster(T_, T_, j + 1, pf, st, ids_v, ids_k, T_, load_tag);
            phase_end();
        }
        if (j + 1 < n) {
            vector_cluster(j, st, pf, load_tag);
            phase_end();
            matrix_cluster(T_, T_, j, pf, st, ids_v, ids_k, T_, load_tag);
            phase_end();
        }
        vector_cluster(n - 1, st, pf, load_tag);
        phase_end();
        // The group's last tile may hold the sequence end: clear V past it.
        if ((tile_begin + n) * kTileKeys > total) pv(n - 1, pf, T_);
        else matrix_cluster(T_, F_, n - 1, pf, st, ids_v, ids_k, F_, load_tag);
        phase_end();
    };
    if (n > 0) {
        if (loader) run_tiles(std::true_type{});
        else run_tiles(std::false_type{});
    }
    while (ph < phases) phase_end();

    if constexpr (ROWS) {
        // ---- row halves: every group saw all keys of its rows; normalise, store ----
        // (the last phase's barrier is behind every read of the tile buffers)
        const float inv = 1.f / (l_run + ((lane & 16) ? tsum[1] : tsum[0]));
        char *stage = &lds[0][0] + wave * (32 * D * 2);
#pragma unroll
        for (int k = 0; k < MT; ++k)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                f32x4 v;
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = o_acc[k][4 * r4 + c] * inv;
                stage_row<D>(stage, lane, 4 * k + r4, v);
            }
        store_rows<D>(stage, lane, orow, out, 0);
        return;
    }

    // ---- key halves: merge the two halves through LDS, normalise, store ----
    // Each group finalises half of the head dims (group 0 the first MT/2 blocks of 32,
    // group 1 the rest): it sends the partner wave holding the same rows the other half
    // of its accumulator and its (m, l), then merges the half it received.
    const float l_tot = l_run + ((lane & 16) ? tsum[1] : tsum[0]);   // plus the group's last tile
    const bool has_ref = thr > -INFINITY;      // this row saw a real score in this key half
    constexpr int MH = MT / 2;
    constexpr int XW = 4 * MH + 1;                 // float4 slots per lane: half of O, then (m, l)
    static_assert(2 * kGroupWaves * XW * 64 * 16 <= (int)sizeof(lds), "merge area");
    const int my0 = grp ? MH : 0, other0 = grp ? 0 : MH;
    __syncthreads();
    f32x4 *xch = reinterpret_cast<f32x4 *>(&lds[0][0]);
    {
        f32x4 *xo = xch + (size_t)(grp * kGroupWaves + wg) * XW * 64;
#pragma unroll
        for (int k = 0; k < MH; ++k)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                f32x4 v;
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = o_acc[other0 + k][4 * r4 + c];
                xo[(k * 4 + r4) * 64 + lane] = v;
            }
        xo[(XW - 1) * 64 + lane] = f32x4{has_ref ? m_ref : -INFINITY, l_tot, 0.f, 0.f};
    }
    __syncthreads();

    const f32x4 *xi = xch + (size_t)((1 - grp) * kGroupWaves + wg) * XW * 64;
    const f32x4 ml = xi[(XW - 1) * 64 + lane];
    const float m1 = ml[0], l1 = ml[1];
    const float m0 = has_ref ? m_ref : -INFINITY;
    const float mm = fmaxf(m0, m1);
    const float a0 = (m0 == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f((m0 - mm) * scale_log2);
    const float a1 = (m1 == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f((m1 - mm) * scale_log2);
    if constexpr (MODE == kKeySplit) {
        if (part >= 0) {
            // A chunk's partial result, in the lane layout (1 KB per wave-wide store).
            if (orow >= 0) {
                f32x4 *po = reinterpret_cast<f32x4 *>(&split_o[0][0][0] + (int64_t)part * kSplitPartO) +
                            wg * MT * 4 * 64 + lane;
                f32x2 *pml = reinterpret_cast<f32x2 *>(&split_ml[0][0][0] + (int64_t)part * kSplitPartML) +
                             wg * 64 + lane;
#pragma unroll
                for (int k = 0; k < MH; ++k)
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) {
                        const f32x4 o1 = xi[(k * 4 + r4) * 64 + lane];
                        f32x4 v;
#pragma unroll
                        for (int c = 0; c < 4; ++c) v[c] = a0 * o_acc[my0 + k][4 * r4 + c] + a1 * o1[c];
                        po[((my0 + k) * 4 + r4) * 64] = v;
                    }
                if (grp == 0) *pml = f32x2{mm, a0 * l_tot + a1 * l1};
            }
            return;
        }
    }
    const float inv = 1.f / (a0 * l_tot + a1 * l1);
    char *stage = &lds[0][0] + 2 * kGroupWaves * XW * 64 * 16 + wave * (32 * MH * 32 * 2);
    static_assert(2 * kGroupWaves * (XW * 64 * 16 + 32 * MH * 32 * 2) <= (int)sizeof(lds), "merge and output area");
#pragma unroll
    for (int k = 0; k < MH; ++k)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
            const f32x4 o1 = xi[(k * 4 + r4) * 64 + lane];
            f32x4 v;
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = (a0 * o_acc[my0 + k][4 * r4 + c] + a1 * o1[c]) * inv;
            stage_row<MH * 32>(stage, lane, 4 * k + r4, v);
        }
    store_rows<MH * 32, D>(stage, lane, orow, out, my0 * 32);
}

// One wave: takes a free slot for the launch with this number, which no other launch has,
// and per_xcd combine workgroups on each XCD (none free: the launch finds no slot and runs
// unsplit). Lane 8 * slot + x reads the slot's owner word and its count of XCD x; the slot
// is free when all eight counts are where its last launch ends. The exchange fails if
// another launch was faster.
__global__ __launch_bounds__(64) void split_claim_kernel(uint64_t launch, unsigned per_xcd)
{
    static_assert(kSplitSlots * kXcds == 64, "one lane per slot and XCD");
    const int lane = threadIdx.x, slot = lane / kXcds, x = lane % kXcds;
    for (int tries = 0; tries < 2 * kSplitSlots; ++tries) {
        unsigned long long own =
            __hip_atomic_load(&split_control.owner[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned count =
            __hip_atomic_load(&split_control.done[slot][x][0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t through = __builtin_amdgcn_ballot_w64((count & 0xFFFFu) == (unsigned)(own & 0xFFFFu));
        const bool is_free = ((through >> (slot * kXcds)) & 0xFFu) == 0xFFu;
        const uint64_t any = __builtin_amdgcn_ballot_w64(is_free);
        if (!any) return;
        bool taken = false;
        if (lane == (int)__builtin_ctzll(any))
            taken = __hip_atomic_compare_exchange_strong(&split_control.owner[slot], &own,
                                                         launch << 16 | ((own + per_xcd) & 0xFFFFu),
                                                         __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
        if (__builtin_amdgcn_ballot_w64(taken)) return;
    }
}

// The same for a captured launch, whose number its replays share: an entry in use under that
// number (it is then through when this replay's workgroups are too: its end moves on by
// them), else the slot an earlier replay had, else the first free entry, slots first. One
// entry at most carries the number. The lock keeps two replays from taking an entry each;
// whoever holds it is a running wave that waits for nothing, and the tries, far more than
// 64 claims take, are bounded all the same (a wave that gives up leaves its launch
// unsplit). Lane: entry.
__global__ __launch_bounds__(64) void split_claim_replay_kernel(uint64_t launch, unsigned per_xcd)
{
    const int lane = threadIdx.x;
    bool locked = false;
    for (int tries = 0; tries < (1 << 14) && !locked; ++tries) {
        unsigned open = 0u;
        bool got = false;
        if (lane == 0)
            got = __hip_atomic_compare_exchange_strong(&split_control.replay_lock, &open, 1u, __ATOMIC_ACQUIRE,
                                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        locked = __builtin_amdgcn_ballot_w64(got) != 0;
        if (!locked) __builtin_amdgcn_s_sleep(8);
    }
    if (!locked) return;
    bool done = false;
    for (int tries = 0; tries < 2 * kSplitEntries && !done; ++tries) {
        unsigned long long own =
            __hip_atomic_load(&split_control.owner[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bool is_free = true;
#pragma unroll
        for (int x = 0; x < kXcds; ++x) {
            const unsigned count =
                __hip_atomic_load(&split_control.done[lane][x][0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            is_free = is_free && (count & 0xFFFFu) == (unsigned)(own & 0xFFFFu);
        }
        const uint64_t mine = __builtin_amdgcn_ballot_w64(own >> 16 == launch);
        const uint64_t free_entries = __builtin_amdgcn_ballot_w64(is_free);
        const bool keep = (mine & ~free_entries) != 0 || (mine & ((1ull << kSplitSlots) - 1)) != 0;
        const uint64_t any = keep ? mine : free_entries;
        bool taken = false;
        // An earlier replay's entry without scratch, free now: another one is taken, unless it
        // is the first free one itself. (Only replays change these, so it is as it was read.)
        if (!keep && mine && any && lane == (int)__builtin_ctzll(mine) && lane != (int)__builtin_ctzll(any))
            __hip_atomic_store(&split_control.owner[lane], own & 0xFFFFu, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (any && lane == (int)__builtin_ctzll(any))
            taken = __hip_atomic_compare_exchange_strong(&split_control.owner[lane], &own,
                                                         launch << 16 | ((own + per_xcd) & 0xFFFFu),
                                                         __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
        done = !any || __builtin_amdgcn_ballot_w64(taken) != 0;
    }
    if (lane == 0)
        __hip_atomic_store(&split_control.replay_lock, 0u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// One wave: gives back the slot of a launch whose combine kernel does not run (it could not
// be enqueued), by the counts that kernel would have added. No entry: nothing.
__global__ __launch_bounds__(64) void split_release_kernel(uint64_t launch, unsigned per_xcd)
{
    const int slot = split_entry(launch);
    if (slot >= 0 && threadIdx.x < kXcds)
        __hip_atomic_fetch_add(&split_control.done[slot][threadIdx.x][0], per_xcd, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
}

// Merges the chunks of every row tile and decode row of a key-split launch:
// out = sum_s 2^(c (m_s - M)) O_s / sum_s 2^(c (m_s - M)) l_s with M = max_s m_s. Grid and
// item order are the split kernel's. The pieces of one row tile (a wave's 32 rows x 8
// dims) are dealt to the waves of all its chunks' workgroups, so the reads of the
// partial results, which bound this kernel, come from every compute unit.
constexpr int kCombineThreads = 512;
template <int D>
__global__ __launch_bounds__(kCombineThreads) void split_combine_kernel(int32_t Hkv, int32_t Hq, int32_t T,
                                                                        float scale_log2, u16 *__restrict__ out,
                                                                        const AttnWorkMap wm)
{
    constexpr int MT = D / 32;
    constexpr int kCombineWaves = kCombineThreads / 64;
    const int slot = split_entry(wm.launch);
    if (slot < 0) return;                            // ran unsplit
    const Item it = locate_item(wm, Hkv);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int G = Hq / Hkv;
    if (it.g < Hkv && slot < kSplitSlots) {          // (past them: ran unsplit, counts itself out)
        const int p = it.p, s = it.s, rows_total = s * G;
        const int ns_seq = (key_tiles(p + s - 1) + wm.chunk - 1) / wm.chunk;
        const int rt = it.local / ns_seq, sp = it.local - rt * ns_seq;
        const int row0 = rt * kRowsPerWG;
        const bool decode_row = s == 1 && G <= decode_wave::kMaxCols;
        const int wg_last = min(rows_total - 1, row0 + kRowsPerWG - 1);
        const int ns = (key_tiles(p + wg_last / G) + wm.chunk - 1) / wm.chunk;   // chunks of this row tile
        // chunk s of the row tile is item j + sp - s (items count down)
        const int64_t part0 = (int64_t)slot * kSplitParts + it.g * wm.per_head + it.j + sp;
        const f32x4 *po = reinterpret_cast<const f32x4 *>(&split_o[0][0][0]);
        const f32x2 *pml = reinterpret_cast<const f32x2 *>(&split_ml[0][0][0]);
        const int waves = (wg_last - row0) / kRowsPerWave + 1;   // of the row tile, with rows
        const int pieces = ns <= 1 || row0 >= rows_total ? 0 : decode_row ? D / 16 : waves * MT * 4;
        const float c = decode_row ? 1.f : scale_log2;    // a decode row's max is scaled already
        for (int pc = sp * kCombineWaves + wave; pc < pieces; pc += ns_seq * kCombineWaves) {
            const int wg = decode_row ? 0 : pc / (MT * 4);
            int64_t tq;
            int h, d0;
            bool ok;
            if (decode_row) {                        // piece = 16 dims; lane = head lane % 16, dims 4 (lane / 16) ..
                h = it.g * G + (lane & 15);
                tq = it.t0;
                d0 = 16 * pc + 4 * (lane >> 4);
                ok = (lane & 15) < G;
            } else {                                 // piece = (wave, 8 dims); lane = row lane % 32, half lane / 32
                const int R = row0 + wg * kRowsPerWave + (lane & 31);
                const int kr = pc - wg * MT * 4;
                h = it.g * G + R % G;
                tq = (int64_t)it.t0 + R / G;
                d0 = 8 * kr + 4 * (lane >> 5);
                ok = R < rows_total;
            }
            if (!ok || tq >= T) continue;            // (lanes without a row)
            // W chunks per pass, their loads in flight together (a chunk past the last is
            // reread with weight 0); the running sums are rescaled between passes.
            float M = -INFINITY, L = 0.f;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            auto merge = [&](auto width) __attribute__((always_inline)) {
                constexpr int W = decltype(width)::value;
                for (int k0 = 0; k0 < ns; k0 += W) {
                    f32x2 ml[W];
                    f32x4 o[W];
#pragma unroll
                    for (int i = 0; i < W; ++i) {
                        const int64_t pt = part0 - min(k0 + i, ns - 1);
                        ml[i] = pml[pt * (kSplitPartML / 8) + wg * 64 + lane];
                        o[i] = po[pt * (kSplitPartO / 16) + pc * 64 + lane];
                    }
                    // -inf after a pass only if every score so far is (overflowed products): its
                    // chunks then weigh 0, as in an unsplit launch
                    float Mn = M;
#pragma unroll
                    for (int i = 0; i < W; ++i) Mn = fmaxf(Mn, ml[i][0]);
                    const float r = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((M - Mn) * c);
                    M = Mn;
                    L *= r;
                    acc *= r;
#pragma unroll
                    for (int i = 0; i < W; ++i) {
                        const float w = k0 + i < ns && ml[i][0] != -INFINITY
                                            ? __builtin_amdgcn_exp2f((ml[i][0] - M) * c) : 0.f;
                        L += w * ml[i][1];
                        acc += w * o[i];
                    }
                }
            };
            if (ns <= 4) merge(std::integral_constant<int, 4>{});
            else merge(std::integral_constant<int, 16>{});
            const bf16x4 bv = __builtin_convertvector(acc * (1.f / L), bf16x4);
            *reinterpret_cast<u32x2 *>(out + (tq * Hq + h) * D + d0) = __builtin_bit_cast(u32x2, bv);
        }
    }
    // This workgroup is through with the slot: it only reads it, and every read has returned
    // its value before the barrier.
    __syncthreads();
    if (threadIdx.x == 0)
        __hip_atomic_fetch_add(&split_control.done[slot][blockIdx.x % kXcds][0], 1u, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace

int attn_rows_per_workgroup(int) { return kRowsPerWG; }

namespace {
// Schedule override (pcr_prefill_attn_set_schedule): 0 chooses per launch.
std::atomic<int> g_schedule{PCR_ATTN_SCHEDULE_AUTO};

// The number of a key-split launch: never one that an earlier launch of the process had
// (48 bits are not used up).
uint64_t next_launch()
{
    static std::atomic<uint64_t> n{0};
    return n.fetch_add(1, std::memory_order_relaxed) + 1;
}

// Enqueues a kernel and returns this launch's own error (hipGetLastError may hold an older one).
template <class T> struct Same { typedef T type; };   // (a parameter's type comes from the kernel alone)
template <class... P>
hipError_t enqueue(void (*kernel)(P...), dim3 grid, int threads, hipStream_t s, const typename Same<P>::type &...a)
{
    void *args[] = {const_cast<void *>(static_cast<const void *>(&a))...};
    return hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, dim3(threads), args, 0, s);
}

template <int D, int MODE>
void launch_attn(dim3 grid, hipStream_t s, const u16 *qq, const u16 *pk, const u16 *pv, const pcr_kv_pool &pool,
                 const int32_t *block_tables, int32_t max_blocks, int32_t num_q_heads, int32_t T, float scale_log2,
                 float rescale_thr, u16 *oo, const AttnWorkMap &wm)
{
    hipLaunchKernelGGL((prefill_attn_kernel<D, MODE>), grid, dim3(kThreads), 0, s, qq, pk, pv, pool.num_blocks,
                       pool.num_kv_heads, block_tables, max_blocks, num_q_heads, T, scale_log2, rescale_thr, oo,
                       wm);
}

// Key split of a key-halves launch: the key tiles of an item, or 0 for none. A launch of
// few workgroups (a short suffix on a long prefix, one GPU's share of the heads) leaves
// compute units idle while each workgroup walks every key; cutting the row tiles' keys
// into chunks gives each compute unit one item. The chunk is the smallest one whose
// items still fit the compute units (and the scratch) in one round.
// It is taken when it is estimated to take 6% less than the launch as a whole, per call
// among others. In us, with f and g the shares of the compute units that have an item
// whole and split, and L and c the key tiles of the longest row and of a chunk, row tiles of
// 128 dims take 8.7 + (0.53 + 0.19 f) L whole and 18 + (0.40 + 0.46 g) c split, decode rows 5.5 + (0.59 +
// 0.20 f) L and 16.5 + (0.26 + 0.65 g) c; with 64 dims 6.9 + (0.51 + 0.09 f) L and 16.5 + (0.44 +
// 0.12 g) c, and 4.7 + (0.29 + 0.12 f) L and 15.5 + (0.31 + 0.06 g) c (fitted to 800 launches, within
// 3% whole and 7% split; a full chip runs at a lower clock, and the three launches of a split
// call are host-bound below 16 us). Measured (32 query / 8 kv heads of 128, whole ->
// split): 43 new tokens on 7985 cached 77 -> 23 us; 16 on 2000 25 -> 18; 128 on 4000 44.5 ->
// 24; 2 on 16000 143 -> 25; 1024 on 15360 twice with 8 / 1 heads 150 -> 124. On the 800, of 20 to
// 140 tiles, one split launch is more than 1% slower than whole, by 2%; 14 tiles above 4/3
// chunk as the line, whatever the rows and dims, had 73 slower ones, up to 57% (a decode
// row of 64 dims on 1250 keys). (Chunks of at least 4, 6, 8, 12 or 16 tiles: 4 to 8 alike, 12
// and 16 up to 20% slower on prefixes of 2k.)
int32_t split_chunk(const int32_t *seq, int n, const int32_t *host_prefix_lens, const int32_t *host_cu_suffix, int G,
                    int Hkv, int D, int n_cu)
{
    const int64_t cap = std::min(n_cu, kSplitParts);
    int32_t longest[2] = {0, 0};             // key tiles: of the row tiles, of the decode rows
    for (int k = 0; k < n; ++k) {
        const int32_t b = seq[k], sb = host_cu_suffix[b + 1] - host_cu_suffix[b];
        int32_t &l = longest[sb == 1 && G <= decode_wave::kMaxCols];
        l = std::max(l, key_tiles(host_prefix_lens[b] + sb - 1));
    }
    auto items = [&](int32_t c) {            // of chunks of c tiles (0: whole)
        int64_t w = 0;
        for (int k = 0; k < n; ++k) {
            const int32_t b = seq[k], sb = host_cu_suffix[b + 1] - host_cu_suffix[b];
            w += ((int64_t)sb * G + kRowsPerWG - 1) / kRowsPerWG *
                 (c ? (key_tiles(host_prefix_lens[b] + sb - 1) + c - 1) / c : 1);
        }
        return w * Hkv;
    };
    int32_t lo = kSplitMinChunk, hi = (std::max(longest[0], longest[1]) - 14) * 3 / 4;   // (never taken above)
    if (lo > hi || items(hi) > cap) return 0;
    while (lo < hi) {
        const int32_t mid = lo + (hi - lo) / 2;
        if (items(mid) <= cap) hi = mid; else lo = mid + 1;
    }
    static const float kTime[2][2][6] = {    // [64 dims, 128][row tile, decode row]
        {{6.9f, 0.51f, 0.09f, 16.5f, 0.44f, 0.12f}, {4.7f, 0.29f, 0.12f, 15.5f, 0.31f, 0.06f}},
        {{8.7f, 0.53f, 0.19f, 18.f, 0.40f, 0.46f}, {5.5f, 0.59f, 0.20f, 16.5f, 0.26f, 0.65f}}};
    const float f = (float)items(0) / n_cu, g = (float)items(hi) / n_cu;
    float whole = 0.f, split = 0.f;
    for (int kind = 0; kind < 2; ++kind) {
        if (!longest[kind]) continue;
        const float *t = kTime[D == 128][kind];
        whole = std::max(whole, t[0] + (t[1] + t[2] * f) * longest[kind]);
        split = std::max(split, t[3] + (t[4] + t[5] * g) * std::min(hi, longest[kind]));
    }
    return split < 0.94f * whole ? hi : 0;
}

// Estimated time in us of a launch on row tiles of rpw rows (128: key halves, 256: row
// halves) over the sequences in launch order. An item takes a fixed part plus its key
// tiles: with 128 dims (64 dims) 7.3 (5.6) us and 0.79 (0.57) a tile with key halves, 10 (7.6)
// and 1.45 (0.99) with row halves, where one copy of a tile serves twice the rows; a
// decode row 5 (3.6) and 0.98 (0.45) per 64 keys. With `simulate` (at most kSimItems items) each
// XCD's items are dealt in launch order to whichever of its compute units is free first,
// as the hardware does: sequences of short prefixes have items of 2 to 30 tiles, and the
// mean of them says little about the last to end. While compute units idle the others
// run at a higher clock (the power they leave): idle time counts 70% (88%). Without
// `simulate`: the work over the compute units, for launches of many rounds.
// Measured on 440 launches of 1 to 9 rounds (8 to 96 query / 1 to 8 kv heads, ragged and not,
// decode rows among them): the choice below loses 0.4% against always the faster one and
// 1.2% at worst against the line of two row-halves items per compute unit, which itself loses 3.7%;
// an estimate from the items' mean lost up to 11% against that line in 29 of them, and
// 30% on two sequences of 2100 new tokens on 90 cached with 28 / 4 heads (103 -> 79 us).
constexpr int kSimItems = 1024;
double schedule_time(const int32_t *order, int n, const int32_t *host_prefix_lens, const int32_t *host_cu_suffix,
                     int G, int Hkv, int D, int rpw, int n_cu, bool simulate)
{
    const bool rows = rpw > kRowsPerWG, wide = D == 128;
    const float fixed = rows ? (wide ? 10.f : 7.6f) : (wide ? 7.3f : 5.6f);
    const float tile = rows ? (wide ? 1.45f : 0.99f) : (wide ? 0.79f : 0.57f);
    const float dec_fixed = wide ? 5.f : 3.6f, dec_tile = wide ? 0.98f : 0.45f;
    float cost[kSimItems];                   // one kv head's items
    int items = 0;
    double total = 0.0;
    for (int k = 0; k < n; ++k) {
        const int32_t b = order[k], p = host_prefix_lens[b], sb = host_cu_suffix[b + 1] - host_cu_suffix[b];
        if (sb == 1 && G <= decode_wave::kMaxCols) {
            const float t = dec_fixed + dec_tile * key_tiles(p);
            total += t;
            if (simulate) cost[items++] = t;
            continue;
        }
        const int64_t r = (int64_t)sb * G, nt = (r + rpw - 1) / rpw;
        if (!simulate) {
            const int first = key_tiles(p + (int)((std::min<int64_t>(r, rpw) - 1) / G)), last = key_tiles(p + sb - 1);
            total += nt * (fixed + tile * 0.5 * (first + last));
            continue;
        }
        for (int64_t t = nt - 1; t >= 0; --t) {
            cost[items++] = fixed + tile * key_tiles(p + (int)((std::min<int64_t>(r, (t + 1) * rpw) - 1) / G));
        }
    }
    if (!simulate) return total * Hkv / n_cu;
    const int n_xcd_cu = std::max(1, std::min(n_cu / kXcds, 64));
    const float idle = wide ? 0.70f : 0.88f;
    // As locate_item deals them: whole heads to each XCD (then all eight do the same), or
    // an eighth of all items.
    const bool whole = Hkv % kXcds == 0;
    const int all = items * Hkv, per = whole ? all / kXcds : (all + kXcds - 1) / kXcds;
    float longest = 0.f;
    for (int x = 0; x < (whole ? 1 : kXcds); ++x) {
        float end[64] = {};                  // a heap: when each compute unit is free
        float sum = 0.f, last = 0.f;
        int at = (x * per) % items;
        for (int w = x * per; w < std::min(all, (x + 1) * per); ++w) {
            const float c = cost[at], t = end[0] + c;
            at = at + 1 == items ? 0 : at + 1;
            sum += c;
            last = std::max(last, t);
            int i = 0;
            for (int c1; (c1 = 2 * i + 1) < n_xcd_cu; i = c1) {
                if (c1 + 1 < n_xcd_cu && end[c1 + 1] < end[c1]) ++c1;
                if (end[c1] >= t) break;
                end[i] = end[c1];
            }
            end[i] = t;
        }
        longest = std::max(longest, idle * last + (1.f - idle) * sum / n_xcd_cu);
    }
    return longest;
}

// One launch over the sequences seq[0..n) (each with new tokens, n <= kMaxMapSeqs,
// longest context first): builds the work map, picks the schedule, launches.
hipError_t launch_group(const int32_t *seq, int n, const u16 *qq, const pcr_kv_pool &pool,
                        const int32_t *block_tables, int32_t max_blocks, const int32_t *host_prefix_lens,
                        const int32_t *host_cu_suffix, int32_t num_q_heads, int32_t T, float scale_log2,
                        float rescale_thr, u16 *oo, hipStream_t s, int auto_schedule, int n_cu, bool can_split)
{
    const int Hkv = pool.num_kv_heads, G = num_q_heads / Hkv;
    auto rows_of = [&](int32_t b) { return ((int64_t)host_cu_suffix[b + 1] - host_cu_suffix[b]) * G; };
    const int sched = g_schedule.load(std::memory_order_relaxed);
    const bool prefer_keys = auto_schedule == PCR_ATTN_SCHEDULE_KEY_HALVES;
    // Slot order: the given order (longest context first), with the decode rows (one
    // new token, one workgroup each, bound by HBM) spread evenly over the prefill
    // tiles (bound by the matrix cores): run back to back they would take every
    // compute unit at once and queue on HBM.
    auto slot_order = [&](auto tiles_of, int32_t *order) {
        const bool dec_rows = G <= decode_wave::kMaxCols;
        int32_t pre[kMaxMapSeqs], dec[kMaxMapSeqs];
        int np = 0, nd = 0;
        int64_t pre_tiles = 0;
        for (int k = 0; k < n; ++k) {
            if (dec_rows && rows_of(seq[k]) == G) {
                dec[nd++] = seq[k];
            } else {
                pre[np++] = seq[k];
                pre_tiles += tiles_of(seq[k]);
            }
        }
        int m = 0, di = 0;
        int64_t done = 0;
        for (int k = 0; k < np; ++k) {
            order[m++] = pre[k];
            done += tiles_of(pre[k]);
            for (; di < nd && (int64_t)di * pre_tiles < (int64_t)nd * done; ++di) order[m++] = dec[di];
        }
        for (; di < nd; ++di) order[m++] = dec[di];
    };

    // More key-halves items than compute units: row halves from two of their items per
    // compute unit on (each then pays its start and end for twice the work), and on either
    // side of that line the other schedule when it is estimated to take 4% less. Key
    // halves win where the fewer row-halves items leave more of the last round idle, and
    // where the suffixes are shorter than their tiles. A caller that prefers key halves (whose
    // shorter workgroups free a compute unit sooner for copy kernels that share the device)
    // gets row halves only if they are estimated so and all fit the compute units at once.
    // Against the line alone (32 query / 8 kv heads of 128): 64 sequences of 32 new tokens on
    // 3000 cached 200 -> 154 us (key halves), 16 of 128 on 4096 142 -> 129 (row halves), one of
    // 1280 on 8192 199 -> 180.
    bool rows = sched == PCR_ATTN_SCHEDULE_ROW_HALVES;
    if (sched == PCR_ATTN_SCHEDULE_AUTO) {
        int64_t tiles = 0, tiles2 = 0;   // row tiles of 128 and of 256 rows, all kv heads
        for (int k = 0; k < n; ++k) {
            tiles += (rows_of(seq[k]) + kRowsPerWG - 1) / kRowsPerWG;
            tiles2 += (rows_of(seq[k]) + 2 * kRowsPerWG - 1) / (2 * kRowsPerWG);
        }
        tiles *= Hkv;
        tiles2 *= Hkv;
        if (tiles > n_cu && (!prefer_keys || tiles2 <= n_cu)) {
            const bool simulate = tiles <= std::min(4 * n_cu, kSimItems);
            auto time_of = [&](int rpw) {
                int32_t order[kMaxMapSeqs];
                slot_order([&](int32_t b) { return (rows_of(b) + rpw - 1) / rpw; }, order);
                return schedule_time(order, n, host_prefix_lens, host_cu_suffix, G, Hkv, pool.head_dim, rpw, n_cu,
                                     simulate);
            };
            const bool line = tiles2 >= 2 * (int64_t)n_cu;
            rows = time_of(2 * kRowsPerWG) < (line ? 1.04 : 0.96) * time_of(kRowsPerWG);
        }
    }
    const int64_t rpw = rows ? 2 * kRowsPerWG : kRowsPerWG;
    // Key tiles per item, 0: no key split.
    const int32_t chunk =
        sched == PCR_ATTN_SCHEDULE_AUTO && !prefer_keys && !rows && can_split
            ? split_chunk(seq, n, host_prefix_lens, host_cu_suffix, G, Hkv, pool.head_dim, n_cu)
            : 0;
    auto keys_of = [&](int32_t b) { return host_prefix_lens[b] + host_cu_suffix[b + 1] - host_cu_suffix[b]; };
    auto tiles_of = [&](int32_t b) {
        const int64_t t = (rows_of(b) + rpw - 1) / rpw;
        return chunk ? t * ((key_tiles(keys_of(b) - 1) + chunk - 1) / chunk) : t;
    };

    AttnWorkMap wm;
    slot_order(tiles_of, wm.seq);
    int32_t cum = 0;
    for (int k = 0; k < n; ++k) {
        const int32_t b = wm.seq[k];
        cum += (int32_t)tiles_of(b);
        wm.tiles_end[k] = cum;
        wm.prefix[k] = host_prefix_lens[b];
        wm.first[k] = host_cu_suffix[b];
        wm.count[k] = host_cu_suffix[b + 1] - host_cu_suffix[b];
    }
    wm.n_seq = n;
    wm.per_head = cum;
    wm.chunk = chunk;
    wm.launch = chunk ? next_launch() : 0;
    const int64_t n_items = (Hkv % kXcds == 0) ? (int64_t)cum * Hkv : ((int64_t)cum * Hkv + kXcds - 1) / kXcds * kXcds;
    const dim3 grid((unsigned)n_items);
    auto *pk = static_cast<const u16 *>(pool.k);
    auto *pv = static_cast<const u16 *>(pool.v);
    auto launch = [&](auto dim) -> hipError_t {
        constexpr int D = decltype(dim)::value;
        auto attn = [&](auto mode) {
            launch_attn<D, decltype(mode)::value>(grid, s, qq, pk, pv, pool, block_tables, max_blocks, num_q_heads,
                                                  T, scale_log2, rescale_thr, oo, wm);
        };
        if (rows) {
            attn(std::integral_constant<int, kRowHalves>{});
        } else if (!chunk) {
            attn(std::integral_constant<int, kKeyHalves>{});
        } else {
            // (the grid is a multiple of the XCD count) A claim without its combine kernel
            // would hold its slot for good.
            const unsigned per_xcd = grid.x / kXcds;
            hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
            hipError_t e = s ? hipStreamIsCapturing(s, &capture) : hipSuccess;   // (the null stream never is)
            if (e != hipSuccess) return e;
            e = enqueue(capture == hipStreamCaptureStatusNone ? split_claim_kernel : split_claim_replay_kernel,
                        dim3(1), 64, s, wm.launch, per_xcd);
            if (e != hipSuccess) return e;
            e = enqueue(prefill_attn_kernel<D, kKeySplit>, grid, kThreads, s, qq, pk, pv, pool.num_blocks, Hkv,
                        block_tables, max_blocks, num_q_heads, T, scale_log2, rescale_thr, oo, wm);
            if (e == hipSuccess)
                e = enqueue(split_combine_kernel<D>, grid, kCombineThreads, s, Hkv, num_q_heads, T, scale_log2, oo,
                            wm);
            if (e != hipSuccess) {
                (void)enqueue(split_release_kernel, dim3(1), 64, s, wm.launch, per_xcd);
                return e;
            }
        }
        return hipGetLastError();
    };
    if (pool.head_dim == 128) return launch(std::integral_constant<int, 128>{});
    return launch(std::integral_constant<int, 64>{});
}
}  // namespace

void attn_set_schedule(int schedule) { g_schedule.store(schedule, std::memory_order_relaxed); }

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_hold_mu;
uint64_t g_held[kMaxDevices][kSplitSlots];   // numbers under which attn_hold_scratch claimed; 0: none
}  // namespace

hipError_t attn_hold_scratch(int n, int *free_entries)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess && (dev < 0 || dev >= kMaxDevices)) e = hipErrorInvalidDevice;
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lk(g_hold_mu);
    // Each slot is claimed twice under its number, as by two overlapping replays of one
    // captured launch, and given back twice.
    for (uint64_t &id : g_held[dev]) {
        for (int k = 0; k < 2 && id && e == hipSuccess; ++k)
            e = enqueue(split_release_kernel, dim3(1), 64, nullptr, id, 1u);
        id = 0;
    }
    for (int i = 0; i < n && i < kSplitSlots && e == hipSuccess; ++i) {
        g_held[dev][i] = next_launch();
        for (int k = 0; k < 2 && e == hipSuccess; ++k)
            e = enqueue(split_claim_replay_kernel, dim3(1), 64, nullptr, g_held[dev][i], 1u);
    }
    if (e == hipSuccess) e = hipDeviceSynchronize();
    static SplitControl c;                   // (under the mutex)
    if (e == hipSuccess) e = hipMemcpyFromSymbol(&c, HIP_SYMBOL(split_control), sizeof(c));
    if (e != hipSuccess) return e;
    *free_entries = 0;
    for (int s = 0; s < kSplitEntries; ++s) {
        bool through = true;
        for (int x = 0; x < kXcds; ++x) through = through && (c.done[s][x][0] & 0xFFFFu) == (c.owner[s] & 0xFFFFu);
        *free_entries += through;
    }
    return hipSuccess;
}

hipError_t launch_prefix_prefill_attn(const void *q, const pcr_kv_pool &pool,
                                      const int32_t *block_tables, int32_t max_blocks,
                                      const int32_t *host_prefix_lens, const int32_t *host_cu_suffix,
                                      int32_t B, int32_t num_q_heads, int32_t T, float sm_scale, void *out,
                                      hipStream_t s, int auto_schedule, int n_cu)
{
    // The sequences with new tokens, longest context first.
    std::vector<int32_t> seq;
    seq.reserve((size_t)std::max(B, 0));
    for (int32_t b = 0; b < B; ++b)
        if (host_cu_suffix[b + 1] > host_cu_suffix[b]) seq.push_back(b);
    if (seq.empty()) return hipSuccess;
    auto keys = [&](int32_t b) { return (int64_t)host_prefix_lens[b] + host_cu_suffix[b + 1] - host_cu_suffix[b]; };
    std::stable_sort(seq.begin(), seq.end(), [&](int32_t a, int32_t c) { return keys(a) > keys(c); });
    const float scale_log2 = sm_scale * kLog2e;
    const float rescale_thr = kRescaleThreshold / scale_log2;   // in units of <q,k>
    auto *qq = static_cast<const u16 *>(q);
    auto *oo = static_cast<u16 *>(out);
    // More sequences than one work map holds: consecutive launches on the stream, the
    // sequences dealt round robin (sequence k of the sorted list to launch k mod
    // n_launch), so that every launch gets the same mix of long and short ones.
    const int n_act = (int)seq.size();
    const int n_launch = (n_act + kMaxMapSeqs - 1) / kMaxMapSeqs;
    int32_t group[kMaxMapSeqs];
    // A key-split launch's chunks read q until its combine kernel writes out, and its rows
    // that need no merge are written beside them: not for outputs that overlap q.
    const uintptr_t qa = (uintptr_t)q, oa = (uintptr_t)out;
    const uintptr_t bytes = (uintptr_t)T * num_q_heads * pool.head_dim * 2;
    const bool can_split = n_launch == 1 && (qa + bytes <= oa || oa + bytes <= qa);
    for (int l = 0; l < n_launch; ++l) {
        int n = 0;
        for (int k = l; k < n_act; k += n_launch) group[n++] = seq[k];
        const hipError_t e = launch_group(group, n, qq, pool, block_tables, max_blocks, host_prefix_lens,
                                          host_cu_suffix, num_q_heads, T, scale_log2, rescale_thr, oo, s,
                                          auto_schedule, n_cu, can_split);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace pcr
