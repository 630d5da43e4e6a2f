// KV data-movement kernels for gfx950: append (new K/V rows into pool slots),
// gather (pool back to logical order) and the host-pull block copy.
//
// All three are pure bit movement; every access is 16 bytes wide where the
// layout allows, and every block id or slot read from device memory is
// range-checked in the kernel before use, so a bad table entry skips its row
// rather than touching memory outside the pool.
#include <type_traits>

#include "pcr_internal.h"

namespace pcr {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16;

// Output rows per gather workgroup: 16 and 64 were 2-5% slower on 268 MB, 16 20% on two
// kv heads.
constexpr int kGatherTile = 32;
// Bytes of input (append) or output (gather) above which both go past the caches: non-
// temporal loads and, for gather, stores. Appends of 16k, 20k and 32k tokens of 8 kv heads
// of 128 (4 KB a token), ordinary -> non-temporal loads: 40 -> 31, 49 -> 39 and 72 -> 61 us
// when the input has left the caches; 25 -> 28, 31 -> 35 and 49 -> 54 in ragged sequences,
// 22 -> 22, 27 -> 27 and 45 -> 49 in aligned ones, when the layer's passes have just written
// it (28, 34, 54 and 22, 27, 44 with tiles cut at token 32). 16k tokens, the line itself, whose
// input and output fill half of the 256 MB cache, lose 3 us when they are appended again
// and again (22 -> 25 aligned, 25 -> 28 ragged), and smaller inputs 12-20% (14-33 MB).
constexpr int64_t kNtBytes = 64ll << 20;
// Output bytes up to which gather runs one thread per 16 bytes of a row (gather_rows_kernel).
constexpr int64_t kGatherRowsBytes = 4ll << 20;
// Append workgroups up to which each requests the rows it may take after its tile with the
// tile's own rows (append_kv_kernel).
constexpr int kAppendEarly = 256;
// New tokens per append workgroup: 32 measured as fast as 16 on block-aligned slot lists
// and 31% faster on the RAG mix's (whose tiles start inside chunks); 64 was 3.5% slower
// on aligned lists of 128k tokens.
constexpr int kAppendTile = 32;

// ---------------------------------------------------------------------------
// append: grid (ceil(T/TILE), Hkv), 256 threads. One workgroup writes about TILE new
// tokens of one kv head. K rows are copied 16 B at a time. V is written d-major
// inside each block: the tile's V rows go through LDS, and each aligned run of 8
// slots of one dim (a 16-byte chunk of a block's V) that the tile's tokens fill is
// written by one 16-byte store. A chunk the tile fills only in part (a run of
// slots that starts or ends inside it) gets element stores for its filled slots.
// Tokens that go on inside the pool block of the token before the tile belong to the
// tile before, so a tile leaves out up to 15 tokens at its start and takes up to 15
// after its end: no block is written by two workgroups, whose XCDs' L2s would each write
// parts of its lines, and chunks are cut only where a sequence starts or ends in them.
// (18480 tokens of 60 ragged sequences, 151 MB: 39.2 us with tiles cut at token 32,
// 35.8 with whole blocks, 31.9 = 4.7 TB/s with the non-temporal loads; 32 x 1024 aligned
// tokens, 268 MB, 56 us = 4.8 TB/s either way. A 256 MB device copy runs at 5.4.)
// NT: the input rows are read with non-temporal loads. (The pool is written with
// ordinary stores, which merge a block's 16-byte chunks into lines in the L2:
// non-temporal ones took 1.5 to 2 times as long.)
// EARLY: the rows after the tile are requested with the tile's, before the slots say whether
// they are this tile's, since a second round trip to memory is what a small call waits for
// (64 tokens of 8 kv heads 4.6 -> 4.2 us, of 64 dims 4.0 -> 3.6; 1024 ragged ones 5.3 -> 5.0). With more
// workgroups than compute units the extra reads cost more (4096 ragged tokens of 64 dims
// 6.1 -> 6.6).
// ---------------------------------------------------------------------------
template <int D, int TILE, bool NT, bool EARLY>
__global__ __launch_bounds__(256) void append_kv_kernel(
    u16 *__restrict__ pool_k, u16 *__restrict__ pool_v, int32_t num_blocks, int32_t Hkv,
    const u16 *__restrict__ k_new, const u16 *__restrict__ v_new,
    const int32_t *__restrict__ slot_mapping, int32_t T)
{
    constexpr int EXT = kBlockSize - 1;        // tokens after the tile it may take
    constexpr int ROWS = TILE + EXT;
    static_assert(ROWS < 64, "one wave ranks the chunk runs");
    static_assert(TILE >= kBlockSize, "a tile starts a block");
    constexpr int CPR = D / 8;                 // 16-B chunks per row
    constexpr int NCH = (TILE * CPR + 255) / 256;
    static_assert(EXT * CPR <= 256, "one chunk of the rows after the tile per thread");
    __shared__ __attribute__((aligned(16))) u16 vs[ROWS][D + 8];   // +8 elements: stagger rows across banks
    __shared__ int32_t slots[ROWS];            // -1: no slot, or another tile's
    __shared__ int32_t runs[ROWS];             // (first token << 8) | tokens, one per chunk run
    __shared__ int32_t n_runs, n_rows;

    const int tile = blockIdx.x, g = blockIdx.y, tid = threadIdx.x;
    const int tok0 = tile * TILE;

    auto load = [&](const u16 *src) __attribute__((always_inline)) -> u32x4 {
        auto *p = reinterpret_cast<const u32x4 *>(src);
        if constexpr (NT) return __builtin_nontemporal_load(p);
        return *p;
    };
    // The tile's K/V rows do not depend on the slot list: their loads go out first, so the
    // two memory round trips (slots, rows) overlap.
    u32x4 kv[NCH], vv[NCH];
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int c = tid + 256 * i, r = c / CPR, cc = c % CPR;
        kv[i] = u32x4{0u, 0u, 0u, 0u};
        vv[i] = u32x4{0u, 0u, 0u, 0u};
        if (c < TILE * CPR && tok0 + r < T) {
            const int64_t src = ((int64_t)(tok0 + r) * Hkv + g) * D + cc * 8;
            kv[i] = load(k_new + src);
            vv[i] = load(v_new + src);
        }
    }
    u32x4 ke = {0u, 0u, 0u, 0u}, ve = {0u, 0u, 0u, 0u};
    const int re = TILE + tid / CPR, ce = tid % CPR;   // this thread's chunk of the rows after the tile
    auto load_ext = [&]() __attribute__((always_inline)) {
        const int64_t src = ((int64_t)(tok0 + re) * Hkv + g) * D + ce * 8;
        ke = load(k_new + src);
        ve = load(v_new + src);
    };
    if constexpr (EARLY) {
        if (re < ROWS && tok0 + re < T) load_ext();
    }
    int32_t sl = -1;                           // wave 0: the slot of token tok0 + tid
    bool follows = false;                      // and whether it follows the token before's
    if (tid < 64) {
        // Lane 63 reads the slot of the token before the tile (all slots in one load).
        const int t = tid == 63 ? tok0 - 1 : tok0 + tid;
        if ((tid < ROWS || tid == 63) && t >= 0 && t < T) {
            sl = slot_mapping[t];
            if (sl < 0 || sl / kBlockSize >= num_blocks) sl = -1;
        }
        // the slot of the token before this one (the wave rotated by one lane: DPP wave_ror:1)
        const int32_t before = __builtin_amdgcn_update_dpp(sl, sl, 0x13C, 0xf, 0xf, false);
        if (tid == 63) sl = -1;
        follows = sl >= 0 && before >= 0 && sl == before + 1;
        // heads: tokens that do not go on inside the block of the token before them. The
        // tile's own tokens run from its first head to the first head at or after its end
        // (both within 15 tokens: a block has 16 slots).
        const uint64_t heads = ~__builtin_amdgcn_ballot_w64(follows && sl % kBlockSize != 0);
        const uint64_t rest = heads >> TILE;
        const int first = (int)__builtin_ctzll(heads);
        const int last = rest ? min(ROWS, TILE + (int)__builtin_ctzll(rest)) : ROWS;
        if (tid < first || tid >= last) sl = -1;
        if (tid < ROWS) slots[tid] = sl;
        if (tid == 0) n_rows = last;
    }
    __syncthreads();

    auto put_row = [&](int r, int cc, u32x4 kw, u32x4 vw) __attribute__((always_inline)) {
        const int32_t s0 = slots[r];
        if (s0 < 0) return;
        *reinterpret_cast<u32x4 *>(&vs[r][cc * 8]) = vw;
        const int64_t blk = s0 / kBlockSize, o = s0 % kBlockSize;
        *reinterpret_cast<u32x4 *>(pool_k + ((blk * Hkv + g) * kBlockSize + o) * D + cc * 8) = kw;
    };
    const bool ext = re < n_rows;
    if constexpr (!EARLY) {
        if (ext) load_ext();
    }
    if (tid < 64) {                            // wave 0: the chunk runs
        // A token starts a chunk run when its slot is valid and either opens an aligned chunk
        // of 8 slots or does not follow the previous token's slot; the run goes on over the
        // following tokens until the next start or invalid slot (a continuing token's slot
        // is its predecessor's plus one, inside the same chunk).
        const bool valid = sl >= 0;
        const bool start = valid && (tid == 0 || sl % 8 == 0 || !follows);
        const uint64_t starts = __builtin_amdgcn_ballot_w64(start);
        const uint64_t stops = starts | ~__builtin_amdgcn_ballot_w64(valid);   // bits past ROWS are stops
        if (start) {
            const uint64_t after = tid == 63 ? 0ull : stops >> (tid + 1);
            const int len = after ? 1 + __builtin_ctzll(after) : 64 - tid;
            const int idx = __builtin_popcountll(starts & ((1ull << tid) - 1ull));
            runs[idx] = (tid << 8) | len;
        }
        if (tid == 0) n_runs = __builtin_popcountll(starts);
    }
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int c = tid + 256 * i;
        if (c < TILE * CPR) put_row(c / CPR, c % CPR, kv[i], vv[i]);
    }
    if (ext) put_row(re, ce, ke, ve);
    __syncthreads();

    // V: task = (run, dim)
    const int nr = n_runs;
    for (int task = tid; task < nr * D; task += 256) {
        const int k = task / D, x = task % D;
        const int rv = runs[k], r0 = rv >> 8, len = rv & 0xff;
        const int32_t s0 = slots[r0];
        const int64_t blk = s0 / kBlockSize, o = s0 % kBlockSize;
        u16 *dst = pool_v + ((blk * Hkv + g) * D + x) * kBlockSize + o;
        if (len == 8) {   // a whole aligned chunk (a run of 8 starts at a multiple of 8)
            u16 e[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) e[j] = vs[r0 + j][x];
            u32x4 w;
            w.x = e[0] | ((unsigned)e[1] << 16);
            w.y = e[2] | ((unsigned)e[3] << 16);
            w.z = e[4] | ((unsigned)e[5] << 16);
            w.w = e[6] | ((unsigned)e[7] << 16);
            *reinterpret_cast<u32x4 *>(dst) = w;
        } else {
            for (int j = 0; j < len; ++j) dst[j] = vs[r0 + j][x];
        }
    }
}

// ---------------------------------------------------------------------------
// gather: grid (ceil(total/TILE), Hkv), 256 threads; out rows in logical order. One
// workgroup reads TILE output rows of one kv head. K rows are copied 16 B at a time.
// V is d-major inside a block: each aligned chunk of 8 slots of one dim that the tile's
// rows use is read by one 16-byte load (two dims per task), its elements go through LDS,
// and the rows leave it 16 B at a time. Bound by moving the bytes: 19897 ragged tokens
// (163 MB) 58.5 us when V was read by eight 2-byte loads per 16 bytes of output, 39 with
// whole chunks, 31.4 with non-temporal stores, 30.5 = 5.3 TB/s with the K loads
// non-temporal too (NT; V loads stay ordinary: a line's two 16-byte halves are read by
// different tasks, and bypassing the caches took 41 us); 268 MB of aligned tokens
// 99.5 -> 45 us = 5.9 TB/s. Output that passes the caches by costs its reader: gather and a
// kernel that reads its output together, with input out of the caches, took 42 us for 8192
// tokens of 8 kv heads of 128 by 2-byte loads, 43 with non-temporal stores, 38 without;
// 16384 (67 MB out) 82, 73, 68, 65536 308, 224, 222; with cached input 16384 65, 48, 48, 32768
// 151, 93, 103. So they start above kNtBytes.
// A row whose block is not in the pool or past the table is written as zeros.
// ---------------------------------------------------------------------------
template <int D, int TILE, bool NT>
__global__ __launch_bounds__(256) void gather_kv_kernel(
    const u16 *__restrict__ pool_k, const u16 *__restrict__ pool_v, int32_t num_blocks, int32_t Hkv,
    const int32_t *__restrict__ block_tables, int32_t max_blocks,
    const int32_t *__restrict__ starts, const int32_t *__restrict__ cu_out, int32_t B,
    int32_t total, u16 *__restrict__ k_out, u16 *__restrict__ v_out)
{
    static_assert(TILE <= 64, "one wave ranks the chunk runs");
    constexpr int CPR = D / 8;                 // 16-B chunks per row
    constexpr int NCH = (TILE * CPR + 255) / 256;
    __shared__ __attribute__((aligned(16))) u16 vs[TILE][D + 8];
    __shared__ int32_t blks[TILE];             // pool block of each row, -1: none
    __shared__ int32_t offs[TILE];             // slot inside the block
    __shared__ int32_t runs[TILE];             // (first row << 8) | rows, one per chunk run
    __shared__ int32_t n_runs;

    const int g = blockIdx.y, tid = threadIdx.x;
    const int row0 = blockIdx.x * TILE;
    auto put = [&](u16 *dst, u32x4 v) __attribute__((always_inline)) {
        if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(dst));
        else *reinterpret_cast<u32x4 *>(dst) = v;
    };
    if (tid < 64) {                            // wave 0: where each row lies, and the chunk runs
        const int r = row0 + tid;
        int32_t blk = -1, o = 0;
        if (tid < TILE && r < total) {
            int lo = 0, hi = B - 1;            // sequence b with cu_out[b] <= r < cu_out[b+1]
            while (lo < hi) {
                const int mid = (lo + hi + 1) / 2;
                if (cu_out[mid] <= r) lo = mid; else hi = mid - 1;
            }
            const int t = starts[lo] + (r - cu_out[lo]);
            if (t >= 0 && t / kBlockSize < max_blocks) {
                const int32_t id = block_tables[(int64_t)lo * max_blocks + t / kBlockSize];
                if (id >= 0 && id < num_blocks) {
                    blk = id;
                    o = t % kBlockSize;
                }
            }
        }
        // A row starts a run when it has a block and opens an aligned chunk of 8 slots or
        // does not follow the previous row's slot; the run goes on to the next start or
        // row without a block.
        const int32_t pb = __shfl_up(blk, 1), po = __shfl_up(o, 1);
        const bool valid = blk >= 0;
        const bool start = valid && (tid == 0 || o % 8 == 0 || pb != blk || po != o - 1);
        const uint64_t starts_m = __builtin_amdgcn_ballot_w64(start);
        const uint64_t stops = starts_m | ~__builtin_amdgcn_ballot_w64(valid);   // bits past TILE are stops
        if (start) {
            const uint64_t after = tid == 63 ? 0ull : stops >> (tid + 1);
            const int len = after ? 1 + __builtin_ctzll(after) : 64 - tid;
            runs[__builtin_popcountll(starts_m & ((1ull << tid) - 1ull))] = (tid << 8) | len;
        }
        if (tid == 0) n_runs = __builtin_popcountll(starts_m);
        if (tid < TILE) {
            blks[tid] = blk;
            offs[tid] = o;
        }
    }
    __syncthreads();

    u32x4 kv[NCH];
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int c = tid + 256 * i, r = c / CPR, cc = c % CPR;
        kv[i] = u32x4{0u, 0u, 0u, 0u};
        if (c < TILE * CPR && blks[r] >= 0) {
            auto *p = reinterpret_cast<const u32x4 *>(
                pool_k + (((int64_t)blks[r] * Hkv + g) * kBlockSize + offs[r]) * D + cc * 8);
            if constexpr (NT) kv[i] = __builtin_nontemporal_load(p);
            else kv[i] = *p;
        }
    }
    // V: task = (run, two dims)
    const int nr = n_runs;
    for (int task = tid; task < nr * (D / 2); task += 256) {
        const int k = task / (D / 2), x = 2 * (task % (D / 2));
        const int rv = runs[k], r0 = rv >> 8, len = rv & 0xff;
        const int o = offs[r0];
        const u16 *src = pool_v + (((int64_t)blks[r0] * Hkv + g) * D + x) * kBlockSize + (o & ~7);
        const u32x4 a = *reinterpret_cast<const u32x4 *>(src);
        const u32x4 b = *reinterpret_cast<const u32x4 *>(src + kBlockSize);
        const int e0 = o & 7;                  // the chunk's element of row r0
#pragma unroll
        for (int e = 0; e < 8; ++e) {          // element e of both dims, as one 32-bit word
            const uint32_t w = e & 1 ? (a[e >> 1] >> 16) | (b[e >> 1] & 0xFFFF0000u)
                                     : (a[e >> 1] & 0xFFFFu) | (b[e >> 1] << 16);
            if (len == 8 || (e >= e0 && e < e0 + len)) *reinterpret_cast<uint32_t *>(&vs[r0 + e - e0][x]) = w;
        }
    }
    __syncthreads();

#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int c = tid + 256 * i, r = c / CPR, cc = c % CPR;
        if (c < TILE * CPR && row0 + r < total) {
            const int64_t dst = ((int64_t)(row0 + r) * Hkv + g) * D + cc * 8;
            u32x4 vv = {0u, 0u, 0u, 0u};
            if (blks[r] >= 0) vv = *reinterpret_cast<const u32x4 *>(&vs[r][cc * 8]);
            put(k_out + dst, kv[i]);
            put(v_out + dst, vv);
        }
    }
}

// The same for calls of few rows, which wait on latency: one thread per 16 bytes of K and V
// finds its row by itself, and takes V in eight 2-byte loads, all in flight with K's. No
// barrier, and no serial tasks where every row is a sequence of its own (64 one-token
// sequences of 8 kv heads of 128: 4.8 us here, 7.7 in tiles; 64 tokens of one 3.9 and 4.5; 600
// 5.4 and 5.0, 2048, above the line, 9.5 and 7.5; one kv head 4096 4.6 and 5.5, 8192 5.6 and 6.1).
template <int D>
__global__ __launch_bounds__(256) void gather_rows_kernel(
    const u16 *__restrict__ pool_k, const u16 *__restrict__ pool_v, int32_t num_blocks, int32_t Hkv,
    const int32_t *__restrict__ block_tables, int32_t max_blocks,
    const int32_t *__restrict__ starts, const int32_t *__restrict__ cu_out, int32_t B,
    int32_t total, u16 *__restrict__ k_out, u16 *__restrict__ v_out)
{
    constexpr int CPR = D / 8;                 // 16-B chunks per row
    const int g = blockIdx.y, r = blockIdx.x * (256 / CPR) + threadIdx.x / CPR, c = threadIdx.x % CPR;
    if (r >= total) return;
    int lo = 0, hi = B - 1;                    // sequence with cu_out[lo] <= r < cu_out[lo + 1]
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (cu_out[mid] <= r) lo = mid; else hi = mid - 1;
    }
    const int t = starts[lo] + (r - cu_out[lo]), o = t % kBlockSize;
    u32x4 kw = {0u, 0u, 0u, 0u}, vw = {0u, 0u, 0u, 0u};
    if (t >= 0 && t / kBlockSize < max_blocks) {
        const int32_t blk = block_tables[(int64_t)lo * max_blocks + t / kBlockSize];
        if (blk >= 0 && blk < num_blocks) {
            const int64_t payload = ((int64_t)blk * Hkv + g) * kBlockSize * D;
            kw = *reinterpret_cast<const u32x4 *>(pool_k + payload + o * D + c * 8);
            const u16 *vp = pool_v + payload + c * 8 * kBlockSize + o;
            u16 e[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) e[k] = vp[k * kBlockSize];
#pragma unroll
            for (int k = 0; k < 4; ++k) vw[k] = e[2 * k] | ((unsigned)e[2 * k + 1] << 16);
        }
    }
    const int64_t dst = ((int64_t)r * Hkv + g) * D + c * 8;
    *reinterpret_cast<u32x4 *>(k_out + dst) = kw;
    *reinterpret_cast<u32x4 *>(v_out + dst) = vw;
}

// ---------------------------------------------------------------------------
// host pull / push: each workgroup copies whole blocks (K or V of one pair)
// between the pinned host store and the pool, 16 B per lane, 8 loads in flight
// per lane before their stores. Grid-stride over the 2*n block copies. Pull
// (host -> pool) reads the host pages with non-temporal loads; push (pool ->
// host) writes them with non-temporal stores, so host data never occupies L2.
// ---------------------------------------------------------------------------
constexpr int kPullUnroll = 8;
// Workgroups of one pull launch: 32 x 256 lanes x 8 x 16 B = 1 MiB in flight, enough
// to saturate a PCIe 5 x16 host link while leaving the other CUs to the compute stream
// (on MI355X, 16 workgroups reach about 85% of the link, 32 and more the full link).
constexpr int kPullWorkgroups = 32;

enum CopyDir { kHostToDevice = 0, kDeviceToHost = 1, kDeviceToDevice = 2 };

template <int kDir>
__global__ __launch_bounds__(256) void copy_blocks_kernel(
    const u32x4 *__restrict__ src_k, const u32x4 *__restrict__ src_v, int64_t src_blocks,
    u32x4 *__restrict__ dst_k, u32x4 *__restrict__ dst_v, int64_t dst_blocks,
    int64_t block_vecs, const PullArgs args)
{
    const int units = 2 * args.n;
    for (int u = blockIdx.x; u < units; u += gridDim.x) {
        const int pair = u >> 1;
        const bool is_v = u & 1;
        const int64_t sb = args.src[pair], db = args.dst[pair];
        if (sb < 0 || sb >= src_blocks || db < 0 || db >= dst_blocks) continue;
        const u32x4 *src = (is_v ? src_v : src_k) + sb * block_vecs;
        u32x4 *dst = (is_v ? dst_v : dst_k) + db * block_vecs;
        for (int64_t base = 0; base < block_vecs; base += 256 * kPullUnroll) {
            u32x4 r[kPullUnroll];
#pragma unroll
            for (int k = 0; k < kPullUnroll; ++k) {
                const int64_t i = base + k * 256 + threadIdx.x;
                if (i < block_vecs) r[k] = kDir == kHostToDevice ? __builtin_nontemporal_load(src + i) : src[i];
            }
#pragma unroll
            for (int k = 0; k < kPullUnroll; ++k) {
                const int64_t i = base + k * 256 + threadIdx.x;
                if (i < block_vecs) {
                    if (kDir == kDeviceToHost) __builtin_nontemporal_store(r[k], dst + i);
                    else dst[i] = r[k];
                }
            }
        }
    }
}

}  // namespace

hipError_t launch_append_kv(const pcr_kv_pool &pool, const void *k_new, const void *v_new,
                            const int32_t *slot_mapping, int32_t T, hipStream_t s)
{
    const dim3 grid((T + kAppendTile - 1) / kAppendTile, pool.num_kv_heads);
    auto *pk = static_cast<u16 *>(pool.k);
    auto *pv = static_cast<u16 *>(pool.v);
    auto *kn = static_cast<const u16 *>(k_new);
    auto *vn = static_cast<const u16 *>(v_new);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, pk, pv, pool.num_blocks, pool.num_kv_heads, kn, vn,
                           slot_mapping, T);
    };
    const int64_t in_bytes = 2 * (int64_t)T * pool.num_kv_heads * pool.head_dim * 2;
    auto launch_d = [&](auto dim) {
        constexpr int D = decltype(dim)::value;
        if (in_bytes > kNtBytes) launch(append_kv_kernel<D, kAppendTile, true, false>);
        else if ((int64_t)grid.x * grid.y <= kAppendEarly) launch(append_kv_kernel<D, kAppendTile, false, true>);
        else launch(append_kv_kernel<D, kAppendTile, false, false>);
    };
    if (pool.head_dim == 128) launch_d(std::integral_constant<int, 128>{});
    else launch_d(std::integral_constant<int, 64>{});
    return hipGetLastError();
}

hipError_t launch_gather_kv(const pcr_kv_pool &pool, const int32_t *block_tables, int32_t max_blocks,
                            const int32_t *starts, const int32_t *cu_out, int32_t B, int32_t total,
                            void *k_out, void *v_out, hipStream_t s)
{
    const int D = pool.head_dim, Hkv = pool.num_kv_heads;
    const int64_t out_bytes = 2 * (int64_t)total * Hkv * D * 2;
    auto launch = [&](auto kernel, int tile) {
        hipLaunchKernelGGL(kernel, dim3((total + tile - 1) / tile, Hkv), dim3(256), 0, s,
                           static_cast<const u16 *>(pool.k), static_cast<const u16 *>(pool.v), pool.num_blocks, Hkv,
                           block_tables, max_blocks, starts, cu_out, B, total, static_cast<u16 *>(k_out),
                           static_cast<u16 *>(v_out));
    };
    auto launch_d = [&](auto dim) {
        constexpr int DD = decltype(dim)::value;
        if (out_bytes <= kGatherRowsBytes) launch(gather_rows_kernel<DD>, 256 / (DD / 8));
        else if (out_bytes > kNtBytes) launch(gather_kv_kernel<DD, kGatherTile, true>, kGatherTile);
        else launch(gather_kv_kernel<DD, kGatherTile, false>, kGatherTile);
    };
    if (D == 128) launch_d(std::integral_constant<int, 128>{});
    else launch_d(std::integral_constant<int, 64>{});
    return hipGetLastError();
}

hipError_t launch_pull_blocks(const void *host_k, const void *host_v, int64_t host_blocks,
                              void *pool_k, void *pool_v, int32_t pool_blocks, int64_t block_bytes,
                              const PullArgs &args, hipStream_t s)
{
    if (args.n <= 0) return hipSuccess;
    const int units = 2 * args.n;
    const int grid = units < kPullWorkgroups ? units : kPullWorkgroups;
    hipLaunchKernelGGL(copy_blocks_kernel<kHostToDevice>, dim3(grid), dim3(256), 0, s,
                       static_cast<const u32x4 *>(host_k), static_cast<const u32x4 *>(host_v),
                       host_blocks, static_cast<u32x4 *>(pool_k), static_cast<u32x4 *>(pool_v),
                       (int64_t)pool_blocks, block_bytes / 16, args);
    return hipGetLastError();
}

hipError_t launch_push_blocks(const void *pool_k, const void *pool_v, int32_t pool_blocks, void *host_k,
                              void *host_v, int64_t host_blocks, int64_t block_bytes, const PullArgs &args,
                              hipStream_t s)
{
    if (args.n <= 0) return hipSuccess;
    const int units = 2 * args.n;
    const int grid = units < kPullWorkgroups ? units : kPullWorkgroups;
    hipLaunchKernelGGL(copy_blocks_kernel<kDeviceToHost>, dim3(grid), dim3(256), 0, s,
                       static_cast<const u32x4 *>(pool_k), static_cast<const u32x4 *>(pool_v),
                       (int64_t)pool_blocks, static_cast<u32x4 *>(host_k), static_cast<u32x4 *>(host_v),
                       host_blocks, block_bytes / 16, args);
    return hipGetLastError();
}

hipError_t launch_device_blocks(const void *src_k, const void *src_v, int64_t src_blocks, void *dst_k, void *dst_v,
                                int64_t dst_blocks, int64_t block_bytes, const PullArgs &args, hipStream_t s)
{
    if (args.n <= 0) return hipSuccess;
    // HBM to HBM: one workgroup per block copy, all CUs if there is work for them
    const int grid = 2 * args.n;
    hipLaunchKernelGGL(copy_blocks_kernel<kDeviceToDevice>, dim3(grid), dim3(256), 0, s,
                       static_cast<const u32x4 *>(src_k), static_cast<const u32x4 *>(src_v), src_blocks,
                       static_cast<u32x4 *>(dst_k), static_cast<u32x4 *>(dst_v), dst_blocks, block_bytes / 16, args);
    return hipGetLastError();
}

}  // namespace pcr
