// Stage 3: tree-masked verification attention (one target layer).
//
// Every query row (node n, query head h) attends to the cached prefix of its
// sequence and to the tree nodes on its root path.  Rows are packed per KV
// head: row rho = n * G + (h - g * G), so one workgroup serves the G query
// heads that share KV head g and streams each K/V tile through LDS once for
// all of them.  The key sequence of sequence b is virtual: positions
// 0 .. ctx_b-1 read the packed cache, positions ctx_b .. ctx_b+n_nodes-1
// read the tree K/V and are masked by the ancestor bitmask.
//
// bf16 path (matrix cores, v_mfma_f32_32x32x16_bf16).  A workgroup is eight
// waves (two per SIMD), each owning 32 query rows.  Scores are computed
// transposed, S^T = K Q^T: a lane then holds one query row and 16 of the 32
// keys of a block, the row max needs one cross-half swap, and the bf16
// probabilities are already in the B-operand layout of O^T = V^T P^T.  K and
// V sit in LDS row-major (the chunks of a row permuted so that the b128 K reads
// and the transposed ds_read_b64_tr_b16 V reads are free of bank conflicts).
// Four 64-key LDS buffers rotate, filled straight from global memory: tile t is
// consumed, tile t+1 is resident (the blocks of a tile already score those of
// the next), tiles t+2 and t+3 are in flight; one barrier per tile.  Inside a
// wave the P V of block i, the scores of block i+2 and the exponentials of
// block i+1 are issued interleaved, so the matrix cores can run while the
// vector ALUs work.  The running reference maximum only moves when a block
// exceeds it by a margin, which keeps the 64-register accumulator rescale off
// the common path.  The context is split across workgroups when the batch alone
// cannot fill the chip; each split leaves, per query row, its (reference, sum)
// pair and its output divided by its own sum (bf16), which a second kernel
// merges.
#include <math.h>

#include <type_traits>

#include "common.hpp"

namespace presto {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

// Two fp32 -> two bf16 (round to nearest even) in one v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2){lo, hi}, bf16x2));
}

constexpr int kKeyTile = 64;      // keys per LDS tile: two 32-key blocks per barrier
constexpr int kBlocksPerTile = kKeyTile / 32;
constexpr int kRing = 4;          // LDS tile buffers: tile t consumed, t+1 resident, t+2 and t+3 in flight
constexpr int kMaxAncWords = 16;  // ancestor words per node: n_max <= 1024
constexpr int kRowsPerWave = 32;  // one 32-row MFMA block per wave
// Workgroups are 8 waves, two per SIMD, so that one wave's vector work runs
// while the other's MFMAs occupy the matrix core.
constexpr int kAttnWaves = 8;
constexpr int kAttnRows = kAttnWaves * kRowsPerWave;  // query rows per workgroup
constexpr float kLog2e = 1.4426950408889634f;

struct AttnArgs {
    const uint16_t* q;
    const uint16_t* kc;
    const uint16_t* vc;
    const int32_t* ctx_off;
    int32_t ctx_slots;  // 0: ctx_off is [batch + 1] offsets; 1: (start, len) pairs
    const uint16_t* kt;
    const uint16_t* vt;
    const uint64_t* anc;
    const int32_t* n_nodes;
    uint16_t* out;
    // split partials when splits > 1: the normalised output as bf16
    // [b, g, split, rho < G n_max, D] (a workgroup's rows are contiguous, so
    // its writes fill whole cache lines) and (m, l) fp32 [b, g, rho, split]
    uint16_t* part_o;
    float2* part_ml;
    int32_t batch, n_max, hq, hkv, G, W;
    int32_t row_tiles, rows_per_tile, splits, split_len;  // rows_per_tile: a multiple of 32, <= 256
    int32_t n_tasks, n_blocks;
    // shares > 0: the key tiles of all sequences together are cut into that
    // many equal shares (see TileShares); the partials are then [slot, g, row,
    // D] and [g, row, slot], slot = share + sequence < n_slots
    int32_t shares, n_slots;
    int2* slots;  // [batch] first and last slot of each sequence
    int32_t pairs;  // 1: the tasks are the (sequence, split) pairs that exist; the grid is an upper bound
    float scale_log2;  // scale * log2(e)
};

// Cache rows of sequence b: start c0 and length ctx, from packed offsets
// [batch + 1] or from (start, len) pairs [batch, 2].
struct CtxSpan {
    int c0, ctx;
};
__device__ __forceinline__ CtxSpan ctx_span(const int32_t* off, int b, int slots) {
    if (slots) return {off[2 * b], off[2 * b + 1]};
    return {off[b], off[b + 1] - off[b]};
}

__device__ __forceinline__ int clamp_nodes(int nn, int n_max) {
    return nn < 1 ? 1 : (nn > n_max ? n_max : nn);
}

// Ragged batches: the key tiles of all sequences in a row (each sequence led by
// kLeadTiles of them that stand for a workgroup's start on it: query
// fragments, the first tiles' arrival, the partial's store) cut into equal
// shares, the first V % shares one tile longer.  A share holds part of one
// sequence, or the end of one, whole ones and the start of another; it and the
// next sequence never advance together past a boundary, so share + sequence
// numbers the parts.
constexpr int kLeadTiles = 3;
struct TileShares {
    int q, r;
    __device__ __forceinline__ TileShares(int total, int shares) : q(total / shares), r(total % shares) {}
    __device__ __forceinline__ int begin(int c) const { return c * q + min(c, r); }
};
// (lead and key) tiles of sequence bb, 0 past the batch
__device__ __forceinline__ int share_tiles(const AttnArgs& a, int bb) {
    if (bb >= a.batch) return 0;
    const int keys = ctx_span(a.ctx_off, bb, a.ctx_slots).ctx + clamp_nodes(a.n_nodes[bb], a.n_max);
    return (keys + kKeyTile - 1) / kKeyTile + kLeadTiles;
}
// splits that sequence bb really has, 0 past the batch
__device__ __forceinline__ int live_splits(const AttnArgs& a, int bb) {
    if (bb >= a.batch) return 0;
    const int keys = ctx_span(a.ctx_off, bb, a.ctx_slots).ctx + clamp_nodes(a.n_nodes[bb], a.n_max);
    return min((keys + a.split_len - 1) / a.split_len, a.splits);
}
// All tiles of the batch (every wave computes it for itself).
__device__ __forceinline__ int share_total(const AttnArgs& a) {
    int total = 0;
    for (int b0 = 0; b0 < a.batch; b0 += kWave)
        total += __builtin_amdgcn_readlane((int)wave_scan_dpp(share_tiles(a, b0 + lane_id())), kWave - 1);
    return total;
}

// Blocks are dealt to the 8 XCDs round-robin; renumber them so that
// consecutive logical tasks (the row tiles of one KV range) share an XCD
// and its L2.
__device__ __forceinline__ int xcd_task(int bid, int n_blocks) {
    const int per = n_blocks >> 3;
    return (bid & 7) * per + (bid >> 3);
}

// LDS layout of the bf16 kernel (bytes).  A K tile is 64 key rows of D
// bf16 (D*2 bytes, no padding) with the 16-byte chunks of row r permuted by
// chunk ^ (r mod 16); a V tile likewise with chunk ^ 4(r mod 4).  The two
// permutations make the fragment reads free of bank conflicts (sixteen
// consecutive K rows read one chunk each: sixteen different chunks; the
// transposed V reads of four consecutive rows cover four disjoint 64-byte
// chunk groups), and since the global-to-LDS loads write 64 consecutive
// 16-byte chunks per instruction, the permutation is applied by choosing
// which global chunk each lane fetches.  K tiles of the ring sit in the
// first 64 KB and V tiles in the second, so that every fragment read is a
// per-lane base register plus an immediate offset.
// Global-to-LDS load of 16 bytes per lane (global_load_lds_dwordx4): lane
// l's bytes land at LDS address lds + 16 l (lds wave-uniform, in m0).  The
// instruction is issued from inline assembly so that the compiler does not
// guard every later LDS read with a wait for all outstanding loads; the
// kernel waits for each tile itself (vmcnt) before the barrier that
// publishes it.
__device__ __forceinline__ void lds_load16(const void* gptr, uint32_t lds) {
    asm volatile("global_load_lds_dwordx4 %0, off" ::"v"(gptr), "{m0}"(lds) : "memory");
}
// the same with a wave-uniform base and a per-lane 32-bit byte offset (the
// base and the LDS address are read from the first lane, so that they are
// scalar operands whatever registers the caller computed them in)
__device__ __forceinline__ void lds_load16(const void* base, uint32_t off, uint32_t lds) {
    const uint64_t b = (uint64_t)(uintptr_t)base;
    // readfirstlane returns a signed int: both halves go through uint32_t so
    // that the low half is zero-extended, not sign-extended, into the pointer
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    const uint64_t sb = ((uint64_t)hi << 32) | (uint64_t)lo;
    const uint32_t m0v = (uint32_t)__builtin_amdgcn_readfirstlane(lds);
    asm volatile("global_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(sb), "{m0}"(m0v) : "memory");
}

template <int D>
struct AttnLds {
    static constexpr int kTile = kKeyTile * D * 2;           // bytes of one K (or V) tile
    static constexpr int kV = kRing * kTile;                 // start of the V tiles
};

// SHARES: a ragged batch cut into equal shares of key tiles (an instantiation
// of its own: the loop over a share's sequences costs the dense key loop 9%).
//
// TAIL: a tree of 2^i draft nodes has 2^i + 1 rows per query head, so that the
// query rows often end 1 .. 16 past a multiple of 256.  A row tile of its own
// for them streams all keys again through a workgroup that computes next to
// nothing; here the last full tile's workgroup takes them along on 16 x 16
// MFMAs: of every tile in LDS, waves 0 - 3 (one per SIMD) take sixteen keys each
// (scores 16x16x32, P V 16x16x16, the query from LDS), about a tenth of a
// tile's matrix work, and their states are combined at the end.  us per call:
// 4 sequences of 32768 keys, 257 nodes 618 -> 596, 129 nodes 374 -> 319;
// 8 of 2048, 257 nodes 136 -> 92.
template <int D, bool SHARES, bool TAIL>
__global__ __launch_bounds__(kAttnWaves * kWave) void tree_attn_bf16_kernel(AttnArgs a) {
    constexpr int KS = D / 16;                 // S^T contraction steps over the head dimension
    constexpr int DB = D / 32;                 // 32-wide blocks of the output head dimension
    constexpr int CH = D / 8;                  // 16-byte chunks per K/V row
    constexpr int NT = kAttnWaves * kWave;
    constexpr int ROWS = kAttnRows;
    // global-to-LDS loads per thread per tile, K and V each: 64 rows x CH
    // chunks, 64 chunks per instruction
    constexpr int LPT = kKeyTile * CH / 64 / kAttnWaves;
    constexpr int ROWS_PER_LOAD = 64 / CH;     // key rows covered by one load instruction
    static_assert(LPT >= 1 && LPT * kAttnWaves * 64 == kKeyTile * CH, "tile loads must divide evenly");
    static_assert(!(SHARES && TAIL), "registers");
    static_assert(AttnLds<D>::kV + kRing * AttnLds<D>::kTile <= 65536 * 2, "ring must fit 128 KB");
    __shared__ __align__(16) char s_kv[2 * kRing * AttnLds<D>::kTile];
    // ancestor rows of this workgroup's nodes: at most ROWS nodes (G = 1)
    // of at most kMaxAncWords words; with the ring this is 160 KB at D = 128
    __shared__ uint64_t s_anc[ROWS * kMaxAncWords];

    int n_tasks = a.n_tasks, n_blocks = a.n_blocks;
    if constexpr (!SHARES && !TAIL) {
        if (a.pairs) {
            // every wave counts the pairs itself
            int pairs = 0;
            for (int b0 = 0; b0 < a.batch; b0 += kWave)
                pairs += __builtin_amdgcn_readlane((int)wave_scan_dpp(live_splits(a, b0 + lane_id())), kWave - 1);
            n_tasks = pairs * a.hkv * a.row_tiles;
            n_blocks = (n_tasks + 7) / 8 * 8;
            if ((int)blockIdx.x >= n_blocks) return;
        }
    }
    const int task = xcd_task(blockIdx.x, n_blocks);
    if (task >= n_tasks) return;
    const int rt = task % a.row_tiles;
    const int g = (task / a.row_tiles) % a.hkv;

    // One range of keys [key0, key1) (key1 cut at the sequence's end) of
    // sequence b: the workgroup's rows against them.  Partials go to rows
    // part_row + rho, their (m, l) to part_ml[ml_row + rho * ml_stride].
    auto segment = [&](int b, int key0, int key1, int64_t part_row, int64_t ml_row, int ml_stride)
                       __attribute__((always_inline)) {
    const CtxSpan cs = ctx_span(a.ctx_off, b, a.ctx_slots);
    const int c0 = cs.c0, ctx = cs.ctx;
    const int nn = clamp_nodes(a.n_nodes[b], a.n_max);
    const int keys = ctx + nn;
    const int k_begin = key0;
    if (k_begin >= keys) return;  // nothing of this sequence in this split
    const int k_end = min(keys, key1);
    const int ntiles = (k_end - k_begin + kKeyTile - 1) / kKeyTile;
    const int nblocks = (k_end - k_begin + 31) / 32;
    const int live_rows = a.G * nn;
    const int all_rows = a.G * a.n_max;
    const int mask_from = min(ctx, k_end);  // keys at or beyond need a mask

    const int tid = threadIdx.x;
    const int wave = tid / kWave, lane = lane_id();
    const int l32 = lane & 31, h = lane >> 5;
    // Row blocks: wave w takes block w, except that when fewer than
    // kAttnWaves blocks hold live rows (A of them), the last one is shared by
    // waves A-1 .. kAttnWaves-1, each taking every nshare-th key block, and
    // their states are combined at the end: a 4-row tail block then costs a
    // SIMD a fraction of a full one.
    const int RT = a.rows_per_tile;
    const int tile_live = min(max(live_rows - rt * RT, 0), RT);
    const int A = (tile_live + kRowsPerWave - 1) / kRowsPerWave;
    const int nshare = (A >= 1 && A < kAttnWaves) ? kAttnWaves - A + 1 : 1;
    const bool shared = nshare > 1 && wave >= A - 1;
    const int sidx = shared ? wave - (A - 1) : 0;
    const int row0 = rt * RT + (shared ? A - 1 : wave) * kRowsPerWave;  // first query row of this wave
    const bool active = row0 < live_rows;
    // the rows past the last full tile, when they ride along with it
    const int tail0 = a.row_tiles * RT;
    const bool tail_here = TAIL && rt == a.row_tiles - 1;
    const bool tail_on = tail_here && live_rows > tail0;  // (the tile itself is then fully live)
    constexpr int TD = D / 16;  // 16-dim blocks of the tail's O^T
    char* const s_tq = reinterpret_cast<char*>(s_anc + (ROWS * kMaxAncWords - 16 * D / 4));
    const int t16 = lane & 15, tq = lane >> 4;
    const int tnode = min((tail0 + t16) / a.G, a.n_max - 1);
    floatx4 ot[TAIL ? TD : 1];
    float tm = -INFINITY, tl = 0.f;  // reference (log2 units) and this lane's part of the row sum
    if constexpr (TAIL) {
#pragma unroll
        for (int i = 0; i < TD; ++i) ot[i] = (floatx4){0.f, 0.f, 0.f, 0.f};
        if (tail_on && tid < 16 * CH) {
            // scaled queries, chunk c of row r at c ^ r
            const int r = tid / CH, ck = tid % CH;
            const int rr = min(tail0 + r, all_rows - 1);
            const uint4 u = *reinterpret_cast<const uint4*>(
                a.q + (((int64_t)b * a.n_max + rr / a.G) * a.hq + g * a.G + rr % a.G) * D + ck * 8);
            const uint32_t w[4] = {u.x, u.y, u.z, u.w};
            uint32_t x[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                x[j] = pack_bf16x2(__uint_as_float(w[j] << 16) * a.scale_log2,
                                   __uint_as_float(w[j] & 0xffff0000u) * a.scale_log2);
            *reinterpret_cast<uint4*>(s_tq + r * D * 2 + ((ck ^ (r & (CH - 1))) * 16)) =
                make_uint4(x[0], x[1], x[2], x[3]);
        }
    }
    const int rho = row0 + l32;  // this lane's query row
    const int qn = rho / a.G, qh = rho - qn * a.G;
    const int node = min(qn, a.n_max - 1);
    const float c = a.scale_log2;

    // Q fragments, B operand of S^T = K Q^T: lane holds row l32,
    // d = ks*16 + h*8 .. +8, pre-scaled by scale*log2(e) (rounded once to
    // bf16), so that the scores come out in log2 units.
    bf16x8 qf[KS];
    {
        const uint16_t* qp = a.q + (((int64_t)b * a.n_max + qn) * a.hq + g * a.G + qh) * D;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            uint4 u = make_uint4(0, 0, 0, 0);
            if (rho < all_rows) u = *reinterpret_cast<const uint4*>(qp + ks * 16 + h * 8);
            const uint32_t w[4] = {u.x, u.y, u.z, u.w};
            uint32_t r[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                r[j] = pack_bf16x2(__uint_as_float(w[j] << 16) * c, __uint_as_float(w[j] & 0xffff0000u) * c);
            qf[ks] = __builtin_bit_cast(bf16x8, make_uint4(r[0], r[1], r[2], r[3]));
        }
    }
    // ancestor bitmask rows of the nodes this workgroup serves, when the
    // split reaches the tree keys (masks then read LDS, not global memory)
    const int n_first = (rt * RT) / a.G;
    if (k_end > ctx) {
        const int n_last = tail_on ? a.n_max - 1 : min((rt * RT + RT - 1) / a.G, a.n_max - 1);
        const int words = (n_last - n_first + 1) * a.W;
        const uint64_t* src = a.anc + ((int64_t)b * a.n_max + n_first) * a.W;
        for (int w = tid; w < words; w += NT) s_anc[w] = src[w];
    }

    // ---- K/V tiles: global -> LDS directly (global_load_lds_dwordx4), a
    // ring of kRing tiles.  Load instruction j of this wave covers key rows
    // ROWS_PER_LOAD * (wave * LPT + j) .. of the tile; lane l writes chunk
    // l % CH of row l / CH and so fetches the global chunk that the row's
    // permutation puts there.  The byte offsets of those chunks within a
    // tile that lies wholly in the cache are fixed for the whole loop.
    uint32_t goff_k[LPT], goff_v[LPT];
    int lrow[LPT], lck[LPT], lcv[LPT];
#pragma unroll
    for (int j = 0; j < LPT; ++j) {
        const int r = ROWS_PER_LOAD * (wave * LPT + j) + lane / CH;
        const int pc = lane % CH;
        lrow[j] = r;
        lck[j] = pc ^ (r & (CH - 1) & 15);
        lcv[j] = pc ^ ((4 * (r & 3)) & (CH - 1));
        goff_k[j] = (uint32_t)((r * a.hkv * D + lck[j] * 8) * 2);
        goff_v[j] = (uint32_t)((r * a.hkv * D + lcv[j] * 8) * 2);
    }
    const int fast_end = min(ctx, k_end);
    const int64_t tree_row0 = (int64_t)b * a.n_max;
    // all loads of the tile starting at key t0 into ring buffer `buf`
    const uint32_t lds_kv = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)s_kv;
    // the four base pointers as scalars: a per-lane choice between them is
    // then a register select, not a load from the argument block
    auto scalar_ptr = [](const uint16_t* ptr) {
        const uint64_t v = (uint64_t)(uintptr_t)ptr;
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
        return (const uint16_t*)(uintptr_t)(((uint64_t)hi << 32) | lo);
    };
    const uint16_t* const kc_s = scalar_ptr(a.kc);
    const uint16_t* const vc_s = scalar_ptr(a.vc);
    const uint16_t* const kt_s = scalar_ptr(a.kt);
    const uint16_t* const vt_s = scalar_ptr(a.vt);
    auto load_tile = [&](int t0, int buf) {
        const uint32_t kdst = lds_kv + buf * AttnLds<D>::kTile + wave * LPT * 1024;
        const uint32_t vdst = kdst + AttnLds<D>::kV;
        if (t0 + kKeyTile <= fast_end) {
            const int64_t row = ((int64_t)(c0 + t0) * a.hkv + g) * D;
            const uint16_t* kb = a.kc + row;
            const uint16_t* vb = a.vc + row;
#pragma unroll
            for (int j = 0; j < LPT; ++j) {
                lds_load16(kb, goff_k[j], kdst + j * 1024);
                lds_load16(vb, goff_v[j], vdst + j * 1024);
            }
        } else {
            // keys below ctx from the cache, the others from the tree K/V;
            // rows past k_end repeat the last key (their scores are masked)
#pragma unroll
            for (int j = 0; j < LPT; ++j) {
                const int kk = min(t0 + lrow[j], k_end - 1);
                const bool in_ctx = kk < ctx;
                const int64_t base = in_ctx ? ((int64_t)(c0 + kk) * a.hkv + g) * D
                                            : ((tree_row0 + (kk - ctx)) * a.hkv + g) * D;
                const uint16_t* kp = (in_ctx ? kc_s : kt_s) + base + lck[j] * 8;
                const uint16_t* vp = (in_ctx ? vc_s : vt_s) + base + lcv[j] * 8;
                lds_load16(kp, kdst + j * 1024);
                lds_load16(vp, vdst + j * 1024);
            }
        }
    };
    // vmcnt(n) with the other counters left alone (gfx9 encoding)
#define PRESTO_WAIT_VM(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (((n) >> 4) << 14) | 0x0f70)

    floatx16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[db][i] = 0.f;

    // per-lane LDS byte addresses of the fragment reads (ring buffer 0,
    // block 0); buffer, block and step offsets are immediates
    const int vr = 4 * h + ((lane & 15) >> 2);                  // row within an 8-row group
    const int vc = ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1);   // chunk within a 4-chunk group
    // step 0's address; the others differ in the chunk bits only (an xor)
    uint32_t k_base = l32 * (D * 2) + ((h ^ (l32 & 15)) & (CH - 1)) * 16;
    uint32_t v_base = AttnLds<D>::kV + vr * (D * 2) + ((4 * (vr & 3) + vc) & (CH - 1)) * 16 + (lane & 1) * 8;
    uint32_t kaddr[TAIL ? 1 : KS], vaddr[TAIL ? 1 : DB];
    if constexpr (!TAIL) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kaddr[ks] = k_base ^ (ks << 5);
#pragma unroll
        for (int db = 0; db < DB; ++db) vaddr[db] = v_base ^ (db << 6);
    }
    // with tail rows the registers for all twelve are missing: formed anew
    // per read
    auto k_at = [&](int ks) __attribute__((always_inline)) { return TAIL ? k_base ^ (ks << 5) : kaddr[TAIL ? 0 : ks]; };
    auto v_at = [&](int db) __attribute__((always_inline)) { return TAIL ? v_base ^ (db << 6) : vaddr[TAIL ? 0 : db]; };
    auto fresh = [&]() __attribute__((always_inline)) {
        if constexpr (TAIL) asm volatile("" : "+v"(k_base), "+v"(v_base));
    };

    auto row_max = [&](const floatx16& S) {
        float mx = S[0];
#pragma unroll
        for (int e = 1; e < 16; ++e) mx = fmaxf(mx, S[e]);
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx),
                                                         false, false);
        return fmaxf(mx, __uint_as_float(h == 0 ? sw[1] : sw[0]));
    };
    // Visibility of the block's 32 keys for this lane's row as one 32-bit
    // mask (bit t: key j0 + t): context keys, then the row's ancestor bits
    // from tree index j0 - ctx on, cut at the split's end; each element then
    // costs one bit test and one select.
    auto apply_mask = [&](floatx16& S, int j0) {
        const int s0 = j0 - ctx;  // tree index of the block's first key (< 0: it starts in the context)
        uint32_t anc = 0u;
        if (j0 + 32 > ctx) {
            const uint64_t* arow = &s_anc[(node - n_first) * a.W];
            if (s0 >= 0) {
                const int w = s0 >> 6, sh = s0 & 63;
                const uint64_t lo = arow[w];
                const uint64_t hi = w + 1 < a.W ? arow[w + 1] : 0ull;
                anc = (uint32_t)(sh == 0 ? lo : (lo >> sh) | (hi << (64 - sh)));
            } else {
                anc = (uint32_t)(arow[0] << (-s0));  // -s0 in 1 .. 31
            }
        }
        const int nctx = ctx - j0, nend = k_end - j0;
        const uint32_t ctx_mask = nctx >= 32 ? ~0u : (nctx <= 0 ? 0u : (1u << nctx) - 1u);
        const uint32_t end_mask = nend >= 32 ? ~0u : (nend <= 0 ? 0u : (1u << nend) - 1u);
        const uint32_t vis = ((ctx_mask | anc) & end_mask) >> (4 * h);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int t = 8 * (e >> 2) + (e & 3);  // element e is key j0 + 8(e/4) + 4h + e%4
            S[e] = ((vis >> t) & 1u) ? S[e] : -INFINITY;
        }
    };

    // ---- Key loop, pipelined over three key blocks so that the matrix
    // cores always have two independent chains and the vector ALUs work in
    // their shadow.  Step i issues, interleaved,
    //   * the P V MFMAs of block i (probabilities from step i-1),
    //   * the score MFMAs of block i+2 (its tile is resident),
    //   * the exponentials of block i+1 (scores from step i-1).
    // Every score chain starts from -m, so the MFMAs deliver x = s*c - m and
    // a probability costs one v_exp.  m is a lazy reference: no per-block
    // maximum is taken; a row whose block sum exceeds 2^8 (some x above
    // about 3) or that has no mass yet takes an exact step (block maximum,
    // rescale of o and l), which is rare.
    constexpr int EPK = 16 / KS;  // exponentials per score MFMA
    static_assert(EPK * KS == 16 && EPK % 2 == 0 && KS == 2 * DB, "head_dim 64 or 128");
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    float m = 0.f, l_run = 0.f;  // lazy reference (log2 units) and row sum
    floatx16 negm;
#pragma unroll
    for (int e = 0; e < 16; ++e) negm[e] = 0.f;
    typedef __attribute__((address_space(3))) short4_t* lds_s4;
    // scores of block blk of ring buffer buf (compile-time) into Sx
    auto qk = [&](auto bufc, int blk, floatx16& Sx) {
        constexpr int buf = decltype(bufc)::value;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const uint4 u = *reinterpret_cast<const uint4*>(s_kv + k_at(ks) + buf * AttnLds<D>::kTile +
                                                             blk * 32 * D * 2);
            Sx = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, u), qf[ks],
                                                         ks == 0 ? negm : Sx, 0, 0, 0);
        }
    };
    auto exps = [&](const floatx16& Sx, uint32_t (&Px)[8]) {
        float ls = 0.f;
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
            Px[e >> 1] = pack_bf16x2(__builtin_amdgcn_exp2f(Sx[e]), __builtin_amdgcn_exp2f(Sx[e + 1]));
            ls = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, Px[e >> 1]), ones, ls, false);
        }
        return ls;
    };
    auto row_sum = [&](float v) {
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        return v + __uint_as_float(h == 0 ? sw[1] : sw[0]);
    };
    // exact step for the rows that need it: move m to the block's maximum,
    // rescale the accumulated state and recompute the block's probabilities
    // (Sy: a block already scored against the old m, shifted along)
    auto exact = [&](floatx16& Sx, uint32_t (&Px)[8], float& ls, bool need, floatx16& Sy) {
        const float mx = row_max(Sx);
        const float delta = (need && mx != -INFINITY) ? mx : 0.f;
        const float alpha = l_run > 0.f ? __builtin_amdgcn_exp2f(-delta) : 0.f;
        m += delta;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db) o[db] *= alpha;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            Sx[e] -= delta;
            Sy[e] -= delta;
            negm[e] = -m;
        }
        ls = row_sum(exps(Sx, Px));
    };
    auto j0_of = [&](int i) { return k_begin + i * 32; };
    auto masked = [&](int i) { return j0_of(i) + 32 > mask_from; };

    floatx16 Sa = negm, Sb = negm;  // scores of blocks i+1 and i+2
    uint32_t Pp[8];                 // probabilities of block i
    // one block step: block i = 2 t + q; V of tile t in ring buffer bv, the
    // K of block i+2 (tile t+1) in ring buffer bk
    auto step = [&](auto bvc, auto bkc, int i, int q) {
        constexpr int bv = decltype(bvc)::value, bk = decltype(bkc)::value;
        fresh();
        const bool more = i + 1 < nblocks;
        if (more && masked(i + 1)) apply_mask(Sa, j0_of(i + 1));
        const int kblk = (i + 2) % kBlocksPerTile;
        uint32_t Pn[8];
        float ls = 0.f;
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            const bf16x8 pb =
                __builtin_bit_cast(bf16x8, make_uint4(Pp[4 * st], Pp[4 * st + 1], Pp[4 * st + 2], Pp[4 * st + 3]));
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const uint32_t v0 = v_at(db) + bv * AttnLds<D>::kTile + q * 32 * D * 2 + st * 16 * D * 2;
                const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(s_kv + v0));
                const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(s_kv + v0 + 8 * D * 2));
                const uint2 ul = __builtin_bit_cast(uint2, lo), uh = __builtin_bit_cast(uint2, hi);
                const bf16x8 va = __builtin_bit_cast(bf16x8, make_uint4(ul.x, ul.y, uh.x, uh.y));
                o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb, o[db], 0, 0, 0);
                const int ks = st * DB + db;
                const uint4 u = *reinterpret_cast<const uint4*>(s_kv + k_at(ks) + bk * AttnLds<D>::kTile +
                                                                 kblk * 32 * D * 2);
                Sb = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, u), qf[ks],
                                                             ks == 0 ? negm : Sb, 0, 0, 0);
#pragma unroll
                for (int uu = 0; uu < EPK; uu += 2) {
                    const int e = ks * EPK + uu;
                    Pn[e >> 1] = pack_bf16x2(__builtin_amdgcn_exp2f(Sa[e]), __builtin_amdgcn_exp2f(Sa[e + 1]));
                    ls = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, Pn[e >> 1]), ones, ls, false);
                }
            }
        }
        if (more) {
            ls = row_sum(ls);
            const bool need = !(ls <= 256.f) || l_run + ls == 0.f;
            if (__ballot(need)) exact(Sa, Pn, ls, need, Sb);
            l_run += ls;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) Pp[j] = Pn[j];
        Sa = Sb;
    };
    // P V of block q of ring buffer bv with the probabilities P
    auto pv = [&](auto bvc, int q, const uint32_t (&P)[8]) {
        constexpr int bv = decltype(bvc)::value;
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            const bf16x8 pb =
                __builtin_bit_cast(bf16x8, make_uint4(P[4 * st], P[4 * st + 1], P[4 * st + 2], P[4 * st + 3]));
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const uint32_t v0 = v_at(db) + bv * AttnLds<D>::kTile + q * 32 * D * 2 + st * 16 * D * 2;
                const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(s_kv + v0));
                const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(s_kv + v0 + 8 * D * 2));
                const uint2 ul = __builtin_bit_cast(uint2, lo), uh = __builtin_bit_cast(uint2, hi);
                const bf16x8 va = __builtin_bit_cast(bf16x8, make_uint4(ul.x, ul.y, uh.x, uh.y));
                o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb, o[db], 0, 0, 0);
            }
        }
    };
    // a shared block's wave: block i (block q of ring buffer bv) on its own,
    // scores, probabilities and P V in sequence (it takes every nshare-th
    // block only)
    auto shared_step = [&](auto bvc, int i, int q) {
        floatx16 S = negm;
        qk(bvc, q, S);
        if (masked(i)) apply_mask(S, j0_of(i));
        uint32_t P[8];
        float ls = row_sum(exps(S, P));
        const bool need = !(ls <= 256.f) || l_run + ls == 0.f;
        floatx16 none = S;
        if (__ballot(need)) exact(S, P, ls, need, none);
        l_run += ls;
        pv(bvc, q, P);
    };
    // the tail rows against sixteen keys of tile t (ring buffer bv): lane
    // (t16, tq) holds row t16 and keys 4 tq .. 4 tq + 3 of wave's sixteen
    auto tail_step = [&](auto bvc, int t) __attribute__((always_inline)) {
        constexpr int bv = decltype(bvc)::value;
        const int j0 = k_begin + t * kKeyTile + wave * 16;
        if (j0 >= k_end) return;
        const uint32_t toff = (uint32_t)((tq ^ t16) & (CH - 1)) * 16;
        const uint32_t ka = (uint32_t)(wave * 16 + t16) * (D * 2) + bv * AttnLds<D>::kTile;
        floatx4 S = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < D / 32; ++ks) {
            const uint4 kf = *reinterpret_cast<const uint4*>(s_kv + ka + (toff ^ (ks * 64)));
            const uint4 qv = *reinterpret_cast<const uint4*>(s_tq + t16 * (D * 2) + (toff ^ (ks * 64)));
            S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf),
                                                        __builtin_bit_cast(bf16x8, qv), S, 0, 0, 0);
        }
        if (j0 + 16 > mask_from) {
            const uint64_t* arow = &s_anc[(tnode - n_first) * a.W];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int j = j0 + 4 * tq + e, s = j - ctx;
                const bool vis = j < k_end && (s < 0 || ((arow[max(s, 0) >> 6] >> (s & 63)) & 1ull));
                S[e] = vis ? S[e] : -INFINITY;
            }
        }
        float mx = fmaxf(fmaxf(S[0], S[1]), fmaxf(S[2], S[3]));
        if (__ballot(mx > tm + 8.f)) {
            // move the row's reference to its maximum over the sixteen keys
            const auto h16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
            mx = fmaxf(__uint_as_float(h16[0]), __uint_as_float(h16[1]));
            const auto h32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
            mx = fmaxf(__uint_as_float(h32[0]), __uint_as_float(h32[1]));
            const float mn = fmaxf(tm, mx);
            const float al = tm == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(tm - mn);
            tm = mn;
            tl *= al;
#pragma unroll
            for (int i = 0; i < TD; ++i) ot[i] *= al;
        }
        const float mr = tm == -INFINITY ? 0.f : tm;  // no key visible yet: every term is 0
        uint32_t P[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            P[e] = pack_bf16x2(__builtin_amdgcn_exp2f(S[2 * e] - mr), __builtin_amdgcn_exp2f(S[2 * e + 1] - mr));
            tl = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, P[e]), ones, tl, false);
        }
        const short4_t pb = __builtin_bit_cast(short4_t, make_uint2(P[0], P[1]));
        const int x = t16 >> 2;
        const uint32_t va = AttnLds<D>::kV + bv * AttnLds<D>::kTile +
                            (uint32_t)(wave * 16 + 4 * tq + x) * (D * 2) + (t16 & 1) * 8;
        const uint32_t vc0 = (uint32_t)(((t16 & 3) >> 1) ^ ((4 * x) & (CH - 1))) * 16;
#pragma unroll
        for (int i = 0; i < TD; ++i) {
            const short4_t vf = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(s_kv + va + (vc0 ^ (i * 32))));
            ot[i] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vf, pb, ot[i], 0, 0, 0);
        }
    };
    // one tile: its two block steps, then the load of tile t+3 into the
    // buffer of tile t-1 (every wave finished it before the last barrier),
    // and the wait for tile t+2 before the barrier
    auto tile = [&](auto uc, int t) {
        constexpr int u = decltype(uc)::value;
        using BV = std::integral_constant<int, u>;
        using BK = std::integral_constant<int, (u + 1) % kRing>;
        load_tile(k_begin + (t + 3) * kKeyTile, (u + 3) % kRing);
        if (active && !shared) {
            if (2 * t < nblocks) step(BV{}, BK{}, 2 * t, 0);
            if (2 * t + 1 < nblocks) step(BV{}, BK{}, 2 * t + 1, 1);
        } else if (active) {
#pragma unroll
            for (int q = 0; q < kBlocksPerTile; ++q) {
                const int i = 2 * t + q;
                if (i < nblocks && i % nshare == sidx) shared_step(BV{}, i, q);
            }
        }
        if constexpr (TAIL)
            if (tail_on && wave < 4) tail_step(BV{}, t);
        PRESTO_WAIT_VM(2 * LPT);
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave's LDS reads are done
        __builtin_amdgcn_s_barrier();
    };

    // prologue: tiles 0..2 requested, tiles 0 and 1 awaited (and with them
    // Q and the ancestor rows, which were requested first)
    load_tile(k_begin, 0);
    load_tile(k_begin + kKeyTile, 1);
    load_tile(k_begin + 2 * kKeyTile, 2);
    PRESTO_WAIT_VM(2 * LPT);
    __syncthreads();
    using B0 = std::integral_constant<int, 0>;
    if (active && !shared) {
        floatx16 S0 = negm;
        qk(B0{}, 0, S0);
        if (masked(0)) apply_mask(S0, j0_of(0));
        float ls;
        exact(S0, Pp, ls, true, Sb);  // m from block 0; Sb not yet live
        l_run = ls;
        qk(B0{}, 1, Sa);
    }
    for (int t = 0; t < ntiles; t += kRing) {
        tile(std::integral_constant<int, 0>{}, t);
        if (t + 1 < ntiles) tile(std::integral_constant<int, 1>{}, t + 1);
        if (t + 2 < ntiles) tile(std::integral_constant<int, 2>{}, t + 2);
        if (t + 3 < ntiles) tile(std::integral_constant<int, 3>{}, t + 3);
    }
    PRESTO_WAIT_VM(0);  // no load into LDS outlives the workgroup
#undef PRESTO_WAIT_VM

    // ---- the shared block's states, combined pairwise through the (now
    // idle) tile ring: per round the waves at odd multiples of `stride` write
    // (m, l, O) and their partners fold them in
    if (nshare > 1) {
        constexpr int SLOT = kWave * (16 * DB + 2);  // floats per written state
        float* s_state = reinterpret_cast<float*>(s_kv);
        for (int stride = 1; stride < nshare; stride *= 2) {
            __syncthreads();  // every wave's loads have landed; the ring is free
            const bool writer = shared && (sidx % (2 * stride)) == stride;
            const bool reader = shared && (sidx % (2 * stride)) == 0 && sidx + stride < nshare;
            if (writer) {
                float* st = s_state + (sidx / (2 * stride)) * SLOT + lane;
                st[0] = m;
                st[kWave] = l_run;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int e = 0; e < 16; ++e) st[(2 + db * 16 + e) * kWave] = o[db][e];
            }
            __syncthreads();
            if (reader) {
                const float* st = s_state + (sidx / (2 * stride)) * SLOT + lane;
                const float m2 = st[0], l2 = st[kWave];
                const float M = l_run > 0.f ? (l2 > 0.f ? fmaxf(m, m2) : m) : m2;
                const float a1 = l_run > 0.f ? __builtin_amdgcn_exp2f(m - M) : 0.f;
                const float a2 = l2 > 0.f ? __builtin_amdgcn_exp2f(m2 - M) : 0.f;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int e = 0; e < 16; ++e) o[db][e] = a1 * o[db][e] + a2 * st[(2 + db * 16 + e) * kWave];
                l_run = a1 * l_run + a2 * l2;
                m = M;
            }
        }
    }

    // ---- the tail's four states, combined through the (now idle) tile ring
    if constexpr (TAIL) {
        if (tail_here) {
            float* s_to = reinterpret_cast<float*>(s_kv);     // [4][16 rows][D]
            float* s_tml = s_to + 4 * 16 * D;                 // [4][16 rows] m, then l
            __syncthreads();  // every wave's loads have landed; the ring is free
            if (tail_on && wave < 4) {
                const auto h16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(tl), __float_as_uint(tl), false, false);
                float ls = __uint_as_float(h16[0]) + __uint_as_float(h16[1]);
                const auto h32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(ls), __float_as_uint(ls), false, false);
                ls = __uint_as_float(h32[0]) + __uint_as_float(h32[1]);
                if (tq == 0) {
                    s_tml[wave * 16 + t16] = tm;
                    s_tml[64 + wave * 16 + t16] = ls;
                }
#pragma unroll
                for (int i = 0; i < TD; ++i)
                    *reinterpret_cast<floatx4*>(&s_to[(wave * 16 + t16) * D + 16 * i + 4 * tq]) = ot[i];
            }
            __syncthreads();
            for (int i = tid; i < 16 * (D / 4); i += NT) {
                const int r = i / (D / 4), d = i % (D / 4) * 4;
                const int tr = tail0 + r;
                if (tr >= all_rows) break;
                float M = -INFINITY, L = 0.f;
                floatx4 acc = {0.f, 0.f, 0.f, 0.f};
                if (tail_on) {
#pragma unroll
                    for (int w = 0; w < 4; ++w) M = fmaxf(M, s_tml[w * 16 + r]);
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const float mw = s_tml[w * 16 + r];
                        const float f = mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw - M);
                        L += f * s_tml[64 + w * 16 + r];
                        acc += f * *reinterpret_cast<const floatx4*>(&s_to[(w * 16 + r) * D + d]);
                    }
                }
                acc *= L > 0.f ? 1.f / L : 0.f;
                // (rows of padding nodes are zeros whatever their q holds)
                const uint2 o2 = tr < live_rows
                                     ? make_uint2(pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3]))
                                     : make_uint2(0u, 0u);
                if (a.splits == 1) {
                    uint16_t* op = a.out + (((int64_t)b * a.n_max + tr / a.G) * a.hq + g * a.G + tr % a.G) * D + d;
                    *reinterpret_cast<uint2*>(op) = o2;
                } else {
                    *reinterpret_cast<uint2*>(a.part_o + (part_row + tr) * D + d) = o2;
                    if (d == 0) a.part_ml[ml_row + (int64_t)tr * ml_stride] = make_float2(L > 0.f ? M : -INFINITY, L);
                }
            }
        }
    }

    // ---- epilogue: lane holds row l32, d = db*32 + 8(i/4) + 4h + i%4
    // the blocks past the shared one hold padding rows only, which without a
    // merge are the waves' own to clear
    if (!SHARES && a.splits == 1 && nshare > 1 && wave >= A) {
        const int r = rt * RT + wave * kRowsPerWave + l32;
        if (wave * kRowsPerWave < RT && r < all_rows && (!TAIL || r < tail0)) {
            uint16_t* op = a.out + (((int64_t)b * a.n_max + r / a.G) * a.hq + g * a.G + r % a.G) * D;
#pragma unroll
            for (int e = 0; e < D / 16; ++e)
                *reinterpret_cast<uint4*>(op + (2 * e + h) * 8) = make_uint4(0u, 0u, 0u, 0u);
        }
    }
    if (shared && sidx != 0) return;  // a shared block's combined state is wave A-1's
    if (rho >= all_rows || (TAIL && rho >= tail0)) return;
    const float l = l_run;  // whole-row sum
    if (!SHARES && a.splits == 1) {
        uint16_t* op = a.out + (((int64_t)b * a.n_max + qn) * a.hq + g * a.G + qh) * D;
        const float inv = l > 0.f ? 1.f / l : 0.f;
        const bool is_live = rho < live_rows;  // rows of padding nodes are zeros whatever their q holds
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const int dd = db * 32 + 8 * q4 + 4 * h;
                const uint2 v = make_uint2(pack_bf16x2(o[db][4 * q4] * inv, o[db][4 * q4 + 1] * inv),
                                           pack_bf16x2(o[db][4 * q4 + 2] * inv, o[db][4 * q4 + 3] * inv));
                *reinterpret_cast<uint2*>(op + dd) = is_live ? v : make_uint2(0u, 0u);
            }
    } else {
        // normalised here, so bf16 holds it to the output's own precision
        // (a workgroup's rows are contiguous: whole lines; the merge reads a
        // row's (m, l) pairs side by side)
        uint16_t* po = a.part_o + (part_row + rho) * D;
        const float inv = l > 0.f ? 1.f / l : 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const int dd = db * 32 + 8 * q4 + 4 * h;
                *reinterpret_cast<uint2*>(po + dd) =
                    make_uint2(pack_bf16x2(o[db][4 * q4] * inv, o[db][4 * q4 + 1] * inv),
                               pack_bf16x2(o[db][4 * q4 + 2] * inv, o[db][4 * q4 + 3] * inv));
            }
        if (h == 0) a.part_ml[ml_row + (int64_t)rho * ml_stride] = make_float2(l > 0.f ? m : -INFINITY, l);
    }
    };

    const int all = a.G * a.n_max;
    const int item = task / a.row_tiles / a.hkv;
    if constexpr (!SHARES) {
        // task = ((b * splits + split') * hkv + g) * row_tiles + rt with the
        // splits in reverse (split' = 0 is the last split): the XCDs start
        // their workgroups a few microseconds apart in XCD order, and the
        // last split, which holds the tree keys and their masks and so runs
        // longest, then lands on the XCDs that start first.
        int split = a.splits - 1 - item % a.splits;
        int b = item / a.splits;
        if constexpr (!TAIL) {
            if (a.pairs) {
                // item = the pair's index in sequence order, splits in reverse as well
                b = -1;
                for (int b0 = 0, base = 0; b0 < a.batch && b < 0; b0 += kWave) {
                    const int n = live_splits(a, b0 + lane_id()), incl = (int)wave_scan_dpp(n);
                    const uint64_t hit = __ballot(base + incl > item);
                    if (hit) {
                        const int l = __ffsll((unsigned long long)hit) - 1;
                        b = b0 + l;
                        split = base + __builtin_amdgcn_readlane(incl, l) - 1 - item;
                    } else {
                        base += __builtin_amdgcn_readlane(incl, kWave - 1);
                    }
                }
                if (b < 0) return;
            }
        }
        const int64_t bg = (int64_t)b * a.hkv + g;
        segment(b, split * a.split_len, (split + 1) * a.split_len, (bg * a.splits + split) * all,
                bg * all * a.splits + split, a.splits);
        return;
    }
    // task = (share * hkv + g) * row_tiles + rt
    const TileShares sh(share_total(a), a.shares);
    int from = sh.begin(item);
    const int to = sh.begin(item + 1);
    if (from >= to) return;
    int b = -1, base = 0;  // the sequence and its first tile
    for (int b0 = 0; b0 < a.batch && b < 0; b0 += kWave) {
        const int n = share_tiles(a, b0 + lane_id()), incl = (int)wave_scan_dpp(n);
        const uint64_t hit = __ballot(base + incl > from);
        if (hit) {
            const int l = __ffsll((unsigned long long)hit) - 1;
            b = b0 + l;
            base += __builtin_amdgcn_readlane(incl - n, l);
        } else {
            base += __builtin_amdgcn_readlane(incl, kWave - 1);
        }
    }
    if (b < 0) return;
    while (true) {
        const int tiles = __builtin_amdgcn_readfirstlane(share_tiles(a, b));
        const int slot = item + b;
        const int t0 = max(from - base - kLeadTiles, 0), t1 = min(to - base, tiles) - kLeadTiles;
        // the merge's note of the sequence's first and last part
        if (rt == 0 && g == 0 && t1 > t0 && threadIdx.x == 0) {
            if (t0 == 0) a.slots[b].x = slot;
            if (t1 == tiles - kLeadTiles) a.slots[b].y = slot;
        }
        if (t1 > t0)
            segment(b, t0 * kKeyTile, t1 * kKeyTile, ((int64_t)slot * a.hkv + g) * all,
                    (int64_t)g * all * a.n_slots + slot, a.n_slots);
        base += tiles;
        if (base >= to) return;
        from = base;
        ++b;
        __syncthreads();  // the tile ring and the ancestor rows are free again
    }
}

// Merge of the split partials.  D / E lanes per query row, E dims each; every
// lane weighs its row's splits itself, l exp2(m - M), kMergeUnroll of them with
// all loads in flight.  Eight dims (16-byte loads, four or eight rows per wave)
// where that makes a workgroup per CU: memory latency and the partials' bytes
// bound those (split by split with one wave per row and 4-byte loads, weights
// across the lanes, 12.9 us for 16 ragged sequences of 33 nodes, three partials
// per row, and 20.7 us for 4 of 257 nodes, 8 partials; 6.6 and 14.3 now).  A
// small grid has one wave per SIMD, which spends its time on the weights and
// sums (about 25 vector instructions per split and lane), so two dims per lane
// spread it over four times the waves: whole calls of 1 x 4096 keys, 33 nodes
// 22.3 -> 21.8 us, 9 nodes at 2048 keys 17.3 -> 16.4 (72 and 24 workgroups of
// eight dims); at 136 (65 nodes) the merge takes 4.45 us with eight and 4.85
// with two in a round, at 264 (129 nodes) the call 30.2 and 30.7.
constexpr int kMergeUnroll = 8;
template <int E>
struct Bf16Chunk {
    typedef uint32_t type __attribute__((ext_vector_type(E / 2)));
};
template <int D, int E>
__global__ __launch_bounds__(256) void tree_attn_merge_kernel(AttnArgs a) {
    typedef typename Bf16Chunk<E>::type chunk;
    constexpr int LPR = D / E;          // lanes per row
    constexpr int RPB = 256 / LPR;      // rows per workgroup
    // grid: x covers the rows of one (sequence, KV head), y the (sequence, KV
    // head) pairs
    const int rows_g = a.G * a.n_max;
    const int rho = (int)blockIdx.x * RPB + (int)threadIdx.x / LPR;
    const int dl = (int)threadIdx.x % LPR;
    if (rho >= rows_g) return;
    const int bg = (int)blockIdx.y;
    const int b = bg / a.hkv, g = bg - b * a.hkv;
    const int n = rho / a.G, hh = rho - n * a.G;
    const uint16_t* po;  // this lane's dims of the row's first partial
    int64_t sstride;     // elements from one partial of the row to the next
    const float2* mlp;   // the row's (m, l) pairs
    int nsplit;
    const int nn_raw = a.n_nodes[b];
    if (a.shares == 0) {
        po = a.part_o + ((int64_t)bg * a.splits * rows_g + rho) * D + dl * E;
        sstride = (int64_t)rows_g * D;
        mlp = a.part_ml + ((int64_t)bg * rows_g + rho) * a.splits;
        nsplit = a.splits;  // cut below, once the loads are on their way
    } else {
        const int2 s = a.slots[b];
        nsplit = s.y - s.x + 1;
        po = a.part_o + (((int64_t)s.x * a.hkv + g) * rows_g + rho) * D + dl * E;
        sstride = (int64_t)a.hkv * rows_g * D;
        mlp = a.part_ml + ((int64_t)g * rows_g + rho) * a.n_slots + s.x;
    }
    float M = -INFINITY, L = 0.f;
    float acc[E];
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = 0.f;
    const int last = nsplit - 1;
    for (int s0 = 0; s0 < nsplit; s0 += kMergeUnroll) {
        float2 ml[kMergeUnroll];
        chunk v[kMergeUnroll];
#pragma unroll
        for (int u = 0; u < kMergeUnroll; ++u) {
            const int sp = min(s0 + u, last);
            ml[u] = mlp[sp];
            v[u] = *reinterpret_cast<const chunk*>(po + (int64_t)sp * sstride);
        }
        if (s0 == 0 && a.shares == 0) {
            // splits past the sequence's end left nothing
            const int keys = ctx_span(a.ctx_off, b, a.ctx_slots).ctx + clamp_nodes(nn_raw, a.n_max);
            nsplit = min(nsplit, (keys + a.split_len - 1) / a.split_len);
        }
        float Mn = M;
#pragma unroll
        for (int u = 0; u < kMergeUnroll; ++u)
            if (s0 + u < nsplit) Mn = fmaxf(Mn, ml[u].x);
        const float old = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - Mn);
        L *= old;
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] *= old;
        M = Mn;
#pragma unroll
        for (int u = 0; u < kMergeUnroll; ++u) {
            if (s0 + u < nsplit) {
                const float w = ml[u].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[u].x - Mn) * ml[u].y;
                L += w;
#pragma unroll
                for (int e = 0; e < E / 2; ++e) {
                    acc[2 * e] = fmaf(w, bf16lo(v[u][e]), acc[2 * e]);
                    acc[2 * e + 1] = fmaf(w, bf16hi(v[u][e]), acc[2 * e + 1]);
                }
            }
        }
    }
    // rows of padding nodes are zeros; a live row whose every partial is NaN (no
    // part has a maximum then, so L is 0) stays NaN
    const bool live = n < clamp_nodes(nn_raw, a.n_max);
    const float inv = L > 0.f ? 1.f / L : 0.f;
    chunk o;
#pragma unroll
    for (int e = 0; e < E / 2; ++e) o[e] = live ? pack_bf16x2(acc[2 * e] * inv, acc[2 * e + 1] * inv) : 0u;
    uint16_t* op = a.out + (((int64_t)b * a.n_max + n) * a.hq + g * a.G + hh) * D + dl * E;
    *reinterpret_cast<chunk*>(op) = o;
}

// fp32 path, on the fp32 matrix cores (v_mfma_f32_32x32x2_f32: exact fp32
// products, fp32 accumulation), fp32 throughout.  A workgroup serves 32 query
// rows of one KV head (packed as in the bf16 kernel) over one range of keys;
// its four waves take every fourth 32-key block and combine their (m, l, O)
// through LDS.  Scores are computed transposed, S^T = K Q^T, so a lane holds
// one row and 16 of a block's keys, and the probabilities are the B operand of
// O^T = V^T P^T as they are: an MFMA contracts two keys (or two head
// dimensions), one from each half of the wave, and since the order of a
// contraction and of the output rows is free, each lane reads 16 contiguous
// bytes of a K row per four MFMAs (dimensions 8 j + 4 h + 0 .. 3) and D / 32
// contiguous floats of a V row per key.  A block of 32 x 32 takes 2 x 64
// MFMAs of 64 cycles, 8192 in all, for 32 KB of K/V: the matrix cores bound
// it, so K and V come straight from global memory (16 B per clock and CU out
// of the L2), K of the next block under the current P V, V under the scores.
// Q sits in LDS to leave the registers to the loads in flight.
// 2 sequences x 2048 keys, 33 nodes, 32/8 heads of 128: 701 us with one wave
// per query row and a key per lane (uncoalesced reads, each row reading all
// of K and V), 45 now (the matrix cores busy 37% of the cycles; the rest is
// the first blocks' arrival, which all workgroups wait for at once, the
// exponentials of two waves per SIMD and the combination).  8 x 16384 keys, 32
// nodes: 67% of the cycles, 86 TFLOP/s (a large fp32 matrix product reaches 148
// on this card).
struct AttnF32Args {
    const float* q;
    const float* kc;
    const float* vc;
    const int32_t* ctx_off;
    int32_t ctx_slots;
    const float* kt;
    const float* vt;
    const uint64_t* anc;
    const int32_t* n_nodes;
    float* out;
    float* part_o;    // splits > 1: [b, g, split, row, D], normalised
    float2* part_ml;  // [b, g, row, split]
    int32_t n_max, hq, hkv, G, W;
    int32_t row_blocks, splits, split_len;  // split_len: keys, a multiple of 32
    int32_t n_tasks, n_blocks;
    float scale;
};

constexpr int kF32Waves = 4;

template <int N>
struct FloatVec {
    // rows are only 4-byte aligned in general
    typedef float type __attribute__((ext_vector_type(N), aligned(4)));
};

template <int D>
__global__ __launch_bounds__(kF32Waves * kWave, 2) void tree_attn_f32_kernel(AttnF32Args a) {
    constexpr int NW = kF32Waves, NT = NW * kWave;
    constexpr int KJ = D / 8;   // 16-byte chunks of a K row per lane
    constexpr int DB = D / 32;  // 32-row blocks of O^T
    constexpr int QC = D / 4;   // 16-byte chunks of a Q row
    constexpr int SLOT = kWave * (16 * DB + 2);  // floats of a wave's state
    typedef typename FloatVec<4>::type f4;
    typedef typename FloatVec<DB>::type fdb;
    typedef float f4a __attribute__((ext_vector_type(4)));
    // Q rows, chunk c of row r at c ^ r (sixteen rows read one chunk each:
    // different banks); after the key loop the waves' states
    __shared__ __align__(16) float s_mem[NW / 2 * SLOT > 32 * D ? NW / 2 * SLOT : 32 * D];
    __shared__ int s_odd;  // a live row's sums are not all finite

    const int task = xcd_task(blockIdx.x, a.n_blocks);
    if (task >= a.n_tasks) return;
    // task = ((b * hkv + g) * splits + split) * row_blocks + rb: the row
    // blocks that read the same keys share an XCD and its L2
    const int rb = task % a.row_blocks;
    const int split = task / a.row_blocks % a.splits;
    const int bg = task / a.row_blocks / a.splits;
    const int b = bg / a.hkv, g = bg - b * a.hkv;
    const int tid = threadIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int l32 = lane & 31, h = lane >> 5;

    const CtxSpan cs = ctx_span(a.ctx_off, b, a.ctx_slots);
    const int c0 = cs.c0, ctx = cs.ctx;
    const int nn = clamp_nodes(a.n_nodes[b], a.n_max);
    const int keys = ctx + nn;
    const int live = a.G * nn, all_rows = a.G * a.n_max;
    const int k_begin = split * a.split_len;
    if (k_begin >= keys) return;  // the merge does not read this split of b
    const int k_end = min(keys, k_begin + a.split_len);
    const int nblk = (k_end - k_begin + 31) / 32;

    const int row0 = rb * 32, rho = row0 + l32;
    const int qn = rho / a.G, qh = rho - qn * a.G;
    const bool is_live = rho < live;
    if (row0 >= live) {
        // padding nodes only: zeros (the merge writes them when there is one)
        if (a.splits == 1)
            for (int i = tid; i < 32 * D; i += NT) {
                const int r = row0 + i / D;
                if (r < all_rows)
                    a.out[(((int64_t)b * a.n_max + r / a.G) * a.hq + g * a.G + r % a.G) * D + i % D] = 0.f;
            }
        return;
    }
    const uint64_t* arow = a.anc + ((int64_t)b * a.n_max + min(qn, a.n_max - 1)) * a.W;
    const int64_t tree_row0 = (int64_t)b * a.n_max;
    // row `key` of this KV head (keys past the end repeat the last one, masked)
    auto row_of = [&](const float* cache, const float* tree, int key) __attribute__((always_inline)) {
        const int kk = min(key, k_end - 1);
        const bool in_ctx = kk < ctx;
        const int64_t r = in_ctx ? (int64_t)(c0 + kk) : tree_row0 + (kk - ctx);
        return (in_ctx ? cache : tree) + (r * a.hkv + g) * D;
    };
    const int64_t stride = (int64_t)a.hkv * D;  // from one key's row to the next
    auto load_k = [&](int j0, f4 (&kr)[KJ]) __attribute__((always_inline)) {
        const float* kp = row_of(a.kc, a.kt, j0 + l32) + 4 * h;
#pragma unroll
        for (int j = 0; j < KJ; ++j) kr[j] = *reinterpret_cast<const f4*>(kp + 8 * j);
    };
    // V of keys 8 (i / 4) + 4 h + i % 4, i = 8 part .. 8 part + 7
    auto load_v = [&](int j0, int part, fdb (&vr)[8]) __attribute__((always_inline)) {
        if (j0 + 32 <= min(ctx, k_end)) {
            const float* vp = a.vc + ((int64_t)(c0 + j0 + 16 * part + 4 * h) * a.hkv + g) * D + DB * l32;
#pragma unroll
            for (int i = 0; i < 8; ++i) vr[i] = *reinterpret_cast<const fdb*>(vp + (8 * (i / 4) + i % 4) * stride);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int e = 8 * part + i;
                vr[i] = *reinterpret_cast<const fdb*>(row_of(a.vc, a.vt, j0 + 8 * (e / 4) + 4 * h + e % 4) + DB * l32);
            }
        }
    };
    auto swap_half = [&](float v) {
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        return __uint_as_float(h == 0 ? sw[1] : sw[0]);
    };

    floatx16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[db][e] = 0.f;
    float m = -INFINITY, l = 0.f;
    if (tid == 0) s_odd = 0;
    f4 kr[KJ];
    if (wave < nblk) load_k(k_begin + 32 * wave, kr);  // in flight under the staging of Q
    for (int i = tid; i < 32 * QC; i += NT) {
        const int r = i / QC, c = i % QC;
        const int rr = min(row0 + r, all_rows - 1);
        const float* qp = a.q + (((int64_t)b * a.n_max + rr / a.G) * a.hq + g * a.G + rr % a.G) * D;
        const f4 v = *reinterpret_cast<const f4*>(qp + 4 * c);
        *reinterpret_cast<f4a*>(&s_mem[r * D + 4 * (c ^ (r & (QC - 1)))]) = v;
    }
    __syncthreads();

    for (int i = wave; i < nblk; i += NW) {
        const int j0 = k_begin + 32 * i;
        asm volatile("" ::: "memory");  // Q is read anew per block, not kept in (spilled) registers
        fdb va[8], vb[8];
        load_v(j0, 0, va);
        floatx16 S;
#pragma unroll
        for (int e = 0; e < 16; ++e) S[e] = 0.f;
#pragma unroll
        for (int j = 0; j < KJ; ++j) {
            const f4a qv = *reinterpret_cast<const f4a*>(&s_mem[l32 * D + 4 * ((2 * j + h) ^ (l32 & (QC - 1)))]);
#pragma unroll
            for (int c = 0; c < 4; ++c) S = __builtin_amdgcn_mfma_f32_32x32x2f32(kr[j][c], qv[c], S, 0, 0, 0);
        }
        load_v(j0, 1, vb);
#pragma unroll
        for (int e = 0; e < 16; ++e) S[e] *= a.scale;
        if (j0 + 32 > min(ctx, k_end)) {
            // visible keys of this lane's row: the context, then its ancestors
            uint32_t anc = 0u;
            const int s0 = j0 - ctx;  // tree index of the block's first key
            if (j0 + 32 > ctx) {
                if (s0 >= 0) {
                    const int w = s0 >> 6, sh = s0 & 63;
                    const uint64_t lo = w < a.W ? arow[w] : 0ull, hi = w + 1 < a.W ? arow[w + 1] : 0ull;
                    anc = (uint32_t)(sh == 0 ? lo : (lo >> sh) | (hi << (64 - sh)));
                } else {
                    anc = (uint32_t)(arow[0] << (-s0));
                }
            }
            const int nctx = ctx - j0, nend = k_end - j0;
            const uint32_t ctx_mask = nctx >= 32 ? ~0u : (nctx <= 0 ? 0u : (1u << nctx) - 1u);
            const uint32_t end_mask = nend >= 32 ? ~0u : (1u << nend) - 1u;
            const uint32_t vis = ((ctx_mask | anc) & end_mask) >> (4 * h);
#pragma unroll
            for (int e = 0; e < 16; ++e) S[e] = ((vis >> (8 * (e >> 2) + (e & 3))) & 1u) ? S[e] : -INFINITY;
        }
        float mx = S[0];
#pragma unroll
        for (int e = 1; e < 16; ++e) mx = fmaxf(mx, S[e]);
        mx = fmaxf(mx, swap_half(mx));
        if (__ballot(mx > m)) {
            const float mn = fmaxf(m, mx);
            const float al = m == -INFINITY ? 0.f : expf(m - mn);
            l *= al;
#pragma unroll
            for (int db = 0; db < DB; ++db) o[db] *= al;
            m = mn;
        }
        const float mr = m == -INFINITY ? 0.f : m;  // no key visible yet: every term is 0
        float ls = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            S[e] = expf(S[e] - mr);
            ls += S[e];
        }
        l += ls + swap_half(ls);
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int db = 0; db < DB; ++db)
                o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[e][db], S[e], o[db], 0, 0, 0);
        if (i + NW < nblk) load_k(j0 + 32 * NW, kr);
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int db = 0; db < DB; ++db)
                o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vb[e][db], S[8 + e], o[db], 0, 0, 0);
    }

    // A tree node that a row does not see takes no part in it, whatever its V
    // holds, but the MFMAs have added 0 times that, NaN where V is not finite.
    // Where a live row's sums are not all finite, the workgroup starts over key
    // by key (looked for here: a test of V within the key loop cost it 8%).
    float odd[4] = {0.f, 0.f, 0.f, 0.f};  // NaN once a sum is not finite
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) odd[e & 3] = fmaf(o[db][e], 0.f, odd[e & 3]);
    const float any = (odd[0] + odd[1]) + (odd[2] + odd[3]);
    if (__ballot(is_live && any != any)) s_odd = 1;
    __syncthreads();
    if (__builtin_expect(s_odd, 0)) {
        // one row per wave at a time, 64 keys per step, a key per lane for the
        // score and D / 64 dimensions per lane for the output
        constexpr int PER = D / kWave;
        for (int r = wave; r < 32 && row0 + r < all_rows; r += NW) {
            const int row = row0 + r, n = row / a.G;
            const uint64_t* ar = a.anc + ((int64_t)b * a.n_max + n) * a.W;
            float m1 = -INFINITY, l1 = 0.f, acc[PER];
#pragma unroll
            for (int e = 0; e < PER; ++e) acc[e] = 0.f;
            for (int j0 = k_begin; j0 < k_end && n < nn; j0 += kWave) {
                const int j = j0 + lane, s = j - ctx;
                const bool vis = j < k_end && (s < 0 || ((ar[s >> 6] >> (s & 63)) & 1ull));
                const float* kp = row_of(a.kc, a.kt, j);
                float x = 0.f;
                for (int d = 0; d < D; ++d) x = fmaf(s_mem[r * D + 4 * ((d >> 2) ^ (r & (QC - 1))) + (d & 3)], kp[d], x);
                x = vis ? x * a.scale : -INFINITY;
                const float mn = fmaxf(m1, wave_max_f32_dpp(x));
                const float al = m1 == -INFINITY ? 0.f : expf(m1 - mn);
                const float pj = expf(x - (mn == -INFINITY ? 0.f : mn));
                m1 = mn;
                l1 = l1 * al + wave_sum_f32_dpp(pj);
#pragma unroll
                for (int e = 0; e < PER; ++e) acc[e] *= al;
                for (uint64_t left = __ballot(vis); left != 0ull; left &= left - 1ull) {
                    const int t = __ffsll((unsigned long long)left) - 1;
                    const float pt = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(pj), t));
                    const float* vp = row_of(a.vc, a.vt, j0 + t) + lane * PER;
#pragma unroll
                    for (int e = 0; e < PER; ++e) acc[e] = fmaf(pt, vp[e], acc[e]);
                }
            }
            const float inv = l1 == 0.f ? 0.f : 1.f / l1;
            float* op;
            if (a.splits == 1) {
                op = a.out + (((int64_t)b * a.n_max + n) * a.hq + g * a.G + row % a.G) * D;
            } else {
                op = a.part_o + (((int64_t)bg * a.splits + split) * all_rows + row) * D;
                if (lane == 0) a.part_ml[((int64_t)bg * all_rows + row) * a.splits + split] = make_float2(m1, l1);
            }
#pragma unroll
            for (int e = 0; e < PER; ++e) op[lane * PER + e] = acc[e] * inv;
        }
        return;
    }

    // the waves' states, combined pairwise: odd multiples of `step` write,
    // their partners fold them in
#pragma unroll
    for (int step = 1; step < NW; step *= 2) {
        if (step > 1) __syncthreads();
        float* st = s_mem + wave / (2 * step) * SLOT + lane;
        if (wave % (2 * step) == step) {
            st[0] = m;
            st[kWave] = l;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int e = 0; e < 16; ++e) st[(2 + db * 16 + e) * kWave] = o[db][e];
        }
        __syncthreads();
        if (wave % (2 * step) == 0) {
            const float m2 = st[0], l2 = st[kWave];
            const float M = fmaxf(m, m2);
            const float a1 = m == -INFINITY ? 0.f : expf(m - M), a2 = m2 == -INFINITY ? 0.f : expf(m2 - M);
            l = a1 * l + a2 * l2;
            m = M;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int e = 0; e < 16; ++e) o[db][e] = a1 * o[db][e] + a2 * st[(2 + db * 16 + e) * kWave];
        }
    }
    if (wave != 0 || rho >= all_rows) return;
    // lane: row l32, dimensions DB (8 (e / 4) + 4 h + e % 4) + db
    // (a row that sees no key of this split leaves zeros; rows of padding nodes
    // are zeros whatever their q holds)
    const float inv = l == 0.f ? 0.f : 1.f / l;
    float* op;
    if (a.splits == 1) {
        op = a.out + (((int64_t)b * a.n_max + qn) * a.hq + g * a.G + qh) * D;
    } else {
        op = a.part_o + (((int64_t)bg * a.splits + split) * all_rows + rho) * D;
        if (h == 0) a.part_ml[((int64_t)bg * all_rows + rho) * a.splits + split] = make_float2(m, l);
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        fdb v;
#pragma unroll
        for (int db = 0; db < DB; ++db) v[db] = is_live ? o[db][e] * inv : 0.f;
        *reinterpret_cast<fdb*>(op + DB * (8 * (e >> 2) + 4 * h + (e & 3))) = v;
    }
}

// Merge of the fp32 split partials: one wave per query row, lane s weighs
// split s by l exp(m - M); dead rows are written as zeros.
template <int D>
__global__ __launch_bounds__(256) void tree_attn_f32_merge_kernel(AttnF32Args a) {
    constexpr int PER = D / kWave;
    const int lane = lane_id();
    const int rows = a.G * a.n_max;
    const int rho = (int)blockIdx.x * (blockDim.x / kWave) + (int)threadIdx.x / kWave;
    if (rho >= rows) return;
    const int bg = (int)blockIdx.y;
    const int b = bg / a.hkv, g = bg - b * a.hkv;
    const int n = rho / a.G, hh = rho - n * a.G;
    const int nn = clamp_nodes(a.n_nodes[b], a.n_max);
    const int keys = ctx_span(a.ctx_off, b, a.ctx_slots).ctx + nn;
    const int nsplit = min(a.splits, (keys + a.split_len - 1) / a.split_len);
    float acc[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) acc[e] = 0.f;
    if (n < nn) {
        float2 ml = make_float2(-INFINITY, 0.f);
        if (lane < nsplit) ml = a.part_ml[((int64_t)bg * rows + rho) * a.splits + lane];
        const float M = wave_max_f32_dpp(ml.x);
        // (a sum without a maximum is 0, or NaN where no score is a number)
        const float wl = ml.x == -INFINITY ? ml.y : expf(ml.x - M) * ml.y;
        const float L = wave_sum_f32_dpp(wl);
        const float* po = a.part_o + ((int64_t)bg * a.splits * rows + rho) * D + lane * PER;
        for (int s = 0; s < nsplit; ++s) {
            const float w = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wl), s));
#pragma unroll
            for (int e = 0; e < PER; ++e) acc[e] += w * po[(int64_t)s * rows * D + e];
        }
#pragma unroll
        for (int e = 0; e < PER; ++e) acc[e] /= L;
    }
    float* op = a.out + (((int64_t)b * a.n_max + n) * a.hq + g * a.G + hh) * D + lane * PER;
#pragma unroll
    for (int e = 0; e < PER; ++e) op[e] = acc[e];
}

}  // namespace presto

namespace presto_host {

using namespace presto;

struct AttnPlan {
    int G, rows, row_tiles, rows_per_tile, splits, split_len;
    int shares, n_slots;  // shares > 0: equal shares of a ragged batch's key tiles
    bool tail;            // 1 .. 16 rows past the last full tile, taken along by it
    bool pairs;           // workgroups dealt over the (sequence, split) pairs that exist
    double cost;          // modelled time, in 32-key blocks of a workgroup of 256 rows
    int64_t tasks, blocks;
    bool merged() const { return shares > 0 || splits > 1; }
    // query rows that leave a partial
    size_t partial_rows(const presto_attn_desc* d) const {
        return (size_t)(shares > 0 ? n_slots : d->batch * (int64_t)splits) * d->hkv * rows;
    }
};

static bool attn_ragged(const presto_attn_desc* d) {
    return d->batch > 1 && d->total_ctx > 0 && d->total_ctx < (int64_t)d->batch * d->max_ctx;
}

constexpr int kMaxSplits = 64;  // searched; the fastest found is at most about 30

// Row tiles and context splits: one workgroup per CU, so the time in key-block
// units (about 0.85 us each) is (rounds of workgroups) x (key blocks per split
// + about 3 for a workgroup's prologue) plus the merge, whose partials (2 D + 8
// bytes per query row and split, written and read back, about 4 MB per
// key-block time) grow with the split count.  tail: without a row tile for the
// rows past the last full one.  pairs: workgroups only for the (sequence,
// split) pairs that exist, about total / len + batch / 2 of them.
static AttnPlan attn_plan_split(const presto_attn_desc* d, bool tail, bool pairs, int most) {
    AttnPlan p;
    p.G = d->hq / d->hkv;
    p.rows = p.G * d->n_max;
    p.rows_per_tile = kAttnRows;
    p.tail = tail;
    p.pairs = pairs;
    p.row_tiles = p.tail ? p.rows / p.rows_per_tile : (p.rows + p.rows_per_tile - 1) / p.rows_per_tile;
    const int64_t per_pair = (int64_t)d->hkv * p.row_tiles;  // workgroups per (sequence, split)
    const int keys = d->max_ctx + d->n_max;                  // the longest sequence
    const double total_keys = (double)d->total_ctx + (double)d->batch * d->n_max;
    const int max_splits = (keys + 127) / 128;
    const double row_bytes = 2.0 * d->head_dim + 8.0;
    p.cost = 1e30;
    p.shares = p.n_slots = 0;
    p.splits = 1;
    p.split_len = (keys + kKeyTile - 1) / kKeyTile * kKeyTile;
    for (int s = 1; s <= most && s <= max_splits; ++s) {
        int len = (keys + s - 1) / s;
        len = (len + kKeyTile - 1) / kKeyTile * kKeyTile;
        const int se = (keys + len - 1) / len;
        const double all = (double)d->batch * se;
        const double n = pairs ? fmin(all, total_keys / len + 0.5 * d->batch) : all;
        const double rounds = ceil(n * per_pair / 256.0);
        const double merge_bytes = se > 1 ? 2.0 * d->hkv * p.rows * n * row_bytes : 0.0;
        const double cost = rounds * ((len + 31) / 32 + 3) + merge_bytes / 4.0e6;
        if (cost < p.cost - 1e-9) {
            p.cost = cost;
            p.splits = se;
            p.split_len = len;
        }
    }
    p.tasks = (int64_t)d->batch * p.splits * per_pair;  // with pairs an upper bound
    p.blocks = (p.tasks + 7) / 8 * 8;
    // When the whole grid fits one round (one workgroup per CU), the tiles
    // are balanced: the same number of row tiles, each a multiple of 32 rows
    // (a 32-row block never straddles two tiles).  260 rows then make tiles
    // of 160 and 100 rows instead of 256 and 4: a workgroup of 256 rows runs
    // two waves per SIMD through every key block (about 1 us per block), one
    // of 160 rows one and a quarter (the idle waves share the fifth block's
    // keys), and the 4-row tiles, nearly idle, disappear.
    if (p.tasks <= 256 && p.row_tiles > 1 && !p.tail && !p.pairs)
        p.rows_per_tile = kRowsPerWave * ((p.rows + kRowsPerWave * p.row_tiles - 1) / (kRowsPerWave * p.row_tiles));
    return p;
}

// Equal shares of all key tiles, one per workgroup of a (KV head, row tile), so
// that no workgroup waits for a longer one.  A few row tiles only: with more
// than 128 workgroups per share there is no choice of their number left.
static AttnPlan attn_plan_shares(const presto_attn_desc* d) {
    AttnPlan p = attn_plan_split(d, false, false, 1);
    p.cost = 1e30;
    const int64_t per_pair = (int64_t)d->hkv * p.row_tiles;
    if (per_pair > 128) return p;
    const double row_bytes = 2.0 * d->head_dim + 8.0;
    const double tiles = ((double)d->total_ctx + (double)d->batch * d->n_max) / kKeyTile +
                         (kLeadTiles + 0.5) * d->batch;
    // per count of rounds, the shares that balance the keys against the merge
    const double merge = 2.0 * d->hkv * p.rows * row_bytes / 4.0e6;  // of one partial per row
    int lo = 1;
    for (int r = 1; lo <= 256 && r * 2.0 * kLeadTiles < p.cost; ++r) {
        const int hi = (int)(256 * r / per_pair < 256 ? 256 * r / per_pair : 256);
        if (hi < lo) continue;
        const double at = sqrt(2.0 * r * tiles / merge);
        const int c0 = at < lo ? lo : (at < hi ? (int)at : hi);
        for (int c = c0; c <= c0 + 1 && c <= hi; ++c) {
            const double cost = r * (2.0 * tiles / c + 2.0 * kLeadTiles) + merge * (c + d->batch);
            if (cost < p.cost - 1e-9) {
                p.cost = cost;
                p.shares = c;
            }
        }
        lo = hi + 1;
    }
    p.n_slots = p.shares + d->batch - 1;
    p.tasks = p.shares * per_pair;
    p.blocks = (p.tasks + 7) / 8 * 8;
    p.rows_per_tile = kAttnRows;
    if (p.tasks <= 256 && p.row_tiles > 1)
        p.rows_per_tile = kRowsPerWave * ((p.rows + kRowsPerWave * p.row_tiles - 1) / (kRowsPerWave * p.row_tiles));
    return p;
}

// fp32: row blocks of 32, and the context split until the grid gives every
// SIMD about two waves (512 workgroups of four); time in key blocks per wave:
// rounds of workgroups x (blocks per wave + about 1 for the prologue and the
// combination), and about 1 for a merge.  2 x 2048 keys, 33 nodes (80 row
// blocks): 6 splits 48 us, against 59 at 2, 47 at 3, 60 at 4, 64 at 8, 71 at
// 16; 1 x 2048 keys, 8 nodes (8 row blocks): 17 splits 22 us, against 54 at 2,
// 28 at 6, 24 at 9, 31 at 33.
struct AttnF32Plan {
    int G, rows, row_blocks, splits, split_len;
    int64_t tasks, blocks;
};

static AttnF32Plan attn_f32_plan(const presto_attn_desc* d, bool may_split) {
    AttnF32Plan p;
    p.G = d->hq / d->hkv;
    p.rows = p.G * d->n_max;
    p.row_blocks = (p.rows + 31) / 32;
    const int64_t per_split = (int64_t)d->batch * d->hkv * p.row_blocks;
    const int blocks = (d->max_ctx + d->n_max + 31) / 32;  // key blocks of the longest sequence
    // the merge's grid.y and its lane per split bound the splits
    const int most = may_split && (int64_t)d->batch * d->hkv <= 65535 ? kWave : 1;
    double best = 1e30;
    p.splits = 1;
    p.split_len = blocks * 32;
    for (int s = 1; s <= most && s * kF32Waves < blocks + kF32Waves; ++s) {
        const int len = (blocks + s - 1) / s;
        const int se = (blocks + len - 1) / len;
        const double cost = ceil((double)per_split * se / 512.0) * ((len + kF32Waves - 1) / kF32Waves + 1.0) +
                            (se > 1 ? 1.0 : 0.0);
        if (cost < best - 1e-9) {
            best = cost;
            p.splits = se;
            p.split_len = len * 32;
        }
    }
    p.tasks = per_split * p.splits;
    p.blocks = (p.tasks + 7) / 8 * 8;
    return p;
}

// part_o bytes (rounded up), then part_ml
static size_t attn_f32_partial_rows(const presto_attn_desc* d, const AttnF32Plan& p) {
    return (size_t)d->batch * d->hkv * p.rows * p.splits;
}

// Plan p of a grid over all (sequence, split) pairs, or the one where 1 .. 16
// query rows past the last full tile ride along with it.  A key block costs a
// workgroup that takes them along about what a full tile's costs, and one of
// balanced tiles of r rows (a grid of one round) 0.22 + 0.64 r / 256 of that,
// one of full tiles in several rounds 0.78: fitted to 173 shapes (1 .. 32 sequences of 1024 .. 32768 keys, 33 .. 1023
// nodes), where no choice is more than 1% slower than tiles of their own.
// us per call, own tiles / riding along: 8 x 8192 keys, 65 nodes 106 / 95;
// 4 x 4096, 65 nodes 39.5 / 43.0; 8 x 4096, 193 nodes (tiles of 224 rows) 120 /
// 155; 8 x 2048, 257 nodes (three rounds of full tiles against one) 128 / 94;
// 32 x 1024, 257 nodes (five against four) 225 / 237.  Short splits
// keep tiles of their own (1 x 4096 keys, 65 nodes: 25.3 / 30.8), and so does a
// grid that is not split without the tail but would be with it (its rows would
// leave bf16 partials instead of one fp32 accumulator).  G >= 2: the ancestor
// rows of a tile then leave room for the tail's queries.
static AttnPlan attn_plan_tail(const presto_attn_desc* d, const AttnPlan& p, int most) {
    if (p.G < 2 || p.rows <= kAttnRows || (p.rows - 1) % kAttnRows >= 16) return p;
    if (p.tasks <= 256 && p.split_len < 1024) return p;
    const AttnPlan t = attn_plan_split(d, true, false, most);
    if (p.splits == 1 && t.splits > 1) return p;
    const double block = p.tasks <= 256 ? 0.22 + 0.64 * p.rows_per_tile / kAttnRows : 0.78;
    return t.cost < block * p.cost ? t : p;
}

// Ragged contexts whose total the caller knows: one of three schedules, by their
// modelled times with a term for what each costs beside its keys.  The terms
// are fitted to 2 .. 128 sequences of 100 .. 32768 keys, the shortest context an
// eighth of the longest, 9 .. 1023 nodes (us per call, pairs / dense / shares;
// dealing pairs whatever the shape was the rule before: no shape measured is
// more than 2% slower than that, most are 5 to 40% faster):
//   dense    the grid of the longest context; workgroups past a sequence's end
//            leave at once.  Short contexts: 8 x 800 keys 23.5 / 21.5 / 22.9,
//            16 x 400 26.2 / 23.1 / 24.7.
//   pairs    6.5 blocks for finding a workgroup's pair.  A few sequences whose
//            pairs make one round: 6 x 5000 keys 33.4 / 37.5 / 35.9.
//   shares   3 blocks for finding a share, 10% for the loop over its parts.
//            Everything longer: 16 x 8192 keys 104 / 101 / 80.
// A batch whose pairs would not be split is not split: one fp32 accumulator from
// a row's first key to its last, no bf16 partials and no merge (32 x 400 keys
// 24.0 / 23.0 / 36.6, 32 x 1600 47.2 / 45.8 / 53.6).
static AttnPlan attn_plan(const presto_attn_desc* d) {
    // (65536 and more merges fit no schedule with partials: the grid that such batches fill unsplit)
    if (!attn_ragged(d) || (int64_t)d->batch * d->hkv > 65535)
        return attn_plan_tail(d, attn_plan_split(d, false, false, kMaxSplits), kMaxSplits);
    const AttnPlan pr = attn_plan_split(d, false, true, kMaxSplits);
    if (pr.splits == 1) return attn_plan_tail(d, attn_plan_split(d, false, false, 1), 1);
    const AttnPlan de = attn_plan_split(d, false, false, kMaxSplits);
    const AttnPlan sh = attn_plan_shares(d);
    const double c_de = 1.05 * de.cost, c_pr = pr.cost + 6.5, c_sh = 1.1 * sh.cost + 3.0;
    if (c_de <= c_pr && c_de <= c_sh) return attn_plan_tail(d, de, kMaxSplits);
    return c_pr <= c_sh ? pr : sh;
}

size_t attn_workspace_bytes(const presto_attn_desc* d) {
    if (d->dt != PRESTO_DT_BF16) {
        const AttnF32Plan p = attn_f32_plan(d, true);
        if (p.splits <= 1) return 0;
        const size_t prs = attn_f32_partial_rows(d, p);
        return ((prs * d->head_dim * sizeof(float) + 255) & ~(size_t)255) + prs * sizeof(float2) + 256;
    }
    const AttnPlan p = attn_plan(d);
    if (!p.merged()) return 0;
    const size_t prs = p.partial_rows(d);
    return ((prs * d->head_dim * sizeof(uint16_t) + 255) & ~(size_t)255) + prs * sizeof(float2) + 256 +
           (p.shares > 0 ? (size_t)d->batch * sizeof(int2) : 0);
}

static presto_status launch_tree_attention_f32(const presto_attn_desc* d, const void* q, const void* k_cache,
                                               const void* v_cache, const int32_t* ctx_offsets,
                                               const void* k_tree, const void* v_tree, const uint64_t* anc,
                                               const int32_t* n_nodes, void* out, void* ws, hipStream_t stream) {
    const AttnF32Plan p = attn_f32_plan(d, ws != nullptr);
    if (p.blocks >= (int64_t)1 << 31)
        return set_error(PRESTO_ERR_UNSUPPORTED, "tree attention: %lld workgroups", (long long)p.blocks);
    AttnF32Args a;
    a.q = (const float*)q;
    a.kc = (const float*)k_cache;
    a.vc = (const float*)v_cache;
    a.ctx_off = ctx_offsets;
    a.ctx_slots = d->ctx_layout == PRESTO_CTX_SLOTS;
    a.kt = (const float*)k_tree;
    a.vt = (const float*)v_tree;
    a.anc = anc;
    a.n_nodes = n_nodes;
    a.out = (float*)out;
    a.part_o = (float*)ws;
    a.part_ml = nullptr;
    if (p.splits > 1)
        a.part_ml = (float2*)((char*)ws +
                              ((attn_f32_partial_rows(d, p) * d->head_dim * sizeof(float) + 255) & ~(size_t)255));
    a.n_max = d->n_max;
    a.hq = d->hq;
    a.hkv = d->hkv;
    a.G = p.G;
    a.W = (d->n_max + 63) / 64;
    a.row_blocks = p.row_blocks;
    a.splits = p.splits;
    a.split_len = p.split_len;
    a.n_tasks = (int32_t)p.tasks;
    a.n_blocks = (int32_t)p.blocks;
    a.scale = d->scale;
    const dim3 grid((unsigned)p.blocks), block(kF32Waves * kWave);
    if (d->head_dim == 64)
        tree_attn_f32_kernel<64><<<grid, block, 0, stream>>>(a);
    else
        tree_attn_f32_kernel<128><<<grid, block, 0, stream>>>(a);
    presto_status st = check_launch("tree_attn_f32_kernel");
    if (st != PRESTO_OK || p.splits == 1) return st;
    const dim3 mgrid((unsigned)((p.rows + 3) / 4), (unsigned)(d->batch * d->hkv));
    if (d->head_dim == 64)
        tree_attn_f32_merge_kernel<64><<<mgrid, 256, 0, stream>>>(a);
    else
        tree_attn_f32_merge_kernel<128><<<mgrid, 256, 0, stream>>>(a);
    return check_launch("tree_attn_f32_merge_kernel");
}

presto_status launch_tree_attention(const presto_attn_desc* d, const void* q, const void* k_cache,
                                    const void* v_cache, const int32_t* ctx_offsets,
                                    const void* k_tree, const void* v_tree, const uint64_t* anc,
                                    const int32_t* n_nodes, void* out, void* ws,
                                    hipStream_t stream) {
    if (d->dt == PRESTO_DT_F32)
        return launch_tree_attention_f32(d, q, k_cache, v_cache, ctx_offsets, k_tree, v_tree, anc, n_nodes, out,
                                         ws, stream);
    const AttnPlan p = attn_plan(d);
    if (p.merged() && (int64_t)d->batch * d->hkv > 65535)  // the merge's grid.y
        return set_error(PRESTO_ERR_UNSUPPORTED, "tree attention: batch x KV heads %lld above 65535",
                         (long long)d->batch * d->hkv);
    AttnArgs a;
    a.q = (const uint16_t*)q;
    a.kc = (const uint16_t*)k_cache;
    a.vc = (const uint16_t*)v_cache;
    a.ctx_off = ctx_offsets;
    a.ctx_slots = d->ctx_layout == PRESTO_CTX_SLOTS;
    a.kt = (const uint16_t*)k_tree;
    a.vt = (const uint16_t*)v_tree;
    a.anc = anc;
    a.n_nodes = n_nodes;
    a.out = (uint16_t*)out;
    {
        const size_t prs = p.partial_rows(d);
        a.part_o = (uint16_t*)ws;
        a.part_ml = (float2*)((char*)ws + ((prs * d->head_dim * sizeof(uint16_t) + 255) & ~(size_t)255));
        a.slots = (int2*)(a.part_ml + prs);
    }
    a.batch = d->batch;
    a.n_max = d->n_max;
    a.hq = d->hq;
    a.hkv = d->hkv;
    a.G = p.G;
    a.W = (d->n_max + 63) / 64;
    a.row_tiles = p.row_tiles;
    a.rows_per_tile = p.rows_per_tile;
    a.splits = p.splits;
    a.split_len = p.split_len;
    a.n_tasks = (int32_t)p.tasks;
    a.pairs = p.pairs ? 1 : 0;
    a.shares = p.shares;
    a.n_slots = p.n_slots;
    a.n_blocks = (int32_t)p.blocks;
    a.scale_log2 = d->scale * kLog2e;
    const dim3 block(kAttnWaves * kWave), grid((unsigned)p.blocks);
    auto go = [&](auto shares, auto tail) {
        if (d->head_dim == 64)
            tree_attn_bf16_kernel<64, decltype(shares)::value, decltype(tail)::value><<<grid, block, 0, stream>>>(a);
        else
            tree_attn_bf16_kernel<128, decltype(shares)::value, decltype(tail)::value><<<grid, block, 0, stream>>>(a);
    };
    if (p.shares > 0) go(std::true_type{}, std::false_type{});
    else if (p.tail) go(std::false_type{}, std::true_type{});
    else go(std::false_type{}, std::false_type{});
    presto_status st = check_launch("tree_attn_bf16_kernel");
    if (st != PRESTO_OK || !p.merged()) return st;
    const int pairs = d->batch * d->hkv;
    auto merge = [&](auto dims) {
        constexpr int E = decltype(dims)::value;
        const int rpb = 256 * E / d->head_dim;
        const dim3 mgrid((unsigned)((p.rows + rpb - 1) / rpb), (unsigned)pairs);
        if (d->head_dim == 64)
            tree_attn_merge_kernel<64, E><<<mgrid, 256, 0, stream>>>(a);
        else
            tree_attn_merge_kernel<128, E><<<mgrid, 256, 0, stream>>>(a);
    };
    // eight dims per lane where that makes a workgroup for every other CU or so
    const int64_t wide = (int64_t)pairs * ((p.rows * d->head_dim + 2047) / 2048);
    if (wide >= 100) merge(std::integral_constant<int, 8>{});
    else merge(std::integral_constant<int, 2>{});
    return check_launch("tree_attn_merge_kernel");
}

}  // namespace presto_host
