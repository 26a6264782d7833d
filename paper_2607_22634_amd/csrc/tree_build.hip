// Stage 2: prefix-aligned scoring and draft-tree construction.
//
// One workgroup builds one sequence's tree; the batch runs in parallel.
// The kernels:
//   tree_level_kernel   best-first (the budget best prefixes), level by level
//   tree_pop_kernel     the same for few nodes and chains, one node at a time
//   tree_beam_kernel    beam search with global retention
//   tree_alg2_kernel    Alg. 2 as printed
#include <math.h>

#include <type_traits>

#include "common.hpp"

// Scores must round exactly as fl(log q + fl(lambda * log rho)) and
// fl(S(parent) + s): no fused multiply-add anywhere in this file.
#pragma clang fp contract(off)

namespace presto {

struct TreeArgs {
    int32_t D, k, branch, budget, N, W, wbits, per_word;
    const int32_t* ids;
    const float* logprob;
    const float* log_rho;
    const float* lambda;
    int32_t lambda_stride;  // 0: one lambda row shared by the batch, D: one per sequence
    const int32_t* root_token;
    int32_t* n_nodes;
    int32_t* parent;
    int32_t* token;
    int32_t* depth;
    int32_t* rank;
    float* score;
    uint64_t* anc;
    int32_t beam_width;  // beam search only
    uint32_t mag_k, mag_k3;  // ceil(2^32 / k), ceil(2^32 / k^3) (k > 1): n / d = umulhi(n, mag) for n < 2^20
    // LDS byte offsets: the tables of every kernel,
    int o_lp, o_ids, o_rho;
    // the level and beam kernels,
    int o_lam, o_pool, o_key, o_hist, o_fine, o_list, o_place, o_row, o_par, o_misc;
    int32_t cap;  // entries the pool holds, the root included
    // the one-node-at-a-time kernel,
    int o_kord, o_krank, o_rec, o_pkey;
    // literal Alg. 2: T (capacity budget + branch - 1)
    int o_tmeta, o_tS, o_tkey, o_tplace;
};

// Frontier metadata in one word: parent node (10 bits), candidate rank (4),
// depth (6), rank of the parent (4), position among the parent's children
// in commit order (4).
__device__ __forceinline__ uint32_t pack_meta(int p, int r, int d, int rp, int pos) {
    return (uint32_t)p | ((uint32_t)r << 10) | ((uint32_t)d << 14) | ((uint32_t)rp << 20) |
           ((uint32_t)pos << 24);
}

// Number of lanes of this lane's row of 16 holding a larger key (row
// rotations by 1..R, each another lane of the row exactly once).
template <int R>
__device__ __forceinline__ int row_count_greater(uint64_t key) {
    if constexpr (R == 0) {
        return 0;
    } else {
        return (dpp_u64<0x120 + R>(0ull, key) > key ? 1 : 0) + row_count_greater<R - 1>(key);
    }
}

// One compare-exchange layer of a bitonic sort, descending: lane i pairs
// with the lane that DPP control CTRL reads (i ^ m within the group), and
// the lower lane of the pair (bit LOWBIT of i clear) keeps the larger key.
template <int CTRL, int LOWBIT>
__device__ __forceinline__ uint64_t bitonic_layer(uint64_t key, int lane) {
    const uint64_t t = dpp_u64<CTRL>(0ull, key);
    const bool lower = ((lane >> LOWBIT) & 1) == 0;
    return (lower == (t > key)) ? t : key;
}

// Keys of lanes 0..7 of every row sorted descending in place (lane 0 of the
// group holds the largest): blocks of 2, 4, 8, each merged by a flip
// (i ^ (s - 1)) and half-cleaners (i ^ s/4, ..., i ^ 1).
__device__ __forceinline__ uint64_t sort8_desc(uint64_t key, int lane) {
    key = bitonic_layer<0xb1, 0>(key, lane);   // i ^ 1
    key = bitonic_layer<0x1b, 1>(key, lane);   // i ^ 3 (quad_perm [3,2,1,0])
    key = bitonic_layer<0xb1, 0>(key, lane);   // i ^ 1
    key = bitonic_layer<0x141, 2>(key, lane);  // i ^ 7 (row_half_mirror)
    key = bitonic_layer<0x4e, 1>(key, lane);   // i ^ 2
    key = bitonic_layer<0xb1, 0>(key, lane);   // i ^ 1
    return key;
}

// Same within this lane's quad (quad_perm rotations by 1, 2, 3).
__device__ __forceinline__ int quad_count_greater(uint64_t key) {
    return (dpp_u64<0x39>(0ull, key) > key ? 1 : 0) + (dpp_u64<0x4e>(0ull, key) > key ? 1 : 0) +
           (dpp_u64<0x93>(0ull, key) > key ? 1 : 0);
}

// Loads up to U words per lane of src[base ..] (batches of 64 words while
// fewer than n; indices clamped, so every load is unconditional) into r.
template <int U>
__device__ __forceinline__ void load_words(uint32_t (&r)[U], const uint32_t* src, int n, int base, int lane) {
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (base + u * kWave < n) r[u] = src[min(base + u * kWave + lane, n - 1)];
}
template <int U>
__device__ __forceinline__ void store_words(uint32_t* dst, const uint32_t (&r)[U], int n, int base, int lane) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = base + u * kWave + lane;
        if (i < n) dst[i] = r[u];
    }
}

// Copies n 32-bit words from global memory to LDS with one wave, 16 loads
// in flight per lane before the first store.
__device__ __forceinline__ void stage_words(uint32_t* dst, const uint32_t* src, int n, int lane) {
    constexpr int U = 16;
    for (int base = 0; base < n; base += U * kWave) {
        uint32_t r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = base + u * kWave + lane;
            r[u] = i < n ? src[i] : 0u;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = base + u * kWave + lane;
            if (i < n) dst[i] = r[u];
        }
    }
}

// x with lane l replaced by v (v and l are read from the first lane, so they
// are scalar operands whatever registers hold them).
__device__ __forceinline__ uint32_t write_lane(uint32_t x, uint32_t v, int l) {
    const uint32_t sv = (uint32_t)__builtin_amdgcn_readfirstlane(v);
    const uint32_t sl = (uint32_t)__builtin_amdgcn_readfirstlane(l);
    asm("v_writelane_b32 %0, %1, m0" : "+v"(x) : "s"(sv), "{m0}"(sl));
    return x;
}

// Token scores fl(log q + fl(lambda * log rho)), NaN -> -inf, of candidate r
// at drafter row `row` in the trigram context (c2, c1) of candidate ranks.
// RHO: 0 no lattice (s = log q), 1 scores of the whole lattice in LDS, 2
// lattice read from global memory and scored on the fly.
template <int RHO>
struct TokenScores {
    const float* s_lp;
    const float* s_lam;
    const float* s_rho;
    const float* g_rho;
    int k;
    __device__ __forceinline__ TokenScores(const TreeArgs& a, const char* lds)
        : s_lp(reinterpret_cast<const float*>(lds + a.o_lp)),
          s_lam(reinterpret_cast<const float*>(lds + a.o_lam)),
          s_rho(reinterpret_cast<const float*>(lds + a.o_rho)),
          g_rho(RHO ? a.log_rho + (int64_t)blockIdx.x * a.D * a.k * a.k * a.k : nullptr),
          k(a.k) {}
    __device__ __forceinline__ float operator()(int row, int c2, int c1, int r) const {
        if constexpr (RHO == 0) return s_lp[row * k + r];
        const int i = ((row * k + c2) * k + c1) * k + r;
        if constexpr (RHO == 1) return s_rho[i];
        const float lr = g_rho[i];
        const float t = s_lam[row] * lr;
        const float v = s_lp[row * k + r] + t;
        return (v == v) ? v : -INFINITY;
    }
};

// Stages the candidate table and lambda of this workgroup's sequence and, with
// the lattice in LDS, the token scores of every context in its place (so that
// scoring a child is one read).  Every thread has up to U lattice words in
// flight, the first batch requested before the barrier that publishes log q
// and lambda; ends with a barrier.  (With one wave staging and a separate
// scoring pass, a lattice of 16,000 words took about 45 k cycles; one thread
// per word with 32 in flight about 23 k.)
template <int NT, int RHO>
__device__ __forceinline__ void stage_tables(const TreeArgs& a, char* lds) {
    const int tid = threadIdx.x, lane = lane_id();
    const int b = blockIdx.x, D = a.D, k = a.k;
    float* s_lp = reinterpret_cast<float*>(lds + a.o_lp);
    float* s_lam = reinterpret_cast<float*>(lds + a.o_lam);
    float* s_rho = reinterpret_cast<float*>(lds + a.o_rho);
    int32_t* s_ids = reinterpret_cast<int32_t*>(lds + a.o_ids);
    const int64_t tb = (int64_t)b * D * k;
    if (tid < kWave) {
        uint32_t r_lp[8], r_ids[8];  // D * k <= 512 words
        load_words(r_lp, reinterpret_cast<const uint32_t*>(a.logprob + tb), D * k, 0, lane);
        load_words(r_ids, reinterpret_cast<const uint32_t*>(a.ids + tb), D * k, 0, lane);
        const float lam = lane < D ? a.lambda[(int64_t)b * a.lambda_stride + lane] : 0.f;
        store_words(reinterpret_cast<uint32_t*>(s_lp), r_lp, D * k, 0, lane);
        store_words(reinterpret_cast<uint32_t*>(s_ids), r_ids, D * k, 0, lane);
        if (lane < D) s_lam[lane] = lam;
    }
    if constexpr (RHO == 1) {
        const int rho_n = D * k * k * k;
        const uint32_t* gr = reinterpret_cast<const uint32_t*>(a.log_rho + (int64_t)b * rho_n);
        auto stage = [&](auto uc) __attribute__((always_inline)) {
            constexpr int U = decltype(uc)::value;
            for (int base = 0; base < rho_n; base += U * NT) {
                // words of this batch per thread that exist for some thread
                const int nu = U > 8 ? U : min(U, (rho_n - base + NT - 1) / NT);
                float x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = base + u * NT + tid;
                    x[u] = (u < nu && i < rho_n) ? __uint_as_float(gr[i]) : 0.f;
                }
                if (base == 0) __syncthreads();
                // every log q and lambda of the batch read before the first
                // store (a store between them would order each read after it)
                float lq[U], lm[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    lq[u] = lm[u] = 0.f;
                    if (u < nu) {
                        const int i = min(base + u * NT + tid, rho_n - 1);
                        const int row = k == 1 ? i : (int)__umulhi((uint32_t)i, a.mag_k3);
                        const int r = k == 1 ? 0 : i - (int)__umulhi((uint32_t)i, a.mag_k) * k;
                        lq[u] = s_lp[row * k + r];
                        lm[u] = s_lam[row];
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int i = base + u * NT + tid;
                    const float t = lm[u] * x[u];
                    const float v = lq[u] + t;
                    if (u < nu && i < rho_n) s_rho[i] = (v == v) ? v : -INFINITY;
                }
            }
        };
        if (rho_n <= 8 * NT)
            stage(std::integral_constant<int, 8>{});
        else
            stage(std::integral_constant<int, 16>{});
    } else {
        __syncthreads();
        if constexpr (RHO == 0) {
            for (int i = tid; i < D * k; i += NT) {
                const float v = s_lp[i];
                s_lp[i] = (v == v) ? v : -INFINITY;
            }
        }
    }
    __syncthreads();
}

// Best-first search one node at a time, by one wave, for trees of at most 64
// rows (see pops_first).  Per committed node LDS holds one 8-byte record (parent,
// rank, depth, S) and its children in commit order; the frontier lives in
// registers, one entry per lane, (S, packed metadata) each: a pop is a DPP wave
// max and a ballot.  The frontier holds, for every committed node, only its next
// not-yet-committed child in commit order: committing a node pushes its first
// child, committing a child pushes its next sibling, so it never holds more than
// (committed + 1) entries.  Rank-path keys are only derived when several entries
// share the best S.  About 1300 cycles per pop; the tables have been staged.
// QUAD: k <= 4 (known at compile time a pop takes 0.05 us less).
template <int RHO, bool QUAD>
__device__ void tree_pop_search(const TreeArgs& a, char* lds) {
    const int lane = lane_id();
    const int b = blockIdx.x;
    const int D = a.D, k = a.k, N = a.N, wbits = a.wbits, per_word = a.per_word;
    const TokenScores<RHO> scores(a, lds);
    const int32_t* s_ids = reinterpret_cast<const int32_t*>(lds + a.o_ids);
    // children of every committed node in commit order: ord(S) (0 ends the
    // list) and candidate rank
    uint32_t* s_kord = reinterpret_cast<uint32_t*>(lds + a.o_kord);  // [N][k]
    uint8_t* s_krank = reinterpret_cast<uint8_t*>(lds + a.o_krank);  // [N][k]
    uint2* s_rec = reinterpret_cast<uint2*>(lds + a.o_rec);          // [N] (meta, S bits)

    // Children of node n (depth d, own rank rn, parent's rank rp, score Sn):
    // lane r < k scores candidate r, the children are ranked by (S desc,
    // rank asc) and stored in that order; returns the first child as (ord S,
    // rank), ord 0 if none.  A node at the depth limit (d == D) has no
    // children: nothing is stored and ord 0 is returned.
    auto expand = [&](int n, int d, int rn, int rp, float Sn, uint32_t& c_ord, int& c_rank) {
        const bool live = d < D;
        const int dr = min(d, D - 1);      // drafter row read (clamped at the depth limit)
        const int ctx2 = d >= 2 ? rp : 0;  // grandparent slot of the trigram
        const int ctx1 = d >= 1 ? rn : 0;  // parent slot of the trigram
        // every lane reads (lanes >= k at a clamped index) so that no branch
        // separates the reads from their use; only lanes < k are kept
        float s = scores(dr, ctx2, ctx1, min(lane, k - 1));
        s = lane < k ? s : -INFINITY;
        bool in = lane < k && live;
        if (a.branch < k) {
            // keep the top-`branch` by token score (larger s, then lower rank)
            int sel = 0;
            for (int j = 0; j < k; ++j) {
                const float sj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s), j));
                sel += (sj > s || (sj == s && j < lane)) ? 1 : 0;
            }
            in = in && sel < a.branch;
        }
        const float sc = Sn + s;
        const uint32_t o = ord32(sc);  // nonzero for every non-NaN score
        const uint64_t key = in ? (((uint64_t)o << 8) | (uint64_t)(255 - lane)) : 0ull;
        if (!QUAD && k > 4 && k <= 8) {
            // sorted in place: lane p holds the p-th child (key 0 past the
            // last child, which writes the end marker)
            const uint64_t sk = sort8_desc(key, lane);
            if (lane < k && live) {
                s_kord[n * k + lane] = (uint32_t)(sk >> 8);
                s_krank[n * k + lane] = (uint8_t)(255 - (uint32_t)(sk & 255));
            }
            const uint64_t top = readlane_u64(sk, 0);
            c_ord = (uint32_t)(top >> 8);
            c_rank = c_ord ? 255 - (int)(top & 255) : 0;
        } else {
            // the lanes that are not children all land on the first free
            // position and write the end marker there
            const int pos = QUAD || k <= 4 ? quad_count_greater(key) : row_count_greater<15>(key);
            if (lane < k && live) {
                s_kord[n * k + pos] = in ? o : 0u;
                s_krank[n * k + pos] = (uint8_t)lane;
            }
            const uint64_t first = __ballot(in && pos == 0);
            c_rank = first ? __ffsll((unsigned long long)first) - 1 : 0;
            c_ord = first ? (uint32_t)__builtin_amdgcn_readlane((int)o, c_rank) : 0u;
        }
    };

    // Rank-path keys (four 32-bit words, most significant first): the key of
    // a node is its parent's key with the digit rank + 1 at its depth.  They
    // only break ties of S, so they are derived when a tie needs them: the
    // parent chain of a tied entry is walked up to the nearest node whose key
    // is known (the root, or a node whose key an earlier tie stored: every
    // non-root key has a nonzero first word) and the parent's key is stored.
    uint4* s_pkey = reinterpret_cast<uint4*>(lds + a.o_pkey);  // [N], 0 = not known yet
    const uint32_t pw_magic = (65536u + per_word - 1) / per_word;  // t / per_word = t * magic >> 16 (t < 128)
    auto add_digit = [&](uint4 key, int d, int r) {
        const uint32_t t = (uint32_t)(d - 1);
        const uint32_t wi = (t * pw_magic) >> 16;
        const uint32_t v = (uint32_t)(r + 1) << (32 - (t - wi * per_word + 1) * wbits);
        key.x |= wi == 0 ? v : 0u;
        key.y |= wi == 1 ? v : 0u;
        key.z |= wi == 2 ? v : 0u;
        key.w |= wi == 3 ? v : 0u;
        return key;
    };
    for (int i = lane; i < N; i += kWave) s_pkey[i] = make_uint4(0u, 0u, 0u, 0u);

    if (lane == 0) s_rec[0] = make_uint2(0xffffffffu, __float_as_uint(0.f));
    uint32_t c_ord;
    int c_rank;
    expand(0, 0, 0, 0, 0.f, c_ord, c_rank);

    // the frontier: entry l in lane l (S as ord32, 0 for none)
    uint32_t fS = lane == 0 ? c_ord : 0u, fM = lane == 0 ? pack_meta(0, c_rank, 1, 0, 0) : 0u;
    int fcount = 1, committed = 1;

    // commit the best frontier entry and push its successors, until the budget
    // is spent or the frontier exhausted (the whole candidate tree committed)
    while (committed - 1 < a.budget) {
        const uint32_t M = wave_max_u32_dpp(fS);
        if (M == 0u) break;
        // winner: the unique entry holding M, else the one with the smallest path key
        const uint64_t any = __ballot(fS == M);
        int w;
        if (__popcll(any) == 1) {
            w = __ffsll((unsigned long long)any) - 1;
        } else {
            bool t = fS == M;
            uint32_t kw[4] = {~0u, ~0u, ~0u, ~0u};
            if (t) {
                const int p = fM & 1023;
                uint4 acc = make_uint4(0u, 0u, 0u, 0u);
                int y = p;
                uint4 st = s_pkey[y];
                uint32_t m = s_rec[y].x;
                while (y != 0 && st.x == 0u) {
                    acc = add_digit(acc, (m >> 14) & 63, (m >> 10) & 15);
                    y = m & 1023;
                    st = s_pkey[y];
                    m = s_rec[y].x;
                }
                const uint4 kp = make_uint4(acc.x | st.x, acc.y | st.y, acc.z | st.z, acc.w | st.w);
                if (y != p) s_pkey[p] = kp;  // lanes storing the same node store the same key
                const uint4 kv = add_digit(kp, (fM >> 14) & 63, (fM >> 10) & 15);
                kw[0] = kv.x; kw[1] = kv.y; kw[2] = kv.z; kw[3] = kv.w;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t mq = wave_min_u32_dpp(t ? kw[q] : ~0u);
                t = t && kw[q] == mq;
            }
            w = __ffsll((unsigned long long)__ballot(t)) - 1;
        }
        const uint32_t meta = (uint32_t)__builtin_amdgcn_readlane((int)fM, w);
        const int p = meta & 1023, r = (meta >> 10) & 15, d = (meta >> 14) & 63, rp = (meta >> 20) & 15;
        const int pos = (meta >> 24) & 15;
        const float S = unord32(M);

        // commit node n: one record; everything else is derived after the search
        const int n = committed++;
        if (lane == 0) s_rec[n] = make_uint2(meta, __float_as_uint(S));

        // next sibling of n: the next entry of its parent's ordered children
        // (read unconditionally, at a clamped index, so that its latency
        // overlaps the expansion's reads)
        const int si = p * k + min(pos + 1, k - 1);
        const uint32_t sib_raw = s_kord[si];
        const int sib_rank = s_krank[si];
        // first child of n
        uint32_t kid_ord = 0u;
        int kid_rank = 0;
        expand(n, d, r, rp, S, kid_ord, kid_rank);
        const uint32_t sib_ord = pos + 1 < k ? sib_raw : 0u;

        // pushes: the first takes the popped entry's lane, the second a fresh one
        uint32_t xS = 0u, xM = 0u, yS = 0u, yM = 0u;
        if (kid_ord != 0u) {
            xS = kid_ord;
            xM = pack_meta(n, kid_rank, d + 1, r, 0);
        }
        if (sib_ord != 0u) {
            const uint32_t m = pack_meta(p, sib_rank, d, rp, pos + 1);
            if (xS != 0u) {
                yS = sib_ord;
                yM = m;
            } else {
                xS = sib_ord;
                xM = m;
            }
        }
        fS = write_lane(fS, xS, w);
        fM = write_lane(fM, xM, w);
        if (yS != 0u) {
            fS = write_lane(fS, yS, fcount);
            fM = write_lane(fM, yM, fcount);
            ++fcount;
        }
    }
    __builtin_amdgcn_wave_barrier();

    // Output rows and ancestor masks, one node per lane: the mask of node n has
    // the bits of n and of every node on its parent chain.
    const int64_t ob = (int64_t)b * N;
    const int root_tok = __builtin_amdgcn_readfirstlane(a.root_token[b]);
    if (lane < N) {
        int par = -1, tok = -1, dep = -1, rank = -1;
        float S = -INFINITY;
        uint64_t mask = 0ull;
        if (lane < committed) {
            const uint2 rec = s_rec[lane];
            dep = lane == 0 ? 0 : (int)(rec.x >> 14) & 63;
            const int r = (int)(rec.x >> 10) & 15;
            tok = lane == 0 ? root_tok : s_ids[(dep > 0 ? dep - 1 : 0) * k + r];
            par = lane == 0 ? -1 : (int)(rec.x & 1023);
            rank = lane == 0 ? -1 : r;
            S = __uint_as_float(rec.y);
            int x = lane;
            while (true) {
                mask |= 1ull << x;
                if (x == 0) break;
                x = (int)(s_rec[x].x & 1023);
            }
        }
        a.parent[ob + lane] = par;
        a.token[ob + lane] = tok;
        a.depth[ob + lane] = dep;
        a.rank[ob + lane] = rank;
        a.score[ob + lane] = S;
        a.anc[ob + lane] = mask;
    }
    if (lane == 0) a.n_nodes[b] = committed;
}

// ---------------------------------------------------------------------------
// Level search and beam search: what the two kernels share.
//
// A workgroup collects prefixes level by level (depth by depth) in a pool in
// LDS: per entry (S, parent entry | rank << 13 | parent's rank << 17 | depth
// << 21) and the rank-path key.  Entry 0 is the root (S = 0, ranks 0: the
// slots its children's contexts read), a level's entries are contiguous.
// Afterwards finish_tree places the entries in the total order (S desc, rank
// path asc, a prefix before its extensions) and writes the rows.

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kPoolMax = 8191;  // 13 bits of parent entry
constexpr int kBins = 512;      // histogram of -S, see score_bin

// Monotone bin of a score: 32 bins per octave of 1 - S, so a bin is 1/32 nat
// wide near S = 0 and 1/4 nat near S = -10; everything below -65535 is in the
// last one.  score_bin(x) < score_bin(y) implies x > y.
constexpr int kBinBits = 5;  // bins per octave: 2^kBinBits
__device__ __forceinline__ uint32_t score_bin(float S) {
    const uint32_t u = __float_as_uint(fmaxf(1.f - S, 1.f)) >> (23 - kBinBits);
    return min(u - (127u << kBinBits), (uint32_t)(kBins - 1));
}

__device__ __forceinline__ int lanes_below(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// The bin holding the `budget`-th best entry counted so far (kBins - 1 if
// fewer are counted), and the number counted up to it.  Every wave computes
// it for itself; a histogram that other waves are still adding to gives a
// bin no better than the true one, since only entries that exist are counted.
__device__ __forceinline__ uint32_t threshold_bin(const uint32_t* s_hist, uint32_t budget, uint32_t& counted) {
    const uint4* h = reinterpret_cast<const uint4*>(s_hist) + 2 * lane_id();
    const uint4 x = h[0], y = h[1];
    const uint32_t v[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
    uint32_t sum = 0u;
#pragma unroll
    for (int i = 0; i < 8; ++i) sum += v[i];
    const uint32_t incl = wave_scan_dpp(sum);
    const uint64_t m = __ballot(incl >= budget);
    if (m == 0ull) {
        counted = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
        return kBins - 1;
    }
    uint32_t c = incl - sum, j = 0u;
    uint32_t upto = c + v[0];
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        c += v[i];
        j += c < budget ? 1u : 0u;
        upto = c < budget ? c + v[i + 1] : upto;
    }
    const int l = __ffsll((unsigned long long)m) - 1;
    counted = (uint32_t)__builtin_amdgcn_readlane((int)upto, l);
    return (uint32_t)__builtin_amdgcn_readlane((int)(8 * l + j), l);
}

template <int KW>
struct PathKey;
template <>
struct PathKey<2> {
    typedef u32x2 type;
};
template <>
struct PathKey<4> {
    typedef u32x4 type;
};
template <int KW>
__device__ __forceinline__ bool key_less(typename PathKey<KW>::type x, typename PathKey<KW>::type y) {
    const uint64_t xa = ((uint64_t)x[0] << 32) | (uint64_t)x[1], ya = ((uint64_t)y[0] << 32) | (uint64_t)y[1];
    if constexpr (KW == 2) {
        return xa < ya;
    } else {
        const uint64_t xb = ((uint64_t)x[2] << 32) | (uint64_t)x[3], yb = ((uint64_t)y[2] << 32) | (uint64_t)y[3];
        return (xa < ya) | ((xa == ya) & (xb < yb));
    }
}

// The pool and the scratch of finish_tree.  KW: words of a rank-path key
// (most significant first; digit rank + 1 at the entry's depth).
template <int KW>
struct Pool {
    typedef typename PathKey<KW>::type Key;
    uint2* rec;       // [cap]
    Key* key;         // [cap]
    uint32_t* hist;   // [kBins] entries per score bin
    uint32_t* fine;   // [fine bins + 1] counts, then offsets
    uint16_t* list;   // [cap] entries in the order of the fine bins
    uint16_t* place;  // [cap] place within the bin, then the entry's row
    uint16_t* row;    // [N] entry of a row
    uint16_t* par;    // [N] parent row
    uint32_t* misc;   // [64]: level counts by depth (then wave sums), 63: a flag
    __device__ __forceinline__ Pool(const TreeArgs& a, char* lds)
        : rec(reinterpret_cast<uint2*>(lds + a.o_pool)), key(reinterpret_cast<Key*>(lds + a.o_key)),
          hist(reinterpret_cast<uint32_t*>(lds + a.o_hist)), fine(reinterpret_cast<uint32_t*>(lds + a.o_fine)),
          list(reinterpret_cast<uint16_t*>(lds + a.o_list)), place(reinterpret_cast<uint16_t*>(lds + a.o_place)),
          row(reinterpret_cast<uint16_t*>(lds + a.o_row)), par(reinterpret_cast<uint16_t*>(lds + a.o_par)),
          misc(reinterpret_cast<uint32_t*>(lds + a.o_misc)) {}
    __device__ __forceinline__ float S(int e) const { return __uint_as_float(rec[e].x); }
    static __device__ __forceinline__ uint32_t meta(int parent, int rank, int prank, int depth) {
        return (uint32_t)parent | ((uint32_t)rank << 13) | ((uint32_t)prank << 17) | ((uint32_t)depth << 21);
    }
    // the key of a child of rank r, whose digit sits in word wi at shift sh
    static __device__ __forceinline__ Key child_key(Key x, int wi, int sh, int r) {
        const uint32_t v = (uint32_t)(r + 1) << sh;
#pragma unroll
        for (int w = 0; w < KW; ++w) x[w] |= w == wi ? v : 0u;
        return x;
    }
};

// Fine bins of finish_tree's sort, at least the workgroup's threads: 512 for
// the small trees (budget 64: 10.2 us, 11.4 with 1024), 1024 for the others
// and the beam (budget 512: 27 us, 32 with 512).
constexpr int kFineMax = 1024;
// A fine bin is crowded (equal scores) from here on: placing its entries takes
// 0.3 us per four of them, finding the budget-th best first about 10 us.
constexpr int kCrowd = 128;

template <int NT, int NF, int KW>
__device__ __forceinline__ void init_pool(const TreeArgs& a, const Pool<KW>& P) {
    const int tid = threadIdx.x;
    for (int i = tid; i < kBins; i += NT) P.hist[i] = 0u;
    for (int i = tid; i < NF; i += NT) P.fine[i] = 0u;
    if (tid < 64) P.misc[tid] = 0u;
    if (tid == 0) {
        P.rec[0] = make_uint2(__float_as_uint(0.f), 0u);
        typename Pool<KW>::Key z;
#pragma unroll
        for (int w = 0; w < KW; ++w) z[w] = 0u;
        P.key[0] = z;
    }
}

// Drops the entries that keep(S, key) refuses (with all their descendants: keep
// refuses none that precedes one it takes) and closes the gaps; the parents'
// indices and the frontier [lo, hi) move along.  Ends with a barrier.
template <int NT, int KW, typename Keep>
__device__ __forceinline__ void compact_pool(const Pool<KW>& P, const Keep& keep, int& lo, int& hi) {
    const int tid = threadIdx.x, lane = lane_id();
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    uint32_t* s_wave = P.misc + 40;  // [NT / kWave], past the level counts
    int n = 1, below_lo = 0;
    if (tid == 0) P.place[0] = 0;
    for (int e0 = 1; e0 < hi; e0 += NT) {
        const int e = e0 + tid;
        uint2 rec = make_uint2(0u, 0u);
        typename Pool<KW>::Key key = P.key[0];
        bool alive = false;
        if (e < hi) {
            rec = P.rec[e];
            key = P.key[e];
            alive = keep(__uint_as_float(rec.x), key);
        }
        const uint64_t m = __ballot(alive), ml = __ballot(alive & (e < lo));
        if (lane == 0) s_wave[wv] = (uint32_t)__popcll(m) | ((uint32_t)__popcll(ml) << 16);
        __syncthreads();
        uint32_t off = 0u, all = 0u;
#pragma unroll
        for (int w = 0; w < NT / kWave; ++w) {
            const uint32_t c = s_wave[w];
            off += w < wv ? c : 0u;
            all += c;
        }
        const int at = n + (int)(off & 0xffffu) + lanes_below(m);
        if (alive) P.place[e] = (uint16_t)at;
        __syncthreads();  // this chunk is read; its entries move down, never past it
        if (alive) {
            P.rec[at] = make_uint2(rec.x, (rec.y & ~8191u) | P.place[rec.y & 8191u]);
            P.key[at] = key;
        }
        n += (int)(all & 0xffffu);
        below_lo += (int)(all >> 16);
    }
    hi = n;
    lo = 1 + below_lo;
    __syncthreads();
}

// The place of the `budget`-th best of a set of prefixes in the total order:
// a prefix is among them iff at_most(S, key).
template <int KW>
struct Bound {
    typedef typename PathKey<KW>::type Key;
    uint32_t s;  // ~ord32(S)
    Key key;
    __device__ __forceinline__ bool at_most(float S, Key k) const {
        const uint32_t x = ~ord32(S);
        return (x < s) | ((x == s) & !key_less<KW>(key, k));
    }
};

// That bound over the members member(i, S, key), i < n, that return true (at
// least `budget` of them), by nine bits of (~ord32(S), rank path) at a time: a
// count of the members that agree with the bits known so far, in P.fine (zeros
// on entry and on return).  Each pass takes every member anew, so that nothing
// but the counts is stored; it ends as soon as the members left are the ones
// missing.  Ends with a barrier.  (Eight bits and four sets of counters, one
// barrier a pass instead of three, took 10% less here and, by the registers it
// takes from the kernel, 20% more of the searches without ties at depth 32.)
template <int NT, int KW, typename Member>
__device__ __forceinline__ Bound<KW> select_best(const Pool<KW>& P, int n, uint32_t budget, const Member& member) {
    const int tid = threadIdx.x, lane = lane_id();
    uint32_t want[KW + 1];
#pragma unroll
    for (int w = 0; w <= KW; ++w) want[w] = 0u;
    uint32_t need = budget;
    int word = 0, shift = 23;  // shifts 23, 14, 5, and the last five bits
    while (true) {
        const uint32_t above = shift == 23 ? 0u : (~0u << (shift == 0 ? 5 : shift + 9));  // known bits of this word
        for (int i0 = 0; i0 < n; i0 += NT) {
            float S = 0.f;
            typename Pool<KW>::Key key = P.key[0];
            bool in = i0 + tid < n;
            if (in) in = member(i0 + tid, S, key);
            uint32_t x[KW + 1];
            x[0] = ~ord32(S);
#pragma unroll
            for (int w = 0; w < KW; ++w) x[w + 1] = key[w];
            uint32_t digit = 0u;
#pragma unroll
            for (int w = 0; w <= KW; ++w) {
                in &= w >= word || x[w] == want[w];
                if (w == word) {
                    in &= (x[w] & above) == (want[w] & above);
                    digit = shift == 0 ? x[w] & 31u : (x[w] >> shift) & 511u;
                }
            }
            // equal digits, as ties have them, as one addition
            const uint64_t m = __ballot(in);
            if (m != 0ull) {
                const int first = __ffsll((unsigned long long)m) - 1;
                const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)digit, first);
                const uint64_t same = __ballot(in & (digit == d0));
                if (lane == first) atomicAdd(&P.fine[d0], (uint32_t)__popcll(same));
                if (in & (digit != d0)) atomicAdd(&P.fine[digit], 1u);
            }
        }
        __syncthreads();
        uint32_t upto;
        const uint32_t digit = threshold_bin(P.fine, need, upto);
        const uint32_t here = P.fine[digit];
        need -= upto - here;
        const bool done = here == need;
#pragma unroll
        for (int w = 0; w <= KW; ++w) {
            if (w == word) want[w] |= (digit << shift) | (done ? (1u << shift) - 1u : 0u);
            if (w > word && done) want[w] = ~0u;
        }
        __syncthreads();  // the counts have been read
        for (int i = tid; i < 512; i += NT) P.fine[i] = 0u;
        __syncthreads();
        if (done) break;
        shift = shift == 0 ? 23 : (shift == 5 ? 0 : shift - 9);
        word += shift == 23 ? 1 : 0;
        if (word > KW) break;  // not reached: the paths are distinct
    }
    Bound<KW> r;
    r.s = want[0];
#pragma unroll
    for (int w = 0; w < KW; ++w) r.key[w] = want[w + 1];
    return r;
}

// Rows nt + 1 .. budget from prefixes of S = -inf, which follow every finite
// one, in rank-path order: a depth-first walk of the candidate tree by one
// wave (every lane the same) that descends through the finite entries (child:
// the entry of every (entry, rank), 0 if not finite) and takes the -inf
// children as it meets them, each before its own descendants.  They become
// entries n .. of the pool.  At most two steps per row; a prefix of S = -inf
// has all its siblings' descendants tied with it, so the level search cannot
// bound them.  Returns the non-root rows.
template <int KW, typename Scores>
__device__ int fill_below(const TreeArgs& a, const Pool<KW>& P, const uint16_t* child, int n, int nt,
                          const Scores& scores) {
    const int D = a.D, k = a.k;
    uint32_t* stack = P.misc;  // per depth: entry | next rank << 16
    int d = 0, node = 0, next = 0, rank = 0, prank = 0;
    bool below = false;  // the node's own S is -inf
    while (nt < a.budget) {
        if (d == D || next == k) {
            if (d == 0) break;
            --d;
            const uint32_t s = (uint32_t)__builtin_amdgcn_readfirstlane((int)stack[d]);
            node = (int)(s & 0xffffu);
            next = (int)(s >> 16);
            const uint2 r = P.rec[node];
            below = __builtin_amdgcn_readfirstlane((int)r.x) == (int)0xff800000u;
            const uint32_t y = (uint32_t)__builtin_amdgcn_readfirstlane((int)r.y);
            rank = (int)(y >> 13) & 15;
            prank = (int)(y >> 17) & 15;
            continue;
        }
        const int r = next++;
        int c = below ? 0 : __builtin_amdgcn_readfirstlane((int)child[node * k + r]);
        const bool finite = c != 0;
        if (!finite) {
            if (a.branch < k) {
                // only the top-`branch` by token score are children
                const float s = scores(d, prank, rank, r);
                int sel = 0;
                for (int j = 0; j < k; ++j) {
                    const float sj = scores(d, prank, rank, j);
                    sel += ((sj > s) | ((sj == s) & (j < r))) ? 1 : 0;
                }
                if (__builtin_amdgcn_readfirstlane(sel) >= a.branch) continue;
            }
            c = n++;
            ++nt;
            P.rec[c] = make_uint2(0xff800000u, Pool<KW>::meta(node, r, rank, d + 1));
            P.place[c] = (uint16_t)nt;
            P.row[nt] = (uint16_t)c;
        }
        stack[d] = (uint32_t)node | ((uint32_t)next << 16);
        ++d;
        node = c;
        next = 0;
        prank = rank;
        rank = r;
        below = !finite;
    }
    return nt;
}

// Places the pool's entries 1 .. n - 1 whose bin is at most the budget-th
// best entry's and writes the tree: the `budget` best in the total order
// (parents are among them: an entry never precedes its parent).  A counting
// sort over fine bins of S, then each entry's place within its bin by
// comparing it with the bin's few others; a handful of barriers, where
// comparing all pairs of 1000 entries took about as long as the search.
// `fill`: fewer than `budget` entries, and candidates of S = -inf were left
// out of the pool (fill_below).
// CUT: entries past `bound` are left out.  Without it, false is returned, with
// nothing written, where a bin is crowded and many entries are too many.
template <int NT, int NF, int KW, bool CUT, typename Scores>
__device__ __forceinline__ bool place_tree(const TreeArgs& a, char* lds, const Pool<KW>& P, int n,
                                           const Scores& scores, bool fill, const Bound<KW>& bound) {
    constexpr int PER = NF / NT;
    static_assert(PER >= 1 && PER * NT == NF && NF <= kFineMax, "whole bins per thread");
    const int tid = threadIdx.x, lane = lane_id();
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int b = blockIdx.x, k = a.k, N = a.N, W = a.W;
    const int budget = a.budget;
    const int32_t* s_ids = reinterpret_cast<const int32_t*>(lds + a.o_ids);
    uint32_t M;
    const uint32_t J = threshold_bin(P.hist, budget, M);
    // lower edge (in S) of the last bin that holds entries, below the
    // catch-all bin: the fine bins cover 0 .. edge, quadratically spaced
    // (scores crowd towards the threshold)
    float inv;
    {
        const uint4* h = reinterpret_cast<const uint4*>(P.hist) + 2 * lane;
        const uint4 x = h[0], y = h[1];
        const uint32_t v[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
        int last = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) last = (v[i] != 0u && 8 * lane + i <= (int)min(J, (uint32_t)kBins - 2)) ? 8 * lane + i : last;
        last = (int)wave_max_u32_dpp((uint32_t)last);
        inv = 1.f / (__uint_as_float((uint32_t)(last + 1 + (127 << kBinBits)) << (23 - kBinBits)) - 1.f);
    }
    auto fine_bin = [&](float S) {
        const float u = fminf(fmaxf(-S * inv, 0.f), 1.f);
        return (int)fminf(u * u * (float)NF, (float)(NF - 1));
    };
    if constexpr (CUT) M = budget;
    auto takes = [&](int e, float S) __attribute__((always_inline)) {
        if constexpr (CUT) return score_bin(S) <= J && bound.at_most(S, P.key[e]);
        return score_bin(S) <= J;
    };
    for (int e = 1 + tid; e < n; e += NT) {
        const float S = P.S(e);
        if (takes(e, S)) P.place[e] = (uint16_t)atomicAdd(&P.fine[fine_bin(S)], 1u);
    }
    __syncthreads();
    // counts -> offsets, PER consecutive bins per thread
    {
        uint32_t c[PER], sum = 0u, most = 0u;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            c[i] = P.fine[tid * PER + i];
            sum += c[i];
            most = max(most, c[i]);
        }
        const uint32_t incl = wave_scan_dpp(sum);
        if (lane == kWave - 1) P.misc[wv] = incl;
        if (!CUT && most > kCrowd) P.misc[61] = 1u;
        __syncthreads();
        uint32_t off = incl - sum;
        for (int w = 0; w < wv; ++w) off += P.misc[w];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            P.fine[tid * PER + i] = off;
            off += c[i];
        }
        if (tid == NT - 1) P.fine[NF] = off;
    }
    __syncthreads();
    if (!CUT && __builtin_expect((int)M >= budget + kCrowd / 2 && P.misc[61] != 0u, 0)) return false;
    for (int e = 1 + tid; e < n; e += NT) {
        const float S = P.S(e);
        if (takes(e, S)) P.list[P.fine[fine_bin(S)] + P.place[e]] = (uint16_t)e;
    }
    __syncthreads();
    int nt = min((int)M, budget);  // non-root rows
    for (int t = tid; t < (int)M; t += NT) {
        const int e = P.list[t];
        const float S = P.S(e);
        const int f = fine_bin(S);
        const int q0 = (int)P.fine[f], q1 = (int)P.fine[f + 1];
        int at = q0;
        if (q1 - q0 > 1) {
            // four members of the bin at a time, every read unconditional (a
            // key read behind the comparison of S made each member of a bin
            // of 256 equal scores a chain of three LDS round trips)
            const typename Pool<KW>::Key ke = P.key[e];
            for (int q = q0; q < q1; q += 4) {
                int o[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) o[u] = P.list[min(q + u, q1 - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float So = P.S(o[u]);
                    const bool less = key_less<KW>(P.key[o[u]], ke);
                    at += ((q + u < q1) & ((So > S) | ((So == S) & less))) ? 1 : 0;
                }
            }
        }
        P.place[e] = (uint16_t)(at + 1);
        if (at < nt) P.row[at + 1] = (uint16_t)e;
    }
    if (tid == 0) P.place[0] = 0;
    __syncthreads();
    if (__builtin_expect(fill, 0)) {
        uint16_t* child = reinterpret_cast<uint16_t*>(P.key);  // the keys have done their part
        for (int i = tid; i < n * k; i += NT) child[i] = 0;
        __syncthreads();
        for (int e = 1 + tid; e < n; e += NT) {
            const uint32_t y = P.rec[e].y;
            child[(y & 8191u) * k + ((y >> 13) & 15u)] = (uint16_t)e;
        }
        __syncthreads();
        if (tid < kWave) {
            const int rows = fill_below<KW>(a, P, child, n, nt, scores);
            if (tid == 0) P.misc[62] = (uint32_t)rows;
        }
        __syncthreads();
        nt = (int)P.misc[62];
    }
    // rows
    const int64_t ob = (int64_t)b * N;
    const int root_tok = __builtin_amdgcn_readfirstlane(a.root_token[b]);
    for (int i = tid; i < N; i += NT) {
        int par = -1, tok = -1, dep = -1, rank = -1;
        float S = -INFINITY;
        if (i == 0) {
            tok = root_tok;
            dep = 0;
            S = 0.f;
        } else if (i <= nt) {
            const uint2 r = P.rec[P.row[i]];
            rank = (int)(r.y >> 13) & 15;
            dep = (int)(r.y >> 21);
            tok = s_ids[(dep - 1) * k + rank];
            par = min((int)P.place[r.y & 8191u], i - 1);
            S = __uint_as_float(r.x);
            P.par[i] = (uint16_t)par;
        }
        a.parent[ob + i] = par;
        a.token[ob + i] = tok;
        a.depth[ob + i] = dep;
        a.rank[ob + i] = rank;
        a.score[ob + i] = S;
    }
    __syncthreads();
    // ancestor masks: the parent chain downwards in row index, one 64-bit
    // word at a time
    for (int i = tid; i < N; i += NT) {
        int y = i <= nt ? i : -1;
        for (int q = W - 1; q >= 0; --q) {
            uint64_t w = 0ull;
            while (y >= q * 64) {
                w |= 1ull << (y & 63);
                y = y == 0 ? -1 : (int)P.par[y];
            }
            a.anc[(ob + i) * W + q] = w;
        }
    }
    if (tid == 0) a.n_nodes[b] = nt + 1;
    return true;
}

template <int NT, int NF, int KW, typename Scores>
__device__ __forceinline__ void finish_tree(const TreeArgs& a, char* lds, const Pool<KW>& P, int n,
                                            const Scores& scores, bool fill) {
    if (__builtin_expect(place_tree<NT, NF, KW, false>(a, lds, P, n, scores, fill, Bound<KW>()), 1)) return;
    // without the entries past the budget-th best
    for (int i = threadIdx.x; i < NF; i += NT) P.fine[i] = 0u;
    __syncthreads();
    uint32_t M;
    const uint32_t J = threshold_bin(P.hist, a.budget, M);
    const Bound<KW> bound =
        select_best<NT, KW>(P, n - 1, a.budget, [&](int i, float& S, typename Pool<KW>::Key& key) {
            S = P.S(i + 1);
            key = P.key[i + 1];
            return score_bin(S) <= J;
        });
    place_tree<NT, NF, KW, true>(a, lds, P, n, scores, fill, bound);
}

// Best-first tree, level by level.
//
// Every token score is <= 0, so S never increases along a path and an
// ancestor precedes its descendants in the total order: the nodes that
// best-first search commits, in pop order, are the `budget` best non-root
// prefixes in that order (the closed form of Sec. 4.2), sorted.  The kernel
// collects that set: level d's candidates are the children of level d - 1's
// entries, one thread per candidate, and a candidate enters the pool unless
// `budget` better entries are known, which a histogram of the scores tells
// (threshold_bin: entries in bins past the one holding the budget-th best
// cannot be in the tree, nor can their descendants).  A level with more
// candidates than threads is counted first and entered afterwards, so that
// its own scores already bound it.  The search ends when a level enters
// nothing: the trees are wide and shallow (6 to 15 levels at depths 16 to 32,
// 1.2 to 4 entries per budgeted node on peaked, flat and Gaussian drafters),
// and finish_tree sorts what remains at or above the threshold.  One barrier
// per level, two where it is counted first.  A level that overflows the pool
// is entered again after the entries that its own scores have ruled out are
// dropped, and where (nearly) equal scores at the threshold alone are more than
// the pool holds, after the budget-th best is found exactly, path and all
// (select_best, 10 to 40 us; its bound also holds for the levels below).
// All scores alike, 8 sequences, against the merged set: depth 12, k = 12,
// budget 256 207 -> 38 us; 32, 4, 128 44 -> 24; 16, 16, 512 925 -> 66.  Two
// candidates of probability 1 in every row, which no softmax gives, tie at
// every level anew: 16, 4, 64 55 -> 101; 32, 4, 128 238 -> 510; larger budgets
// gain (16, 10, 1023 1953 -> 577).
//
// Latency bounds it: a level is a chain of LDS round trips (count, record,
// score, place, record) of about 1000 cycles, on one workgroup per sequence.
// Measured per call, against merging a sorted set of the best prefixes sweep
// by sweep (budgets 33 - 512) or popping one node at a time (others): budget
// 64, k = 4: 29.8 -> 11.1 us; 32 sequences of budget 128, depth 32: 33.2 ->
// 14.8; budget 256, k = 8: 89.4 -> 16.4.
// Candidates of S = -inf are left out (all their descendants tie with them);
// where only they can fill the tree, a depth-first walk adds them (fill_below).
//
// search_levels: levels d .. D from the pool's entries [lo, hi) of the one above.
// False (TIES = false only): more (nearly) equal scores at the threshold than
// the pool holds; the pool is as before level d, but for entries past hi, the
// histogram holds all the level's candidates.  TIES goes on from there.
template <int NT, int RHO, int KW, bool TIES>
__device__ __forceinline__ bool search_levels(const TreeArgs& a, const Pool<KW>& P, const TokenScores<RHO>& scores,
                                              int& d, int& lo, int& hi, uint32_t& J, bool& below) {
    typedef typename Pool<KW>::Key Key;
    const int tid = threadIdx.x, lane = lane_id();
    const int D = a.D, k = a.k;
    bool again = false;    // the level is entered for the second time, counted as it is
    bool over = TIES;      // its ties are too many
    bool recount = false;  // entered after that, to be counted anew
    bool bounded = false;  // candidates past `bound` are dropped
    Bound<KW> bound;
    uint32_t known = 0u;
    while (d <= D) {
        const int total = (hi - lo) * k;
        const int wi = (d - 1) / a.per_word, sh = 32 - ((d - 1) % a.per_word + 1) * a.wbits;
        // candidate i of the level: entry p's child of rank r
        auto score = [&](int i, int& p, int& r, uint2& rec, uint32_t& bin) __attribute__((always_inline)) {
            const int q = k == 1 ? i : (int)__umulhi((uint32_t)i, a.mag_k);
            r = i - q * k;
            p = lo + q;
            rec = P.rec[p];
            const int rank = (int)(rec.y >> 13) & 15, prank = (int)(rec.y >> 17) & 15;
            const float s = scores(d - 1, prank, rank, r);
            bool in = true;
            if (a.branch < k) {
                // the top-`branch` by token score (larger s, then lower rank)
                int sel = 0;
                for (int j = 0; j < k; ++j) {
                    const float sj = scores(d - 1, prank, rank, j);
                    sel += ((sj > s) | ((sj == s) & (j < r))) ? 1 : 0;
                }
                in = sel < a.branch;
            }
            const float S = __uint_as_float(rec.x) + s;
            below |= in & (S == -INFINITY);
            rec.x = __float_as_uint(S);
            bin = score_bin(S);
            in = in & (S > -INFINITY) & (bin <= J);
            if constexpr (TIES)
                if (bounded) in = in && bound.at_most(S, Pool<KW>::child_key(P.key[p], wi, sh, r));
            return in;
        };
        if constexpr (TIES) {
            if (over) {
                // the exact bound over the pool and the level, and the pool without what it rules out
                const int held = hi - 1;
                bound = select_best<NT, KW>(P, held + total, a.budget, [&](int i, float& S, Key& key) {
                    if (i < held) {
                        S = P.S(i + 1);
                        key = P.key[i + 1];
                        return true;
                    }
                    int p, r;
                    uint2 rec;
                    uint32_t bin;
                    const bool in = score(i - held, p, r, rec, bin);
                    S = __uint_as_float(rec.x);
                    key = Pool<KW>::child_key(P.key[p], wi, sh, r);
                    return in;
                });
                bounded = true;
                if (tid == 0) P.misc[d] = 0u;
                compact_pool<NT, KW>(P, [&](float S, Key key) { return bound.at_most(S, key); }, lo, hi);
                for (int i = tid; i < kBins; i += NT) P.hist[i] = 0u;
                __syncthreads();
                for (int e = 1 + tid; e < hi; e += NT) atomicAdd(&P.hist[score_bin(P.S(e))], 1u);
                over = again = false;
                recount = true;
                continue;
            }
        }
        const bool counted = (total > NT && !recount) || again;
        if (counted && !again) {
            for (int i = tid; i < total; i += NT) {
                int p, r;
                uint2 rec;
                uint32_t bin;
                if (score(i, p, r, rec, bin)) atomicAdd(&P.hist[bin], 1u);
            }
            __syncthreads();
            J = threshold_bin(P.hist, a.budget, known);
        }
        for (int i0 = 0; i0 < total; i0 += NT) {
            int p = 0, r = 0;
            uint2 rec = make_uint2(0u, 0u);
            uint32_t bin = 0u;
            bool in = false;
            if (i0 + tid < total) in = score(i0 + tid, p, r, rec, bin);
            const uint64_t m = __ballot(in);
            if (m != 0ull) {
                uint32_t at = 0u;
                if (lane == 0) at = atomicAdd(&P.misc[d], (uint32_t)__popcll(m));
                at = hi + (uint32_t)__builtin_amdgcn_readlane((int)at, 0) + lanes_below(m);
                if (in & (at < (uint32_t)a.cap)) {
                    const Key pk = P.key[p];
                    P.rec[at] = make_uint2(rec.x, Pool<KW>::meta(p, r, (int)(rec.y >> 13) & 15, d));
                    P.key[at] = Pool<KW>::child_key(pk, wi, sh, r);
                }
                if (in & !counted) atomicAdd(&P.hist[bin], 1u);
            }
        }
        __syncthreads();
        const int entered = (int)P.misc[d];
        if (__builtin_expect(hi + entered > a.cap, 0)) {
            // the histogram holds every candidate of the level, entered or not
            J = threshold_bin(P.hist, a.budget, known);
            __syncthreads();  // every wave has read the level's count
            if ((int)known >= a.cap) {
                if constexpr (!TIES) return false;
                over = true;
                continue;
            }
            if (tid == 0) P.misc[d] = 0u;
            compact_pool<NT, KW>(P, [&](float S, Key) { return score_bin(S) <= J; }, lo, hi);
            again = true;
            continue;
        }
        again = recount = false;
        lo = hi;
        hi += entered;
        ++d;
        if (entered == 0) break;
        if (!counted && hi > a.budget) J = threshold_bin(P.hist, a.budget, known);
    }
    return true;
}

template <int NT, int RHO, int KW>
__global__ __launch_bounds__(NT) void tree_level_kernel(TreeArgs a) {
    extern __shared__ __align__(16) char lds[];
    const Pool<KW> P(a, lds);
    constexpr int NF = NT < 512 ? 512 : kFineMax;
    init_pool<NT, NF, KW>(a, P);
    stage_tables<NT, RHO>(a, lds);
    const TokenScores<RHO> scores(a, lds);
    int d = 1, lo = 0, hi = 1;  // next level, entries of the one above
    uint32_t J = kBins - 1;     // candidates in later bins are dropped
    bool below = false;         // a candidate of S = -inf was left out
    if (__builtin_expect(!search_levels<NT, RHO, KW, false>(a, P, scores, d, lo, hi, J, below), 0))
        search_levels<NT, RHO, KW, true>(a, P, scores, d, lo, hi, J, below);
    // the counts are shared, so the whole workgroup agrees on the outcome (a
    // wave's J may differ, finish_tree takes it anew)
    bool fill = false;
    if (hi - 1 < a.budget) {
        if (below) P.misc[63] = 1u;
        __syncthreads();
        fill = P.misc[63] != 0u;
    }
    finish_tree<NT, NF, KW>(a, lds, P, hi, scores, fill);
}

// The one-node-at-a-time search as a kernel of its own, one wave, for the
// smallest trees (see pops_first).  The lattice is not staged: a node's children
// are scored from global memory as it is expanded (raw in LDS, 1024 words took
// 0.3 us more and a pop as long).
template <int RHO, bool QUAD>
__global__ __launch_bounds__(kWave) void tree_pop_kernel(TreeArgs a) {
    static_assert(RHO != 1, "the lattice is not scored ahead");
    extern __shared__ __align__(16) char lds[];
    const int lane = lane_id(), n = a.D * a.k;
    const int64_t tb = (int64_t)blockIdx.x * n;
    uint32_t r_lp[8], r_ids[8];  // D * k <= 512 words
    load_words(r_lp, reinterpret_cast<const uint32_t*>(a.logprob + tb), n, 0, lane);
    load_words(r_ids, reinterpret_cast<const uint32_t*>(a.ids + tb), n, 0, lane);
    const float lam = lane < a.D ? a.lambda[(int64_t)blockIdx.x * a.lambda_stride + lane] : 0.f;
    if constexpr (RHO == 0) {
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (u * kWave < n) {
                const float v = __uint_as_float(r_lp[u]);
                r_lp[u] = __float_as_uint((v == v) ? v : -INFINITY);
            }
    }
    store_words(reinterpret_cast<uint32_t*>(lds + a.o_lp), r_lp, n, 0, lane);
    store_words(reinterpret_cast<uint32_t*>(lds + a.o_ids), r_ids, n, 0, lane);
    if (lane < a.D) reinterpret_cast<float*>(lds + a.o_lam)[lane] = lam;
    __builtin_amdgcn_wave_barrier();
    tree_pop_search<RHO, QUAD>(a, lds);
}

// Beam search with global retention (Alg. 1): per depth, every beam entry's
// top-`branch` children join T, and the `beam_width` best of them (S desc,
// rank path asc) form the next beam; depths are taken while T holds fewer
// than `budget` nodes.  T never exceeds budget - 1 + beam_width * k entries, so it
// is kept whole, and the tree is its `budget` best (finish_tree).
//
// One thread per candidate (beam_width * k <= 256).  The beam is kept in
// rank-path order, so a candidate's index orders it by path among its depth:
// its place comes from comparing (ord S, index) keys with every candidate's,
// and the chosen ones keep their order by a prefix count.  Three barriers per
// depth.  k = 10, width 10, budget 512: 27.8 us per call, where a best-first
// search restricted to T, one node at a time (about 1300 cycles each), took
// 367.
constexpr int kBeamThreads = 256;
template <int RHO, int KW>
__global__ __launch_bounds__(kBeamThreads) void tree_beam_kernel(TreeArgs a) {
    constexpr int NT = kBeamThreads;
    extern __shared__ __align__(16) char lds[];
    __shared__ __align__(16) uint64_t s_keys[NT];
    __shared__ uint16_t s_beam[2][64];  // pool entries of the beam, in rank-path order
    __shared__ uint32_t s_wave[NT / kWave];
    const int tid = threadIdx.x, lane = lane_id();
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int D = a.D, k = a.k, width = a.beam_width;
    const Pool<KW> P(a, lds);
    init_pool<NT, kFineMax, KW>(a, P);
    if (tid == 0) s_beam[0][0] = 0;
    stage_tables<NT, RHO>(a, lds);
    const TokenScores<RHO> scores(a, lds);

    int nb = 1, n = 1, cur = 0;
    for (int d = 1; d <= D && n - 1 < a.budget && nb > 0; ++d) {
        const int total = nb * k;
        const int wi = (d - 1) / a.per_word, sh = 32 - ((d - 1) % a.per_word + 1) * a.wbits;
        bool in = tid < total;
        const int pb = k == 1 ? tid : (int)__umulhi((uint32_t)tid, a.mag_k), r = tid - pb * k;
        int p = 0, rank = 0;
        float S = 0.f;
        if (in) {
            p = s_beam[cur][pb];
            const uint2 rec = P.rec[p];
            rank = (int)(rec.y >> 13) & 15;
            const int prank = (int)(rec.y >> 17) & 15;
            const float s = scores(d - 1, prank, rank, r);
            if (a.branch < k) {
                int sel = 0;
                for (int j = 0; j < k; ++j) {
                    const float sj = scores(d - 1, prank, rank, j);
                    sel += ((sj > s) | ((sj == s) & (j < r))) ? 1 : 0;
                }
                in = sel < a.branch;
            }
            S = __uint_as_float(rec.x) + s;
        }
        // larger S first, then the lower index; 0: no candidate
        const uint64_t key = in ? ((uint64_t)ord32(S) << 32) | (uint64_t)(0xffffffffu - (uint32_t)tid) : 0ull;
        s_keys[tid] = key;
        __syncthreads();
        int before = 0;
        const ulonglong2* kv = reinterpret_cast<const ulonglong2*>(s_keys);
        for (int j = 0; j < (total + 1) / 2; ++j) {
            const ulonglong2 x = kv[j];
            before += (x.x > key ? 1 : 0) + (x.y > key ? 1 : 0);
        }
        const bool sel = in & (before < width);
        const uint64_t mi = __ballot(in), ms = __ballot(sel);
        if (lane == 0) s_wave[wv] = (uint32_t)__popcll(mi) | ((uint32_t)__popcll(ms) << 16);
        __syncthreads();
        uint32_t off = 0u, all = 0u;
#pragma unroll
        for (int w = 0; w < NT / kWave; ++w) {
            const uint32_t c = s_wave[w];
            off += w < wv ? c : 0u;
            all += c;
        }
        const int at = n + (int)(off & 0xffffu) + lanes_below(mi);
        if (in & (at < a.cap)) {
            P.rec[at] = make_uint2(__float_as_uint(S), Pool<KW>::meta(p, r, rank, d));
            P.key[at] = Pool<KW>::child_key(P.key[p], wi, sh, r);
            atomicAdd(&P.hist[score_bin(S)], 1u);
            if (sel) s_beam[cur ^ 1][(int)(off >> 16) + lanes_below(ms)] = (uint16_t)at;
        }
        n += (int)(all & 0xffffu);
        nb = (int)(all >> 16);
        cur ^= 1;
        __syncthreads();
    }
    finish_tree<NT, kFineMax, KW>(a, lds, P, min(n, a.cap), scores, false);
}

// Literal Alg. 2 (Sec. 4.2): T grows by whole expansions.  The root is
// expanded first; every later pop takes the best node of T not yet expanded
// (total order: S desc, rank path asc) and appends its top-`branch`
// children to T.  The search stops once T holds `budget` non-root nodes (the
// last expansion may overshoot by branch - 1) or nothing is left to expand,
// and the tree is TopB(T): the `budget` best nodes of T, in the total order,
// after the root.  One wavefront per sequence: T lives in LDS (per node the
// parent, rank and depth in one word, S, and the rank-path key, built from
// the parent's key when the node is appended); node e of T is "not yet
// expanded" while slot e / 64 of lane e % 64 holds ord(S) (0 once expanded).
// TopB(T) places every node by counting the nodes before it.
template <int SLT, int RHO>
__global__ __launch_bounds__(kWave) void tree_alg2_kernel(TreeArgs a) {
    extern __shared__ __align__(16) char lds[];
    const int lane = lane_id();
    const int b = blockIdx.x;
    const int D = a.D, k = a.k, N = a.N, W = a.W, wbits = a.wbits, per_word = a.per_word;
    const int branch = a.branch, budget = a.budget;
    float* s_lp = reinterpret_cast<float*>(lds + a.o_lp);
    int32_t* s_ids = reinterpret_cast<int32_t*>(lds + a.o_ids);
    float* s_rho = reinterpret_cast<float*>(lds + a.o_rho);
    // T node c: (parent + 1, 0 for the root) | rank << 11 | depth << 15
    // (T holds up to budget + branch - 1 <= 1038 nodes: 11 bits of parent)
    uint32_t* s_tmeta = reinterpret_cast<uint32_t*>(lds + a.o_tmeta);
    float* s_tS = reinterpret_cast<float*>(lds + a.o_tS);
    uint4* s_tkey = reinterpret_cast<uint4*>(lds + a.o_tkey);  // x: most significant word
    int32_t* s_tplace = reinterpret_cast<int32_t*>(lds + a.o_tplace);
    const int rho_n = D * k * k * k;
    const float* g_rho = RHO ? a.log_rho + (int64_t)b * rho_n : nullptr;

    // every load of the tables requested before the first store, as in the
    // best-first kernel
    const float lam_lane = lane < D ? a.lambda[(int64_t)b * a.lambda_stride + lane] : 0.f;
    const int64_t tb = (int64_t)b * D * k;
    {
        uint32_t r_lp[8], r_ids[8], r_rho[16];  // D * k <= 512 words
        load_words(r_lp, reinterpret_cast<const uint32_t*>(a.logprob + tb), D * k, 0, lane);
        load_words(r_ids, reinterpret_cast<const uint32_t*>(a.ids + tb), D * k, 0, lane);
        if constexpr (RHO == 1) load_words(r_rho, reinterpret_cast<const uint32_t*>(g_rho), rho_n, 0, lane);
        store_words(reinterpret_cast<uint32_t*>(s_lp), r_lp, D * k, 0, lane);
        store_words(reinterpret_cast<uint32_t*>(s_ids), r_ids, D * k, 0, lane);
        if constexpr (RHO == 1) {
            store_words(reinterpret_cast<uint32_t*>(s_rho), r_rho, rho_n, 0, lane);
            if (rho_n > 16 * kWave)
                stage_words(reinterpret_cast<uint32_t*>(s_rho) + 16 * kWave,
                            reinterpret_cast<const uint32_t*>(g_rho) + 16 * kWave, rho_n - 16 * kWave,
                            lane);
        }
    }
    __builtin_amdgcn_wave_barrier();

    // Appends the top-`branch` children (by s desc, rank asc) of the node v
    // (T index, -1 for the root; depth d < D, own rank rn, parent's rank rp,
    // score Sv, key kv) to T at index nT.  Lane r scores candidate r.
    auto expand = [&](int v, int d, int rn, int rp, float Sv, uint4 kv, int nT) {
        const int ctx2 = d >= 2 ? rp : 0;
        const int ctx1 = d >= 1 ? rn : 0;
        const int rl = min(lane, k - 1);
        float s = s_lp[d * k + rl];
        if constexpr (RHO != 0) {
            const float lam_d = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lam_lane), d));
            const int ri = ((d * k + ctx2) * k + ctx1) * k + rl;
            const float lr = RHO == 1 ? s_rho[ri] : g_rho[ri];
            const float t = lam_d * lr;
            s = s + t;
        }
        s = (s == s && lane < k) ? s : -INFINITY;
        int sel = 0;
        for (int j = 0; j < k; ++j) {
            const float sj = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s), j));
            sel += (sj > s || (sj == s && j < lane)) ? 1 : 0;
        }
        if (lane < k && sel < branch) {
            const int c = nT + sel;
            s_tmeta[c] = (uint32_t)(v + 1) | ((uint32_t)lane << 11) | ((uint32_t)(d + 1) << 15);
            s_tS[c] = Sv + s;
            const int wi = d / per_word, sh = 32 - (d % per_word + 1) * wbits;
            const uint32_t dig = (uint32_t)(lane + 1) << sh;
            s_tkey[c] = make_uint4(kv.x | (wi == 0 ? dig : 0u), kv.y | (wi == 1 ? dig : 0u),
                                   kv.z | (wi == 2 ? dig : 0u), kv.w | (wi == 3 ? dig : 0u));
        }
        __builtin_amdgcn_wave_barrier();
    };
    // marks T nodes n0 .. n0 + cnt - 1 as not yet expanded
    uint32_t fO[SLT];
#pragma unroll
    for (int j = 0; j < SLT; ++j) fO[j] = 0u;
    auto mark_open = [&](int n0, int cnt) {
#pragma unroll
        for (int j = 0; j < SLT; ++j) {
            const int e = j * kWave + lane;
            if (e >= n0 && e < n0 + cnt) fO[j] = ord32(s_tS[e]);
        }
    };
    auto key_less = [](uint4 x, uint4 y) {
        return x.x != y.x ? x.x < y.x : (x.y != y.y ? x.y < y.y : (x.z != y.z ? x.z < y.z : x.w < y.w));
    };

    expand(-1, 0, 0, 0, 0.f, make_uint4(0u, 0u, 0u, 0u), 0);  // depth >= 1: the root has children
    mark_open(0, branch);
    int nT = branch;
    while (nT < budget) {
        uint32_t lm = 0u;
#pragma unroll
        for (int j = 0; j < SLT; ++j) lm = max(lm, fO[j]);
        const uint32_t M = wave_max_u32_dpp(lm);
        if (M == 0u) break;  // every node of T expanded
        int cnt = 0, jsel = 0;
#pragma unroll
        for (int j = SLT - 1; j >= 0; --j) {
            const bool hit = fO[j] == M;
            cnt += hit ? 1 : 0;
            jsel = hit ? j : jsel;
        }
        const uint64_t any = __ballot(cnt > 0);
        int w;
        if (__popcll(any) == 1 && __ballot(cnt > 1) == 0ull) {
            w = __ffsll((unsigned long long)any) - 1;
        } else {
            // several nodes share the best S: the smallest rank-path key wins
            uint4 bk = make_uint4(~0u, ~0u, ~0u, ~0u);
            int bj = 0;
            for (int j = 0; j < SLT; ++j) {
                if (fO[j] == M) {
                    const uint4 kj = s_tkey[j * kWave + lane];
                    if (key_less(kj, bk)) {
                        bk = kj;
                        bj = j;
                    }
                }
            }
            bool t = cnt > 0;
            uint32_t m;
            m = wave_min_u32_dpp(t ? bk.x : ~0u); t = t && bk.x == m;
            m = wave_min_u32_dpp(t ? bk.y : ~0u); t = t && bk.y == m;
            m = wave_min_u32_dpp(t ? bk.z : ~0u); t = t && bk.z == m;
            m = wave_min_u32_dpp(t ? bk.w : ~0u); t = t && bk.w == m;
            w = __ffsll((unsigned long long)__ballot(t)) - 1;
            jsel = bj;
        }
        const int es = __builtin_amdgcn_readlane(jsel, w);
        const int e = es * kWave + w;
#pragma unroll
        for (int j = 0; j < SLT; ++j) fO[j] = (lane == w && j == es) ? 0u : fO[j];
        const uint32_t meta = s_tmeta[e];
        const int d = (meta >> 15) & 63;
        if (d < D) {
            const int pv = (int)(meta & 2047) - 1;
            const int rp = pv >= 0 ? (int)((s_tmeta[pv] >> 11) & 15) : 0;
            expand(e, d, (meta >> 11) & 15, rp, s_tS[e], s_tkey[e], nT);
            mark_open(nT, branch);
            nT += branch;
        }
    }

    // TopB(T): the place of node i in the total order is the number of nodes
    // of T before it (S larger, or S equal and rank-path key smaller)
    const int keep = min(nT, budget);
    uint32_t oT[SLT];
#pragma unroll
    for (int q = 0; q < SLT; ++q) {
        const int i = q * kWave + lane;
        oT[q] = i < nT ? ord32(s_tS[i]) : 0u;
    }
    int place[SLT];
#pragma unroll
    for (int q = 0; q < SLT; ++q) place[q] = 0;
#pragma unroll
    for (int sj = 0; sj < SLT; ++sj) {
        for (int l = 0; l < kWave; ++l) {
            const int j = sj * kWave + l;
            if (j >= nT) break;
            const uint32_t oj = (uint32_t)__builtin_amdgcn_readlane((int)oT[sj], l);
            bool tie = false;
#pragma unroll
            for (int q = 0; q < SLT; ++q) {
                place[q] += oj > oT[q] ? 1 : 0;
                tie = tie || (oj == oT[q] && q * kWave + lane != j && q * kWave + lane < nT);
            }
            if (__ballot(tie)) {
                const uint4 kj = s_tkey[j];
#pragma unroll
                for (int q = 0; q < SLT; ++q) {
                    const int i = q * kWave + lane;
                    if (oj == oT[q] && i != j && i < nT && key_less(kj, s_tkey[i])) ++place[q];
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < SLT; ++q) {
        const int i = q * kWave + lane;
        if (i < nT) s_tplace[i] = place[q];
    }
    __builtin_amdgcn_wave_barrier();

    // output: row 0 the root, rows 1 .. keep the kept nodes in order, then padding
    const int64_t ob = (int64_t)b * N;
    constexpr int SLW = SLT + 1;  // mask words: N = budget + 1 <= 64 * SLT + 1
    for (int i = lane; i < nT; i += kWave) {
        const int pl = s_tplace[i];
        if (pl >= keep) continue;
        const int o = pl + 1;
        const uint32_t meta = s_tmeta[i];
        const int pv = (int)(meta & 2047) - 1, r = (meta >> 11) & 15, d = (meta >> 15) & 63;
        int po = 0;
        if (pv >= 0) po = s_tplace[pv] < keep ? s_tplace[pv] + 1 : -2;
        a.parent[ob + o] = po;
        a.token[ob + o] = s_ids[(d - 1) * k + r];
        a.depth[ob + o] = d;
        a.rank[ob + o] = r;
        a.score[ob + o] = s_tS[i];
        // ancestor bits: this node, then the parent chain until the root
        // (or a parent that TopB(T) dropped, which ends the chain)
        uint64_t words[SLW];
#pragma unroll
        for (int q = 0; q < SLW; ++q) words[q] = 0ull;
        int x = i, xo = o;
        while (true) {
#pragma unroll
            for (int q = 0; q < SLW; ++q) words[q] |= q == (xo >> 6) ? 1ull << (xo & 63) : 0ull;
            const int xv = (int)(s_tmeta[x] & 2047) - 1;
            if (xv < 0) {
                words[0] |= 1ull;  // the root
                break;
            }
            if (s_tplace[xv] >= keep) break;
            x = xv;
            xo = s_tplace[xv] + 1;
        }
#pragma unroll
        for (int q = 0; q < SLW; ++q)
            if (q < W) a.anc[(ob + o) * W + q] = words[q];
    }
    const int root_tok = __builtin_amdgcn_readfirstlane(a.root_token[b]);
    for (int i = lane; i < N; i += kWave) {
        if (i != 0 && i <= keep) continue;
        const bool root = i == 0;
        a.parent[ob + i] = -1;
        a.token[ob + i] = root ? root_tok : -1;
        a.depth[ob + i] = root ? 0 : -1;
        a.rank[ob + i] = -1;
        a.score[ob + i] = root ? 0.f : -INFINITY;
        for (int q = 0; q < W; ++q) a.anc[(ob + i) * W + q] = (root && q == 0) ? 1ull : 0ull;
    }
    if (lane == 0) a.n_nodes[b] = keep + 1;
}
}  // namespace presto

namespace presto_host {

using namespace presto;

static int align16(int x) { return (x + 15) & ~15; }

// gfx950 gives one workgroup up to 160 KiB of LDS; one sequence's search runs
// alone on its CU anyway.
static constexpr int kTreeLdsBudget = 160 * 1024;
static constexpr int kDefaultLds = 64 * 1024;

// Dynamic LDS above the default needs the kernel's own limit raised (once
// per instantiation and process).
template <typename K>
static presto_status allow_lds(K* kernel, int bytes) {
    if (bytes <= kDefaultLds) return PRESTO_OK;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e != hipSuccess)
        return set_error(PRESTO_ERR_HIP, "tree build: %d bytes of LDS refused: %s", bytes,
                         hipGetErrorString(e));
    return PRESTO_OK;
}

int tree_key_bits(int k) {
    int wbits = 1;
    while ((1 << wbits) < k + 1) ++wbits;
    return wbits;
}

// Deepest tree whose rank-path key fits four 32-bit words (digits never
// straddle a word).
int tree_max_depth(int k) { return 4 * (32 / tree_key_bits(k)); }

// Literal Alg. 2: candidate table, then T (capacity budget + branch - 1:
// the last expansion may overshoot the budget), then the lattice.
struct Alg2Layout {
    int cap, total_no_rho, total_with_rho;
    int o_lp, o_ids, o_tmeta, o_tS, o_tkey, o_tplace, o_rho;
};

static Alg2Layout alg2_layout(int D, int k, int branch, int budget) {
    Alg2Layout L;
    L.cap = budget + branch - 1;
    int off = 0;
    L.o_lp = off; off = align16(off + D * k * 4);
    L.o_ids = off; off = align16(off + D * k * 4);
    L.o_tmeta = off; off = align16(off + L.cap * 4);
    L.o_tS = off; off = align16(off + L.cap * 4);
    L.o_tkey = off; off = align16(off + L.cap * 16);
    L.o_tplace = off; off = align16(off + L.cap * 4);
    L.total_no_rho = off;
    L.o_rho = off;
    L.total_with_rho = align16(off + D * k * k * k * 4);
    return L;
}

// Threads of the level kernel: enough that a level's candidates (up to about
// budget * k / 2, usually budget) take few rounds, few enough that the
// barriers stay cheap.
static int level_threads(int budget) { return budget <= 128 ? 256 : (budget <= 256 ? 512 : 1024); }

// Trees of few nodes, or of one per level, go one node at a time: a pop takes
// about 0.5 us, a level 0.6 and its start and end (the staged lattice, the sort)
// about 3 us more.  us per call, pops / levels: 10 nodes, depth 16, k = 4 8.9 /
// 9.6, 12 nodes 9.9 / 9.5; with the 16,000 words of k = 10's lattice 16 nodes
// 15.4 / 18.3, 24 nodes 20.6 / 19.4; a chain of 32 nodes 21.9 / 28.3.
static bool pops_first(int D, int k, int branch, int budget, bool lattice) {
    if (branch == 1) return budget < kWave;
    return budget <= (lattice && D * k * k * k > 8192 ? 20 : 10);
}

// Level and beam kernels: candidate table, lambda, the pool with its sort
// scratch, then the lattice.
struct PoolLayout {
    int kw, cap, total;
    bool rho_in_lds;
    int o_lp, o_ids, o_lam, o_pool, o_key, o_hist, o_fine, o_list, o_place, o_row, o_par, o_misc, o_rho;
};

static PoolLayout pool_layout_cap(int D, int k, int N, bool lattice, int cap) {
    PoolLayout L;
    L.kw = D <= 2 * (32 / tree_key_bits(k)) ? 2 : 4;
    L.cap = cap;
    int off = 0;
    L.o_lp = off; off = align16(off + D * k * 4);
    L.o_ids = off; off = align16(off + D * k * 4);
    L.o_lam = off; off = align16(off + D * 4);
    L.o_pool = off; off = align16(off + cap * 8);
    L.o_key = off; off = align16(off + cap * 4 * L.kw);
    L.o_hist = off; off = align16(off + kBins * 4);
    L.o_fine = off; off = align16(off + (kFineMax + 1) * 4);
    L.o_list = off; off = align16(off + cap * 2);
    L.o_place = off; off = align16(off + cap * 2);
    L.o_row = off; off = align16(off + N * 2);
    L.o_par = off; off = align16(off + N * 2);
    L.o_misc = off; off = align16(off + 64 * 4);
    L.o_rho = off;
    L.rho_in_lds = lattice;
    L.total = lattice ? align16(off + D * k * k * k * 4) : off;
    return L;
}

// The pool holds five entries per budgeted node (three to four is what most
// searches enter) and 256 more, or what fits; the lattice is in LDS whenever
// that leaves room for two per node and 256.
static PoolLayout level_layout(int D, int k, int budget, bool lattice) {
    const int N = budget + 1;
    const int want = 5 * budget + 257 < kPoolMax ? 5 * budget + 257 : kPoolMax;
    for (int in_lds = lattice ? 1 : 0; in_lds >= 0; --in_lds)
        for (int cap = want; cap >= 2 * budget + 257; cap -= 64) {
            const PoolLayout L = pool_layout_cap(D, k, N, in_lds != 0, cap);
            if (L.total <= kTreeLdsBudget) return L;
        }
    return pool_layout_cap(D, k, N, false, 2 * budget + 257);
}

// static LDS of the beam kernel, taken off the dynamic budget
static constexpr int kBeamStatic = 4096;

static PoolLayout beam_layout(int D, int k, int budget, int width, bool lattice) {
    const int cap = budget + width * k + 1;  // root, T below the budget, one more depth
    const PoolLayout L = pool_layout_cap(D, k, budget + 1, lattice, cap);
    if (!lattice || L.total <= kTreeLdsBudget - kBeamStatic) return L;
    return pool_layout_cap(D, k, budget + 1, false, cap);
}

bool tree_build_fits(int D, int k, int branch, int N, int beam_width, bool alg2) {
    if (alg2) return alg2_layout(D, k, branch, N - 1).total_no_rho <= kTreeLdsBudget;
    if (beam_width > 0) return beam_layout(D, k, N - 1, beam_width, false).total <= kTreeLdsBudget - kBeamStatic;
    return level_layout(D, k, N - 1, false).total <= kTreeLdsBudget;
}

presto_status launch_build_tree(const presto_tree_desc* desc, const int32_t* ids,
                                const float* logprob, const float* log_rho, const float* lambda,
                                const int32_t* root_token, int32_t* n_nodes, int32_t* parent,
                                int32_t* token, int32_t* depth, int32_t* rank, float* score,
                                uint64_t* anc, hipStream_t stream) {
    TreeArgs a{};
    a.D = desc->depth;
    a.k = desc->k;
    a.branch = desc->branch;
    a.budget = desc->budget;
    a.N = desc->budget + 1;
    a.W = (a.N + 63) / 64;
    a.wbits = tree_key_bits(a.k);
    a.per_word = 32 / a.wbits;
    a.ids = ids;
    a.logprob = logprob;
    a.log_rho = log_rho;
    a.lambda = lambda;
    a.lambda_stride = desc->lambda_per_seq ? desc->depth : 0;
    a.root_token = root_token;
    a.n_nodes = n_nodes;
    a.parent = parent;
    a.token = token;
    a.depth = depth;
    a.rank = rank;
    a.score = score;
    a.anc = anc;
    presto_status st = PRESTO_OK;
    if (desc->mode == PRESTO_TREE_BEST_FIRST_ALG2) {
        const Alg2Layout L = alg2_layout(a.D, a.k, a.branch, a.budget);
        a.beam_width = 0;
        a.o_lp = L.o_lp; a.o_ids = L.o_ids; a.o_rho = L.o_rho;
        a.o_tmeta = L.o_tmeta; a.o_tS = L.o_tS; a.o_tkey = L.o_tkey; a.o_tplace = L.o_tplace;
        const bool rho_in_lds = log_rho != nullptr && L.total_with_rho <= kTreeLdsBudget;
        const int lds = rho_in_lds ? L.total_with_rho : L.total_no_rho;
        const int slt = (L.cap + kWave - 1) / kWave;
        const int rho_mode = log_rho == nullptr ? 0 : (rho_in_lds ? 1 : 2);
        auto go = [&](auto kernel) {
            st = allow_lds(kernel, lds);
            if (st == PRESTO_OK) kernel<<<desc->batch, kWave, lds, stream>>>(a);
        };
#define PRESTO_ALG2(S)                                    \
    if (rho_mode == 0) go(tree_alg2_kernel<S, 0>);        \
    else if (rho_mode == 1) go(tree_alg2_kernel<S, 1>);   \
    else go(tree_alg2_kernel<S, 2>)
        if (slt <= 1) { PRESTO_ALG2(1); }
        else if (slt <= 2) { PRESTO_ALG2(2); }
        else if (slt <= 4) { PRESTO_ALG2(4); }
        else if (slt <= 9) { PRESTO_ALG2(9); }
        else { PRESTO_ALG2(17); }
#undef PRESTO_ALG2
        if (st != PRESTO_OK) return st;
        return check_launch("tree_alg2_kernel");
    }
    const bool beam = desc->mode == PRESTO_TREE_BEAM;
    const bool lattice = log_rho != nullptr;
    a.beam_width = beam ? desc->beam_width : 0;
    if (!beam && pops_first(a.D, a.k, a.branch, a.budget, lattice)) {
        // candidate table, lambda, then per node its children, record and path key
        int lds = 0;
        auto take = [&](int& at, int bytes) { at = lds; lds = align16(lds + bytes); };
        take(a.o_lp, a.D * a.k * 4);
        take(a.o_ids, a.D * a.k * 4);
        take(a.o_lam, a.D * 4);
        take(a.o_kord, a.N * a.k * 4);
        take(a.o_krank, a.N * a.k);
        take(a.o_rec, a.N * 8);
        take(a.o_pkey, a.N * 16);
        auto go = [&](auto kernel) { kernel<<<desc->batch, kWave, lds, stream>>>(a); };
        if (a.k <= 4) {
            if (lattice) go(tree_pop_kernel<2, true>);
            else go(tree_pop_kernel<0, true>);
        } else {
            if (lattice) go(tree_pop_kernel<2, false>);
            else go(tree_pop_kernel<0, false>);
        }
        return check_launch("tree_pop_kernel");
    }
    const PoolLayout L = beam ? beam_layout(a.D, a.k, a.budget, a.beam_width, lattice)
                              : level_layout(a.D, a.k, a.budget, lattice);
    a.o_lp = L.o_lp; a.o_ids = L.o_ids; a.o_lam = L.o_lam; a.o_rho = L.o_rho;
    a.o_pool = L.o_pool; a.o_key = L.o_key; a.o_hist = L.o_hist; a.o_fine = L.o_fine; a.o_list = L.o_list;
    a.o_place = L.o_place; a.o_row = L.o_row; a.o_par = L.o_par; a.o_misc = L.o_misc;
    a.cap = L.cap;
    const uint64_t k3 = (uint64_t)a.k * a.k * a.k;
    a.mag_k = (uint32_t)(((1ull << 32) + a.k - 1) / a.k);  // k > 1 only
    a.mag_k3 = (uint32_t)(((1ull << 32) + k3 - 1) / k3);
    const int rho_mode = !lattice ? 0 : (L.rho_in_lds ? 1 : 2);
    const int threads = beam ? kBeamThreads : level_threads(a.budget);
    auto go = [&](auto kernel) {
        st = allow_lds(kernel, L.total);
        if (st == PRESTO_OK) kernel<<<desc->batch, threads, L.total, stream>>>(a);
    };
    if (beam) {
#define PRESTO_BEAM(K)                                    \
    if (rho_mode == 0) go(tree_beam_kernel<0, K>);        \
    else if (rho_mode == 1) go(tree_beam_kernel<1, K>);   \
    else go(tree_beam_kernel<2, K>)
        if (L.kw == 2) { PRESTO_BEAM(2); } else { PRESTO_BEAM(4); }
#undef PRESTO_BEAM
        if (st != PRESTO_OK) return st;
        return check_launch("tree_beam_kernel");
    }
#define PRESTO_LEVEL3(T, K)                                   \
    if (rho_mode == 0) go(tree_level_kernel<T, 0, K>);        \
    else if (rho_mode == 1) go(tree_level_kernel<T, 1, K>);   \
    else go(tree_level_kernel<T, 2, K>)
#define PRESTO_LEVEL(T) \
    if (L.kw == 2) { PRESTO_LEVEL3(T, 2); } else { PRESTO_LEVEL3(T, 4); }
    if (threads == 256) { PRESTO_LEVEL(256) }
    else if (threads == 512) { PRESTO_LEVEL(512) }
    else { PRESTO_LEVEL(1024) }
#undef PRESTO_LEVEL
#undef PRESTO_LEVEL3
    if (st != PRESTO_OK) return st;
    return check_launch("tree_level_kernel");
}

}  // namespace presto_host
