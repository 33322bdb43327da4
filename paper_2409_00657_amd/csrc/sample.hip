// hopgnn_sample: counter-hash k-hop sampling, one micrograph per root vertex
// (paper section 2 "sampling", section 4 "micrograph definition").
//
// One workgroup owns one micrograph and walks its levels in order; a level is
// written to HBM (coalesced inside the micrograph's slice of the level-major
// array) and read back by the same workgroup after a barrier, so all hops of
// all micrographs run in a single launch.  Work per slot is two dependent
// random reads (row bounds, then one neighbour) - latency bound, hidden by
// keeping every micrograph's workgroup resident at once.
#include <type_traits>

#include "pregather_internal.hpp"

namespace hopgnn {

struct SampleShape {
    int32_t n_layers;
    int32_t f[kMaxLayers + 1];      // f[h], h = 1..L
    int32_t P[kMaxLayers + 1];      // P[h] = slots per micrograph at level h
    int32_t base[kMaxLayers + 2];   // base[h] = first slot of level h; base[L+1] = T
};

__device__ __forceinline__ uint64_t finalise64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Exact unsigned 64-bit remainder (a multiply-high range reduction would pick
// different neighbours and is not an acceptable substitute).
__device__ __forceinline__ uint64_t mod_u64(uint64_t x, uint64_t d) {
    return x % d;
}

// Batches sampled by one launch: blockIdx.y picks the batch, i.e. its seeds, its key (first
// hash round already applied on the host) and its slice of the outputs.
constexpr int kMaxBatchesPerLaunch = 64;
struct BatchKeys {
    uint64_t keyed[kMaxBatchesPerLaunch];
};

constexpr int kSampleUnroll = 4;

template <typename OffT>
__global__ void __launch_bounds__(256)
sample_micrographs(const OffT* __restrict__ offsets, const int32_t* __restrict__ indices,
                   const int32_t* __restrict__ seeds, int32_t n_seeds, SampleShape sh,
                   BatchKeys keys, int32_t* ids, int32_t* indptr, int32_t* slot_idx, int64_t slot_idx_stride,
                   uint8_t* __restrict__ present, int32_t m_offset, int32_t seeds_per_key, int32_t has_edges) {
    // Two ways to carry several keys: blockIdx.y = one batch (own seeds, key and output slices) of
    // n_seeds micrographs each, or ONE level-major batch whose micrographs m_offset + blockIdx.x
    // take the key of their block of seeds_per_key consecutive seeds (then gridDim.y = 1).
    const int32_t m = m_offset + (int32_t)blockIdx.x;
    const int32_t B = n_seeds;
    const uint32_t batch = blockIdx.y;
    const uint64_t keyed = keys.keyed[batch + blockIdx.x / (uint32_t)seeds_per_key];
    seeds += (int64_t)batch * B;
    ids += (int64_t)batch * sh.base[sh.n_layers + 1];
    if (slot_idx != nullptr) slot_idx += (int64_t)batch * slot_idx_stride;
    if (batch != 0) indptr = nullptr;      // the segment offsets are the same for every batch of one shape
    const int32_t root = seeds[m];
    if (threadIdx.x == 0) {
        ids[m] = root;
        if (present != nullptr && root >= 0) present[root] = 1;   // the pre-gather's presence map
        if (indptr != nullptr && m == 0) indptr[sh.base[sh.n_layers]] = sh.base[sh.n_layers + 1] - B;
    }
    for (int32_t h = 1; h <= sh.n_layers; ++h) {
        const uint32_t f = sh.f[h];
        const int32_t P = sh.P[h];
        const int32_t* parents = ids + sh.base[h - 1] + (int64_t)m * sh.P[h - 1];
        int32_t* children = ids + sh.base[h] + (int64_t)m * P;
        // Several slots per thread and round: every slot is a chain of dependent random reads
        // (parent, its two row bounds, one neighbour), so the chains of a round are issued side by
        // side - all bounds, then all neighbours - instead of one after the other.  Loads are
        // unconditional from clamped, in-bounds addresses; what must not count is masked afterwards.
        auto level = [&](auto unroll) {
        constexpr int U = decltype(unroll)::value;
        for (uint32_t c0 = threadIdx.x; c0 < (uint32_t)P; c0 += blockDim.x * U) {
            uint32_t q[U], j[U];
            int32_t v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t c = c0 + u * blockDim.x;
                const uint32_t cc = c < (uint32_t)P ? c : 0u;
                q[u] = cc / f;
                j[u] = cc - q[u] * f;
                v[u] = (h == 1) ? root : parents[q[u]];
                if (c >= (uint32_t)P) v[u] = -1;
            }
            int64_t o0[U], deg[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t vv = v[u] >= 0 ? v[u] : 0;
                o0[u] = has_edges ? (int64_t)offsets[vv] : 0;             // no edges: no vertex has a row to read
                deg[u] = has_edges ? (int64_t)offsets[vv + 1] - o0[u] : 0;
                if (v[u] < 0) deg[u] = 0;
            }
            int32_t child[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                uint64_t x = finalise64((keyed ^ (((uint64_t)(uint32_t)root << 32) | (uint32_t)v[u])) +
                                        0x9E3779B97F4A7C15ull);
                x = finalise64((x ^ (((uint64_t)(uint32_t)h << 32) | j[u])) + 0x9E3779B97F4A7C15ull);
                const int64_t e = deg[u] > 0 ? o0[u] + (int64_t)mod_u64(x, (uint64_t)deg[u]) : 0;
                child[u] = has_edges ? indices[e] : -1;
                if (deg[u] <= 0) child[u] = -1;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t c = c0 + u * blockDim.x;
                if (c >= (uint32_t)P) continue;
                children[c] = child[u];
                if (present != nullptr && child[u] >= 0) present[child[u]] = 1;
                if (slot_idx != nullptr && h < sh.n_layers) {   // non-leaf child: its own row in later layers
                    const int32_t slot = sh.base[h] + m * P + (int32_t)c;
                    slot_idx[slot - B] = child[u] >= 0 ? slot : -1;
                }
                if (indptr != nullptr && j[u] == 0)
                    indptr[sh.base[h - 1] + m * sh.P[h - 1] + (int32_t)q[u]] =
                        sh.base[h] + (m * sh.P[h - 1] + (int32_t)q[u]) * (int32_t)f - B;
            }
        }
        };
        // a level no wider than the workgroup has one slot per thread: nothing to batch
        if ((uint32_t)P > blockDim.x) level(std::integral_constant<int, kSampleUnroll>{});
        else level(std::integral_constant<int, 1>{});
        __syncthreads();   // this level is visible to the whole workgroup before the next hop
    }
}

// The same micrographs with every level's parents taken once each.  Equal vertices on one level of a
// micrograph draw the same children (the draws depend on key, root, vertex, hop and draw only), and with
// replacement on skewed graphs most slots are such repeats: of the parents of the last hop 17 to 53 % are
// distinct on power-law graphs, 66 to 78 % on uniform ones.  Per level:
//   A  one thread per distinct parent: its row bounds, the reciprocal of its degree and the first hash round
//   B  one thread per draw of a distinct parent: the second hash round, the remainder by a multiply-high with
//      that reciprocal (exact, below), one neighbour read, the mark
//   C  every slot copies its parent's draw out of LDS; a non-leaf level is then reduced to its distinct vertices
//      (LDS hash table, the first slot of a vertex stands for it, distinct vertices numbered in slot order)
// so that a slot costs an LDS read and its stores where it cost three loads, two hash rounds and a 64-bit remainder.
// floor(x M / 2^64) with M = floor((2^64 - 1) / d) is floor(x / d) or one less: x M / 2^64 > x / d - 1.
// The level lives in LDS throughout; the host takes this kernel where it fits (see lds_shape).
struct DrawParent {
    uint64_t first, degree, recip, hashed;      // row start, row length, M, first hash round
};

struct LdsShape {
    int32_t n_parents;      // capacity: slots of the widest non-leaf level
    int32_t table_mask;     // entries of the hash table - 1 (a power of two, at least twice n_parents)
    int32_t draws_off, vert_off, rank_off, key_off, first_off;      // byte offsets behind the parents
    int32_t bytes;
    uint32_t f_magic[kMaxLayers + 1];      // c / f[h] = __umulhi(c, f_magic[h]) for c < 2^16; 0 for f[h] = 1
};

// Where it pays: with thousands of micrographs the chip is full of workgroups that wait for the graph (page
// translations of random reads, 10 to 13 G/s), and what counts is how few reads they make and how many workgroups are
// resident: two wavefronts (256 threads leave most lanes idle between the barriers of short levels).  With fewer
// micrographs one workgroup's chain of reads is the whole time, and a thread per slot, no barriers between, is shorter.
// us, sampling call alone, slot by slot / this with 256 / 128 / 64 threads:
//   16384 x 10,10,10 (chung_lu, 20 M vertices)   128 / 125 / 95 / 94      4096 x 10,10,10 (100 M)   35 / 33 / 30 / 31
//    4096 x 25,10 (rmat, 16 M)                    13.5 / 16.0 / 12.8 / 11.3     1024 x 15,10,5 (2.4 M)   11.9 / 13.3 / 15.6 / 18.9
// (with marks, 4096 x 10,10,10: 63 / 53; 3296 x 12,16 on a uniform graph of degree 27, 0.7 M slots, whole fetch: 50.1 / 52.1).
// A caller that wants the distinct vertices takes it at any size.
constexpr int kLdsMaxParents = 512, kLdsMaxDraws = 4096, kLdsMinMicrographs = 2048;
constexpr int64_t kLdsMinSlots = 2000000;

template <typename OffT, int NT>
__global__ void __launch_bounds__(NT)
sample_micrographs_lds(const OffT* __restrict__ offsets, const int32_t* __restrict__ indices,
                       const int32_t* __restrict__ seeds, int32_t n_seeds, SampleShape sh, LdsShape ls, BatchKeys keys,
                       int32_t* __restrict__ ids, int32_t* __restrict__ indptr, int32_t* __restrict__ slot_idx,
                       int64_t slot_idx_stride, uint8_t* __restrict__ present, int32_t m_offset, int32_t seeds_per_key,
                       int32_t has_edges, DistinctOut distinct) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
    constexpr int kLdsRounds = kLdsMaxParents / NT, WAVES = NT / kWave;
    __shared__ int32_t wave_reps[kLdsRounds][WAVES];
    DrawParent* parent = reinterpret_cast<DrawParent*>(lds_raw);
    int32_t* draws = reinterpret_cast<int32_t*>(lds_raw + ls.draws_off);      // [distinct parents][f]
    int32_t* vert = reinterpret_cast<int32_t*>(lds_raw + ls.vert_off);        // distinct parents
    uint16_t* rank = reinterpret_cast<uint16_t*>(lds_raw + ls.rank_off);      // parent slot -> distinct parent
    int32_t* key = reinterpret_cast<int32_t*>(lds_raw + ls.key_off);
    int32_t* first = reinterpret_cast<int32_t*>(lds_raw + ls.first_off);      // first slot of the key, then its number
    constexpr uint16_t kNone = 0xFFFF;

    const int32_t m = m_offset + (int32_t)blockIdx.x;
    const int32_t B = n_seeds;
    const uint32_t batch = blockIdx.y;
    const uint64_t keyed = keys.keyed[batch + blockIdx.x / (uint32_t)seeds_per_key];
    seeds += (int64_t)batch * B;
    ids += (int64_t)batch * sh.base[sh.n_layers + 1];
    if (slot_idx != nullptr) slot_idx += (int64_t)batch * slot_idx_stride;
    if (batch != 0) indptr = nullptr;      // the segment offsets are the same for every batch of one shape
    const int32_t root = seeds[m];
    const int64_t mic = (int64_t)batch * B + m;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    if (tid == 0) {
        ids[m] = root;
        if (present != nullptr && root >= 0) present[root] = 1;   // the pre-gather's presence map
        if (indptr != nullptr && m == 0) indptr[sh.base[sh.n_layers]] = sh.base[sh.n_layers + 1] - B;
        vert[0] = root;
        rank[0] = root >= 0 ? (uint16_t)0 : kNone;
    }
    int32_t n_distinct = root >= 0 ? 1 : 0;
    __syncthreads();
    for (int32_t h = 1; h <= sh.n_layers; ++h) {
        const int32_t f = sh.f[h], P = sh.P[h];
        const uint32_t magic = ls.f_magic[h];
        auto over_f = [&](int32_t c) -> int32_t { return f == 1 ? c : (int32_t)__umulhi((uint32_t)c, magic); };
        // A
        for (int32_t i = tid; i < n_distinct; i += NT) {
            const int32_t v = vert[i];
            DrawParent p;
            p.first = has_edges ? (uint64_t)offsets[v] : 0u;             // no edges: no vertex has a row to read
            const uint64_t end = has_edges ? (uint64_t)offsets[(int64_t)v + 1] : 0u;
            p.hashed = finalise64((keyed ^ (((uint64_t)(uint32_t)root << 32) | (uint32_t)v)) + 0x9E3779B97F4A7C15ull);
            p.degree = (int64_t)end > (int64_t)p.first ? end - p.first : 0u;
            p.recip = p.degree > 0 ? ~0ull / p.degree : 0u;
            parent[i] = p;
        }
        const bool leaf = h == sh.n_layers;
        __syncthreads();
        if (!leaf)      // (behind the barrier: the level before may have been reading its numbers up to there)
            for (int32_t i = tid; i <= ls.table_mask; i += NT) {
                key[i] = -1;
                first[i] = 0x7FFFFFFF;
            }
        // B: several draws per thread side by side, unconditional reads from in-bounds addresses
        const int32_t n_draws = n_distinct * f;
        auto draw = [&](auto unroll) {
            constexpr int U = decltype(unroll)::value;
            for (int32_t t0 = tid; t0 < n_draws; t0 += NT * U) {
                int32_t child[U];
                bool some[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int32_t t = t0 + u * NT < n_draws ? t0 + u * NT : t0;
                    const int32_t q = over_f(t), j = t - q * f;
                    const DrawParent p = parent[q];
                    const uint64_t x = finalise64((p.hashed ^ (((uint64_t)(uint32_t)h << 32) | (uint32_t)j)) + 0x9E3779B97F4A7C15ull);
                    uint64_t r = x - __umul64hi(x, p.recip) * p.degree;
                    r = r >= p.degree ? r - p.degree : r;
                    some[u] = p.degree > 0;
                    child[u] = has_edges ? indices[some[u] ? p.first + r : 0u] : -1;
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int32_t t = t0 + u * NT;
                    if (t >= n_draws) continue;
                    if (!some[u]) child[u] = -1;
                    draws[t] = child[u];
                    if (present != nullptr && child[u] >= 0) present[child[u]] = 1;
                }
            }
        };
        if (n_draws > NT) draw(std::integral_constant<int, kSampleUnroll>{});
        else draw(std::integral_constant<int, 1>{});
        __syncthreads();
        // C
        int32_t* children = ids + sh.base[h] + (int64_t)m * P;
        const int32_t slot0 = sh.base[h] + m * P, parent0 = sh.base[h - 1] + m * sh.P[h - 1];
        int32_t q = over_f(tid), j = tid - q * f;      // slot c = q f + j; c advances by NT from call to call
        const int32_t dq = over_f(NT), dj = NT - dq * f;
        auto copy_out = [&](int32_t c) -> int32_t {
            const int32_t i = rank[q];
            const int32_t child = i != kNone ? draws[i * f + j] : -1;
            children[c] = child;
            if (slot_idx != nullptr && !leaf) slot_idx[slot0 + c - B] = child >= 0 ? slot0 + c : -1;   // its own row in later layers
            if (indptr != nullptr && j == 0) indptr[parent0 + q] = slot0 + c - B;
            j += dj;
            q += dq;
            if (j >= f) {
                j -= f;
                ++q;
            }
            return child;
        };
        if (leaf) {
            for (int32_t c = tid; c < P; c += NT) copy_out(c);
            break;
        }
        int32_t child[kLdsRounds], at[kLdsRounds];
#pragma unroll
        for (int u = 0; u < kLdsRounds; ++u) {
            child[u] = -1;
            at[u] = 0;
            if (u * NT >= P) continue;        // uniform, as below
            const int32_t c = u * NT + tid;
            if (c < P) child[u] = copy_out(c);
            if (child[u] >= 0) {
                uint32_t s = ((uint32_t)child[u] * 2654435761u) >> 16;
                for (;; ++s) {                // at most half of the entries are ever taken
                    s &= (uint32_t)ls.table_mask;
                    const int32_t was = atomicCAS(&key[s], -1, child[u]);
                    if (was == -1 || was == child[u]) break;
                }
                at[u] = (int32_t)s;
                atomicMin(&first[s], c);
            }
        }
        __syncthreads();
        uint64_t reps[kLdsRounds];
#pragma unroll
        for (int u = 0; u < kLdsRounds; ++u) {
            if (u * NT >= P) continue;
            reps[u] = __ballot(child[u] >= 0 && first[at[u]] == u * NT + tid);
            if (lane == 0) wave_reps[u][wave] = __popcll(reps[u]);
        }
        __syncthreads();
        int32_t before = 0;
#pragma unroll
        for (int u = 0; u < kLdsRounds; ++u) {
            if (u * NT >= P) continue;
            int32_t mine = before;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                if (w < wave) mine += wave_reps[u][w];
                before += wave_reps[u][w];
            }
            if ((reps[u] >> lane) & 1ull) {
                const int32_t n = mine + __popcll(reps[u] & ((1ull << lane) - 1ull));
                vert[n] = child[u];
                first[at[u]] = n;
                if (distinct.rank[h] != nullptr) distinct.slot[h][mic * P + n] = (uint16_t)(u * NT + tid);
            }
        }
        n_distinct = before;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kLdsRounds; ++u) {
            const int32_t c = u * NT + tid;
            if (c >= P) continue;
            rank[c] = child[u] >= 0 ? (uint16_t)first[at[u]] : kNone;
            if (distinct.rank[h] != nullptr) distinct.rank[h][mic * P + c] = rank[c];
        }
        if (distinct.rank[h] != nullptr && tid == 0) distinct.count[h][mic] = n_distinct;
        // (the next level's first barrier stands between these writes and their readers)
    }
}

static uint64_t host_finalise64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// LDS of sample_micrographs_lds for this shape, or false where a level does not fit: more than 512 slots on the widest
// non-leaf level (four rounds of the workgroup, their state in registers) or more than 4096 leaves (16 KB; a larger
// level leaves too few workgroups on a CU to hide its reads): the kernel above takes those.
static bool lds_shape(const SampleShape& sh, LdsShape& ls) {
    const int32_t L = sh.n_layers;
    if (sh.P[L - 1] > kLdsMaxParents || sh.P[L] > kLdsMaxDraws) return false;
    ls = LdsShape{};
    ls.n_parents = sh.P[L - 1];
    int32_t entries = 64;
    while (entries < 2 * ls.n_parents) entries *= 2;
    ls.table_mask = entries - 1;
    int32_t o = ls.n_parents * (int32_t)sizeof(DrawParent);
    ls.vert_off = o;
    o += ls.n_parents * 4;
    // the leaves' draws lie where the hash table was (which stands behind the draws of the levels that need it)
    ls.draws_off = o;
    ls.key_off = o + ls.n_parents * 4;
    ls.first_off = ls.key_off + entries * 4;
    const int32_t table_end = L > 1 ? ls.first_off + entries * 4 : o, draws_end = o + sh.P[L] * 4;
    o = table_end > draws_end ? table_end : draws_end;
    ls.rank_off = o;
    o += ls.n_parents * 2;
    ls.bytes = o;
    for (int32_t h = 1; h <= L; ++h) ls.f_magic[h] = sh.f[h] > 1 ? (uint32_t)((((uint64_t)1 << 32) + sh.f[h] - 1) / sh.f[h]) : 0u;
    return true;
}

template <typename OffT>
static void launch_sample(dim3 grid, int threads, hipStream_t s, const hopgnn_csr* g, const int32_t* seeds, int32_t n_seeds,
                          const SampleShape& sh, const BatchKeys& keys, int32_t* ids, int32_t* indptr, int32_t* slot_idx,
                          int64_t slot_idx_stride, uint8_t* present, int32_t m_offset, int32_t seeds_per_key,
                          const DistinctOut& distinct) {
    const OffT* offsets = static_cast<const OffT*>(g->offsets);
    const int32_t has_edges = g->n_edges > 0 ? 1 : 0;
    LdsShape ls;
    const bool many = (int64_t)grid.x * grid.y >= kLdsMinMicrographs;
    const bool large = many && (int64_t)grid.x * grid.y * (sh.base[sh.n_layers + 1] / n_seeds) >= kLdsMinSlots;
    if ((large || distinct.rank[sh.n_layers - 1] != nullptr) && lds_shape(sh, ls))
        hipLaunchKernelGGL((many ? sample_micrographs_lds<OffT, 128> : sample_micrographs_lds<OffT, 256>), grid,
                           dim3(many ? 128 : 256), ls.bytes, s, offsets, g->indices, seeds, n_seeds, sh, ls, keys, ids, indptr,
                           slot_idx, slot_idx_stride, present, m_offset, seeds_per_key, has_edges, distinct);
    else
        hipLaunchKernelGGL(sample_micrographs<OffT>, grid, dim3(threads), 0, s, offsets, g->indices, seeds, n_seeds, sh, keys,
                           ids, indptr, slot_idx, slot_idx_stride, present, m_offset, seeds_per_key, has_edges);
}

}  // namespace hopgnn

using namespace hopgnn;

extern "C" int64_t hopgnn_slots_per_seed(const int32_t* fanouts, int32_t n_layers) {
    if (fanouts == nullptr || n_layers < 1 || n_layers > kMaxLayers) return -1;
    int64_t p = 1, t = 1;
    for (int32_t h = 0; h < n_layers; ++h) {
        if (fanouts[h] < 1) return -1;
        p *= fanouts[h];
        if (p > (int64_t)1 << 31) return -1;
        t += p;
    }
    return t;
}

namespace hopgnn {

bool sample_gives_distinct(const int32_t* fanouts, int32_t n_layers) {
    if (n_layers < 2 || n_layers > kMaxLayers || hopgnn_slots_per_seed(fanouts, n_layers) < 0) return false;
    SampleShape sh{};
    sh.n_layers = n_layers;
    sh.P[0] = 1;
    for (int32_t h = 1; h <= n_layers; ++h) {
        sh.f[h] = fanouts[h - 1];
        sh.P[h] = sh.P[h - 1] * sh.f[h];
    }
    LdsShape ls;
    return lds_shape(sh, ls);
}

hopgnn_status sample_batches(const hopgnn_csr* g, const int32_t* seeds, int32_t n_seeds, const int32_t* fanouts,
                             int32_t n_layers, const uint64_t* keys, int32_t n_batches, int32_t* ids, int32_t* indptr,
                             int32_t* slot_idx, int64_t slot_idx_stride, uint8_t* present, void* stream,
                             const DistinctOut& distinct) {
    if (g == nullptr || fanouts == nullptr || n_seeds < 0 || n_batches < 0) return HOPGNN_EINVAL;
    const int64_t t_seed = hopgnn_slots_per_seed(fanouts, n_layers);
    if (t_seed < 0) return HOPGNN_EINVAL;
    if (g->n_vertices < 0 || g->n_edges < 0 || g->n_vertices > ((int64_t)1 << 31)) return HOPGNN_EINVAL;
    if (n_seeds == 0 || n_batches == 0) return HOPGNN_OK;
    if (g->offsets == nullptr || seeds == nullptr || ids == nullptr || keys == nullptr) return HOPGNN_EINVAL;
    if (g->n_edges > 0 && g->indices == nullptr) return HOPGNN_EINVAL;
    const int64_t T = (int64_t)n_seeds * t_seed;
    if (T * n_batches >= ((int64_t)1 << 31)) return HOPGNN_ERANGE;

    SampleShape sh{};
    sh.n_layers = n_layers;
    sh.P[0] = 1;
    sh.base[0] = 0;
    for (int32_t h = 1; h <= n_layers; ++h) {
        sh.f[h] = fanouts[h - 1];
        sh.P[h] = sh.P[h - 1] * sh.f[h];
        sh.base[h] = sh.base[h - 1] + n_seeds * sh.P[h - 1];
    }
    sh.base[n_layers + 1] = sh.base[n_layers] + n_seeds * sh.P[n_layers];
    if (slot_idx != nullptr && n_batches > 1 && slot_idx_stride < (int64_t)sh.base[n_layers] - n_seeds)
        return HOPGNN_EINVAL;              // the batches' neighbour lists would overlap

    int threads = 64;
    while (threads < 256 && threads < sh.P[n_layers]) threads *= 2;
    hipStream_t s = static_cast<hipStream_t>(stream);
    for (int32_t b0 = 0; b0 < n_batches; b0 += kMaxBatchesPerLaunch) {
        const int32_t nb = n_batches - b0 < kMaxBatchesPerLaunch ? n_batches - b0 : kMaxBatchesPerLaunch;
        BatchKeys bk{};
        for (int32_t i = 0; i < nb; ++i) bk.keyed[i] = host_finalise64(keys[b0 + i] + 0x9E3779B97F4A7C15ull);
        const int32_t* sd = seeds + (int64_t)b0 * n_seeds;
        int32_t* id = ids + (int64_t)b0 * T;
        int32_t* ip = b0 == 0 ? indptr : nullptr;
        int32_t* si = slot_idx != nullptr ? slot_idx + (int64_t)b0 * slot_idx_stride : nullptr;
        const dim3 grid((unsigned)n_seeds, (unsigned)nb);
        DistinctOut dn = distinct;
        for (int32_t h = 1; h < n_layers; ++h) {
            if (dn.rank[h] == nullptr) continue;
            const int64_t m0 = (int64_t)b0 * n_seeds;
            dn.rank[h] += m0 * sh.P[h];
            dn.slot[h] += m0 * sh.P[h];
            dn.count[h] += m0;
        }
        (g->offsets_i64 ? launch_sample<int64_t> : launch_sample<int32_t>)(grid, threads, s, g, sd, n_seeds, sh, bk, id, ip, si,
                                                                           slot_idx_stride, present, 0, n_seeds, dn);
        HOPGNN_LAUNCH_CHECK();
    }
    return HOPGNN_OK;
}

hopgnn_status sample_merged(const hopgnn_csr* g, const int32_t* seeds, int32_t n_seeds, int32_t seeds_per_key,
                            const int32_t* fanouts, int32_t n_layers, const uint64_t* keys, int32_t* ids,
                            int32_t* indptr, int32_t* slot_idx, uint8_t* present, void* stream,
                            const DistinctOut& distinct) {
    if (g == nullptr || fanouts == nullptr || n_seeds < 0 || seeds_per_key < 1) return HOPGNN_EINVAL;
    const int64_t t_seed = hopgnn_slots_per_seed(fanouts, n_layers);
    if (t_seed < 0) return HOPGNN_EINVAL;
    if (g->n_vertices < 0 || g->n_edges < 0 || g->n_vertices > ((int64_t)1 << 31)) return HOPGNN_EINVAL;
    if (n_seeds == 0) return HOPGNN_OK;
    if (g->offsets == nullptr || seeds == nullptr || ids == nullptr || keys == nullptr) return HOPGNN_EINVAL;
    if (g->n_edges > 0 && g->indices == nullptr) return HOPGNN_EINVAL;
    if ((int64_t)n_seeds * t_seed >= ((int64_t)1 << 31)) return HOPGNN_ERANGE;

    SampleShape sh{};
    sh.n_layers = n_layers;
    sh.P[0] = 1;
    sh.base[0] = 0;
    for (int32_t h = 1; h <= n_layers; ++h) {
        sh.f[h] = fanouts[h - 1];
        sh.P[h] = sh.P[h - 1] * sh.f[h];
        sh.base[h] = sh.base[h - 1] + n_seeds * sh.P[h - 1];
    }
    sh.base[n_layers + 1] = sh.base[n_layers] + n_seeds * sh.P[n_layers];
    int threads = 64;
    while (threads < 256 && threads < sh.P[n_layers]) threads *= 2;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int32_t n_keys = (int32_t)ceil_div(n_seeds, seeds_per_key);
    for (int32_t k0 = 0; k0 < n_keys; k0 += kMaxBatchesPerLaunch) {     // 64 keys fit one launch's arguments
        const int32_t nk = n_keys - k0 < kMaxBatchesPerLaunch ? n_keys - k0 : kMaxBatchesPerLaunch;
        BatchKeys bk{};
        for (int32_t i = 0; i < nk; ++i) bk.keyed[i] = host_finalise64(keys[k0 + i] + 0x9E3779B97F4A7C15ull);
        const int64_t m0 = (int64_t)k0 * seeds_per_key;
        const int64_t count = (int64_t)nk * seeds_per_key < n_seeds - m0 ? (int64_t)nk * seeds_per_key : n_seeds - m0;
        const dim3 grid((unsigned)count, 1u);
        (g->offsets_i64 ? launch_sample<int64_t> : launch_sample<int32_t>)(grid, threads, s, g, seeds, n_seeds, sh, bk, ids, indptr,
                                                                           slot_idx, 0, present, (int32_t)m0, seeds_per_key, distinct);
        HOPGNN_LAUNCH_CHECK();
    }
    return HOPGNN_OK;
}

}  // namespace hopgnn

extern "C" hopgnn_status hopgnn_sample_merged(const hopgnn_csr* g, const int32_t* seeds, int32_t n_seeds,
                                              int32_t seeds_per_key, const int32_t* fanouts, int32_t n_layers,
                                              const uint64_t* keys, int32_t* ids, int32_t* indptr, int32_t* slot_idx,
                                              void* stream) {
    return sample_merged(g, seeds, n_seeds, seeds_per_key, fanouts, n_layers, keys, ids, indptr, slot_idx, nullptr,
                         stream);
}

extern "C" hopgnn_status hopgnn_sample(const hopgnn_csr* g, const int32_t* seeds, int32_t n_seeds,
                                       const int32_t* fanouts, int32_t n_layers, uint64_t key,
                                       int32_t* ids, int32_t* indptr, int32_t* slot_idx,
                                       void* stream) {
    return sample_batches(g, seeds, n_seeds, fanouts, n_layers, &key, 1, ids, indptr, slot_idx, 0, nullptr, stream);
}

extern "C" hopgnn_status hopgnn_sample_group(const hopgnn_csr* g, const int32_t* seeds, int32_t n_seeds,
                                             const int32_t* fanouts, int32_t n_layers, const uint64_t* keys,
                                             int32_t n_batches, int32_t* ids, int32_t* indptr, int32_t* slot_idx,
                                             int64_t slot_idx_stride, void* stream) {
    return sample_batches(g, seeds, n_seeds, fanouts, n_layers, keys, n_batches, ids, indptr, slot_idx, slot_idx_stride,
                          nullptr, stream);
}

extern "C" const char* hopgnn_status_str(hopgnn_status s) {
    switch (s) {
        case HOPGNN_OK: return "ok";
        case HOPGNN_EINVAL: return "invalid argument";
        case HOPGNN_ENOMEM_WS: return "workspace too small";
        case HOPGNN_ERANGE: return "size out of range";
        case HOPGNN_EHIP: return "HIP launch failed";
    }
    return "unknown status";
}
