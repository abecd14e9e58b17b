// Group-shared rewiring of the supports (Alg. 3), the discrete phase of training:
//   1. score each (group k, slot j) by the |w| of the group's labels at that slot (fp32 sum over
//      the G labels in order: the algorithm's mean divides every score by the same G);
//   2. prune the m = floor(K F rho) smallest scores over all groups, ties to the lower flat index;
//   3. give each pruned slot a feature drawn uniformly from those its group does not keep (slots
//      in ascending order, each draw excluding the earlier ones), then re-sort the row, carrying
//      every slot's weight column (and velocity) with it;
//   4. reinitialise the pruned slots' weights: zero, or uniform in [-1/sqrt(F), 1/sqrt(F)].
// Draws come from SplitMix64 (Steele, Lea and Flood, 2014) in counter form: draw k F + j for the
// new feature of slot j of group k, draw K F + l F + j for label l's new weight at slot j.
#include "common.hpp"

namespace {

__device__ __forceinline__ uint64_t splitmix64_at(uint64_t s, uint64_t i) {
    uint64_t z = s + (i + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Selection state of the radix select: the prefix of the threshold's key found so far, the bits it
// covers, the rank of the wanted key among the keys that share the prefix, the number of blocks that
// have added their counts, and whether every key equal to the threshold is pruned.
struct RwState {
    uint32_t prefix, pmask;
    uint64_t rank;
    uint32_t done, all;
};

__global__ void k_rw_init(uint32_t *__restrict__ hist, RwState *__restrict__ st, uint64_t rank) {
    const int t = threadIdx.x;
    if (t < 256) hist[t] = 0u;
    if (t == 0) *st = RwState{0u, 0u, rank, 0u, 0u};
}

// Digit counts of one workgroup in LDS: 16 copies, by lane, at an odd stride, because the keys of
// trained weights share one or two values of their leading digit and a wave's 64 additions to one
// counter are served one after the other.
constexpr int kRwRep = 16, kRwRepStride = 257;

__device__ __forceinline__ void rw_clear(uint32_t *h) {
    for (int i = threadIdx.x; i < kRwRep * kRwRepStride; i += blockDim.x) h[i] = 0u;
    __syncthreads();
}

// Adds the workgroup's counts to the digit's histogram; the last workgroup to do so picks the digit
// whose cumulative count passes the wanted rank and clears the histogram for the next pass.  What
// crosses workgroups goes through device-scope atomics alone, each done (its old value is back)
// before the workgroup's barrier and so before its addition to st->done: no fence, which would write
// back the L2 with the keys just stored (one per workgroup: 690 us for the score pass).
__device__ void rw_pick(const uint32_t *h, uint32_t *hist, RwState *st, int shift) {
    __shared__ uint32_t scan[256];
    __shared__ bool last;
    const int t = threadIdx.x;   // 256 threads or more
    __syncthreads();
    uint32_t own = 0u;
    if (t < 256)
        for (int r = 0; r < kRwRep; ++r) own += h[r * kRwRepStride + t];
    const uint32_t old = own ? __hip_atomic_fetch_add(&hist[t], own, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    if (__syncthreads_or(old == 0xFFFFFFFFu)) return;   // waits for old; never taken (fewer than 2^31 keys)
    if (t == 0)
        last = __hip_atomic_fetch_add(&st->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    __syncthreads();
    if (!last) return;   // workgroup-uniform
    uint32_t n = 0u;
    if (t < 256) {
        n = __hip_atomic_load(&hist[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&hist[t], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        scan[t] = n;
    }
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const uint32_t a = t >= off && t < 256 ? scan[t - off] : 0u;
        __syncthreads();
        if (t < 256) scan[t] += a;
        __syncthreads();
    }
    const uint64_t rank = st->rank, upto = t < 256 ? scan[t] : 0u, before = upto - n;   // (fewer than 2^31 keys)
    __syncthreads();
    if (before <= rank && rank < upto) {   // one thread
        st->prefix |= (uint32_t)t << shift;
        st->pmask |= 255u << shift;
        st->rank = rank - before;
        st->all = rank - before + 1 == n ? 1u : 0u;
        st->done = 0u;
    }
}

// keys[k F + j] = bits of the fp32 sum over the group's labels of |W[l, j]| (non-negative, so the
// bit patterns order as the values), and the count of their leading digit.  NE neighbouring slots
// per thread, read together (NE divides F and W is 16-byte aligned): the pass is
// bound by memory (2.9M x 64: 101 to 118 us with 2 bytes, 8 bytes or 16 a load, the leading digit's
// count included; that count took 53 us in a pass of its own, the scores 88).
template <typename T, int NE>
__global__ __launch_bounds__(256) void k_rw_scores(const T *__restrict__ W, int64_t K, int G, int F,
                                                   uint32_t *__restrict__ keys, uint32_t *__restrict__ hist,
                                                   RwState *__restrict__ st) {
    typedef T Vec __attribute__((ext_vector_type(NE)));
    __shared__ uint32_t h[kRwRep * kRwRepStride];
    rw_clear(h);
    uint32_t *mine = h + (threadIdx.x & (kRwRep - 1)) * kRwRepStride;
    for (int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * NE; i < K * F;
         i += (int64_t)gridDim.x * blockDim.x * NE) {
        const int64_t k = (uint32_t)i / (uint32_t)F;   // K F < 2^29
        const int j = (int)(i - k * F);
        // the labels' weights 8 at a time, all 8 loads in flight before they are summed in order
        float s[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e) s[e] = 0.0f;
        const T *w = W + k * G * F + j;
        auto load = [&](int g) { return *reinterpret_cast<const Vec *>(w + (int64_t)g * F); };
        auto add = [&](Vec v) {
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                const T x = v[e];
                s[e] += fabsf(load_f32(&x, 0));
            }
        };
        int g = 0;
        for (; g + 8 <= G; g += 8) {
            Vec v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = load(g + u);
#pragma unroll
            for (int u = 0; u < 8; ++u) add(v[u]);
        }
        for (; g < G; ++g) add(load(g));
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const uint32_t key = __float_as_uint(s[e]);
            keys[i + e] = key;
            atomicAdd(&mine[key >> 24], 1u);
        }
    }
    rw_pick(h, hist, st, 24);
}

// histogram of the next 8-bit digit (at `shift`) of the keys that share the current prefix
__global__ __launch_bounds__(1024) void k_rw_hist(const uint32_t *__restrict__ keys, int64_t n,
                                                 RwState *__restrict__ st, int shift, uint32_t *__restrict__ hist) {
    __shared__ uint32_t h[kRwRep * kRwRepStride];
    rw_clear(h);
    uint32_t *mine = h + (threadIdx.x & (kRwRep - 1)) * kRwRepStride;
    const uint32_t prefix = st->prefix, pmask = st->pmask;
    // four keys per 16-byte load, four loads in flight per thread (the keys array is 256-byte
    // aligned); the last n mod 4 keys one by one
    const uint4 *k4 = reinterpret_cast<const uint4 *>(keys);
    const int64_t n4 = n / 4, stride = (int64_t)gridDim.x * blockDim.x;
    auto count = [&](uint32_t key) {
        if ((key & pmask) == prefix) atomicAdd(&mine[(key >> shift) & 255u], 1u);
    };
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += 4 * stride) {
        uint4 v[4];
        bool ok[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            ok[u] = i + u * stride < n4;
            v[u] = ok[u] ? k4[i + u * stride] : make_uint4(0u, 0u, 0u, 0u);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (ok[u]) {
                count(v[u].x);
                count(v[u].y);
                count(v[u].z);
                count(v[u].w);
            }
    }
    if (blockIdx.x == 0 && threadIdx.x < n - 4 * n4) count(keys[4 * n4 + threadIdx.x]);
    rw_pick(h, hist, st, shift);
}

constexpr int kRwBlock = 1024;   // keys per block of the tie count (256 threads x 4)

// number of keys equal to the threshold per block of kRwBlock keys (nothing reads it where every
// such key is pruned)
__global__ __launch_bounds__(256) void k_rw_eqcount(const uint32_t *__restrict__ keys, int64_t n,
                                                    const RwState *__restrict__ st, uint32_t *__restrict__ cnt) {
    __shared__ uint32_t tot;
    if (st->all) return;   // uniform
    if (threadIdx.x == 0) tot = 0u;
    __syncthreads();
    const uint32_t T = st->prefix;
    const int64_t i0 = (int64_t)blockIdx.x * kRwBlock + 4 * threadIdx.x;
    uint32_t c = 0;
    for (int e = 0; e < 4; ++e) c += (i0 + e < n && keys[i0 + e] == T) ? 1u : 0u;
    if (c) atomicAdd(&tot, c);
    __syncthreads();
    if (threadIdx.x == 0) cnt[blockIdx.x] = tot;
}

// exclusive prefix of the per-block counts, in block order (one workgroup of 1024 threads): each
// thread sums a contiguous run of counts, one scan of the 1024 run sums, then each thread writes
// its run's prefixes (integer sums: the same values in any order)
constexpr int kRwScanThreads = 1024;
__global__ __launch_bounds__(kRwScanThreads) void k_rw_scan(uint32_t *__restrict__ cnt, int64_t nb,
                                                            const RwState *__restrict__ st) {
    if (st->all) return;   // uniform
    __shared__ uint32_t part[kRwScanThreads];
    const int t = threadIdx.x;
    const int64_t per = (nb + kRwScanThreads - 1) / kRwScanThreads;
    const int64_t b = t * per, e = b + per < nb ? b + per : nb;
    uint32_t sum = 0u;
#pragma unroll 8
    for (int64_t i = b; i < e; ++i) sum += cnt[i];
    part[t] = sum;
    __syncthreads();
    for (int off = 1; off < kRwScanThreads; off <<= 1) {   // inclusive Hillis-Steele scan
        const uint32_t a = t >= off ? part[t - off] : 0u;
        __syncthreads();
        part[t] += a;
        __syncthreads();
    }
    uint32_t run = part[t] - sum;
    for (int64_t i = b; i < e; ++i) {
        const uint32_t v = cnt[i];
        cnt[i] = run;
        run += v;
    }
}

// Regrowth, one wave per group with a pruned slot.  F <= 256 slots (up to four per lane), H <= 1024
// features (one 32-bit word of the wave's used-feature bitmap per lane).
constexpr int kRwWaves = 4;
// A wave moves up to CH weights (or velocities) at a time: 1024, or 256 where a group has no more, whose
// registers leave room for more waves (172K groups of one slot: 142 us with 1024, 3 waves per SIMD).
constexpr int kRwChunk = 1024, kRwChunkSmall = 256;
constexpr int kRwMaxRows = 64;
// LDS words of a chunk: rows of F values at an odd number of words, at least one word apart
constexpr int rw_chunk_words(int ch) { return ch + 2 * kRwMaxRows; }

typedef uint32_t rw_word __attribute__((may_alias));
typedef uint16_t rw_half __attribute__((may_alias));
template <int BYTES> struct RwVec { typedef uint32_t type __attribute__((ext_vector_type(BYTES / 4))); };
template <> struct RwVec<4> { typedef uint32_t type; };
template <> struct RwVec<2> { typedef uint16_t type; };

// A chunk of whole label rows, VB bytes per lane and access (a row is a whole number of them)
template <typename T, int VB, int CH> struct RwRows {
    typedef typename RwVec<VB>::type V;
    static constexpr int kVe = VB / (int)sizeof(T), kNv = CH > 64 * kVe ? CH / (64 * kVe) : 1;
    V v[kNv];

    static __device__ __forceinline__ int stride_words(int F) { return ((F * (int)sizeof(T) + 3) / 4 + 1) | 1; }

    __device__ __forceinline__ void load(const T *p, int n, int lane) {
#pragma unroll
        for (int i = 0; i < kNv; ++i) {
            const int e = kVe * (lane + 64 * i);
            if (e < n) v[i] = *reinterpret_cast<const V *>(p + e);
        }
    }
    __device__ __forceinline__ void put(uint32_t *lds, int n, int F, uint32_t magic, int lane) const {
        const int sw = stride_words(F);
#pragma unroll
        for (int i = 0; i < kNv; ++i) {
            const int e = kVe * (lane + 64 * i);
            if (e >= n) continue;
            const int row = (int)((uint32_t)e * magic >> 20), pos = e - row * F;
            if constexpr (VB == 2) {
                reinterpret_cast<rw_half *>(lds + row * sw)[pos] = v[i];
            } else if constexpr (VB == 4) {
                reinterpret_cast<rw_word *>(lds + row * sw)[pos * (int)sizeof(T) / 4] = v[i];
            } else {
#pragma unroll
                for (int u = 0; u < VB / 4; ++u)
                    reinterpret_cast<rw_word *>(lds + row * sw)[pos * (int)sizeof(T) / 4 + u] = v[i][u];
            }
        }
    }
    // the value of row `row`, slot j
    static __device__ __forceinline__ void set(uint32_t *lds, int F, int row, int j, float x) {
        if constexpr (sizeof(T) == 2) reinterpret_cast<rw_half *>(lds + row * stride_words(F))[j] = f32_to_bf16(x);
        else reinterpret_cast<rw_word *>(lds + row * stride_words(F))[j] = __float_as_uint(x);
    }
    // position p of each row takes slot src[p]
    static __device__ __forceinline__ void store(const uint32_t *lds, const uint16_t *src, T *p, int n, int F,
                                                 uint32_t magic, int lane) {
        const int sw = stride_words(F);
#pragma unroll
        for (int i = 0; i < kNv; ++i) {
            const int e = kVe * (lane + 64 * i);
            if (e >= n) continue;
            const int row = (int)((uint32_t)e * magic >> 20), pos = e - row * F;
            uint32_t x[kVe];
#pragma unroll
            for (int u = 0; u < kVe; ++u) {
                const int j = src[pos + u];
                if constexpr (sizeof(T) == 2) x[u] = reinterpret_cast<const rw_half *>(lds + row * sw)[j];
                else x[u] = reinterpret_cast<const rw_word *>(lds + row * sw)[j];
            }
            V o;
            if constexpr (VB == 2) {
                o = (uint16_t)x[0];
            } else if constexpr (VB == 4) {
                if constexpr (sizeof(T) == 2) o = x[0] | x[1] << 16;
                else o = x[0];
            } else {
#pragma unroll
                for (int u = 0; u < VB / 4; ++u) {
                    if constexpr (sizeof(T) == 2) o[u] = x[2 * u] | x[2 * u + 1] << 16;
                    else o[u] = x[u];
                }
            }
            *reinterpret_cast<V *>(p + e) = o;
        }
    }
};

// Bound by memory: the weights and velocities of nearly every group move once.  A group's first
// chunk of both is requested before the draws, which are a serial chain of about 20 instructions
// each; whole chunks of rows then pass through LDS in the widest accesses that the rows allow, the
// pruned slots' new values written there by dense lanes.  (One row at a time, each a load, an LDS
// write, a gather and a store that waited for each other, and draws of 45 instructions: 727 us at
// 2.9M labels x 64, rho 0.1, of 2.26 GB moved; 410 here, 5.5 TB/s.)
//
// A slot is pruned if its key is below the threshold, or equal to it and among the first need keys
// that are: cnt holds the equal keys before each block of kRwBlock, and the wave counts those between
// its block's start and its slots (only where not all of them are pruned).
//
// NPL: 64-slot words of a support (F <= 64 NPL); VB, VM: bytes per access of W and of the velocity
template <typename T, int NPL, int VB, int VM, int CH>
__global__ __launch_bounds__(64 * kRwWaves) void k_rw_regrow(int32_t *__restrict__ idx, T *__restrict__ W,
                                                             float *__restrict__ mom, const uint32_t *__restrict__ keys,
                                                             const RwState *__restrict__ st,
                                                             const uint32_t *__restrict__ cnt, int64_t K, int G, int F,
                                                             int H, int init_random, uint64_t seed, float scale,
                                                             uint32_t fmagic) {
    __shared__ uint32_t used_s[kRwWaves][32];
    __shared__ uint32_t upre_s[kRwWaves][32];
    __shared__ int32_t feat_s[kRwWaves][64 * NPL];
    __shared__ __align__(16) uint16_t src_s[kRwWaves][64 * NPL];
    __shared__ uint16_t pl_s[kRwWaves][64 * NPL];
    __shared__ uint32_t rows_s[kRwWaves][rw_chunk_words(CH)];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t k = (int64_t)blockIdx.x * kRwWaves + wv;
    if (k >= K) return;   // wave-uniform; this kernel has no workgroup barrier
    uint32_t *used = used_s[wv], *upre = upre_s[wv], *rows = rows_s[wv];
    int32_t *feat = feat_s[wv];
    uint16_t *src = src_s[wv], *pl = pl_s[wv];
    const int64_t KF = K * F;
    constexpr int NPW = NPL;

    // the group's slots and their marks as one 64-bit ballot per 64 slots
    used[lane & 31] = 0u;
    uint64_t pm[NPW];
    int32_t ft[NPW];
    int n_pruned = 0;
    const uint32_t T0 = st->prefix;
    const bool all = st->all != 0u;
    const uint64_t need = st->rank + 1;   // the wanted key is the rank-th (0-based) among those equal
    bool tie = false;
#pragma unroll
    for (int w = 0; w < NPW; ++w) {
        const int j = lane + 64 * w;
        const uint32_t key = j < F ? keys[k * F + j] : 0xFFFFFFFFu;
        ft[w] = j < F ? idx[k * F + j] : 0;
        pm[w] = __builtin_amdgcn_ballot_w64(j < F && (key < T0 || (all && key == T0)));
        tie |= j < F && key == T0;
    }
    if (!all && __builtin_amdgcn_ballot_w64(tie) != 0u) {   // wave-uniform
        const int64_t b0 = k * F / kRwBlock * kRwBlock;
        uint64_t before = cnt[k * F / kRwBlock];
        for (int64_t i = b0; i < k * F; i += 64)
            before += __popcll(__builtin_amdgcn_ballot_w64(i + lane < k * F && keys[i + lane] == T0));
        // a support may cross into later blocks: the running count goes on over its own slots
#pragma unroll
        for (int w = 0; w < NPW; ++w) {
            const int j = lane + 64 * w;
            const bool eq = j < F && keys[k * F + j] == T0;
            const uint64_t em = __builtin_amdgcn_ballot_w64(eq);
            const uint64_t r = before + __popcll(em & ((1ull << lane) - 1ull));
            pm[w] |= __builtin_amdgcn_ballot_w64(eq && r < need);
            before += __popcll(em);
        }
    }
#pragma unroll
    for (int w = 0; w < NPW; ++w) n_pruned += __popcll(pm[w]);
    if (n_pruned == 0) return;   // wave-uniform

    // rows per chunk, at most CH values; the first chunk is on its way during the draws
    int R = (int)((CH * fmagic) >> 20);   // CH / F
    R = R < kRwMaxRows ? R : kRwMaxRows;
    R = R < G ? R : G;
    T *wg = W + k * G * F;
    float *mg = mom + k * G * F;
    RwRows<T, VB, CH> wr;
    RwRows<float, VM, CH> mr;
    wr.load(wg, R * F, lane);
    if (mom) mr.load(mg, R * F, lane);

    // the kept features, and the list of pruned slots
    int d0 = 0;   // pruned slots in earlier words
    // Draws, pruned slots in ascending order: the (r mod n_free)-th free feature, r the slot's
    // SplitMix64 value.  The d-th draw has n_free = H - (F - n_pruned) - d, so every draw's
    // r mod n_free is computed at once, on the lane of its slot; only the selection is sequential.
    // In 32-bit steps (n_free <= H <= 1024, so every product fits):
    //   r mod n = ((r_hi mod n) (2^32 mod n) + r_lo mod n) mod n.
    uint32_t tt[NPW];
#pragma unroll
    for (int w = 0; w < NPW; ++w) {
        const int j = lane + 64 * w;
        tt[w] = 0u;
        if ((pm[w] >> lane) & 1u) {
            const int d = d0 + __popcll(pm[w] & ((1ull << lane) - 1ull));
            pl[d] = (uint16_t)j;
            const uint64_t r = splitmix64_at(seed, (uint64_t)(k * F + j));
            const uint32_t nf = (uint32_t)(H - (F - n_pruned) - d);
            const uint32_t p32 = (0xFFFFFFFFu % nf + 1u) % nf;   // 2^32 mod nf
            tt[w] = ((uint32_t)(r >> 32) % nf * p32 % nf + (uint32_t)r % nf) % nf;
        } else if (j < F) {
            atomicOr(&used[ft[w] >> 5], 1u << (ft[w] & 31));
        }
        d0 += __popcll(pm[w]);
    }
    // Lane w holds the free bits of bitmap word w (words past H have none) and the inclusive
    // prefix of the free counts, scanned once; a draw removes one bit, so the lane that held it
    // and every later prefix drop by one, with no further scan.  The holder is the first lane whose
    // prefix passes t, and its word's wanted bit the set one with as many set bits below it as are
    // left to pass, which 32 lanes test at once.
    const int nw = (H + 31) >> 5;
    uint32_t freew = 0u, valid = 0u;
    if (lane < nw) {
        const int lo = 32 * lane;
        valid = H - lo >= 32 ? 0xFFFFFFFFu : ((1u << (H - lo)) - 1u);
        freew = ~used[lane] & valid;
    }
    uint32_t inc = __popc(freew);
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t a = __shfl_up(inc, off, 64);
        if (lane >= off) inc += a;
    }
    const uint32_t lanebit = lane < 32 ? 1u << lane : 0u;
#pragma unroll
    for (int w = 0; w < NPW; ++w)
        for (uint64_t rem = pm[w]; rem != 0u; rem &= rem - 1u) {
            const int sl = (int)__builtin_ctzll(rem);
            const uint32_t t = __builtin_amdgcn_readlane(tt[w], sl);
            const int holder = (int)__builtin_ctzll(__builtin_amdgcn_ballot_w64(t < inc));
            const uint32_t fw = __builtin_amdgcn_readlane(freew, holder);
            const uint32_t left = t - (__builtin_amdgcn_readlane(inc, holder) - __popc(fw));
            const int pos = (int)__builtin_ctzll(
                __builtin_amdgcn_ballot_w64((fw & lanebit) != 0u && __builtin_amdgcn_mbcnt_lo(fw, 0u) == left));
            if (lane == holder) freew &= ~(1u << pos);
            if (lane >= holder) --inc;
            if (lane == sl) ft[w] = 32 * holder + pos;
        }

    // new positions: the rank of each slot's feature among the row's features, from the final
    // bitmap (the features are distinct): used features in earlier words, plus the used bits of
    // its word below it
    {
        const uint32_t usedw = ~freew & valid;
        const uint32_t uc = __popc(usedw);
        uint32_t ui = uc;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t a = __shfl_up(ui, off, 64);
            if (lane >= off) ui += a;
        }
        if (lane < nw) {
            used[lane] = usedw;
            upre[lane] = ui - uc;
        }
    }
#pragma unroll
    for (int w = 0; w < NPW; ++w) {
        const int j = lane + 64 * w;
        if (j >= F) continue;
        const int f = ft[w];
        const int p = (int)(upre[f >> 5] + __popc(used[f >> 5] & ((1u << (f & 31)) - 1u)));
        src[p] = (uint16_t)j;
        feat[p] = f;
    }
    for (int p = lane; p < F; p += 64) idx[k * F + p] = feat[p];

    // each label's weights (and velocity) follow their slots; pruned slots are reinitialised
    const uint32_t pmagic = ((1u << 20) + (uint32_t)n_pruned - 1u) / (uint32_t)n_pruned;
    for (int g0 = 0; g0 < G; g0 += R) {
        const int nr = G - g0 < R ? G - g0 : R, n = nr * F;
        const int nx = G - g0 - nr < R ? (G - g0 - nr) * F : R * F;   // values of the next chunk
        wr.put(rows, n, F, fmagic, lane);
        if (nx > 0) wr.load(wg + (int64_t)(g0 + nr) * F, nx, lane);
        for (int e = lane; e < nr * n_pruned; e += 64) {
            const int row = (int)((uint32_t)e * pmagic >> 20), j = pl[e - row * n_pruned];
            float v = 0.0f;
            if (init_random) {
                const uint64_t r = splitmix64_at(seed, (uint64_t)(KF + (k * G + g0 + row) * F + j)) >> 40;
                v = (float)((int32_t)(2 * r) - (1 << 24)) * scale;
            }
            RwRows<T, VB, CH>::set(rows, F, row, j, v);
        }
        RwRows<T, VB, CH>::store(rows, src, wg + (int64_t)g0 * F, n, F, fmagic, lane);
        if (!mom) continue;   // uniform
        mr.put(rows, n, F, fmagic, lane);
        if (nx > 0) mr.load(mg + (int64_t)(g0 + nr) * F, nx, lane);
        for (int e = lane; e < nr * n_pruned; e += 64) {
            const int row = (int)((uint32_t)e * pmagic >> 20);
            RwRows<float, VM, CH>::set(rows, F, row, pl[e - row * n_pruned], 0.0f);
        }
        RwRows<float, VM, CH>::store(rows, src, mg + (int64_t)g0 * F, n, F, fmagic, lane);
    }
}

}  // namespace

namespace haste {

// 256 slots: four per lane of the regrowth; it addresses a group's weights (and velocity) with 32-bit offsets within its block
bool rewire_supported(const TailArgs &a) {
    return a.F_in <= 256 && a.F_s <= kMaxFs && a.G * a.F_in * 4 < ((int64_t)1 << 31);
}

static int64_t rw_blocks(const TailArgs &a) { return cdiv((a.L / a.G) * a.F_in, kRwBlock); }

size_t rewire_ws(const TailArgs &a) {
    const int64_t KF = (a.L / a.G) * a.F_in;
    return (size_t)round_up(KF * 4, 256) + (size_t)round_up(KF, 256) + (size_t)round_up(rw_blocks(a) * 4, 256) +
           256 * 4 + 256;
}

hipError_t rewire(const TailArgs &a, int32_t *idx, void *W, float *m, int64_t n_prune, int init_random, uint64_t seed,
                  void *ws, hipStream_t s) {
    const int64_t K = a.L / a.G, KF = K * a.F_in;
    char *p = static_cast<char *>(ws);
    uint32_t *keys = reinterpret_cast<uint32_t *>(p);
    p += round_up(KF * 4, 256) + round_up(KF, 256);   // (the KF bytes after the keys are not used)
    uint32_t *cnt = reinterpret_cast<uint32_t *>(p);
    p += round_up(rw_blocks(a) * 4, 256);
    uint32_t *hist = reinterpret_cast<uint32_t *>(p);
    RwState *st = reinterpret_cast<RwState *>(p + 256 * 4);
    const bool bf = a.dtype == HASTE_DTYPE_BF16;
    const int F = (int)a.F_in;
    hipLaunchKernelGGL(k_rw_init, dim3(1), dim3(256), 0, s, hist, st, (uint64_t)(n_prune - 1));
    // every workgroup adds to the same few counters, one addition after the other (2.9M x 64: digits 24 us a
    // pass with 1024 workgroups of 256 threads, 11 with 256 of 1024; scores with 2 bytes a load 300 with one
    // workgroup per 256 slots, 120 with 1024)
    auto blocks = [](int64_t want, int64_t most) { return want < most ? want : most; };
    auto scores = [&](auto tag, auto ne) {
        using T = decltype(tag);
        constexpr int NE = decltype(ne)::value;
        hipLaunchKernelGGL((k_rw_scores<T, NE>), dim3((unsigned)blocks(cdiv(KF / NE, 256), 1024)), dim3(256), 0, s,
                           (const T *)W, K,
                           (int)a.G, F, keys, hist, st);
    };
    if (bf) {
        if (F % 4 == 0) scores(bf16_t{}, std::integral_constant<int, 4>{});
        else if (F % 2 == 0) scores(bf16_t{}, std::integral_constant<int, 2>{});
        else scores(bf16_t{}, std::integral_constant<int, 1>{});
    } else {
        if (F % 4 == 0) scores(float{}, std::integral_constant<int, 4>{});
        else scores(float{}, std::integral_constant<int, 1>{});
    }
    for (int shift = 16; shift >= 0; shift -= 8)
        hipLaunchKernelGGL(k_rw_hist, dim3((unsigned)blocks(cdiv(KF, 4096), 256)), dim3(1024), 0, s, keys, KF, st,
                           shift, hist);
    const int64_t nb = rw_blocks(a);
    hipLaunchKernelGGL(k_rw_eqcount, dim3((unsigned)nb), dim3(256), 0, s, keys, KF, st, cnt);
    hipLaunchKernelGGL(k_rw_scan, dim3(1), dim3(kRwScanThreads), 0, s, cnt, nb, st);
    const float scale = (float)(1.0 / sqrt((double)a.F_in)) * 5.9604644775390625e-08f;   // a 2^-24, exact
    const uint32_t fmagic = ((1u << 20) + (uint32_t)F - 1u) / (uint32_t)F;   // e / F = e fmagic >> 20, e <= 1024
    const dim3 g2((unsigned)cdiv(K, kRwWaves));
    auto regrow = [&](auto tag, auto npl, auto vb, auto vm) {
        using T = decltype(tag);
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, g2, dim3(64 * kRwWaves), 0, s, idx, (T *)W, m, keys, st, cnt, K, (int)a.G, F, (int)a.F_s,
                               init_random, seed, scale, fmagic);
        };
        constexpr int NPL = decltype(npl)::value, VB = decltype(vb)::value, VM = decltype(vm)::value;
        if (a.G * F <= kRwChunkSmall) go(k_rw_regrow<T, NPL, VB, VM, kRwChunkSmall>);
        else go(k_rw_regrow<T, NPL, VB, VM, kRwChunk>);
    };
    // accesses that divide a row: 16 bytes where every row is aligned to them, else 4, else one value
    using c16 = std::integral_constant<int, 16>;
    using c4 = std::integral_constant<int, 4>;
    using c2 = std::integral_constant<int, 2>;
    auto by_access = [&](auto npl) {
        if (bf) {
            if (F % 8 == 0) regrow(bf16_t{}, npl, c16{}, c16{});
            else if (F % 2 == 0) regrow(bf16_t{}, npl, c4{}, c4{});
            else regrow(bf16_t{}, npl, c2{}, c4{});
        } else {
            if (F % 4 == 0) regrow(float{}, npl, c16{}, c16{});
            else regrow(float{}, npl, c4{}, c4{});
        }
    };
    if (F <= 64) by_access(std::integral_constant<int, 1>{});
    else if (F <= 128) by_access(std::integral_constant<int, 2>{});
    else by_access(std::integral_constant<int, 4>{});
    return hipGetLastError();
}

}  // namespace haste
