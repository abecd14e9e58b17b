// Semantic grouping of labels (Alg. 2): coarse spherical k-means into C = max(1, N / (beta G))
// clusters, then greedy groups inside each cluster: a random unassigned seed together with its
// top-(G - 1) unassigned neighbours by cosine similarity (Section 3.1, "Label Grouping").
// Embeddings are int8 (unit vectors x 127).  A centre is the direction of its members' sum s, kept
// exactly as an int32 vector; a label goes to the centre maximising e.s / |s| (the cosine up to the
// label's own norm), where e.s is an exact integer and |s| the correctly rounded square root of
// the exact |s|^2, and the quotient is one fp64 division.  The products e.s run on int8 MFMA: s is
// split into balanced base-256 digit planes, s = sum_p 256^p d_p with d_p in [-128, 127], and the
// planes' exact int32 products are recombined in int64.  Greedy similarities are the fp64 cosine
// (e_i.e_s) / sqrt(|e_i|^2 |e_s|^2) of exact integers.
// Draws: SplitMix64 (Steele, Lea and Flood, 2014) in counter form.
#include <cfloat>
#include <climits>

#include "common.hpp"

namespace {

typedef int i32x4_t __attribute__((ext_vector_type(4)));

constexpr int kGlPlanes = 4;   // |s| < 2^31 (N < 2^24 members of |e_d| <= 127) needs four digits

__device__ __forceinline__ uint64_t splitmix64_at(uint64_t s, uint64_t i) {
    uint64_t z = s + (i + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__global__ void k_gl_iota(int32_t *__restrict__ a, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] = (int32_t)i;
}

// the first C entries of a partial Fisher-Yates shuffle of [0, N): swap partner of i is
// i + out(i) mod (N - i)
__global__ void k_gl_shuffle(int32_t *__restrict__ a, int64_t N, int64_t C, uint64_t seed) {
    if (threadIdx.x != 0) return;
    for (int64_t i = 0; i < C; ++i) {
        const int64_t j = i + (int64_t)(splitmix64_at(seed, (uint64_t)i) % (uint64_t)(N - i));
        const int32_t t = a[i];
        a[i] = a[j];
        a[j] = t;
    }
}

// The same entries without the swaps' chain of memory accesses: before step i, position p holds p, or, if
// the last earlier step k with partner p exists, what position k held before step k.  One workgroup; every
// thread follows its entries' chains through the partners in LDS (C <= kGlShuffleMax).  C = 256: 129 us
// swap by swap, 5 us.
constexpr int kGlShuffleMax = 8192;
__global__ __launch_bounds__(1024) void k_gl_draw(int32_t *__restrict__ a, int64_t N, int C, uint64_t seed) {
    extern __shared__ int32_t partner[];          // [C]
    for (int i = threadIdx.x; i < C; i += blockDim.x)
        partner[i] = i + (int32_t)(splitmix64_at(seed, (uint64_t)i) % (uint64_t)(N - i));
    __syncthreads();
    for (int i = threadIdx.x; i < C; i += blockDim.x) {
        int32_t p = partner[i];
        for (int k = i - 1; k >= 0; --k)
            if (partner[k] == p) p = k;           // from here, position k before step k
        a[i] = p;
    }
}

// Centre c is the direction of the int32 vector s_c (a label's embedding at the start, then the
// sum of its members).  The assignment reads it as digit planes cp[p][c][D] (s_c = sum_p 256^p
// cp[p][c]), the number of planes it needs cnp[c] (higher planes are zero), and its norm cn[c].
constexpr int kGlWaves = 8;
constexpr int kGlMaxD = 1024;
constexpr int kGlThreads = 256;

// Writes centre c from the int32 vector held by the workgroup (sum[t] = s[threadIdx.x + 256 t]):
// the exact |s|^2 (128-bit), its correctly rounded square root, the digit planes and their count.
// A zero vector leaves the centre as it was (the caller's "keep" rule).  Workgroup-uniform.
__device__ void gl_store_centre(const int32_t (&sum)[kGlMaxD / kGlThreads], int D, int64_t C, int c,
                                int32_t *__restrict__ cs, int8_t *__restrict__ cp, double *__restrict__ cn,
                                int32_t *__restrict__ cnp) {
    __shared__ unsigned __int128 red[kGlThreads];
    __shared__ int32_t rmax[kGlThreads];
    uint64_t q = 0;   // at most four squares below 2^62 each: exact in 64 bits
    int need = 1;
#pragma unroll
    for (int t = 0; t < kGlMaxD / kGlThreads; ++t) {
        const int d = threadIdx.x + kGlThreads * t;
        if (d < D) {
            q += (uint64_t)((int64_t)sum[t] * (int64_t)sum[t]);
            int32_t r = sum[t];
            for (int p = 0; p < kGlPlanes && r != 0; ++p) {
                const int32_t dp = (int32_t)(int8_t)(r & 0xFF);   // balanced digit in [-128, 127]
                r = (r - dp) / 256;                                // exact
                need = p + 1 > need ? p + 1 : need;
            }
        }
    }
    red[threadIdx.x] = q;
    rmax[threadIdx.x] = need;
    __syncthreads();
    for (int off = kGlThreads / 2; off > 0; off >>= 1) {
        if (threadIdx.x < off) {
            red[threadIdx.x] += red[threadIdx.x + off];
            rmax[threadIdx.x] = rmax[threadIdx.x] > rmax[threadIdx.x + off] ? rmax[threadIdx.x] : rmax[threadIdx.x + off];
        }
        __syncthreads();
    }
    const unsigned __int128 tot = red[0];
    const int np = rmax[0];
    __syncthreads();   // red and rmax may be reused by the caller's next centre
    if (tot == 0) return;
#pragma unroll
    for (int t = 0; t < kGlMaxD / kGlThreads; ++t) {
        const int d = threadIdx.x + kGlThreads * t;
        if (d < D) {
            int32_t r = sum[t];
            cs[(int64_t)c * D + d] = r;
            for (int p = 0; p < kGlPlanes; ++p) {
                const int32_t dp = (int32_t)(int8_t)(r & 0xFF);
                r = (r - dp) / 256;
                cp[((int64_t)p * C + c) * D + d] = (int8_t)dp;
            }
        }
    }
    if (threadIdx.x == 0) {
        cn[c] = sqrt((double)tot);   // one rounding of the exact integer, one correctly rounded root
        cnp[c] = np;
    }
}

// initial centres: the embeddings of labels a[0 .. C) (one workgroup per centre)
__global__ __launch_bounds__(kGlThreads) void k_gl_pick_centres(const int8_t *__restrict__ E,
                                                                const int32_t *__restrict__ a, int64_t C, int D,
                                                                int32_t *__restrict__ cs, int8_t *__restrict__ cp,
                                                                double *__restrict__ cn, int32_t *__restrict__ cnp) {
    const int c = blockIdx.x;
    const int8_t *e = E + (int64_t)a[c] * D;
    int32_t sum[kGlMaxD / kGlThreads];
#pragma unroll
    for (int t = 0; t < kGlMaxD / kGlThreads; ++t) {
        const int d = threadIdx.x + kGlThreads * t;
        sum[t] = d < D ? (int32_t)e[d] : 0;
    }
    gl_store_centre(sum, D, C, c, cs, cp, cn, cnp);
}

// cl[l] = argmax_c (E[l].s_c) / |s_c| (ties: the lower c).  A wave takes 16 MT labels, a workgroup of
// 8 waves 256, or 128 where 256 would leave half of the CUs without one, or with up to 256 dimensions (less
// work per centre) some (60000 labels and centres, 64 dimensions: 9.9 ms with 256, 7.8 the kernel before it;
// 30000 labels, 512 dimensions, the whole grouping: 1165 us with 256, 1056 with 128; 65536 labels, 768: 1417, 1555); centres pass through LDS 16 at a time, as many digit planes as the 16 need, and the next
// 16 wait in registers.  v_mfma_i32_16x16x64_i8, M = 16 labels, N = 16 centres, K = 64 dimensions: both
// operands hold, per lane, 16 consecutive dimensions (16 q .. 16 q + 15 of the 64-chunk) of their row, so
// each lane group contracts the same dimensions; result lane (centre l16, q) holds labels 4q .. 4q+3.
// Rows of the tile are 16 bytes longer than whole 64-chunks, so that the 16 lanes of a read meet 64
// different banks (1 KiB rows put them all on one).
// The quotient is compared through dot * (1 / |s_c|), which lies within 2^-51 of it: only scores closer
// than 2^-48 of the best are divided.  131K labels, 256 centres, 768 dimensions, three planes: 530 us with
// 16 labels a wave, 1 KiB rows and a division per score, 110 us.
template <int NK, int MT>
__global__ __launch_bounds__(64 * kGlWaves) void k_gl_assign(const int8_t *__restrict__ E, int64_t N, int D,
                                                             const int8_t *__restrict__ cp,
                                                             const double *__restrict__ cn,
                                                             const int32_t *__restrict__ cnp, int64_t C,
                                                             int32_t *__restrict__ cl) {
    constexpr int RS = 64 * NK + 16;              // bytes of a tile row
    constexpr int SL = kGlPlanes * 16 * 4 * NK / (64 * kGlWaves) > 0 ? kGlPlanes * 16 * 4 * NK / (64 * kGlWaves) : 1;
    __shared__ __align__(16) int8_t tile[kGlPlanes * 16 * RS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int l16 = lane & 15, q = lane >> 4;
    const int64_t l0 = (int64_t)blockIdx.x * (16 * MT * kGlWaves) + 16 * MT * wave;
    // this lane's A rows: label l0 + 16 m + l16, dims 64 kk + 16 q .. +15 (zero past D or past N)
    const Buf eb(E, (uint32_t)(N * D));
    i32x4_t a[MT][NK];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int kk = 0; kk < NK; ++kk) {
            const int d0 = 64 * kk + 16 * q;
            const int64_t l = l0 + 16 * m + l16;
            a[m][kk] = __builtin_bit_cast(i32x4_t, eb.ld16(d0 < D && l < N ? (uint32_t)(l * D + d0) : kOob));
        }
    // best so far per label: the score's stand-in, the exact product and the centre
    double bv[MT][4], bd[MT][4];
    int bi[MT][4];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            bv[m][i] = bd[m][i] = 0.0;
            bi[m][i] = INT_MAX;
        }
    // 16-byte piece e of a tile: plane e / (64 NK), centre, chunk (zero past D and past C)
    const Buf cb(cp, (uint32_t)(kGlPlanes * C * D));
    uint4 st[SL];
    auto load = [&](int64_t c0) {
#pragma unroll
        for (int i = 0; i < SL; ++i) {
            const int e = threadIdx.x + 64 * kGlWaves * i, p = e / (64 * NK), r = (e / (4 * NK)) & 15, ch = e % (4 * NK);
            st[i] = cb.ld16(p < kGlPlanes && c0 + r < C && 16 * ch < D ? (uint32_t)(((int64_t)p * C + c0 + r) * D + 16 * ch) : kOob);
        }
    };
    auto planes = [&](int64_t c0) -> int {        // of the 16 centres (wave-uniform)
        const int v = c0 + l16 < C ? cnp[c0 + l16] : 1;
        return __ballot(v > 3) ? 4 : __ballot(v > 2) ? 3 : __ballot(v > 1) ? 2 : 1;
    };
    load(0);
    int npn = planes(0);
    for (int64_t c0 = 0; c0 < C; c0 += 16) {
        const int npt = npn;
        __syncthreads();                          // the previous tile is no longer read
#pragma unroll
        for (int i = 0; i < SL; ++i) {
            const int e = threadIdx.x + 64 * kGlWaves * i, r = e / (4 * NK), ch = e % (4 * NK);   // row: plane 16 + centre
            if (r < 16 * kGlPlanes) *reinterpret_cast<uint4 *>(&tile[r * RS + 16 * ch]) = st[i];
        }
        __syncthreads();
        if (c0 + 16 < C) {
            load(c0 + 16);
            npn = planes(c0 + 16);
        }
        i32x4_t acc[kGlPlanes][MT];
#pragma unroll
        for (int p = 0; p < kGlPlanes; ++p) {
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[p][m] = i32x4_t{0, 0, 0, 0};
            if (p >= npt) continue;
#pragma unroll
            for (int kk = 0; kk < NK; ++kk) {
                const i32x4_t b = *reinterpret_cast<const i32x4_t *>(&tile[(16 * p + l16) * RS + 64 * kk + 16 * q]);
#pragma unroll
                for (int m = 0; m < MT; ++m) acc[p][m] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[m][kk], b, acc[p][m], 0, 0, 0);
            }
        }
        const int c = (int)(c0 + l16);
        if (c < C) {
            const double nc = cn[c], inv = 1.0 / nc;
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    // exact: |dot| < 2^31 127 1024 < 2^53
                    const double dot = fma((double)acc[3][m][i], 16777216.0,
                                           fma((double)acc[2][m][i], 65536.0, fma((double)acc[1][m][i], 256.0, (double)acc[0][m][i])));
                    const double v = dot * inv, t = fabs(bv[m][i]) * 0x1p-48, d = v - bv[m][i];
                    // centres ascend per lane: ties keep the lower one; a lane's first centre is always
                    // taken, so a label always gets a valid centre (even from NaN scores of zero rows)
                    bool take = d > t || bi[m][i] == INT_MAX;
                    if (!take && d >= -t) take = dot / nc > bd[m][i] / cn[bi[m][i]];
                    if (take) {
                        bv[m][i] = v;
                        bd[m][i] = dot;
                        bi[m][i] = c;
                    }
                }
        }
    }
    // best over the 16 lanes of each row group: larger value, then lower centre
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            double v = bi[m][i] != INT_MAX ? bd[m][i] / cn[bi[m][i]] : 0.0;
            int bc = bi[m][i];
            for (int off = 1; off < 16; off <<= 1) {
                const double ov = __shfl_xor(v, off, 64);
                const int oi = __shfl_xor(bc, off, 64);
                if (oi != INT_MAX && (bc == INT_MAX || ov > v || (ov == v && oi < bc))) {
                    v = ov;
                    bc = oi;
                }
            }
            const int64_t l = l0 + 16 * m + 4 * q + i;
            if (l16 == 0 && l < N) cl[l] = bc;
        }
}

__global__ void k_gl_zero(int32_t *__restrict__ p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

__global__ void k_gl_count(const int32_t *__restrict__ cl, int64_t N, int32_t *__restrict__ cnt) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) atomicAdd(&cnt[cl[i]], 1);
}

// block-wide inclusive sum of one value per thread (256 threads)
__device__ __forceinline__ int32_t block_incl_scan(int32_t v, int32_t *s) {
    s[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const int32_t a = threadIdx.x >= off ? s[threadIdx.x - off] : 0;
        __syncthreads();
        s[threadIdx.x] += a;
        __syncthreads();
    }
    const int32_t r = s[threadIdx.x];
    __syncthreads();
    return r;
}

// start[c] = sum of cnt[< c]; gstart[c] = sum of ceil(cnt[< c] / G); start[C], gstart[C] the totals
// (one workgroup)
__global__ __launch_bounds__(256) void k_gl_starts(const int32_t *__restrict__ cnt, int64_t C, int64_t G,
                                                   int32_t *__restrict__ start, int32_t *__restrict__ gstart,
                                                   int64_t *__restrict__ n_groups) {
    __shared__ int32_t s[256];
    __shared__ int32_t carry[2];
    if (threadIdx.x == 0) carry[0] = carry[1] = 0;
    __syncthreads();
    for (int64_t base = 0; base < C; base += 256) {
        const int64_t c = base + threadIdx.x;
        const int32_t v = c < C ? cnt[c] : 0;
        const int32_t g = (int32_t)((v + G - 1) / G);
        const int32_t iv = block_incl_scan(v, s);
        const int32_t ig = block_incl_scan(g, s);
        if (c < C) {
            start[c] = carry[0] + iv - v;
            gstart[c] = carry[1] + ig - g;
        }
        __syncthreads();
        if (threadIdx.x == 255) {
            carry[0] += iv;
            carry[1] += ig;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        start[C] = carry[0];
        gstart[C] = carry[1];
        *n_groups = carry[1];
    }
}

// members[start[c] ..] = the labels of cluster c in ascending order (one workgroup per cluster)
__global__ __launch_bounds__(256) void k_gl_collect(const int32_t *__restrict__ cl, int64_t N,
                                                    const int32_t *__restrict__ start, int32_t *__restrict__ members) {
    __shared__ int32_t s[256];
    const int c = blockIdx.x;
    int32_t pos = start[c];
    for (int64_t base = 0; base < N; base += 256) {
        const int64_t l = base + threadIdx.x;
        const int32_t f = (l < N && cl[l] == c) ? 1 : 0;
        const int32_t inc = block_incl_scan(f, s);
        if (f) members[pos + inc - 1] = (int32_t)l;
        pos += s[255];   // s still holds the scan: the block total
        __syncthreads();
    }
}

// The same lists as a stable counting sort over tiles of TL labels, one wave per tile, where the clusters'
// counters fit the LDS (C <= kGlSortMax): counts per (tile, cluster), their exclusive sums over the tiles,
// and then every tile writes its labels behind them.  131K labels, 256 clusters: 600 us for the three
// kernels above (each cluster scanned all labels), 31 us.
constexpr int kGlSortMax = 16384;
constexpr int kGlScanSegs = 16;

__global__ __launch_bounds__(64) void k_gl_hist(const int32_t *__restrict__ cl, int64_t N, int64_t TL, int C,
                                                int32_t *__restrict__ hist) {
    extern __shared__ int32_t hc[];               // [C]
    for (int c = threadIdx.x; c < C; c += 64) hc[c] = 0;
    __syncthreads();
    const int64_t l0 = blockIdx.x * TL, l1 = l0 + TL < N ? l0 + TL : N;
    for (int64_t l = l0 + threadIdx.x; l < l1; l += 64) atomicAdd(&hc[cl[l]], 1);
    __syncthreads();
    for (int c = threadIdx.x; c < C; c += 64) hist[(int64_t)blockIdx.x * C + c] = hc[c];
}

// hist[t][c] becomes the sum over earlier tiles; cnt[c] the total.  64 clusters x 16 runs of tiles.
__global__ __launch_bounds__(64 * kGlScanSegs) void k_gl_scan(int32_t *__restrict__ hist, int nt, int C,
                                                              int32_t *__restrict__ cnt) {
    __shared__ int32_t part[kGlScanSegs][64];
    const int c = blockIdx.x * 64 + (threadIdx.x & 63), sg = threadIdx.x >> 6;
    const int per = (nt + kGlScanSegs - 1) / kGlScanSegs, t0 = sg * per, t1 = t0 + per < nt ? t0 + per : nt;
    int32_t sum = 0;
    if (c < C) {
#pragma unroll 8
        for (int t = t0; t < t1; ++t) sum += hist[(int64_t)t * C + c];
    }
    part[sg][threadIdx.x & 63] = sum;
    __syncthreads();
    if (c >= C) return;
    int32_t run = 0;
    for (int j = 0; j < sg; ++j) run += part[j][threadIdx.x & 63];
#pragma unroll 8
    for (int t = t0; t < t1; ++t) {
        const int32_t v = hist[(int64_t)t * C + c];
        hist[(int64_t)t * C + c] = run;
        run += v;
    }
    if (sg == kGlScanSegs - 1) cnt[c] = run;
}

__global__ __launch_bounds__(64) void k_gl_fill(const int32_t *__restrict__ cl, int64_t N, int64_t TL, int C,
                                                const int32_t *__restrict__ hist, const int32_t *__restrict__ start,
                                                int32_t *__restrict__ members) {
    extern __shared__ int32_t hc[];               // [C]: where the tile's next label of the cluster goes
    for (int c = threadIdx.x; c < C; c += 64) hc[c] = start[c] + hist[(int64_t)blockIdx.x * C + c];
    __syncthreads();
    const int64_t l0 = blockIdx.x * TL, l1 = l0 + TL < N ? l0 + TL : N;
    const uint64_t lt = __lanemask_lt();
    for (int64_t base = l0; base < l1; base += 64) {
        const int64_t l = base + threadIdx.x;
        const int c = l < l1 ? cl[l] : -1;
        uint64_t left = __ballot(c >= 0);
        int rank = 0, same = 0;                   // labels of this lane's cluster before it, and in all
        while (left) {                            // cluster by cluster (wave-uniform)
            const int cc = __builtin_amdgcn_readlane(c, (int)__builtin_ctzll(left));
            const uint64_t m = __ballot(c == cc);
            if (c == cc) {
                rank = __popcll(m & lt);
                same = __popcll(m);
            }
            left &= ~m;
        }
        if (c >= 0) members[hc[c] + rank] = (int32_t)l;
        __syncthreads();
        if (c >= 0 && rank == same - 1) hc[c] += same;
        __syncthreads();
    }
}

// cs[c] += the sums of the clusters' member rows (cs zeroed before): a workgroup takes `rows`
// consecutive places of the member lists, run by run of one cluster; its 8 waves take every eighth member,
// a lane 16 dimensions, and the waves' sums meet in LDS before they are added (whole numbers: any order
// gives the same sum).  131K x 768: one workgroup per cluster reading single bytes 785 us, 22 us (and 5 for the centres).
// A run takes about 1.5 us, one after the other, so `rows` holds about four clusters of the average size.
constexpr int kGlSumRows = 256;                   // at most
__global__ __launch_bounds__(512) void k_gl_sum(const int8_t *__restrict__ E, int64_t N, int D,
                                                const int32_t *__restrict__ members, const int32_t *__restrict__ cl,
                                                const int32_t *__restrict__ start, int32_t *__restrict__ cs, int rows) {
    __shared__ int32_t wsum[8 * kGlMaxD];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t p0 = (int64_t)blockIdx.x * rows, p1 = p0 + rows < N ? p0 + rows : N;
    const bool own = 16 * lane < D;
    for (int64_t q0 = p0; q0 < p1;) {             // workgroup-uniform
        const int c = cl[members[q0]];
        const int64_t q1 = start[c + 1] < p1 ? start[c + 1] : p1;
        int32_t acc[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) acc[k] = 0;
        for (int64_t m0 = q0 + wave; m0 < q1; m0 += 64) {   // 8 members of this wave
            uint4 v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const bool ok = own && m0 + 8 * j < q1;
                v[j] = ok ? *reinterpret_cast<const uint4 *>(E + (int64_t)members[m0 + 8 * j] * D + 16 * lane) : make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint32_t w[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
#pragma unroll
                for (int k = 0; k < 16; ++k)      // a dot product with one 1 adds one signed byte
                    acc[k] = __builtin_amdgcn_sdot4((int)w[k >> 2], 1 << (8 * (k & 3)), acc[k], false);
            }
        }
        if (own) {
#pragma unroll
            for (int k = 0; k < 16; ++k) wsum[wave * kGlMaxD + 16 * lane + k] = acc[k];
        }
        __syncthreads();
        for (int d = threadIdx.x; d < D; d += 512) {
            int32_t t = 0;
#pragma unroll
            for (int w = 0; w < 8; ++w) t += wsum[w * kGlMaxD + d];
            if (t != 0) atomicAdd(&cs[(int64_t)c * D + d], t);
        }
        __syncthreads();
        q0 = q1;
    }
}

// centre c from the sum in cs (one workgroup per cluster; an empty cluster, or one whose members sum to
// zero, keeps its centre)
__global__ __launch_bounds__(kGlThreads) void k_gl_centroid(int D, int64_t C, const int32_t *__restrict__ start,
                                                            int32_t *__restrict__ cs, int8_t *__restrict__ cp,
                                                            double *__restrict__ cn, int32_t *__restrict__ cnp) {
    const int c = blockIdx.x;
    if (start[c + 1] == start[c]) return;   // workgroup-uniform
    int32_t sum[kGlMaxD / kGlThreads];
#pragma unroll
    for (int t = 0; t < kGlMaxD / kGlThreads; ++t) {
        const int d = threadIdx.x + kGlThreads * t;
        sum[t] = d < D ? cs[(int64_t)c * D + d] : 0;
    }
    gl_store_centre(sum, D, C, c, cs, cp, cn, cnp);
}

// |e|^2 of every label (exact integers below 2^24), 16 lanes per label
__global__ __launch_bounds__(256) void k_gl_norms(const int8_t *__restrict__ E, int64_t N, int D, int32_t *__restrict__ nrm) {
    const int64_t l = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
    const int l16 = threadIdx.x & 15;
    int32_t acc = 0;
    if (l < N) {
        for (int d = 16 * l16; d < D; d += 256) {
            const uint4 v = *reinterpret_cast<const uint4 *>(E + l * D + d);
            acc = __builtin_amdgcn_sdot4((int)v.x, (int)v.x, acc, false);
            acc = __builtin_amdgcn_sdot4((int)v.y, (int)v.y, acc, false);
            acc = __builtin_amdgcn_sdot4((int)v.z, (int)v.z, acc, false);
            acc = __builtin_amdgcn_sdot4((int)v.w, (int)v.w, acc, false);
        }
    }
    for (int off = 8; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 16);
    if (l < N && l16 == 0) nrm[l] = acc;
}

// Greedy groups of clusters of up to kGlSmall members (one workgroup per cluster; the larger ones take
// the kernel below).  The unassigned members' places stay compact and ascending in LDS, so the seed
// is read directly; 16 lanes form one member's product with the seed's row; and instead of k - 1 passes
// of a workgroup maximum, a radix selection over the upper halves of the similarities finds the value
// that the group's other members lie above, and only those at it are compared in full.  131K labels, 256
// clusters (the largest of about 2000): 6.4 ms with the kernel below, 0.48 ms.
constexpr int kGlSmall = 2048;
constexpr int kGlSmallThreads = 1024;
__global__ __launch_bounds__(kGlSmallThreads) void k_gl_greedy_small(
    const int8_t *__restrict__ E, int64_t N, int D, const int32_t *__restrict__ members, const int32_t *__restrict__ start,
    const int32_t *__restrict__ gstart, int64_t G, uint64_t seed, const int32_t *__restrict__ nrm, int32_t *__restrict__ order,
    int32_t *__restrict__ gsize) {
    constexpr int T = kGlSmallThreads, PT = kGlSmall / T;   // members per thread
    constexpr int RU = 4;                         // rows in flight per 16 lanes
    __shared__ int32_t un[2][kGlSmall];           // places of the unassigned members, ascending
    __shared__ int32_t lab[kGlSmall];             // their labels
    __shared__ int32_t dot[kGlSmall];
    __shared__ uint2 eq[kGlSmall];                // members at the threshold: lower half, place
    __shared__ int32_t hist[256], wcnt[2][T / 64];
    __shared__ int32_t s_bin, s_above, s_eq;
    const int c = blockIdx.x;
    const int32_t m0 = start[c], n = start[c + 1] - m0;
    if (n > kGlSmall) return;                     // workgroup-uniform
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l16 = lane & 15;
    int32_t g = gstart[c], pos = m0;
    for (int i = tid; i < n; i += T) un[0][i] = i;
    __syncthreads();
    int cur = 0;
    for (int64_t t = 0, nu = n; nu > 0; ++t, cur ^= 1) {
        const int u = (int)nu, k = u < (int)G ? u : (int)G;
        const int r = (int)(splitmix64_at(seed, (uint64_t)(N + (int64_t)c * N + t)) % (uint64_t)nu);
        for (int i = tid; i < u; i += T) lab[i] = members[m0 + un[cur][i]];
        if (tid == 0) s_eq = 0;
        __syncthreads();
        int need = k - 1;                         // members to choose beside the seed
        uint32_t thr = 0;                         // those whose upper half lies above it, and `need` of those at it
        uint64_t key[PT];                         // ordered as the similarities
#pragma unroll
        for (int j = 0; j < PT; ++j) key[j] = 0;
        if (need > 0 && need < u - 1) {           // workgroup-uniform; else none or all of them
            const int8_t *es = E + (int64_t)lab[r] * D;
            uint4 sv[kGlMaxD / 256];
#pragma unroll
            for (int q = 0; q < kGlMaxD / 256; ++q)
                sv[q] = 16 * l16 + 256 * q < D ? *reinterpret_cast<const uint4 *>(es + 16 * l16 + 256 * q) : make_uint4(0, 0, 0, 0);
            for (int i0 = tid >> 4; i0 < u; i0 += RU * (T / 16)) {
                int32_t acc[RU];
#pragma unroll
                for (int x = 0; x < RU; ++x) {
                    const int i = i0 + x * (T / 16);
                    const int8_t *e = E + (int64_t)lab[i < u ? i : i0] * D + 16 * l16;
                    acc[x] = 0;
#pragma unroll
                    for (int q = 0; q < kGlMaxD / 256; ++q) {
                        if (16 * l16 + 256 * q >= D) continue;
                        const uint4 v = *reinterpret_cast<const uint4 *>(e + 256 * q);
                        acc[x] = __builtin_amdgcn_sdot4((int)v.x, (int)sv[q].x, acc[x], false);
                        acc[x] = __builtin_amdgcn_sdot4((int)v.y, (int)sv[q].y, acc[x], false);
                        acc[x] = __builtin_amdgcn_sdot4((int)v.z, (int)sv[q].z, acc[x], false);
                        acc[x] = __builtin_amdgcn_sdot4((int)v.w, (int)sv[q].w, acc[x], false);
                    }
                }
#pragma unroll
                for (int x = 0; x < RU; ++x) {
                    const int i = i0 + x * (T / 16);
                    for (int off = 8; off > 0; off >>= 1) acc[x] += __shfl_xor(acc[x], off, 16);
                    if (l16 == 0 && i < u) dot[i] = acc[x];
                }
            }
            __syncthreads();
            const int64_t ns = nrm[lab[r]];
#pragma unroll
            for (int j = 0; j < PT; ++j) {
                const int i = tid + T * j;
                if (i >= u) continue;
                const uint64_t b = __builtin_bit_cast(uint64_t, (double)dot[i] / sqrt((double)((int64_t)nrm[lab[i]] * ns)));
                key[j] = b >> 63 ? ~b : b | (uint64_t)1 << 63;
            }
            for (int sh = 24; sh >= 0; sh -= 8) {
                for (int i = tid; i < 256; i += T) hist[i] = 0;
                __syncthreads();
#pragma unroll
                for (int j = 0; j < PT; ++j) {
                    const int i = tid + T * j;
                    const uint32_t hi = (uint32_t)(key[j] >> 32);
                    if (i < u && i != r && (sh == 24 || hi >> (sh + 8) == thr >> (sh + 8))) atomicAdd(&hist[(hi >> sh) & 255], 1);
                }
                __syncthreads();
                if (wave == 0) {                  // the bin that holds the need-th from above: lane -> 4 bins downward
                    int32_t cnt[4], sum = 0;
#pragma unroll
                    for (int x = 0; x < 4; ++x) sum += cnt[x] = hist[255 - 4 * lane - x];
                    int32_t incl = sum;
                    for (int off = 1; off < 64; off <<= 1) {
                        const int32_t o = __shfl_up(incl, off);
                        if (lane >= off) incl += o;
                    }
                    int32_t above = incl - sum;
                    if (above < need && incl >= need) {
                        int x = 0;
                        while (above + cnt[x] < need) above += cnt[x++];
                        s_bin = 255 - 4 * lane - x;
                        s_above = above;
                    }
                }
                __syncthreads();
                thr |= (uint32_t)s_bin << sh;
                need -= s_above;
            }
#pragma unroll
            for (int j = 0; j < PT; ++j) {
                const int i = tid + T * j;
                if (i < u && i != r && (uint32_t)(key[j] >> 32) == thr) eq[atomicAdd(&s_eq, 1)] = make_uint2((uint32_t)key[j], (uint32_t)i);
            }
            __syncthreads();
        }
        // the group in ascending order, and the rest: T places at a time
        const bool all_in = k == u;
        int gone = 0;                             // chosen members before this run of T
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            if (T * j >= u) break;                // workgroup-uniform
            const int i = tid + T * j;
            bool in = i < u && (all_in || i == r);
            if (i < u && i != r && !all_in && k > 1) {
                const uint32_t hi = (uint32_t)(key[j] >> 32), lo = (uint32_t)key[j];
                in = hi > thr;
                if (hi == thr) {                  // larger similarity first, then the lower place
                    int rank = 0;
                    for (int x = 0; x < s_eq; ++x) rank += eq[x].x > lo || (eq[x].x == lo && (int)eq[x].y < i);
                    in = rank < need;
                }
            }
            const uint64_t m = __ballot(in);
            if (lane == 0) wcnt[j & 1][wave] = __popcll(m);
            __syncthreads();
            int before = gone, all = gone;
            for (int w = 0; w < T / 64; ++w) {
                before += w < wave ? wcnt[j & 1][w] : 0;
                all += wcnt[j & 1][w];
            }
            before += __popcll(m & __lanemask_lt());
            if (i < u) {
                if (in) order[pos + before] = lab[i];
                else un[cur ^ 1][i - before] = un[cur][i];
            }
            gone = all;
        }
        if (tid == 0) gsize[g] = k;
        __syncthreads();
        pos += k;
        ++g;
        nu -= k;
    }
}

// Greedy groups inside each cluster of more than kGlSmall members (one workgroup per cluster): the seed is the (out(N + c N + t)
// mod nu)-th unassigned member in ascending order; the group is the seed and its top-(k - 1)
// unassigned members by cosine to it (k = min(G, nu), ties to the lower label), listed in ascending
// label order.
__global__ __launch_bounds__(kGlThreads) void k_gl_greedy(const int8_t *__restrict__ E, int64_t N, int D,
                                                          const int32_t *__restrict__ members,
                                                          const int32_t *__restrict__ start,
                                                          const int32_t *__restrict__ gstart, int64_t G,
                                                          uint64_t seed, const int32_t *__restrict__ nrm,
                                                          uint8_t *__restrict__ taken, double *__restrict__ sims,
                                                          int32_t *__restrict__ order, int32_t *__restrict__ gsize) {
    __shared__ int32_t s[kGlThreads];
    __shared__ double rv[kGlThreads];
    __shared__ int32_t ri[kGlThreads];
    __shared__ int32_t sel[256];
    __shared__ int32_t bpos;
    const int c = blockIdx.x;
    const int32_t m0 = start[c], n = start[c + 1] - m0;
    if (n <= kGlSmall) return;                    // workgroup-uniform
    int32_t g = gstart[c], pos = m0;
    for (int32_t i = threadIdx.x; i < n; i += kGlThreads) taken[m0 + i] = 0;
    __syncthreads();
    for (int64_t t = 0, nu = n; nu > 0; ++t) {
        // the seed: the r-th unassigned member, by a block scan over the members in order
        const int64_t r = (int64_t)(splitmix64_at(seed, (uint64_t)(N + (int64_t)c * N + t)) % (uint64_t)nu);
        int32_t before = 0;
        if (threadIdx.x == 0) bpos = -1;
        __syncthreads();
        for (int32_t base = 0; base < n; base += kGlThreads) {
            const int32_t i = base + threadIdx.x;
            const int32_t f = (i < n && !taken[m0 + i]) ? 1 : 0;
            const int32_t inc = block_incl_scan(f, s);
            if (f && before + inc - 1 == r) bpos = i;
            before += s[kGlThreads - 1];
            __syncthreads();
            if (bpos >= 0) break;   // workgroup-uniform after the barrier
        }
        if (bpos < 0) break;   // cannot happen (r < nu unassigned members); never index E with it
        const int32_t sp = bpos, bc = members[m0 + sp];
        const int8_t *es = E + (int64_t)bc * D;
        const int64_t ns = nrm[bc];
        // cosines of the other unassigned members to the seed
        for (int32_t i = threadIdx.x; i < n; i += kGlThreads) {
            if (taken[m0 + i] || i == sp) continue;
            const int32_t lab = members[m0 + i];
            const int8_t *e = E + (int64_t)lab * D;
            int32_t acc = 0;
            for (int d = 0; d < D; d += 4)
                acc = __builtin_amdgcn_sdot4(*reinterpret_cast<const int32_t *>(e + d),
                                             *reinterpret_cast<const int32_t *>(es + d), acc, false);
            sims[m0 + i] = (double)acc / sqrt((double)((int64_t)nrm[lab] * ns));
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            sel[0] = bc;
            taken[m0 + sp] = 1;
        }
        __syncthreads();
        // the other k - 1 by repeated block argmax (larger cosine, then lower member position,
        // i.e. lower label: members ascend)
        const int32_t k = (int32_t)(nu < G ? nu : G);
        for (int32_t j = 1; j < k; ++j) {
            double best = -DBL_MAX;
            int32_t bi = INT_MAX;
            for (int32_t i = threadIdx.x; i < n; i += kGlThreads) {
                if (taken[m0 + i]) continue;
                const double v = sims[m0 + i];
                if (bi == INT_MAX || v > best || (v == best && i < bi)) {   // any unassigned member first
                    best = v;
                    bi = i;
                }
            }
            rv[threadIdx.x] = best;
            ri[threadIdx.x] = bi;
            __syncthreads();
            for (int off = kGlThreads / 2; off > 0; off >>= 1) {
                if (threadIdx.x < off) {
                    const double ov = rv[threadIdx.x + off];
                    const int32_t oi = ri[threadIdx.x + off];
                    if (oi != INT_MAX &&
                        (ri[threadIdx.x] == INT_MAX || ov > rv[threadIdx.x] || (ov == rv[threadIdx.x] && oi < ri[threadIdx.x]))) {
                        rv[threadIdx.x] = ov;
                        ri[threadIdx.x] = oi;
                    }
                }
                __syncthreads();
            }
            if (threadIdx.x == 0) {
                // k <= nu, so an unassigned member exists and ri[0] < n; never index past it
                const int32_t pick = ri[0] < n ? ri[0] : 0;
                sel[j] = members[m0 + pick];
                taken[m0 + pick] = 1;
            }
            __syncthreads();
        }
        // the group, ascending (insertion sort of at most G <= 256 labels)
        if (threadIdx.x == 0) {
            for (int32_t i = 1; i < k; ++i) {
                const int32_t v = sel[i];
                int32_t j = i - 1;
                while (j >= 0 && sel[j] > v) {
                    sel[j + 1] = sel[j];
                    --j;
                }
                sel[j + 1] = v;
            }
            gsize[g] = k;
        }
        __syncthreads();
        for (int32_t i = threadIdx.x; i < k; i += kGlThreads) order[pos + i] = sel[i];
        __syncthreads();
        pos += k;
        ++g;
        nu -= k;
    }
}

}  // namespace

namespace haste {

static int64_t gl_clusters(int64_t N, int64_t G, int64_t beta) {
    const int64_t C = N / (beta * G);
    return C < 1 ? 1 : C;
}

bool group_supported(int64_t N, int64_t D, int64_t G, int64_t beta) {
    // N < 2^24 keeps a cluster's int32 sums of int8 rows (|e_d| <= 127) exact and inside four
    // balanced base-256 digits; the digit planes (4 C D bytes) stay addressable by 32-bit offsets
    if (!(N > 0 && N < ((int64_t)1 << 24) && D > 0 && D % 16 == 0 && D <= kGlMaxD && G >= 1 && G <= 256 &&
          beta >= 1 && N * D < ((int64_t)1 << 31)))
        return false;
    return kGlPlanes * gl_clusters(N, G, beta) * D < ((int64_t)1 << 31);
}

size_t group_ws(int64_t N, int64_t D, int64_t G, int64_t beta) {
    const int64_t C = gl_clusters(N, G, beta);
    return (size_t)(round_up(N * 4, 256) * 4 + round_up(N * 8, 256) + round_up(N, 256) + round_up(C * D * 4, 256) +
                    round_up(kGlPlanes * C * D, 256) + round_up(C * 8, 256) + round_up((C + 1) * 4, 256) * 4 + 256);
}

hipError_t group_labels(int64_t N, int64_t D, const int8_t *E, int64_t G, int64_t beta, int64_t iters, uint64_t seed,
                        int32_t *order, int32_t *gsize, int64_t *n_groups, int32_t *cluster, void *ws, hipStream_t s) {
    const int64_t C = gl_clusters(N, G, beta);
    char *p = static_cast<char *>(ws);
    auto take = [&](int64_t bytes) {
        char *q = p;
        p += round_up(bytes, 256);
        return q;
    };
    int32_t *a = reinterpret_cast<int32_t *>(take(N * 4));
    int32_t *cl = cluster ? cluster : reinterpret_cast<int32_t *>(take(N * 4));
    if (cluster) take(N * 4);
    int32_t *members = reinterpret_cast<int32_t *>(take(N * 4));
    int32_t *nrm = reinterpret_cast<int32_t *>(take(N * 4));
    double *sims = reinterpret_cast<double *>(take(N * 8));
    uint8_t *taken = reinterpret_cast<uint8_t *>(take(N));
    int32_t *cs = reinterpret_cast<int32_t *>(take(C * D * 4));
    int8_t *cp = reinterpret_cast<int8_t *>(take(kGlPlanes * C * D));
    double *cn = reinterpret_cast<double *>(take(C * 8));
    int32_t *cnp = reinterpret_cast<int32_t *>(take((C + 1) * 4));
    int32_t *cnt = reinterpret_cast<int32_t *>(take((C + 1) * 4));
    int32_t *start = reinterpret_cast<int32_t *>(take((C + 1) * 4));
    int32_t *gstart = reinterpret_cast<int32_t *>(take((C + 1) * 4));
    const int Di = (int)D;
    if (C <= kGlShuffleMax) {
        hipLaunchKernelGGL(k_gl_draw, dim3(1), dim3(1024), (size_t)C * 4, s, a, N, (int)C, seed);
    } else {
        hipLaunchKernelGGL(k_gl_iota, dim3((unsigned)cdiv(N, 256)), dim3(256), 0, s, a, N);
        hipLaunchKernelGGL(k_gl_shuffle, dim3(1), dim3(64), 0, s, a, N, C, seed);
    }
    hipLaunchKernelGGL(k_gl_pick_centres, dim3((unsigned)C), dim3(kGlThreads), 0, s, E, a, C, Di, cs, cp, cn, cnp);
    auto assign = [&](auto nk) {
        constexpr int NK = decltype(nk)::value;
        auto go = [&](auto kern, int mt) {
            hipLaunchKernelGGL(kern, dim3((unsigned)cdiv(N, 16 * mt * kGlWaves)), dim3(64 * kGlWaves), 0, s, E, N, Di, cp, cn, cnp, C, cl);
        };
        if (cdiv(N, 32 * kGlWaves) <= (NK == 4 ? kXcds * kCusPerXcd : kXcds * kCusPerXcd / 2)) go(k_gl_assign<NK, 1>, 1);
        else go(k_gl_assign<NK, 2>, 2);
    };
    // tiles of the counting sort: about 512, and few enough that their counts fit the similarities' space
    // (8 N bytes; those come later)
    int64_t TL = cdiv(N, 512) > 256 ? cdiv(N, 512) : 256;
    if (TL < cdiv(C, 2)) TL = cdiv(C, 2);
    const int nt = (int)cdiv(N, TL);
    const bool sorted = C <= kGlSortMax && (int64_t)nt * C * 4 <= N * 8;
    int32_t *hist = reinterpret_cast<int32_t *>(sims);
    hipError_t e = hipSuccess;
    if (sorted) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_gl_hist), hipFuncAttributeMaxDynamicSharedMemorySize, (int)C * 4);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_gl_fill), hipFuncAttributeMaxDynamicSharedMemorySize, (int)C * 4);
        if (e != hipSuccess) return e;
    }
    auto assign_and_collect = [&]() {
        if (D <= 256) assign(std::integral_constant<int, 4>{});
        else if (D <= 512) assign(std::integral_constant<int, 8>{});
        else if (D <= 768) assign(std::integral_constant<int, 12>{});
        else assign(std::integral_constant<int, 16>{});
        if (sorted) {
            hipLaunchKernelGGL(k_gl_hist, dim3((unsigned)nt), dim3(64), (size_t)C * 4, s, cl, N, TL, (int)C, hist);
            hipLaunchKernelGGL(k_gl_scan, dim3((unsigned)cdiv(C, 64)), dim3(64 * kGlScanSegs), 0, s, hist, nt, (int)C, cnt);
            hipLaunchKernelGGL(k_gl_starts, dim3(1), dim3(256), 0, s, cnt, C, G, start, gstart, n_groups);
            hipLaunchKernelGGL(k_gl_fill, dim3((unsigned)nt), dim3(64), (size_t)C * 4, s, cl, N, TL, (int)C, hist, start, members);
            return;
        }
        hipLaunchKernelGGL(k_gl_zero, dim3((unsigned)cdiv(C, 256)), dim3(256), 0, s, cnt, C);
        hipLaunchKernelGGL(k_gl_count, dim3((unsigned)cdiv(N, 256)), dim3(256), 0, s, cl, N, cnt);
        hipLaunchKernelGGL(k_gl_starts, dim3(1), dim3(256), 0, s, cnt, C, G, start, gstart, n_groups);
        hipLaunchKernelGGL(k_gl_collect, dim3((unsigned)C), dim3(256), 0, s, cl, N, start, members);
    };
    const int sum_rows = (int)(4 * N / C < kGlSumRows ? 4 * N / C : kGlSumRows);
    for (int64_t it = 0; it < iters; ++it) {
        assign_and_collect();
        hipLaunchKernelGGL(k_gl_zero, dim3((unsigned)cdiv(C * D, 256)), dim3(256), 0, s, cs, C * D);
        hipLaunchKernelGGL(k_gl_sum, dim3((unsigned)cdiv(N, sum_rows)), dim3(512), 0, s, E, N, Di, members, cl, start, cs, sum_rows);
        hipLaunchKernelGGL(k_gl_centroid, dim3((unsigned)C), dim3(kGlThreads), 0, s, Di, C, start, cs, cp, cn, cnp);
    }
    assign_and_collect();
    hipLaunchKernelGGL(k_gl_norms, dim3((unsigned)cdiv(N, 16)), dim3(256), 0, s, E, N, Di, nrm);
    hipLaunchKernelGGL(k_gl_greedy_small, dim3((unsigned)C), dim3(kGlSmallThreads), 0, s, E, N, Di, members, start, gstart,
                       G, seed, nrm, order, gsize);
    hipLaunchKernelGGL(k_gl_greedy, dim3((unsigned)C), dim3(kGlThreads), 0, s, E, N, Di, members, start, gstart, G,
                       seed, nrm, taken, sims, order, gsize);
    return hipGetLastError();
}

}  // namespace haste
