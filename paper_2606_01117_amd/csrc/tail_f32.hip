// The tail's three products for fp32 layers on v_mfma_f32_16x16x4_f32: fp32 inputs and accumulation,
// at twice the rate of the vector ALUs' multiply-adds, each operand element read once per 16 products.
// Any group size, support width up to 256 slots, feature width and label count.
//
// Every kernel works on units: up to 16 labels of one group, which share the group's gathered
// features.  A matrix instruction takes 4 K positions, one per 16-lane group q of the wave; four
// consecutive instructions j = 0 .. 3 cover 16 consecutive K indices 4q + j, so that a lane's four
// operand elements are neighbours and one 16-byte access brings all of them.
//
// Slots past the support have zero weights and meet a row of zeros (forward) or an accumulator row that
// nothing reads (backward-feature); labels past the group and rows past the batch read as zeros or are
// not stored.  So an infinity or a NaN reaches what the definition says and nothing else.
#include <type_traits>

#include "common.hpp"

namespace {

__device__ __forceinline__ f32x4_t mfma16x16x4(float a, float b, const f32x4_t &c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// four fp32 (or int32) at byte offset o, of which the first nv are read and the others zero; VEC: o is a
// multiple of 16 bytes from an aligned base, and nv is 4 or more, or 0 or less
template <bool VEC>
__device__ __forceinline__ uint4 load4(const Buf &b, uint32_t o, int nv) {
    if constexpr (VEC) return b.ld16(nv > 0 ? o : kOob);
    return make_uint4(b.ld4(nv > 0 ? o : kOob), b.ld4(nv > 1 ? o + 4 : kOob), b.ld4(nv > 2 ? o + 8 : kOob),
                      b.ld4(nv > 3 ? o + 12 : kOob));
}

// A workgroup's 32-row slab of X (rows past B zero): thread -> rows 4 w .. 4 w + 3 of features lane + 64 i
// (w: its wave), so that the global reads run along the features.  put(f, row quad, four values)
template <class Put>
__device__ __forceinline__ void load_slab32(const float *__restrict__ X, int b0, int B, int F_s, Put &&put) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int f = lane; f < F_s; f += 64) {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = b0 + 4 * w + r < B ? X[(int64_t)(b0 + 4 * w + r) * F_s + f] : 0.0f;
        put(f, w, v);
    }
}

// ---------------------------------------------------------------------------------------------
// Forward: Y^T tile [16 labels][16 rows] = W (16 labels x slots) times the gathered X^T (slots x rows).
// A workgroup of 8 waves keeps a 32-row slab of X^T in LDS, a feature's rows interleaved so that rows l16
// and 16 + l16 are neighbours (one 8-byte read brings the operands of both row tiles), and sweeps a
// segment of units, one per wave at a time, 64 slots (a chunk) at a time; the next chunk's supports and
// weights are loaded while the current one is multiplied.  A lane ends with 4 consecutive labels of a row.
// ---------------------------------------------------------------------------------------------
constexpr int kF32Waves = 8;
__host__ __device__ constexpr int f32_fwd_lds(int F_s) { return (F_s + 1) * 128; }

// VEC: F_in is a multiple of 4.  VST: G and L are, so that a lane's four logits are one store.
template <bool VEC, bool VST>
__global__ __launch_bounds__(512) void k_fwd_f32(const float *__restrict__ X, const int32_t *__restrict__ idx,
                                                 const float *__restrict__ W, const float *__restrict__ bias,
                                                 float *__restrict__ Y, int B, int F_s, int64_t L, int G, int F_in, int nt,
                                                 int64_t nunit, int64_t ups, int nbt) {
    extern __shared__ __align__(16) float xs32[];   // [F_s + 1][16][2]: feature F_s is zero
    const int w = blockIdx.x, xcd = w % kXcds, jj = w / kXcds;
    const int b0 = (jj % nbt) * 32;
    const int64_t seg = (int64_t)(jj / nbt) * kXcds + xcd;
    const int64_t u0 = seg * ups, u1 = u0 + ups < nunit ? u0 + ups : nunit;
    if (u0 >= u1) return;                         // workgroup-uniform
    load_slab32(X, b0, B, F_s, [&](int f, int rq, const float (&v)[4]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) xs32[f * 32 + ((4 * rq + r) & 15) * 2 + (rq >> 2)] = v[r];
    });
    if (threadIdx.x < 32) xs32[F_s * 32 + threadIdx.x] = 0.0f;
    __syncthreads();
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, q = lane >> 4;
    const int nch = (F_in + 63) >> 6;             // chunks of 64 slots
    struct Chunk {
        uint4 f[4], w[4];                         // slots 16 s + 4q .. + 3: features, weights of label l16
    };
    // unit u: labels lab .. of group k
    auto where = [&](int64_t u, int64_t &k, int &l0) {
        k = nt == 1 ? u : u / nt;
        l0 = 16 * (int)(u - k * nt);
    };
    auto load = [&](int64_t u, int c, Chunk &ch) {
        int64_t k;
        int l0;
        where(u, k, l0);
        const Buf ib(idx + k * F_in, (uint32_t)(F_in * 4));
        const Buf wb(W + k * G * F_in, (uint32_t)((int64_t)G * F_in * 4));   // labels past the group: zero
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int t = 64 * c + 16 * s + 4 * q;
            ch.f[s] = load4<VEC>(ib, (uint32_t)(t * 4), F_in - t);
            ch.w[s] = load4<VEC>(wb, (uint32_t)(((l0 + l16) * F_in + t) * 4), F_in - t);
        }
    };
    f32x4_t acc[2] = {f32x4_t{0, 0, 0, 0}, f32x4_t{0, 0, 0, 0}};
    auto chunk = [&](int64_t u, int c, const Chunk &ch) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int t = 64 * c + 16 * s + 4 * q;
            if (64 * c + 16 * s >= F_in) break;   // wave-uniform
            const uint32_t fs[4] = {ch.f[s].x, ch.f[s].y, ch.f[s].z, ch.f[s].w};
            const uint32_t ws[4] = {ch.w[s].x, ch.w[s].y, ch.w[s].z, ch.w[s].w};
            float2 x[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int f = t + j < F_in ? (int)fs[j] : F_s;
                x[j] = *reinterpret_cast<const float2 *>(xs32 + f * 32 + 2 * l16);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[0] = mfma16x16x4(__uint_as_float(ws[j]), x[j].x, acc[0]);
                acc[1] = mfma16x16x4(__uint_as_float(ws[j]), x[j].y, acc[1]);
            }
        }
        if (c + 1 < nch) return;                  // wave-uniform
        int64_t k;
        int l0;
        where(u, k, l0);
        const int nl = G - l0 - 4 * q;            // labels from this lane's first
        const int64_t lab = k * G + l0 + 4 * q;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int b = b0 + 16 * m + l16;
            if (b < B && nl > 0) {
                float v[4] = {acc[m][0], acc[m][1], acc[m][2], acc[m][3]};
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] += bias && r < nl ? bias[lab + r] : 0.0f;
                float *y = Y + (int64_t)b * L + lab;
                if constexpr (VST) {
                    *reinterpret_cast<float4 *>(y) = make_float4(v[0], v[1], v[2], v[3]);
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (r < nl) y[r] = v[r];
                }
            }
            acc[m] = f32x4_t{0, 0, 0, 0};
        }
    };
    // this wave's (unit, chunk) steps in order, each loaded one step ahead (past the last: a repeat)
    int64_t u = u0 + wave;
    if (u >= u1) return;
    int c = 0;
    Chunk ca, cb;
    load(u, 0, ca);
    auto next = [&](int64_t &nu, int &nc) {
        nc = c + 1 < nch ? c + 1 : 0;
        nu = c + 1 < nch ? u : u + kF32Waves;
    };
    for (;;) {
        int64_t nu;
        int nc;
        next(nu, nc);
        load(nu < u1 ? nu : u, nc, cb);
        chunk(u, c, ca);
        if (nu >= u1) break;
        u = nu;
        c = nc;
        next(nu, nc);
        load(nu < u1 ? nu : u, nc, ca);
        chunk(u, c, cb);
        if (nu >= u1) break;
        u = nu;
        c = nc;
    }
}

// ---------------------------------------------------------------------------------------------
// Backward-weight: dW^T tile [16 slots][16 labels] = X^T (slots x rows) times dY (rows x labels).  A wave
// owns UPW units for the whole batch (their tiles stay in registers) and the workgroup stages the batch's
// X^T in 32-row slabs, 36-float feature rows; the next slab waits in registers.  A lane reads its dY
// values straight from memory (4 rows of 16 labels per instruction), one unit ahead.  16 rows are summed
// from zero and then added, which over a batch rounds less than one chain (128 rows: relative error
// 1.0e-7 against 2.1e-7).
// ---------------------------------------------------------------------------------------------
constexpr int kBwRow = 36;                        // floats per staged feature row: 32 rows + pad
__host__ __device__ constexpr int f32_bw_lds(int F_s) { return F_s * kBwRow * 4; }
// units per wave: up to 8 tiles, which the registers hold beside the next slab (16 tiles: without it)
__host__ __device__ constexpr int f32_bw_upw(int nst) { return nst >= 8 ? 1 : 2; }

// NST: 16-slot tiles (16 NST >= F_in).  XI: features per thread of a slab (64 XI >= F_s).
template <int NST, int XI>
__global__ __launch_bounds__(512) void k_bwd_w_f32(const float *__restrict__ X, const int32_t *__restrict__ idx,
                                                   const float *__restrict__ dY, float *__restrict__ dW,
                                                   float *__restrict__ dbias, int beta, int B, int F_s, int64_t L, int G,
                                                   int F_in, int nt, int64_t nunit) {
    constexpr int UPW = f32_bw_upw(NST);
    constexpr bool AHEAD = NST <= 8;              // the next slab waits in registers
    extern __shared__ __align__(16) float xs32[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, q = lane >> 4;
    const int64_t u0 = ((int64_t)blockIdx.x * kF32Waves + wave) * UPW;
    int f[UPW][NST];
    int64_t lab[UPW];
    int nl[UPW];                                  // labels of the unit (none past the last unit)
#pragma unroll
    for (int j = 0; j < UPW; ++j) {
        const int64_t u = u0 + j < nunit ? u0 + j : nunit - 1;
        const int64_t k = nt == 1 ? u : u / nt;
        const int l0 = 16 * (int)(u - k * nt);
        lab[j] = k * G + l0;
        nl[j] = u0 + j < nunit ? (G - l0 < 16 ? G - l0 : 16) : 0;
#pragma unroll
        for (int st = 0; st < NST; ++st) f[j][st] = idx[k * F_in + (16 * st + l16 < F_in ? 16 * st + l16 : F_in - 1)];
    }
    float4 xr[XI];
    auto load_x = [&](int b0) {
#pragma unroll
        for (int i = 0; i < XI; ++i) {
            const int ff = lane + 64 * i;
            float v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int b = b0 + 4 * wave + r;
                v[r] = ff < F_s && b < B ? X[(int64_t)b * F_s + ff] : 0.0f;
            }
            xr[i] = make_float4(v[0], v[1], v[2], v[3]);
        }
    };
    // dY of unit j in the slab at b0: rows 16 h + 4q + r of label l16
    auto load_y = [&](int j, int b0, float (&y)[8]) {
        const bool ok = l16 < nl[j];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int b = b0 + 16 * (e >> 2) + 4 * q + (e & 3);
            y[e] = ok && b < B ? dY[(int64_t)b * L + lab[j] + l16] : 0.0f;
        }
    };
    f32x4_t acc[UPW][NST];
    float db[UPW];
#pragma unroll
    for (int j = 0; j < UPW; ++j) {
        db[j] = 0.0f;
#pragma unroll
        for (int st = 0; st < NST; ++st) acc[j][st] = f32x4_t{0, 0, 0, 0};
    }
    float y[2][8];
    if constexpr (AHEAD) load_x(0);
    load_y(0, 0, y[0]);
    for (int b0 = 0; b0 < B; b0 += 32) {
        __syncthreads();                          // the previous slab is no longer read
        if constexpr (!AHEAD) load_x(b0);
#pragma unroll
        for (int i = 0; i < XI; ++i)
            if (lane + 64 * i < F_s) *reinterpret_cast<float4 *>(xs32 + (lane + 64 * i) * kBwRow + 4 * wave) = xr[i];
        __syncthreads();
        if constexpr (AHEAD)
            if (b0 + 32 < B) load_x(b0 + 32);
#pragma unroll
        for (int j = 0; j < UPW; ++j) {
            constexpr bool ONE = UPW == 1;
            float(&yc)[8] = y[ONE ? 0 : j & 1];
            if constexpr (!ONE) {
                if (j + 1 < UPW) load_y(j + 1, b0, y[(j + 1) & 1]);
                else load_y(0, b0 + 32, y[(j + 1) & 1]);
            }
#pragma unroll
            for (int st = 0; st < NST; ++st) {
                f32x4_t d[2] = {f32x4_t{0, 0, 0, 0}, f32x4_t{0, 0, 0, 0}};
                float4 a[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) a[h] = *reinterpret_cast<const float4 *>(xs32 + f[j][st] * kBwRow + 16 * h + 4 * q);
#pragma unroll
                for (int h = 0; h < 2; ++h) d[h] = mfma16x16x4(a[h].x, yc[4 * h], d[h]);
#pragma unroll
                for (int h = 0; h < 2; ++h) d[h] = mfma16x16x4(a[h].y, yc[4 * h + 1], d[h]);
#pragma unroll
                for (int h = 0; h < 2; ++h) d[h] = mfma16x16x4(a[h].z, yc[4 * h + 2], d[h]);
#pragma unroll
                for (int h = 0; h < 2; ++h) d[h] = mfma16x16x4(a[h].w, yc[4 * h + 3], d[h]);
                acc[j][st] += d[0];
                acc[j][st] += d[1];
                // tile by tile (several tiles' sums at once would not fit the registers)
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) db[j] += yc[e];
            if constexpr (ONE) load_y(0, b0 + 32, y[0]);
        }
    }
    // lane (label l16, q) holds slots 16 st + 4q .. + 3
#pragma unroll
    for (int j = 0; j < UPW; ++j) {
        if (l16 < nl[j]) {
            float *row = dW + (lab[j] + l16) * F_in;
#pragma unroll
            for (int st = 0; st < NST; ++st) {
                const int t = 16 * st + 4 * q;
                if ((F_in & 3) == 0) {            // kernel-uniform
                    if (t < F_in) {
                        float4 v = make_float4(acc[j][st][0], acc[j][st][1], acc[j][st][2], acc[j][st][3]);
                        if (beta) {
                            const float4 o = *reinterpret_cast<const float4 *>(row + t);
                            v = make_float4(o.x + v.x, o.y + v.y, o.z + v.z, o.w + v.w);
                        }
                        *reinterpret_cast<float4 *>(row + t) = v;
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (t + r < F_in) row[t + r] = beta ? row[t + r] + acc[j][st][r] : acc[j][st][r];
                }
            }
        }
        if (dbias) {                              // kernel-uniform
            float s = db[j];
            s += __shfl_xor(s, 16);
            s += __shfl_xor(s, 32);
            if (q == 0 && l16 < nl[j]) dbias[lab[j] + l16] = beta ? dbias[lab[j] + l16] + s : s;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Backward-feature: tile [16 rows][16 slots] = dY (rows x labels) times W (labels x slots), added onto
// the accumulator dX^T [F_s][16 rows] in LDS by plain read-add-write through the matrix core's
// accumulator input.  A workgroup is one wave: it owns 16 batch rows and a segment of groups, and the LDS
// holds three such workgroups per CU, so no two waves touch a cell and the order of the sums is fixed.
// Tile st covers slots SPL l16 + st of a chunk of 16 SPL, so that one 16-byte load of a label's row
// brings a lane's weights of all tiles.  The loads run three steps ahead; the segments' partials are
// summed in index order.
// ---------------------------------------------------------------------------------------------
__host__ __device__ constexpr int f32_bx_lds(int F_s) { return (F_s + 1) * 64; }

// VEC: F_in is a multiple of 4.  VY: G and L are.
template <bool VEC, bool VY>
__global__ __launch_bounds__(64) void k_bwd_x_f32(const int32_t *__restrict__ idx, const float *__restrict__ W,
                                                  const float *__restrict__ dY, float *__restrict__ part, int B, int Bp,
                                                  int F_s, int64_t L, int G, int F_in, int64_t K, int64_t gps, int nbt) {
    extern __shared__ __align__(16) char acc32[];   // row f: 64 bytes, its 16-byte chunk c at c ^ ((f >> 2) & 3)
    constexpr int RING = 4;
    const int lane = threadIdx.x, l16 = lane & 15, q = lane >> 4;
    const int b0 = (int)(blockIdx.x % nbt) * 16;
    const int64_t seg = blockIdx.x / nbt;
    const int64_t k0 = seg * gps, k1 = k0 + gps < K ? k0 + gps : K;
    for (int e = lane; e < (F_s + 1) * 4; e += 64) *reinterpret_cast<float4 *>(acc32 + 16 * e) = make_float4(0, 0, 0, 0);
    float *pp = part + (size_t)seg * F_s * Bp + b0;
    const int nch = (F_in + 63) >> 6, nlt = (G + 15) >> 4;
    const int nst = nch * nlt;                    // steps per group: chunk by chunk, 16 labels at a time
    const int64_t n = k1 > k0 ? (k1 - k0) * nst : 0;
    const int rows = B - b0 < 16 ? B - b0 : 16;
    struct Step {
        uint4 y, w[4], f;                         // dY of labels 4q .. + 3 of row l16; W of label 4q + j; features
    };
    struct At {
        int64_t k;
        int c, lt;
    };
    auto advance = [&](At &a) {
        if (++a.lt == nlt) {
            a.lt = 0;
            if (++a.c == nch) {
                a.c = 0;
                ++a.k;
            }
        }
    };
    auto load = [&](const At &a, Step &s) {
        const bool in = a.k < k1;                 // past the segment: all zeros
        const int64_t k = in ? a.k : k0;
        const int l = 16 * a.lt + 4 * q, t = 64 * a.c + 4 * l16;
        const int nv = in ? F_in - t : 0;
        const Buf yb(dY + (int64_t)b0 * L + k * G, (uint32_t)(((int64_t)(rows - 1) * L + G) * 4));
        s.y = load4<VY>(yb, (uint32_t)(((int64_t)l16 * L + l) * 4), in && l16 < rows ? G - l : 0);
        const Buf wb(W + k * G * F_in, (uint32_t)((int64_t)G * F_in * 4));   // labels past the group: zero
#pragma unroll
        for (int j = 0; j < 4; ++j) s.w[j] = load4<VEC>(wb, (uint32_t)(((l + j) * F_in + t) * 4), nv);
        const Buf ib(idx + k * F_in, (uint32_t)(F_in * 4));
        s.f = load4<VEC>(ib, (uint32_t)(t * 4), nv);
    };
    At ld{k0, 0, 0}, at{k0, 0, 0};
    Step ring[RING];
#pragma unroll
    for (int i = 0; i < RING - 1; ++i) {
        load(ld, ring[i]);
        advance(ld);
        __builtin_amdgcn_sched_barrier(0);
    }
    f32x4_t d[4];
    char *ao[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        d[i] = f32x4_t{0, 0, 0, 0};
        ao[i] = acc32;
    }
    __syncthreads();
    auto step = [&](const Step &s, Step &next) {
        load(ld, next);
        advance(ld);
        __builtin_amdgcn_sched_barrier(0);
        if (at.lt == 0) {                         // wave-uniform: a chunk begins
            const uint32_t fs[4] = {s.f.x, s.f.y, s.f.z, s.f.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                // slots past the support (and steps past the segment) meet the row nothing reads
                const uint32_t f = at.k < k1 && 64 * at.c + 4 * l16 + i < F_in ? fs[i] : (uint32_t)F_s;
                ao[i] = acc32 + f * 64 + ((q ^ ((f >> 2) & 3)) << 4);
                d[i] = *reinterpret_cast<const f32x4_t *>(ao[i]);
            }
        }
        const uint32_t ys[4] = {s.y.x, s.y.y, s.y.z, s.y.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t ws[4] = {s.w[j].x, s.w[j].y, s.w[j].z, s.w[j].w};
#pragma unroll
            for (int i = 0; i < 4; ++i) d[i] = mfma16x16x4(__uint_as_float(ys[j]), __uint_as_float(ws[i]), d[i]);
        }
        if (at.lt == nlt - 1) {                   // wave-uniform: it ends
#pragma unroll
            for (int i = 0; i < 4; ++i) *reinterpret_cast<f32x4_t *>(ao[i]) = d[i];
        }
        advance(at);
    };
    for (int64_t t = 0; t < n; t += RING) {
#pragma unroll
        for (int i = 0; i < RING; ++i) step(ring[i], ring[(i + RING - 1) % RING]);
    }
    __syncthreads();
    for (int e = lane; e < F_s * 4; e += 64) {
        const int f = e >> 2, c = e & 3;
        *reinterpret_cast<float4 *>(pp + (size_t)f * Bp + 4 * c) =
            *reinterpret_cast<const float4 *>(acc32 + f * 64 + ((c ^ ((f >> 2) & 3)) << 4));
    }
}

int64_t f32_units(const haste::TailArgs &a) { return a.L / a.G * haste::cdiv(a.G, 16); }

struct F32BxGeom {
    int nbt;
    int64_t nseg, gps;
};

F32BxGeom f32_bx_geom(const haste::TailArgs &a) {
    F32BxGeom g;
    g.nbt = (int)haste::cdiv(a.B, 16);
    // as many one-wave workgroups as the LDS of the chip holds, and at least 8 groups each
    const int64_t per_cu = 160 * 1024 / f32_bx_lds((int)a.F_s);
    int64_t nseg = kXcds * kCusPerXcd * per_cu / g.nbt;
    const int64_t most = haste::cdiv(a.L / a.G, 8);
    if (nseg > most) nseg = most;
    g.nseg = nseg < 1 ? 1 : nseg;
    g.gps = haste::cdiv(a.L / a.G, g.nseg);
    return g;
}

template <typename K>
hipError_t lds_limit(K k, int bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

}  // namespace

namespace haste {

// fp32; a group's weights, and 16 rows of dY, within the 31-bit range of a buffer offset
static bool f32_shape(const TailArgs &a) {
    return a.dtype == HASTE_DTYPE_F32 && a.F_in <= 256 && a.F_s <= kMaxFs &&
           (a.G + 16) * a.F_in * 4 < ((int64_t)1 << 31);
}

struct F32FwdGeom {
    int nbt;
    int64_t nunit, nseg, ups;
};

static F32FwdGeom f32_fwd_geom(const TailArgs &a) {
    F32FwdGeom g;
    g.nbt = (int)cdiv(a.B, 32);
    g.nunit = f32_units(a);
    g.nseg = round_up(cdiv(kXcds * kCusPerXcd, g.nbt), kXcds);
    const int64_t most = round_up(cdiv(g.nunit, kF32Waves), kXcds);
    if (g.nseg > most) g.nseg = most;
    g.ups = round_up(cdiv(g.nunit, g.nseg), kF32Waves);
    return g;
}

// a workgroup stages its slab of X^T, then every wave takes one unit after the other, chunk by chunk
double fwd_f32_us(const TailArgs &a) {
    const F32FwdGeom g = f32_fwd_geom(a);
    const int64_t nseg = cdiv(g.nunit, g.ups), fit = 160 * 1024 / f32_fwd_lds((int)a.F_s);
    const double R = xcd_rounds(nseg, g.nbt, 1), Rp = xcd_rounds(nseg, g.nbt, fit < 1 ? 1 : fit > 4 ? 4 : fit);
    const double S = (double)(g.ups / kF32Waves), ch = (double)cdiv(a.F_in, 64);
    return 1.7 + Rp * (2.4 + 0.012 * a.F_s + 0.37 * S * ch) +
           R * S * (0.3 * cdiv(a.F_in, 16) + (a.F_in % 4 ? 0.36 * ch : 0.0) + (a.G % 4 ? 0.27 : 0.0)) + 1.0e-6 * a.B * a.L;
}

// Groups of 1 or 2 labels leave most of a 16-label unit empty, and the vector ALUs are then as fast
// (131K labels, 64 slots, 128 rows, us: G = 1 / 2 / 4 / 8 / 16: 357 / 302 / 218 / 211 / 207 on the vector
// ALUs, 495 / 260 / 143 / 79 / 50 here).  Larger ones with few slots (G = 3, 8 slots of 128 features, 194K
// labels, 168 rows: 47 there, 320 here) or few units per workgroup (1064 rows, 816 labels, 32 slots of
// 768: 18 and 34) too: the estimates decide (of 1210 random layers 217 more than 6% slower here than there
// without them, 38 with them).
bool fwd_f32_preferred(const TailArgs &a) {
    return a.G > 2 && f32_shape(a) && valu_supported(a) && f32_fwd_lds((int)a.F_s) <= 160 * 1024 && fwd_f32_us(a) < fwd_valu_us(a);
}

hipError_t fwd_f32(const TailArgs &a, const void *X, const int32_t *idx, const void *W, const float *bias, void *Y,
                   hipStream_t s) {
    const int lds = f32_fwd_lds((int)a.F_s);
    const F32FwdGeom g = f32_fwd_geom(a);
    auto go = [&](auto kern) {
        hipError_t e = lds_limit(kern, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)(g.nseg * g.nbt)), dim3(512), lds, s, (const float *)X, idx, (const float *)W,
                           bias, (float *)Y, (int)a.B, (int)a.F_s, a.L, (int)a.G, (int)a.F_in, (int)cdiv(a.G, 16), g.nunit, g.ups,
                           g.nbt);
        return hipGetLastError();
    };
    const bool vst = a.G % 4 == 0;                // L then is too, and every unit starts at a multiple of 4
    if (a.F_in % 4 == 0) return vst ? go(k_fwd_f32<true, true>) : go(k_fwd_f32<true, false>);
    return vst ? go(k_fwd_f32<false, true>) : go(k_fwd_f32<false, false>);
}

static int f32_bw_nst(const TailArgs &a) { return a.F_in <= 32 ? 2 : a.F_in <= 64 ? 4 : a.F_in <= 128 ? 8 : 16; }

// a workgroup sweeps the batch in slabs of 32 rows for 8 or 16 units
double bwd_w_f32_us(const TailArgs &a) {
    const int nst = f32_bw_nst(a), xi = a.F_s <= 512 ? 8 : a.F_s <= 768 ? 12 : 16;
    const double R = (double)cdiv(cdiv(f32_units(a), kF32Waves * f32_bw_upw(nst)), 256);
    return 2.5 + R * (1.3 + 0.13 * nst + cdiv(a.B, 32) * (0.88 + 0.18 * nst + 0.21 * xi)) + 0.35e-6 * a.B * a.L + 0.53e-6 * a.L * a.F_in;
}

// (as above: 444 / 424 / 331 / 405 / 405 on the vector ALUs, about 600 / 345 / 179 / 96 / 55 here; G = 2 with 32
// slots 182 there, 193 here; G = 3 with 8 slots of 128 features, 194K labels, 168 rows 56 there, 307 here)
bool bwd_w_f32_preferred(const TailArgs &a) {
    return (a.G > 2 || (a.G == 2 && a.F_in > 32)) && f32_shape(a) && valu_supported(a) && f32_bw_lds((int)a.F_s) <= 160 * 1024 &&
           bwd_w_f32_us(a) < bwd_w_valu_us(a);
}

hipError_t bwd_w_f32(const TailArgs &a, const void *X, const int32_t *idx, const void *dY, float *dW, float *dbias,
                     int beta, hipStream_t s) {
    const int lds = f32_bw_lds((int)a.F_s);
    const int64_t nunit = f32_units(a);
    auto go = [&](auto kern, int upw) {
        hipError_t e = lds_limit(kern, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)cdiv(nunit, kF32Waves * upw)), dim3(512), lds, s, (const float *)X, idx,
                           (const float *)dY, dW, dbias, beta, (int)a.B, (int)a.F_s, a.L, (int)a.G, (int)a.F_in,
                           (int)cdiv(a.G, 16), nunit);
        return hipGetLastError();
    };
    auto wide = [&](auto nst) {
        constexpr int NST = decltype(nst)::value;
        if (a.F_s <= 512) return go(k_bwd_w_f32<NST, 8>, f32_bw_upw(NST));
        if (a.F_s <= 768) return go(k_bwd_w_f32<NST, 12>, f32_bw_upw(NST));
        return go(k_bwd_w_f32<NST, 16>, f32_bw_upw(NST));
    };
    switch (f32_bw_nst(a)) {
        case 2: return wide(std::integral_constant<int, 2>{});
        case 4: return wide(std::integral_constant<int, 4>{});
        case 8: return wide(std::integral_constant<int, 8>{});
    }
    return wide(std::integral_constant<int, 16>{});
}

// a one-wave workgroup takes its groups one after the other, 64 slots and 16 labels a step, slower the more
// waves share its CU
double bwd_x_f32_us(const TailArgs &a) {
    const F32BxGeom g = f32_bx_geom(a);
    const int64_t wgs = g.nseg * g.nbt, fit = 160 * 1024 / f32_bx_lds((int)a.F_s), occ = cdiv(wgs, 256) < fit ? cdiv(wgs, 256) : fit;
    const double R = (double)cdiv(wgs, 256 * fit), chunks = (double)(g.gps * cdiv(a.F_in, 64)), odd = a.F_in % 4 ? 1.0 : 0.0;
    return R * (7.6 + 0.0044 * a.F_s + chunks * (0.21 + cdiv(a.G, 16) * (0.26 + 0.067 * odd + (0.086 + 0.052 * odd) * occ))) +
           0.3e-6 * bwd_x_f32_ws(a);
}

// (as above: 512 / 516 / 517 / 513 / 510 on the vector ALUs, 1032 / 525 / 255 / 141 / 82 here.)  A segment is
// at least 8 groups, so layers of few large groups have few workgroups with long chains (275 rows, 952 labels,
// G = 119, 195 slots of 256: 53 there, 155 here; of 1210 random layers 40 more than 6% slower here than there
// without the estimates, 11 with them).
bool bwd_x_f32_preferred(const TailArgs &a) {
    return a.G > 2 && f32_shape(a) && valu_supported(a) && (a.L * 15 + a.G) * 4 < ((int64_t)1 << 31) &&
           bwd_x_f32_us(a) < bwd_x_valu_us(a);
}

size_t bwd_x_f32_ws(const TailArgs &a) {
    const F32BxGeom g = f32_bx_geom(a);
    return (size_t)g.nseg * (size_t)a.F_s * (size_t)(g.nbt * 16) * 4;
}

hipError_t bwd_x_f32(const TailArgs &a, const int32_t *idx, const void *W, const void *dY, float *dX, int beta, void *ws,
                     hipStream_t s) {
    const F32BxGeom g = f32_bx_geom(a);
    const int lds = f32_bx_lds((int)a.F_s);
    float *part = reinterpret_cast<float *>(ws);
    auto go = [&](auto kern) {
        hipError_t e = lds_limit(kern, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)(g.nseg * g.nbt)), dim3(64), lds, s, idx, (const float *)W, (const float *)dY,
                           part, (int)a.B, g.nbt * 16, (int)a.F_s, a.L, (int)a.G, (int)a.F_in, a.L / a.G, g.gps, g.nbt);
        return hipGetLastError();
    };
    const bool vy = a.G % 4 == 0;
    hipError_t e;
    if (a.F_in % 4 == 0) e = vy ? go(k_bwd_x_f32<true, true>) : go(k_bwd_x_f32<true, false>);
    else e = vy ? go(k_bwd_x_f32<false, true>) : go(k_bwd_x_f32<false, false>);
    if (e != hipSuccess) return e;
    return reduce_fmajor(part, (int)g.nseg, g.nbt * 16, a.B, a.F_s, dX, beta, s);
}

}  // namespace haste
