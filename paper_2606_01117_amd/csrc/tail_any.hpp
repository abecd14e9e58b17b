// Backward-feature as a dense matrix-core product over scattered weight tiles, for groups of any
// size and supports of any width (bf16).
//
//   dX[rows, f] = sum over labels l of dY[rows, l] W'[l, f],   W'[l, f] = W[l, t] where
//   idx[g(l), t] = f, and 0 where f is not in the support of l's group   (Section 3.2, the
//   backward-feature product; W' is the weight grid of Fig. 2 (d) with its empty cells as zeros).
//
// A workgroup owns 16 MT batch rows and FR features (dX^T [FR][16 MT] fp32 in the matrix-core
// accumulators) for a segment of labels, which it takes in steps of 32:
//   - four producer waves clear the cells that an earlier step left in a [FR][32 labels] bf16 tile in
//     LDS, write the step's weights into it (W'[l, idx[g(l), t]] = W[l, t]) and stage the step's dY;
//   - four consumer waves (one per SIMD, each beside a producer) form D += A B with A = dY[16 MT
//     rows][32 labels] and B = the tile, v_mfma_f32_16x16x32_bf16, FR / 64 feature tiles each.
// Three tiles rotate, with one barrier per step: the one being read, the next one being written, and
// the previous one, whose reads may still be in flight at the barrier (so the consumers wait there
// for the producers only).  The consumers' reads run three feature tiles ahead of their products,
// across the barrier too.
//
// The product does F_s / F_in times the multiply-adds the layer needs, and its cost does not
// depend on the groups: it replaces accumulators in LDS, whose read-add-write costs 8 bytes per
// (group, slot, row), where those are wider than the dense product is long.  Labels of one group
// share their features, so PK of them (the largest power of two up to 8 that divides G) go into
// the tile with one write per slot, 2 PK bytes.
#pragma once

#include "common.hpp"

namespace {

typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) uint16_t lds_u16_t;
typedef __attribute__((address_space(3))) uint32_t lds_u32_t;
typedef __attribute__((address_space(3))) u32x2_t lds_u32x2_t;
typedef __attribute__((address_space(3))) u32x4_t lds_u32x4_t;
typedef __attribute__((address_space(3))) bf16x8_t lds_bf16x8_t;

constexpr int kAxCons = 4;                        // consumer waves
constexpr int kAxThreads = 64 * (kAxCons + 4);    // and four producers
constexpr int kAxStageRow = 80;                   // bytes per staged dY row: 32 labels + pad
// steps whose loads are in flight per producer lane (16 slot pairs a lane leave registers for one,
// and their step is long enough to cover a load's latency)
__host__ __device__ constexpr int ax_ring(int ni) { return ni <= 8 ? 3 : 1; }

// three tiles of 64-byte rows, three staged dY steps, and a spare cell for writes of no slot (cheaper
// than lane masks around the writes: 196 against 201 us on 655K labels in groups of 4)
__host__ __device__ constexpr int ax_lds(int fr, int mt) { return 3 * fr * 64 + 3 * 16 * mt * kAxStageRow + 64; }

// How dY rows (8 labels per lane) and weight pairs are read: 16 bytes and a dword where dY's rows
// are 16-byte aligned (L a multiple of 8) and F_in is even; dwords where L and F_in are even; 2
// bytes at a time otherwise.
constexpr int kRead16 = 0, kRead4 = 1, kRead2 = 2;

// x / d for a run-time d, as a multiply-high by mul = ceil(2^32 / d) (x d < 2^32); mul = 0: d is 1
__device__ __forceinline__ uint32_t div_by(uint32_t x, uint32_t mul) { return mul ? __umulhi(x, mul) : x; }

// 8 bf16 at byte offset o of which the first nv may be read (others: zero)
template <int READ>
__device__ __forceinline__ u32x4_t load_row8(const Buf &b, uint32_t o, int64_t nv) {
    if constexpr (READ == kRead16) {
        return __builtin_bit_cast(u32x4_t, b.ld16(nv > 0 ? o : kOob));
    } else if constexpr (READ == kRead4) {
        u32x4_t v;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = b.ld4(nv > 2 * k ? o + 4 * k : kOob);
        return v;
    } else {
        u32x4_t v;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            v[k] = (uint32_t)b.ld2(nv > 2 * k ? o + 4 * k : kOob) | ((uint32_t)b.ld2(nv > 2 * k + 1 ? o + 4 * k + 2 : kOob) << 16);
        return v;
    }
}

// MT: 16-row tiles per workgroup.  NFT: 16-feature tiles per consumer wave (tiles w, w + 4, ...).
// PK: labels per tile write.  NI: slot pairs per producer lane and step (32 / PK packs of
// ceil(F_in / 2) pairs over 256 lanes).  READ: as above.  The workgroup covers features f0 .. f0 +
// FR - 1 of the layer's (all of them, or one of nsplit shares).
template <int MT, int NFT, int PK, int NI, int READ>
__global__ __attribute__((amdgpu_flat_work_group_size(kAxThreads, kAxThreads), amdgpu_waves_per_eu(2, 2)))
void k_bwd_x_any(const int32_t *__restrict__ idx, const bf16_t *__restrict__ W, const bf16_t *__restrict__ dY,
                 float *__restrict__ part, int B, int Bp, int F_s, int64_t L, int G, uint32_t gmul, int F_in, int nbt,
                 int nsplit, int64_t lps) {
    constexpr int FR = 16 * kAxCons * NFT;
    constexpr int TB = FR * 64;                   // bytes of a tile
    constexpr int SB = 16 * MT * kAxStageRow;     // bytes of a staged dY step
    constexpr int RW = 16 * MT;
    extern __shared__ __align__(16) char ax[];
    const int w = blockIdx.x, xcd = w % kXcds;
    int jj = w / kXcds;
    const int bt = jj % nbt;
    jj /= nbt;
    const int f0 = (jj % nsplit) * FR;
    const int64_t seg = (int64_t)(jj / nsplit) * kXcds + xcd;
    const int b0 = bt * RW;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, q = lane >> 4;
    const int nf = F_s - f0 < FR ? F_s - f0 : FR;   // the workgroup's features
    float *pp = part + ((size_t)seg * F_s + f0) * Bp + b0;
    const int64_t l_begin = seg * lps;
    const int64_t l_end = l_begin + lps < L ? l_begin + lps : L;
    if (l_begin >= l_end) {                       // empty segment: the partial is zero (workgroup-uniform)
        for (int e = tid; e < nf * RW; e += kAxThreads) pp[(size_t)(e / RW) * Bp + (e % RW)] = 0.0f;
        return;
    }
    const int n = (int)((l_end - l_begin + 63) / 64) * 2;   // steps (even: those past the end add zeros)
    const uint32_t lbase = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)ax;
    const uint32_t sbase = lbase + 3 * TB;
    for (int e = tid; e < 3 * TB / 16; e += kAxThreads) *(lds_u32x4_t *)(uintptr_t)(lbase + 16 * e) = u32x4_t{0u, 0u, 0u, 0u};
    __syncthreads();                              // tiles zeroed

    if (wave >= kAxCons) {
        // ---- producers ----
        constexpr uint32_t kNone = 3 * TB + 3 * SB;   // the spare cell, as an offset from the first tile
        const int pt = tid - 64 * kAxCons;
        // Wave wv writes labels 8 wv .. 8 wv + 7 of every step, one 16-byte chunk of each tile row (with
        // random features and the chunk swizzle those cells lie in all of a tile's banks), so that its
        // clears and writes of a cell are ordered by its own program order.  This lane: the pack of
        // labels lo .. lo + PK - 1, slots sl[i] and sl[i] + 1 (-2: none).
        constexpr int LPK = 8 * PK;               // lanes of one pack
        const int wv = pt >> 6;
        const int lo = 8 * wv + lane / LPK * PK;
        int sl[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int p = lane % LPK + LPK * i;
            sl[i] = 2 * p < F_in ? 2 * p : -2;
        }
        const Buf wseg(W + l_begin * F_in, (uint32_t)((l_end - l_begin) * F_in * 2));
        const int64_t g0 = l_begin / G;
        const uint32_t r0 = (uint32_t)(l_begin - g0 * G);   // labels of group g0 before the segment
        const int64_t g_end = (l_end + G - 1) / G;
        const Buf iseg(idx + g0 * F_in, (uint32_t)((g_end - g0) * F_in * 4));
        // dY: lane -> row pt / 4 of 64 (MT = 2: row pt / 4 of 32, lanes past them none), 8 labels
        const int rows = B - b0 < RW ? B - b0 : RW;
        const int dr = pt >> 2, dp = pt & 3;
        const bool ylane = dr < RW;
        const Buf dseg(dY + (int64_t)b0 * L, (uint32_t)((int64_t)rows * L * 2));
        const uint32_t yst = sbase + (uint32_t)(dr * kAxStageRow + 16 * dp);

        struct Slot {
            uint32_t w[NI][PK];
            int32_t f[NI][2];
            u32x4_t y;
        };
        constexpr int RD = ax_ring(NI);
        Slot rg[RD];
        auto load_step = [&](int st, Slot &r) __attribute__((always_inline)) {
            const uint32_t lr = (uint32_t)(st * 32 + lo);
            const uint32_t wo = lr * (uint32_t)F_in * 2u, io0 = div_by(lr + r0, gmul) * (uint32_t)F_in * 4u;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const bool ok = sl[i] >= 0;
#pragma unroll
                for (int j = 0; j < PK; ++j) {
                    const uint32_t o = wo + (uint32_t)(j * F_in + sl[i]) * 2u;
                    if constexpr (READ == kRead2) r.w[i][j] = (uint32_t)wseg.ld2(ok ? o : kOob) | ((uint32_t)wseg.ld2(ok ? o + 2 : kOob) << 16);
                    else r.w[i][j] = wseg.ld4(ok ? o : kOob);
                }
                const uint32_t io = ok ? io0 + (uint32_t)sl[i] * 4u : kOob;
                if constexpr (READ == kRead2) {
                    r.f[i][0] = (int32_t)iseg.ld4(io);
                    r.f[i][1] = (int32_t)iseg.ld4(ok ? io + 4 : kOob);
                } else {
                    const uint2 v = iseg.ld8(io);
                    r.f[i][0] = (int32_t)v.x;
                    r.f[i][1] = (int32_t)v.y;
                }
            }
            const int64_t lab = l_begin + (int64_t)st * 32 + 8 * dp;
            r.y = load_row8<READ>(dseg, (uint32_t)(((int64_t)dr * L + lab) * 2), dr < rows ? l_end - lab : 0);
        };
        // offsets from the tile's base of the cells written by a step, to be cleared three steps later
        // (a pair of slots per word: a tile is less than 64 KiB)
        uint32_t ca[3][NI];
        const uint32_t lcol = (uint32_t)((lo >> 3) << 4 | (lo & 7) << 1);   // chunk and label of the pack
        auto cell = [&](int32_t f) __attribute__((always_inline)) -> uint32_t {
            const uint32_t fr = (uint32_t)(f - f0);
            return (fr << 6) | (lcol ^ ((fr << 2) & 0x30u));
        };
        auto put = [&](uint32_t a, const uint32_t (&v)[PK / 2 > 0 ? PK / 2 : 1]) __attribute__((always_inline)) {
            if constexpr (PK == 1) *(lds_u16_t *)(uintptr_t)a = (uint16_t)v[0];
            else if constexpr (PK == 2) *(lds_u32_t *)(uintptr_t)a = v[0];
            else if constexpr (PK == 4) *(lds_u32x2_t *)(uintptr_t)a = u32x2_t{v[0], v[1]};
            else *(lds_u32x4_t *)(uintptr_t)a = u32x4_t{v[0], v[1], v[2], v[3]};
        };
        constexpr uint32_t kNo = 0xffffu;          // no cell (a tile's last byte is never a cell's first)
        auto scatter = [&](const Slot &r, int tb, uint32_t (&c)[NI]) __attribute__((always_inline)) {
            const uint32_t base = lbase + (uint32_t)(tb * TB);
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                uint32_t v0[PK / 2 > 0 ? PK / 2 : 1], v1[PK / 2 > 0 ? PK / 2 : 1];
                if constexpr (PK == 1) {
                    v0[0] = r.w[i][0];
                    v1[0] = r.w[i][0] >> 16;
                } else {
#pragma unroll
                    for (int j = 0; j < PK / 2; ++j) {
                        v0[j] = __builtin_amdgcn_perm(r.w[i][2 * j + 1], r.w[i][2 * j], 0x05040100u);
                        v1[j] = __builtin_amdgcn_perm(r.w[i][2 * j + 1], r.w[i][2 * j], 0x07060302u);
                    }
                }
                const bool ok0 = sl[i] >= 0 && (uint32_t)(r.f[i][0] - f0) < (uint32_t)FR;
                const bool ok1 = sl[i] >= 0 && (uint32_t)(r.f[i][1] - f0) < (uint32_t)FR &&
                                 (READ != kRead2 || sl[i] + 1 < F_in);
                const uint32_t c0 = ok0 ? cell(r.f[i][0]) : kNo, c1 = ok1 ? cell(r.f[i][1]) : kNo;
                c[i] = c0 | (c1 << 16);
                put(ok0 ? base + c0 : lbase + kNone, v0);
                put(ok1 ? base + c1 : lbase + kNone, v1);
            }
        };
        auto clear = [&](int tb, const uint32_t (&c)[NI]) __attribute__((always_inline)) {
            const uint32_t base = lbase + (uint32_t)(tb * TB);
            const uint32_t z[PK / 2 > 0 ? PK / 2 : 1] = {};
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const uint32_t c0 = c[i] & 0xffffu, c1 = c[i] >> 16;
                put(c0 != kNo ? base + c0 : lbase + kNone, z);
                put(c1 != kNo ? base + c1 : lbase + kNone, z);
            }
        };
        auto stage_y = [&](const Slot &r, int sb) __attribute__((always_inline)) {
            if (ylane) *(lds_u32x4_t *)(uintptr_t)(yst + (uint32_t)(sb * SB)) = r.y;
        };
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int i = 0; i < NI; ++i) ca[k][i] = kNo | (kNo << 16);
        // step s waits in ring slot s mod RD, is written into tile and stage s mod 3, and leaves its
        // cells in ca[s mod 3]
#pragma unroll
        for (int k = 0; k < RD; ++k) {
            load_step(k, rg[k]);
            __builtin_amdgcn_sched_barrier(0);
        }
        scatter(rg[0], 0, ca[0]);
        stage_y(rg[0], 0);
        load_step(RD, rg[0]);
        __syncthreads();                          // step 0 in its tile
        // interval t: tile (t + 1) mod 3, last read in interval t - 2, loses step t - 2 and takes step t + 1
        auto interval = [&](int t, auto uc) __attribute__((always_inline)) {
            constexpr int N = (decltype(uc)::value + 1) % 3;
            clear(N, ca[N]);
            scatter(rg[N % RD], N, ca[N]);
            stage_y(rg[N % RD], N);
            __builtin_amdgcn_sched_barrier(0);
            load_step(t + 1 + RD, rg[N % RD]);
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
        };
        for (int t = 0; t < n; t += 3) {
            interval(t, std::integral_constant<int, 0>{});
            if (t + 1 >= n) break;
            interval(t + 1, std::integral_constant<int, 1>{});
            if (t + 2 >= n) break;
            interval(t + 2, std::integral_constant<int, 2>{});
        }
        return;
    }

    // ---- consumers ----
    __builtin_amdgcn_s_setprio(2);
    f32x4_t acc[MT][NFT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int i = 0; i < NFT; ++i) acc[m][i] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    // A rows 16 m + l16, labels 8q .. 8q + 7 of the step; B rows 16 (wave + 4 i) + l16, chunk q
    const uint32_t aoff = sbase + (uint32_t)(l16 * kAxStageRow + 16 * q);
    const uint32_t boff = lbase + (uint32_t)(wave * 1024 + l16 * 64 + ((q ^ ((l16 >> 2) & 3)) << 4));
    constexpr int PD = 3, SC = 1024 * kAxCons;    // feature tiles read ahead; bytes from one to the next
    static_assert(NFT >= PD && 2 * NFT % 4 == 0, "ring of four operands over two steps");
    bf16x8_t oa[2][MT], ob[4];
    auto read_a = [&](uint32_t a, bf16x8_t (&o)[MT]) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < MT; ++m) o[m] = *(lds_bf16x8_t *)(uintptr_t)(a + 16 * m * kAxStageRow);
    };
    int sl3 = 0;                                  // the step's tile and stage
    __syncthreads();                              // step 0 in its tile
    read_a(aoff, oa[0]);
#pragma unroll
    for (int i = 0; i < PD; ++i) ob[i] = *(lds_bf16x8_t *)(uintptr_t)(boff + SC * i);
    auto step = [&](auto pc) __attribute__((always_inline)) {
        constexpr int P = decltype(pc)::value;
        const uint32_t bcur = boff + (uint32_t)(sl3 * TB);
        const int nx = sl3 == 2 ? 0 : sl3 + 1;
        const uint32_t bnext = boff + (uint32_t)(nx * TB);
#pragma unroll
        for (int i = 0; i < NFT; ++i) {
            if (i == NFT - PD) {
                // The next step is in its tile.  The reads of this one's need not have returned: its
                // tile is written again two barriers on, when its products have been issued.
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                read_a(aoff + (uint32_t)(nx * SB), oa[1 - P]);
            }
            ob[(P * NFT + i + PD) & 3] = i + PD < NFT ? *(lds_bf16x8_t *)(uintptr_t)(bcur + SC * (i + PD))
                                                      : *(lds_bf16x8_t *)(uintptr_t)(bnext + SC * (i + PD - NFT));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < MT; ++m)
                acc[m][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(oa[P][m], ob[(P * NFT + i) & 3], acc[m][i], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        sl3 = nx;
    };
    for (int t = 0; t < n; t += 2) {
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
    }
    // partial dX^T of the segment: lane (l16, q) of feature tile ft holds feature 16 ft + l16, rows
    // 16 m + 4q .. + 3
#pragma unroll
    for (int i = 0; i < NFT; ++i) {
        const int f = 16 * (wave + kAxCons * i) + l16;
        if (f < nf) {
#pragma unroll
            for (int m = 0; m < MT; ++m)
                *reinterpret_cast<float4 *>(pp + (size_t)f * Bp + 16 * m + 4 * q) =
                    make_float4(acc[m][i][0], acc[m][i][1], acc[m][i][2], acc[m][i][3]);
        }
    }
}

// Labels that share a tile write: the largest power of two that divides G, up to 8, or 4 where that
// gives every producer lane its slot pair (up to 64 slots; with 8 half of the lanes would write
// nothing: 118 against 107 us on 328K labels in groups of 8, and 124 against 142 with 128 slots).
// Segments start at multiples of 64 labels, so a step's packs never straddle groups.
inline int pack_of(int64_t G, int64_t F_in) {
    return G % 8 == 0 && F_in > 64 ? 8 : G % 4 == 0 ? 4 : G % 2 == 0 ? 2 : 1;
}

inline uint32_t div_mul(int64_t d) { return d == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); }

struct AxGeom {
    int mt, nft, nbt, nsplit, pk, ni;
    int64_t nseg, lps;
    size_t lds;
};

inline AxGeom ax_geom(const haste::TailArgs &a) {
    AxGeom g;
    g.mt = a.B > 32 ? 4 : 2;
    g.nbt = (int)haste::cdiv(a.B, 16 * g.mt);
    // three tiles of 768 features fill the LDS: wider inputs split their features over workgroups
    g.nsplit = (int)haste::cdiv(a.F_s, 768);
    const int64_t fr = haste::cdiv(a.F_s, g.nsplit);
    g.nft = g.mt == 4 && fr <= 512 ? 8 : 12;
    g.pk = pack_of(a.G, a.F_in);
    const int64_t items = (32 / g.pk) * haste::cdiv(a.F_in, 2), per = haste::cdiv(items, 256);
    // the instantiated counts of slot pairs per lane (0: more than the registers hold)
    static const int kNi[4][4] = {{4, 8, 16, 0}, {2, 4, 8, 0}, {1, 2, 4, 0}, {1, 2, 0, 0}};
    const int *ni = kNi[g.pk == 1 ? 0 : g.pk == 2 ? 1 : g.pk == 4 ? 2 : 3];
    while (*ni && *ni < per) ++ni;
    g.ni = *ni;
    // one workgroup per CU; a segment is at least 256 labels, so that the partials stay few
    int64_t nseg = haste::round_up(haste::cdiv(kXcds * kCusPerXcd, g.nbt * g.nsplit), kXcds);
    const int64_t max_seg = haste::round_up(haste::cdiv(a.L, 256), kXcds);
    g.nseg = nseg < max_seg ? nseg : max_seg;
    g.lps = haste::round_up(haste::cdiv(a.L, g.nseg), 64);
    g.lds = (size_t)ax_lds(16 * kAxCons * g.nft, g.mt);
    return g;
}

// one launch of the kernel for MT row tiles and NFT feature tiles
template <int MT, int NFT>
struct AxRun {
    const haste::TailArgs &a;
    const AxGeom &g;
    const int32_t *idx;
    const void *W, *dY;
    float *part;
    hipStream_t s;

    template <int PK, int NI, int READ>
    hipError_t go() const {
        auto kern = k_bwd_x_any<MT, NFT, PK, NI, READ>;
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)g.lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)(g.nseg * g.nbt * g.nsplit)), dim3(kAxThreads), g.lds, s, idx, (const bf16_t *)W,
                           (const bf16_t *)dY, part, (int)a.B, g.nbt * 16 * MT, (int)a.F_s, a.L, (int)a.G, div_mul(a.G),
                           (int)a.F_in, g.nbt, g.nsplit, g.lps);
        return hipGetLastError();
    }
    template <int PK, int NI>
    hipError_t read() const {
        if (a.F_in % 2 == 0) {
            if (a.L % 8 == 0 && (reinterpret_cast<uintptr_t>(dY) & 15) == 0) return go<PK, NI, kRead16>();
            if constexpr (PK < 8)
                if (a.L % 2 == 0) return go<PK, NI, kRead4>();
        }
        return go<PK, NI, kRead2>();
    }
    hipError_t run() const {
        switch (g.pk * 100 + g.ni) {
            case 104: return read<1, 4>();
            case 108: return read<1, 8>();
            case 116: return read<1, 16>();
            case 202: return read<2, 2>();
            case 204: return read<2, 4>();
            case 208: return read<2, 8>();
            case 401: return read<4, 1>();
            case 402: return read<4, 2>();
            case 404: return read<4, 4>();
            case 801: return read<8, 1>();
            case 802: return read<8, 2>();
        }
        return hipErrorInvalidValue;
    }
};

}  // namespace
