// Backward-feature and forward as dense matrix-core products over scattered weight tiles, for groups of
// any size and supports of any width (bf16).  Backward-feature first:
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

// three tiles of 64-byte rows, three staged dY steps, and 64 bytes: a spare cell for writes of no slot
// (cheaper than lane masks around the writes: 196 against 201 us on 655K labels in groups of 4), at
// kAxBad one bit per row whose dY is not finite somewhere, and at kAxFix what the pass over such rows
// needs (kept in registers, it would crowd the producers' loop)
__host__ __device__ constexpr int ax_lds(int fr, int mt) { return 3 * fr * 64 + 3 * 16 * mt * kAxStageRow + 160; }
constexpr int kAxBad = 32, kAxFix = 64;
struct AxFix {
    const int32_t *idx;
    const bf16_t *W, *dY;
    float *pp;
    int64_t L, l_begin, l_end;
    int b0, Bp, nf, f0, G, F_in;
};
static_assert(sizeof(AxFix) <= 96, "fits behind kAxFix");

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

// The producers' side of a [FR][32 labels] tile: four waves write a step's weights and clear an earlier
// step's.  Wave wv writes labels 8 wv .. 8 wv + 7 of every step, one 16-byte chunk of each tile row (with
// random features and the chunk swizzle those cells lie in all of a tile's banks), so that its clears
// and writes of a cell are ordered by its own program order.  A lane owns one pack of PK labels and NI
// slot pairs of their group.  SPARE: features outside f0 .. f0 + FR - 1 (and pairs past the support) are
// written to a spare cell at offset `none`; without it every feature lies in the tile, and lanes with
// no pair of their own repeat the last one.
template <int PK, int NI, int READ, int FR, bool SPARE>
struct AxTiles {
    static constexpr int TB = FR * 64;            // bytes of a tile
    static constexpr int LPK = 8 * PK;            // lanes of one pack
    static constexpr int NV = PK / 2 > 0 ? PK / 2 : 1;
    static constexpr uint32_t kNo = 0xffffu;      // no cell (a tile's last byte is never a cell's first)
    struct Slot {                                 // a step's loads
        uint32_t w[NI][PK];
        int32_t f[NI][2];
    };
    Buf wseg, iseg;
    uint32_t lbase, none, lcol, r0, gmul;
    int lo, F_in, f0;
    int sl[NI];                                   // the pairs' first slots (-2: none)

    // pt: producer thread 0 .. 255; the segment's labels are l_begin .. l_end - 1
    __device__ __forceinline__ AxTiles(const int32_t *idx, const bf16_t *W, int64_t l_begin, int64_t l_end, int G,
                                       uint32_t gmul_, int F_in_, int f0_, uint32_t lbase_, uint32_t none_, int pt)
        : wseg(W + l_begin * F_in_, (uint32_t)((l_end - l_begin) * F_in_ * 2)),
          iseg(idx + l_begin / G * F_in_, (uint32_t)(((l_end + G - 1) / G - l_begin / G) * F_in_ * 4)), lbase(lbase_),
          none(none_), r0((uint32_t)(l_begin % G)), gmul(gmul_), F_in(F_in_), f0(f0_) {
        const int lane = pt & 63;
        lo = 8 * (pt >> 6) + lane / LPK * PK;
        lcol = (uint32_t)((lo >> 3) << 4 | (lo & 7) << 1);
        const int last = (F_in - 1) & ~1;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int t = 2 * (lane % LPK + LPK * i);
            sl[i] = t <= last ? t : SPARE ? -2 : last;
        }
    }
    // step st of the segment; labels past its end have zero weights
    __device__ __forceinline__ void load(int st, Slot &r) const {
        const uint32_t lr = (uint32_t)(st * 32 + lo);
        const uint32_t wo = lr * (uint32_t)F_in * 2u, io0 = div_by(lr + r0, gmul) * (uint32_t)F_in * 4u;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const bool ok = !SPARE || sl[i] >= 0;
#pragma unroll
            for (int j = 0; j < PK; ++j) {
                const uint32_t o = wo + (uint32_t)(j * F_in + sl[i]) * 2u;
                if constexpr (READ == kRead2)
                    r.w[i][j] = (uint32_t)wseg.ld2(ok ? o : kOob) | ((uint32_t)wseg.ld2(ok ? o + 2 : kOob) << 16);
                else
                    r.w[i][j] = wseg.ld4(ok ? o : kOob);
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
    }
    __device__ __forceinline__ uint32_t cell(uint32_t fr) const { return (fr << 6) | (lcol ^ ((fr << 2) & 0x30u)); }
    __device__ __forceinline__ void put(uint32_t a, const uint32_t (&v)[NV]) const {
        if constexpr (PK == 1) *(lds_u16_t *)(uintptr_t)a = (uint16_t)v[0];
        else if constexpr (PK == 2) *(lds_u32_t *)(uintptr_t)a = v[0];
        else if constexpr (PK == 4) *(lds_u32x2_t *)(uintptr_t)a = u32x2_t{v[0], v[1]};
        else *(lds_u32x4_t *)(uintptr_t)a = u32x4_t{v[0], v[1], v[2], v[3]};
    }
    // Cells written by a step, as offsets from the tile's base, a pair of slots per word (a tile is less
    // than 64 KiB).  Before the first step: none, or this lane's own cell of feature 0 (still zero).
    __device__ __forceinline__ void no_cells(uint32_t (&c)[NI]) const {
#pragma unroll
        for (int i = 0; i < NI; ++i) c[i] = SPARE ? kNo | (kNo << 16) : lcol | (lcol << 16);
    }
    __device__ __forceinline__ void scatter(const Slot &r, int tb, uint32_t (&c)[NI]) const {
        const uint32_t base = lbase + (uint32_t)(tb * TB);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            uint32_t v0[NV], v1[NV];
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
            const bool two = READ != kRead2 || sl[i] + 1 < F_in;
            if constexpr (SPARE) {
                const uint32_t fa = (uint32_t)(r.f[i][0] - f0), fb = (uint32_t)(r.f[i][1] - f0);
                const bool ok0 = sl[i] >= 0 && fa < (uint32_t)FR, ok1 = sl[i] >= 0 && fb < (uint32_t)FR && two;
                const uint32_t c0 = ok0 ? cell(fa) : kNo, c1 = ok1 ? cell(fb) : kNo;
                c[i] = c0 | (c1 << 16);
                put(ok0 ? base + c0 : none, v0);
                put(ok1 ? base + c1 : none, v1);
            } else {
                const uint32_t fa = min((uint32_t)r.f[i][0], (uint32_t)(FR - 1));
                const uint32_t fb = two ? min((uint32_t)r.f[i][1], (uint32_t)(FR - 1)) : fa;
                if (!two)
#pragma unroll
                    for (int j = 0; j < NV; ++j) v1[j] = v0[j];
                const uint32_t c0 = cell(fa), c1 = cell(fb);
                c[i] = c0 | (c1 << 16);
                put(base + c0, v0);
                put(base + c1, v1);
            }
        }
    }
    __device__ __forceinline__ void clear(int tb, const uint32_t (&c)[NI]) const {
        const uint32_t base = lbase + (uint32_t)(tb * TB);
        const uint32_t z[NV] = {};
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const uint32_t c0 = c[i] & 0xffffu, c1 = c[i] >> 16;
            put(SPARE && c0 == kNo ? none : base + c0, z);
            put(SPARE && c1 == kNo ? none : base + c1, z);
        }
    }
};

// All threads of the workgroup: adds to its stored partial pp[f][row] the products of the elements of dY
// that are not finite, of the marked rows.  32 rows at a time sum in LDS (the tiles' space); a wave takes
// every eighth run of 64 labels.
template <int MT, int FR>
__device__ __forceinline__ void ax_add_not_finite(char *lds, const AxFix *fix, const uint32_t *bad) {
    const AxFix x = *fix;
    float *sum = reinterpret_cast<float *>(lds);   // [32 rows][FR]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int r0 = 0; r0 < 16 * MT; r0 += 32) {
        const uint32_t mask = bad[r0 >> 5];
        if (mask == 0u) continue;                 // workgroup-uniform
        for (int e = tid; e < 32 * FR; e += kAxThreads) sum[e] = 0.0f;
        __syncthreads();
        for (uint32_t m = mask; m != 0u; m &= m - 1u) {
            const int r = __builtin_ctz(m);
            const bf16_t *y = x.dY + (int64_t)(x.b0 + r0 + r) * x.L;
            for (int64_t l0 = x.l_begin + 64 * wave; l0 < x.l_end; l0 += kAxThreads) {
                const bf16_t v = l0 + lane < x.l_end ? y[l0 + lane] : (bf16_t)0;
                for (uint64_t at = __ballot((v & 0x7f80) == 0x7f80); at != 0u; at &= at - 1u) {
                    const int j = (int)__builtin_ctzll(at);
                    const int64_t l = l0 + j;
                    const float yv = bf16_to_f32((bf16_t)__builtin_amdgcn_readlane((int)v, j));
                    for (int t = lane; t < x.F_in; t += 64) {
                        const int f = x.idx[l / x.G * x.F_in + t] - x.f0;
                        if (f >= 0 && f < x.nf) atomicAdd(&sum[r * FR + f], yv * bf16_to_f32(x.W[l * x.F_in + t]));
                    }
                }
            }
        }
        __syncthreads();
        for (int e = tid; e < 32 * x.nf; e += kAxThreads) {
            const int r = e & 31, f = e >> 5;
            if ((mask >> r) & 1u) x.pp[(size_t)f * x.Bp + r0 + r] += sum[r * FR + f];
        }
        __syncthreads();
    }
}

// An empty cell of the tile contributes dY times zero, which is zero only for finite dY.  So an infinity
// or a NaN of dY is staged as the smallest normal number of its sign (which leaves zero cells zero, and
// infinite and NaN weights what they are) and its row marked, and in a workgroup with marked rows all waves
// go over those rows of dY once more and add each such element's own products, feature by feature.  What
// they sum to is an infinity or a NaN in any order.  (The test costs a producer lane 11 instructions a
// step.)
//
// MT: 16-row tiles per workgroup.  NFT: 16-feature tiles per consumer wave (tiles w, w + 4, ...).
// PK: labels per tile write.  NI: slot pairs per producer lane and step (32 / PK packs of
// ceil(F_in / 2) pairs over 256 lanes).  READ: as above.  The workgroup covers features f0 .. f0 +
// FR - 1 of the layer's (all of them, or one of nsplit shares).
template <int MT, int NFT, int PK, int NI, int READ>
__global__ __attribute__((amdgpu_flat_work_group_size(kAxThreads, kAxThreads), amdgpu_waves_per_eu(2, 2)))
void k_bwd_x_any(const int32_t *__restrict__ idx, const bf16_t *__restrict__ W, const bf16_t *__restrict__ dY,
                 float *__restrict__ part, int B, int Bp, int F_s, int64_t L, int G, uint32_t gmul, int F_in, int nbt,
                 int nsplit, int64_t nseg, int64_t lps) {
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
    if (seg >= nseg) return;                      // workgroup-uniform (the grid holds whole rows of 8 segments)
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
    uint32_t *bad = reinterpret_cast<uint32_t *>(ax + 3 * TB + 3 * SB + kAxBad);   // [2]: one bit per row
    AxFix *fix = reinterpret_cast<AxFix *>(ax + 3 * TB + 3 * SB + kAxFix);
    if (tid < 2) bad[tid] = 0u;
    if (tid == 0) *fix = AxFix{idx, W, dY, pp, L, l_begin, l_end, b0, Bp, nf, f0, G, F_in};
    __syncthreads();                              // tiles zeroed
    const int rows = B - b0 < RW ? B - b0 : RW;

    if (wave >= kAxCons) {
        // ---- producers ----
        const int pt = tid - 64 * kAxCons;
        using Tiles = AxTiles<PK, NI, READ, FR, true>;
        const Tiles tl(idx, W, l_begin, l_end, G, gmul, F_in, f0, lbase, lbase + 3 * TB + 3 * SB, pt);
        // dY: lane -> row pt / 4 of 64 (MT = 2: row pt / 4 of 32, lanes past them none), 8 labels
        const int dr = pt >> 2, dp = pt & 3;
        const bool ylane = dr < RW;
        const Buf dseg(dY + (int64_t)b0 * L, (uint32_t)((int64_t)rows * L * 2));
        const uint32_t yst = sbase + (uint32_t)(dr * kAxStageRow + 16 * dp);

        struct Slot {
            typename Tiles::Slot w;
            u32x4_t y;
        };
        constexpr int RD = ax_ring(NI);
        Slot rg[RD];
        auto load_step = [&](int st, Slot &r) __attribute__((always_inline)) {
            tl.load(st, r.w);
            const int64_t lab = l_begin + (int64_t)st * 32 + 8 * dp;
            r.y = load_row8<READ>(dseg, (uint32_t)(((int64_t)dr * L + lab) * 2), dr < rows ? l_end - lab : 0);
        };
        uint32_t ca[3][NI];                       // cells written, to be cleared three steps later
        auto stage_y = [&](const Slot &r, int sb) __attribute__((always_inline)) {
            u32x4_t v = r.y;
            uint32_t top = 0u;                    // bit 15 or 31 of a dword: that half's exponent is all ones
#pragma unroll
            for (int k = 0; k < 4; ++k) top |= (v[k] & 0x7fff7fffu) + 0x00800080u;
            if (top & 0x80008000u) {              // (rows past the batch are zero)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t t = ((v[k] & 0x7fff7fffu) + 0x00800080u) & 0x80008000u;
                    const uint32_t m = (t >> 15) * 0xffffu;
                    v[k] = (v[k] & ~(m & 0x7fff7fffu)) | (m & 0x00800080u);
                }
                atomicOr(&bad[dr >> 5], 1u << (dr & 31));
            }
            if (ylane) *(lds_u32x4_t *)(uintptr_t)(yst + (uint32_t)(sb * SB)) = v;
        };
#pragma unroll
        for (int k = 0; k < 3; ++k) tl.no_cells(ca[k]);
        // step s waits in ring slot s mod RD, is written into tile and stage s mod 3, and leaves its
        // cells in ca[s mod 3]
#pragma unroll
        for (int k = 0; k < RD; ++k) {
            load_step(k, rg[k]);
            __builtin_amdgcn_sched_barrier(0);
        }
        tl.scatter(rg[0].w, 0, ca[0]);
        stage_y(rg[0], 0);
        load_step(RD, rg[0]);
        __syncthreads();                          // step 0 in its tile
        // interval t: tile (t + 1) mod 3, last read in interval t - 2, loses step t - 2 and takes step t + 1
        auto interval = [&](int t, auto uc) __attribute__((always_inline)) {
            constexpr int N = (decltype(uc)::value + 1) % 3;
            tl.clear(N, ca[N]);
            tl.scatter(rg[N % RD].w, N, ca[N]);
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
    } else {
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
    __syncthreads();                              // partial stored, rows marked
    if ((bad[0] | bad[1]) != 0u)                  // workgroup-uniform
        ax_add_not_finite<MT, FR>(ax, fix, bad);
}

// ---------------------------------------------------------------------------------------------
// Forward on the same tiles: Y[rows, l] = bias[l] + sum over f of X[rows, f] W'[l, f], or with the rows'
// positives the loss gradient of the rounded logits.
//
// A workgroup owns 128 batch rows and a segment of labels: consumer wave w keeps X for rows 32 w ..
// 32 w + 31 and all FR features in registers (192 at FR = 768) and per step forms D[32 labels][32 rows]
// with v_mfma_f32_32x32x16_bf16, A read from the feature-major tile with ds_read_b64_tr_b16 (two reads
// per 16 features).  Every row costs the tile's writes once per 128 rows, and the reads of a tile (48
// KiB per wave, about 105 bytes per cycle and CU) set the pace, a little above the products.  The bf16
// logits go to a [32 rows][32 labels] LDS block of the wave, from which its producer wave stores them two
// steps later (and takes the sigmoid, whose transcendentals the consumers then need not wait for).
//
// An empty cell contributes X times zero, which is zero only for finite X.  A workgroup whose rows hold an
// infinity or a NaN therefore takes each label's own slots one by one instead, hundreds of times slower (128
// rows, 131K labels, 256 slots: 39 us, 18 ms with one infinity).
// ---------------------------------------------------------------------------------------------
constexpr int kFaStage = 2 * 4 * 2048;            // two steps of four waves' blocks
__host__ __device__ constexpr int fa_lds(int fr) { return 3 * fr * 64 + kFaStage; }

// element e of row b is a positive of the row (sorted ascending)
__device__ __forceinline__ bool is_positive(const int32_t *row, int P, int64_t e) {
    int lo = 0, hi = P;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if ((int64_t)row[mid] < e) lo = mid + 1;
        else hi = mid;
    }
    return lo < P && (int64_t)row[lo] == e;
}

// NC: 16-feature K chunks (FR = 16 NC >= F_s).
template <int NC, int PK, int NI, int READ>
__global__ __attribute__((amdgpu_flat_work_group_size(kAxThreads, kAxThreads), amdgpu_waves_per_eu(2, 2)))
void k_fwd_any(const bf16_t *__restrict__ X, const int32_t *__restrict__ idx, const bf16_t *__restrict__ W,
               const float *__restrict__ bias, bf16_t *__restrict__ Y, int B, int F_s, int64_t L, int G, uint32_t gmul,
               int F_in, int nbt, int64_t lps, const int32_t *__restrict__ spos, int P) {
    constexpr int FR = 16 * NC, TB = FR * 64;
    extern __shared__ __align__(16) char ax[];
    const int w = blockIdx.x, xcd = w % kXcds, jj = w / kXcds;
    const int bt = jj % nbt;
    const int64_t seg = (int64_t)(jj / nbt) * kXcds + xcd;
    const int b0 = bt * 128;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t l_begin = seg * lps;
    const int64_t l_end = l_begin + lps < L ? l_begin + lps : L;
    if (l_begin >= l_end) return;                 // workgroup-uniform
    const int n = (int)((l_end - l_begin + 31) / 32);   // steps
    const uint32_t lbase = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)ax;
    const uint32_t sbase = lbase + 3 * TB;
    for (int e = tid; e < 3 * TB / 16; e += kAxThreads) *(lds_u32x4_t *)(uintptr_t)(lbase + 16 * e) = u32x4_t{0u, 0u, 0u, 0u};
    if (tid == 0) *(lds_u32_t *)(uintptr_t)sbase = 0u;   // becomes 1 if X is not finite

    // X of the consumers' rows: lane -> row l32, features 16 c + 8 h .. + 7
    const int l32 = lane & 31, h = lane >> 5;
    const int row0 = b0 + 32 * (wave & 3);
    const int rows = B - row0 < 32 ? B - row0 : 32;   // of this wave (or its consumer); none if <= 0
    bf16x8_t xb[NC];
    bool bad = false;
    if (wave < kAxCons && rows > 0) {
        const Buf xr(X + (int64_t)row0 * F_s, (uint32_t)(rows * F_s * 2));
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int f = 16 * c + 8 * h;
            const int nv = l32 < rows ? F_s - f : 0;
            const uint32_t o = (uint32_t)((l32 * F_s + f) * 2);
            uint4 v;
            if ((F_s & 7) == 0) {                 // kernel-uniform
                v = xr.ld16(nv > 0 ? o : kOob);
            } else if ((F_s & 3) == 0) {
                const uint2 lo = xr.ld8(nv > 0 ? o : kOob), hi = xr.ld8(nv > 4 ? o + 8 : kOob);
                v = make_uint4(lo.x, lo.y, hi.x, hi.y);
            } else if ((F_s & 1) == 0) {
                v = __builtin_bit_cast(uint4, load_row8<kRead4>(xr, o, nv));
            } else {
                v = __builtin_bit_cast(uint4, load_row8<kRead2>(xr, o, nv));
            }
            const uint32_t d[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) bad |= (d[k] & 0x7f80u) == 0x7f80u || (d[k] & 0x7f800000u) == 0x7f800000u;
            xb[c] = as_bf16x8(v);
        }
    }
    __syncthreads();                              // tiles zeroed
    if (bad) *(lds_u32_t *)(uintptr_t)sbase = 1u;
    __syncthreads();
    if (*(lds_u32_t *)(uintptr_t)sbase != 0u) {   // workgroup-uniform
        const int nr = B - b0 < 128 ? B - b0 : 128;
        for (int64_t l = l_begin + tid; l < l_end; l += kAxThreads) {
            const int32_t *ip = idx + l / G * F_in;
            for (int r = b0; r < b0 + nr; ++r) {
                float a = 0.0f;
                for (int t = 0; t < F_in; ++t) a = fmaf(bf16_to_f32(X[(int64_t)r * F_s + ip[t]]), bf16_to_f32(W[l * F_in + t]), a);
                bf16_t y = f32_to_bf16(bias ? a + bias[l] : a);
                if (spos) y = f32_to_bf16(bce_grad_f32(bf16_to_f32(y), is_positive(spos + (int64_t)r * P, P, l)));
                Y[(int64_t)r * L + l] = y;
            }
        }
        return;
    }

    if (wave >= kAxCons) {
        // ---- producers ----
        const int pt = tid - 64 * kAxCons;
        using Tiles = AxTiles<PK, NI, READ, FR, false>;
        const Tiles tl(idx, W, l_begin, l_end, G, gmul, F_in, 0, lbase, 0u, pt);
        // output of consumer wave - 4: this lane's rows (lane / 4) and 16 + (lane / 4), labels 8 (lane mod 4) ..
        const int orow = lane >> 2, piece = lane & 3;
        const Buf yo(Y + (int64_t)row0 * L, (uint32_t)(rows > 0 ? (int64_t)rows * L * 2 : 0));
        // whole half-lines stream past the L2; pieces that straddle lines must meet there (328K labels in
        // groups of 24, rows not 128-byte aligned: 179 us streaming, 109 through the L2; aligned 108, 114)
        const bool lines = L % 64 == 0;
        PosCursor tg[2];
        if (spos) {
#pragma unroll
            for (int k = 0; k < 2; ++k)
                if (orow + 16 * k < rows) tg[k].init(spos + (int64_t)(row0 + orow + 16 * k) * P, P, l_begin + 8 * piece);
        }
        const uint32_t rd = sbase + (uint32_t)((wave & 3) * 2048 + orow * 64 + ((piece ^ ((orow >> 2) & 3)) << 4));
        auto flush = [&](int t) __attribute__((always_inline)) {
            const int64_t lab = l_begin + (int64_t)t * 32 + 8 * piece;
            const int64_t nv = l_end - lab;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int r = orow + 16 * k;
                if (r >= rows || nv <= 0) continue;
                u32x4_t v = *(lds_u32x4_t *)(uintptr_t)(rd + (uint32_t)((t & 1) * 8192 + k * 1024));
                if (spos) {                       // kernel-uniform
                    const uint32_t m = tg[k].bits(lab, 8);
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[j] = bce_pair(v[j], m >> (2 * j));
                }
                const uint32_t o = (uint32_t)(((int64_t)r * L + lab) * 2);
                if constexpr (READ == kRead16) {
                    if (lines) yo.st16<kStreaming>(__builtin_bit_cast(uint4, v), o);
                    else yo.st16(__builtin_bit_cast(uint4, v), o);
                } else if constexpr (READ == kRead4) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) yo.st4(v[j], nv > 2 * j ? o + 4 * j : kOob);
                } else {
#pragma unroll
                    for (int j = 0; j < 8; ++j) yo.st2((uint16_t)(v[j >> 1] >> (16 * (j & 1))), nv > j ? o + 2 * j : kOob);
                }
            }
        };
        constexpr int RD = ax_ring(NI);
        typename Tiles::Slot rg[RD];
        uint32_t ca[3][NI];
#pragma unroll
        for (int k = 0; k < 3; ++k) tl.no_cells(ca[k]);
#pragma unroll
        for (int k = 0; k < RD; ++k) {
            tl.load(k, rg[k]);
            __builtin_amdgcn_sched_barrier(0);
        }
        tl.scatter(rg[0], 0, ca[0]);
        tl.load(RD, rg[0]);
        __syncthreads();                          // step 0 in its tile
        // interval t: as in backward-feature; the logits of step t - 2 were written in interval t - 1
        auto interval = [&](int t, auto uc) __attribute__((always_inline)) {
            constexpr int N = (decltype(uc)::value + 1) % 3;
            tl.clear(N, ca[N]);
            tl.scatter(rg[N % RD], N, ca[N]);
            __builtin_amdgcn_sched_barrier(0);
            tl.load(t + 1 + RD, rg[N % RD]);
            __builtin_amdgcn_sched_barrier(0);
            if (t >= 2) flush(t - 2);
            __syncthreads();
        };
        for (int t = 0; t < n; t += 3) {
            interval(t, std::integral_constant<int, 0>{});
            if (t + 1 >= n) break;
            interval(t + 1, std::integral_constant<int, 1>{});
            if (t + 2 >= n) break;
            interval(t + 2, std::integral_constant<int, 2>{});
        }
        if (n >= 2) flush(n - 2);
        __syncthreads();                          // the last step's logits
        flush(n - 1);
        return;
    }

    // ---- consumers ----
    __syncthreads();                              // step 0 in its tile
    if (rows <= 0) {                              // wave-uniform: no rows, only the barriers
        for (int t = 0; t <= n; ++t) __syncthreads();
        return;
    }
    __builtin_amdgcn_s_setprio(2);
    constexpr int RING = NC % 6 == 0 ? 6 : 8, PD = RING - 1;   // operands held; read ahead
    static_assert(NC % RING == 0, "whole rings per step");
    // A operand source lanes (ds_read_b64_tr_b16): 16-lane group g = lane / 16 names labels 16 (g & 1) ..
    // of features 16 c + 8 (g >> 1) + 4 i + jq (read i), 4 labels 4 aq .. + 3 per lane
    const int g = lane >> 4, jq = (lane & 15) >> 2, aq = lane & 3;
    uint32_t ao[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
        ao[i] = lbase + (uint32_t)((8 * (g >> 1) + 4 * i + jq) * 64 +
                                   (((2 * (g & 1) + (aq >> 1)) ^ ((2 * (g >> 1) + i) & 3)) << 4) + 8 * (aq & 1));
    auto read_a = [&](uint32_t tile, int c) __attribute__((always_inline)) -> bf16x8_t {
        const bf16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_t *)(uintptr_t)(ao[0] + tile + 1024 * c));
        const bf16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_t *)(uintptr_t)(ao[1] + tile + 1024 * c));
        const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
        return as_bf16x8(make_uint4(l2.x, l2.y, h2.x, h2.y));
    };
    // this lane's logits of a step: row l32, labels 8 i + 4 h .. + 3
    const uint32_t wr = sbase + (uint32_t)(wave * 2048 + l32 * 64 + 8 * h);
    bf16x8_t oa[RING];
#pragma unroll
    for (int c = 0; c < PD; ++c) oa[c] = read_a(0u, c);
    const Buf bseg(bias ? bias + l_begin : bias, (uint32_t)(bias ? (l_end - l_begin) * 4 : 0));
    int s3 = 0;                                   // the step's tile
    for (int t = 0; t < n; ++t) {
        const uint32_t cur = (uint32_t)(s3 * TB);
        s3 = s3 == 2 ? 0 : s3 + 1;
        const uint32_t nxt = (uint32_t)(s3 * TB);
        f32x16_t acc = f32x16_t{0};
        if (bias) {                               // kernel-uniform; labels past the segment read as zero
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x4_t v = __builtin_bit_cast(f32x4_t, bseg.ld16((uint32_t)(128 * t + 16 * h + 32 * i)));
                acc[4 * i] = v[0];
                acc[4 * i + 1] = v[1];
                acc[4 * i + 2] = v[2];
                acc[4 * i + 3] = v[3];
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (c == NC - PD) {
                // the next step is in its tile (this one's reads may still be in flight: its tile is
                // written again two barriers on)
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            oa[(c + PD) % RING] = c + PD < NC ? read_a(cur, c + PD) : read_a(nxt, c + PD - NC);
            __builtin_amdgcn_sched_barrier(0);
            acc = mfma32x32x16(oa[c % RING], xb[c], acc);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *(lds_u32x2_t *)(uintptr_t)(wr + (uint32_t)((t & 1) * 8192 + ((i ^ ((l32 >> 2) & 3)) << 4))) =
                u32x2_t{pack_bf16(acc[4 * i], acc[4 * i + 1]), pack_bf16(acc[4 * i + 2], acc[4 * i + 3])};
    }
    __syncthreads();                              // the last step's logits are written
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

// ws_bytes: of the partials; fewer segments where it holds no more (0 segments: not even one)
inline AxGeom ax_geom(const haste::TailArgs &a, size_t ws_bytes = SIZE_MAX) {
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
    const size_t fit = ws_bytes / ((size_t)a.F_s * (size_t)(g.nbt * 16 * g.mt) * 4);
    if (fit < (size_t)g.nseg) g.nseg = (int64_t)fit;
    g.lps = g.nseg ? haste::round_up(haste::cdiv(a.L, g.nseg), 64) : 0;
    g.lds = (size_t)ax_lds(16 * kAxCons * g.nft, g.mt);
    return g;
}

struct FaGeom {
    int nc, nbt, pk, ni;
    int64_t nseg, lps;
};

inline FaGeom fa_geom(const haste::TailArgs &a) {
    const AxGeom x = ax_geom(a);
    FaGeom g;
    g.nc = a.F_s <= 512 ? 32 : 48;
    g.nbt = (int)haste::cdiv(a.B, 128);
    g.pk = x.pk;
    g.ni = x.ni;
    int64_t nseg = haste::round_up(haste::cdiv(kXcds * kCusPerXcd, g.nbt), kXcds);
    const int64_t max_seg = haste::round_up(haste::cdiv(a.L, 64), kXcds);
    g.nseg = nseg < max_seg ? nseg : max_seg;
    g.lps = haste::round_up(haste::cdiv(a.L, g.nseg), 64);
    return g;
}

// f.go<PK, NI, READ>() for the layer's packs, slot pairs and access width (the entry points refuse arrays
// that are not 16-byte aligned)
template <class F>
hipError_t ax_pick(const haste::TailArgs &a, int pk, int ni, const F &f) {
    auto read = [&](auto p, auto i) -> hipError_t {
        constexpr int PK = decltype(p)::value, NI = decltype(i)::value;
        if (a.F_in % 2 == 0) {
            if (a.L % 8 == 0) return f.template go<PK, NI, kRead16>();
            if constexpr (PK < 8)
                if (a.L % 2 == 0) return f.template go<PK, NI, kRead4>();
        }
        return f.template go<PK, NI, kRead2>();
    };
#define HASTE_AX(p, i) \
    case 100 * p + i: return read(std::integral_constant<int, p>{}, std::integral_constant<int, i>{})
    switch (100 * pk + ni) {
        HASTE_AX(1, 4);
        HASTE_AX(1, 8);
        HASTE_AX(1, 16);
        HASTE_AX(2, 2);
        HASTE_AX(2, 4);
        HASTE_AX(2, 8);
        HASTE_AX(4, 1);
        HASTE_AX(4, 2);
        HASTE_AX(4, 4);
        HASTE_AX(8, 1);
        HASTE_AX(8, 2);
    }
#undef HASTE_AX
    return hipErrorInvalidValue;
}

// one launch of the forward for NC feature chunks
template <int NC>
struct FaRun {
    const haste::TailArgs &a;
    const FaGeom &g;
    const void *X;
    const int32_t *idx;
    const void *W;
    const float *bias;
    void *Y;
    const int32_t *spos;
    int P;
    hipStream_t s;

    template <int PK, int NI, int READ>
    hipError_t go() const {
        auto kern = k_fwd_any<NC, PK, NI, READ>;
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           fa_lds(16 * NC));
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)(g.nseg * g.nbt)), dim3(kAxThreads), fa_lds(16 * NC), s, (const bf16_t *)X, idx,
                           (const bf16_t *)W, bias, (bf16_t *)Y, (int)a.B, (int)a.F_s, a.L, (int)a.G, div_mul(a.G), (int)a.F_in,
                           g.nbt, g.lps, spos, P);
        return hipGetLastError();
    }
    hipError_t run() const { return ax_pick(a, g.pk, g.ni, *this); }
};

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
        hipLaunchKernelGGL(kern, dim3((unsigned)(haste::round_up(g.nseg, kXcds) * g.nbt * g.nsplit)), dim3(kAxThreads), g.lds, s,
                           idx, (const bf16_t *)W, (const bf16_t *)dY, part, (int)a.B, g.nbt * 16 * MT, (int)a.F_s, a.L, (int)a.G,
                           div_mul(a.G), (int)a.F_in, g.nbt, g.nsplit, g.nseg, g.lps);
        return hipGetLastError();
    }
    hipError_t run() const { return ax_pick(a, g.pk, g.ni, *this); }
};

}  // namespace
