// Backward-feature on scattered tiles for any group: geometry and dispatch (kernel: tail_any.hpp),
// with the instantiations for 64 rows and up to 768 features.
#include "tail_any.hpp"

namespace haste {

hipError_t bwd_x_any_4_8(const TailArgs &a, const int32_t *idx, const void *W, const void *dY, float *part,
                           size_t ws_bytes, hipStream_t s);
hipError_t bwd_x_any_2_12(const TailArgs &a, const int32_t *idx, const void *W, const void *dY, float *part,
                           size_t ws_bytes, hipStream_t s);

hipError_t fwd_any_48(const TailArgs &a, const void *X, const int32_t *idx, const void *W, const float *bias, void *Y,
                      const int32_t *spos, int P, hipStream_t s);
hipError_t fwd_any_32(const TailArgs &a, const void *X, const int32_t *idx, const void *W, const float *bias, void *Y,
                      const int32_t *spos, int P, hipStream_t s);

// forward: as backward-feature, with up to 768 features (the tiles and two steps' logits fill the LDS)
bool fwd_any_supported(const TailArgs &a) {
    if (a.F_s > 768 || !bwd_x_any_supported(a)) return false;
    const FaGeom g = fa_geom(a);
    const int64_t far = g.lps + 256;
    return far * a.F_in * 4 < ((int64_t)1 << 31) && (far + a.G) * a.G < ((int64_t)1 << 32);
}

// A workgroup clears its tiles and reads X for 128 rows (by 2, 4 or 16 bytes), then takes steps of 32 labels;
// a step's cost is that of the product over all features, or of the producers' slot pairs
double fwd_any_us(const TailArgs &a) {
    const FaGeom g = fa_geom(a);
    const double R = xcd_rounds(cdiv(a.L, g.lps), g.nbt, 1), S = R * (g.lps / 32);
    const bool halves = a.F_in % 2 != 0 || a.L % 2 != 0 || (g.pk == 8 && a.L % 8 != 0);
    return 0.56 + R * (1.3 + g.nc * (0.21 + (a.F_s % 2 ? 0.23 : a.F_s % 8 ? 0.057 : 0.0))) +
           S * (0.0055 * g.nc + g.ni * (0.07 + 0.024 * g.pk) + (halves ? 0.015 + 0.075 * g.ni * g.pk : 0.0)) + 0.82e-6 * a.B * a.L;
}

// Where another kernel takes the layer too, measured per call at F_s = 768 (us; 328K labels):
//   - groups of 1 or 2 labels: the scattered tiles of 32 rows per workgroup are written once per 32 rows
//     there, once per 128 here (G = 1, 64 slots, 32 / 64 / 128 / 256 rows: 37 / 60 / 111 / 204 there, 51 /
//     54 / 65 / 110 here);
//   - groups of 4 or 8: their gathers cost about (20 + 3 F_in / G) / 3.3 us per 32 rows, this 53 per 128
//     (256 rows, G = 4, 32 / 64 / 128 slots: 101 / 153 / 284 there, 104 / 107 / 113 here; G = 8: 79 /
//     104 / 169 against 102 / 104 / 109);
//   - larger groups share each gather among 16 labels or more (G = 16, 64 slots: 65 there, 104 here);
//   - everything else (other group sizes and widths) runs on the vector ALUs, 8 times slower.
// So much for large layers.  Here the cost of a step does not depend on the slots, and a workgroup's
// prologue takes 8 to 13 us (twice that at odd F_s), so with few slots, rows or features, or few labels per
// workgroup, the others are faster, and the estimates decide (4 rows, 334K labels, G = 16, 8 slots of 128
// features: 8 there, 34 here; 1606 rows, 2432 labels, G = 8, 128 slots of 128: 13 against 21; 2600 random
// layers: 539 more than 6% slower here than there without the estimates, 69 with them).
bool fwd_any_preferred(const TailArgs &a) {
    if (!fwd_any_supported(a)) return false;
    if (fwd_dn_supported(a)) return a.B > 32 && fwd_any_us(a) < fwd_dn_us(a);
    if (fwd_sg_supported(a))
        return cdiv(a.B, 32) * (20 + 3 * a.F_in / a.G) * 48 > 177 * cdiv(a.B, 128) * fa_geom(a).nc && fwd_any_us(a) < fwd_sg_us(a);
    return !fwd_mfma_supported(a) && valu_supported(a) && fwd_any_us(a) < fwd_valu_us(a);
}

hipError_t fwd_any(const TailArgs &a, const void *X, const int32_t *idx, const void *W, const float *bias, void *Y,
                   hipStream_t s, const int32_t *spos, int P) {
    return a.F_s <= 512 ? fwd_any_32(a, X, idx, W, bias, Y, spos, P, s) : fwd_any_48(a, X, idx, W, bias, Y, spos, P, s);
}

// bf16; 64 rows of dY, and a segment's weights and supports, within the 31-bit range of a buffer
// offset (the loads run five steps past a segment's end); the group of a label by multiply-high.
bool bwd_x_any_supported(const TailArgs &a) {
    if (a.dtype != HASTE_DTYPE_BF16 || a.F_s > kMaxFs || a.L * 128 >= ((int64_t)1 << 31)) return false;
    return bwd_x_any_fits(a, SIZE_MAX);
}

bool bwd_x_any_fits(const TailArgs &a, size_t ws_bytes) {
    const AxGeom g = ax_geom(a, ws_bytes);
    const int64_t far = g.lps + 256;
    return g.ni != 0 && g.nseg != 0 && far * a.F_in * 4 < ((int64_t)1 << 31) && (far + a.G) * a.G < ((int64_t)1 << 32);
}

// Where another kernel takes the layer too, measured per call at F_s = 768 (us; 328K labels):
//   - one label per group, up to 64 slots or 32 rows: the scattered-tile kernel whose waves all do both
//     jobs (64 slots, 32 / 64 / 256 rows: 52 / 68 / 162 there, 58 / 63 / 167 here; 128 slots 69 / 92 /
//     280 against 86 / 89 / 245);
//   - groups in LDS accumulators (general kernel, plus its transposition of W): that costs a
//     read-add-write per (group, slot, row), the dense product FR multiply-adds per label, so the
//     accumulators win where a group has few slots for its labels (256 rows, G = 32: 32 / 64 / 128 slots
//     61 / 90 / 166 there, 113 / 119 / 126 here; G = 16: 91 / 134 / 235 against 111 / 117 / 125), and
//     up to 64 rows the transposition does not pay back (32 rows, G = 32: 45 / 54 / 79 against 44 / 48
//     / 47; 64 rows 64 slots 52 / 52);
//   - everything else (other group sizes and widths: vector ALUs, or small groups of wide inputs)
//     20 times slower there.
// That is for large layers; between the accumulators and this, for groups of 12 to 32 labels, the estimates decide
// (440 rows, 51K labels, G = 12, 32 slots of 512: 44 there, 65 here; of 434 random layers of up to 32 labels
// a group 14 more than 6% slower here than there without them, 2 with them).  Groups of 2, 4 and 8 labels with 32 or 64
// slots, and of one with 128, once ran on the tiles of k_bwd_x_dn, which are faster for some small layers (4% of
// 747 random ones by more than 6%, F_s = 128 and 32 slots by up to half) but turn a whole row of dX to NaN
// where dY is not finite; so they stay here.
double bwd_x_any_us(const TailArgs &a) {
    const AxGeom g = ax_geom(a);
    const double R = xcd_rounds(cdiv(a.L, g.lps), g.nbt * g.nsplit, 1), S = R * (g.lps / 32);
    const bool halves = a.F_in % 2 != 0 || a.L % 2 != 0 || (g.pk == 8 && a.L % 8 != 0);
    return 6.2 + R * 0.099 * g.nft * g.mt + S * (0.063 + 0.012 * g.nft + g.ni * (0.16 + 0.013 * g.pk) + (halves ? 0.21 + 0.1 * g.ni * g.pk : 0.0)) +
           0.36e-6 * bwd_x_any_ws(a);
}

bool bwd_x_any_preferred(const TailArgs &a) {
    if (!bwd_x_any_supported(a) || bwd_x_dn_supported(a)) return false;
    if (bwd_x_mfma_supported(a)) {
        const AxGeom g = ax_geom(a);
        const int64_t per = a.G < 32 ? a.G : 32;
        return (a.B <= 64 || a.F_in * 768 >= 4 * per * (g.nsplit * 64 * g.nft)) &&
               (a.G <= 8 || a.G > 32 || bwd_x_any_us(a) < bwd_x_mfma_us(a));
    }
    return bwd_x_sg_supported(a) || valu_supported(a);
}

size_t bwd_x_any_ws(const TailArgs &a) {
    const AxGeom g = ax_geom(a);
    return (size_t)round_up(g.nseg * a.F_s * (g.nbt * 16 * g.mt) * 4, 256);
}

hipError_t bwd_x_any(const TailArgs &a, const int32_t *idx, const void *W, const void *dY, float *dX, int beta, void *ws,
                     size_t ws_bytes, hipStream_t s) {
    const AxGeom g = ax_geom(a, ws_bytes);
    float *part = reinterpret_cast<float *>(ws);
    const hipError_t e = g.mt == 2    ? bwd_x_any_2_12(a, idx, W, dY, part, ws_bytes, s)
                         : g.nft == 8 ? bwd_x_any_4_8(a, idx, W, dY, part, ws_bytes, s)
                                      : AxRun<4, 12>{a, g, idx, W, dY, part, s}.run();
    if (e != hipSuccess) return e;
    return reduce_fmajor(part, (int)g.nseg, g.nbt * 16 * g.mt, a.B, a.F_s, dX, beta, s);
}

}  // namespace haste
