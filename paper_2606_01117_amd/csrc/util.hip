// Small helper kernels: fills, fixed-order partial reductions, idx validation, gather export.
#include "common.hpp"

namespace {

__global__ void k_fill(float *__restrict__ p, int64_t n, float v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// dX[b, f] = beta dX[b, f] + sum_{k < S} part[k][f][b], in a fixed order: the partials in four runs, a run
// eight at a time in pairs, the eights in ascending k, and the runs' sums in pairs.  A workgroup takes 8
// features x 32 rows, each of its waves one of the runs: a lane reads 4 consecutive rows (16 bytes, 128
// contiguous bytes per feature) of every partial, with the loads of 8 partials in flight, and the waves'
// sums meet in LDS.  With all partials in one wave, a chain of S / 8 waits, and 8 x 128 rows a workgroup, 77
// rows x 500 features ran on 63 CUs: that training step (65K labels, G = 24) 95.7 us, 92.1 now; 128 rows x
// 768 (131K labels, G = 16) 72.1 and 71.4; from 256 rows on, where the read rate bounds it, no different.
__global__ __launch_bounds__(256) void k_reduce_fmajor(const float *__restrict__ part, int S, int64_t ldp, int64_t B,
                                                       int64_t F_s, float *__restrict__ dX, int beta, unsigned nfb) {
    __shared__ __align__(16) float tile[4][8][32 + 4];
    const int64_t f0 = (int64_t)(blockIdx.x % nfb) * 8, b0 = (int64_t)(blockIdx.x / nfb) * 32;
    const int t = threadIdx.x, bq = t & 7, fr = (t >> 3) & 7, run = t >> 6;
    const int64_t f = f0 + fr, b = b0 + 4 * bq;
    const int len = ((S + 3) / 4 + 7) / 8 * 8, k1 = (run + 1) * len < S ? (run + 1) * len : S;
    float4 acc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (f < F_s && b < ldp) {
        const float4 *p = reinterpret_cast<const float4 *>(part + f * ldp + b);
        const int64_t ks = F_s * ldp / 4;   // float4 stride between partials
        int k = run * len;
        for (; k + 8 <= k1; k += 8) {
            float4 v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = p[(int64_t)(k + j) * ks];
            // the eight in pairs, then onto the running sum, whose roundings are the largest
#pragma unroll
            for (int d = 1; d < 8; d *= 2)
#pragma unroll
                for (int j = 0; j < 8; j += 2 * d) {
                    v[j].x += v[j + d].x;
                    v[j].y += v[j + d].y;
                    v[j].z += v[j + d].z;
                    v[j].w += v[j + d].w;
                }
            acc.x += v[0].x;
            acc.y += v[0].y;
            acc.z += v[0].z;
            acc.w += v[0].w;
        }
        for (; k < k1; ++k) {
            const float4 v = p[(int64_t)k * ks];
            acc.x += v.x;
            acc.y += v.y;
            acc.z += v.z;
            acc.w += v.w;
        }
    }
    *reinterpret_cast<float4 *>(&tile[run][fr][4 * bq]) = acc;
    __syncthreads();
    // thread -> row b0 + t / 8, feature f0 + t % 8
    const int r = t >> 3, c = t & 7;
    if (b0 + r < B && f0 + c < F_s) {
        const float v = (tile[0][c][r] + tile[1][c][r]) + (tile[2][c][r] + tile[3][c][r]);
        float *q = dX + (b0 + r) * F_s + f0 + c;
        *q = beta ? *q + v : v;
    }
}

// C[i] (+)= sum_{k < S} part[k][i] in ascending k, four consecutive elements per thread (16-byte
// loads) with the loads of 16 partials in flight: the partial sums are read once, at a rate the
// one-float-per-thread loop below does not reach (its loads wait one by one).  MN % 4 == 0 and
// 16-byte aligned arrays.
__global__ __launch_bounds__(256) void k_reduce_rmajor4(const float4 *__restrict__ part, int S, int64_t MN4,
                                                        float4 *__restrict__ C, int beta) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= MN4) return;
    float4 acc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    int k = 0;
    for (; k + 16 <= S; k += 16) {
        float4 v[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = part[(int64_t)(k + j) * MN4 + i];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            acc.x += v[j].x;
            acc.y += v[j].y;
            acc.z += v[j].z;
            acc.w += v[j].w;
        }
    }
    for (; k < S; ++k) {
        const float4 v = part[(int64_t)k * MN4 + i];
        acc.x += v.x;
        acc.y += v.y;
        acc.z += v.z;
        acc.w += v.w;
    }
    if (beta) {
        const float4 o = C[i];
        acc.x = o.x + acc.x;
        acc.y = o.y + acc.y;
        acc.z = o.z + acc.z;
        acc.w = o.w + acc.w;
    }
    C[i] = acc;
}

__global__ void k_reduce_rmajor(const float *__restrict__ part, int S, int64_t MN, float *__restrict__ C, int beta) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < MN; i += (int64_t)gridDim.x * blockDim.x) {
        float s = 0.0f;
        for (int k = 0; k < S; ++k) s += part[(int64_t)k * MN + i];
        C[i] = beta ? C[i] + s : s;
    }
}

__global__ void k_validate(const int32_t *__restrict__ idx, int64_t rows, int64_t F_in, int64_t F_s,
                           int32_t *__restrict__ n_bad) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < rows; r += (int64_t)gridDim.x * blockDim.x) {
        const int32_t *p = idx + r * F_in;
        bool ok = true;
        int64_t prev = -1;
        for (int64_t t = 0; t < F_in; ++t) {
            const int64_t v = p[t];
            if (v <= prev || v >= F_s) ok = false;
            prev = v;
        }
        if (!ok) atomicAdd(n_bad, 1);
    }
}

__global__ void k_zero_i32(int32_t *p) { *p = 0; }

template <typename T>
__global__ void k_gather(const T *__restrict__ X, const int32_t *__restrict__ idx, int64_t B, int64_t F_s,
                         int64_t F_in, int64_t k0, int64_t nk, T *__restrict__ out) {
    const int64_t n = nk * B * F_in;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t t = i % F_in, b = (i / F_in) % B, k = i / (F_in * B);
        out[i] = X[b * F_s + idx[(k0 + k) * F_in + t]];
    }
}

unsigned grid_for(int64_t n) {
    int64_t g = haste::cdiv(n, 256);
    if (g > 4096) g = 4096;
    return (unsigned)(g < 1 ? 1 : g);
}


// BCE gradient of stored logits (Section 3.3 objective): dY[b, n] = sigmoid(Y[b, n]) - T[b, n], with
// T[b, n] = 1 where n occurs in pos[b, 0..P-1].  A workgroup takes 2048 columns of one row and a
// thread 8 of them.  Y and dY may be the same buffer
// (each element is read before it is written, by the same thread).
// Which 8 columns a thread takes: 8 consecutive bf16 (16 bytes), two runs of 4 consecutive fp32 (16 bytes
// each, 1024 columns apart), or, where rows are not whole 16-byte groups, 8 single columns 256 apart, so
// that every access of a wave is one contiguous run.  (Eight consecutive columns one by one touched each
// line eight times: 131K fp32 columns, 128 rows: 73 us, 21 so.)
// A few positives are read by every thread (workgroup-uniform); more are set in a bitmap of the workgroup's
// columns by the threads together, whose barriers cost 3% (256 rows of 655K bf16 columns, 5 / 40 positives:
// 110 / 239 us one by one, 114 / 114 in the bitmap).
constexpr int kBceFew = 8;
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void k_bce_grad(const T *Y, const int32_t *__restrict__ pos, int P, T *dY,
                                                  int64_t N, int64_t nchunk) {
    constexpr int RUN = VEC ? 16 / (int)sizeof(T) : 1;   // consecutive columns
    const int64_t b = blockIdx.x / nchunk;
    const int64_t c0 = (blockIdx.x - b * nchunk) * 2048;
    const int tid = threadIdx.x;
    uint32_t t = 0;                               // bit RUN i + e: column c0 + 256 RUN i + RUN tid + e
    if (P <= kBceFew) {                           // kernel-uniform
        for (int p = 0; p < P; ++p) {
            const int64_t d = (int64_t)pos[b * P + p] - c0;
            if (d < 0 || d >= 2048) continue;     // workgroup-uniform
            const int i = (int)d / (256 * RUN), e = (int)d % (256 * RUN) - RUN * tid;
            if (e >= 0 && e < RUN) t |= 1u << (RUN * i + e);
        }
    } else {
        __shared__ uint32_t hit[64];              // one bit per column
        if (tid < 64) hit[tid] = 0u;
        __syncthreads();
        for (int p = tid; p < P; p += 256) {
            const int64_t d = (int64_t)pos[b * P + p] - c0;
            if (d >= 0 && d < 2048) atomicOr(&hit[d >> 5], 1u << (d & 31));
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 8 / RUN; ++i) {
            const int c = 256 * RUN * i + RUN * tid;
            t |= (hit[c >> 5] >> (c & 31) & ((1u << RUN) - 1u)) << (RUN * i);
        }
    }
    const T *y = Y + b * N;
    T *o = dY + b * N;
    if constexpr (VEC) {
#pragma unroll
        for (int i = 0; i < 8 / RUN; ++i) {
            const int64_t c = c0 + 256 * RUN * i + RUN * tid;
            if (c >= N) continue;
            const uint4 v = *reinterpret_cast<const uint4 *>(y + c);
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
            uint32_t r[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                r[k] = sizeof(T) == 2 ? bce_pair(w[k], t >> (2 * k))
                                      : __float_as_uint(bce_grad_f32(__uint_as_float(w[k]), (t >> (RUN * i + k)) & 1));
            *reinterpret_cast<uint4 *>(o + c) = make_uint4(r[0], r[1], r[2], r[3]);
        }
    } else {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int64_t c = c0 + 256 * i + tid;
            v[i] = c < N ? load_f32(y, c) : 0.0f;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int64_t c = c0 + 256 * i + tid;
            if (c < N) store_out(o, c, bce_grad_f32(v[i], (t >> i) & 1));
        }
    }
}

// Each batch row's positives sorted ascending (one wave per row): element i goes to its rank
// #{j : v_j < v_i, or v_j == v_i and j < i}; ids outside [0, N) (the -1 padding) sort last as
// INT32_MAX.
__global__ __launch_bounds__(256) void k_sort_pos(const int32_t *__restrict__ pos, int P, int64_t B, int64_t N,
                                                  int32_t *__restrict__ spos) {
    __shared__ int32_t v[4][haste::kSortPosMax];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t b = (int64_t)blockIdx.x * 4 + w;
    if (b >= B) return;   // wave-uniform; no barrier follows
    for (int i = lane; i < P; i += 64) {
        const int32_t x = pos[b * P + i];
        v[w][i] = x >= 0 && x < N ? x : INT32_MAX;
    }
    __builtin_amdgcn_wave_barrier();
    for (int i = lane; i < P; i += 64) {
        const int32_t x = v[w][i];
        int r = 0;
        for (int j = 0; j < P; ++j) {
            const int32_t y = v[w][j];
            r += (y < x) || (y == x && j < i);
        }
        spos[b * P + r] = x;
    }
}

// One momentum step per weight (sgd_step), four consecutive weights per thread: 16-byte velocity and
// gradient accesses and 8- or 16-byte weight accesses when n is a multiple of 4 and the buffers are
// aligned (VEC), else one weight per thread.  W_next may be W: each weight is read before it is
// written, by the same thread.  g == NULL: a zero gradient.
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void k_sgd_momentum(const T *W, const float *__restrict__ g, float *__restrict__ m,
                                                      T *W_next, int64_t n, float lr, float momentum,
                                                      float weight_decay) {
    const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * (VEC ? 4 : 1);
    if (i0 >= n) return;
    if constexpr (VEC) {
        const float4 gv = g ? *reinterpret_cast<const float4 *>(g + i0) : make_float4(0.f, 0.f, 0.f, 0.f);
        float4 mv = *reinterpret_cast<const float4 *>(m + i0);
        float w[4], o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = load_f32(W, i0 + j);
        sgd_step(w[0], gv.x, mv.x, o[0], lr, momentum, weight_decay);
        sgd_step(w[1], gv.y, mv.y, o[1], lr, momentum, weight_decay);
        sgd_step(w[2], gv.z, mv.z, o[2], lr, momentum, weight_decay);
        sgd_step(w[3], gv.w, mv.w, o[3], lr, momentum, weight_decay);
        *reinterpret_cast<float4 *>(m + i0) = mv;
        if constexpr (sizeof(T) == 2)
            *reinterpret_cast<uint2 *>(W_next + i0) = make_uint2(pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3]));
        else
            *reinterpret_cast<float4 *>(W_next + i0) = make_float4(o[0], o[1], o[2], o[3]);
    } else {
        float mm = m[i0], o;
        sgd_step(load_f32(W, i0), g ? g[i0] : 0.0f, mm, o, lr, momentum, weight_decay);
        m[i0] = mm;
        store_out(W_next, i0, o);
    }
}
}  // namespace

namespace haste {

hipError_t fill_f32(float *p, int64_t n, float v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill, dim3(grid_for(n)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t reduce_fmajor(const float *part, int S, int64_t ldp, int64_t B, int64_t F_s, float *dX, int beta,
                         hipStream_t s) {
    if (B <= 0) return hipSuccess;
    const int64_t nfb = cdiv(F_s, 8);
    hipLaunchKernelGGL(k_reduce_fmajor, dim3((unsigned)(nfb * cdiv(B, 32))), dim3(256), 0, s, part, S, ldp, B, F_s, dX,
                       beta, (unsigned)nfb);
    return hipGetLastError();
}

hipError_t reduce_rmajor(const float *part, int S, int64_t M, int64_t N, float *C, int beta, hipStream_t s) {
    const int64_t MN = M * N;
    if (MN <= 0) return hipSuccess;
    if (MN % 4 == 0 && (reinterpret_cast<uintptr_t>(part) & 15) == 0 && (reinterpret_cast<uintptr_t>(C) & 15) == 0) {
        hipLaunchKernelGGL(k_reduce_rmajor4, dim3((unsigned)cdiv(MN / 4, 256)), dim3(256), 0, s,
                           reinterpret_cast<const float4 *>(part), S, MN / 4, reinterpret_cast<float4 *>(C), beta);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_reduce_rmajor, dim3(grid_for(MN)), dim3(256), 0, s, part, S, MN, C, beta);
    return hipGetLastError();
}

hipError_t validate_idx(const int32_t *idx, int64_t rows, int64_t F_in, int64_t F_s, int32_t *n_bad,
                        hipStream_t s) {
    hipLaunchKernelGGL(k_zero_i32, dim3(1), dim3(1), 0, s, n_bad);
    if (rows > 0) hipLaunchKernelGGL(k_validate, dim3(grid_for(rows)), dim3(256), 0, s, idx, rows, F_in, F_s, n_bad);
    return hipGetLastError();
}

hipError_t debug_gather(const void *X, int32_t dtype, const int32_t *idx, int64_t B, int64_t F_s, int64_t F_in,
                        int64_t k0, int64_t nk, void *out, hipStream_t s) {
    const int64_t n = nk * B * F_in;
    if (n <= 0) return hipSuccess;
    if (dtype == HASTE_DTYPE_BF16)
        hipLaunchKernelGGL(k_gather<bf16_t>, dim3(grid_for(n)), dim3(256), 0, s, (const bf16_t *)X, idx, B, F_s, F_in,
                           k0, nk, (bf16_t *)out);
    else
        hipLaunchKernelGGL(k_gather<float>, dim3(grid_for(n)), dim3(256), 0, s, (const float *)X, idx, B, F_s, F_in, k0,
                           nk, (float *)out);
    return hipGetLastError();
}


hipError_t bce_grad(int64_t B, int64_t N, int32_t dtype, const void *Y, const int32_t *pos, int P, void *dY,
                    hipStream_t s) {
    const int64_t nchunk = cdiv(N, 2048);
    const dim3 grid((unsigned)(B * nchunk)), block(256);
    const bool vec = N % (dtype == HASTE_DTYPE_BF16 ? 8 : 4) == 0 &&
                     ((reinterpret_cast<uintptr_t>(Y) | reinterpret_cast<uintptr_t>(dY)) & 15) == 0;
    if (dtype == HASTE_DTYPE_BF16) {
        if (vec)
            hipLaunchKernelGGL((k_bce_grad<bf16_t, true>), grid, block, 0, s, (const bf16_t *)Y, pos, P, (bf16_t *)dY, N, nchunk);
        else
            hipLaunchKernelGGL((k_bce_grad<bf16_t, false>), grid, block, 0, s, (const bf16_t *)Y, pos, P, (bf16_t *)dY, N, nchunk);
    } else {
        if (vec)
            hipLaunchKernelGGL((k_bce_grad<float, true>), grid, block, 0, s, (const float *)Y, pos, P, (float *)dY, N, nchunk);
        else
            hipLaunchKernelGGL((k_bce_grad<float, false>), grid, block, 0, s, (const float *)Y, pos, P, (float *)dY, N, nchunk);
    }
    return hipGetLastError();
}


hipError_t sort_positives(int64_t B, int64_t N, const int32_t *pos, int P, int32_t *spos, hipStream_t s) {
    if (B <= 0 || P <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_sort_pos, dim3((unsigned)cdiv(B, 4)), dim3(256), 0, s, pos, P, B, N, spos);
    return hipGetLastError();
}

hipError_t sgd_momentum(int64_t n, int32_t dtype, const void *W, const float *g, float *m, const haste_sgd_t &opt,
                        void *W_next, hipStream_t s) {
    const uintptr_t al = reinterpret_cast<uintptr_t>(W) | reinterpret_cast<uintptr_t>(g) |
                         reinterpret_cast<uintptr_t>(m) | reinterpret_cast<uintptr_t>(W_next);
    const bool vec = (n % 4) == 0 && (al & 15) == 0;
    const dim3 grid((unsigned)cdiv(n, vec ? 1024 : 256)), block(256);
    if (dtype == HASTE_DTYPE_BF16) {
        if (vec)
            hipLaunchKernelGGL((k_sgd_momentum<bf16_t, true>), grid, block, 0, s, (const bf16_t *)W, g, m,
                               (bf16_t *)W_next, n, opt.lr, opt.momentum, opt.weight_decay);
        else
            hipLaunchKernelGGL((k_sgd_momentum<bf16_t, false>), grid, block, 0, s, (const bf16_t *)W, g, m,
                               (bf16_t *)W_next, n, opt.lr, opt.momentum, opt.weight_decay);
    } else {
        if (vec)
            hipLaunchKernelGGL((k_sgd_momentum<float, true>), grid, block, 0, s, (const float *)W, g, m,
                               (float *)W_next, n, opt.lr, opt.momentum, opt.weight_decay);
        else
            hipLaunchKernelGGL((k_sgd_momentum<float, false>), grid, block, 0, s, (const float *)W, g, m,
                               (float *)W_next, n, opt.lr, opt.momentum, opt.weight_decay);
    }
    return hipGetLastError();
}

}  // namespace haste
