// get_hermitian + get_bias for fp32 factors as two fp16 parts per value (tiles_x3.h, PARTS = 2) where the NW wavefronts of
// a workgroup share a system (f = 256, tile rows ROWS per wavefront).
//
// With fp32 MFMAs every wavefront gathers every row for itself and runs 8 x 17 instructions of 32 cycles per 32 entries:
// the matrix pipelines are the bound (k_hermitian_wide 123 of 141 TFLOP/s).  Two parts need 3 x 17 instructions of 16
// cycles, and then the gathering and cutting would be: so a step's 32 rows are gathered once per workgroup.  Wavefront w
// fetches entries 4w .. 4w+3, cuts them and puts the parts into LDS in operand layout (1 KB per tile and part,
// 32 KB a step, two buffers in turn, one barrier a step), from where every wavefront reads the tile columns it needs, 16
// bytes per lane, conflict-free.  Per step and CU about 200 KB of LDS reads (1,600 cycles at 128 bytes) stand against
// 1,632 cycles of MFMAs per SIMD.
// Measured (120,047 x 17,770, 25M entries, f = 256, CG(6)): 28.2 -> 16.4 ms per sweep; k_hermitian_wide 8.5 -> 4.7 ms with twice the
// work items (3.3e12 flops of both kernels in 14.5 ms instead of 26.7).
//
// b_u: fp32 FMAs of the uncut values by the lanes that gather them, summed over the wavefronts at the end.
// Producer lane (i, kq): entry pair p = kq % 2 of the wavefront's four entries, feature half kq / 2 (tiles 8 (kq / 2) ..
// + 7, the usual lane -> feature map), so that both entries of an operand word are in one lane.
#pragma once
#include "tiles_x3.h"

namespace als {

constexpr int x2_shared_words(int F) { return 2 * 2 * tiles_1d(F) * 256; }

// Same contract as accumulate_tiles<F, ..., ROWS, true, kExplicit>.  Every wavefront of the workgroup must call, with the
// same s0 and len.  stage: x2_shared_words(F) words of LDS, free again after the workgroup's next barrier.
template <int F, int NW, bool WIDE, uint32_t ROWS>
__device__ __forceinline__ void accumulate_tiles_x2_shared(const int32_t *__restrict__ idx, const float *__restrict__ val,
                                                           const void *__restrict__ Theta, int64_t s0, int len,
                                                           v4f (&acc)[tiles_in(ROWS)], float (&b)[tiles_1d(F)],
                                                           uint32_t *stage, int wave, uint32_t absmax_bits) {
    static_assert(F == 256 && NW == 8, "16 tiles, two 16-byte loads per row and lane, 8 wavefronts x 4 entries");
    constexpr int NT = tiles_1d(F);
    constexpr int RMAX = 31 - __builtin_clz(ROWS);
    constexpr int STAGE = 2 * NT * 256;   // words per staging buffer: tile T, part k at (2 T + k) * 256
    const int lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
    const int p = kq & 1, hf = kq >> 1;
    float scale, inv_scale;
    two_part_scale(absmax_bits, scale, inv_scale);
    const int32_t *__restrict__ ib = idx + s0;
    const float *__restrict__ vb = val + s0;
    constexpr int kRsrcFlags = 0x00020000;
    const __amdgpu_buffer_rsrc_t ids_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(ib), 0, 4 * len, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t val_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(vb), 0, 4 * len, kRsrcFlags);
    const int nsteps = (len + 31) >> 5;
    const int e_in_step = 4 * wave + 2 * p;                 // first of this lane's two entries inside a step
    const uint32_t e_off = 4u * (uint32_t)e_in_step;
    const uint32_t lane_a = 16u * (uint32_t)i + 512u * (uint32_t)hf;   // bytes into the row: tiles 8hf .. 8hf+7
    // word of (tile, part, this lane's pair) in a staging buffer: lane (i, kq') of the consumers, register m
    const int P = 2 * wave + p;
    const int w_base = 8 * hf * 512 + (16 * (P >> 2) + i) * 4 + (P & 3);

    struct Pair { uint32_t a, b; };
    auto load_pair_ids = [&](int t) -> Pair {   // (beyond the end of the work item: 0, i.e. row 0, masked below)
        Pair r;
        r.a = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(ids_rsrc, e_off + 128u * (uint32_t)t, 0, 0);
        r.b = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(ids_rsrc, e_off + 4u + 128u * (uint32_t)t, 0, 0);
        return r;
    };
    struct Rows { v4f v[2][2]; float r[2]; };   // 8 features of two rows, their ratings
    auto gather = [&](uint32_t c, v4f (&v)[2]) {
        const char *q = reinterpret_cast<const char *>(Theta);
        if constexpr (WIDE) q += (int64_t)c * (4 * F) + lane_a;
        else q += row_offset<(uint32_t)(4 * F)>(c, lane_a);
        v[0] = *reinterpret_cast<const v4f *>(q);
        v[1] = *reinterpret_cast<const v4f *>(q + 256);
    };
    auto fetch = [&](Rows &w, const Pair &ids, int t) {
        gather(ids.a, w.v[0]);
        gather(ids.b, w.v[1]);
        w.r[0] = bits_to_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b32(val_rsrc, e_off + 128u * (uint32_t)t, 0, 0));
        w.r[1] = bits_to_float((uint32_t)__builtin_amdgcn_raw_buffer_load_b32(val_rsrc, e_off + 4u + 128u * (uint32_t)t, 0, 0));
    };
    float bacc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) bacc[k] = 0.f;
    // rows of step t -> staging buffer and b_u; entries beyond the work item count as zero
    auto stage_rows = [&](const Rows &w, int t, uint32_t *buf) {
        const int e = 32 * t + e_in_step;
        const bool ok0 = e < len, ok1 = e + 1 < len;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float x0 = ok0 ? w.v[0][k >> 2][k & 3] : 0.f, x1 = ok1 ? w.v[1][k >> 2][k & 3] : 0.f;
            bacc[k] = fmaf(w.r[1], x1, fmaf(w.r[0], x0, bacc[k]));
            uint32_t h, l;
            split_two(x0, x1, scale, h, l);
            buf[w_base + 512 * k] = h;
            buf[w_base + 512 * k + 256] = l;
        }
    };

    // Gathers run PD steps ahead of their use; the column ids one step further
    constexpr int PD = ALS_X2_SHARED_DEPTH;
    Rows raw[PD];
    Pair ids = load_pair_ids(0);
#pragma unroll
    for (int u = 0; u < PD; ++u) {   // (steps beyond the last read row 0 and are never used)
        fetch(raw[u], ids, u);
        ids = load_pair_ids(u + 1);
    }
    stage_rows(raw[0], 0, stage);
    fetch(raw[0], ids, PD);
    ids = load_pair_ids(PD + 1);
    __syncthreads();
    auto step = [&](auto utag, int t) {
        constexpr int S = (decltype(utag)::value + 1) % PD;   // register set of step t+1, reused for step t+1+PD
        const uint32_t *cur = stage + (t & 1) * STAGE;
        if (t + 1 < nsteps) {   // rows of the next step into the other buffer, then their registers take new gathers
            stage_rows(raw[S], t + 1, stage + ((t + 1) & 1) * STAGE);
            fetch(raw[S], ids, t + 1 + PD);
            ids = load_pair_ids(t + 2 + PD);
        }
        auto part = [&](int T, int k) -> v4u { return *reinterpret_cast<const v4u *>(cur + (2 * T + k) * 256 + 4 * lane); };
        v4u hr[NT], lr[NT];   // (only those of ROWS are ever loaded)
#pragma unroll
        for (int R = 0; R < NT; ++R)
            if ((ROWS >> R) & 1u) { hr[R] = part(R, 0); lr[R] = part(R, 1); }
#pragma unroll
        for (int C = 0; C <= RMAX; ++C) {
            const v4u h = ((ROWS >> C) & 1u) ? hr[C] : part(C, 0), l = ((ROWS >> C) & 1u) ? lr[C] : part(C, 1);
#pragma unroll
            for (int R = C; R < NT; ++R)
                if ((ROWS >> R) & 1u) {
                    v4f &a = acc[tiles_below(ROWS, R) + C];
                    mfma_16x16x32<ALS_F16>(a, hr[R], l);
                    mfma_16x16x32<ALS_F16>(a, lr[R], h);
                    mfma_16x16x32<ALS_F16>(a, hr[R], h);
                }
        }
        __syncthreads();   // the next buffer is complete; everybody is done reading this one
    };
    for (int t0 = 0; t0 < nsteps; t0 += PD) {
        [&]<int... u>(std::integer_sequence<int, u...>) {
            ((t0 + u < nsteps ? step(std::integral_constant<int, u>{}, t0 + u) : void()), ...);
        }(std::make_integer_sequence<int, PD>{});
    }
    const float inv2 = inv_scale * inv_scale;   // sums of (s theta)(s theta'): back to the caller's scale, exactly
#pragma unroll
    for (int q = 0; q < tiles_in(ROWS); ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[q][r] *= inv2;
    // b_u: the two entry pairs of a wavefront, then the wavefronts in order
    float *red = reinterpret_cast<float *>(stage);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        bacc[k] += __shfl_xor(bacc[k], 16);
        if (p == 0) red[wave * F + 16 * (8 * hf + k) + i] = bacc[k];
    }
    __syncthreads();
#pragma unroll
    for (int T = 0; T < NT; ++T) {
        float s = 0.f;
        if ((ROWS >> T) & 1u)
            for (int w = 0; w < NW; ++w) s += red[w * F + 16 * T + i];
        b[T] = s;
    }
}

}  // namespace als
