// Column family: layer / RMS normalisation over a dimension that is NOT the innermost one.
//
// A channels-first tensor [outer, C, S] (S = everything after the normalised dimension, contiguous) normalised
// over C is usually written as: move C to the end, normalise rows, move it back -- three kernels and three times
// the bytes when each step is a kernel of its own.  The paper's rewriting (section 5: operators swapped across
// data movement until reads and writes of the same slice merge) removes both layout changes: the reduction runs
// over a strided dimension instead.  Here a workgroup of T lanes owns a slab [C, 8 vectors of S]: lane (row group
// rg = tid / 8, column col = tid % 8) loads the 16-byte vectors of rows rg, rg + T / 8, ... at column col -- every load
// instruction of a wave reads 8 rows x 128 contiguous bytes, like the tile transposition -- and keeps them in
// registers (KC vectors per lane, so C <= T / 8 * KC).  The statistics of one position are spread over the row groups:
// three lane exchanges inside a wave (lanes 8, 16, 32 apart hold the same column), then one LDS exchange between the
// waves (one barrier each).  Mean first (as differences from a pivot row), then centred squares: no cancellation; RMS
// needs one exchange.  Every input element is read once and every output element written once; nothing is transposed.
//
// Bound: with few slabs the chain load -> exchange -> exchange -> store of a workgroup, not bandwidth.  [64, 384, 14, 14]
// fp16, 256 slabs: 18.0 us; with the parameters fetched once per workgroup and neighbouring slabs on one die 17.1; with
// 1024 lanes to a slab instead of 256 9.5.
#pragma once
#include "pf_device.hpp"

namespace pf {

constexpr uint32_t kColMax = 1024u;  // longest column (normalised extent)

// v + the same value of the lane 8, 16 and 32 further on: a row rotation and the two lane-row swaps
PF_DEVICE float col_wave_sum(float v) {
    v += dpp_move<0x128>(v);  // row_ror:8
    {
        const uint32_t w = __builtin_bit_cast(uint32_t, v);
        const auto s = __builtin_amdgcn_permlane16_swap(w, w, false, false);
        const uint32_t s0 = s[0], s1 = s[1];
        v = __builtin_bit_cast(float, s0) + __builtin_bit_cast(float, s1);
    }
    const uint32_t w = __builtin_bit_cast(uint32_t, v);
    const auto s = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    const uint32_t s0 = s[0], s1 = s[1];
    return __builtin_bit_cast(float, s0) + __builtin_bit_cast(float, s1);
}

// Sum over all row groups, per position: every lane ends with the sums of its own column's VEC positions.  part: [waves]
// [8 * VEC] partial sums, total: [waves][8 * VEC] a copy of the result per wave (each exchange of a kernel has LDS areas
// of its own: no barrier in front).
template <int VEC, int T>
PF_DEVICE void col_all_reduce(float (&v)[VEC], float* part, float* total, uint32_t wave, uint32_t col, uint32_t lane) {
    constexpr uint32_t P = 8u * VEC, W = (uint32_t)T / 64u;
#pragma unroll
    for (int j = 0; j < VEC; ++j) v[j] = col_wave_sum(v[j]);
    if (lane < 8u) {
#pragma unroll
        for (int j = 0; j < VEC; ++j) part[wave * P + col * VEC + j] = v[j];
    }
    __syncthreads();
    // one position per lane, all waves alike; the copy a wave reads back is its own, so no barrier is needed
    if (lane < P) {
        float s = part[lane];
#pragma unroll
        for (uint32_t w = 1; w < W; ++w) s += part[w * P + lane];
        total[wave * P + lane] = s;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < VEC; ++j) v[j] = total[wave * P + col * VEC + j];
}

// The slab stays in registers in its storage form between the passes: the compiler may not keep the unpacked values
// of one pass alive for the next.
template <int KC>
PF_DEVICE void keep_packed(u32x4 (&raw)[KC]) {
#pragma unroll
    for (int k = 0; k < KC; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t w = raw[k][i];
            asm volatile("" : "+v"(w));
            raw[k][i] = w;
        }
}

// RAGGED: the extent after the normalised dimension is not a whole number of 16-byte vectors (7 x 7 or 14 x 14
// positions of 16-bit data): rows start at element alignment and the last vector of a row is partial.
template <int DT, int KC, bool RMS, bool RAGGED = false, int T = 256>
__global__ void __launch_bounds__(T) colnorm_kernel(const ColArgs a) {
    using S = Storage<DT>;
    constexpr int VEC = S::VEC;
    constexpr uint32_t RG = (uint32_t)T / 8u;  // row groups
    constexpr int NP = (int)(((uint32_t)KC * RG < kColMax ? (uint32_t)KC * RG : kColMax) + T - 1) / T;
    __shared__ float lds_part[2][T / 64 * 8 * VEC], lds_total[2][T / 64 * 8 * VEC];
    __shared__ float lds_gamma[NP * T], lds_beta[NP * T];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, col = tid & 7u, rg = tid >> 3;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Workgroups are dealt to the eight compute dies round-robin; neighbouring slabs, which share memory lines wherever rows
    // are not whole lines, are numbered so that they fall on the same die (each has its own L2).
    const uint32_t tile = (blockIdx.x & 7u) * a.tiles_per_die + (blockIdx.x >> 3);
    if (tile >= a.tiles) return;
    const uint32_t o = tile / a.tiles_per_outer, t = tile - o * a.tiles_per_outer;
    const uint32_t sv = t * 8u + col;
    const bool col_ok = sv < a.s_vecs;
    const uint32_t cnt = RAGGED ? elems_below<VEC>(sv * VEC, a.s) : (uint32_t)VEC;  // elements of this lane's vector inside the row
    const uint64_t base = ((uint64_t)o * a.c) * a.s + (uint64_t)sv * VEC;  // element offset of row 0 at this column

    // Whole vectors are loaded without a branch: a lane whose row or column does not exist reads the last one that does
    // (the line a neighbour reads anyway) and never uses or stores the value.  Behind a guard every load would merge
    // with a fill value at the join, which the compiler resolves by waiting for it: the loads of a lane, all
    // independent, would then go to memory one round trip after the other.
    const uint64_t base_ld = RAGGED ? base : ((uint64_t)o * a.c) * a.s + (uint64_t)min(sv, a.s_vecs - 1u) * VEC;
    // (RAGGED: a lane's vector is whole, partial or absent for all its rows alike, so the three cases are told apart once,
    // outside the loop over the rows, and each runs its loads back to back)
    u32x4 raw[KC];
    if (!RAGGED || cnt == (uint32_t)VEC) {
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            const uint64_t elem = base_ld + (uint64_t)min(rg + RG * (uint32_t)k, a.c - 1u) * a.s;
            raw[k] = RAGGED ? load_elems<DT>(a.x, elem, (uint32_t)VEC, 0u) : load_stream(a.x, elem * S::ESIZE);
        }
    } else if (cnt != 0u) {
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            // (what follows a partial vector is the next row of the tensor, unless this is its last row)
            const uint32_t c = min(rg + RG * (uint32_t)k, a.c - 1u);
            raw[k] = load_elems<DT>(a.x, base + (uint64_t)c * a.s, cnt, 0u, c + 1u < a.c || tile + a.tiles_per_outer < a.tiles);
        }
    } else {
#pragma unroll
        for (int k = 0; k < KC; ++k) raw[k] = u32x4{0u, 0u, 0u, 0u};
    }
    // mean = piv + mean[]: kept as a pivot (row 0 of the same position) plus the mean of the differences from it, so
    // that a large common offset of the values eats the digits neither of the sum nor of x - mean
    // (every lane fetches the pivot row itself: the row groups of a column read the same 16 bytes, which the cache
    // serves, and no barrier is needed to share them)
    u32x4 piv_raw = u32x4{0u, 0u, 0u, 0u};
    if (!RMS) {
        if (!RAGGED) piv_raw = load_cached(a.x, base_ld * S::ESIZE);
        else if (col_ok) piv_raw = load_elems<DT>(a.x, base, cnt, 0u);
    }
    // The parameters, once per workgroup, shared through LDS by the barrier of the first exchange (fetched by every lane for
    // its own rows they were two 2-byte loads per 16-byte vector of the slab: twice the load instructions of the data).
    float gam_own[NP], bet_own[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const uint64_t off = (uint64_t)min(tid + (uint32_t)(p * T), a.c - 1u) * S::ESIZE;
        float tmp[VEC];
        S::unpack(S::splat(static_cast<const char*>(a.gamma) + off), tmp);
        gam_own[p] = tmp[0];
        S::unpack(S::splat(static_cast<const char*>(RMS ? a.gamma : a.beta) + off), tmp);
        bet_own[p] = RMS ? 0.0f : tmp[0];
    }
    float piv[VEC], mean[VEC], acc[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) piv[j] = 0.0f, mean[j] = 0.0f, acc[j] = 0.0f;
    if (!RMS) {
        S::unpack(piv_raw, piv);
#pragma unroll
        for (int k = 0; k < KC; ++k) {
            if (rg + RG * (uint32_t)k < a.c) {
                float x[VEC];
                S::unpack(raw[k], x);
#pragma unroll
                for (int j = 0; j < VEC; ++j) mean[j] += x[j] - piv[j];
            }
        }
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        lds_gamma[tid + (uint32_t)(p * T)] = gam_own[p];
        lds_beta[tid + (uint32_t)(p * T)] = bet_own[p];
    }
    if (!RMS) {
        col_all_reduce<VEC, T>(mean, lds_part[0], lds_total[0], wave, col, lane);
#pragma unroll
        for (int j = 0; j < VEC; ++j) mean[j] *= a.inv_c;
        keep_packed<KC>(raw);
    }
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        if (rg + RG * (uint32_t)k < a.c) {
            float x[VEC];
            S::unpack(raw[k], x);
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                const float d = (x[j] - piv[j]) - mean[j];
                acc[j] = fmaf(d, d, acc[j]);
            }
        }
    }
    col_all_reduce<VEC, T>(acc, lds_part[1], lds_total[1], wave, col, lane);
    keep_packed<KC>(raw);
    float rstd[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) rstd[j] = pf_rsqrt<S::PRECISE>(fmaf(acc[j], a.inv_c, a.eps));
#pragma unroll
    for (int k = 0; k < KC; ++k) {
        const uint32_t c = rg + RG * (uint32_t)k;
        if (!(col_ok && c < a.c)) continue;
        const float gam = lds_gamma[c], bet = lds_beta[c];
        float x[VEC];
        S::unpack(raw[k], x);
#pragma unroll
        for (int j = 0; j < VEC; ++j) x[j] = fmaf(((x[j] - piv[j]) - mean[j]) * rstd[j], gam, bet);
        if (RAGGED) store_elems<DT>(a.out, base + (uint64_t)c * a.s, cnt, S::pack(x));
        else store_stream(a.out, (base + (uint64_t)c * a.s) * S::ESIZE, S::pack(x));
    }
}

}  // namespace pf
