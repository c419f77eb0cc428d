// GroupNorm over slabs of whole groups: a workgroup owns (sample, slab of whole groups, slice of the positions), held packed in
// its registers (NV vectors a lane).  A slab that is one slice has its statistics to itself: nothing is exchanged between workgroups, no workgroup
// waits.  Several slices of a slab exchange one word a group each, and a workgroup reads the words of its own groups, where a
// workgroup of whole positions (group_kernel) reads those of every group of the sample.
//
// Bound: the chain load -> statistics -> (exchange) -> store of a workgroup, all of them resident at once.
#pragma once
#include "pf_group_kernels.hpp"

namespace pf {

// Statistics: per element slot the mean over the lane's positions (its first value and the mean distance from that), then the squared deviations from it; PACKED (16-bit storage, an even
// number of channels to a group, nothing but the load in front): sums and sums of squares per pair of elements, as in the
// general group kernels.  They are merged as (count, mean, M2) triples, one per group the vector touches.
//
// Exchange (SLICED): as in group_kernel, self-describing words in two parities, with the launch's number kept on the device: a word of the
// workgroup's own, which nobody else touches.  All workgroups of a launch with slices are resident together on an idle device; where
// two such launches share it, the order of the workgroups (group_slab_place) lets runs of slabs complete and make room.
template <int DT, int NV, int CVS, class Spec, bool SLICED, bool PACKED>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(NV > 16 ? 2 : 4))) group_slab_kernel(const ChainArgs a, const GroupSlabGeom g) {
    using S = Storage<DT>;
    constexpr int VEC = S::VEC;
    constexpr uint32_t PPS = 512u / (uint32_t)CVS;  // positions per step
    extern __shared__ float lds[];                  // [512][parts] (count, mean, M2)
    __shared__ float lds_stat[2 * 512];
    using P = typename Spec::Pro;
    static_assert(Spec::kStatic && P::n == 1 && P::at(0).code == U_MOV && P::at(0).kind == K_FULL, "nothing but the load in front");
    // What the address of the first load takes of the arguments, asked for together: where the compiler places them they are up to four
    // trips to memory, one behind the other (0.2 to 0.4 us of every call: [1, 64, 64, 448] fp32 11.4 -> 11.0, [2, 72, 72, 544] bf16 16.4 -> 15.7)
    asm volatile("" ::"s"(a.full[P::at(0).slot]), "s"(g.hw), "s"(g.channels), "s"(g.cpg), "s"(g.slab_groups), "s"(g.blocks), "s"(g.blocks_per_die), "s"(g.div_sample.m));
    if (SLICED) asm volatile("" ::"s"(g.slice_len), "s"(g.slice_rest), "s"(g.div_run.m), "s"(g.div_run_slabs.m), "s"(g.ws_epoch));
    const GroupSlabPlace place = group_slab_place<SLICED>(blockIdx.x, g.blocks_per_die, g.div_run, g.div_sample, g.div_run_slabs);
    const uint32_t at = place.at, sample = place.sample, in_sample = place.slab, slice = place.slice;
    if (at >= g.blocks) return;  // (the grid is rounded up to a multiple of eight)
    const uint32_t p_begin = SLICED ? slice * g.slice_len + min(slice, g.slice_rest) : 0u;
    const uint32_t p_count = SLICED ? g.slice_len + (slice < g.slice_rest ? 1u : 0u) : g.hw;
    const uint32_t epoch = SLICED ? g.ws_epoch[at] : 0u;
    const uint32_t grp0 = in_sample * g.slab_groups;
    const uint32_t ch0 = grp0 * g.cpg, ch1 = ch0 + g.slab_groups * g.cpg;
    const uint32_t v0 = ch0 / (uint32_t)VEC;
    const uint32_t t = threadIdx.x;
    const uint32_t pstep = t / (uint32_t)CVS, cvl = t - pstep * (uint32_t)CVS;
    const uint32_t ch = (v0 + cvl) * (uint32_t)VEC;  // the lane's first channel
    const bool active = pstep < PPS && ch < ch1;

    // ---- the slab into registers.  No branch around a load: a lane without a vector reads the slice's first.
    const uint64_t slice_bytes = ((uint64_t)sample * g.hw + p_begin) * g.channels * S::ESIZE;
    const char* base = static_cast<const char*>(a.full[P::at(0).slot]) + slice_bytes;
    const uint32_t step_bytes = PPS * g.channels * (uint32_t)S::ESIZE;
    const uint32_t first_bytes = v0 * 16u;
    const uint32_t lane_bytes = active ? pstep * g.channels * (uint32_t)S::ESIZE + (v0 + cvl) * 16u : first_bytes;
    const bool last_valid = active && (uint32_t)(NV - 1) * PPS + pstep < p_count;  // (every step but the last is whole)
    // (a slice one position shorter than the others may have nothing in the last step: its first vector again)
    const uint32_t last_step = (uint32_t)(NV - 1) * PPS < p_count ? (uint32_t)(NV - 1) : 0u;
    u32x4 raw[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i)
        raw[i] = *reinterpret_cast<const u32x4*>(base + (size_t)((i + 1 < NV ? (uint32_t)i : last_step) * step_bytes) + (i + 1 < NV || last_valid ? lane_bytes : first_bytes));
    LaneState<DT, 1, Spec> s;
    s.col[0] = ch;
    constexpr int gs = Spec::kGamma, bs = Spec::kBeta;
#pragma unroll
    for (int v = 0; v < Spec::NV; ++v) s.vraw[v][0] = load_vec_operand<DT, Spec::kVecMode>(a.vec[v], 0u, active ? ch : v0 * (uint32_t)VEC, g.channels);
    auto keep_packed = [&](int i) {  // (the widened values are not kept from pass to pass)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t w = raw[i][j];
            asm volatile("" : "+v"(w));
            raw[i][j] = w;
        }
    };

    // ---- statistics
    {
        const float npos = active ? (float)(NV - 1) + (last_valid ? 1.0f : 0.0f) : 0.0f;
        const float inv = npos > 0.0f ? 1.0f / npos : 0.0f;
        constexpr int SLOTS = PACKED ? VEC / 2 : VEC, PER = VEC / SLOTS;  // elements to a slot
        float mean_e[SLOTS], m2_e[SLOTS];
#pragma unroll
        for (int e = 0; e < SLOTS; ++e) mean_e[e] = m2_e[e] = 0.0f;
        if constexpr (PACKED) {
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                if (i + 1 < NV || last_valid) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const uint32_t w = raw[i][j];
                        if (DT == DT_F16) {
                            const f16x2 x = __builtin_bit_cast(f16x2, w), ones = {(_Float16)1.0f, (_Float16)1.0f};
                            mean_e[j % SLOTS] = __builtin_amdgcn_fdot2(x, ones, mean_e[j % SLOTS], false);
                            m2_e[j % SLOTS] = __builtin_amdgcn_fdot2(x, x, m2_e[j % SLOTS], false);
                        } else {
                            const bf16x2 x = __builtin_bit_cast(bf16x2, w), ones = {(__bf16)1.0f, (__bf16)1.0f};
                            mean_e[j % SLOTS] = __builtin_amdgcn_fdot2_f32_bf16(x, ones, mean_e[j % SLOTS], false);
                            m2_e[j % SLOTS] = __builtin_amdgcn_fdot2_f32_bf16(x, x, m2_e[j % SLOTS], false);
                        }
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < SLOTS; ++j) {
                // (with its remainder: the mean of seven positions off by the rounded reciprocal's error, the same way in every lane, would
                // put the variance around an offset of 100 off by 4e-4)
                const float sum = mean_e[j], q = sum * (inv * 0.5f);
                mean_e[j] = __builtin_fmaf(__builtin_fmaf(-2.0f * npos, q, sum), inv * 0.5f, q);
                m2_e[j] = fmaxf(m2_e[j] - sum * mean_e[j], 0.0f);
            }
        } else {
            // From the lane's first value on: a sum times the rounded reciprocal of seven is off the same way in every lane (fp32 around 1000: the
            // mean by 0.7 of its last place), and equal values would not be their own mean.
            float first_x[VEC];
            S::unpack(raw[0], first_x);
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                float x[VEC];
                S::unpack(raw[i], x);
                if (i + 1 < NV || last_valid) {
#pragma unroll
                    for (int e = 0; e < SLOTS; ++e) mean_e[e] += x[e] - first_x[e];
                }
            }
#pragma unroll
            for (int e = 0; e < SLOTS; ++e) mean_e[e] = npos > 0.0f ? __builtin_fmaf(mean_e[e], inv, first_x[e]) : 0.0f;
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                keep_packed(i);
                float x[VEC];
                S::unpack(raw[i], x);
                if (i + 1 < NV || last_valid) {
#pragma unroll
                    for (int e = 0; e < SLOTS; ++e) {
                        const float d = x[e] - mean_e[e];
                        m2_e[e] = __builtin_fmaf(d, d, m2_e[e]);
                    }
                }
            }
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) keep_packed(i);
        // one triple per group the vector touches, adjacent slots merged
        const uint32_t first = fast_div(min(ch, g.channels - 1u), g.div_cpg);
        const float n_slot = npos * (float)PER;
        Stat cur = {n_slot, mean_e[0], m2_e[0]};
        uint32_t part = 0;
#pragma unroll
        for (int e = 1; e <= SLOTS; ++e) {
            const uint32_t next = e < SLOTS ? fast_div(min(ch + (uint32_t)(e * PER), g.channels - 1u), g.div_cpg) - first : g.parts;
            const bool flush = next != part;
            if (flush) {
                float* q = lds + (t * g.parts + part) * 3u;
                q[0] = cur.n;
                q[1] = cur.mean;
                q[2] = cur.m2;
            }
            if (e < SLOTS) {
                const Stat slot = {n_slot, mean_e[e % SLOTS], m2_e[e % SLOTS]};
                cur = flush ? slot : stat_merge<S::PRECISE>(cur, slot);
                part = next;
            }
        }
    }
    __syncthreads();
    {
        // 2^log2_lanes adjacent lanes share a group and walk the lanes whose vectors touch it
        const uint32_t lanes = 1u << g.log2_lanes, q = t >> g.log2_lanes, j = t & (lanes - 1u);
        const bool in_range = q < g.slab_groups;
        Stat st = {0.0f, 0.0f, 0.0f};
        if (in_range) {
            const uint32_t lo = (ch0 + q * g.cpg) / (uint32_t)VEC, hi = (ch0 + (q + 1u) * g.cpg - 1u) / (uint32_t)VEC;
            const uint32_t ncv = hi - lo + 1u;
            uint32_t ps = j / ncv, k = j - ps * ncv;
            const uint32_t d_ps = lanes / ncv, d_k = lanes - d_ps * ncv;
            while (ps < PPS) {
                const uint32_t part = grp0 + q - fast_div((lo + k) * (uint32_t)VEC, g.div_cpg);
                const float* w = lds + ((ps * (uint32_t)CVS + lo - v0 + k) * g.parts + part) * 3u;
                st = stat_merge<S::PRECISE>(st, Stat{w[0], w[1], w[2]});
                ps += d_ps;
                k += d_k;
                if (k >= ncv) k -= ncv, ++ps;
            }
        }
        for (uint32_t m = 1; m < lanes; m <<= 1) st = stat_merge<S::PRECISE>(st, stat_shfl_xor(st, (int)m));
        if constexpr (SLICED) {
            if (in_range) {
                uint64_t* words = g.ws_gather + (epoch & 1u) * g.gather_words + ((uint64_t)sample * g.groups + grp0 + q) * g.slices;
                if (j == 0u) {
                    uint64_t* other = g.ws_gather + ((epoch & 1u) ^ 1u) * g.gather_words + ((uint64_t)sample * g.groups + grp0 + q) * g.slices;
                    __hip_atomic_store(other + slice, kSlotEmpty, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(words + slice, pack_slot(st.mean, st.m2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                st = Stat{0.0f, 0.0f, 0.0f};
                uint32_t spins = 0;
                for (uint32_t b = j; b < g.slices; b += lanes) {
                    uint64_t w;
                    for (;;) {
                        w = __hip_atomic_load(words + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if (w != kSlotEmpty) break;
                        if (++spins >= g.spin_limit) {
                            __hip_atomic_store(g.ws_error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            break;
                        }
                        __builtin_amdgcn_s_sleep(8);
                    }
                    if (w == kSlotEmpty) continue;
                    st = stat_merge<S::PRECISE>(st, Stat{(float)((g.slice_len + (b < g.slice_rest ? 1u : 0u)) * g.cpg), __builtin_bit_cast(float, (uint32_t)w),
                                             __builtin_bit_cast(float, (uint32_t)(w >> 32))});
                }
            }
            for (uint32_t m = 1; m < lanes; m <<= 1) st = stat_merge<S::PRECISE>(st, stat_shfl_xor(st, (int)m));
        }
        if (in_range && j == 0u) {
            lds_stat[q * 2u] = st.mean;
            lds_stat[q * 2u + 1u] = 1.0f / sqrtf((st.n > 0.0f ? st.m2 / st.n : 0.0f) + a.eps);
        }
    }
    __syncthreads();
    if (SLICED && t == 0u) g.ws_epoch[at] = epoch + 1u;

    // ---- normalise from registers, as group_kernel does: one multiply-add an element; fp32 chains subtract the mean first
    constexpr bool kCentre = DT == DT_F32;
    float A[VEC], B[VEC], M[VEC];
    {
        float gm[VEC], bt[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            gm[e] = 1.0f;
            bt[e] = 0.0f;
        }
        if (gs >= 0) fetch_vec<DT, 1, Spec>(s, gs, gm);
        if (bs >= 0) fetch_vec<DT, 1, Spec>(s, bs, bt);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const uint32_t q = fast_div(min(ch + (uint32_t)e, ch1 - 1u), g.div_cpg) - grp0;
            M[e] = lds_stat[q * 2u];
            A[e] = lds_stat[q * 2u + 1u] * gm[e];
            B[e] = kCentre ? bt[e] : bt[e] - M[e] * A[e];
        }
    }
    char* out_base = static_cast<char*>(a.out[0]) + slice_bytes;
    // (multiplied anew: kept from the loads, the steps' offsets need more scalar registers than there are)
    uint32_t out_step_bytes = step_bytes;
    asm volatile("" : "+s"(out_step_bytes));
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        float x[VEC];
        S::unpack(raw[i], x);
        s.fraw[P::at(0).slot][0] = raw[i];  // (the steps behind may read the input again: x + norm(x))
        s.row[0] = sample * g.hw + p_begin + (uint32_t)i * PPS + pstep;  // (a mask reads the position)
#pragma unroll
        for (int e = 0; e < VEC; ++e) s.acc[e] = __builtin_fmaf(kCentre ? x[e] - M[e] : x[e], A[e], B[e]);
        run_program<DT, 1, Spec>(ProgView<typename Spec::Epi>{a.epi}, s, NoStore{});
        if (i + 1 < NV ? active : last_valid) *reinterpret_cast<u32x4*>(out_base + (size_t)((uint32_t)i * out_step_bytes) + lane_bytes) = S::pack(s.acc);
    }
}

}  // namespace pf
