// Pool family: prologue -> reduction over the positions of a channels-last tensor (sum, maximum or mean over
// every dimension between the first and the last: global pooling of x [n, spatial.., c] into [n, 1.., c]) ->
// epilogue on the pooled values.
//
// This is the reduce basic operator (paper section 6) along dimensions that are not contiguous in memory.  A
// workgroup walks a channel slab of each position of its slice (whole positions, fully contiguous, where a position is one
// slab), and every lane owns one channel vector, so the running reduction lives in registers and no value crosses lanes
// until the workgroup's slice is done (one pass through LDS).  A slab's positions are spread over several workgroups: each
// publishes its per-channel partial result; the slab's last workgroup waits for those words, merges them, runs the epilogue
// and stores -- the device-scope synchronisation of section 5.1.
#pragma once
#include "pf_group_kernels.hpp"

namespace pf {

enum PoolOp : int32_t { POOL_SUM = 0, POOL_MAX = 1, POOL_MEAN = 2 };


template <int OP>
PF_DEVICE float pool_identity() { return OP == POOL_MAX ? -__builtin_inff() : 0.0f; }
// maximum that keeps a NaN once it has seen one (the operator's definition: a NaN element poisons the result)
template <int OP>
PF_DEVICE float pool_combine(float acc, float x) {
    if (OP != POOL_MAX) return acc + x;
    return pf_max_nan(acc, x);
}

// A partial result as a published word: all-ones means "not written in this launch" (a NaN that arithmetic never
// produces; a NaN result with that payload is published as the canonical one).
constexpr uint32_t kPoolEmpty = ~0u;
PF_DEVICE uint32_t pool_word(float x) {
    const uint32_t w = __builtin_bit_cast(uint32_t, x);
    return w == kPoolEmpty ? 0x7fc00000u : w;
}

// log2 of the largest power of two that is at most v, and at most 64 lanes
constexpr uint32_t floor_log2_64(uint32_t v) { return v >= 64u ? 6u : v >= 2u ? 1u + floor_log2_64(v / 2u) : 0u; }
// One value per channel from `rows` rows of `words` channels in LDS, returned to lane t for channel t.  2^log2_lanes adjacent lanes share a
// channel, each takes a strided subset of the rows, a shuffle tree merges them and the value is passed on through out[channel]
// (another area); one lane to a channel (log2_lanes 0) needs no more than its own reads.  words << log2_lanes is at most the workgroup.
// Callers put a barrier in front.  (Rows merged one LDS read after the other, then eight channels by one lane, were a chain
// of 256 reads for 16 channels: mean over [5, 64, 64, 16] fp16 9.3 us, 5.4 so; [36, 28, 28, 64] bf16 7.2, 5.8.  A plain loop: instructions
// come from memory at the start of a launch, and reads unrolled four deep cost [32, 56, 56, 240] + SiLU 0.4 us of 13.2.)
template <int OP>
PF_DEVICE float pool_reduce_rows(const float* rows_lds, float* out, uint32_t rows, uint32_t words, uint32_t log2_lanes) {
    const uint32_t ch = threadIdx.x >> log2_lanes, lanes = 1u << log2_lanes, r = threadIdx.x & (lanes - 1u);
    float m = pool_identity<OP>();
    if (ch < words) {
#pragma unroll 1
        for (uint32_t q = r; q < rows; q += lanes) m = pool_combine<OP>(m, rows_lds[q * words + ch]);
    }
    if (log2_lanes != 0u) {
#pragma unroll 1
        for (uint32_t x = 1; x < lanes; x <<= 1) m = pool_combine<OP>(m, __shfl_xor(m, (int)x, 64));
        if (ch < words && r == 0u) out[ch] = m;
        __syncthreads();
        if (threadIdx.x < words) m = out[threadIdx.x];
    }
    return m;
}

// A group normalisation in front of the pooling (U_GNORM in the prologue).  Its statistics come from an earlier launch (the
// group family's statistics kernel); a workgroup lies in one sample and a lane owns its channels, so mean and scale of
// the lane's channels are merged once and every element costs a subtraction and a multiply-add.  The normalised
// tensor, which only the pooling reads, never exists in memory: the chain reads x twice and writes the pooled
// values, where a normalisation kernel and a pooling kernel with an fp32 tensor between them moved nine times x
// (GroupNorm + SiLU + mean of [32, 64, 64, 320] fp16).  Many (sample, group) pairs take norm_pool_slab_kernel below instead.
template <int VEC>
struct PoolNorm {
    float mean[VEC], scale[VEC], shift[VEC];
    template <int DT, int K, class Spec>
    PF_DEVICE void operator()(int, const LaneState<DT, K, Spec>&) const {}
};
template <int VEC, int DT, class Spec>
PF_DEVICE void hook_norm(const PoolNorm<VEC>& h, LaneState<DT, 1, Spec>& s) {
    using P = typename Spec::Pro;
    // fp16 straight from memory: widened by the subtraction itself (v_fma_mix_f32: x * 1 - mean, one rounding either way)
    if constexpr (DT == DT_F16 && P::n >= 2 && P::at(0).code == U_MOV && P::at(0).kind == K_FULL && P::at(1).code == U_GNORM) {
        const u32x4 x = s.fraw[P::at(0).slot][0];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t xp = x[j];
            float d0, d1;
            asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(d0) : "v"(xp), "v"(h.mean[(2 * j) % VEC]));
            asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(d1) : "v"(xp), "v"(h.mean[(2 * j + 1) % VEC]));
            s.acc[(2 * j) % VEC] = __builtin_fmaf(d0, h.scale[(2 * j) % VEC], h.shift[(2 * j) % VEC]);
            s.acc[(2 * j + 1) % VEC] = __builtin_fmaf(d1, h.scale[(2 * j + 1) % VEC], h.shift[(2 * j + 1) % VEC]);
        }
        return;
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) s.acc[e] = __builtin_fmaf(s.acc[e] - h.mean[e], h.scale[e], h.shift[e]);
}

// RAGGED: a channel count that is not a whole number of 16-byte vectors.  A position then starts at element alignment
// and its last vector holds `cnt` channels: elements past them are never read or stored (their accumulator slots carry
// whatever the prologue makes of the fill value and stay in the lane).
//
// A workgroup owns (sample, channel slab, slice of the positions): at most 512 channels, so a slice's partial result is a
// word per lane at most, and as many slices as fill the device.
//
// Bound: one trip to memory, the steps of the slice, then the exchange (3 us).  [32, 56, 56, 240] fp16 + SiLU, 48 MB: 12.7 us with
// slices of one chunk, 12.1 with two chunks that refill; [24, 35, 35, 832] fp16 15.7 us in one slab of 104 vectors, 11.6 in two, 12.3 in the thirteen that
// the plan takes (whole memory lines).  CHUNKED: false when a slice is NV steps at most.
// Registers for two workgroups to a unit: [32, 56, 56, 244] behind four steps 62 us, 81 with one (the plan takes shorter chunks where
// vectors would not fit).
template <int DT, int NV, class Spec, int OP, bool RAGGED = false, bool CHUNKED = true>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(Spec::kStatic ? 4 : 1))) pool_kernel(const ChainArgs a, const PoolGeom g) {
    using S = Storage<DT>;
    constexpr int VEC = S::VEC;
    __shared__ float lds[512 * VEC];
    __shared__ float lds_ch[512];  // a value per channel of the slab
    const uint32_t t = threadIdx.x;
    const uint32_t pstep = fast_div(t, g.div_cv);
    const uint32_t unit = blockIdx.x / g.blocks_per_sample;  // (sample, slab)
    const uint32_t bx = blockIdx.x - unit * g.blocks_per_sample;
    const uint32_t sample = unit / g.slabs;
    const uint32_t slab_cv = (unit - sample * g.slabs) * g.cv;  // first channel vector of the slab
    const uint32_t cvl = t - pstep * g.cv;                      // channel vector inside the slab ...
    const uint32_t cvi = slab_cv + cvl;                         // ... and inside the position
    const bool active = pstep < g.pos_per_step && cvi * (uint32_t)VEC < g.channels;
    const uint32_t slab_channels = min(g.cv * (uint32_t)VEC, g.channels - slab_cv * (uint32_t)VEC);
    const uint32_t p_begin = bx * g.pos_per_block;
    const uint32_t p_count = min(g.hw - p_begin, g.pos_per_block);  // (p_begin + pos_per_block may be past 2^32)
    const uint32_t pro_full = Spec::kStatic ? list_operand_mask<typename Spec::Pro>(K_FULL) : ~g.epi_full_mask;
    const uint32_t pro_vec = Spec::kStatic ? list_operand_mask<typename Spec::Pro>(K_VEC) : ~g.epi_vec_mask;
    const uint32_t epi_full = Spec::kStatic ? list_operand_mask<typename Spec::Epi>(K_FULL) : g.epi_full_mask;
    const uint32_t epi_vec = Spec::kStatic ? list_operand_mask<typename Spec::Epi>(K_VEC) : g.epi_vec_mask;

    LaneState<DT, 1, Spec> s;
    s.col[0] = cvi * VEC;
    const uint32_t cnt = RAGGED ? elems_below<VEC>(cvi * (uint32_t)VEC, g.channels) : (uint32_t)VEC;
    // (what follows a position's partial vector is the next position, unless it is the tensor's last)
    const uint64_t total_elems = (uint64_t)g.samples * g.hw * g.channels;
    auto load_ragged = [&](const void* base, uint64_t elem) { return load_elems<DT>(base, elem, cnt, 0u, elem + (uint64_t)VEC <= total_elems); };

    // ---- the slice in chunks of NV position steps.  No branch around a whole vector's load (an element-aligned one has
    // the branch of load_elems, and waits): a lane without a position at step i reads the
    // slice's first vector and leaves it out of the reduction.  (Behind guards the compiler loses count of what is in flight
    // and waits for all of the chunk's loads before the first vector is worked on.)  A vector's address is a scalar, the
    // step's, plus one offset of the lane's.
    const uint64_t pos0 = (uint64_t)sample * g.hw + p_begin;
    const uint32_t step_elems = g.pos_per_step * g.channels;
    const uint32_t lane_elems = pstep * g.channels + cvi * (uint32_t)VEC;
    const uint32_t p_left = active ? (p_count > pstep ? p_count - pstep : 0u) : 0u;  // step i is the lane's while i * pos_per_step < p_left
    auto valid_of = [&](uint32_t step) { return step * g.pos_per_step < p_left; };
    auto load_step = [&](uint32_t step) {
        // (a step wholly past the slice's end: step 0)
        const uint64_t at = pos0 * g.channels + (step * g.pos_per_step < p_count ? (uint64_t)step * step_elems : 0u);
        if (RAGGED) return load_ragged(a.full[0], at + (valid_of(step) ? lane_elems : 0u));
        return load_stream(static_cast<const char*>(a.full[0]) + at * S::ESIZE, (valid_of(step) ? lane_elems : 0u) * (uint32_t)S::ESIZE);
    };

    // ---- mean and scale of the lane's channels.  What they are made of is asked for in front of the slice: loads come back in
    // order, and the merging is done while the slice is on its way.
    constexpr bool kNorm = Spec::kStatic && list_has<typename Spec::Pro>(U_GNORM);
    PoolNorm<VEC> norm;
    u32x4 raw[NV];
    if constexpr (!kNorm) {
#pragma unroll
        for (int i = 0; i < NV; ++i) raw[i] = load_step((uint32_t)i);
    }
    if constexpr (kNorm) {
        constexpr int gs = Spec::kGamma, bs = Spec::kBeta;
        float gm[VEC], bt[VEC];
        const u32x4 graw = RAGGED ? load_vec_operand_elems<DT>(a.vec[gs], 0u, cvi * VEC, g.channels, active ? cnt : 0u)
                                  : load_vec_operand<DT>(a.vec[gs], 0u, active ? cvi * VEC : 0u, g.channels);
        const u32x4 braw = RAGGED ? load_vec_operand_elems<DT>(a.vec[bs], 0u, cvi * VEC, g.channels, active ? cnt : 0u)
                                  : load_vec_operand<DT>(a.vec[bs], 0u, active ? cvi * VEC : 0u, g.channels);
        // the statistics of the groups the slab touches: 2^norm_log2 adjacent lanes share a group, each merges a strided subset
        // of the sample's partials, four of them in flight at a time, then the lanes are merged by a shuffle tree
        const uint32_t grp0 = fast_div(slab_cv * (uint32_t)VEC, g.div_norm_cpg);
        const uint32_t grps = fast_div(slab_cv * (uint32_t)VEC + slab_channels - 1u, g.div_norm_cpg) + 1u - grp0;
        const uint32_t lanes = 1u << g.norm_log2, grp = t >> g.norm_log2;
        const f32x4* part = reinterpret_cast<const f32x4*>(g.norm_partial) + (uint64_t)sample * g.norm_slices * g.norm_groups + grp0 + min(grp, grps - 1u);
        Stat st = {0.0f, 0.0f, 0.0f};
        f32x4 q[4];
        auto fetch = [&](uint32_t b) {
#pragma unroll
            for (int u = 0; u < 4; ++u) q[u] = part[(uint64_t)min(b + (uint32_t)u * lanes, g.norm_slices - 1u) * g.norm_groups];
        };
        auto merge = [&](uint32_t b) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float n = b + (uint32_t)u * lanes < g.norm_slices ? q[u][0] : 0.0f;
                st = stat_merge(st, Stat{n, n > 0.0f ? q[u][1] : 0.0f, n > 0.0f ? q[u][2] : 0.0f});
            }
        };
        uint32_t b = t & (lanes - 1u);
        fetch(b);
#pragma unroll
        for (int i = 0; i < NV; ++i) raw[i] = load_step((uint32_t)i);
        merge(b);
        for (b += 4u * lanes; b < g.norm_slices; b += 4u * lanes) {
            fetch(b);
            merge(b);
        }
        for (uint32_t m = 1; m < lanes; m <<= 1) st = stat_merge(st, stat_shfl_xor(st, (int)m));
        if (grp < grps && (t & (lanes - 1u)) == 0u) {
            lds[grp * 2u] = st.mean;
            lds[grp * 2u + 1u] = 1.0f / sqrtf((st.n > 0.0f ? st.m2 / st.n : 0.0f) + a.eps);
        }
        S::unpack(graw, gm);
        S::unpack(braw, bt);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const uint32_t my = fast_div(min(cvi * (uint32_t)VEC + (uint32_t)e, slab_cv * (uint32_t)VEC + slab_channels - 1u), g.div_norm_cpg) - grp0;
            norm.mean[e] = lds[my * 2u];
            norm.scale[e] = lds[my * 2u + 1u] * gm[e];
            norm.shift[e] = bt[e];
        }
        __syncthreads();  // (the area is used again below)
    }

    float acc[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = pool_identity<OP>();
    // (the state is passed, not captured: the interpreter's accesses by operand number, made through a closure, put it into scratch
    // memory)
    auto work_on = [&](LaneState<DT, 1, Spec>& s, const u32x4& x, uint32_t step) {
        const uint32_t pos = (uint32_t)pos0 + pstep + step * g.pos_per_step;
        s.row[0] = pos;
        s.fraw[0][0] = x;
#pragma unroll
        for (int f = 1; f < Spec::NF; ++f)
            if (f < Spec::n_full(a) && ((pro_full >> f) & 1u)) {
                s.fraw[f][0] = u32x4{0u, 0u, 0u, 0u};
                if (valid_of(step)) {
                        const uint64_t elem = (uint64_t)pos * g.channels + cvi * VEC;
                        s.fraw[f][0] = RAGGED ? load_ragged(a.full[f], elem) : load_stream(a.full[f], elem * S::ESIZE);
                    }
            }
#pragma unroll
        for (int v = 0; v < Spec::NV; ++v)
            if (v < Spec::n_vec(a) && ((pro_vec >> v) & 1u)) {
                s.vraw[v][0] = u32x4{0u, 0u, 0u, 0u};
                if (valid_of(step))
                    s.vraw[v][0] = RAGGED ? load_vec_operand_elems<DT, Spec::kVecMode>(a.vec[v], pos, s.col[0], g.channels, cnt)
                                          : load_vec_operand<DT, Spec::kVecMode>(a.vec[v], pos, s.col[0], g.channels);
            }
        if constexpr (kNorm) run_program<DT, 1, Spec>(ProgView<typename Spec::Pro>{a.pro}, s, norm);
        else run_program<DT, 1, Spec>(ProgView<typename Spec::Pro>{a.pro}, s, NoStore{});
        if (valid_of(step)) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[e] = pool_combine<OP>(acc[e], s.acc[e]);
        }
    };
    uint32_t step = 0;
    if constexpr (Spec::kStatic) {
        // Every chunk but the last: a vector's place is refilled from the next chunk as soon as it has been worked on, so memory and
        // arithmetic overlap inside a wave.  (The last chunk has a copy of the code without the refill: the barrier behind it waits
        // for whatever is in flight, needed or not.)
        if constexpr (CHUNKED) {
            for (; (step + (uint32_t)NV) * g.pos_per_step < p_count; step += (uint32_t)NV) {
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    work_on(s, raw[i], step + (uint32_t)i);
                    raw[i] = load_step(step + (uint32_t)(NV + i));
                }
            }
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) work_on(s, raw[i], step + (uint32_t)i);
    } else {
        // The interpreter: one copy of the steps, a chunk's loads together in front of them.  (Vectors that change places in a
        // rolled loop wait for the newest load at every step.)
        for (;;) {
#pragma unroll
            for (int i = 0; i < NV; ++i) work_on(s, raw[i], step + (uint32_t)i);
            step += (uint32_t)NV;
            if (step * g.pos_per_step >= p_count) break;
#pragma unroll
            for (int i = 0; i < NV; ++i) raw[i] = load_step(step + (uint32_t)i);
        }
    }

    // ---- the position steps of the workgroup, through LDS: a value per channel of the slab
#pragma unroll
    for (int e = 0; e < VEC; ++e) lds[t * VEC + e] = acc[e];
    __syncthreads();
    const uint32_t row_words = g.cv * (uint32_t)VEC;
    float mine = pool_reduce_rows<OP>(lds, lds_ch, g.pos_per_step, row_words, g.log2_lanes);  // (channel t of the slab)
    // A slab split over several workgroups: every slice but the last publishes its per-channel partial result as
    // self-describing words (kPoolEmpty = not written in this launch; consecutive lanes, consecutive words); the slab's
    // LAST slice (dispatched after the others) reads them all, re-reading the ones still empty, puts them back to empty for
    // the next launch and merges.  The critical path is one coherent store followed by one coherent load: no flag, no wait
    // for the stores' acknowledgement in between.
    if (bx + 1u != g.blocks_per_sample) {
        uint32_t* part = g.ws_partial + (uint64_t)blockIdx.x * row_words;
        if (t < slab_channels) __hip_atomic_store(part + t, pool_word(mine), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    // The merger (a slab that is one slice merges nothing): merge_rows row groups of threads, each a channel per lane
    // (consecutive lanes, consecutive words); row group r takes the slices r, r + merge_rows, ..., eight of them in flight
    // at a time.  Every wait is bounded: after spin_limit re-reads the error word is set and the missing slice is left out.
    const uint32_t others = g.blocks_per_sample - 1u;
    if (others != 0u) {
        const uint32_t r = t / row_words, idx = t - r * row_words;
        uint32_t* base = g.ws_partial + (uint64_t)unit * g.blocks_per_sample * row_words;
        uint32_t spins = 0;
        float merged = pool_identity<OP>();
        if (r < g.merge_rows && idx < slab_channels) {
            if (r == 0u) merged = mine;  // the merger's own slice
            for (uint32_t b0 = r; b0 < others; b0 += 8u * g.merge_rows) {
                uint32_t w[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const uint32_t b = b0 + (uint32_t)u * g.merge_rows;
                    w[u] = b < others ? __hip_atomic_load(base + (uint64_t)b * row_words + idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                      : pool_word(pool_identity<OP>());
                }
                // words still empty are re-read together (one trip to memory per round, not one per word)
                for (;;) {
                    bool waiting = false;
#pragma unroll
                    for (int u = 0; u < 8; ++u) waiting = waiting || w[u] == kPoolEmpty;
                    if (!waiting) break;
                    if (++spins > g.spin_limit) {
                        __hip_atomic_store(g.ws_error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        break;
                    }
                    __builtin_amdgcn_s_sleep(8);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const uint32_t b = b0 + (uint32_t)u * g.merge_rows;
                        if (w[u] == kPoolEmpty) w[u] = __hip_atomic_load(base + (uint64_t)b * row_words + idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const uint32_t b = b0 + (uint32_t)u * g.merge_rows;
                    if (b >= others || w[u] == kPoolEmpty) continue;
                    __hip_atomic_store(base + (uint64_t)b * row_words + idx, kPoolEmpty, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    merged = pool_combine<OP>(merged, __builtin_bit_cast(float, w[u]));
                }
            }
        }
        __syncthreads();  // (the positions' rows have been read)
        if (r < g.merge_rows) lds[t] = merged;
        __syncthreads();
        mine = pool_reduce_rows<OP>(lds, lds_ch, g.merge_rows, row_words, g.log2_lanes);
    }
    if (g.log2_lanes == 0u) {
        if (t < row_words) lds_ch[t] = mine;
        __syncthreads();
    }
    // lane t: channel vector t of the slab's result
    const bool owner = t < g.cv && (slab_cv + t) * (uint32_t)VEC < g.channels;
    if (!owner) return;
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = lds_ch[t * VEC + e];

    // ---- epilogue on the pooled values of (sample, channel vector slab_cv + t), addressed in the result's layout [n, c]
    if (OP == POOL_MEAN) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] *= g.inv_hw;
    }
    s.row[0] = sample;
    // (the slab's channel vector t is the lane's own: pstep is 0 there)
    const uint64_t out_elem = (uint64_t)sample * g.channels + cvi * VEC;
    const uint64_t out_off = out_elem * S::ESIZE;
#pragma unroll
    for (int f = 0; f < Spec::NF; ++f)
        if (f < Spec::n_full(a) && ((epi_full >> f) & 1u)) s.fraw[f][0] = RAGGED ? load_elems<DT>(a.full[f], out_elem, cnt, 0u) : load_cached(a.full[f], out_off);
#pragma unroll
    for (int v = 0; v < Spec::NV; ++v)
        if (v < Spec::n_vec(a) && ((epi_vec >> v) & 1u))
            s.vraw[v][0] = RAGGED ? load_vec_operand_elems<DT, Spec::kVecMode>(a.vec[v], sample, s.col[0], g.channels, cnt)
                                  : load_vec_operand<DT, Spec::kVecMode>(a.vec[v], sample, s.col[0], g.channels);
#pragma unroll
    for (int e = 0; e < VEC; ++e) s.acc[e] = acc[e];
    run_program<DT, 1, Spec>(ProgView<typename Spec::Epi>{a.epi}, s, NoStore{});
    if (RAGGED) store_elems<DT>(a.out[0], out_elem, cnt, S::pack(s.acc));
    else store_stream(a.out[0], out_off, S::pack(s.acc));
}

// GroupNorm -> steps -> pooling in one launch: a workgroup owns (sample, slab of whole groups) and all positions, held packed in
// its registers (NV vectors a lane).  The statistics, which are the groups' alone, and the pooled values then never leave
// the workgroup: x is read once, nothing is exchanged between workgroups and no second launch waits for the first.
//
// A slab starts and ends where its groups do, inside a 16-byte vector as it may be: lanes hold the whole vectors that the slab
// touches, and elements of a neighbour's groups are left out of the statistics and of the result.  Slabs are rarely whole
// memory lines either; neighbouring slabs run on one die, whose L2 serves the lines they share.
//
// Statistics: per element slot the mean over the lane's positions, then the squared deviations from it, merged as (count, mean,
// M2) triples, one per group the vector touches.
//
// Bound: the arithmetic behind the normalisation, with few waves to cover its waits.  [32, 64, 64, 320] fp16, GroupNorm(32) + SiLU +
// mean, 84 MB: 48.9 us in two launches, 44.6 in one, 41.5 with a channel's rows merged by lanes (pool_reduce_rows).
template <int DT, int NV, int CVS, class Spec, int OP>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(NV > 16 ? 2 : 4))) norm_pool_slab_kernel(const ChainArgs a, const SlabGeom g) {
    using S = Storage<DT>;
    constexpr int VEC = S::VEC;
    constexpr uint32_t PPS = 512u / (uint32_t)CVS;  // positions per step
    extern __shared__ float lds[];                  // [512][parts] (count, mean, M2), then [512][VEC] pooled values
    __shared__ float lds_stat[2 * 512];
    using P = typename Spec::Pro;
    static_assert(Spec::kStatic && P::n >= 2 && P::at(0).code == U_MOV && P::at(0).kind == K_FULL && P::at(1).code == U_GNORM, "the load, then the normalisation");
    const uint32_t slab = (blockIdx.x & 7u) * g.slabs_per_die + (blockIdx.x >> 3);
    if (slab >= g.slabs) return;  // (the grid is rounded up to a multiple of eight)
    const uint32_t sample = slab / g.slabs_per_sample;
    const uint32_t grp0 = (slab - sample * g.slabs_per_sample) * g.slab_groups;
    const uint32_t ch0 = grp0 * g.cpg, ch1 = ch0 + g.slab_groups * g.cpg;
    const uint32_t v0 = ch0 / (uint32_t)VEC;
    const uint32_t t = threadIdx.x;
    const uint32_t pstep = t / (uint32_t)CVS, cvl = t - pstep * (uint32_t)CVS;
    const uint32_t ch = (v0 + cvl) * (uint32_t)VEC;  // the lane's first channel
    const bool active = pstep < PPS && ch < ch1;

    // ---- the slab into registers.  No branch around a load: a lane without a vector reads the step's first.
    const char* base = static_cast<const char*>(a.full[P::at(0).slot]) + (uint64_t)sample * g.hw * g.channels * S::ESIZE;
    const uint32_t step_bytes = PPS * g.channels * (uint32_t)S::ESIZE;
    const uint32_t first_bytes = v0 * 16u;
    const uint32_t lane_bytes = active ? pstep * g.channels * (uint32_t)S::ESIZE + (v0 + cvl) * 16u : first_bytes;
    const bool last_valid = active && (uint32_t)(NV - 1) * PPS + pstep < g.hw;  // (every step but the last is whole)
    u32x4 raw[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) raw[i] = *reinterpret_cast<const u32x4*>(base + (size_t)((uint32_t)i * step_bytes) + (i + 1 < NV || last_valid ? lane_bytes : first_bytes));
    constexpr int gs = Spec::kGamma, bs = Spec::kBeta;
    const u32x4 graw = load_vec_operand<DT>(a.vec[gs], 0u, active ? ch : v0 * (uint32_t)VEC, g.channels);
    const u32x4 braw = load_vec_operand<DT>(a.vec[bs], 0u, active ? ch : v0 * (uint32_t)VEC, g.channels);

    // ---- statistics
    {
        const float npos = active ? (float)(NV - 1) + (last_valid ? 1.0f : 0.0f) : 0.0f;
        const float inv = npos > 0.0f ? 1.0f / npos : 0.0f;
        float mean_e[VEC], m2_e[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) mean_e[e] = m2_e[e] = 0.0f;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            float x[VEC];
            S::unpack(raw[i], x);
            if (i + 1 < NV || last_valid) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) mean_e[e] += x[e];
            }
        }
        auto keep_packed = [&](int i) {  // (the widened values are not kept from pass to pass)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t w = raw[i][j];
                asm volatile("" : "+v"(w));
                raw[i][j] = w;
            }
        };
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            keep_packed(i);
            float x[VEC];
            S::unpack(raw[i], x);
            if (i + 1 < NV || last_valid) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const float d = __builtin_fmaf(-mean_e[e], inv, x[e]);  // (the sum still; straight from the packed value in fp16)
                    m2_e[e] = __builtin_fmaf(d, d, m2_e[e]);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) keep_packed(i);
        // (the mean with what the reciprocal was rounded by: a sum times the rounded one of seven is not the mean of equal values)
        const float inv_rest = __builtin_fmaf(-npos, inv, 1.0f) * inv;
#pragma unroll
        for (int e = 0; e < VEC; ++e) mean_e[e] = __builtin_fmaf(mean_e[e], inv, mean_e[e] * inv_rest);
        // one triple per group the vector touches, adjacent slots merged
        const uint32_t first = fast_div(min(ch, g.channels - 1u), g.div_cpg);
        Stat cur = {npos, mean_e[0], m2_e[0]};
        uint32_t part = 0;
#pragma unroll
        for (int e = 1; e <= VEC; ++e) {
            const uint32_t next = e < VEC ? fast_div(min(ch + (uint32_t)e, g.channels - 1u), g.div_cpg) - first : g.parts;
            const bool flush = next != part;
            if (flush) {
                float* q = lds + (t * g.parts + part) * 3u;
                q[0] = cur.n;
                q[1] = cur.mean;
                q[2] = cur.m2;
            }
            if (e < VEC) {
                const Stat slot = {npos, mean_e[e % VEC], m2_e[e % VEC]};
                cur = flush ? slot : stat_merge(cur, slot);
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
                st = stat_merge(st, Stat{w[0], w[1], w[2]});
                ps += d_ps;
                k += d_k;
                if (k >= ncv) k -= ncv, ++ps;
            }
        }
        for (uint32_t m = 1; m < lanes; m <<= 1) st = stat_merge(st, stat_shfl_xor(st, (int)m));
        if (in_range && j == 0u) {
            lds_stat[q * 2u] = st.mean;
            lds_stat[q * 2u + 1u] = 1.0f / sqrtf((st.n > 0.0f ? st.m2 / st.n : 0.0f) + a.eps);
        }
    }
    __syncthreads();

    // ---- normalise, the steps behind, pool
    PoolNorm<VEC> norm;
    {
        float gm[VEC], bt[VEC];
        S::unpack(graw, gm);
        S::unpack(braw, bt);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            // (a neighbour's elements: the nearest group of the slab)
            const uint32_t q = fast_div(min(max(ch + (uint32_t)e, ch0), ch1 - 1u), g.div_cpg) - grp0;
            norm.mean[e] = lds_stat[q * 2u];
            norm.scale[e] = lds_stat[q * 2u + 1u] * gm[e];
            norm.shift[e] = bt[e];
        }
    }
    LaneState<DT, 1, Spec> s;
    s.col[0] = ch;
    s.row[0] = 0u;
    float acc[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = pool_identity<OP>();
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        s.fraw[P::at(0).slot][0] = raw[i];
        run_program<DT, 1, Spec>(ProgView<P>{a.pro}, s, norm);
        if (i + 1 < NV || last_valid) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[e] = pool_combine<OP>(acc[e], s.acc[e]);
        }
        // (the sums stay where they are written: sunk behind the last step by the compiler, they keep every step's values alive)
#pragma unroll
        for (int e = 0; e < VEC; ++e) asm volatile("" : "+v"(acc[e]));
    }

    // ---- the position steps, through LDS (the statistics' area has been read)
    constexpr uint32_t row_words = (uint32_t)(CVS * VEC);
    constexpr uint32_t log2_lanes = floor_log2_64(512u / row_words);
#pragma unroll
    for (int e = 0; e < VEC; ++e) lds[t * VEC + e] = acc[e];
    __syncthreads();
    const float mine = pool_reduce_rows<OP>(lds, lds_stat, PPS, row_words, log2_lanes);
    if (log2_lanes == 0u) {
        if (t < row_words) lds_stat[t] = mine;
        __syncthreads();
    }
    if (t >= (uint32_t)CVS || !active) return;
#pragma unroll
    for (int e = 0; e < VEC; ++e) s.acc[e] = OP == POOL_MEAN ? lds_stat[t * VEC + e] * g.inv_hw : lds_stat[t * VEC + e];

    // ---- epilogue, addressed in the result's layout [n, c]
    constexpr uint32_t epi_full = list_operand_mask<typename Spec::Epi>(K_FULL), epi_vec = list_operand_mask<typename Spec::Epi>(K_VEC);
    s.row[0] = sample;
    const uint64_t out_elem = (uint64_t)sample * g.channels + ch;
#pragma unroll
    for (int f = 0; f < Spec::NF; ++f)
        if ((epi_full >> f) & 1u) s.fraw[f][0] = load_cached(a.full[f], out_elem * S::ESIZE);
#pragma unroll
    for (int v = 0; v < Spec::NV; ++v)
        if ((epi_vec >> v) & 1u) s.vraw[v][0] = load_vec_operand<DT, Spec::kVecMode>(a.vec[v], sample, ch, g.channels);
    run_program<DT, 1, Spec>(ProgView<typename Spec::Epi>{a.epi}, s, NoStore{});
    const u32x4 packed = S::pack(s.acc);
    if (ch >= ch0 && ch + (uint32_t)VEC <= ch1) {
        store_stream(a.out[0], out_elem * S::ESIZE, packed);
        return;
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        if (ch + (uint32_t)e < ch0 || ch + (uint32_t)e >= ch1) continue;
        if (DT == DT_F32) {
            static_cast<uint32_t*>(a.out[0])[out_elem + (uint64_t)e] = packed[e % 4];
        } else {
            const uint32_t w = packed[e / 2];
            static_cast<uint16_t*>(a.out[0])[out_elem + (uint64_t)e] = (uint16_t)((e & 1) ? w >> 16 : w & 0xffffu);
        }
    }
}

}  // namespace pf
