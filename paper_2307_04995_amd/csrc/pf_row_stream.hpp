// Row family, streaming variant: rows that do not fit the registers of one workgroup.
//
// A workgroup owns a row and walks it twice in chunks of blockDim * K vectors.  The first walk runs the
// prologue and accumulates the row statistics per lane in a form that can be merged (running maximum and
// rescaled sum for softmax, (count, mean, M2) for LayerNorm, a sum of squares for RMSNorm, a sum or a
// maximum for the keep-dim reductions); one block-scope exchange merges them.  The second walk re-reads the
// operands (the row was just touched, so this read is served by the caches for rows of up to a few MB),
// re-runs the prologue, normalises, runs the epilogue and stores.  HBM traffic stays at one read and one
// write per element as long as a row fits the last-level cache; what the register-resident kernels keep in
// registers this one recomputes.
//
// The synchronisation structure is the same as in the resident kernels (paper section 5.1: one
// reduce -> broadcast exchange at workgroup scope); only the slice held per lane differs.
#pragma once
#include "pf_row_kernels.hpp"

namespace pf {

constexpr int kStreamThreads = 512;
constexpr int kStreamWaves = kStreamThreads / 64;

// merge (count, mean, M2) triples over the workgroup; every thread gets the result
PF_DEVICE Stat block_merge_stat(Stat st, uint32_t wave, uint32_t lane, float* lds) {
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) st = stat_merge(st, stat_shfl_xor(st, m));
    if (lane == 0) {
        lds[wave * 3 + 0] = st.n;
        lds[wave * 3 + 1] = st.mean;
        lds[wave * 3 + 2] = st.m2;
    }
    __syncthreads();
    Stat r = {lds[0], lds[1], lds[2]};
    for (int w = 1; w < kStreamWaves; ++w) r = stat_merge(r, Stat{lds[w * 3], lds[w * 3 + 1], lds[w * 3 + 2]});
    return r;
}

template <int DT, bool RAGGED, class Spec>
__global__ void __launch_bounds__(kStreamThreads) row_stream_kernel(const ChainArgs a) {
    using S = Storage<DT>;
    constexpr int VEC = S::VEC;
    constexpr int K = 2;
    constexpr int E = K * VEC;
    constexpr bool PR = S::PRECISE;
    __shared__ float red[2][16];
    __shared__ float lds_stat[kStreamWaves * 3];

    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t row = blockIdx.x;
    const uint32_t n = a.n_inner;
    const uint64_t row_byte = (uint64_t)row * n * S::ESIZE;
    const uint32_t chunk = (uint32_t)kStreamThreads * E;
    const int core = Spec::core(a);

    // causal mask: columns beyond the diagonal never need loading (they are overwritten by the mask, or the
    // folded mask treats them as -inf)
    uint32_t i_row = 0, load_limit = n;
    if (a.mask_si != 0u) {
        i_row = row - fast_div(row, a.mask_div) * a.mask_si;
        const uint32_t keep = (i_row + VEC) / VEC * VEC;
        load_limit = n < keep ? n : keep;
    }
    const bool fill_inf = a.core_mask == 2u;
    const uint32_t fill = fill_inf ? (DT == DT_F32 ? 0xff800000u : (DT == DT_F16 ? 0xfc00fc00u : 0xff80ff80u)) : 0u;
    const float cs = a.core_scale;
    const float c2 = cs * kLog2e;

    LaneState<DT, K, Spec> s;
    auto load_chunk = [&](uint32_t c0) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            s.row[k] = row;
            s.col[k] = c0 + ((uint32_t)k * kStreamThreads + threadIdx.x) * VEC;
        }
        load_row_operands<DT, K, K, Spec, RAGGED>(a, s, 0, row_byte, row, load_limit, n, fill, n);
    };
    // the mask folded into a softmax core, applied by position
    auto folded_mask = [&]() {
        if (core == CORE_SOFTMAX && a.core_mask != 0u) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int32_t last = (int32_t)i_row - (int32_t)s.col[k];
#pragma unroll
                for (int e = 0; e < VEC; ++e) s.acc[k * VEC + e] = (e > last) ? -__builtin_inff() : s.acc[k * VEC + e];
            }
        }
    };
    auto valid_elem = [&](int k, int e) { return RAGGED ? s.col[k] + (uint32_t)e < n : s.col[k] < n; };

    // ---- first walk: statistics
    float run_max = -__builtin_inff(), run_sum = 0.0f, nan_seen = 0.0f;
    LaneAcc la;
    for (uint32_t c0 = 0; c0 < n; c0 += chunk) {
        load_chunk(c0);
        run_program<DT, K, Spec>(ProgView<typename Spec::Pro>{a.pro}, s, NoStore{});
        folded_mask();
        if (core == CORE_SOFTMAX) {
            float cm = -__builtin_inff();
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    s.acc[k * VEC + e] = valid_elem(k, e) ? s.acc[k * VEC + e] : -__builtin_inff();
                    cm = fmaxf(cm, s.acc[k * VEC + e]);
                }
            const float m_new = fmaxf(run_max, cm);
            // exp(c * (x - m)) with m the running maximum; -inf terms contribute nothing.  A NaN element slips
            // past the maximum but poisons the sum, hence the whole row, as the definition does.
            if (m_new != run_max) run_sum *= PR ? expf((run_max - m_new) * cs) : __builtin_amdgcn_exp2f((run_max - m_new) * c2);
            run_max = m_new;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const float x = s.acc[e];
                const float t = PR ? expf((x - m_new) * cs) : __builtin_amdgcn_exp2f((x - m_new) * c2);
                run_sum += (x == -__builtin_inff()) ? 0.0f : t;
            }
        } else if (core == CORE_LAYERNORM) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                if (!RAGGED || s.col[k] + (uint32_t)VEC <= n) {
                    if (s.col[k] < n) la.template add_vector<VEC>(s.acc + k * VEC);
                } else {
#pragma unroll
                    for (int e = 0; e < VEC; ++e)
                        if (s.col[k] + (uint32_t)e < n) la.template add_vector<1>(s.acc + k * VEC + e);
                }
            }
        } else if (core == CORE_REDUCE_MAX) {
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const float x = s.acc[k * VEC + e];
                    if (valid_elem(k, e)) {
                        run_max = fmaxf(run_max, x);
                        nan_seen = (x != x) ? 1.0f : nan_seen;
                    }
                }
        } else {  // RMSNorm: sum of squares; REDUCE_SUM / REDUCE_MEAN: sum
            const bool sq = core == CORE_RMSNORM;
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const float x = s.acc[k * VEC + e];
                    run_sum += valid_elem(k, e) ? (sq ? x * x : x) : 0.0f;
                }
        }
    }

    // ---- block-scope exchange
    float row_max = 0.0f, row_inv = 0.0f, mean = 0.0f, rstd = 0.0f, value = 0.0f;
    if (core == CORE_SOFTMAX) {
        row_max = row_allreduce<OpMax>(run_max, kStreamWaves, wave, 0u, lane, red[0]);
        if (run_max != row_max) run_sum *= PR ? expf((run_max - row_max) * cs) : __builtin_amdgcn_exp2f((run_max - row_max) * c2);
        const float sum = row_allreduce<OpSum>(run_sum, kStreamWaves, wave, 0u, lane, red[1]);
        row_inv = pf_rcp<PR>(sum);
    } else if (core == CORE_LAYERNORM) {
        const Stat st = block_merge_stat(la.finish(), wave, lane, lds_stat);
        mean = st.mean;
        rstd = pf_rsqrt<PR>(st.m2 / (float)n + a.eps);
    } else if (core == CORE_RMSNORM) {
        const float ss = row_allreduce<OpSum>(run_sum, kStreamWaves, wave, 0u, lane, red[0]);
        rstd = pf_rsqrt<PR>(ss / (float)n + a.eps);
    } else if (core == CORE_REDUCE_MAX) {
        const float m = row_allreduce<OpMax>(run_max, kStreamWaves, wave, 0u, lane, red[0]);
        const float ns = row_allreduce<OpMax>(nan_seen, kStreamWaves, wave, 0u, lane, red[1]);
        value = ns > 0.0f ? __builtin_nanf("") : m;
    } else {
        value = row_allreduce<OpSum>(run_sum, kStreamWaves, wave, 0u, lane, red[0]);
        if (core == CORE_REDUCE_MEAN) value = value / (float)n;
    }

    if (core == CORE_REDUCE_SUM || core == CORE_REDUCE_MAX || core == CORE_REDUCE_MEAN) {
        // one value per row: the epilogue (unary and constant steps only) runs on it, one lane stores it
        LaneState<DT, 1, Spec> t;
        t.row[0] = row;
        t.col[0] = 0;
#pragma unroll
        for (int e = 0; e < VEC; ++e) t.acc[e] = value;
        run_program<DT, 1, Spec>(ProgView<typename Spec::Epi>{a.epi}, t, NoStore{});
        if (threadIdx.x == 0) {
            if (DT == DT_F32) {
                static_cast<float*>(a.out[0])[row] = t.acc[0];
            } else {
                const u32x4 packed = S::pack(t.acc);
                static_cast<uint16_t*>(a.out[0])[row] = (uint16_t)(packed[0] & 0xffffu);
            }
        }
        return;
    }

    // ---- second walk: normalise and store
    const RowStore<RAGGED> store_fn{a.out[0], a.out[1], row_byte, n};
    char* out_row = static_cast<char*>(a.out[0]) + row_byte;
    for (uint32_t c0 = 0; c0 < n; c0 += chunk) {
        load_chunk(c0);
        run_program<DT, K, Spec>(ProgView<typename Spec::Pro>{a.pro}, s, store_fn);
        folded_mask();
        if (core == CORE_SOFTMAX) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const float t = PR ? expf((s.acc[e] - row_max) * cs) : __builtin_amdgcn_exp2f((s.acc[e] - row_max) * c2);
                s.acc[e] = t * row_inv;
            }
        } else {
            float gm[E], bt[E];
#pragma unroll
            for (int e = 0; e < E; ++e) {
                gm[e] = 1.0f;
                bt[e] = 0.0f;
            }
            if (Spec::gamma(a) >= 0) fetch_vec<DT, K, Spec>(s, Spec::gamma(a), gm);
            if (core == CORE_LAYERNORM && Spec::beta(a) >= 0) fetch_vec<DT, K, Spec>(s, Spec::beta(a), bt);
#pragma unroll
            for (int e = 0; e < E; ++e) s.acc[e] = (s.acc[e] - mean) * rstd * gm[e] + bt[e];
        }
        run_program<DT, K, Spec>(ProgView<typename Spec::Epi>{a.epi}, s, store_fn);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (RAGGED) store_elems<DT>(out_row, s.col[k], elems_below<VEC>(s.col[k], n), S::pack(s.acc + k * VEC));
            else if (s.col[k] < n) store_stream(out_row, s.col[k] * (uint32_t)S::ESIZE, S::pack(s.acc + k * VEC));
        }
    }
}

// Row family, held variant: rows longer than the row kernel keeps (it holds them widened to fp32) but short enough for
// the registers of one workgroup in their storage form -- a 100 KB row of a 50 257-entry vocabulary is 28 registers a
// lane.  The row is read once: K vectors a lane, all requested before the first is used; every pass over it (maximum,
// sum of exponentials, result) widens the packed vectors again, which costs a conversion where the streaming variant
// costs a second trip to memory.
//
// The vectors lie on a grid that starts at the last 128-byte line boundary at or before the row, not at the row's first
// element: every access is aligned, a wave's 1 KB is eight whole lines, and what the first and last vectors hold of
// the neighbouring rows (or before and behind the row altogether) is replaced by a neutral value where it is used and
// never stored.
//
// Bound: HBM, with the vector units half busy (two exponentials per element, the second instead of keeping 104 fp32
// values a lane).  Softmax of [1024, 50257] fp16, 206 MB: 70.9 us streamed, 46 us held with vectors that start at the row's
// first element, 40.6 us on the grid of lines (5.1 TB/s); [300, 50257] fp32 57.1 -> 38.7 us; one row of 128 256 bf16
// 28.3 -> 17.2 us.
template <int DT>
struct HeldGrid {
    static constexpr uint32_t VEC = Storage<DT>::VEC;
    uint32_t first;  // elements between the grid's origin and the row's first (less than a line)
    uint32_t n;
    PF_DEVICE uint32_t below(uint32_t g) const { return elems_below<(int)VEC>(g, first); }           // elements of the vector at g in front of the row
    PF_DEVICE uint32_t limit(uint32_t g) const { return elems_below<(int)VEC>(g, first + n); }       // ... up to the row's end
    PF_DEVICE bool whole(uint32_t g) const { return g >= first && g + VEC <= first + n; }
};

// Elements [lo, hi) of a vector, one by one (the two vectors at a row's ends).
template <int DT>
PF_DEVICE void store_between(void* base, int64_t elem, uint32_t lo, uint32_t hi, u32x4 v) {
#pragma unroll
    for (uint32_t e = 0; e < (uint32_t)Storage<DT>::VEC; ++e) {
        if (e < lo || e >= hi) continue;
        if (DT == DT_F32) {
            static_cast<uint32_t*>(base)[elem + (int64_t)e] = v[e % 4u];
        } else {
            const uint32_t w = v[e / 2u];
            static_cast<uint16_t*>(base)[elem + (int64_t)e] = (uint16_t)((e & 1u) ? w >> 16 : w & 0xffffu);
        }
    }
}

// Stores of a held row: the accumulator's vector at grid position g.
template <int DT>
struct HeldStore {
    HeldGrid<DT> grid;
    void* out0;
    void* out1;
    int64_t origin;  // the grid's origin in elements from the tensor's start
    const uint32_t* g;
    PF_DEVICE void put_whole(void* dst, u32x4 v) const {
        char* p = static_cast<char*>(dst) + origin * Storage<DT>::ESIZE + *g * (uint32_t)Storage<DT>::ESIZE;
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p));
    }
    PF_DEVICE void put(void* dst, u32x4 v) const {
        const uint32_t at = *g;
        if (grid.whole(at)) put_whole(dst, v);
        else store_between<DT>(dst, origin + (int64_t)at, grid.below(at), grid.limit(at), v);
    }
    template <int D, int K, class Spec>
    PF_DEVICE void operator()(int slot, const LaneState<D, K, Spec>& st) const {
        put(slot == 0 ? out0 : out1, Storage<D>::pack(st.acc));
    }
};

template <int DT, int K, int T, bool RAGGED, class Spec>
__global__ void __launch_bounds__(T) row_held_kernel(const ChainArgs a) {
    using S = Storage<DT>;
    constexpr int VEC = S::VEC;
    constexpr bool PR = S::PRECISE;
    constexpr uint32_t W = (uint32_t)T / 64u;
    static_assert(Spec::kStatic && Spec::NF == 1, "one full operand, specialised chains only");
    __shared__ float red[3][16];
    warm_chain_arguments<Spec>();

    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t row = blockIdx.x;
    const uint32_t n = a.n_inner;
    const int core = Spec::core(a);
    const uint64_t row_addr = (uint64_t)a.full[0] + (uint64_t)row * n * S::ESIZE;
    const char* origin = reinterpret_cast<const char*>(row_addr & ~(uint64_t)127u);
    const HeldGrid<DT> grid{(uint32_t)(row_addr & 127u) / (uint32_t)S::ESIZE, n};
    auto g_of = [&](int k) { return ((uint32_t)k * T + tid) * (uint32_t)VEC; };
    // Slots that may hold a partial or an absent vector, known when the kernel is compiled: the first, and (a row needs
    // between K T - T - 8 and K T vectors, its place on the grid included) the last two.
    auto edge = [](int k) { return k == 0 || k + 2 >= K; };

    // Lanes in front of the row or behind it read its first or last vector.  The last vector of the tensor's last row
    // may reach past the tensor: it is gathered element by element.
    const uint32_t lo = grid.first / (uint32_t)VEC * (uint32_t)VEC;
    const bool short_end = RAGGED && row + 1u == a.rows && (grid.first + n) % (uint32_t)VEC != 0u;
    const uint32_t hi = short_end ? (grid.first + n) / (uint32_t)VEC * (uint32_t)VEC - (uint32_t)VEC
                                  : (grid.first + n - 1u) / (uint32_t)VEC * (uint32_t)VEC;
    u32x4 raw[K];
#pragma unroll
    for (int k = 0; k < K; ++k) raw[k] = load_stream(origin, min(max(g_of(k), lo), hi) * (uint32_t)S::ESIZE);
    if (short_end) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (g_of(k) == hi + (uint32_t)VEC) raw[k] = load_elems<DT>(origin, g_of(k), (grid.first + n) % (uint32_t)VEC, 0u);
    }

    // With nothing but the load in front of the reduction, elements that are not the row's become neutral in their packed
    // form, once; the passes then need no masks (LayerNorm's second does: its neutral value is the mean).
    constexpr bool kFill = Spec::Pro::n == 1;
    if (kFill) {
        const bool low = core == CORE_SOFTMAX || core == CORE_REDUCE_MAX;
        const uint32_t fill = !low ? 0u : DT == DT_F32 ? 0xff800000u : DT == DT_F16 ? 0xfc00fc00u : 0xff80ff80u;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (!edge(k)) continue;
            const uint32_t b = grid.below(g_of(k)), l = grid.limit(g_of(k));
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t w = raw[k][j];
                if (DT == DT_F32) {
                    raw[k][j] = (uint32_t)j >= b && (uint32_t)j < l ? w : fill;
                } else {
                    const uint32_t e0 = 2u * (uint32_t)j, e1 = e0 + 1u;
                    raw[k][j] = (e0 >= b && e0 < l ? w & 0xffffu : fill & 0xffffu) | (e1 >= b && e1 < l ? w & 0xffff0000u : fill & 0xffff0000u);
                }
            }
        }
    }

    LaneState<DT, 1, Spec> s;
    s.row[0] = row;
    uint32_t g_now = 0;
    constexpr uint32_t pro_vec = list_operand_mask<typename Spec::Pro>(K_VEC);
    auto load_vecs = [&](int k, bool all) {
        const uint32_t g = g_of(k);
#pragma unroll
        for (int v = 0; v < Spec::NV; ++v) {
            if (!all && !((pro_vec >> v) & 1u)) continue;
            if (!edge(k) || grid.whole(g)) {
                s.vraw[v][0] = RAGGED || grid.first != 0u ? load_vec_operand_elems<DT, Spec::kVecMode>(a.vec[v], row, g - grid.first, n, (uint32_t)VEC)
                                                          : load_vec_operand<DT, Spec::kVecMode>(a.vec[v], row, g, n);
                continue;
            }
            // the row's ends: element by element, columns outside the row read its first or last
            uint32_t bits[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                const uint32_t c = min(max(g + (uint32_t)e, grid.first) - grid.first, n - 1u);
                const u32x4 one = load_vec_operand_elems<DT, Spec::kVecMode>(a.vec[v], row, c, n, 1u);
                bits[e] = one[0];
            }
            if (DT == DT_F32) s.vraw[v][0] = u32x4{bits[0], bits[1], bits[2], bits[3]};
            else
                s.vraw[v][0] = u32x4{(bits[0] & 0xffffu) | (bits[1] << 16), (bits[2 % VEC] & 0xffffu) | (bits[3 % VEC] << 16),
                                     (bits[4 % VEC] & 0xffffu) | (bits[5 % VEC] << 16), (bits[6 % VEC] & 0xffffu) | (bits[7 % VEC] << 16)};
        }
    };
    // vector k through the prologue, into s.acc
    auto value_of = [&](int k, const auto& store_fn) {
        g_now = g_of(k);
        s.col[0] = g_now - grid.first;
        s.fraw[0][0] = raw[k];
        run_program<DT, 1, Spec>(ProgView<typename Spec::Pro>{a.pro}, s, store_fn);
    };
    // the same for a reduction: what is not the row's becomes `neutral`
    auto counted = [&](int k, float neutral, bool filled) {
        if (pro_vec) load_vecs(k, false);
        value_of(k, NoStore{});
        if (edge(k) && !filled) {
            const uint32_t b = grid.below(g_of(k)), l = grid.limit(g_of(k));
#pragma unroll
            for (int e = 0; e < VEC; ++e) s.acc[e] = (uint32_t)e >= b && (uint32_t)e < l ? s.acc[e] : neutral;
        }
    };
    // (the packed vectors are what stays between passes, not their widened values)
    auto keep = [&]() {
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                uint32_t w = raw[k][j];
                asm volatile("" : "+v"(w));
                raw[k][j] = w;
            }
    };
    auto sum_over_row = [&](float v, int area) { return row_allreduce<OpSum>(v, W, wave, 0u, lane, red[area]); };

    // (a vector's elements are added pairwise before they join the lane's running sum: the rounding of a row's sum, which every
    // element of a softmax shares, stays below that of the streaming walk)
    auto vector_sum = [&]() {
        float v = 0.0f;
#pragma unroll
        for (int e = 0; e < VEC; e += 4) v += (s.acc[e] + s.acc[e + 1]) + (s.acc[e + 2] + s.acc[e + 3]);
        return v;
    };

    float row_max = 0.0f, mc = 0.0f, row_inv = 0.0f, mean = 0.0f, rstd = 0.0f, value = 0.0f;
    const float cs = a.core_scale, c2 = cs * kLog2e;
    // The maximum is subtracted before the multiplication: in x * c2 - max * c2 the rounding of max * c2, a common factor of the
    // row that the division takes out, is an exponent of its own where the maximum is large (2^328 in a bf16 row masked
    // throughout with -1e10).  Where the planner knows that it is not (kSmallScores) one fused step does both: [1024, 50257]
    // fp16 39.1 us against 40.9.
    auto exp_below_max = [&](float x) {
        if (PR) return expf((x - row_max) * cs);
        return __builtin_amdgcn_exp2f(Spec::kSmallScores ? __builtin_fmaf(x, c2, mc) : (x - row_max) * c2);
    };
    if (core == CORE_SOFTMAX || core == CORE_REDUCE_MAX) {
        float m = -__builtin_inff(), nan_seen = 0.0f;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            counted(k, -__builtin_inff(), kFill);
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                m = fmaxf(m, s.acc[e]);
                if (core == CORE_REDUCE_MAX) nan_seen = (s.acc[e] != s.acc[e]) ? 1.0f : nan_seen;
            }
        }
        row_max = row_allreduce<OpMax>(m, W, wave, 0u, lane, red[0]);
        if (core == CORE_REDUCE_MAX) {
            nan_seen = row_allreduce<OpMax>(nan_seen, W, wave, 0u, lane, red[1]);
            value = nan_seen > 0.0f ? __builtin_nanf("") : row_max;
        } else {
            mc = -row_max * c2;
            keep();
            float sum = 0.0f;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                counted(k, -__builtin_inff(), kFill);
#pragma unroll
                for (int e = 0; e < VEC; ++e) s.acc[e] = exp_below_max(s.acc[e]);
                sum += vector_sum();
            }
            row_inv = pf_rcp<PR>(sum_over_row(sum, 1));
        }
    } else {
        const bool sq = core == CORE_RMSNORM;
        float sum = 0.0f;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            counted(k, 0.0f, kFill);
#pragma unroll
            for (int e = 0; e < VEC; ++e) s.acc[e] = sq ? s.acc[e] * s.acc[e] : s.acc[e];
            sum += vector_sum();
        }
        value = sum_over_row(sum, 0);
        if (core == CORE_REDUCE_MEAN) value = value / (float)n;
        if (core == CORE_RMSNORM) rstd = pf_rsqrt<PR>(value / (float)n + a.eps);
        if (core == CORE_LAYERNORM) {
            // the deviations from the first mean carry what its rounding left over: mean and M2 are corrected by their sum
            keep();
            const float first = value / (float)n;
            float d1 = 0.0f, d2 = 0.0f;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                counted(k, first, false);
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const float d = s.acc[e] - first;
                    d1 += d;
                    d2 = __builtin_fmaf(d, d, d2);
                }
            }
            d1 = sum_over_row(d1, 1) / (float)n;
            d2 = sum_over_row(d2, 2) / (float)n;
            mean = first + d1;
            rstd = pf_rsqrt<PR>(fmaxf(__builtin_fmaf(-d1, d1, d2), 0.0f) + a.eps);
        }
    }

    if (core == CORE_REDUCE_SUM || core == CORE_REDUCE_MAX || core == CORE_REDUCE_MEAN) {
        // one value per row: the epilogue (unary and constant steps only) runs on it, one lane stores it
        s.col[0] = 0;
#pragma unroll
        for (int e = 0; e < VEC; ++e) s.acc[e] = value;
        run_program<DT, 1, Spec>(ProgView<typename Spec::Epi>{a.epi}, s, NoStore{});
        if (tid == 0) {
            if (DT == DT_F32) static_cast<float*>(a.out[0])[row] = s.acc[0];
            else static_cast<uint16_t*>(a.out[0])[row] = (uint16_t)(S::pack(s.acc)[0] & 0xffffu);
        }
        return;
    }

    // ---- normalise and store
    keep();
    const HeldStore<DT> store_fn{grid, a.out[0], a.out[1], (int64_t)row * n - (int64_t)grid.first, &g_now};
#pragma unroll
    for (int k = 0; k < K; ++k) {
        load_vecs(k, true);
        value_of(k, store_fn);
        if (core == CORE_SOFTMAX) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) s.acc[e] = exp_below_max(s.acc[e]) * row_inv;
        } else {
            float gm[VEC], bt[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                gm[e] = 1.0f;
                bt[e] = 0.0f;
            }
            if (Spec::gamma(a) >= 0) fetch_vec<DT, 1, Spec>(s, Spec::gamma(a), gm);
            if (core == CORE_LAYERNORM && Spec::beta(a) >= 0) fetch_vec<DT, 1, Spec>(s, Spec::beta(a), bt);
#pragma unroll
            for (int e = 0; e < VEC; ++e) s.acc[e] = (s.acc[e] - mean) * rstd * gm[e] + bt[e];
        }
        run_program<DT, 1, Spec>(ProgView<typename Spec::Epi>{a.epi}, s, store_fn);
        const u32x4 v = S::pack(s.acc);
        if (!edge(k)) store_fn.put_whole(a.out[0], v);
        else store_fn.put(a.out[0], v);
    }
}

}  // namespace pf
