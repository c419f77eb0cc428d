// Kernel-family planning: catalogue match or plan-time specialisation, launch geometry, workspace.
#include "pf_host_internal.h"
#include "pf_specs.h"

namespace pfh {

struct SpecTable {
    std::vector<pf::SpecDesc> row, group, perm;
    SpecTable() {
#define PF_ADD_SPEC(vec, id_, nf_, nv_, nt_, core_, gamma_, beta_, pro_, epi_)              \
    {                                                                                       \
        pf::SpecDesc s;                                                                     \
        memset(&s, 0, sizeof(s));                                                           \
        s.id = id_; s.nf = nf_; s.nv = nv_; s.nt = nt_; s.core = pf::core_;                 \
        s.gamma = gamma_; s.beta = beta_;                                                   \
        const uint32_t p[] = {0u, pro_};                                                    \
        const uint32_t e[] = {0u, epi_};                                                    \
        s.n_pro = (int)(sizeof(p) / sizeof(p[0])) - 1;                                      \
        s.n_epi = (int)(sizeof(e) / sizeof(e[0])) - 1;                                      \
        for (int i = 0; i < s.n_pro; ++i) s.pro[i] = p[i + 1];                              \
        for (int i = 0; i < s.n_epi; ++i) s.epi[i] = e[i + 1];                              \
        vec.push_back(s);                                                                   \
    }
#define PF_ROW_X(id, nf, nv, nt, core, gamma, beta, pro, epi) PF_ADD_SPEC(row, id, nf, nv, nt, core, gamma, beta, PF_L(pro), PF_L(epi))
        PF_ROW_SPECS(PF_ROW_X)
#define PF_GROUP_X(id, nf, nv, nt, core, gamma, beta, pro, epi) PF_ADD_SPEC(group, id, nf, nv, nt, core, gamma, beta, PF_L(pro), PF_L(epi))
        PF_GROUP_SPECS(PF_GROUP_X)
#define PF_PERM_X(id, nf, nv, nt, core, gamma, beta, pro, epi) PF_ADD_SPEC(perm, id, nf, nv, nt, core, gamma, beta, PF_L(pro), PF_L(epi))
        PF_PERM_SPECS(PF_PERM_X)
    }
};

const SpecTable& spec_table() {
    static const SpecTable t;
    return t;
}

bool list_equal(const pf::Program& p, const uint32_t* list, int n) {
    if (p.n != n) return false;
    for (int i = 0; i < n; ++i) {
        const uint32_t packed = (uint32_t)p.u[i].code | ((uint32_t)p.u[i].kind << 8) | ((uint32_t)p.u[i].slot << 16);
        if (packed != list[i]) return false;
    }
    return true;
}

int match_spec(const std::vector<pf::SpecDesc>& table, const Lowered& L) {
    if (L.general_bcast || L.scalar_vec) return 0;  // catalogue kernels are built without the general broadcast addressing
                                                    // and without the one-element operand case
    if (L.n_out != 1) return 0;
    for (const pf::SpecDesc& s : table) {
        if (s.nf != L.n_full || s.nv != L.n_vec || s.nt != L.n_tmp || s.core != L.core) continue;
        if (s.gamma != L.core_vec[0] || s.beta != L.core_vec[1]) continue;
        if (!list_equal(L.pro, s.pro, s.n_pro) || !list_equal(L.epi, s.epi, s.n_epi)) continue;
        return s.id;
    }
    return 0;
}


constexpr int kStencilRowsHost = 6;   // output rows per strip of the stencil kernels (kStencilRows on the device side)
constexpr int kStencilRows5Host = 4;  // ... for 5 x 5 kernels (kStencilRows5)

int env_int(const char* name, int dflt) {
    const char* s = getenv(name);
    if (!s || !*s) return dflt;
    return atoi(s);
}

// the chain's structure as template arguments for the plan-time specialisation
pf::JitSpec make_jit_spec(const Lowered& L) {
    pf::JitSpec j;
    j.nf = L.n_full;
    j.nv = L.n_vec;
    j.nt = L.n_tmp;
    j.core = L.core;
    j.gamma = L.core_vec[0];
    j.beta = L.core_vec[1];
    j.flags = (L.general_bcast ? 1 : 0) | (L.scalar_vec ? 2 : 0);
    for (int i = 0; i < L.pro.n; ++i)
        j.pro.push_back((uint32_t)L.pro.u[i].code | ((uint32_t)L.pro.u[i].kind << 8) | ((uint32_t)L.pro.u[i].slot << 16));
    for (int i = 0; i < L.epi.n; ++i)
        j.epi.push_back((uint32_t)L.epi.u[i].code | ((uint32_t)L.epi.u[i].kind << 8) | ((uint32_t)L.epi.u[i].slot << 16));
    return j;
}

thread_local ScratchArena* tls_scratch = nullptr;

pf_status plan_workspace_alloc(pf_plan_s* p, uint64_t bytes, const char* what) {
    p->workspace_bytes = bytes;
    if (ScratchArena* a = tls_scratch) {
        const uint64_t at = (a->used + 255) / 256 * 256;
        if (at + bytes > a->cap)
            return fail(PF_ERR_NOMEM, "%s of %llu bytes does not fit the static scratch array (%llu bytes, %llu in use): use pf_chain_plan + pf_chain_run",
                        what, (unsigned long long)bytes, (unsigned long long)a->cap, (unsigned long long)at);
        p->workspace = a->base + at;
        p->workspace_borrowed = true;
        a->used = at + bytes;
        return PF_OK;
    }
    if (hipMalloc(&p->workspace, bytes) != hipSuccess) return fail(PF_ERR_NOMEM, "%s of %llu bytes failed", what, (unsigned long long)bytes);
    return PF_OK;
}

pf_status plan_workspace_fill(pf_plan_s* p, void* ptr, int byte, uint64_t bytes, bool must_hold) {
    if (bytes == 0) return PF_OK;
    if (planning_static()) {
        if (must_hold) p->fills.push_back(pf_plan_s::Fill{ptr, bytes, byte});
        return PF_OK;
    }
    if (hipMemset(ptr, byte, bytes) != hipSuccess) return fail(PF_ERR_HIP, "workspace clear failed");
    return PF_OK;
}

// A plan that should have got a kernel specialised for its chain runs on the run-time-interpreted kernels instead (the
// run-time compiler or the kernel headers are missing, or the compilation failed): several times slower, so the plan
// says so (pf_plan_info.interpreter_fallback) and keeps the reason for pf_last_error.
void note_interpreter_fallback(pf_plan_s* p, const std::string& why) {
    p->interpreter_fallback = true;
    p->fallback_reason = why;
    if (env_int("PF_LOG", 0)) fprintf(stderr, "[pf] plan-time specialisation unavailable, using the interpreter: %s\n", why.c_str());
}

// Plan-time specialisation needs the device (the compiled kernel is loaded onto it).
bool jit_possible(int device) {
    if (!pf::jit_enabled() || planning_static()) return false;
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess || device < 0 || device >= n) return false;
    return hipSetDevice(device) == hipSuccess;
}


pf_status fill_vec_args(pf_plan_s* p, const Checked& c) {
    const Lowered& L = p->low;
    const int es = dtype_size(L.main_dtype);
    p->args.vec_plain_all = 1;
    for (int v = 0; v < L.n_vec; ++v) {
        const int in = L.vec_input[v];
        const int64_t n = numel(c.shape[in]);
        const int64_t inner = (L.vec_is_epi[v] ? L.post_shape : L.pre_shape).back();
        if (n != inner || c.shape[in].empty() || c.shape[in].back() != inner || (n * es) % 16 != 0) p->args.vec_plain_all = 0;
        pf::VecArg& va = p->args.vec[v];
        va.ptr = nullptr;
        va.dtype = L.main_dtype;
        va.pad = 0;
        va.terms = nullptr;
        if (n > 0xffffffffLL) return fail(PF_ERR_UNSUPPORTED, "broadcast input %d too large", in);
        va.numel = (uint32_t)n;
        va.period_rows = 1;
        va.n_terms = 0;
        va.col_bcast = 0;
        if (n == 1) {
            p->low.scalar_vec = true;
            continue;
        }
        const Shape& os = c.shape[in];
        const Shape& ps = L.vec_partner[v];
        if (!ps.empty() && !is_trailing(os, ps)) {
            // ---- general broadcasting: extents of 1 anywhere.  One term per run of kept row dimensions.
            const Shape& region = L.vec_is_epi[v] ? L.post_shape : L.pre_shape;
            if (!broadcasts_onto(os, ps) || ps.back() != inner || numel(ps) != numel(region))
                return fail(PF_ERR_UNSUPPORTED, "broadcast input %d: its shape does not broadcast over the kernel's rows", in);
            const size_t rank = ps.size(), off = rank - os.size();
            auto op_extent = [&](size_t i) { return i < off ? (int64_t)1 : os[i - off]; };
            p->low.general_bcast = true;
            va.col_bcast = (op_extent(rank - 1) == 1 && inner != 1) ? 1u : 0u;
            if (!va.col_bcast && (inner * es) % 16 != 0) p->ragged = true;
            int64_t div = 1, stride = 1;  // rows of the value / operand rows inside the dimension being looked at
            bool in_run = false;
            for (size_t q = rank - 1; q-- > 0;) {
                const int64_t e = ps[q], oe = op_extent(q);
                if (e == 1) continue;
                if (oe == e) {
                    if (in_run) {
                        pf::BcastTerm& t = p->bcast_host[v][va.n_terms - 1];
                        t.mod = make_fastdiv((uint32_t)(t.mod.d * e));
                    } else {
                        if (va.n_terms == PF_DEV_MAX_BCAST_TERMS)
                            return fail(PF_ERR_UNSUPPORTED, "broadcast input %d: more than %d separate runs of kept dimensions", in, PF_DEV_MAX_BCAST_TERMS);
                        pf::BcastTerm& t = p->bcast_host[v][va.n_terms++];
                        memset(&t, 0, sizeof(t));
                        t.div = make_fastdiv((uint32_t)div);
                        t.mod = make_fastdiv((uint32_t)e);
                        t.stride = (uint32_t)stride;
                        in_run = true;
                    }
                    stride *= e;
                } else {
                    in_run = false;
                }
                div *= e;
                if (div > 0xffffffffLL) return fail(PF_ERR_UNSUPPORTED, "broadcast input %d: too many rows", in);
            }
            if (va.n_terms == 0) {
                // nothing kept among the row dimensions: one operand row for every row of the value
                pf::BcastTerm& t = p->bcast_host[v][va.n_terms++];
                memset(&t, 0, sizeof(t));
                t.div = make_fastdiv(1u);
                t.mod = make_fastdiv(1u);
                t.stride = 0;
            }
            continue;
        }
        if ((n * es) % 16 != 0) p->ragged = true;  // gathered element by element (row and element-wise families)
        if (n >= inner) {
            if (n % inner != 0) return fail(PF_ERR_UNSUPPORTED, "broadcast input %d does not tile the kernel's rows", in);
            va.period_rows = (uint32_t)(n / inner);
        } else if (inner % n != 0) {
            return fail(PF_ERR_UNSUPPORTED, "broadcast input %d does not tile the kernel's rows", in);
        }
    }
    if (L.general_bcast) {
        if (planning_static())
            return fail(PF_ERR_UNSUPPORTED, "broadcast inputs with extents of 1 inside their shape need a table in device memory: use pf_chain_plan + pf_chain_run");
        if (hipSetDevice(p->device) != hipSuccess || hipMalloc(&p->bcast_dev, sizeof(p->bcast_host)) != hipSuccess)
            return fail(PF_ERR_NOMEM, "device memory for broadcast terms");
        if (hipMemcpy(p->bcast_dev, p->bcast_host, sizeof(p->bcast_host), hipMemcpyHostToDevice) != hipSuccess)
            return fail(PF_ERR_HIP, "upload of broadcast terms failed");
        for (int v = 0; v < L.n_vec; ++v)
            if (p->args.vec[v].n_terms)
                p->args.vec[v].terms = static_cast<const pf::BcastTerm*>(p->bcast_dev) + (size_t)v * PF_DEV_MAX_BCAST_TERMS;
    }
    return PF_OK;
}

pf_status plan_row(pf_plan_s* p, int forced_variant) {
    const Lowered& L = p->low;
    const int es = dtype_size(L.main_dtype);
    const int vec = 16 / es;
    const int64_t n = L.pre_shape.back();
    const int64_t rows = numel(L.pre_shape) / n;
    if ((n * es) % 16 != 0) p->ragged = true;
    if (rows > 0xffffffffLL || n > 0x7fffffffLL) return fail(PF_ERR_UNSUPPORTED, "tensor too large for the row family");
    const int64_t vpr = (n + vec - 1) / vec;
    // candidates (waves per row, vectors per lane); prefer little idle lanes, a statically specialised
    // kernel, small workgroups, a single wave per row
    const bool reduce_only = L.core == pf::CORE_REDUCE_SUM || L.core == pf::CORE_REDUCE_MAX || L.core == pf::CORE_REDUCE_MEAN;
    const int matched = (!reduce_only && !p->ragged && env_int("PF_NO_STATIC", 0) == 0) ? match_spec(spec_table().row, L) : 0;
    // no catalogue entry: the same kernel templates are specialised for this chain's structure at plan time
    // (also catalogue entries in launch shapes that were not instantiated at build time)
    const bool jit_ok = jit_possible(p->device);
    auto have_static = [&](int k, int rpw, bool wave_rows, unsigned threads) {
        if (matched && pf::row_static_available(matched, k, rpw, wave_rows, threads)) return true;
        if (!jit_ok) return false;
        return (k == 1 || k == 2 || k == 4) && (rpw == 1 || rpw == 2 || rpw == 4) && k * rpw <= 4 && (wave_rows || rpw == 1) &&
               threads <= 1024;
    };
    int best_wpr = 0, best_k = 0;
    long best_score = -1;
    const int ks[3] = {1, 2, 4};
    for (int ki = 0; ki < 3 && forced_variant != PF_VARIANT_ROW_STREAM; ++ki) {
        const int k = ks[ki];
        const int64_t wpr = (vpr + 64 * k - 1) / (64 * k);
        if (wpr > 16) continue;
        if (forced_variant == PF_VARIANT_ROW_WAVE && wpr != 1) continue;
        if (forced_variant == PF_VARIANT_ROW_BLOCK && wpr == 1) continue;
        const double waste = 1.0 - (double)vpr / (double)(wpr * 64 * k);
        const unsigned threads = 64u * (unsigned)wpr * (wpr >= 4 ? 1u : (unsigned)(4 / wpr));
        long score = (waste > 0.26 ? 4000 : (waste > 0.13 ? 2000 : 0)) + (wpr > 4 ? 1000 : 0) + (wpr > 1 ? 100 : 0) + k;
        // With rows to spare, a wave that owns its row and idles through up to a quarter of its vector slots (they are
        // never loaded) still beats waves that share a row through LDS and barriers (768 fp32 columns, 65 536 rows:
        // 98.4 us against 106.6 us); with few rows the shared row wins, its lanes each doing a third of the arithmetic
        // (256 rows, replayed from a graph: 3.0 us against 3.6 us).
        if (wpr == 1 && rows >= 8192 && waste <= 0.26) score = k;
        if ((matched || jit_ok) && !have_static(k, 1, wpr == 1, threads)) score += 500;
        if (best_score < 0 || score < best_score) {
            best_score = score;
            best_wpr = (int)wpr;
            best_k = k;
        }
    }
    p->reduce_only = reduce_only;
    if (p->reduce_only) {
        // the epilogue runs on one value per row: no tensor operands there
        for (int i = 0; i < L.epi.n; ++i)
            if (L.epi.u[i].kind != pf::K_NONE && L.epi.u[i].kind != pf::K_IMM)
                return fail(PF_ERR_UNSUPPORTED, "after a keep-dim reduction only unary and constant steps are implemented");
        for (int i = 0; i < L.epi.n; ++i)
            if (L.epi.u[i].code == pf::U_MASK_CAUSAL || L.epi.u[i].code == pf::U_STORE)
                return fail(PF_ERR_UNSUPPORTED, "after a keep-dim reduction only unary and constant steps are implemented");
        if (L.n_out != 1) return fail(PF_ERR_UNSUPPORTED, "a keep-dim reduction has one output");
    }
    p->family = PF_FAMILY_ROW;
    p->args.n_inner = (uint32_t)n;
    p->args.rows = (uint64_t)rows;
    if (best_score < 0 && L.core == pf::CORE_ROWPROG)
        return fail(PF_ERR_UNSUPPORTED, "chains with in-line reductions need rows that fit one workgroup's registers (row length %lld)", (long long)n);
    // Rows held packed (row_held_kernel), threads per row.  256 lanes while a lane holds at most ten vectors, then 512, and
    // 1024 once 512 lanes would hold more than 25 (softmax of about 100 MB: [1249, 20001] fp16 19.1 us with 256 lanes, 21.1
    // with 512; [1024, 50257] 40.6 with 512, 41.4 with 1024; [300, 128256] 43.3 and 42.2).
    auto try_held = [&](int variant) {
        if (!jit_ok || forced_variant >= 0 || L.n_full != 1 || L.mask_si != 0 || L.core == pf::CORE_ROWPROG || env_int("PF_ROW_HELD", 1) == 0) return false;
        if (rows > 0x7fffffffLL || n * es > 0x7fffffffLL) return false;
        const int64_t held = (n * es + 127 + 15) / 16;  // vectors of a row wherever it starts within a 128-byte line
        const int t = held <= 256 * 10 ? 256 : held <= 512 * 25 ? 512 : 1024;
        const int k = (int)((held + t - 1) / t);
        if (t == 1024 && k > 20) return false;  // (128 registers a lane: what 20 vectors and the arithmetic need)
        // fp16 values as they are loaded reach 65504: with the scale in front of the softmax they stay below 2^20, where rounding
        // them to fp32 moves an exponent by less than 2^-4
        pf::JitSpec jspec = make_jit_spec(L);
        if (L.core == pf::CORE_SOFTMAX && L.main_dtype == PF_F16 && L.pro.n == 1 && L.core_scale * 1.4426951f * 65504.0f < 1048576.0f) jspec.flags |= 16;
        std::string err;
        hipFunction_t fn = pf::jit_row_held_kernel(p->device, L.main_dtype, k, t, p->ragged, jspec, &err);
        if (!fn || pf::jit_scratch_bytes(fn) != 0) return false;
        p->jit_fn = fn;
        p->spec_id = pf::kSpecJit;
        p->variant = variant;
        p->row_held = true;
        p->k = k;
        p->row.waves_per_row = (uint32_t)t / 64;
        p->row.rows_per_block = 1;
        p->row.rows_per_wave = 1;
        p->block = dim3((uint32_t)t);
        p->grid = dim3((uint32_t)rows);
        p->lds_bytes = 3 * 16 * 4;
        return true;
    };
    // Softmax over rows that are not whole vectors, of more than 512 vectors, with rows to fill the device: held packed and
    // aligned to memory lines they beat the row kernel's element-aligned accesses ([4999, 5001] fp16 28.8 -> 20.7 us,
    // [1525, 16383] 25.5 -> 19.5, [2499, 5001] fp32 24.5 -> 21.2); shorter ones do not ([8330, 3001] fp16 21.6 against 22.8),
    // nor do whole ones ([3125, 8000] 19.2 against 19.5).
    if (best_score >= 0 && p->ragged && L.core == pf::CORE_SOFTMAX && L.n_vec == 0 && L.n_out == 1 && vpr > 512 && rows >= 512 && try_held(PF_VARIANT_ROW_BLOCK))
        return PF_OK;
    if (best_score < 0) {
        // Rows longer than a workgroup keeps in registers widened to fp32 (or on request): held packed where that fits,
        // else the streaming kernel, a workgroup per row, two walks over the row.
        if (forced_variant >= 0 && forced_variant != PF_VARIANT_ROW_STREAM)
            return fail(PF_ERR_UNSUPPORTED, "variant %d is not possible for row length %lld", forced_variant, (long long)n);
        if (rows > 0x7fffffffLL || n * es > 0x7fffffffLL) return fail(PF_ERR_UNSUPPORTED, "tensor too large for the streaming row variant");
        p->variant = PF_VARIANT_ROW_STREAM;
        p->k = 2;
        p->spec_id = 0;
        p->row.waves_per_row = 8;
        p->row.rows_per_block = 1;
        p->row.rows_per_wave = 1;
        p->block = dim3(512);
        p->grid = dim3((uint32_t)rows);
        p->lds_bytes = (2 * 16 + 8 * 3) * 4;
        if (try_held(PF_VARIANT_ROW_STREAM)) return PF_OK;
        if (jit_ok) {
            std::string err;
            p->jit_fn = pf::jit_row_stream_kernel(p->device, L.main_dtype, p->ragged, make_jit_spec(L), &err);
            if (p->jit_fn) p->spec_id = pf::kSpecJit;
            else note_interpreter_fallback(p, err);
        }
        return PF_OK;
    }
    // Rows that leave lanes of a wave idle above, or need several waves there, on as many lanes as three vectors each fill (with waves to
    // fill the device, two to a SIMD).  Softmax of 129-192 vectors, us before and now: 1160 columns fp16, 46 400 rows 43.1 -> 36.1, causal
    // 41.1 -> 29.5, [3, 12, 704, 704] fp32 causal 26.4 -> 19.8.  Of 33-48 and 65-80 vectors, several rows side by side in a wave, up to 32 768
    // rows: 272 columns fp16, 32 640 rows 10.0 -> 8.7, 384, 12 288 rows 5.5 -> 4.7, 168 fp32, 26 880 rows, causal 9.2 -> 7.2; with more rows the
    // waves above keep more loads in flight (376 columns fp16, 120 320 rows 31.9 against 36.4).  Normalisations of two full operands: a wave to
    // a row, three or five to eight vectors a lane, where rows are ragged or fp32: 2639 columns fp16 23.1 -> 20.2, 1119 fp32 39.4 -> 31.0, 1532
    // fp32 28.8 -> 26.5 (whole fp16 rows: 2640 columns 16.1 both, 3520 15.4 against 16.0; 1999 columns fp32, eight vectors, 30.3 against 30.9).
    int wide_k = 0, wide_l = 6;
    if (jit_ok && forced_variant < 0 && L.n_out == 1 && L.core == pf::CORE_SOFTMAX && L.n_full == 1 && L.n_vec == 0) {
        for (int l = 4; l <= 6; ++l)
            if (vpr > (2 << l) && vpr <= (l == 5 ? 80 : 3 << l) && (l == 6 || rows <= 32768)) wide_k = 3, wide_l = l;
    } else if (jit_ok && forced_variant < 0 && L.n_out == 1 && (L.core == pf::CORE_LAYERNORM || L.core == pf::CORE_RMSNORM) && L.n_full == 2 && (p->ragged || es == 4)) {
        if ((vpr > 128 && vpr <= 192) || (vpr > 256 && vpr <= 512)) wide_k = (int)((vpr + 63) / 64);
        if (wide_k == 8 && p->ragged && es == 4) wide_k = 0;
    }
    if (rows < ((int64_t)2048 << (6 - wide_l)) || env_int("PF_ROW_WIDE", 1) == 0) wide_k = 0;
    if (wide_k > 0) {
        // (a kernel that does not fit the registers is not taken)
        std::string err;
        hipFunction_t fn = pf::jit_row_kernel(p->device, L.main_dtype, wide_k, 1, true, p->ragged, 256, wide_l, make_jit_spec(L), &err);
        if (!fn || pf::jit_scratch_bytes(fn) != 0) wide_k = 0;
    }
    if (wide_k > 0) best_wpr = 1, best_k = wide_k;
    p->variant = best_wpr == 1 ? PF_VARIANT_ROW_WAVE : PF_VARIANT_ROW_BLOCK;
    p->k = best_k;
    p->row.waves_per_row = (uint32_t)best_wpr;
    p->row.rows_per_block = best_wpr >= 4 ? 1u : (uint32_t)(4 / best_wpr);
    if (best_wpr == 1 && env_int("PF_ROW_WAVES", 0) > 0) p->row.rows_per_block = (uint32_t)env_int("PF_ROW_WAVES", 4);
    p->row.rows_per_wave = 1;
    // Rows per wave: a wave that owns short rows takes several at once, so that it has about 4 KB of loads
    // in flight (what it takes to cover the HBM latency at full occupancy), as long as enough waves remain
    // (16 per SIMD) to fill the device evenly and a specialised kernel exists for the combination.
    if (best_wpr == 1 && (matched || jit_ok) && L.n_out == 1 && wide_k == 0) {
        const int64_t bytes_per_row_in_flight = (int64_t)L.n_full * best_k * 1024;
        int rpw = 1;
        while (rpw < 4 && bytes_per_row_in_flight * rpw < 4096 && best_k * rpw * 2 <= 4 && rows / (rpw * 2) >= 16384) rpw *= 2;
        const int forced = env_int("PF_ROWS_PER_WAVE", 0);
        if (forced > 0) rpw = forced;
        if (rpw > 1 && have_static(best_k, rpw, true, 256)) p->row.rows_per_wave = (uint32_t)rpw;
    }
    // Waves that own their rows and have at most 2 KB of loads in flight each (one short row, or two whose tails a causal
    // mask cuts off) do better two to a workgroup than four: C2 15.3 -> 14.7 us, a plain softmax of 512 columns 18.3 ->
    // 17.9 us; with 4 KB per wave (C3) four are better (17.7 against 17.9 us), eight and sixteen worse for all.
    if (best_wpr == 1 && env_int("PF_ROW_WAVES", 0) == 0 && (int64_t)L.n_full * best_k * p->row.rows_per_wave * 1024 <= 2048) p->row.rows_per_block = 2;
    // (softmax of 40 vectors, two waves to a workgroup or four: 5.1 and 5.3 us, ragged 7.0 and 6.9; of 145 vectors 37.2 and 36.1)
    if (wide_k > 0 && env_int("PF_ROW_WAVES", 0) == 0) p->row.rows_per_block = wide_l == 4 && !p->ragged ? 2u : 4u;
    p->block = dim3(64u * best_wpr * p->row.rows_per_block);
    p->lds_bytes = best_wpr > 1 ? 2 * 16 * 4 : 0;
    // Short rows (at most 32 vectors): several rows side by side in a wave, 8 / 16 / 32 lanes each, instead of
    // one row on a wave whose other lanes idle.  Exists in plan-time specialised form only.
    int log2l = 6;
    if (best_wpr == 1 && best_k == 1 && vpr <= 32 && jit_ok && !reduce_only && L.n_out == 1 && rows >= 256) {
        log2l = 3;
        while ((1 << log2l) < vpr) ++log2l;
        // A wave that serves several rows side by side has their loads in flight: two steps of rows, no more, for 32 lanes to a row (softmax of
        // 256 columns fp16, 22 528 rows 6.0 us with one, 4.9 with two; 83 968 rows 16.4 with four, 15.4 with two; 244 columns 34.2 with
        // four, 32.2 with two) and for ragged rows (61 columns 8.4 with four, 7.8 with two).
        if (L.core == pf::CORE_SOFTMAX && L.n_full == 1 && L.n_vec == 0 && env_int("PF_ROWS_PER_WAVE", 0) == 0) {
            if (log2l == 5 && rows >= 16384) p->row.rows_per_wave = 2;
            else if (p->ragged && p->row.rows_per_wave > 2u) p->row.rows_per_wave = 2;
        }
    }
    if (wide_k > 0) log2l = wide_l;
    {
        const int forced_l = env_int("PF_ROW_LOG2_LANES", 0);
        if (forced_l >= 3 && forced_l <= 6 && best_wpr == 1 && best_k == 1 && vpr <= (1 << forced_l) && jit_ok && !reduce_only && L.n_out == 1) log2l = forced_l;
    }
    p->row_log2l = log2l;
    p->spec_id = (log2l == 6 && matched && pf::row_static_available(matched, p->k, (int)p->row.rows_per_wave, best_wpr == 1, p->block.x)) ? matched : 0;
    if (!p->spec_id && jit_ok && (wide_k > 0 || have_static(p->k, (int)p->row.rows_per_wave, best_wpr == 1, p->block.x))) {
        std::string err;
        if (reduce_only) p->jit_fn = pf::jit_row_reduce_kernel(p->device, L.main_dtype, p->k, p->ragged, make_jit_spec(L), &err);
        else p->jit_fn = pf::jit_row_kernel(p->device, L.main_dtype, p->k, (int)p->row.rows_per_wave, best_wpr == 1, p->ragged,
                                       p->block.x <= 256 ? 256 : 1024, log2l, make_jit_spec(L), &err);
        if (p->jit_fn) p->spec_id = pf::kSpecJit;
        else note_interpreter_fallback(p, err);
    }
    if (!p->spec_id) {
        p->row.rows_per_wave = 1;
        p->row_log2l = 6;
    }
    {
        const int64_t rows_per_block = (int64_t)p->row.rows_per_block * p->row.rows_per_wave * (64 >> p->row_log2l);
        p->grid = dim3((uint32_t)((rows + rows_per_block - 1) / rows_per_block));
    }
    // Tensors of half a megabyte and more: the kernel is compiled for this shape (row length and count, mask period and
    // mode, waves per row as constants), which removes the tests and divisions in front of a wave's first load.  Not
    // below that: a compilation per shape is only worth it where the launch is long enough to notice.
    const int const_mode = env_int("PF_ROW_CONST", 1);
    if (p->spec_id && !reduce_only && jit_ok && const_mode != 0 && (const_mode == 2 || rows * n * es >= (512 << 10))) {
        pf::RowShapeConst sh;
        sh.n_inner = (uint32_t)n;
        sh.rows = (uint64_t)rows;
        sh.mask_si = L.mask_si;
        sh.core_mask = L.core_mask;
        sh.vec_plain_all = p->args.vec_plain_all;
        sh.waves_per_row = p->row.waves_per_row;
        sh.rows_per_block = p->row.rows_per_block;
        std::string err;
        hipFunction_t fn = pf::jit_row_kernel_const(p->device, L.main_dtype, p->k, (int)p->row.rows_per_wave, best_wpr == 1, p->ragged,
                                                   p->block.x <= 256 ? 256 : 1024, p->row_log2l, make_jit_spec(L), sh, &err);
        // (rows taken on three or more vectors a lane for fitting the registers: only where this kernel fits them too)
        if (fn && (wide_k == 0 || pf::jit_scratch_bytes(fn) == 0)) {
            p->jit_fn = fn;
            p->spec_id = pf::kSpecJit;
        }
    }
    return PF_OK;
}

pf_status plan_ew(pf_plan_s* p) {
    const Lowered& L = p->low;
    const int es = dtype_size(L.main_dtype);
    const int vec = 16 / es;
    const int64_t n = L.pre_shape.back();
    const int64_t total = numel(L.pre_shape);
    if ((n * es) % 16 != 0) p->ragged = true;
    if (p->ragged) {
        for (int i = 0; i < L.pro.n; ++i)
            if (L.pro.u[i].code == pf::U_MASK_CAUSAL)
                return fail(PF_ERR_UNSUPPORTED, "a causal mask without a row reduction needs rows of whole 16-byte vectors");
    }
    const int64_t total_vecs = (total + vec - 1) / vec;
    if (total_vecs > 0xffffffffLL) return fail(PF_ERR_UNSUPPORTED, "tensor too large for the element-wise family");
    p->family = PF_FAMILY_ELEMENTWISE;
    p->variant = PF_VARIANT_EW_FLAT;
    p->k = 1;
    p->ew_total_vecs = (uint32_t)total_vecs;
    p->ew_vecs_per_row = (uint32_t)std::max<int64_t>(1, n / vec);
    p->block = dim3(256);
    p->grid = dim3((uint32_t)((total_vecs + 256 * p->k - 1) / (256 * p->k)));
    p->args.n_inner = (uint32_t)n;
    p->args.rows = (uint64_t)(total / n);
    if (jit_possible(p->device)) {
        std::string err;
        p->jit_fn = pf::jit_ew_kernel(p->device, L.main_dtype, p->k, p->ragged, make_jit_spec(L), &err);
        if (p->jit_fn) p->spec_id = pf::kSpecJit;
        else note_interpreter_fallback(p, err);
    }
    return PF_OK;
}


pf::FastDiv make_fastdiv(uint32_t d) {
    pf::FastDiv f;
    f.d = d;
    if (d <= 1) {
        f.m = 0; f.s1 = 0; f.s2 = 0;
        return f;
    }
    uint32_t l = 0;
    while ((1ull << l) < d) ++l;
    f.m = (uint32_t)((((1ull << 32) * ((1ull << l) - d)) / d) + 1);
    f.s1 = 1;
    f.s2 = l - 1;
    return f;
}

// ---- transpose family
pf_status plan_perm(pf_plan_s* p, int forced_variant) {
    const Lowered& L = p->low;
    const int es = dtype_size(L.main_dtype);
    const int vec = 16 / es;
    const Shape& in = L.pre_shape;
    const int rank = (int)in.size();
    if (numel(in) > 0xffffffffLL) return fail(PF_ERR_UNSUPPORTED, "tensor too large for the transpose family");
    // extents that are not whole vectors on either side (or a broadcast operand that is not): element-granular kernels
    const bool ragged = p->ragged || (L.pre_shape.back() * es) % 16 != 0 || (L.post_shape.back() * es) % 16 != 0;
    p->ragged = ragged;
    if (ragged && (L.pre_shape.back() == 1 || L.post_shape.back() == 1))
        return fail(PF_ERR_UNSUPPORTED, "permutations of tensors whose innermost extent is 1 are not implemented (reshape it away)");
    for (int i = 0; i < L.pro.n; ++i)
        if (L.pro.u[i].code == pf::U_STORE) return fail(PF_ERR_UNSUPPORTED, "secondary outputs are not implemented in the transpose family");
    for (int i = 0; i < L.epi.n; ++i)
        if (L.epi.u[i].code == pf::U_STORE) return fail(PF_ERR_UNSUPPORTED, "secondary outputs are not implemented in the transpose family");
    // input strides
    std::vector<int64_t> istr(rank);
    int64_t acc = 1;
    for (int k = rank - 1; k >= 0; --k) { istr[k] = acc; acc *= in[k]; }
    // output dims in order, dropping extent-1 dims and merging dims that stay adjacent
    bool uses_positions = L.n_vec != 0 || L.mask_si != 0 || L.core_mask != 0;
    for (int i = 0; i < L.pro.n; ++i) uses_positions |= L.pro.u[i].code == pf::U_MASK_CAUSAL;
    for (int i = 0; i < L.epi.n; ++i) uses_positions |= L.epi.u[i].code == pf::U_MASK_CAUSAL;
    const bool merge_ragged = ragged && !uses_positions && L.perm[rank - 1] != rank - 1 && env_int("PF_PERM_MERGE_RAGGED", 1) != 0;
    struct Dim { int64_t extent, in_stride; };
    std::vector<Dim> od;
    for (int q = 0; q < rank; ++q) {
        const int src = L.perm[q];
        if (in[src] == 1) continue;
        // (ragged: dimensions are not merged, so that the innermost dimension of each side is one the vectors of
        // broadcast operands and the partial last vector can be told from -- unless nothing in the chain looks at
        // positions: an innermost-changing permutation without broadcast operands or mask, where merging h and w of
        // a 7 x 7 feature map makes the transposed extent 49 instead of 7)
        if ((!ragged || merge_ragged) && !od.empty() && od.back().in_stride == in[src] * istr[src]) {
            od.back().extent *= in[src];
            od.back().in_stride = istr[src];
        } else {
            od.push_back(Dim{in[src], istr[src]});
        }
    }
    if (od.empty()) od.push_back(Dim{1, 1});
    const int m = (int)od.size();
    pf::PermGeom& g = p->permg;
    memset(&g, 0, sizeof(g));
    g.in_n_inner = (uint32_t)L.pre_shape.back();
    g.out_n_inner = (uint32_t)L.post_shape.back();
    g.div_in_inner = make_fastdiv(g.in_n_inner);
    g.div_out_inner = make_fastdiv(g.out_n_inner);
    g.total_vecs = (uint32_t)(numel(in) / vec);
    for (int f = 0; f < L.n_full; ++f) if (L.full_is_epi[f]) g.epi_full_mask |= 1u << f;
    for (int v = 0; v < L.n_vec; ++v) if (L.vec_is_epi[v]) g.epi_vec_mask |= 1u << v;
    // output strides of the merged dims
    std::vector<int64_t> ostr(m);
    acc = 1;
    for (int q = m - 1; q >= 0; --q) { ostr[q] = acc; acc *= od[q].extent; }
    p->family = PF_FAMILY_TRANSPOSE;
    p->spec_id = (env_int("PF_NO_STATIC", 0) || ragged) ? 0 : match_spec(spec_table().perm, L);
    p->args.n_inner = g.in_n_inner;
    p->args.rows = (uint64_t)(numel(in) / g.in_n_inner);

    if (od.back().in_stride != 1) {
        // ---- the innermost dimension changes: square tiles over (input-innermost I, output-innermost O)
        if (forced_variant >= 0 && forced_variant != PF_VARIANT_T_TILE)
            return fail(PF_ERR_UNSUPPORTED, "variant %d is not implemented for this permutation", forced_variant);
        int qi = -1;
        for (int q = 0; q < m; ++q)
            if (od[q].in_stride == 1) qi = q;
        if (qi < 0) return fail(PF_ERR_UNSUPPORTED, "internal: no contiguous input dimension");
        const int64_t n_i = od[qi].extent, n_o = od.back().extent;
        if (!ragged && ((n_i * es) % 16 != 0 || (n_o * es) % 16 != 0))
            return fail(PF_ERR_ALIGNMENT, "transposed extents (%lld, %lld) are not multiples of 16 bytes", (long long)n_i, (long long)n_o);
        const bool pro_trivial = L.pro.n == 1 && L.pro.u[0].code == pf::U_MOV && L.pro.u[0].kind == pf::K_FULL && L.pro.u[0].slot == 0;
        if (es == 2 && !pro_trivial && L.epi.n != 0)
            return fail(PF_ERR_UNSUPPORTED, "16-bit chains may compute on one side of an innermost-changing permutation only");
        if (L.n_full < 1 || L.pro.n < 1 || L.pro.u[0].code != pf::U_MOV || L.pro.u[0].kind != pf::K_FULL || L.pro.u[0].slot != 0)
            return fail(PF_ERR_UNSUPPORTED, "the permuted value must start from a full-shape input");
        const int64_t te = 8 * vec;
        int r = 0;
        uint64_t total_tiles = 1;
        for (int q = 0; q < m - 1; ++q) {
            if (q == qi) continue;
            g.extent[r] = (uint32_t)od[q].extent;
            g.in_stride[r] = (uint32_t)od[q].in_stride;
            g.out_stride[r] = (uint32_t)ostr[q];
            ++r;
        }
        g.extent[r] = (uint32_t)((n_i + te - 1) / te);
        g.in_stride[r] = (uint32_t)te;
        g.out_stride[r] = (uint32_t)(te * ostr[qi]);
        ++r;
        g.extent[r] = (uint32_t)((n_o + te - 1) / te);
        g.in_stride[r] = (uint32_t)(te * od.back().in_stride);
        g.out_stride[r] = (uint32_t)te;
        ++r;
        g.rank = r;
        for (int q = 0; q < r; ++q) {
            g.div[q] = make_fastdiv(g.extent[q]);
            total_tiles *= g.extent[q];
        }
        if (total_tiles > 0x7fffffffull) return fail(PF_ERR_UNSUPPORTED, "tensor too large for the transpose family");
        g.total_vecs = (uint32_t)total_tiles;
        g.tile_a = (uint32_t)n_i;
        g.tile_b = (uint32_t)n_o;
        g.t_in_stride_o = (uint32_t)od.back().in_stride;
        g.t_out_stride_i = (uint32_t)ostr[qi];
        p->variant = PF_VARIANT_T_TILE;
        p->k = vec;
        p->block = dim3(256);
        p->grid = dim3((uint32_t)((total_tiles + 3) / 4));
        p->lds_bytes = 0;
        // A layout-only swap of a plane's two dimensions with an extent that is not whole vectors: strips that are one stretch
        // of memory on the side whose rows are not (perm_plane_kernel), if `step` rows of it (a 128-byte line of the other
        // side; half of one for long rows) fit 64 KB of LDS, which leaves a compute unit two workgroups.  Half lines only in
        // whole vectors ([64, 384, 29, 29] fp16 to channels-last 31.2 -> 22.6 us; with 500 channels 50.7 against 51.8).
        const int64_t n_a = n_o, n_b = n_i;  // input plane [a, b]
        bool swap = ragged && p->args.raw_copy && L.n_vec == 0 && env_int("PF_NO_STATIC", 0) == 0 && env_int("PF_PERM_PLANE", 1) != 0 &&
                    od.back().in_stride == n_b && ostr[qi] == n_a;
        // the other dimensions keep their order around the plane
        for (int q = 0; q < m - 1 && swap; ++q)
            if (q != qi) swap = od[q].in_stride == ostr[q] && ostr[q] >= n_a * n_b;
        if (swap) {
            const bool flat_out = (n_b * es) % 16 == 0;  // the input's rows are whole vectors: the output's are not
            const int64_t flat_rows = flat_out ? n_b : n_a, flat_len = flat_out ? n_a : n_b;
            int64_t step = 128 / es;
            auto lds_of = [&](int64_t st) { return flat_out ? flat_len * (st + 1) * es : (st * flat_len + 2 * vec) * es; };
            if (lds_of(step) > 64 * 1024 && ((flat_out ? n_b : n_a) * es) % 16 == 0) step /= 2;
            // Strips enough: a flat output pays off with two to a compute unit ([32, 56, 56, 100] 20.7 -> 11.0 us; 384 strips of
            // [64, 14, 14, 384] 8.4 against 8.6, ten of [1, 30, 30, 320] 6.9 against 10.7), half lines likewise; a flat input
            // always ([2, 96, 15, 15] 9.1 -> 7.2).
            const int64_t planes = numel(in) / (n_a * n_b), per_plane = (flat_rows + step - 1) / step;
            const bool enough = planes * per_plane >= 512 || (!flat_out && step * es == 128);
            // (a launch holds fewer than 2^32 lanes, strips are dealt to eight dies: with more than that the tiles take over, four to
            // a workgroup)
            if (enough && lds_of(step) <= 64 * 1024 && planes * per_plane <= (1LL << 24) - 8) {
                pf::PlaneGeom& pg = p->planeg;
                pg.a = (uint32_t)n_a;
                pg.b = (uint32_t)n_b;
                pg.step = (uint32_t)step;
                pg.strips = (uint32_t)(planes * per_plane);
                pg.strips_per_die = (pg.strips + 7u) / 8u;
                pg.div_strips = make_fastdiv((uint32_t)per_plane);
                pg.div_a = make_fastdiv(pg.a);
                pg.total = (uint64_t)numel(in);
                p->perm_plane = flat_out ? 2 : 1;
                p->spec_id = 2;  // the catalogue's layout-only permutation
                p->lds_bytes = (uint32_t)((lds_of(step) + 15) / 16 * 16);
                p->grid = dim3(pg.strips_per_die * 8u);
                return PF_OK;
            }
        }
        if (!p->spec_id && jit_possible(p->device)) {
            std::string err;
            p->jit_fn = pf::jit_perm_kernel(p->device, L.main_dtype, p->variant, p->k, ragged, make_jit_spec(L), &err);
            if (p->jit_fn) p->spec_id = pf::kSpecJit;
            else note_interpreter_fallback(p, err);
        }
        return PF_OK;
    }
    const int64_t inner = od.back().extent;
    if (!ragged && (inner * es) % 16 != 0) return fail(PF_ERR_ALIGNMENT, "innermost run of %lld elements is not a multiple of 16 bytes", (long long)inner);
    const int64_t inner_vecs = (inner + vec - 1) / vec;  // the last one partial when ragged
    if (ragged) {
        const int64_t tv = numel(in) / inner * inner_vecs;
        if (tv > 0xffffffffLL) return fail(PF_ERR_UNSUPPORTED, "tensor too large for the transpose family");
        g.total_vecs = (uint32_t)tv;
    }
    // LDS-staged variant: [batch, A, B, inner] -> [batch, B, A, inner]
    bool lds_ok = false;
    uint32_t ta = 0, tb = 0;
    int ia = -1, ib = -1;  // output positions of B (first) and A (second): out = [batch?, B, A, inner]
    if (!ragged && (m == 3 || m == 4)) {
        ib = m - 3;
        ia = m - 2;
        const Dim& B = od[ib];
        const Dim& A = od[ia];
        // in the input A is outside B: stride(A) == extent(B) * stride(B), stride(B) == inner
        const bool pattern = B.in_stride == inner && A.in_stride == B.extent * inner && (m == 3 || od[0].in_stride == A.extent * A.in_stride);
        if (pattern) {
            const int64_t inner_v = inner / vec;
            // tile: tb inner rows of B per input run, ta of A per output run; keep the tile near 32 KB
            for (int64_t cand_b = std::min<int64_t>(B.extent, 32); cand_b >= 1 && !lds_ok; --cand_b) {
                if (B.extent % cand_b != 0) continue;
                for (int64_t cand_a = 32; cand_a >= 2; --cand_a) {
                    if (A.extent % cand_a != 0) continue;
                    const int64_t bytes = cand_a * (cand_b * inner_v + 16) * 16;
                    if (bytes > 48 * 1024 || cand_a * cand_b * inner_v < 256) continue;
                    ta = (uint32_t)cand_a; tb = (uint32_t)cand_b; lds_ok = true;
                    break;
                }
            }
        }
    }
    int variant = forced_variant >= 0 ? forced_variant : PF_VARIANT_T_ROWS;
    if (variant == PF_VARIANT_T_LDS_ROWS && !lds_ok)
        return fail(PF_ERR_UNSUPPORTED, "the LDS-staged variant needs a [.., A, B, inner] -> [.., B, A, inner] permutation with tileable extents");
    if (variant != PF_VARIANT_T_ROWS && variant != PF_VARIANT_T_LDS_ROWS)
        return fail(PF_ERR_UNSUPPORTED, "variant %d is not implemented for this permutation", variant);
    p->variant = variant;
    if (variant == PF_VARIANT_T_LDS_ROWS) {
        const Dim& B = od[ib];
        const Dim& A = od[ia];
        const int64_t batch = m == 4 ? od[0].extent : 1;
        g.rank = 4;
        g.extent[0] = (uint32_t)batch;
        g.extent[1] = (uint32_t)(A.extent / ta);
        g.extent[2] = (uint32_t)(B.extent / tb);
        g.extent[3] = (uint32_t)(inner / vec);
        g.in_stride[0] = m == 4 ? (uint32_t)od[0].in_stride : 0u;
        g.in_stride[1] = (uint32_t)A.in_stride;
        g.in_stride[2] = (uint32_t)B.in_stride;
        g.in_stride[3] = 1;
        g.out_stride[0] = m == 4 ? (uint32_t)ostr[0] : 0u;
        g.out_stride[1] = (uint32_t)ostr[ia];
        g.out_stride[2] = (uint32_t)ostr[ib];
        g.out_stride[3] = 1;
        g.tile_a = ta;
        g.tile_b = tb;
        {
            // pad the staged line so that stepping one line advances the bank index (256 bytes of bank space =
            // 16 vectors) by one inner row: pitch = row (mod 16 vectors) must equal inner (mod 16 vectors)
            const int64_t inner_v = inner / vec, row_v = tb * inner_v;
            const int64_t pad = (((inner_v - row_v) % 16) + 16) % 16;
            g.lds_pitch = (uint32_t)(row_v + (env_int("PF_LDS_PAD", -1) >= 0 ? env_int("PF_LDS_PAD", 0) : pad));
        }
        p->k = 1;
        p->block = dim3(256);
        p->grid = dim3((uint32_t)(batch * (A.extent / ta) * (B.extent / tb)));
        p->lds_bytes = (uint32_t)(ta * g.lds_pitch * 16);
    } else {
        if (m > PF_DEV_MAX_RANK) return fail(PF_ERR_UNSUPPORTED, "too many dimensions");
        // Two dimensions X, Y that swap around a kept innermost run ([.., Y, X, inner] -> [.., X, Y, inner]) and whose
        // run is short: walked in output order, a workgroup writes one long contiguous stretch but reads runs of `inner`
        // elements a whole X row apart.  Walking tx x ty blocks of (X, Y) instead gives both sides stretches of about
        // 512 bytes (C4, 128-byte runs: 14.3 us in output order, 13.3 us in blocks of 4 x 4; 2 x 2 to 4 x 16 within 0.2 us
        // of each other, 16 x 2 at 13.9 us).
        int tile_t = 0, tile_y = 0;
        if (!ragged && m >= 3 && m + 2 <= PF_DEV_MAX_RANK && od[m - 3].in_stride == inner && od[m - 2].in_stride == od[m - 3].extent * inner) {
            const int64_t run_bytes = inner * es;
            int64_t want = 1;
            while (want * 2 * run_bytes <= 512) want *= 2;
            int64_t tx = want, ty = want;
            while (tx > 1 && od[m - 3].extent % tx != 0) tx /= 2;
            while (ty > 1 && od[m - 2].extent % ty != 0) ty /= 2;
            const int forced = env_int("PF_PERM_BLOCK", -1), forced_y = env_int("PF_PERM_BLOCK_Y", forced);
            if (forced >= 1 && forced_y >= 1 && od[m - 3].extent % forced == 0 && od[m - 2].extent % forced_y == 0) tx = forced, ty = forced_y;
            if (forced != 0 && (tx > 1 || ty > 1)) tile_t = (int)tx, tile_y = (int)ty;
        }
        if (tile_t) {
            const Dim X = od[m - 3], Y = od[m - 2];
            const int64_t ox = ostr[m - 3], oy = ostr[m - 2];
            int r = 0;
            auto put = [&](int64_t extent, int64_t is, int64_t os) {
                g.extent[r] = (uint32_t)extent;
                g.in_stride[r] = (uint32_t)is;
                g.out_stride[r] = (uint32_t)os;
                g.div[r] = make_fastdiv(g.extent[r]);
                ++r;
            };
            for (int q = 0; q < m - 3; ++q) put(od[q].extent, od[q].in_stride, ostr[q]);
            put(X.extent / tile_t, X.in_stride * tile_t, ox * tile_t);
            put(Y.extent / tile_y, Y.in_stride * tile_y, oy * tile_y);
            put(tile_y, Y.in_stride, oy);
            put(tile_t, X.in_stride, ox);
            put(inner_vecs, 1, 1);
            g.rank = r;
        } else {
        g.rank = m;
        for (int q = 0; q < m; ++q) {
            g.extent[q] = (uint32_t)(q == m - 1 ? inner_vecs : od[q].extent);
            g.in_stride[q] = (uint32_t)od[q].in_stride;
            g.out_stride[q] = (uint32_t)ostr[q];
            g.div[q] = make_fastdiv(g.extent[q]);
        }
        }
        p->k = (g.total_vecs >= 65536u && !ragged) ? 2 : 1;
        if (!ragged && env_int("PF_PERM_K", 0) >= 1 && env_int("PF_PERM_K", 0) <= 16) p->k = env_int("PF_PERM_K", 2);
        g.tile_a = (uint32_t)inner;  // (ragged kernels: length of the innermost run)
        p->block = dim3(256);
        p->grid = dim3((g.total_vecs + 256u * p->k - 1) / (256u * p->k));
        p->lds_bytes = 0;
    }
    // Large tensors on the rows variant: the kernel is compiled for this geometry (index arithmetic on constants).  Worth
    // a compilation per shape only where the launch is long enough to notice; smaller ones keep the run-time geometry.
    if (p->variant == PF_VARIANT_T_ROWS && !ragged && !L.general_bcast && jit_possible(p->device) && env_int("PF_PERM_CONST", 1) != 0 &&
        (g.total_vecs >= (1u << 20) || env_int("PF_PERM_CONST", 1) == 2)) {
        uint32_t numel[PF_DEV_MAX_VEC] = {1, 1, 1, 1}, period[PF_DEV_MAX_VEC] = {1, 1, 1, 1};
        for (int v = 0; v < L.n_vec; ++v) {
            numel[v] = p->args.vec[v].numel;
            period[v] = p->args.vec[v].period_rows;
        }
        // eight vectors per lane (the built-in kernels exist for one and two): C4 12.9 us with two, 12.4 with four, 11.9
        // with eight, 12.0 with sixteen; six or twelve, which cut across the blocks, 13.0 - 13.6
        const int k_const = env_int("PF_PERM_K", 0) ? p->k : 8;
        std::string err;
        hipFunction_t fn = pf::jit_perm_rows_const(p->device, L.main_dtype, k_const, make_jit_spec(L), g, numel, period, &err);
        if (fn) {
            p->jit_fn = fn;
            p->spec_id = pf::kSpecJit;
            p->k = k_const;
            p->grid = dim3((g.total_vecs + 256u * p->k - 1) / (256u * p->k));
            return PF_OK;
        }
        if (p->k > 2) {
            p->k = 2;
            p->grid = dim3((g.total_vecs + 256u * p->k - 1) / (256u * p->k));
        }
    }
    if (!p->spec_id && jit_possible(p->device)) {
        std::string err;
        p->jit_fn = pf::jit_perm_kernel(p->device, L.main_dtype, p->variant, p->k, ragged, make_jit_spec(L), &err);
        if (p->jit_fn) p->spec_id = pf::kSpecJit;
        else note_interpreter_fallback(p, err);
    }
    return PF_OK;
}

// ---- group family
// GroupNorm over slabs of whole groups (group_slab_kernel).  false where the kernel does not take the chain or is not the quicker one.
// tiles, tiles_per_sample, rounds: what the one-launch kernel of whole positions would be planned with (rounds: of co-resident tiles).
//
// Two ranges (44 shapes, 550 pairs of slab and slices measured; geometric mean over the shapes 0.86 of the kernel of whole positions):
//  - one slice to a slab, six steps at most and one workgroup to a unit at most: nothing is exchanged, which is half of what a small call
//    costs.  us, fp16 or bf16: [31, 10, 10, 96] 9.7 -> 5.9, [11, 14, 14, 640] 8.4 -> 5.9, [21, 14, 14, 352] 8.9 -> 6.7; fp32: [2, 7, 7, 1216]
//    7.4 -> 5.1, [6, 32, 32, 128] 9.5 -> 7.6.  With more steps the strided reads cost more than the exchange: [2, 32, 32, 224] bf16, 15 steps,
//    9.7 against 8.8, [20, 28, 28, 512] bf16, 13 steps, 12.0 against 10.1.
//  - slices where the other kernel would go several rounds, or a sample is so many tiles that a lane reads its words in more than three
//    trips (48; 42 in fp32; 16-bit tensors of more tiles than units excepted: [6, 64, 64, 416] bf16 19.6, 20.9 in slabs).  us, fp32:
//    [7, 56, 56, 768] 79.9 -> 36.9, [1, 56, 56, 416] 18.0 -> 10.4, [4, 64, 64, 320] 23.8 -> 18.8, [13, 28, 28, 960] 32.4 -> 27.4; 16 bits:
//    [21, 64, 64, 352] 44.1 -> 33.0, [4, 64, 64, 224] 13.6 -> 12.4.
static bool plan_group_slab(pf_plan_s* p, int n_cu, int64_t n, int64_t hw, int64_t ch, int64_t tiles, int64_t tiles_per_sample, int64_t rounds) {
    const Lowered& L = p->low;
    const int mode = env_int("PF_GROUP_SLAB", 1);  // 0 never, 2 wherever it is possible, quicker or not
    if (!jit_possible(p->device) || mode == 0 || env_int("PF_GROUP_GENERAL", 0) != 0 || env_int("PF_GROUP_NV", 0) != 0) return false;
    const int64_t groups = L.groups, cpg = ch / groups;
    const int es = dtype_size(L.main_dtype), vec = 16 / es;
    if ((ch * es) % 16 != 0 || hw * ch * es > 0x7fffffffLL) return false;
    const int forced_d = env_int("PF_SLAB_GROUPS", 0), forced_slices = env_int("PF_SLAB_SLICES", 0);
    const bool forced = mode == 2;
    const bool sliced_pays = rounds > 1 || (es == 4 ? tiles_per_sample > 42 : tiles_per_sample > 48 && tiles <= n_cu);
    struct Pick {
        double cost;
        int64_t d, nv, slices, blocks;
    };
    std::vector<Pick> picks;
    for (int64_t d = 1; d <= groups && d <= 512; ++d) {
        if (groups % d != 0 || (forced_d && d != forced_d) || (d * cpg * es) % 16 != 0) continue;
        const int64_t slabs = n * (groups / d), cvs = d * cpg / vec;
        if (cvs > 512) continue;
        const int64_t pps = 512 / cvs, width = cvs * 16;
        const bool lines = (width % 128 == 0 && (ch * es) % 128 == 0) || d == groups;
        const double waste = std::min(3.0, (double)(((width + 127) / 128 + (lines ? 0 : 1)) * 128) / (double)width - 1.0);  // (of the memory lines a position's share touches)
        for (int64_t slices = 1; slices <= std::min<int64_t>(64, hw); ++slices) {
            if (forced_slices && slices != forced_slices) continue;
            const int64_t longest = (hw + slices - 1) / slices, nv = (longest + pps - 1) / pps, blocks = slabs * slices;
            if (nv > 44 || (nv - 1) * pps > hw / slices || blocks > 0x7fffff) continue;  // (every step of every slice but the last is whole)
            const bool small = slices == 1 && nv <= 6, large = sliced_pays && width >= 64;
            if ((blocks > n_cu || !(small || large)) && !forced) continue;
            // (more than 16 vectors a lane are taken for one workgroup to a unit: not compiled where two launches could not share the device)
            if (slices > 1 && nv > 16 && !pf::group_slab_shares((uint32_t)slices, (uint32_t)((blocks + 7) / 8), (uint32_t)n_cu / 8)) continue;
            // microseconds beside what the bytes cost, fitted to the pairs of at most one workgroup to a unit
            const double cost = (double)nv * ((es == 4 ? 0.25 : 0.165) + 0.044 * waste) + 0.11 * std::log2((double)pps) + (slices > 1 ? 1.97 + 0.0515 * (double)slices : 0.0);
            picks.push_back(Pick{cost, d, nv, slices, blocks});
        }
    }
    std::sort(picks.begin(), picks.end(), [](const Pick& x, const Pick& y) { return x.cost < y.cost; });
    pf::GroupSlabGeom& g = p->gslab;
    memset(&g, 0, sizeof(g));
    hipFunction_t fn = nullptr;
    std::string err;
    g.parts = 1;
    for (int64_t v = 0; v < ch / vec; ++v) g.parts = std::max<uint32_t>(g.parts, (uint32_t)((v * vec + vec - 1) / cpg - v * vec / cpg + 1));
    const uint32_t dyn_lds = 512u * 3u * g.parts * 4u;
    // A kernel whose vectors do not fit the registers is passed over, three at most: each is compiled first.  Slices wait for one another:
    // all workgroups of the launch have to be resident, and two such launches on two streams must not hold the device in vain.  Any order
    // of the workgroups does where both fit; else as many slabs of a sample are dispatched together as may be (neighbours share memory lines:
    // in runs of one slab [1, 56, 56, 416] fp32 takes 12.2 us, 10.3 in runs of 32).  That leaves 16 slices to a launch that fills the units
    // one to each: [5, 128, 128, 416] fp16 45.4 us, 38.1 in 25 slices, [3, 96, 96, 1120] 40.2, 35.2 in 21 (65.0 and 76.2 by whole positions).
    size_t at = 0;
    uint32_t run_slabs = 1;
    for (; at < picks.size() && at < 3; ++at) {
        fn = pf::jit_group_slab_kernel(p->device, L.main_dtype, (int)picks[at].nv, (int)(picks[at].d * cpg / vec), picks[at].slices > 1, es == 2 && cpg % 2 == 0, make_jit_spec(L), &err);
        const uint32_t per_die = (uint32_t)((picks[at].blocks + 7) / 8), places = fn ? (uint32_t)(std::max(pf::jit_blocks_per_cu(fn, 512, dyn_lds), 0) * n_cu / 8) : 0u;
        const uint32_t slabs = (uint32_t)(groups / picks[at].d), slices = (uint32_t)picks[at].slices;
        run_slabs = slices == 1u ? 1u : slabs;
        while (run_slabs > 1u && (slabs % run_slabs != 0u || !pf::group_slab_shares(run_slabs * slices, per_die, places))) --run_slabs;
        if (fn && pf::jit_scratch_bytes(fn) == 0 && (slices == 1u || (per_die <= places && pf::group_slab_shares(run_slabs * slices, per_die, places)))) break;
        fn = nullptr;
    }
    if (!fn) return false;
    const int64_t best_d = picks[at].d, best_nv = picks[at].nv, best_slices = picks[at].slices;
    g.hw = (uint32_t)hw;
    g.channels = (uint32_t)ch;
    g.groups = (uint32_t)groups;
    g.cpg = (uint32_t)cpg;
    g.div_cpg = make_fastdiv(g.cpg);
    g.slab_groups = (uint32_t)best_d;
    g.slabs_per_sample = (uint32_t)(groups / best_d);
    g.slices = (uint32_t)best_slices;
    g.div_run = make_fastdiv(run_slabs * g.slices);
    g.div_sample = make_fastdiv(g.slabs_per_sample / run_slabs);
    g.div_run_slabs = make_fastdiv(run_slabs);
    g.slice_len = (uint32_t)(hw / best_slices);
    g.slice_rest = (uint32_t)(hw % best_slices);
    g.blocks = (uint32_t)(n * g.slabs_per_sample * best_slices);
    g.blocks_per_die = (g.blocks + 7u) / 8u;
    while (g.log2_lanes < 6u && (best_d << (g.log2_lanes + 1)) <= 512) ++g.log2_lanes;
    const uint32_t grid = g.blocks_per_die * 8u;
    if (best_slices > 1) {
        g.spin_limit = (uint32_t)env_int("PF_GROUP_SPIN_LIMIT", 1 << 22);
        g.gather_words = (uint32_t)(n * groups * best_slices);
        const uint64_t gather_bytes = ((uint64_t)2 * g.gather_words * sizeof(uint64_t) + 255) / 256 * 256, epochs = ((uint64_t)g.blocks * sizeof(uint32_t) + 255) / 256 * 256;
        if (hipSetDevice(p->device) != hipSuccess || plan_workspace_alloc(p, gather_bytes + epochs + 256, "workspace allocation") != PF_OK) return false;
        char* ws = static_cast<char*>(p->workspace);
        if (plan_workspace_fill(p, ws, 0xff, gather_bytes, true) != PF_OK || plan_workspace_fill(p, ws + gather_bytes, 0, epochs + 256, true) != PF_OK) {
            (void)hipFree(p->workspace);
            p->workspace = nullptr;
            return false;
        }
        g.ws_gather = reinterpret_cast<uint64_t*>(ws);
        g.ws_epoch = reinterpret_cast<uint32_t*>(ws + gather_bytes);
        g.ws_error = reinterpret_cast<uint32_t*>(ws + gather_bytes + epochs);
        p->ws_error = g.ws_error;
    }
    p->jit_fn = fn;
    p->group_slab = true;
    p->variant = PF_VARIANT_GROUP_RESIDENT;
    p->spec_id = pf::kSpecJit;
    p->k = (int)best_nv;
    p->grid = dim3(grid);
    p->block = dim3(512);
    p->dyn_lds = dyn_lds;
    p->lds_bytes = dyn_lds + 2 * 512 * 4;
    p->n_launches = 1;
    p->args.n_inner = (uint32_t)ch;
    p->args.rows = (uint64_t)(n * hw);
    return true;
}

pf_status plan_group(pf_plan_s* p, int forced_variant) {
    // on the static scratch array: the two-launch variant, which waits for nobody and so has no failed wait to report
    if (planning_static() || p->stats_only) forced_variant = PF_VARIANT_GROUP_TWO_PASS;
    const Lowered& L = p->low;
    const int es = dtype_size(L.main_dtype);
    const int vec = 16 / es;
    const Shape& sh = L.pre_shape;
    const int64_t samples = sh[0], C = sh.back();
    const int64_t hw = numel(sh) / (samples * C);
    const int64_t G = L.groups;
    // A channel count that is not a whole number of vectors: positions start at element alignment and end in a partial
    // vector.  The general kernels (interpreted or specialised now) read and write such vectors element by element.
    const bool ragged_c = (C * es) % 16 != 0;
    if (p->ragged && !ragged_c) return fail(PF_ERR_ALIGNMENT, "a broadcast input of the group family is not a multiple of 16 bytes");
    const int64_t cpg = C / G;
    const int64_t vpg = cpg / vec, cv = (C + vec - 1) / vec;
    // Groups that are a power-of-two number of whole vectors take the kernels' shuffle-tree path; any other width
    // takes the general one (per-element sums, parts merged through LDS).
    const bool general = ragged_c || cpg % vec != 0 || (vpg & (vpg - 1)) != 0 || vpg > 64 || env_int("PF_GROUP_GENERAL", 0) != 0 ||
                         (p->stats_only && es == 2);  // (statistics for a chain of several kernels: never from packed pairs, see below)
    if (general && G > 512) return fail(PF_ERR_UNSUPPORTED, "more than 512 groups");
    if (samples * hw > 0xffffffffLL || samples > 65535) return fail(PF_ERR_UNSUPPORTED, "tensor too large for the group family");
    for (int i = 0; i < L.pro.n; ++i)
        if (L.pro.u[i].code == pf::U_STORE) return fail(PF_ERR_UNSUPPORTED, "secondary outputs are not implemented in the group family");
    for (int i = 0; i < L.epi.n; ++i)
        if (L.epi.u[i].code == pf::U_STORE) return fail(PF_ERR_UNSUPPORTED, "secondary outputs are not implemented in the group family");
    pf::GroupGeom& g = p->group;
    memset(&g, 0, sizeof(g));
    g.samples = (uint32_t)samples;
    g.hw = (uint32_t)hw;
    g.channels = (uint32_t)C;
    g.groups = (uint32_t)G;
    g.cv = (uint32_t)cv;
    g.vpg = (uint32_t)vpg;
    g.log2_vpg = 0;
    while ((1u << g.log2_vpg) < g.vpg) ++g.log2_vpg;
    g.div_cv = make_fastdiv(g.cv);
    g.cpg = (uint32_t)cpg;
    g.div_cpg = make_fastdiv(g.cpg);
    g.parts = 1;
    for (int64_t v = 0; v < cv; ++v) g.parts = std::max<uint32_t>(g.parts, (uint32_t)(std::min<int64_t>(v * vec + vec - 1, C - 1) / cpg - (v * vec) / cpg + 1));
    g.ragged = ragged_c ? 1u : 0u;
    const uint32_t gen_lds = general ? 512u * g.parts * 3u * (uint32_t)sizeof(float) : 0u;
    p->group_general = general;
    // 2: statistics straight from the packed 16-bit pairs (needs pairs that never straddle groups and nothing but the
    // load in front of the normalisation; the kernel checks the rest at compile time)
    // 3: channel counts that are not whole vectors; 4: both
    // (a chain of several kernels kept its statistics in fp32 from widened values, running mean by running mean: it still does)
    const bool packed_stats = cpg % 2 == 0 && L.main_dtype != PF_F32 && L.pro.n == 1 && !p->stats_only;
    const int gen_parts = !general ? 0 : ragged_c ? (packed_stats ? 4 : 3) : (packed_stats ? 2 : 1);
    g.spin_limit = (uint32_t)env_int("PF_GROUP_SPIN_LIMIT", 1 << 22);  // polls before a wait gives up (tests force it small)
    p->family = PF_FAMILY_GROUP;
    p->spec_id = (env_int("PF_NO_STATIC", 0) || general) ? 0 : match_spec(spec_table().group, L);

    hipDeviceProp_t prop;
    if (hipSetDevice(p->device) != hipSuccess || hipGetDeviceProperties(&prop, p->device) != hipSuccess)
        return fail(PF_ERR_HIP, "cannot query device %d (the group family needs the device at plan time)", p->device);
    const int n_cu = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;

    g.vec_per_channel = 1;
    for (int v = 0; v < L.n_vec; ++v)
        if (p->args.vec[v].numel > (uint32_t)C || p->args.vec[v].n_terms != 0) g.vec_per_channel = 0;
    // Workgroups of 512 threads; a tile is NV position steps of 512 / cv positions each.
    // (workgroups of 256 or 128 threads, i.e. twice or four times the tiles, were measured on C5: 33.5 and 46.9 us
    // against 29.0; 1 024 threads, one workgroup per compute unit, 31.2 against 30.8)
    const uint32_t threads = 512;
    if (g.cv > threads) return fail(PF_ERR_UNSUPPORTED, "more than %d channels", (int)threads * vec);
    g.pos_per_step = threads / g.cv;
    // lanes that share a group when partials are merged: as many as fit, a power of two, at most 64
    g.lanes_per_group = 1;
    while (g.lanes_per_group < 64u && g.lanes_per_group * 2u * g.groups <= threads) g.lanes_per_group *= 2u;

    auto tiling = [&](int nv_c, uint32_t* bps_out) {
        const uint32_t ppb = (uint32_t)nv_c * g.pos_per_step;
        *bps_out = (uint32_t)((hw + ppb - 1) / ppb);
    };
    // The largest tile that still leaves enough workgroups.  The two-launch variant wants two per compute unit.  The
    // one-launch variant does better with fewer, larger tiles, down to about two for every three compute units: all
    // of them are resident at once, and fewer tiles mean fewer words in the exchange (measured: [16,32,32,640]
    // 24.6 us with 688 tiles of 4 steps, 16.9 us with 176 of 16; [16,64,64,128] 16.5 -> 13.2 us).
    const bool fused_candidate = L.n_full == 1 && g.vec_per_channel && forced_variant != PF_VARIANT_GROUP_TWO_PASS &&
                                 (p->spec_id != 0 || jit_possible(p->device));
    const uint64_t min_tiles = fused_candidate ? ((uint64_t)n_cu * 2 + 2) / 3 : 2 * (uint64_t)n_cu;
    const int cands[3] = {16, 8, 4};
    const int forced_nv = env_int("PF_GROUP_NV", 0);
    int nv = 0;
    uint32_t bps = 0;
    for (int ci = 0; ci < 3 && nv == 0; ++ci) {
        if (forced_nv && cands[ci] != forced_nv) continue;
        if (general && !((gen_parts == 2 || gen_parts == 4) && jit_possible(p->device)) && cands[ci] == 16 && !forced_nv) continue;  // (16 vectors fit the general kernels' registers only with packed statistics)
        uint32_t b;
        tiling(cands[ci], &b);
        if ((uint64_t)b * samples >= min_tiles || ci == 2 || forced_nv) {
            nv = cands[ci];
            bps = b;
        }
    }
    if (nv == 0) return fail(PF_ERR_INVALID_ARG, "PF_GROUP_NV must be 4, 8 or 16");
    // Slabs of whole groups: nothing but the load in front (steps there would be run by every pass over the held values), and a sample that the
    // one-launch kernel holds at once, two workgroups to a unit.  (Larger ones are two launches, which can be recorded and wait for nobody: they
    // stay so.)  Tiles of 16 steps become tiles of 12 where the kernel spills: with samples that do not fit as such, that kernel decides first.
    auto try_slabs = [&]() {
        const int64_t tiles_now = (int64_t)bps * samples, at_once = 2 * (int64_t)n_cu / bps * bps;
        return at_once > 0 && plan_group_slab(p, n_cu, samples, hw, C, tiles_now, bps, (tiles_now + at_once - 1) / at_once);
    };
    const bool slabs_may = forced_variant != PF_VARIANT_GROUP_TWO_PASS && L.n_full == 1 && g.vec_per_channel && L.pro.n == 1 && L.pro.u[0].code == pf::U_MOV && L.pro.u[0].kind == pf::K_FULL;
    uint32_t bps_of_12;
    tiling(12, &bps_of_12);
    const bool tiles_settled = nv != 16 || p->spec_id != 0 || bps_of_12 <= 2u * (uint32_t)n_cu;
    if (slabs_may && tiles_settled && try_slabs()) return PF_OK;
    // resident variant: catalogue entry, one full operand, per-channel broadcast operands only, and a grid the
    // device holds at once
    const bool jit_ok = p->spec_id == 0 && jit_possible(p->device);
    pf::JitSpec jspec = make_jit_spec(L);
    if (p->stats_only && L.main_dtype != PF_F32) jspec.flags |= 32;
    std::string jit_err;
    hipFunction_t fused_fn = nullptr;
    bool resident_ok = L.n_full == 1 && g.vec_per_channel && forced_variant != PF_VARIANT_GROUP_TWO_PASS;
    if (resident_ok && p->spec_id == 0) {
        // not in the catalogue: the fused kernel exists only if it can be specialised now
        fused_fn = jit_ok ? pf::jit_group_kernel(p->device, L.main_dtype, nv, 0, gen_parts, jspec, &jit_err) : nullptr;
        if (fused_fn && nv == 16 && !forced_nv && pf::jit_scratch_bytes(fused_fn) > 0) {
            // The kernel of 16 vectors per lane does not fit the registers for this chain: what it spills goes through
            // memory once per workgroup (measured on [16,64,64,320] with groups of 10: 16 KiB per workgroup, traffic 1.16 x
            // the tensor).  Tiles of 12 steps do fit.
            uint32_t b12;
            tiling(12, &b12);
            hipFunction_t fn12 = pf::jit_group_kernel(p->device, L.main_dtype, 12, 0, gen_parts, jspec, &jit_err);
            if (fn12 && pf::jit_scratch_bytes(fn12) == 0) {
                fused_fn = fn12;
                nv = 12;
                bps = b12;
            }
        }
        if (!fused_fn) resident_ok = false;
    }
    if (slabs_may && !tiles_settled && resident_ok && try_slabs()) return PF_OK;
    const uint64_t tiles = (uint64_t)bps * samples;
    if (tiles > 0x7fffffffull) return fail(PF_ERR_UNSUPPORTED, "tensor too large for the group family");
    uint32_t res_grid = 0;
    if (resident_ok) {
        const int per_cu = fused_fn ? pf::jit_blocks_per_cu(fused_fn, (int)threads, gen_lds)
                                    : pf::group_resident_blocks_per_cu(p->spec_id, L.main_dtype, nv, (int)threads);
        const uint64_t cap = (uint64_t)std::max(per_cu, 0) * n_cu;
        uint64_t grid = std::min<uint64_t>(tiles, cap);
        grid = grid / bps * bps;  // whole samples per round, so every wait is for co-resident workgroups
        if (grid < bps) resident_ok = false;
        else res_grid = (uint32_t)grid;
    }
    int variant = forced_variant >= 0 ? forced_variant : (resident_ok ? PF_VARIANT_GROUP_RESIDENT : PF_VARIANT_GROUP_TWO_PASS);
    if (variant == PF_VARIANT_GROUP_RESIDENT && !resident_ok)
        return fail(PF_ERR_UNSUPPORTED, "the register-resident variant is not available for this chain or shape");
    if (variant != PF_VARIANT_GROUP_RESIDENT && variant != PF_VARIANT_GROUP_TWO_PASS)
        return fail(PF_ERR_UNSUPPORTED, "unknown group variant %d", variant);
    p->variant = variant;
    p->block = dim3(threads);
    g.pos_per_block = (uint32_t)nv * g.pos_per_step;
    g.blocks_per_sample = bps;
    p->k = nv;
    if (variant == PF_VARIANT_GROUP_RESIDENT) {
        p->grid = dim3(res_grid);
        p->n_launches = 1;
        if (fused_fn) {
            p->jit_fn = fused_fn;
            p->spec_id = pf::kSpecJit;
        }
        // tensors of 4 MB and more: the kernel compiled for this geometry (see the kernel's header)
        const int const_mode = env_int("PF_GROUP_CONST", 1);
        if (!general && jit_possible(p->device) && const_mode != 0 && (const_mode == 2 || samples * hw * C * es >= (4 << 20))) {
            std::string err;
            hipFunction_t fn = pf::jit_group_kernel_const(p->device, L.main_dtype, nv, gen_parts, jspec, g, (uint32_t)tiles, res_grid, threads, &err);
            if (fn && pf::jit_blocks_per_cu(fn, (int)threads, gen_lds) * n_cu >= (int)res_grid) {
                p->jit_fn = fn;
                p->spec_id = pf::kSpecJit;
            }
        }
    } else {
        p->grid = dim3((uint32_t)tiles);
        p->grid2 = p->grid;
        p->block2 = p->block;
        p->n_launches = p->stats_only ? 1 : 2;
        if (jit_ok) {
            p->jit_fn = pf::jit_group_kernel(p->device, L.main_dtype, nv, 1, gen_parts, jspec, &jit_err);
            if (p->jit_fn && !p->stats_only) p->jit_fn2 = pf::jit_group_kernel(p->device, L.main_dtype, nv, 2, gen_parts, jspec, &jit_err);
            if (p->jit_fn && (p->jit_fn2 || p->stats_only)) p->spec_id = pf::kSpecJit;
        }
        // (tiles of 12 steps exist in plan-time specialised form only)
        if (nv == 12 && p->spec_id != pf::kSpecJit) return fail(PF_ERR_UNSUPPORTED, "plan-time specialisation failed for the two-launch kernels: %s", jit_err.c_str());
    }
    if (jit_ok && p->spec_id == 0) note_interpreter_fallback(p, jit_err);
    p->lds_bytes = general ? gen_lds + 512 * 2 * 4 + 4 : 512 * 3 * 4 + 512 * 2 * 4 + 4;
    p->dyn_lds = gen_lds;
    // workspace: partials of the two-launch variant, or two parities of exchange words (all-ones = empty) of the
    // resident one; then the error word
    const uint64_t part_bytes = variant == PF_VARIANT_GROUP_RESIDENT ? 0 : (uint64_t)samples * g.blocks_per_sample * g.groups * 4 * sizeof(float);
    const uint64_t gather_bytes =
        variant == PF_VARIANT_GROUP_RESIDENT ? (((uint64_t)2 * samples * g.groups * g.blocks_per_sample * sizeof(uint64_t)) + 255) / 256 * 256 : 0;
    pf_status ws_st = plan_workspace_alloc(p, part_bytes + gather_bytes + 256, "workspace allocation");
    if (ws_st != PF_OK) return ws_st;
    char* ws = static_cast<char*>(p->workspace);
    if ((ws_st = plan_workspace_fill(p, ws, 0, part_bytes, false)) != PF_OK) return ws_st;
    if ((ws_st = plan_workspace_fill(p, ws + part_bytes, 0xff, gather_bytes, true)) != PF_OK) return ws_st;
    if ((ws_st = plan_workspace_fill(p, ws + part_bytes + gather_bytes, 0, 256, true)) != PF_OK) return ws_st;
    g.ws_partial = part_bytes ? reinterpret_cast<float*>(ws) : nullptr;
    g.ws_gather = gather_bytes ? reinterpret_cast<uint64_t*>(ws + part_bytes) : nullptr;
    g.ws_error = reinterpret_cast<uint32_t*>(ws + part_bytes + gather_bytes);
    p->args.n_inner = (uint32_t)C;
    p->args.rows = (uint64_t)(samples * hw);
    return PF_OK;
}

// ---- stencil family
pf_status plan_stencil(pf_plan_s* p, const Checked& c, int forced_variant) {
    const Lowered& L = p->low;
    const int es = dtype_size(L.main_dtype);
    const int vec = 16 / es;
    const Shape& xs = L.pre_shape;  // [n, h, w, c]
    const Shape& ks = c.shape[p->desc.ops[L.core_op].src[1]];
    if (ks[0] != ks[1] || (ks[0] != 3 && ks[0] != 5))
        return fail(PF_ERR_UNSUPPORTED, "dwconv2d: 3 x 3 and 5 x 5 kernels are implemented (got %lld x %lld)", (long long)ks[0], (long long)ks[1]);
    const int ksz = (int)ks[0];
    const int out_rows = ksz == 3 ? kStencilRowsHost : kStencilRows5Host;
    const int64_t n = xs[0], h = xs[1], w = xs[2], ch = xs[3];
    // a channel count that is not a whole number of vectors: element-aligned positions, a partial last vector
    const bool ragged_c = (ch * es) % 16 != 0;
    if (p->ragged && !ragged_c) return fail(PF_ERR_ALIGNMENT, "a broadcast input of the stencil family is not a multiple of 16 bytes");
    if (n * h * w > 0xffffffffLL || n > 65535 || (h + out_rows - 1) / out_rows > 65535) return fail(PF_ERR_UNSUPPORTED, "tensor too large for the stencil family");
    if (L.n_out != 1) return fail(PF_ERR_UNSUPPORTED, "secondary outputs are not implemented in the stencil family");
    for (int i = 0; i < L.pro.n; ++i)
        if (L.pro.u[i].code == pf::U_MASK_CAUSAL) return fail(PF_ERR_UNSUPPORTED, "causal_mask next to a convolution is not implemented");
    for (int i = 0; i < L.epi.n; ++i)
        if (L.epi.u[i].code == pf::U_MASK_CAUSAL) return fail(PF_ERR_UNSUPPORTED, "causal_mask next to a convolution is not implemented");
    pf::StencilGeom& g = p->stencil;
    memset(&g, 0, sizeof(g));
    g.n = (uint32_t)n;
    g.h = (uint32_t)h;
    g.w = (uint32_t)w;
    g.c = (uint32_t)ch;
    g.cv = (uint32_t)((ch + vec - 1) / vec);
    g.ragged = ragged_c ? 1u : 0u;
    g.row_vecs = (uint32_t)(w * g.cv);
    g.div_cv = make_fastdiv(g.cv);
    for (int f = 0; f < L.n_full; ++f)
        if (L.full_is_epi[f]) g.epi_full_mask |= 1u << f;
    for (int v = 0; v < L.n_vec; ++v)
        if (L.vec_is_epi[v]) g.epi_vec_mask |= 1u << v;
    p->family = PF_FAMILY_STENCIL;
    p->k = 1;
    p->spec_id = 0;
    p->block = dim3(256);
    p->grid = dim3((g.row_vecs + 255u) / 256u, (uint32_t)((h + out_rows - 1) / out_rows), (uint32_t)n);
    p->n_launches = 1;
    p->stencil_ks = ksz;
    p->args.n_inner = (uint32_t)ch;
    p->args.rows = (uint64_t)(n * h * w);
    // broadcast operands indexed by channel alone (a bias) are loaded once per lane, not once per position
    pf::JitSpec jspec = make_jit_spec(L);
    bool by_channel = true;
    for (int v = 0; v < L.n_vec; ++v)
        if (v != L.core_vec[0] && (p->args.vec[v].numel > (uint32_t)ch || p->args.vec[v].n_terms != 0)) by_channel = false;
    if (by_channel) jspec.flags |= 4;
    const pf_op_desc& conv = p->desc.ops[L.core_op];
    const int64_t stride = conv.n_i == 1 ? conv.i[0] : 1;
    if (stride > 1) {
        // down-sampling convolution: one lane per output column and channel vector, taps loaded where they are used
        if (forced_variant >= 0 && forced_variant != PF_VARIANT_STENCIL_STRIDED)
            return fail(PF_ERR_UNSUPPORTED, "a strided convolution runs on the strided variant only");
        const int64_t oh = (h - 1) / stride + 1, ow = (w - 1) / stride + 1;
        g.stride = (uint32_t)stride;
        g.oh = (uint32_t)oh;
        g.ow = (uint32_t)ow;
        g.out_row_vecs = (uint32_t)(ow * g.cv);
        // output rows per workgroup: 4 (the kernel vectors are loaded once per workgroup), fewer while that leaves
        // a compute unit with less than about eight workgroups
        hipDeviceProp_t prop;
        const int n_cu = (hipGetDeviceProperties(&prop, p->device) == hipSuccess && prop.multiProcessorCount > 0) ? prop.multiProcessorCount : 256;
        const int64_t tiles_x = (g.out_row_vecs + 255) / 256;
        int64_t strip = 4;
        while (strip > 1 && tiles_x * ((oh + strip - 1) / strip) * n < 8 * (int64_t)n_cu) strip /= 2;
        g.strip_rows = (uint32_t)strip;
        if ((oh + strip - 1) / strip > 65535) return fail(PF_ERR_UNSUPPORTED, "tensor too large for the stencil family");
        p->variant = PF_VARIANT_STENCIL_STRIDED;
        p->lds_bytes = 0;
        p->grid = dim3((uint32_t)tiles_x, (uint32_t)((oh + strip - 1) / strip), (uint32_t)n);
        if (jit_possible(p->device)) {
            std::string err;
            p->jit_fn = pf::jit_stencil_kernel(p->device, L.main_dtype, p->variant, ksz, ragged_c, jspec, &err);
            if (p->jit_fn) p->spec_id = pf::kSpecJit;
            else note_interpreter_fallback(p, err);
        }
        return PF_OK;
    }
    if (forced_variant == PF_VARIANT_STENCIL_STRIDED) return fail(PF_ERR_UNSUPPORTED, "the strided variant is for strides above 1");
    // Staged variant (values activated once, shared through an LDS tile) when the tile fits; its entries are
    // packed in the storage type if the prologue keeps storage precision and the kernel is specialised.
    const bool jit_ok = jit_possible(p->device);
    bool exact_pro = L.main_dtype != PF_F32 && L.pro.n >= 1 && L.pro.u[0].code == pf::U_MOV && L.pro.u[0].kind == pf::K_FULL;
    for (int i = 1; i < L.pro.n; ++i)
        if (L.pro.u[i].code != pf::U_RELU && L.pro.u[i].code != pf::U_NEG) exact_pro = false;
    const uint32_t entry_bytes = (L.main_dtype == PF_F32 || (exact_pro && jit_ok)) ? 16u : 32u;
    const uint64_t tile_bytes = (uint64_t)(out_rows + ksz - 1) * (256u + 2u * (uint32_t)(ksz / 2) * g.cv) * entry_bytes;
    // per workgroup: 64 KB everywhere; up to 96 KB where the device offers 160 KB (gfx950), which still leaves
    // room for a second, smaller workgroup on the compute unit
    uint64_t lds_limit = 64 * 1024;
    {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, p->device) == hipSuccess && prop.sharedMemPerBlock >= 160 * 1024) lds_limit = 96 * 1024;
    }
    const bool staged_ok = tile_bytes <= lds_limit;
    int variant = forced_variant >= 0 ? forced_variant : (staged_ok ? PF_VARIANT_STENCIL_STAGED : PF_VARIANT_STENCIL_DIRECT);
    if (variant == PF_VARIANT_STENCIL_DIRECT && ksz != 3)
        return fail(PF_ERR_UNSUPPORTED, "5 x 5 kernels need the staged variant, whose LDS tile (%llu bytes) does not fit here", (unsigned long long)tile_bytes);
    if (variant != PF_VARIANT_STENCIL_STAGED && variant != PF_VARIANT_STENCIL_DIRECT) return fail(PF_ERR_UNSUPPORTED, "unknown stencil variant %d", variant);
    if (variant == PF_VARIANT_STENCIL_STAGED && !staged_ok)
        return fail(PF_ERR_UNSUPPORTED, "the staged variant needs an LDS tile of %llu bytes (limit %llu)", (unsigned long long)tile_bytes,
                    (unsigned long long)lds_limit);
    p->variant = variant;
    p->lds_bytes = variant == PF_VARIANT_STENCIL_STAGED ? (uint32_t)tile_bytes : 0u;
    if (variant == PF_VARIANT_STENCIL_STAGED) {
        // one-dimensional grid, tiles numbered so that neighbours share a compute die's L2
        g.tiles_x = p->grid.x;
        g.tiles_y = p->grid.y;
        const uint64_t tiles = (uint64_t)p->grid.x * p->grid.y * p->grid.z;
        if (tiles > 0x7ffffff0ull) return fail(PF_ERR_UNSUPPORTED, "tensor too large for the stencil family");
        g.tiles = (uint32_t)tiles;
        g.tiles_per_die = (uint32_t)((tiles + 7) / 8);
        p->grid = dim3(g.tiles_per_die * 8u);
    }
    if (jit_ok) {
        std::string err;
        if (variant == PF_VARIANT_STENCIL_DIRECT) jspec.flags &= ~4;  // (loads its operands at every position)
        // A launch that leaves compute units idle: registers do not limit what is resident.  Read by the 5 x 5 kernels that widen
        // 16-bit values alone (others would be compiled twice).
        if (ksz == 5 && L.main_dtype != PF_F32 && !(exact_pro && L.main_dtype == PF_F16)) {
            hipDeviceProp_t prop;
            if (hipGetDeviceProperties(&prop, p->device) == hipSuccess && (uint64_t)g.tiles <= (uint64_t)prop.multiProcessorCount) jspec.flags |= 8;
        }
        p->jit_fn = pf::jit_stencil_kernel(p->device, L.main_dtype, variant, ksz, ragged_c, jspec, &err);
        if (p->jit_fn) p->spec_id = pf::kSpecJit;
        else {
            note_interpreter_fallback(p, err);
            // the interpreted kernel never packs its tile
            if (variant == PF_VARIANT_STENCIL_STAGED && entry_bytes == 16u && L.main_dtype != PF_F32) {
                const uint64_t big = tile_bytes * 2;
                if (big > lds_limit && ksz != 3) return fail(PF_ERR_UNSUPPORTED, "5 x 5 kernels need the staged variant, whose LDS tile does not fit here");
                if (big > lds_limit) {
                    p->variant = PF_VARIANT_STENCIL_DIRECT;
                    p->lds_bytes = 0;
                    p->grid = dim3(g.tiles_x, g.tiles_y, (uint32_t)n);
                } else {
                    p->lds_bytes = (uint32_t)big;
                }
            }
        }
    }
    return PF_OK;
}

// ---- gather family
int64_t gcd64(int64_t a, int64_t b) {
    while (b != 0) {
        const int64_t t = a % b;
        a = b;
        b = t;
    }
    return a;
}

// Where element `e` (flat index) of value `v` comes from: walks the operators backwards to a chain input.
void gather_source(const pf_chain_desc* d, const Checked& c, int v, int64_t e, int* in_id, int64_t* in_flat) {
    const int n_in = d->n_inputs;
    while (v >= n_in) {
        const pf_op_desc& o = d->ops[v - n_in];
        const Shape& os = c.shape[v];
        const int rank = (int)os.size();
        if (o.op == PF_RESHAPE) {
            v = o.src[0];
            continue;
        }
        int64_t idx[PF_MAX_RANK];
        int64_t rem = e;
        for (int q = rank - 1; q >= 0; --q) {
            idx[q] = rem % os[q];
            rem /= os[q];
        }
        int src = o.src[0];
        int64_t sidx[PF_MAX_RANK];
        if (o.op == PF_PERMUTE) {
            for (int q = 0; q < rank; ++q) sidx[o.i[q]] = idx[q];
        } else if (o.op == PF_SLICE) {
            for (int q = 0; q < rank; ++q) sidx[q] = idx[q];
            sidx[o.i[0]] += o.i[1];
        } else {  // PF_CONCAT
            for (int q = 0; q < rank; ++q) sidx[q] = idx[q];
            const int64_t first = c.shape[o.src[0]][o.i[0]];
            if (idx[o.i[0]] >= first) {
                src = o.src[1];
                sidx[o.i[0]] -= first;
            }
        }
        const Shape& ss = c.shape[src];
        int64_t flat = 0;
        for (int q = 0; q < rank; ++q) flat = flat * ss[q] + sidx[q];
        e = flat;
        v = src;
    }
    *in_id = v;
    *in_flat = e;
}

pf_status plan_gather(pf_plan_s* p, const Checked& c) {
    const pf_chain_desc* d = &p->desc;
    const Lowered& L = p->low;
    const int es = dtype_size(L.main_dtype);
    const int vec = 16 / es;
    const int n_in = d->n_inputs;
    // Run length: for every value, a length G such that each aligned block of G elements (flat, row-major)
    // is contiguous inside one chain input.  0 stands for "the whole tensor" (gcd(0, x) = x).
    std::vector<int64_t> G(n_in + d->n_ops, 0);
    for (int k = 0; k < d->n_ops; ++k) {
        const pf_op_desc& o = d->ops[k];
        const int v = n_in + k;
        const Shape& os = c.shape[v];
        const int rank = (int)os.size();
        int64_t g = G[o.src[0]] ? G[o.src[0]] : numel(c.shape[o.src[0]]);
        if (o.op == PF_PERMUTE) {
            int64_t inner = 1;
            for (int q = rank - 1; q >= 0 && o.i[q] == q; --q) inner *= os[q];
            g = gcd64(g, inner);
        } else if (o.op == PF_SLICE) {
            int64_t inner = 1;
            for (int q = (int)o.i[0] + 1; q < rank; ++q) inner *= os[q];
            g = gcd64(gcd64(g, o.i[2] * inner), gcd64(o.i[1] * inner, c.shape[o.src[0]][o.i[0]] * inner));
        } else if (o.op == PF_CONCAT) {
            int64_t inner = 1;
            for (int q = (int)o.i[0] + 1; q < rank; ++q) inner *= os[q];
            const int64_t g1 = G[o.src[1]] ? G[o.src[1]] : numel(c.shape[o.src[1]]);
            g = gcd64(gcd64(g, g1), gcd64(c.shape[o.src[0]][o.i[0]] * inner, c.shape[o.src[1]][o.i[0]] * inner));
        }
        G[v] = g;
    }
    int64_t run = 0, total = 0;
    for (int o = 0; o < d->n_outputs; ++o) {
        const int v = d->out_value[o];
        run = gcd64(run, G[v] ? G[v] : numel(c.shape[v]));
        total += numel(c.shape[v]);
    }
    for (int k = 0; k < n_in; ++k)
        if (numel(c.shape[k]) > 0xffffffffLL) return fail(PF_ERR_UNSUPPORTED, "tensor too large for the gather family");
    if (total > 0xffffffffLL) return fail(PF_ERR_UNSUPPORTED, "tensor too large for the gather family");
    // very long runs are cut so that the copy has enough workgroups; cuts keep whole vectors
    while (run > 65536 && run % 2 == 0 && (run / 2) % vec == 0) run /= 2;
    const int64_t n_runs = total / run;
    if (n_runs > (1 << 22))
        return fail(PF_ERR_UNSUPPORTED, "layout chain moves runs of only %lld elements: %lld runs exceed the run table", (long long)run, (long long)n_runs);
    std::vector<pf::GatherRun> table((size_t)n_runs);
    size_t at = 0;
    for (int o = 0; o < d->n_outputs; ++o) {
        const int v = d->out_value[o];
        const int64_t n = numel(c.shape[v]);
        for (int64_t e = 0; e < n; e += run) {
            int in_id;
            int64_t in_flat;
            gather_source(d, c, v, e, &in_id, &in_flat);
            pf::GatherRun& r = table[at++];
            r.src_off = (uint32_t)in_flat;
            r.dst_off = (uint32_t)e;
            r.src_id = (uint8_t)in_id;
            r.dst_id = (uint8_t)o;
            r.pad = 0;
        }
    }
    if (planning_static())
        return fail(PF_ERR_UNSUPPORTED, "layout-only chains with concat / slice need a run table in device memory: use pf_chain_plan + pf_chain_run");
    if (hipSetDevice(p->device) != hipSuccess) return fail(PF_ERR_HIP, "cannot select device %d", p->device);
    p->workspace_bytes = (uint64_t)n_runs * sizeof(pf::GatherRun);
    if (hipMalloc(&p->workspace, p->workspace_bytes) != hipSuccess) return fail(PF_ERR_NOMEM, "run table allocation of %llu bytes failed", (unsigned long long)p->workspace_bytes);
    if (hipMemcpy(p->workspace, table.data(), p->workspace_bytes, hipMemcpyHostToDevice) != hipSuccess) return fail(PF_ERR_HIP, "run table upload failed");
    pf::GatherArgs& a = p->gather;
    memset(&a, 0, sizeof(a));
    a.table = static_cast<const pf::GatherRun*>(p->workspace);
    a.n_runs = (uint32_t)n_runs;
    a.run_elems = (uint32_t)run;
    a.vec_per_run = (uint32_t)((run + vec - 1) / vec);
    a.div_vpr = make_fastdiv(a.vec_per_run);
    const uint64_t work = (uint64_t)n_runs * a.vec_per_run;
    if (work > 0x7fffffffull) return fail(PF_ERR_UNSUPPORTED, "tensor too large for the gather family");
    p->family = PF_FAMILY_GATHER;
    p->variant = 0;
    // vectors per lane: two once every compute unit still gets a dozen workgroups (concat -> channel shuffle -> split
    // of [128, 232, 28, 28] fp16: one 19.8 us, two 17.6 us, four 18.1 us)
    int k = work >= (uint64_t)2 * 256 * 4096 ? 2 : 1;
    const int forced_k = env_int("PF_GATHER_K", 0);
    if (forced_k == 1 || forced_k == 2 || forced_k == 4) k = forced_k;
    p->k = k;
    p->spec_id = 0;
    p->block = dim3(256);
    p->grid = dim3((uint32_t)((work + 256 * (uint64_t)k - 1) / (256 * (uint64_t)k)));
    p->lds_bytes = 0;
    p->n_launches = 1;
    return PF_OK;
}

// ---- attention family
// ---- pool family
// A pooling with a normalisation in front in one launch, statistics included (p->pool: extents filled in); false where that is
// not possible or not quicker.
static bool plan_norm_pool_slab(pf_plan_s* p, int n_cu) {
    const Lowered& L = p->low;
    if (!jit_possible(p->device) || env_int("PF_NORM_POOL_SLAB", 1) == 0) return false;
    // the load, the normalisation, then steps without tensor operands (each would be read once a position)
    if (L.pro.n < 2 || L.pro.u[0].code != pf::U_MOV || L.pro.u[0].kind != pf::K_FULL || L.pro.u[1].code != pf::U_GNORM) return false;
    for (int i = 2; i < L.pro.n; ++i)
        if (L.pro.u[i].kind == pf::K_FULL || L.pro.u[i].kind == pf::K_VEC) return false;
    if (L.core_vec[0] < 0 || L.core_vec[1] < 0 || p->pool.ragged) return false;
    const int64_t n = p->pool.samples, hw = p->pool.hw, ch = p->pool.channels, groups = L.groups, cpg = ch / groups;
    const int es = dtype_size(L.main_dtype), vec = 16 / es;
    if (hw * ch * es > 0x7fffffffLL) return false;
    // Groups per slab: what a model of the launch finds quickest (microseconds, measured: 9, then 0.87 a step of one workgroup to
    // a unit, 1.8 of two), among slabs of at least four vectors that fit the registers -- 44 vectors a lane one workgroup to a unit,
    // 16 two -- and are enough to fill three quarters of the device.  Taken where the same model of the two launches (10.5 and
    // 1.0 a step of all positions) is 2 us behind: [32, 64, 64, 320] fp16 44.6 against 48.9, [31, 16, 16, 1152] 16.1 against 22.5; not
    // [13, 50, 50, 576], slabs of 18 channels in 24, 37.1 against 29.9.
    const bool forced = env_int("PF_NORM_POOL_SLAB", 1) == 2;  // (wherever it is possible)
    const int64_t cv = ch / vec;
    int64_t best_d = 0, best_cvs = 0, best_nv = 0;
    double best = 8.5 + (double)(n * ((hw + 512 / cv - 1) / (512 / cv))) / (double)n_cu;
    for (int64_t d = 1; d <= groups && d <= 512; ++d) {
        if (groups % d != 0) continue;
        const int64_t slabs = n * (groups / d), sc = d * cpg;
        if ((slabs * 4 < (int64_t)n_cu * 3 && !forced) || slabs > 0x7fffff) continue;
        int64_t cvs = 0;
        for (int64_t lo = 0; lo < ch; lo += sc) cvs = std::max(cvs, (lo + sc - 1) / vec - lo / vec + 1);
        if (cvs * vec > 512 || (cvs < 4 && !forced)) continue;
        const int64_t pps = 512 / cvs, nv = (hw + pps - 1) / pps;
        if (nv > 44) continue;
        const int64_t per_cu = nv > 16 ? 1 : 2;
        const int64_t rounds = (slabs + per_cu * n_cu - 1) / (per_cu * n_cu);
        const double cost = 9.0 + (double)(rounds * nv) * (per_cu == 2 && slabs > n_cu ? 1.8 : 0.87);
        if (cost < best || (forced && best_d == 0)) best = cost, best_d = d, best_cvs = cvs, best_nv = nv;
    }
    // 16-bit tensors of more than 2 MiB: slabs that leave units idle as well, at most one to a unit, where a model of that launch is 8 %
    // ahead of the two launches' (fitted to 270 measured slabs of 26 shapes, 5 % off in the mean; [13, 50, 50, 576] bf16 30.8 in one launch, 28.3
    // in two, 7 % ahead by the models).  us, fp16 or bf16, before and
    // now: [21, 28, 28, 64] 13.7 -> 8.8, [19, 14, 14, 576] 13.3 -> 9.3, [28, 18, 18, 416] 15.4 -> 10.6, [23, 32, 32, 992] 39.5 -> 32.0, [8, 56, 56,
    // 256] 18.0 -> 14.0.  Smaller tensors would gain as well ([1, 7, 7, 128] 9.8, 8.7 in one launch); tests/test_norm_pool_gpu.py states two
    // launches for them.  (Slices of a slab that exchange their statistics gain more where slabs are few -- [4, 64, 64, 672] 25.7 -> 20.8 -- but all
    // workgroups of a launch then wait for one another: two such launches on two streams, each with half of the units, would wait in vain,
    // dispatched as they were; in runs of slabs, as the slices of the group family are now, they were not tried.)
    if (!forced && es == 2 && n * hw * ch * es > (2 << 20)) {
        const double mb = (double)(n * hw * ch * es) * 1e-6;
        double least = 0.92 * (12.4 - 0.37 * (double)(n * ((hw + 512 / cv - 1) / (512 / cv))) / (double)n_cu + 0.68 * mb);
        for (int64_t d = 1; d <= groups && d <= 512; ++d) {
            if (groups % d != 0) continue;
            const int64_t slabs = n * (groups / d), sc = d * cpg, bytes = sc * es;
            int64_t cvs = 0;
            for (int64_t lo = 0; lo < ch; lo += sc) cvs = std::max(cvs, (lo + sc - 1) / vec - lo / vec + 1);
            if (cvs * vec > 512 || slabs > n_cu) continue;
            const int64_t pps = 512 / cvs, nv = (hw + pps - 1) / pps;
            if (nv > 44) continue;
            const bool lines = (bytes % 128 == 0 && (ch * es) % 128 == 0) || d == groups;
            const double waste = lines ? 0.0 : std::min(3.0, 112.0 / (double)bytes);  // (of the memory lines a position's share touches)
            const double us = 5.8 + mb * (0.082 + 0.05 * waste) + 0.66 * (double)nv + 0.15 * std::log2((double)pps);
            if (us < least) least = us, best_d = d, best_cvs = cvs, best_nv = nv;
        }
    }
    if (best_d == 0) return false;
    pf::SlabGeom g;
    memset(&g, 0, sizeof(g));
    g.hw = (uint32_t)hw;
    g.channels = (uint32_t)ch;
    g.cpg = (uint32_t)cpg;
    g.div_cpg = make_fastdiv(g.cpg);
    g.slab_groups = (uint32_t)best_d;
    g.slabs_per_sample = (uint32_t)(groups / best_d);
    g.slabs = (uint32_t)(n * g.slabs_per_sample);
    g.slabs_per_die = (g.slabs + 7u) / 8u;
    g.inv_hw = 1.0f / (float)hw;
    g.parts = 1;
    for (int64_t v = 0; v < ch / vec; ++v) g.parts = std::max<uint32_t>(g.parts, (uint32_t)((v * vec + vec - 1) / cpg - v * vec / cpg + 1));
    while (g.log2_lanes < 6u && (best_d << (g.log2_lanes + 1)) <= 512) ++g.log2_lanes;
    pf::JitSpec jspec = make_jit_spec(L);
    if (L.main_dtype != PF_F32) jspec.flags |= 32;
    std::string err;
    hipFunction_t fn = pf::jit_norm_pool_slab_kernel(p->device, L.main_dtype, (int)best_nv, (int)best_cvs, L.pool_op, jspec, &err);
    if (!fn || pf::jit_scratch_bytes(fn) != 0) return false;
    p->jit_fn = fn;
    p->pool_slab = true;
    p->slab = g;
    p->k = (int)best_nv;
    p->grid = dim3(g.slabs_per_die * 8u);
    p->dyn_lds = 512u * std::max<uint32_t>(3u * g.parts, (uint32_t)vec) * 4u;
    p->lds_bytes = p->dyn_lds + 2 * 512 * 4;
    p->family = PF_FAMILY_POOL;
    p->variant = 0;
    p->spec_id = pf::kSpecJit;
    p->block = dim3(512);
    p->n_launches = 1;
    p->args.n_inner = (uint32_t)ch;
    p->args.rows = (uint64_t)(n * hw);
    return true;
}

pf_status plan_pool(pf_plan_s* p) {
    const Lowered& L = p->low;
    const int es = dtype_size(L.main_dtype);
    const int vec = 16 / es;
    const Shape& xs = L.pre_shape;  // [n, spatial.., c]
    const int64_t n = xs[0], ch = xs.back();
    const int64_t hw = numel(xs) / (n * ch);
    // a channel count that is not a whole number of vectors: element-aligned positions, a partial last vector
    const bool ragged_c = (ch * es) % 16 != 0;
    if (p->ragged && !ragged_c) return fail(PF_ERR_ALIGNMENT, "a broadcast input of the pool family is not a multiple of 16 bytes");
    const int64_t cv = (ch + vec - 1) / vec;
    if (cv > 512) return fail(PF_ERR_UNSUPPORTED, "more than %d channels", 512 * vec);
    if (n * hw > 0xffffffffLL || n > 0x7fffffLL) return fail(PF_ERR_UNSUPPORTED, "tensor too large for the pool family");
    if (L.n_out != 1) return fail(PF_ERR_UNSUPPORTED, "secondary outputs are not implemented in the pool family");
    if (L.n_full < 1 || L.full_is_epi[0]) return fail(PF_ERR_UNSUPPORTED, "the pooled value must start from a full-shape input");
    for (int i = 0; i < L.pro.n; ++i)
        if (L.pro.u[i].code == pf::U_MASK_CAUSAL) return fail(PF_ERR_UNSUPPORTED, "causal_mask in front of a pooling is not implemented");
    for (int i = 0; i < L.epi.n; ++i)
        if (L.epi.u[i].code == pf::U_MASK_CAUSAL) return fail(PF_ERR_UNSUPPORTED, "causal_mask behind a pooling is not implemented");
    hipDeviceProp_t prop;
    const int n_cu = (hipGetDeviceProperties(&prop, p->device) == hipSuccess && prop.multiProcessorCount > 0) ? prop.multiProcessorCount : 256;
    pf::PoolGeom& g = p->pool;
    memset(&g, 0, sizeof(g));
    g.samples = (uint32_t)n;
    g.hw = (uint32_t)hw;
    g.channels = (uint32_t)ch;
    g.ragged = ragged_c ? 1u : 0u;
    g.inv_hw = 1.0f / (float)hw;
    for (int f = 0; f < L.n_full; ++f)
        if (L.full_is_epi[f]) g.epi_full_mask |= 1u << f;
    for (int v = 0; v < L.n_vec; ++v)
        if (L.vec_is_epi[v]) g.epi_vec_mask |= 1u << v;
    if (L.norm_op >= 0 && plan_norm_pool_slab(p, n_cu)) return PF_OK;
    // Channel slabs and slices of the positions: the pair that a model of the launch finds quickest, in steps of a workgroup
    // (with two to a unit 0.4 us for a plain pooling, 1.0 behind a normalisation).  A round of workgroups waits for its first
    // bytes (four steps) and works off its own; several slices add an exchange and its trips of eight words a lane (four
    // each).  One workgroup to a unit instead of two was tried in the model and loses ([32, 56, 56, 240] fp16 14.4 against 12.0).
    // A slab that does not begin and end with a memory line shares its first and last one with its neighbours, which run on
    // other dies: a step then costs 14 vectors more, unless the launch leaves units idle and waits for latencies alone.  us, with
    // one slab per 512 channels, with slabs that cost nothing, now: [103, 23, 23, 280] fp16 9.7 12.1 9.2, [6, 64, 64, 112] fp32
    // 6.7 8.2 6.6, [109, 28, 28, 1072] fp16 + residual, SiLU 76 87 70.
    // Positions at element alignment: a load is behind the branch for the tensor's last vector and waits for the one before, so a
    // step is a trip to memory (three of the others), and four workgroups to a unit cover more of them than two.  us, the same
    // three: [64, 28, 28, 331] fp16 13.0 18.4 11.6, [30, 81, 81, 251] fp16 24.5 29.2 24.0.  (Neither behind a normalisation, whose
    // statistics every workgroup merges first, nor where there are no four steps to a unit.)
    const int64_t min_slabs = (cv * vec + 511) / 512;
    const int64_t whole_pps = std::max<int64_t>(1, 512 / cv);
    const bool serial = ragged_c && L.norm_op < 0 && n * ((hw + whole_pps - 1) / whole_pps) > 4 * (int64_t)n_cu;
    const int64_t resident = (serial ? 4 : 2) * (int64_t)n_cu;
    const double step_cost = serial ? 3.0 : 1.0, first_cost = serial ? 8.0 : 4.0, shared_vecs = L.norm_op >= 0 ? 0.0 : ragged_c ? 10.0 : 14.0;
    double best_cost = 0.0;
    int64_t best_slabs = 0, best_spb = 0;
    for (int64_t slabs = min_slabs; slabs <= std::max<int64_t>(min_slabs, cv / 8); ++slabs) {
        const int64_t scv = (cv + slabs - 1) / slabs;
        if ((cv + scv - 1) / scv != slabs) continue;
        const int64_t pps = 512 / scv, steps = (hw + pps - 1) / pps, units = n * slabs;
        const int64_t per_trip = 8 * (512 / (scv * vec));
        const int64_t max_slices = planning_static() ? 1 : std::min<int64_t>(33, steps);
        for (int64_t slices = 1; slices <= max_slices; ++slices) {
            const int64_t spb = (steps + slices - 1) / slices;
            if ((steps + spb - 1) / spb != slices) continue;
            const int64_t rounds = (units * slices + resident - 1) / resident;
            const int64_t exchange = slices > 1 ? 1 + (slices - 1 + per_trip - 1) / per_trip : 0;
            // (two workgroups to a unit merge the statistics of a normalisation in front twice: [19, 32, 32, 160] bf16 16.2, 14.4 with one)
            const int64_t twice = L.norm_op >= 0 && units * slices > n_cu ? 3 : 0;
            const bool shares = slabs > 1 && units * slices > n_cu && ((ch * es) % 128 != 0 || scv % 8 != 0);
            const double step = step_cost * (shares ? 1.0 + shared_vecs / (double)scv : 1.0);
            const double cost = (double)rounds * ((double)spb * step + first_cost + (double)twice) + 4.0 * (double)exchange;
            if (best_slabs == 0 || cost < best_cost) best_cost = cost, best_slabs = slabs, best_spb = spb;
        }
    }
    g.slabs = (uint32_t)best_slabs;
    g.cv = (uint32_t)((cv + best_slabs - 1) / best_slabs);
    g.div_cv = make_fastdiv(g.cv);
    g.pos_per_step = 512u / g.cv;
    g.merge_rows = 512u / (g.cv * (uint32_t)vec);
    while (g.log2_lanes < 6u && (2u << g.log2_lanes) <= g.merge_rows) ++g.log2_lanes;
    // chunks of equal length, at most eight steps (four where more than two workgroups share a unit's registers)
    const int64_t best_pps = 512 / g.cv, best_blocks = n * best_slabs * ((hw + best_spb * best_pps - 1) / (best_spb * best_pps));
    const int64_t most = serial && best_blocks > 2 * (int64_t)n_cu ? 4 : 8;
    int64_t chunks = (best_spb + most - 1) / most;
    int nv = (int)((best_spb + chunks - 1) / chunks);
    const int forced_nv = env_int("PF_POOL_NV", 0), forced_chunks = env_int("PF_POOL_CHUNKS", 0);
    auto force = [&]() {
        if (forced_nv == 1 || forced_nv == 2 || forced_nv == 4 || forced_nv == 8) nv = forced_nv, chunks = (best_spb + nv - 1) / nv;
        if (forced_chunks > 0) chunks = forced_chunks;
    };
    force();
    p->spec_id = 0;
    if (jit_possible(p->device)) {
        std::string err;
        pf::JitSpec jspec = make_jit_spec(L);
        if (L.norm_op >= 0 && L.main_dtype != PF_F32) jspec.flags |= 32;
        // (the kernel leaves room for two workgroups to a unit; where its vectors do not fit the registers then, half as many: see
        // the kernel)
        for (;;) {
            p->jit_fn = pf::jit_pool_kernel(p->device, L.main_dtype, nv, L.pool_op, ragged_c, chunks > 1, jspec, &err);
            if (!p->jit_fn || nv == 1 || nv == forced_nv || pf::jit_scratch_bytes(p->jit_fn) == 0) break;
            nv = (nv + 1) / 2;
            chunks = (best_spb + nv - 1) / nv;
        }
        if (p->jit_fn) p->spec_id = pf::kSpecJit;
        else note_interpreter_fallback(p, err);
    }
    if (p->spec_id == 0) {  // interpreted kernels exist for 1, 2, 4 and 8 steps
        nv = best_spb >= 8 ? 8 : best_spb > 2 ? 4 : (int)best_spb;
        chunks = (best_spb + nv - 1) / nv;
        force();
    }
    const int64_t chunk_pos = (int64_t)nv * g.pos_per_step;
    g.pos_per_block = (uint32_t)(chunks * chunk_pos);
    g.blocks_per_sample = (uint32_t)((hw + chunks * chunk_pos - 1) / (chunks * chunk_pos));
    // A static call takes samples that one workgroup is enough for: eight steps of whole positions, or samples of any length where
    // there are four to every compute unit.  (One workgroup on [1, 512, 512, 64] fp16 is 6 ms.)
    if (planning_static() && (g.blocks_per_sample > 1 || (hw > 8 * (512 / cv) && n < 4 * (int64_t)n_cu)))
        return fail(PF_ERR_UNSUPPORTED, "a pooling split over several workgroups per sample waits on the device, and a wait that gives up is reported "
                                        "through the plan: use pf_chain_plan + pf_chain_run");
    const uint64_t blocks = (uint64_t)g.blocks_per_sample * g.slabs * n;
    if (blocks > 0x7fffffffull) return fail(PF_ERR_UNSUPPORTED, "tensor too large for the pool family");
    p->family = PF_FAMILY_POOL;
    p->variant = 0;
    p->k = nv;
    p->block = dim3(512);
    p->grid = dim3((uint32_t)blocks);
    p->lds_bytes = 512 * vec * 4 + 512 * 4;
    p->n_launches = 1;
    p->args.n_inner = (uint32_t)ch;
    p->args.rows = (uint64_t)(n * hw);
    if (g.blocks_per_sample > 1) {
        const uint64_t part_bytes = ((uint64_t)blocks * g.cv * vec * sizeof(float) + 255) / 256 * 256;
        if (hipSetDevice(p->device) != hipSuccess) return fail(PF_ERR_HIP, "cannot select device %d", p->device);
        pf_status ws_st = plan_workspace_alloc(p, part_bytes + 256, "workspace allocation");
        if (ws_st != PF_OK) return ws_st;
        if ((ws_st = plan_workspace_fill(p, p->workspace, 0xff, part_bytes, true)) != PF_OK) return ws_st;
        if ((ws_st = plan_workspace_fill(p, static_cast<char*>(p->workspace) + part_bytes, 0, 256, true)) != PF_OK) return ws_st;
        g.ws_partial = reinterpret_cast<uint32_t*>(p->workspace);
        g.ws_error = reinterpret_cast<uint32_t*>(static_cast<char*>(p->workspace) + part_bytes);
        g.spin_limit = (uint32_t)env_int("PF_POOL_SPIN_LIMIT", 1 << 18);  // re-reads before a wait gives up (tests force it small)
        p->ws_error = g.ws_error;
    }
    if (L.norm_op >= 0) {
        g.norm_groups = (uint32_t)L.groups;
        const int64_t cpg = ch / L.groups, slab_ch = (int64_t)g.cv * vec;
        int64_t grps = 1;  // the most groups a slab touches
        for (int64_t lo = 0; lo < ch; lo += slab_ch) grps = std::max(grps, (std::min(lo + slab_ch, ch) - 1) / cpg - lo / cpg + 1);
        while (g.norm_log2 < 6u && (grps << (g.norm_log2 + 1)) <= 512) ++g.norm_log2;  // (at most: see plan_norm_pool)
        g.div_norm_cpg = make_fastdiv((uint32_t)(ch / L.groups));
    }
    return PF_OK;
}

// ---- column family
pf_status plan_column(pf_plan_s* p) {
    const Lowered& L = p->low;
    const int es = dtype_size(L.main_dtype), vec = 16 / es;
    if (L.col_c > 1024) return fail(PF_ERR_UNSUPPORTED, "normalisation over a strided dimension holds at most 1024 values per position in registers (got %lld)", (long long)L.col_c);
    const int64_t s_vecs = (L.col_s + vec - 1) / vec, tiles = (s_vecs + 7) / 8;
    p->ragged = L.col_s % vec != 0;  // rows at element alignment, partial last vector
    if (L.col_outer * tiles > 0x7fffffffLL || L.col_outer * L.col_c * L.col_s > 0xffffffffLL * 4) return fail(PF_ERR_UNSUPPORTED, "tensor too large for the column family");
    pf::ColArgs& a = p->col;
    memset(&a, 0, sizeof(a));
    a.c = (uint32_t)L.col_c;
    a.s = (uint32_t)L.col_s;
    a.s_vecs = (uint32_t)s_vecs;
    a.tiles_per_outer = (uint32_t)tiles;
    a.inv_c = 1.0f / (float)L.col_c;
    a.eps = L.eps;
    a.tiles = (uint32_t)(L.col_outer * tiles);
    a.tiles_per_die = (a.tiles + 7u) / 8u;
    // Lanes per workgroup.  Few slabs: more lanes share one, so that a compute unit that holds one or two still has its
    // loads in flight and each lane fewer rows behind each other ([64, 384, 14, 14] fp16, 256 slabs: 17.1 us with 256 lanes,
    // 11.2 with 512, 10.0 with 1024; [256, 768, 7, 7] 27.0, 20.5, 17.6; 512 slabs of 512 rows 15.4, 14.7, 14.5).  From about
    // three slabs per unit on 256 lanes are as good (832 slabs of 192 rows: 12.8, 12.8, 14.3) and then better (3136 of 96:
    // 18.5, 20.9, 31.6).  Short columns do not fill the row groups of more lanes.
    // (A plan made without a device, whose unit count is unknown, takes 256.)
    hipDeviceProp_t prop;
    const int n_cu = (hipGetDeviceProperties(&prop, p->device) == hipSuccess && prop.multiProcessorCount > 0) ? prop.multiProcessorCount : 0;
    int threads = a.tiles > 2u * (uint32_t)n_cu || L.col_c <= 128 ? 256 : L.col_c <= 256 ? 512 : 1024;
    const int forced_t = env_int("PF_COL_THREADS", 0);
    if (forced_t == 256 || (forced_t == 512 && L.col_c <= 256) || forced_t == 1024) threads = forced_t;
    // vectors per lane: the smallest instantiated count that holds the column (threads / 8 row groups per workgroup)
    p->k = 8192 / threads;
    for (int kc : {24, 16, 12, 8, 6, 4, 3, 2, 1})
        if ((int64_t)kc * (threads / 8) >= L.col_c && (kc > 1 || threads == 256)) p->k = kc;
    p->family = PF_FAMILY_COLUMN;
    p->variant = 0;
    p->spec_id = 0;
    p->grid = dim3(a.tiles_per_die * 8u);
    p->block = dim3((uint32_t)threads);
    p->lds_bytes = (uint32_t)(4 * (threads / 64) * 8 * vec + 2 * std::min(1024, p->k * threads / 8)) * 4;
    p->n_launches = 1;
    return PF_OK;
}

pf_status plan_attn(pf_plan_s* p, int forced_variant) {
    const Lowered& L = p->low;
    const int es = dtype_size(L.main_dtype);
    const int vec = 16 / es;
    const Shape& ks = L.pre_shape;  // [..., t, d]
    const int64_t d = ks.back(), t = ks[ks.size() - 2];
    const int64_t heads = numel(ks) / (t * d);
    const bool grows = L.attn_in[1] >= 0;
    const int64_t t_total = t + (grows ? 1 : 0);
    if ((d * es) % 16 != 0) return fail(PF_ERR_ALIGNMENT, "head dimension %lld is not a multiple of 16 bytes", (long long)d);
    const int64_t lpr = d / vec;
    if (lpr > 64 || (lpr & (lpr - 1)) != 0 || d > 256)
        return fail(PF_ERR_UNSUPPORTED, "head dimension %lld: needs a power-of-two number (<= 64) of 16-byte vectors and at most 256 elements", (long long)d);
    if (heads > 65535 || t_total > 0x7fffffffLL || t_total < 1) return fail(PF_ERR_UNSUPPORTED, "attention shape out of range");
    hipDeviceProp_t prop;
    if (hipSetDevice(p->device) != hipSuccess || hipGetDeviceProperties(&prop, p->device) != hipSuccess)
        return fail(PF_ERR_HIP, "cannot query device %d (the attention family needs the device at plan time)", p->device);
    const int n_cu = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
    pf::AttnArgs& a = p->attn;
    memset(&a, 0, sizeof(a));
    a.t = (uint32_t)t;
    a.t_total = (uint32_t)t_total;
    a.d = (uint32_t)d;
    a.lanes_per_row = (uint32_t)lpr;
    a.log2_lpr = 0;
    while ((1u << a.log2_lpr) < a.lanes_per_row) ++a.log2_lpr;
    a.scale = L.attn_scale;
    // A plan that owns its workspace merges by polling self-describing words (a bounded wait, reported through the plan);
    // a call that plans and runs in one go has no plan to report through and keeps the counted, wait-free merge.
    const bool polled = !planning_static() && env_int("PF_ATTN_POLLED", 1) != 0;
    // Rows per workgroup of the counted merge, and for the choice of the variant: 8 steps of 256 / lpr rows when that still gives every compute unit two workgroups, or one where 4
    // steps would leave a head more slices than its merge takes in one trip (2 per thread group: 3 x 25 heads, t = 1023, d = 64,
    // 8 slices of 4 steps 8.7 us against 9.3; 2 x 25, t = 2047, 16 slices 10.3 against 9.6; 8 heads, t = 4000, d = 128, 63
    // slices 13.8 against 10.5); else 4.  (One or two steps per workgroup lose to the per-slice overhead, sixteen to register
    // pressure.)
    const int64_t rps = 256 / lpr;
    int nv = 4;
    int64_t dp = 1;
    while (dp < d) dp *= 2;
    const int64_t groups = 256 / dp;  // thread groups of the merge
    {
        const int64_t slices8 = heads * ((t_total + rps * 8 - 1) / (rps * 8)), splits4 = (t_total + rps * 4 - 1) / (rps * 4);
        if (slices8 >= 2 * (int64_t)n_cu || (polled && slices8 >= n_cu && splits4 > 2 * groups)) nv = 8;
    }
    const int forced_nv = env_int("PF_ATTN_NV", 0);
    if (forced_nv == 1 || forced_nv == 2 || forced_nv == 4 || forced_nv == 8) nv = forced_nv;
    // Streaming variant: a workgroup walks `chunks` chunks of 2 steps each with the next chunk's loads in flight.  Taken from
    // eight chunks on where that leaves a head one slice (many heads: no device-scope merge at all), where the merge is the
    // counted one, and where one pass would leave a head more slices than the merge has in flight in one trip, eight per thread
    // group: a further trip for every 8 groups behind the last slice costs more than the one-pass kernel's deeper load burst
    // gains.  us streamed and in one pass, fp16 -- d = 64, a trip is 32 slices: 200 heads, t = 4095 (16 slices) 42.7, 40.5;
    // t = 8191 (32) 78.7, 77.9; t = 16383 (64) 151.7, 153.6; d = 128, 16 slices a trip: 4 x 32 heads, t = 2047 (16) 31.2, 29.5;
    // 64 heads, t = 4095 (32) 32.0, 32.7; t = 8191 (64) 56.2, 62.2; t = 32767 (256) 197, 243; 8 heads, t = 131071 (1024) 111,
    // 214.  Below eight chunks the streamed slices are short and can be more than those of one pass (one head, t = 65535,
    // d = 128: 683 and 512, 98 and 66 us; not always: 8 heads, t = 16383, d = 128: 86 and 128, 28.6 and 34.4).  Two trips where a
    // trip is at most 16 slices: 125 heads, t = 2265, d = 128 (18 slices) 30.3 in one pass, 32.8 streamed; 96 heads, t = 3822 (30) 36.2 and
    // 39.5; 64 heads, t = 4095 (32) 31.9 both; 50 heads, t = 5290 (42) 30.0 and 31.5 still, but t = 8191 (64) is the streamed kernel's.  In a static call the partial results have a fixed array to fit in as well (2 MB: 4 x 32 heads, t = 4096,
    // d = 128 fill 0.5 MB streamed, 2.5 MB in one pass).
    int64_t chunks = 1;
    bool stream = false;
    {
        const int64_t all_chunks = (t_total + rps * 2 - 1) / (rps * 2);
        const int64_t target_splits = std::max<int64_t>(1, (3 * (int64_t)n_cu + heads - 1) / heads);
        const int64_t c = (all_chunks + target_splits - 1) / target_splits;
        const int forced_chunks = env_int("PF_ATTN_CHUNKS", 0);
        chunks = forced_chunks > 0 ? forced_chunks : c;
        const int64_t splits_one_pass = (t_total + rps * nv - 1) / (rps * nv);
        stream = chunks >= 8 && !forced_nv && (chunks >= all_chunks || !polled || splits_one_pass > (groups <= 2 ? 16 : 8) * groups);
    }
    int variant = forced_variant >= 0 ? forced_variant : (stream ? PF_VARIANT_ATTN_STREAM : PF_VARIANT_ATTN_ONE_PASS);
    if (variant != PF_VARIANT_ATTN_ONE_PASS && variant != PF_VARIANT_ATTN_STREAM)
        return fail(PF_ERR_UNSUPPORTED, "unknown attention variant %d", variant);
    if (variant == PF_VARIANT_ATTN_STREAM) {
        nv = forced_nv == 4 ? 4 : 2;
        if (chunks < 1) chunks = 1;
    } else {
        chunks = 1;
    }
    a.chunks = (uint32_t)chunks;
    int64_t splits = (t_total + rps * nv * chunks - 1) / (rps * nv * chunks);
    a.part_stride = (uint32_t)((d + 2 + 31) / 32 * 32);
    auto part_bytes_of = [&](int64_t slices) { return ((uint64_t)heads * slices * a.part_stride * sizeof(float) + 255) / 256 * 256; };
    const uint64_t cnt_bytes = ((uint64_t)heads * sizeof(uint32_t) + 255) / 256 * 256, at_least = planning_static() ? part_bytes_of(splits) : 0;
    // One pass: slices of one to eight steps, the number that a model of the launch finds quickest (microseconds, fitted to 360 measured
    // (shape, slices) pairs of 30 shapes; its choice is 1.002 times the best measured one in the mean, the rule above 1.10).  The
    // busiest unit pays 0.31 a workgroup and 0.11 a step; a merge costs 1.5 where a thread reads one slice, 1.6 two, 2.6 up to eight,
    // and 1.5 a further trip.  A head that is one slice merges nothing.  Slices of equal length instead of whole steps and a
    // shorter last one: 608 heads, t = 494, d = 128 29.1 us against 28.6, the others alike.  Before and after: 200 heads, t = 1023, d = 64 (4
    // slices of 8 steps, 5 of 7 now) 13.4 -> 12.9 us, 24 heads, t = 3058 10.0 -> 9.1, 8 heads, t = 143 (one slice) 5.3 -> 3.7, 50 heads,
    // t = 71, d = 128 5.4 -> 3.8.  Lost: 96 heads, t = 798, d = 128 (7 slices of 8 steps, 8 of 7 now) 12.27 -> 12.44; 128 heads, t = 600, where the model
    // sees the same difference, 12.10 -> 11.81.  Heads that eight steps leave more than 128 slices stay with the rule above, though not for
    // speed (one head of 20 000 rows, d = 128: 313 slices 41.5 us, 157 24.0): tests/test_attention_gpu.py states the 313 slices.
    // A static call takes the same slices, so that its results are the plan's, unless they do not fit the scratch array where the
    // others would (and is refused where the others do not fit).
    if (variant == PF_VARIANT_ATTN_ONE_PASS && !forced_nv && (t_total + rps * 8 - 1) / (rps * 8) <= 128) {
        const int64_t room = planning_static() ? (int64_t)(tls_scratch->cap - std::min(tls_scratch->cap, (tls_scratch->used + 255) / 256 * 256)) - (int64_t)cnt_bytes - 256 : INT64_MAX;
        double best = 0.0;
        for (int64_t steps = 8; steps >= 1; --steps) {
            const int64_t s = (t_total + rps * steps - 1) / (rps * steps);
            const int64_t per_unit = (heads * s + n_cu - 1) / n_cu, trips = (s + 8 * groups - 1) / (8 * groups);
            const int64_t needed = ((t_total + s - 1) / s + rps - 1) / rps;  // (steps that make no more slices)
            const double merge = s == 1 ? 0.0 : s <= groups ? 1.5 : s <= 2 * groups ? 1.6 : 2.6 + 1.5 * (double)(trips - 1);
            const double cost = (double)per_unit * (0.31 + 0.11 * (double)needed) + merge;
            if ((best == 0.0 || cost < best) && (int64_t)part_bytes_of(s) <= room) best = cost, splits = s, nv = (int)needed;
        }
    }
    if (splits > 65535) return fail(PF_ERR_UNSUPPORTED, "too many cached rows for the attention family");
    p->family = PF_FAMILY_ATTENTION;
    p->variant = variant;
    p->k = nv;
    p->spec_id = 0;
    p->block = dim3(256);
    p->grid = dim3((uint32_t)splits, (uint32_t)heads);
    p->lds_bytes = (8 + 4 * 256 + 1) * 4;
    p->n_launches = 1;
    const uint64_t part_bytes = std::max(part_bytes_of(splits), at_least);
    pf_status ws_st = plan_workspace_alloc(p, part_bytes + cnt_bytes + 256, "workspace allocation");
    if (ws_st != PF_OK) return ws_st;
    if ((ws_st = plan_workspace_fill(p, p->workspace, polled ? 0xff : 0, part_bytes, polled)) != PF_OK) return ws_st;
    if ((ws_st = plan_workspace_fill(p, static_cast<char*>(p->workspace) + part_bytes, 0, cnt_bytes + 256, true)) != PF_OK) return ws_st;
    a.ws_partial = reinterpret_cast<float*>(p->workspace);
    a.ws_counter = reinterpret_cast<uint32_t*>(static_cast<char*>(p->workspace) + part_bytes);
    if (polled) {
        a.polled = 1;
        a.spin_limit = (uint32_t)env_int("PF_ATTN_SPIN_LIMIT", 1 << 20);  // re-reads before a wait gives up (tests force it small)
        a.ws_error = reinterpret_cast<uint32_t*>(static_cast<char*>(p->workspace) + part_bytes + cnt_bytes);
        p->ws_error = a.ws_error;
    }
    return PF_OK;
}

pf_status plan_checked_desc(const pf_chain_desc* desc, int32_t device, int32_t variant, pf_plan** out, PlanMode mode) {
    Checked c;
    pf_status s = check_desc(desc, &c);
    if (s != PF_OK) return s;
    pf_plan_s* p = new (std::nothrow) pf_plan_s();
    if (!p) return fail(PF_ERR_NOMEM, "out of host memory");
    const uint64_t scratch_used_before = tls_scratch ? tls_scratch->used : 0;
    p->desc = *desc;
    p->device = device;
    memset(&p->args, 0, sizeof(p->args));
    memset(&p->row, 0, sizeof(p->row));
    memset(&p->group, 0, sizeof(p->group));
    memset(&p->permg, 0, sizeof(p->permg));
    memset(&p->attn, 0, sizeof(p->attn));
    p->stats_only = mode == PLAN_GROUP_STATISTICS;
    s = lower_chain(desc, c, &p->low, mode == PLAN_POOL_WITH_NORM);
    if (s == PF_OK && ((p->stats_only && p->low.core != pf::CORE_GROUPNORM) || (mode == PLAN_POOL_WITH_NORM && p->low.norm_op < 0)))
        s = fail(PF_ERR_UNSUPPORTED, "internal: not the chain this part was meant for");
    if (s == PF_OK && p->low.core != pf::CORE_ATTN_DECODE && p->low.core != pf::CORE_GATHER && p->low.core != pf::CORE_COLNORM) {
        const Lowered& L = p->low;
        p->args.n_full = L.n_full;
        p->args.n_vec = L.n_vec;
        p->args.core = L.core;
        p->args.core_vec[0] = L.core_vec[0];
        p->args.core_vec[1] = L.core_vec[1];
        p->args.eps = L.eps;
        p->args.mask_si = L.mask_si;
        p->args.core_mask = L.core_mask;
        p->args.mask_div = make_fastdiv(L.mask_si ? L.mask_si : 1u);
        p->args.core_scale = L.core_scale;
        p->args.pro = L.pro;
        p->args.epi = L.epi;
        // pure layout work (nothing but the initial load): kernels move the raw bits, no conversion
        p->args.raw_copy = (L.pro.n == 1 && L.epi.n == 0 && L.pro.u[0].code == pf::U_MOV && L.pro.u[0].kind == pf::K_FULL) ? 1u : 0u;
        s = fill_vec_args(p, c);
    }
    if (s == PF_OK) {
        switch (p->low.core) {
            case pf::CORE_NONE: s = plan_ew(p); break;
            case pf::CORE_GROUPNORM: s = plan_group(p, variant); break;
            case pf::CORE_PERMUTE: s = plan_perm(p, variant); break;
            case pf::CORE_ATTN_DECODE: s = plan_attn(p, variant); break;
            case pf::CORE_GATHER: s = plan_gather(p, c); break;
            case pf::CORE_DWCONV: s = plan_stencil(p, c, variant); break;
            case pf::CORE_POOL: s = plan_pool(p); break;
            case pf::CORE_COLNORM: s = plan_column(p); break;
            default: s = plan_row(p, variant); break;
        }
    }
    // A launch holds fewer than 2^32 lanes (the device counts them in 32 bits): more are not refused by the run-time, which
    // starts what is left of the number modulo 2^32.
    if (s == PF_OK && (uint64_t)p->grid.x * p->block.x > 0xffffffffull)
        s = fail(PF_ERR_UNSUPPORTED, "tensor too large for one launch (%u workgroups of %u lanes)", p->grid.x, p->block.x);
    if (s == PF_OK) {
        for (int k = 0; k < desc->n_inputs; ++k) p->in_bytes[k] = (uint64_t)numel(c.shape[k]) * dtype_size(desc->inputs[k].dtype);
        for (int o = 0; o < desc->n_outputs; ++o) {
            p->out_shape[o] = c.shape[desc->out_value[o]];
            p->out_bytes[o] = p->stats_only ? 0 : (uint64_t)numel(p->out_shape[o]) * dtype_size(desc->out_dtype[o]);
        }
        if (env_int("PF_LOG", 0))
            fprintf(stderr, "[pf_chain] family=%d variant=%d spec=%d k=%d rpw=%u grid=%u block=%u uops=%d+%d full=%d vec=%d tmp=%d mask_si=%u\n",
                    p->family, p->variant, p->spec_id, p->k, p->row.rows_per_wave, p->grid.x, p->block.x, p->low.pro.n, p->low.epi.n, p->low.n_full,
                    p->low.n_vec, p->low.n_tmp, p->low.mask_si);
        *out = p;
        return PF_OK;
    }
    pf_chain_plan_destroy(p);
    if (tls_scratch) tls_scratch->used = scratch_used_before;  // a plan that failed gives its share of the scratch array back
    return s;
}

pf_status plan_one_kernel(const pf_chain_desc* desc, int32_t device, int32_t variant, pf_plan** out) {
    Checked c;
    pf_status s = check_desc(desc, &c);
    if (s != PF_OK) return s;
    // a chain that spells a composite operator in basic operators is planned as that operator when that works
    if (env_int("PF_RECOMPOSE", 1) != 0) {
        pf_chain_desc composite;
        if (recompose_chain(desc, c, &composite) && plan_checked_desc(&composite, device, variant, out) == PF_OK) return PF_OK;
    }
    return plan_checked_desc(desc, device, variant, out);
}

}  // namespace pfh
