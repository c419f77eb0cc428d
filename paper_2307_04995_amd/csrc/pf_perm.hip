// Build-time instantiations of the transpose family (catalogue entries and the run-time-interpreted form),
// their launcher, and the copy probes every chain is measured against.
#include "pf_launch.h"
#include "pf_perm_kernels.hpp"
#include "pf_specs.h"

namespace pf {

// ---------------------------------------------------------------------------------------------
template <int ID>
struct PermSpecOf;
#define PF_DEF_SPEC(id, nf, nv, nt, core, gamma, beta, pro, epi)                                              \
    template <>                                                                                                \
    struct PermSpecOf<id> {                                                                                    \
        using type = StaticSpec<nf, nv, nt, core, gamma, beta, StaticList<pro>, StaticList<epi>>;              \
    };
PF_PERM_SPECS(PF_DEF_SPEC)
#undef PF_DEF_SPEC
template <>
struct PermSpecOf<0> {
    using type = GenericSpec;
};

template <int ID, int DT>
static hipError_t launch_perm_spec_dt(const ChainArgs& a, const PermGeom& g, int variant, int k, bool ragged, dim3 grid, dim3 block,
                                      uint32_t lds, hipStream_t st) {
    using Spec = typename PermSpecOf<ID>::type;
    if (ragged) {
        // extents that are not whole vectors: built in the run-time-interpreted form only (specialised when the plan is made)
        if constexpr (ID == 0) {
            if (variant == 2) hipLaunchKernelGGL((perm_tile_kernel<DT, Spec, true>), grid, block, 0, st, a, g);
            else if (variant == 0 && k == 1) hipLaunchKernelGGL((perm_rows_kernel<DT, 1, Spec, true>), grid, block, 0, st, a, g);
            else return hipErrorInvalidValue;
            return hipGetLastError();
        }
        return hipErrorInvalidValue;
    }
    if (variant == 2) {
        hipLaunchKernelGGL((perm_tile_kernel<DT, Spec>), grid, block, 0, st, a, g);
    } else if (variant == 1) {
        hipLaunchKernelGGL((perm_lds_rows_kernel<DT, Spec>), grid, block, lds, st, a, g);
    } else if (k == 2) {
        hipLaunchKernelGGL((perm_rows_kernel<DT, 2, Spec>), grid, block, 0, st, a, g);
    } else {
        hipLaunchKernelGGL((perm_rows_kernel<DT, 1, Spec>), grid, block, 0, st, a, g);
    }
    return hipGetLastError();
}

template <int ID>
static hipError_t launch_perm_spec(int dtype, const ChainArgs& a, const PermGeom& g, int variant, int k, bool ragged, dim3 grid,
                                   dim3 block, uint32_t lds, hipStream_t st) {
    switch (dtype) {
        case DT_F32: return launch_perm_spec_dt<ID, DT_F32>(a, g, variant, k, ragged, grid, block, lds, st);
        case DT_F16: return launch_perm_spec_dt<ID, DT_F16>(a, g, variant, k, ragged, grid, block, lds, st);
        case DT_BF16: return launch_perm_spec_dt<ID, DT_BF16>(a, g, variant, k, ragged, grid, block, lds, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_perm(int spec_id, int dtype, const ChainArgs& a, const PermGeom& g, int variant, int k, bool ragged, dim3 grid,
                       dim3 block, uint32_t lds, hipStream_t st) {
    switch (spec_id) {
        case 0: return launch_perm_spec<0>(dtype, a, g, variant, k, ragged, grid, block, lds, st);
#define PF_CASE(id, ...) \
    case id: return launch_perm_spec<id>(dtype, a, g, variant, k, ragged, grid, block, lds, st);
            PF_PERM_SPECS(PF_CASE)
#undef PF_CASE
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_perm_plane(int dtype, bool flat_out, const void* in, void* out, const PlaneGeom& g, dim3 grid, uint32_t lds, hipStream_t st) {
    // (the bits travel untouched: the element size is all that matters of the type)
    if (dtype == DT_F32) {
        if (flat_out) hipLaunchKernelGGL((perm_plane_kernel<DT_F32, true>), grid, dim3(256), lds, st, in, out, g);
        else hipLaunchKernelGGL((perm_plane_kernel<DT_F32, false>), grid, dim3(256), lds, st, in, out, g);
    } else {
        if (flat_out) hipLaunchKernelGGL((perm_plane_kernel<DT_F16, true>), grid, dim3(256), lds, st, in, out, g);
        else hipLaunchKernelGGL((perm_plane_kernel<DT_F16, false>), grid, dim3(256), lds, st, in, out, g);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// copy probe: the plain streaming copy every chain is measured against
// ---------------------------------------------------------------------------------------------
template <int K, bool NT>
__global__ void __launch_bounds__(256) copy_probe_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst, uint64_t n_vec) {
    const uint64_t base = (uint64_t)blockIdx.x * (256u * K) + threadIdx.x;
    u32x4 r[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint64_t v = base + 256u * k;
        r[k] = u32x4{0u, 0u, 0u, 0u};
        if (v < n_vec) r[k] = NT ? __builtin_nontemporal_load(src + v) : src[v];
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint64_t v = base + 256u * k;
        if (v < n_vec) {
            if (NT) __builtin_nontemporal_store(r[k], dst + v);
            else dst[v] = r[k];
        }
    }
}

// persistent form: a fixed grid, each workgroup strides over the buffer
template <int K>
__global__ void __launch_bounds__(256) copy_persistent_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst, uint64_t n_vec) {
    const uint64_t step = (uint64_t)gridDim.x * (256u * K);
    for (uint64_t base = (uint64_t)blockIdx.x * (256u * K) + threadIdx.x; base < n_vec; base += step) {
        u32x4 r[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint64_t v = base + 256u * k;
            r[k] = u32x4{0u, 0u, 0u, 0u};
            if (v < n_vec) r[k] = __builtin_nontemporal_load(src + v);
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint64_t v = base + 256u * k;
            if (v < n_vec) __builtin_nontemporal_store(r[k], dst + v);
        }
    }
}

// read-only and write-only streams, to see how the two directions share the memory system
template <int K>
__global__ void __launch_bounds__(256) read_probe_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst, uint64_t n_vec) {
    const uint64_t base = (uint64_t)blockIdx.x * (256u * K) + threadIdx.x;
    u32x4 acc = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint64_t v = base + 256u * k;
        if (v < n_vec) acc ^= __builtin_nontemporal_load(src + v);
    }
    // the data is random-free (benchmark buffers hold a constant), so this store never happens; it only
    // keeps the loads alive
    if ((acc[0] ^ acc[1] ^ acc[2] ^ acc[3]) == 0x9e3779b9u) dst[base % n_vec] = acc;
}
template <int K>
__global__ void __launch_bounds__(256) write_probe_kernel(u32x4* __restrict__ dst, uint64_t n_vec) {
    const uint64_t base = (uint64_t)blockIdx.x * (256u * K) + threadIdx.x;
    const u32x4 val = u32x4{(uint32_t)base, 1u, 2u, 3u};
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint64_t v = base + 256u * k;
        if (v < n_vec) __builtin_nontemporal_store(val, dst + v);
    }
}

hipError_t launch_copy_probe(const void* src, void* dst, uint64_t bytes, int variant, hipStream_t st) {
    const uint64_t n_vec = bytes / 16;
    if (n_vec == 0) return hipSuccess;
    const u32x4* s = static_cast<const u32x4*>(src);
    u32x4* d = static_cast<u32x4*>(dst);
    // variant = unroll (1, 2, 4) | 16: plain (temporal) accesses | 32: read only | 64: write only
    //           | 128: persistent grid with (variant >> 8) workgroups per compute unit
    const bool nt = (variant & 16) == 0;
    const int k = variant & 15;
    const uint64_t per_block = 256ull * (uint64_t)(k ? k : 1);
    const uint64_t blocks = (n_vec + per_block - 1) / per_block;
    if (blocks > 0x7fffffffull) return hipErrorInvalidValue;
    dim3 grid((uint32_t)blocks), block(256);
    if (variant & 128) {
        // persistent: (variant >> 8) workgroups per compute unit, 256 compute units assumed
        const uint32_t per_cu = (uint32_t)(variant >> 8) ? (uint32_t)(variant >> 8) : 8u;
        dim3 pgrid(256u * per_cu);
        switch (k) {
            case 1: hipLaunchKernelGGL((copy_persistent_kernel<1>), pgrid, block, 0, st, s, d, n_vec); break;
            case 2: hipLaunchKernelGGL((copy_persistent_kernel<2>), pgrid, block, 0, st, s, d, n_vec); break;
            case 4: hipLaunchKernelGGL((copy_persistent_kernel<4>), pgrid, block, 0, st, s, d, n_vec); break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    if (variant & 32) {
        switch (k) {
            case 1: hipLaunchKernelGGL((read_probe_kernel<1>), grid, block, 0, st, s, d, n_vec); break;
            case 2: hipLaunchKernelGGL((read_probe_kernel<2>), grid, block, 0, st, s, d, n_vec); break;
            case 4: hipLaunchKernelGGL((read_probe_kernel<4>), grid, block, 0, st, s, d, n_vec); break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    if (variant & 64) {
        switch (k) {
            case 1: hipLaunchKernelGGL((write_probe_kernel<1>), grid, block, 0, st, d, n_vec); break;
            case 2: hipLaunchKernelGGL((write_probe_kernel<2>), grid, block, 0, st, d, n_vec); break;
            case 4: hipLaunchKernelGGL((write_probe_kernel<4>), grid, block, 0, st, d, n_vec); break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
#define PF_COPY(KK)                                                                                   \
    if (nt) hipLaunchKernelGGL((copy_probe_kernel<KK, true>), grid, block, 0, st, s, d, n_vec);       \
    else hipLaunchKernelGGL((copy_probe_kernel<KK, false>), grid, block, 0, st, s, d, n_vec);
    switch (k) {
        case 1: PF_COPY(1) break;
        case 2: PF_COPY(2) break;
        case 4: PF_COPY(4) break;
        default: return hipErrorInvalidValue;
    }
#undef PF_COPY
    return hipGetLastError();
}

}  // namespace pf
