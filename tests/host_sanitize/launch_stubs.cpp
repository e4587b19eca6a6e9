// Host-only stand-ins for the kernel launchers and the three HIP runtime calls
// of api.cpp, for the AddressSanitizer / UndefinedBehaviorSanitizer build of
// the C ABI's host code (tests/test_host_sanitize.py).  Nothing here touches a
// GPU.  Each launcher checks what the host hands to the kernels: descriptor
// counts within the argument tables, first-workgroup offsets that never
// decrease, and every workspace range the kernels would write inside the
// workspace the caller passed (set by the driver).  The noise launcher also
// counts, per tensor, the launches that add Gaussian noise to it, so that the
// driver can check that every gradient gets its noise exactly once.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>

#include "bk_kernels.h"

uintptr_t g_ws_lo = 0, g_ws_hi = 0;   // [lo, hi): the caller's workspace
long g_launches = 0;
long g_ghost_wgs = 0;                 // most workgroups of a ghost-norm launch
long g_ghost_launches = 0;
long g_gemm_wgs = 0;                  // ... of the last a^T g launch
long g_gemm_launches = 0;
long g_gemm_min_wgs = 0;              // ... of the smallest one (0: none yet)
int g_gemm_remap = 0, g_gemm_first_T = 0;   // its XCD deal, the T of its first layer
bk::GemmVariant g_gemm_variant = bk::GemmVariant::Scalar;   // ... of the last one
std::map<uintptr_t, int> g_noised;    // tensor -> launches that add noise to it

namespace {
void need(bool ok, const char* what) {
    if (!ok) {
        std::fprintf(stderr, "launch check failed: %s\n", what);
        std::abort();
    }
}
void in_ws(const void* base, int64_t off_elems, int64_t n_elems, size_t es, const char* what) {
    if (n_elems <= 0) return;
    const uintptr_t b = reinterpret_cast<uintptr_t>(base);
    need(b != 0 && off_elems >= 0, what);
    const uintptr_t lo = b + (uintptr_t)off_elems * es, hi = lo + (uintptr_t)n_elems * es;
    need(lo >= g_ws_lo && hi <= g_ws_hi, what);
}
template <typename L>
void monotone(const L* layers, int n, int max_n, int64_t n_wg, const char* what) {
    if (n_wg <= 0) return;   // the launchers return at once
    need(n >= 1 && n <= max_n, what);
    int64_t prev = 0;
    for (int k = 0; k < n; ++k) {
        if (!((int64_t)layers[k].wg_begin >= prev && (int64_t)layers[k].wg_begin < n_wg))
            std::fprintf(stderr, "descriptor %d of %d: first workgroup %lld after %lld, %lld workgroups\n", k, n,
                         (long long)layers[k].wg_begin, (long long)prev, (long long)n_wg);
        need((int64_t)layers[k].wg_begin >= prev && (int64_t)layers[k].wg_begin < n_wg, what);
        prev = layers[k].wg_begin;
    }
}
}  // namespace

extern "C" {
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
    *v = 256;
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "stub"; }
}

namespace bk {

hipError_t launch_ghost_full(const GhostArgs& a, int n_wg, bool, hipStream_t) {
    ++g_launches;
    monotone(a.L, a.n, kMaxGhost, n_wg, "ghost_full descriptors");
    for (int k = 0; k < a.n; ++k) in_ws(a.part, a.L[k].part_off, (int64_t)a.B * a.L[k].npairs, 4, "ghost_full partials");
    return hipSuccess;
}
hipError_t launch_ghost(const GhostArgs& a, int n_wg, bool, bool, bool, hipStream_t) {
    ++g_launches;
    ++g_ghost_launches;
    g_ghost_wgs = std::max(g_ghost_wgs, (long)n_wg);
    monotone(a.L, a.n, kMaxGhost, n_wg, "ghost descriptors");
    int64_t red = 0;
    for (int k = 0; k < a.n; ++k) {
        const GhostLayer& L = a.L[k];
        in_ws(a.part, L.part_off, (int64_t)a.B * L.npairs, 4, "ghost partials");
        need(L.red_begin == red, "ghost slice reduction");
        if (L.ksplit <= 1) continue;
        // column slices: every pair's partial Grams, and kGhostSplitParts partials
        const int64_t pairs = (int64_t)L.nsb * (L.nsb + 1) / 2;
        need(L.npairs == pairs * kGhostSplitParts && L.ka >= 1 && L.ka < L.ksplit && !L.Pb, "ghost slices");
        in_ws(a.tiles, L.tile_off, a.B * pairs * L.ksplit * kGhostSplitTile, 4, "ghost partial Grams");
        red += (int64_t)a.B * L.npairs;
    }
    for (int k = 0; k < a.n && a.small; ++k) {
        // whole samples to a workgroup: their rows fit its block
        const int rows = a.small == 1 ? 32 : a.small == 2 ? 64 : a.small == 3 ? 96 : 128;
        const int64_t last = k + 1 < a.n ? a.L[k + 1].wg_begin : n_wg;
        need(a.L[k].T >= 1 && (int64_t)a.L[k].nsb * a.L[k].T <= rows && (a.small == 1 || a.L[k].nsb == 1) &&
                 (last - a.L[k].wg_begin) * a.L[k].nsb >= a.B,
             "few-token samples");
    }
    need(a.n_red == red && (red == 0 || !a.small), "ghost slice reduction grid");
    return hipSuccess;
}
hipError_t launch_embed_join(const GhostArgs& a, int n_wg, bool, int ct, hipStream_t) {
    ++g_launches;
    monotone(a.L, a.n, kMaxGhost, n_wg, "join descriptors");
    need(ct == 8 || ct == 32, "join column threads");
    for (int k = 0; k < a.n; ++k) {
        need(a.L[k].T >= 1 && a.L[k].T <= kEmbedJoinMaxT && a.L[k].p % 8 == 0, "join shape");
        need((int64_t)a.L[k].npairs * 8 * ct >= a.L[k].p, "join column chunks");
        in_ws(a.part, a.L[k].part_off, (int64_t)a.B * a.L[k].npairs, 4, "join partials");
    }
    return hipSuccess;
}
hipError_t launch_gemm(const GemmArgs& a, int n_wg, bool, bool inst, GemmVariant v, hipStream_t, int n_remap) {
    ++g_launches;
    g_gemm_wgs = n_wg;
    g_gemm_min_wgs = g_gemm_min_wgs == 0 ? n_wg : std::min(g_gemm_min_wgs, (long)n_wg);
    ++g_gemm_launches;
    g_gemm_variant = v;
    g_gemm_remap = n_remap;
    g_gemm_first_T = a.n > 0 ? a.L[0].T : 0;
    need(n_remap >= 0 || v == GemmVariant::F32 || v == GemmVariant::F32Any, "order of workgroups");
    monotone(a.L, a.n, kMaxGemm, n_wg, "gemm descriptors");
    for (int k = 0; k < a.n; ++k) {
        const GemmLayer& L = a.L[k];
        const GemmGeom geo = gemm_geom(v, L.d, L.p);
        need(L.tm == geo.tm && L.tn == geo.tn, "gemm tiles");
        const int64_t tiles = (int64_t)L.tm * L.tn;
        // the fp32 kernel reads C through a 32-bit buffer descriptor
        if (!inst && (v == GemmVariant::F32 || v == GemmVariant::F32Any))
            need((uint64_t)a.B * 4 < 0xFFFFFFF0u, "fp32 clip weights within 32-bit offsets");
        // 16-byte pieces of rows of fewer than 8 columns end inside the batch
        if (v == GemmVariant::WideAny) need((int64_t)a.B * L.T * std::min(L.d, L.p) >= 8, "unaligned bf16 rows");
        if (inst && v == GemmVariant::GradDL) {
            // one workgroup per (sample, tile), never split, no clip weights
            need(L.ksplit <= 1 && a.C == nullptr && (int64_t)a.B * L.T < ((int64_t)1 << 31) && L.T >= 64,
                 "LDS-DMA instantiated norm");
        }
        if (inst) {
            const int64_t parts = L.ksplit > 1 ? tiles * (geo.tile_elems / kSplitRedWG) : tiles;
            in_ws(a.part, L.part_off, (int64_t)a.B * parts, 4, "inst partials");
            if (L.ksplit > 1) in_ws(a.tiles, L.ptile_off, (int64_t)a.B * tiles * L.ksplit * geo.tile_elems, 4, "inst tiles");
        } else if (L.ksplit > 1) {
            need(L.split_from >= 0 && L.split_from <= tiles, "grad split_from");
            in_ws(a.tiles, L.ptile_off, (tiles - L.split_from) * L.ksplit * geo.tile_elems, 4, "grad tiles");
        }
    }
    return hipSuccess;
}
hipError_t launch_split_reduce(const GemmArgs& a, int n_wg, bool inst, GemmVariant v, hipStream_t) {
    ++g_launches;
    need(n_wg > 0 && a.n >= 1 && a.n <= kMaxGemm, "split reduce");
    // the variants whose slices the kernel adds
    need(v == GemmVariant::Wide || v == GemmVariant::Narrow32 || v == GemmVariant::Narrow64 || v == GemmVariant::F32 ||
             v == GemmVariant::F32Any || (!inst && (v == GemmVariant::Grad || v == GemmVariant::GradDL)),
         "split reduce variant");
    int64_t red = 0;
    for (int k = 0; k < a.n; ++k) {
        const GemmLayer& L = a.L[k];
        need(L.red_begin == red, "split reduce descriptors");
        const int64_t tiles = (int64_t)L.tm * L.tn - L.split_from;
        if (L.ksplit > 1) red += (inst ? a.B : 1) * tiles * (gemm_geom(v, L.d, L.p).tile_elems / kSplitRedWG);
    }
    need(red == n_wg, "split reduce grid");
    return hipSuccess;
}
hipError_t launch_reduce(const ReduceArgs& a, hipStream_t) {
    ++g_launches;
    need(a.n >= 1 && a.n <= kMaxReduce && a.B >= 1, "reduce descriptors");
    for (int k = 0; k < a.n; ++k) {
        in_ws(a.part, a.L[k].part_off, (int64_t)a.B * a.L[k].npart, 4, "reduce partials");
        in_ws(a.part, a.L[k].part_off2, (int64_t)a.B * a.L[k].npart2, 4, "reduce second partials");
    }
    return hipSuccess;
}
hipError_t launch_clip(const float*, int64_t L, int64_t B, int, float, float, float*, float*, hipStream_t) {
    ++g_launches;
    need(L >= 0 && B >= 0, "clip sizes");
    return hipSuccess;
}
hipError_t launch_noise(const NoiseArgs& a, int n_wg, hipStream_t) {
    ++g_launches;
    need(a.n >= 1 && a.n <= kMaxNoise && a.bpw >= 256 && a.bpw <= (uint32_t)kNoiseBlocksPerWG && a.bpw % 256 == 0,
         "noise descriptors");
    uint32_t prev = 0;
    for (int k = 0; k < a.n; ++k) {
        need(a.L[k].wg_begin >= prev && (int64_t)a.L[k].wg_begin < n_wg && a.L[k].n > 0, "noise layers");
        prev = a.L[k].wg_begin;
        ++g_noised[reinterpret_cast<uintptr_t>(a.L[k].G)];
    }
    return hipSuccess;
}
hipError_t launch_wsum(const WsumArgs& a, int n_wg, hipStream_t) {
    ++g_launches;
    need(a.n >= 1 && a.n <= kMaxWsum && n_wg > 0, "wsum descriptors");
    return hipSuccess;
}
hipError_t launch_unfold(const void*, void*, const UnfoldShape& s, bool, hipStream_t) {
    ++g_launches;
    need(s.Ho > 0 && s.Wo > 0 && s.T == s.Ho * s.Wo && s.ld >= s.C * s.kh * s.kw, "unfold shape");
    return hipSuccess;
}
hipError_t launch_conv_prep(const ConvPrepLayer*, int n, int64_t B, bool, hipStream_t) {
    ++g_launches;
    need(n >= 1 && B >= 1, "conv prep");
    return hipSuccess;
}
hipError_t launch_tokens(const void*, void*, int64_t B, int64_t C, int64_t HW, bool, hipStream_t) {
    ++g_launches;
    need(B >= 1 && C >= 1 && HW >= 1, "tokens shape");
    return hipSuccess;
}
hipError_t launch_philox_raw(uint64_t, uint32_t, uint32_t, uint64_t, int64_t nq, uint32_t*, hipStream_t) {
    ++g_launches;
    need(nq >= 0, "philox count");
    return hipSuccess;
}
hipError_t launch_embed_grad(const int64_t*, const void*, const float*, bool, int64_t B, int64_t T, int64_t p,
                             int64_t V, float*, void* ws, bool, hipStream_t) {
    ++g_launches;
    need(B * T <= kEmbedMaxTokens && V > 0 && p > 0, "embedding gradient shape");
    in_ws(ws, 0, (int64_t)embed_grad_ws_bytes(B * T, p), 1, "embedding gradient workspace");
    return hipSuccess;
}
hipError_t launch_affine(const AffineArgs& a, int n_wg, bool, hipStream_t) {
    ++g_launches;
    monotone(a.L, a.n, kMaxAffine, n_wg, "affine descriptors");
    for (int k = 0; k < a.n; ++k) in_ws(a.part, a.L[k].part_off, (int64_t)a.B * a.L[k].chunks, 4, "affine partials");
    return hipSuccess;
}

}  // namespace bk
