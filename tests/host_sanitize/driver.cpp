// Driver of the sanitizer build of the C ABI's host code: workspace queries,
// every grouped call over random stacks, and invalid arguments, with the
// launchers stubbed (launch_stubs.cpp).  Device pointers are fake, aligned
// addresses: the host code never dereferences them.  Prints "ok" and exits 0
// when every call returned (sanitizer reports abort the run).
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <map>
#include <vector>

#include "bk.h"
#include "bk_kernels.h"

extern uintptr_t g_ws_lo, g_ws_hi;
extern long g_launches;
extern long g_ghost_wgs, g_ghost_launches, g_gemm_wgs, g_gemm_launches, g_gemm_min_wgs;
extern int g_gemm_remap, g_gemm_first_T;
extern bk::GemmVariant g_gemm_variant;
extern std::map<uintptr_t, int> g_noised;

namespace {
std::mt19937_64 rng(20221001);
int64_t pick(std::initializer_list<int64_t> v) { return *(v.begin() + rng() % v.size()); }
void* fake(uintptr_t k, bool misalign = false) { return reinterpret_cast<void*>((k << 24) + (misalign ? 2 : 0)); }
void* set_ws(size_t bytes) {
    g_ws_lo = (uintptr_t)0x7f0000000000ull;
    g_ws_hi = g_ws_lo + bytes;
    return reinterpret_cast<void*>(g_ws_lo);
}
int64_t dim() { return pick({1, 2, 7, 8, 16, 24, 32, 60, 64, 100, 128, 256, 264, 300, 768, 1024, 1280, 3072, 4096}); }
int64_t tlen() { return pick({0, 1, 16, 49, 64, 70, 100, 128, 129, 197, 256, 300, 784, 1000, 1024, 4096, 16385}); }
}  // namespace

// Every weight and bias gradient with elements got its noise from exactly one
// launch (none without noise), and nothing else got any.
bool noised_once(const std::vector<bk_layer>& L, float sig) {
    std::map<uintptr_t, int> want;
    if (sig != 0.f)
        for (const bk_layer& y : L) {
            if ((y.kind == BK_NORM_AFFINE ? y.p : y.d * y.p) > 0) ++want[reinterpret_cast<uintptr_t>(y.G)];
            if ((y.flags & BK_LAYER_BIAS) && y.p > 0) ++want[reinterpret_cast<uintptr_t>(y.Gb)];
        }
    if (want != g_noised) {
        std::fprintf(stderr, "noise launches per tensor: %zu tensors expected, %zu noised\n", want.size(),
                     g_noised.size());
        return false;
    }
    return true;
}

int main() {
    // 1. workspace queries: random, edge and invalid sizes for every op
    for (int it = 0; it < 20000; ++it) {
        const bk_op op = (bk_op)(rng() % 6);
        const bk_dtype dt = (bk_dtype)(rng() % 3);
        const int64_t B = pick({-1, 0, 1, 2, 16, 64, 4096, 4097, (int64_t)1 << 20});
        const int64_t T = pick({-3, 0, 1, 33, 128, 129, 1024, 16384, 16385, (int64_t)1 << 31});
        const int64_t d = pick({-1, 0, 1, 8, 60, 768, 50257, 8192, (int64_t)1 << 40});
        const int64_t p = pick({0, 1, 8, 60, 64, 264, 1280, 3072});
        (void)bk_workspace_size(op, dt, B, T, d, p);
        const int gs = bk_use_ghost(T, d, p), gt = bk_use_ghost_time(T, d, p);
        if (gt == 1 && gs != 1) {
            std::fprintf(stderr, "time rule ghost where the space rule is not (T=%lld d=%lld p=%lld)\n",
                         (long long)T, (long long)d, (long long)p);
            return 1;
        }
    }

    // 2. random stacks through the grouped calls
    int calls = 0, ok_calls = 0;
    for (int it = 0; it < 4000; ++it) {
        const int n = 1 + (int)(rng() % 110);
        const bk_dtype dt = rng() % 4 ? BK_BF16 : BK_F32;
        const int64_t B = pick({1, 2, 3, 16, 32, 64, 4096, 4097});
        std::vector<bk_layer> L((size_t)n);
        for (int l = 0; l < n; ++l) {
            bk_layer& y = L[(size_t)l];
            const int r = (int)(rng() % 10);
            y.kind = r < 7 ? BK_LINEAR : r < 8 ? BK_EMBEDDING : BK_NORM_AFFINE;
            y.T = tlen();
            y.p = dim();
            y.d = y.kind == BK_EMBEDDING ? pick({1, 300, 50257}) : y.kind == BK_NORM_AFFINE ? y.p : dim();
            const bool mis = rng() % 8 == 0;
            y.x = fake(4 * l + 1, mis && y.kind != BK_EMBEDDING);
            y.g = fake(4 * l + 2, mis);
            y.G = static_cast<float*>(fake(4 * l + 3));
            y.flags = 0;
            if (y.kind != BK_EMBEDDING && rng() % 3 == 0) {
                y.flags |= BK_LAYER_BIAS;
                y.Gb = static_cast<float*>(fake(0x100000 + l));
                y.Pb = static_cast<float*>(fake(0x200000 + l));
            }
            if (rng() % 4 == 0) y.flags |= BK_LAYER_ACCUMULATE;
            if (rng() % 3 == 0) y.flags |= BK_LAYER_TIME_RULE;
            if (y.kind == BK_NORM_AFFINE || (y.kind == BK_LINEAR && rng() % 5 == 0)) {
                if (y.kind == BK_LINEAR) y.flags |= BK_LAYER_MIXOPT;
                y.P = static_cast<float*>(fake(0x300000 + l));
            }
        }
        float* norm = static_cast<float*>(fake(0x400000));
        float* C = static_cast<float*>(fake(0x400001));
        float* tot = static_cast<float*>(fake(0x400002));
        const size_t wn = bk_layer_norms_workspace_size(L.data(), n, dt, B);
        const size_t wg = bk_weighted_grads_workspace_size(L.data(), n, dt, B);
        const size_t wp = bk_private_grad_workspace_size(L.data(), n, dt, B);
        if (wp < wn || wp < wg) {
            std::fprintf(stderr, "private-grad workspace below a phase's\n");
            return 1;
        }
        ++calls;
        ok_calls += bk_layer_norms(L.data(), n, dt, B, norm, set_ws(wn), wn, nullptr) == BK_OK;
        (void)bk_weighted_grads(L.data(), n, C, dt, B, set_ws(wg), wg, nullptr);
        const float sig = rng() % 2 ? 1.f : 0.f;
        g_noised.clear();
        const bk_status pst = bk_private_grad(L.data(), n, dt, B, (bk_clip)(rng() % 2), 1.f, 0.01f, sig, 7,
                                              (uint32_t)it, norm, C, tot, set_ws(wp), wp, nullptr);
        if (pst == BK_OK && !noised_once(L, sig)) return 1;
        if (wp > 0 && bk_private_grad(L.data(), n, dt, B, BK_CLIP_AUTO, 1.f, 0.01f, 1.f, 7, 0, norm, C, tot,
                                      set_ws(wp), wp - 1, nullptr) == BK_OK) {
            std::fprintf(stderr, "a short workspace was accepted\n");
            return 1;
        }
    }

    // 3. single-layer calls and invalid arguments
    for (int it = 0; it < 3000; ++it) {
        const bk_dtype dt = (bk_dtype)(rng() % 2);
        const int64_t B = pick({0, 1, 3, 16}), T = tlen(), d = dim(), p = dim();
        void* a = fake(1, rng() % 6 == 0);
        void* g = fake(2, rng() % 6 == 0);
        float* out = static_cast<float*>(fake(3));
        size_t w = bk_workspace_size(BK_OP_GHOST_NORM, dt, B, T, d, p);
        (void)bk_ghost_norm(a, g, dt, B, T, d, p, out, set_ws(w), w, nullptr);
        w = bk_workspace_size(BK_OP_INST_NORM, dt, B, T, d, p);
        (void)bk_inst_norm(a, g, dt, B, T, d, p, out, set_ws(w), w, nullptr);
        const int64_t V = pick({1, 50257});
        w = bk_workspace_size(BK_OP_EMBED_GHOST_NORM, dt, B, T, V, p);
        (void)bk_embed_ghost_norm(static_cast<const int64_t*>(fake(4)), g, dt, B, T, p, V, out, set_ws(w), w, nullptr);
        w = bk_workspace_size(BK_OP_WEIGHTED_GRAD, dt, B, T, d, p);
        (void)bk_weighted_grad(a, g, out, dt, B, T, d, p, out, set_ws(w), w, nullptr);
        w = bk_workspace_size(BK_OP_EMBED_WEIGHTED_GRAD, dt, B, T, V, p);
        (void)bk_embed_weighted_grad(static_cast<const int64_t*>(fake(4)), g, out, dt, B, T, p, V, out, set_ws(w), w,
                                     nullptr);
        (void)bk_clip_factors(out, pick({0, 1, 48}), B, (bk_clip)(rng() % 3), pick({-1, 0, 1}), pick({-1, 0, 1}),
                              out, out, nullptr);
        (void)bk_add_noise(out, pick({-1, 0, 5, 1 << 20}), pick({-1, 0, 1}), 3, 0, 0, nullptr);
        (void)bk_philox_raw(1, 2, 3, 0, pick({-1, 0, 17}), reinterpret_cast<uint32_t*>(out), nullptr);
        // invalid pointers and sizes: every call must fail validation, not crash
        (void)bk_ghost_norm(nullptr, g, dt, B + 1, T + 1, d, p, out, nullptr, 0, nullptr);
        (void)bk_inst_norm(a, g, (bk_dtype)7, B, T, d, p, out, nullptr, 0, nullptr);
        (void)bk_weighted_grad(a, g, nullptr, dt, -B - 1, T, d, p, out, nullptr, 0, nullptr);
        (void)bk_layer_norms(nullptr, 3, dt, B, out, nullptr, 0, nullptr);
    }
    {   // batches of a thousand million one-token samples
        for (int64_t B : {(int64_t)1 << 28, ((int64_t)1 << 30) - 4, (int64_t)1 << 30, (int64_t)INT32_MAX})
            for (int64_t d : {1, 4}) {
                const size_t w = bk_workspace_size(BK_OP_WEIGHTED_GRAD, BK_F32, B, 1, d, 4);
                float* out = static_cast<float*>(fake(3));
                const bk_status st = bk_weighted_grad(fake(1), fake(2), out, BK_F32, B, 1, d, 4, out, set_ws(w), w, nullptr);
                if (st != BK_OK) {
                    std::fprintf(stderr, "a clipped gradient of %lld samples was refused\n", (long long)B);
                    return 1;
                }
            }
    }
    // long rows, few samples: the rows are cut into column slices at every batch
    for (const bk_dtype dt : {BK_BF16, BK_F32})
        for (int64_t B = 1; B < 64; ++B) {
            struct { int64_t T, d, p; } const heads[] = {{128, 768, 50257}, {128, 768, 50264}, {100, 2048, 128256}, {128, 768, 8192},
                                                         {50, 4096, 6000}, {128, 770, 50257}};
            for (const auto& h : heads) {
                if (h.p * B * h.T > INT32_MAX) continue;
                bk_layer y{};
                y.kind = BK_LINEAR;
                y.T = h.T;
                y.d = h.d;
                y.p = h.p;
                y.x = fake(1);
                y.g = fake(2);
                const size_t w = bk_layer_norms_workspace_size(&y, 1, dt, B);
                g_ghost_wgs = 0;
                const bk_status st = bk_layer_norms(&y, 1, dt, B, static_cast<float*>(fake(3)), set_ws(w), w, nullptr);
                // at least 4 slices a sample, and towards 512 where 128-byte chunks allow 16 to a slice
                const int64_t epc = dt == BK_BF16 ? 64 : 32, ch = (h.d + epc - 1) / epc + (h.p + epc - 1) / epc;
                const int64_t want = B * std::min({(int64_t)64, ch / 16, 512 / B});
                if (st != BK_OK || g_ghost_wgs < want) {
                    std::fprintf(stderr, "column slices: dtype %d B=%lld T=%lld %lld -> %lld: %ld workgroups, %lld wanted\n", (int)dt,
                                 (long long)B, (long long)h.T, (long long)h.d, (long long)h.p, g_ghost_wgs, (long long)want);
                    return 1;
                }
            }
        }
    // clipped gradients of few tiles over many samples are cut into K slices,
    // also past the 256 x 256 kernels' weight table
    for (int64_t B : {bk::kDMaxB, bk::kDMaxB + 1, 2 * bk::kDMaxB})
        for (int64_t T : {64, 70, 150})
            for (int64_t d : {256, 264, 768}) {
                const size_t w = bk_workspace_size(BK_OP_WEIGHTED_GRAD, BK_BF16, B, T, d, 256);
                float* out = static_cast<float*>(fake(3));
                if (bk_weighted_grad(fake(1), fake(2), out, BK_BF16, B, T, d, 256, out, set_ws(w), w, nullptr) != BK_OK || g_gemm_wgs < 128) {
                    std::fprintf(stderr, "B=%lld T=%lld %lld -> 256: %ld workgroups\n", (long long)B, (long long)T, (long long)d, g_gemm_wgs);
                    return 1;
                }
            }
    // a narrow layer of few tokens beside layers on the flat 256 x 256 tiles
    {
        bk_layer L[2] = {};
        for (int l = 0; l < 2; ++l) {
            L[l].T = 50;
            L[l].d = l ? 768 : 1000;
            L[l].p = l ? 5000 : 64;
            L[l].x = fake(3 * l + 1);
            L[l].g = fake(3 * l + 2);
            L[l].G = static_cast<float*>(fake(3 * l + 3));
        }
        const size_t w = bk_weighted_grads_workspace_size(L, 2, BK_BF16, 256);
        g_gemm_min_wgs = 0;
        if (bk_weighted_grads(L, 2, static_cast<float*>(fake(20)), BK_BF16, 256, set_ws(w), w, nullptr) != BK_OK || g_gemm_min_wgs < 64) {
            std::fprintf(stderr, "narrow layer beside flat ones: %ld workgroups\n", g_gemm_min_wgs);
            return 1;
        }
    }
    // many flat tiles of few rows: the 256 x 128 tiles
    for (int64_t B : {7, 511, 512}) {
        const size_t w = bk_workspace_size(BK_OP_WEIGHTED_GRAD, BK_BF16, B, 1, 3072, 3072);
        float* out = static_cast<float*>(fake(3));
        if (bk_weighted_grad(fake(1), fake(2), out, BK_BF16, B, 1, 3072, 3072, out, set_ws(w), w, nullptr) != BK_OK ||
            g_gemm_variant != (B < 512 ? bk::GemmVariant::Wide : bk::GemmVariant::Grad)) {
            std::fprintf(stderr, "3072 x 3072 of %lld rows: kernel variant %d\n", (long long)B, (int)g_gemm_variant);
            return 1;
        }
    }
    // fp32 layers of different T: the largest tiles first, over all XCDs
    {
        bk_layer L[3] = {};
        for (int l = 0; l < 3; ++l) {
            L[l].T = l == 2 ? 300 : 40;
            L[l].d = L[l].p = 768;
            L[l].x = fake(3 * l + 1);
            L[l].g = fake(3 * l + 2);
            L[l].G = static_cast<float*>(fake(3 * l + 3));
        }
        for (int n : {2, 3}) {
            const size_t w = bk_weighted_grads_workspace_size(L, n, BK_F32, 16);
            if (bk_weighted_grads(L, n, static_cast<float*>(fake(20)), BK_F32, 16, set_ws(w), w, nullptr) != BK_OK ||
                (g_gemm_remap == -1) != (n == 3) || g_gemm_first_T != (n == 3 ? 300 : 40)) {
                std::fprintf(stderr, "fp32 layers of different T: deal %d, first T %d\n", g_gemm_remap, g_gemm_first_T);
                return 1;
            }
        }
    }
    // one or two odd rows in all
    for (int64_t B : {1, 2, 3}) {
        float* out = static_cast<float*>(fake(3));
        if (bk_weighted_grad(fake(1), fake(2), out, BK_BF16, B, 1, 1031, 128, out, nullptr, 0, nullptr) != BK_OK ||
            g_gemm_variant != (B < 3 ? bk::GemmVariant::Scalar : bk::GemmVariant::WideAny)) {
            std::fprintf(stderr, "%lld odd rows: kernel variant %d\n", (long long)B, (int)g_gemm_variant);
            return 1;
        }
    }
    // instantiated norms of a few columns by a few rows
    for (int64_t T : {33, 64}) {
        const size_t w = bk_workspace_size(BK_OP_INST_NORM, BK_BF16, 4096, T, 64, 2);
        if (bk_inst_norm(fake(1), fake(2), BK_BF16, 4096, T, 64, 2, static_cast<float*>(fake(3)), set_ws(w), w, nullptr) != BK_OK ||
            g_gemm_variant != (T == 33 ? bk::GemmVariant::Scalar : bk::GemmVariant::WideAny)) {
            std::fprintf(stderr, "64 -> 2 at %lld tokens: kernel variant %d\n", (long long)T, (int)g_gemm_variant);
            return 1;
        }
    }
    // fp32 calls of few rows: the register-transposing kernel
    {
        struct { int64_t B, T, d, p; bk::GemmVariant v; } const cs[] = {
            {4, 16, 64, 64, bk::GemmVariant::Vec},        {64, 1, 4096, 4096, bk::GemmVariant::Vec},
            {1, 96, 1024, 1024, bk::GemmVariant::Vec},    {1, 65, 4096, 4096, bk::GemmVariant::F32},
            {1, 97, 64, 64, bk::GemmVariant::F32},        {64, 1, 65, 63, bk::GemmVariant::Scalar},
            {65, 1, 65, 63, bk::GemmVariant::F32Any},     {4, 16, 4097, 4095, bk::GemmVariant::F32Any}};
        for (const auto& c : cs) {
            const size_t w = bk_workspace_size(BK_OP_WEIGHTED_GRAD, BK_F32, c.B, c.T, c.d, c.p);
            float* out = static_cast<float*>(fake(3));
            if (bk_weighted_grad(fake(1), fake(2), out, BK_F32, c.B, c.T, c.d, c.p, out, set_ws(w), w, nullptr) != BK_OK || g_gemm_variant != c.v) {
                std::fprintf(stderr, "fp32 B=%lld T=%lld %lld -> %lld: kernel variant %d\n", (long long)c.B, (long long)c.T, (long long)c.d, (long long)c.p, (int)g_gemm_variant);
                return 1;
            }
        }
    }
    // bf16 rows of every odd length share one launch
    {
        bk_layer L[3] = {};
        const int64_t p[3] = {2, 9, 1031};
        for (int l = 0; l < 3; ++l) {
            L[l].T = 100;
            L[l].d = 264;
            L[l].p = p[l];
            L[l].x = fake(3 * l + 1);
            L[l].g = fake(3 * l + 2);
            L[l].G = static_cast<float*>(fake(3 * l + 3));
        }
        const size_t w = bk_weighted_grads_workspace_size(L, 3, BK_BF16, 16);
        g_gemm_launches = 0;
        if (bk_weighted_grads(L, 3, static_cast<float*>(fake(20)), BK_BF16, 16, set_ws(w), w, nullptr) != BK_OK || g_gemm_launches != 1) {
            std::fprintf(stderr, "unaligned bf16 gradients: %ld launches\n", g_gemm_launches);
            return 1;
        }
    }
    // The workspace of the full batch serves every smaller one, for stacks
    // without bf16 instantiated layers, and its size never falls as B grows.
    for (int it = 0; it < 400; ++it) {
        const bk_dtype dt = rng() % 3 ? BK_BF16 : BK_F32;
        const int n = 1 + (int)(rng() % 6);
        std::vector<bk_layer> L((size_t)n);
        for (int l = 0; l < n; ++l) {
            bk_layer& y = L[(size_t)l];
            const int r = (int)(rng() % 10);
            y.kind = r < 8 ? BK_LINEAR : r < 9 ? BK_EMBEDDING : BK_NORM_AFFINE;
            do {
                y.T = pick({1, 2, 16, 37, 50, 64, 100, 128, 130, 197, 256, 300, 600, 1024});
                y.p = pick({8, 60, 256, 264, 768, 1000, 3072, 4099, 8192, 50257});
                y.d = y.kind == BK_EMBEDDING ? 50257 : y.kind == BK_NORM_AFFINE ? y.p : pick({8, 60, 264, 768, 1001, 4096});
            } while (y.kind == BK_LINEAR && dt == BK_BF16 && !bk_use_ghost(y.T, y.d, y.p));
            const bool mis = rng() % 6 == 0;
            y.x = fake(4 * l + 1, mis && y.kind != BK_EMBEDDING);
            y.g = fake(4 * l + 2, mis);
            y.G = static_cast<float*>(fake(4 * l + 3));
            y.flags = 0;
            if (y.kind != BK_EMBEDDING && rng() % 3 == 0) {
                y.flags |= BK_LAYER_BIAS;
                y.Gb = static_cast<float*>(fake(0x100000 + l));
                y.Pb = static_cast<float*>(fake(0x200000 + l));
            }
            if (y.kind == BK_NORM_AFFINE) y.P = static_cast<float*>(fake(0x300000 + l));
        }
        float* norm = static_cast<float*>(fake(0x400000));
        float* C = static_cast<float*>(fake(0x400001));
        const int64_t full = pick({16, 63, 64, 65, 128, 512, 600, 4096});
        const size_t w = bk_private_grad_workspace_size(L.data(), n, dt, full);
        size_t more = w;
        for (int64_t B = full; B >= 0; B -= B > 700 ? 1 + (int64_t)(rng() % 400) : B > 80 ? 1 + (int64_t)(rng() % 40) : 1) {
            const size_t need = bk_private_grad_workspace_size(L.data(), n, dt, B);
            if (need > more) {
                std::fprintf(stderr, "workspace grows as the batch shrinks (full %lld): %zu at B=%lld, %zu just above\n", (long long)full, need, (long long)B, more);
                for (const bk_layer& y : L)
                    std::fprintf(stderr, "  dtype %d kind %d T=%lld %lld -> %lld flags %d\n", (int)dt, y.kind, (long long)y.T, (long long)y.d, (long long)y.p, y.flags);
                return 1;
            }
            more = need;
            const bk_status st = bk_private_grad(L.data(), n, dt, B, BK_CLIP_AUTO, 1.f, 0.01f, 0.f, 7, 0, norm, C, nullptr, set_ws(w), w, nullptr);
            if (st != BK_OK) {
                std::fprintf(stderr, "B=%lld on the workspace of B=%lld: %s\n", (long long)B, (long long)full, bk_last_error());
                return 1;
            }
        }
    }
    // few tokens of long rows whose pairs get no slices stay on the few-token
    // kernel (32 / T samples to a workgroup)
    for (const bk_dtype dt : {BK_BF16, BK_F32}) {
        bk_layer y{};
        y.kind = BK_LINEAR;
        y.T = 2;
        y.d = y.p = 8192;
        y.x = fake(1);
        y.g = fake(2);
        const size_t w = bk_layer_norms_workspace_size(&y, 1, dt, 200);
        g_ghost_wgs = 0;
        if (bk_layer_norms(&y, 1, dt, 200, static_cast<float*>(fake(3)), set_ws(w), w, nullptr) != BK_OK || g_ghost_wgs != 13) {
            std::fprintf(stderr, "few tokens of long rows: %ld workgroups\n", g_ghost_wgs);
            return 1;
        }
    }
    // few-token layers beside layers of the pair kernel leave it its slices
    {
        bk_layer L[8] = {};
        for (int l = 0; l < 8; ++l) {
            L[l].T = l < 4 ? 49 : 200;
            L[l].d = l < 4 ? 512 : 768;
            L[l].p = l < 4 ? 512 : 3072;
            L[l].x = fake(2 * l + 1);
            L[l].g = fake(2 * l + 2);
        }
        const size_t w = bk_layer_norms_workspace_size(L, 8, BK_F32, 4);
        g_ghost_wgs = 0;
        if (bk_layer_norms(L, 8, BK_F32, 4, static_cast<float*>(fake(40)), set_ws(w), w, nullptr) != BK_OK || g_ghost_wgs < 4 * 48) {
            std::fprintf(stderr, "pair kernel beside few tokens: %ld workgroups\n", g_ghost_wgs);
            return 1;
        }
    }
    // small calls: samples of few and of more tokens in one launch (fp32: two)
    for (const bk_dtype dt : {BK_BF16, BK_F32}) {
        bk_layer L[4] = {};
        for (int l = 0; l < 4; ++l) {
            L[l].T = l == 0 ? 5 : l == 1 ? 50 : l == 2 ? (dt == BK_F32 ? 80 : 20) : (dt == BK_F32 ? 120 : 33);
            L[l].d = L[l].p = 768;
            L[l].x = fake(2 * l + 1);
            L[l].g = fake(2 * l + 2);
        }
        const size_t w = bk_layer_norms_workspace_size(L, 4, dt, 16);
        g_ghost_launches = 0;
        if (bk_layer_norms(L, 4, dt, 16, static_cast<float*>(fake(40)), set_ws(w), w, nullptr) != BK_OK || g_ghost_launches != (dt == BK_F32 ? 2 : 1)) {
            std::fprintf(stderr, "few and more tokens: %ld launches\n", g_ghost_launches);
            return 1;
        }
    }
    // the fused reduction's grid covers every sample once, threads past the
    // batch stay past it, up to the largest batch
    for (int64_t B : {(int64_t)1, (int64_t)255, (int64_t)257, (int64_t)INT32_MAX - 255, (int64_t)INT32_MAX})
        for (int n : {1, 2, 3, 85, 129, bk::kMaxReduce}) {
            const int per = bk::kReducePairs / n;
            const int64_t wgs = bk::reduce_clip_wgs(n, B);
            const int64_t first = bk::reduce_clip_sample((uint32_t)(wgs - 1), per, 0);
            const int64_t last = bk::reduce_clip_sample((uint32_t)(wgs - 1), per, 2 * per - 1);
            if (first >= B || first + per < B || last != first + per - 1 || per * n > bk::kReducePairs) {
                std::fprintf(stderr, "fused reduction grid: B=%lld n=%d\n", (long long)B, n);
                return 1;
            }
        }
    {   // grouped noise over many tensors (more than one launch's table)
        std::vector<float*> G(400);
        std::vector<int64_t> nel(400);
        std::vector<uint32_t> tid(400);
        for (size_t k = 0; k < G.size(); ++k) {
            G[k] = static_cast<float*>(fake(0x500000 + k));
            nel[k] = pick({0, 1, 3, 1000, 1 << 22});
            tid[k] = (uint32_t)k;
        }
        (void)bk_add_noise_grouped(G.data(), nel.data(), tid.data(), (int64_t)G.size(), 1.f, 9, 1, nullptr);
    }
    {   // convolution preparation
        for (int it = 0; it < 500; ++it) {
            const int n = 1 + (int)(rng() % 30);
            std::vector<bk_conv> cv((size_t)n);
            for (int l = 0; l < n; ++l) {
                bk_conv& c = cv[(size_t)l];
                c.x = rng() % 4 ? fake(0x600000 + l) : nullptr;
                c.dy = rng() % 4 ? fake(0x700000 + l) : nullptr;
                c.a = fake(0x800000 + l);
                c.g = fake(0x900000 + l);
                c.C = pick({1, 3, 64, 512});
                c.H = c.W = pick({1, 7, 14, 56, 224});
                c.kh = c.kw = pick({1, 3, 7});
                c.stride = pick({1, 2});
                c.pad = pick({0, 1, 3});
                c.ld = c.C * c.kh * c.kw + pick({0, 5});
                c.p = pick({1, 64, 512});
            }
            (void)bk_conv_prep(cv.data(), n, (bk_dtype)(rng() % 2), pick({1, 16}), nullptr);
        }
    }
    std::printf("ok: %d stacks (%d with valid norms), %ld launches checked\n", calls, ok_calls, g_launches);
    return 0;
}
