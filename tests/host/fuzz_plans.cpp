// Host-side planning code under AddressSanitizer / UBSan: random layer geometries through the
// planners of the product kernels and through every workspace-size query and entry point of the C
// ABI (with placeholder pointers; without a GPU every call ends before a launch).  Checks the
// invariants the kernels rely on.  Usage: fuzz_plans [cases] [seed]; or fuzz_plans route followed by the
// eleven numbers of a layer's descriptor, any number of times: which kernel computes it, fp32 and packed-sign output;
// or plan and the same numbers: the kernel of the fp32 form and what its plan chose;
// or wbin and the same numbers: the form of the weights-only layer.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <utility>

#include "dab_internal.h"
#include "wbin.h"

namespace {

uint64_t g_state = 1;
uint32_t rnd(uint32_t n) {   // 0 .. n-1
    g_state = g_state * 6364136223846793005ull + 1442695040888963407ull;
    return static_cast<uint32_t>((g_state >> 33) % n);
}
int pick(int lo, int hi) { return lo + static_cast<int>(rnd(static_cast<uint32_t>(hi - lo + 1))); }

#define REQUIRE(cond) \
    do { \
        if (!(cond)) { \
            std::fprintf(stderr, "invariant failed: %s  (B=%d C=%d H=%d W=%d F=%d k=%dx%d pad=%d,%d stride=%d,%d)\n", #cond, d.B, d.C, \
                         d.H, d.W, d.F, d.kh, d.kw, d.pad_h, d.pad_w, d.stride_h, d.stride_w); \
            return 1; \
        } \
    } while (0)

int check_one(const dab_conv_desc& d) {
    using namespace dab;
    const long long Ho = (d.H + 2ll * d.pad_h - d.kh) / d.stride_h + 1, Wo = (d.W + 2ll * d.pad_w - d.kw) / d.stride_w + 1;
    const long long M = 1ll * d.B * Ho * Wo;
    DirectPlan dp;
    if (plan_direct(d, &dp)) {
        const DirectGeom& g = dp.g;
        REQUIRE(dp.lw == 1 || dp.lw == 2 || dp.lw == 4);
        REQUIRE((dp.lw == 1 && (dp.pf == 5 || dp.pf == 6)) || (dp.lw == 2 && (dp.pf == 3 || dp.pf == 4)) ||
                (dp.lw == 4 && (dp.pf == 2 || dp.pf == 3)));
        REQUIRE(dp.waves == 4 || dp.waves == 8);
        REQUIRE(g.M == M && g.Wo == Wo && g.HoWo == Ho * Wo);
        REQUIRE(g.G * dp.lw == g.WH && g.NG == g.T * g.G && g.WH == (g.Cw + 1) / 2);
        REQUIRE(g.n_ent >= g.nk + 1 && g.n_ent <= 37 && (g.n_ent - 1) % (dp.pf * dp.lw) == 0);
        REQUIRE(dp.lds_bytes == static_cast<size_t>(g.n_ent) * 4096 && dp.lds_bytes <= 160 * 1024 - 8192);
        REQUIRE(1ll * g.n_mtiles * 64 * dp.waves >= M && 1ll * (g.n_mtiles - 1) * 64 * dp.waves < M);
        REQUIRE(dp.grid >= 1 && dp.grid <= 4096 && g.wg_per_ntile >= 1 && g.wg_per_ntile <= g.n_mtiles);
        REQUIRE(1ull * g.y_bytes == 4ull * static_cast<unsigned long long>(M) * static_cast<unsigned long long>(d.F));
        REQUIRE(1ull * g.a_bytes == 4ull * d.B * d.H * d.W * g.Cw);
        REQUIRE(!dp.pad || g.T <= 32);
        // the offsets that drop a load or a store lie past the tensors
        REQUIRE(g.y_bytes <= kOobStore && g.a_bytes <= (1u << 30));
    }
    for (int large = 0; large < 2; ++large) {
        BlockPlan bp;
        if (plan_block(d, &bp, large != 0)) {
            REQUIRE(bp.waves == 2 || bp.waves == 4 || bp.waves == 8);
            REQUIRE(bp.g.M == M);
            const long long blocks = 1ll * ((M + 31) / 32) * ((d.F + 31) / 32);
            REQUIRE(bp.bg.n_mblocks == (M + 31) / 32 && bp.bg.units == blocks);
            REQUIRE(8ll * bp.bg.per_xcd >= blocks && 8ll * (bp.bg.per_xcd - 1) < blocks);
            REQUIRE(1ull * bp.grid == 8ull * bp.bg.per_xcd);
            REQUIRE(blocks <= (large ? 8192 : 512) && (!large || blocks * bp.g.nk <= 400000));
            // the load burst: whole loads, and a kernel exists for the combination
            REQUIRE(bp.lw == 1 || (bp.lw == 4 && bp.g.Cw % 8 == 0));
            REQUIRE(bp.depth % bp.lw == 0);
            REQUIRE((bp.lw == 1 && (bp.depth == 4 || ((bp.depth == 8 || bp.depth == 13) && bp.waves == 8))) ||
                    (bp.lw == 4 && (bp.depth == 4 || ((bp.depth == 8 || bp.depth == 16) && bp.waves == 8))));
            REQUIRE(1ll * d.C * d.kh * d.kw < (1ll << 24));
        }
    }
    SplitPlan sp;
    if (plan_split(d, &sp)) {
        const SplitGeom& sg = sp.sg;
        const int ks = 1 << sg.log_ks, tile = 64 * (8 / ks);
        REQUIRE(sp.lw == 1 || sp.lw == 2 || sp.lw == 4);
        REQUIRE(sg.log_ks >= 0 && sg.log_ks <= 3 && 1ll * sg.groups_per_share * ks >= sp.g.NG);
        REQUIRE(sp.g.G * sp.lw == sp.g.WH && sp.g.NG == sp.g.T * sp.g.G && (sp.lw == 1 || sp.g.Cw == 2 * sp.g.WH));
        REQUIRE(1ll * sg.n_mtiles * tile >= M && 1ll * (sg.n_mtiles - 1) * tile < M);
        REQUIRE(1ll * sg.units == 1ll * sg.n_mtiles * ((d.F + 127) / 128));
        REQUIRE(sp.grid == 8u * static_cast<unsigned>(sg.per_xcd) && 8ll * sg.per_xcd >= sg.units);
        REQUIRE(1ull * sg.e_bytes == 4ull * sp.g.T * sp.g.Cw * sp.g.Fp && sg.e_bytes < (1u << 30));
        REQUIRE(sp.g.a_bytes <= (1u << 30));
        REQUIRE((sg.narrow != 0) == (ks > 1 && 1ll * d.C * d.kh * d.kw < (1 << 15)));    // (a sum of 2^15 terms has no 16 bits)
        REQUIRE(sp.lds_bytes == (ks > 1 ? 131072u : 0u));
        REQUIRE(!sp.pad || sp.g.T <= 32);
        REQUIRE(1ll * d.C * d.kh * d.kw < (1ll << 24));
    }
    size_t wneed = 0;
    if (wbin_workspace(d, &wneed) == DAB_OK) {
        WbinPlan wp;
        plan_wbin(d, &wp);
        const WbinGeom& g = wp.g;
        const int pixels = wp.form.rows ? wp.form.rows * 8 / wp.form.v : 32 * wp.form.v;
        const int filters = wp.form.rows ? wp.form.rows * wp.form.nb : 32 * wp.form.nb * (4 / wp.form.v);
        REQUIRE(g.M == M && wp.lds_bytes <= static_cast<size_t>(kWbinMaxLds));
        REQUIRE(g.n_ntiles == (d.F + filters - 1) / filters && 1ll * g.units == (M + pixels - 1) / pixels * g.n_ntiles);
        REQUIRE(wp.grid == 8u * static_cast<unsigned>(g.per_xcd) && 8ll * g.per_xcd >= g.units);
        REQUIRE(1ull * g.x_bytes == 4ull * d.B * d.H * d.W * d.C && g.x_bytes < (1u << 31));
        REQUIRE(1ull * g.e_bytes == 4ull * g.T * g.Cw * g.Fp && g.e_bytes < (1u << 31));
        if (wp.form.rows == 0) {
            // every tile's pixels fit the patch (tiles near image ends and a few hundred others)
            const long long tiles = (M + pixels - 1) / pixels, step = tiles > 300 ? tiles / 300 : 1;
            auto padded = [&](long long m) {
                const long long b = m / g.HoWo, r = m % g.HoWo;
                return (b * g.Hp + r / g.Wo * g.sh) * g.Wp + r % g.Wo * g.sw;
            };
            for (long long t = 0; t < tiles; t += step) {
                const long long last = t * pixels + pixels < M ? t * pixels + pixels : M;
                const long long np = padded(last - 1) + 1ll * (g.kh - 1) * g.Wp + g.kw - padded(t * pixels);
                REQUIRE(np <= 64 * kPatchSlots && 8 * 64 * kPatchSlots + 4 * pixels <= 96 * 64 * kPatchSlots);
            }
        }
    }
    // the public queries and entry points: any status is fine, a crash or a sanitizer report is not
    void* fake = reinterpret_cast<void*>(0x1000);
    const size_t ws = dab_binconv2d_workspace_bytes(&d);
    const size_t wws = dab_wbin_conv2d_workspace_bytes(&d);
    REQUIRE(ws % 256 == 0 && wws % 256 == 0);
    int st = dab_binconv2d(&d, static_cast<const uint32_t*>(fake), static_cast<const uint32_t*>(fake), static_cast<const float*>(fake),
                           static_cast<const float*>(fake), static_cast<float*>(fake), nullptr, ws ? fake : nullptr, ws, nullptr);
    REQUIRE(st >= DAB_OK && st <= DAB_ERR_HIP);
    st = dab_binconv2d_bits(&d, static_cast<const uint32_t*>(fake), static_cast<const uint32_t*>(fake), static_cast<const float*>(fake),
                            static_cast<const float*>(fake), nullptr, static_cast<uint32_t*>(fake), nullptr, 0, nullptr);
    REQUIRE(st >= DAB_OK && st <= DAB_ERR_HIP);
    if (d.H == 1 && d.W == 1 && d.kh == 1 && d.kw == 1) {
        REQUIRE(dab_binfc_workspace_bytes(d.B, d.C, d.F) == ws);
        REQUIRE(dab_wbin_fc_workspace_bytes(d.B, d.C, d.F) % 256 == 0);
    }
    const long long n = 1ll * d.C * d.kh * d.kw;
    if (n < (1ll << 31)) {
        (void)dab_estimate_workspace_bytes(d.F, static_cast<int32_t>(n));
        dab_weight_job job{};
        job.W = static_cast<const float*>(fake); job.F = d.F; job.C = d.C; job.kh = d.kh; job.kw = d.kw;
        job.alpha = job.beta = job.thr_val = static_cast<float*>(fake);
        job.K = job.thr_idx = static_cast<int32_t*>(fake);
        job.alpha_is_upper = static_cast<uint8_t*>(fake);
        const size_t jws = dab_binarize_weights_multi_workspace_bytes(&job, 1);
        REQUIRE(jws == 0 || (n > 4608 && jws >= static_cast<size_t>(d.F)));
        st = dab_binarize_weights_multi(&job, 1, nullptr, 0, nullptr);
        REQUIRE(st >= DAB_OK && st <= DAB_ERR_HIP);
    }
    dab_pack_job pj{static_cast<const float*>(fake), nullptr, static_cast<uint32_t*>(fake), d.B, d.C, d.H, d.W};
    st = dab_pack_activations_multi(&pj, 1, nullptr);
    REQUIRE(st >= DAB_OK && st <= DAB_ERR_HIP);
    return 0;
}

}  // namespace

int main(int argc, char** argv) {
    if (argc > 1 && std::strcmp(argv[1], "wbin") == 0) {
        for (int a = 2; a + 11 <= argc; a += 11) {
            int32_t v[11];
            for (int i = 0; i < 11; ++i) v[i] = std::atoi(argv[a + i]);
            dab::WbinPlan p;
            dab::plan_wbin(dab_conv_desc{v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8], v[9], v[10]}, &p);
            std::printf("%d,%d,%d\n", p.form.rows, p.form.nb, p.form.v);
        }
        return 0;
    }
    if (argc > 1 && std::strcmp(argv[1], "route") == 0) {
        static const char* const names[] = {"block", "direct", "split", "expanded"};
        for (int a = 2; a + 11 <= argc; a += 11) {
            int32_t v[11];
            for (int i = 0; i < 11; ++i) v[i] = std::atoi(argv[a + i]);
            const dab_conv_desc d{v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8], v[9], v[10]};
            for (const bool bits : {false, true}) {
                dab::Product which;
                if (dab::product_of(d, bits, &which) != DAB_OK) return 1;
                std::printf("%s%c", names[static_cast<int>(which)], bits ? '\n' : ' ');
            }
        }
        return 0;
    }
    if (argc > 1 && std::strcmp(argv[1], "plan") == 0) {
        static const char* const stores[] = {"plain", "through", "streamed"};
        for (int a = 2; a + 11 <= argc; a += 11) {
            int32_t v[11];
            for (int i = 0; i < 11; ++i) v[i] = std::atoi(argv[a + i]);
            const dab_conv_desc d{v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8], v[9], v[10]};
            dab::Product which;
            dab::DirectPlan dp;
            dab::SplitPlan sp;
            dab::BlockPlan bp;
            if (dab::product_of(d, false, &which) != DAB_OK) return 1;
            if (which == dab::Product::kDirect && dab::plan_direct(d, &dp)) std::printf("direct %s\n", stores[dp.g.store_policy]);
            else if (which == dab::Product::kSplit && dab::plan_split(d, &sp))
                std::printf("split w%d s%d %s\n", sp.lw, 1 << sp.sg.log_ks, !sp.sg.log_ks ? "alone" : sp.sg.narrow ? "16-bit" : "fp32");
            else if (which == dab::Product::kBlock && dab::plan_block(d, &bp, true))
                std::printf("block w%d s%d depth%d\n", bp.lw, bp.waves, bp.depth);
            else std::printf("expanded\n");
        }
        return 0;
    }
    // outputs of 2^29 - 1, - 2 and - 4 values, the largest that the persistent kernel takes, and one that it does not
    for (const auto& [B, F] : {std::pair{2304167, 233}, {4227330, 127}, {4194303, 128}, {4194304, 128}}) {
        const dab_conv_desc d{B, 32, 1, 1, F, 1, 1, 0, 0, 1, 1};
        dab::DirectPlan dp;
        REQUIRE(dab::plan_direct(d, &dp) == (1ll * B * F < (1ll << 29)));
        if (check_one(d)) return 1;
    }
    const int cases = argc > 1 ? std::atoi(argv[1]) : 20000;
    g_state = argc > 2 ? static_cast<uint64_t>(std::atoll(argv[2])) * 2 + 1 : 1;
    int planned = 0;
    for (int it = 0; it < cases; ++it) {
        dab_conv_desc d{};
        const int shape = static_cast<int>(rnd(4));
        d.B = shape == 0 ? pick(1, 8) : (shape == 1 ? pick(1, 300) : pick(1, 5000));
        d.C = rnd(3) == 0 ? 32 * pick(1, 40) : pick(1, 1300);
        d.F = rnd(3) == 0 ? 64 * pick(1, 16) : pick(1, 1300);
        if (rnd(4) == 0) {                       // fully connected
            d.H = d.W = d.kh = d.kw = 1; d.stride_h = d.stride_w = 1;
            d.C = rnd(2) ? pick(2, 20000) : 64 * pick(1, 300);
        } else {
            d.H = pick(1, 70); d.W = pick(1, 70);
            d.kh = pick(1, 7); d.kw = pick(1, 7);
            d.pad_h = pick(0, 4); d.pad_w = pick(0, 4);             // (also beyond the kernel extent)
            d.stride_h = pick(1, 3); d.stride_w = pick(1, 3);
        }
        if (rnd(50) == 0) d.B = 0;               // an invalid descriptor now and then
        if (rnd(50) == 0) d.kh = d.H + 2 * d.pad_h + 1;
        const bool valid = d.B >= 1 && d.kh <= d.H + 2 * d.pad_h && d.kw <= d.W + 2 * d.pad_w &&
                           1ll * d.C * d.kh * d.kw >= 2;
        if (!valid) {
            // entry points must refuse it, whatever else
            void* fake = reinterpret_cast<void*>(0x1000);
            const int st = dab_binconv2d(&d, static_cast<const uint32_t*>(fake), static_cast<const uint32_t*>(fake),
                                         static_cast<const float*>(fake), static_cast<const float*>(fake), static_cast<float*>(fake),
                                         nullptr, nullptr, 0, nullptr);
            if (st == DAB_OK) { std::fprintf(stderr, "an invalid descriptor was accepted\n"); return 1; }
            (void)dab_binconv2d_workspace_bytes(&d);
            continue;
        }
        if (check_one(d)) return 1;
        ++planned;
    }
    std::printf("%d geometries checked\n", planned);
    return 0;
}
