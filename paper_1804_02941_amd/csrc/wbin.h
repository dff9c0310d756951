// The weights-only layer's plan and launch (wbin.hip).
#pragma once

#include "dab_internal.h"

namespace dab {

constexpr int kWbinMaxLds = 160 * 1024;
constexpr int kPatchSlots = 8;     // 16-byte pieces of the fp32 patch a thread carries: a patch is at most 64 times as many pixels

struct WbinGeom {
    int H, W, C, Cw, C16, F, Fp, kh, kw, ph, pw, sh, sw;
    int Ho, Wo, HoWo, M, T, Hp, Wp;
    int n_ntiles, units, per_xcd;  // filter tiles, workgroups with work, those of one XCD
    uint32_t x_bytes, e_bytes;
    int stream_out;                // the output is larger than the chip's caches keep: streaming stores
    FastDiv d_HoWo, d_Wo, d_Wp, d_HpWp, d_kw, d_C16, d_Cw, d_ntiles;
};
// rows = 0, the patch kernel: wavefronts of 32 pixels x 32 nb filters, v of a workgroup's four along the pixels.
// Otherwise the direct kernel: rows pixels x rows nb filters a wavefront, v of a workgroup's eight share the reduction.
struct WbinForm {
    int rows, nb, v;
};
struct WbinPlan {
    WbinGeom g;
    WbinForm form;
    double us;                     // estimated time of the launch
    unsigned grid;
    size_t lds_bytes;
};
int wbin_workspace(const dab_conv_desc& d, size_t* bytes);
void plan_wbin(const dab_conv_desc& d, WbinPlan* pl);
int launch_wbin(const WbinPlan& pl, hipStream_t st, const float* X, const uint32_t* E, const float* alpha, const float* beta,
                float* Y);
int init_wbin();

}  // namespace dab
