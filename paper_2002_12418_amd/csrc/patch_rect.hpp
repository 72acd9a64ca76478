// The rectangle of output pixels that a workgroup of the sliding-window kernels owns, and the patch of the image it sees.
#pragma once
#include "kernels.hpp"

namespace mnnconv {

struct PatchRect {
    int ni, ty, tx;              // output rectangle: images x rows x columns
    int ph, pw;                  // its patch, per image
    int pws;                     // a patch row is stored as stride_w runs of pws pixels, so that a run holds what consecutive columns read
    int pp, ppr;                 // slots and pixels of the patch, all images
    int tilesX, tilesY;
    int vecD;                    // four columns from a multiple of four on are four floats in a row (conv_patch.hip: and 16-byte aligned)
};

// As few workgroups as `bn` columns allow, then (wide_stores) 16-byte stores, then the smallest patch of at most max_px pixels and max_pp slots.
// False where no patch fits.
inline bool choose_patch_rect(const GemmProblem& p, int bn, int max_px, int max_pp, bool wide_stores, PatchRect* out)
{
    const int Ho = p.L / p.cv_Wo, Wo = p.cv_Wo, N = p.Ncols / p.L;
    bool found = false;
    long long best = 0;
    auto consider = [&](int ni, int ty, int tx) {
        PatchRect a{};
        a.ni = ni; a.ty = ty; a.tx = tx;
        const long long ph = (long long)(ty - 1) * p.cv_sh + (long long)(p.cv_kh - 1) * p.cv_dh + 1;
        const long long pw = (long long)(tx - 1) * p.cv_sw + (long long)(p.cv_kw - 1) * p.cv_dw + 1;
        if (ph > max_px || pw > max_px || ni * ph * pw > max_px) return;
        a.ph = (int)ph; a.pw = (int)pw;
        a.pws = (a.pw + p.cv_sw - 1) / p.cv_sw;
        a.ppr = ni * a.ph * a.pw;
        a.pp = ni * a.ph * a.pws * p.cv_sw;
        if (a.pp > max_pp) return;
        a.tilesX = (Wo + tx - 1) / tx;
        a.tilesY = (Ho + ty - 1) / ty;
        const long long tiles = (long long)a.tilesX * a.tilesY * ((N + ni - 1) / ni);
        // runs of columns, a row of the rectangle or all its rows where they span the plane, that 16-byte stores can take
        a.vecD = (tx == Wo ? ty * tx % 4 == 0 && p.L % 4 == 0 : tx % 4 == 0 && Wo % 4 == 0) ? 1 : 0;
        const int wide = wide_stores ? a.vecD - out->vecD : 0;
        if (found && (tiles > best || (tiles == best && (wide < 0 || (wide == 0 && a.pp >= out->pp))))) return;
        found = true;
        best = tiles;
        *out = a;
    };
    auto level = [](int size, int most) { const int parts = (size + most - 1) / most; return (size + parts - 1) / parts; };
    if ((long long)Ho * Wo <= bn) consider(level(N, bn / (Ho * Wo)), Ho, Wo);
    const int least = (Wo + bn - 1) / bn;                 // columns of rectangles
    for (int parts = least; parts < least + 12; ++parts) {
        const int tx = (Wo + parts - 1) / parts;
        consider(1, level(Ho, bn / tx), tx);
        if (tx <= 4) break;
    }
    return found;
}

}  // namespace mnnconv
