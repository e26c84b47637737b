// Kernels of each grid length, as launchers: the variants that the autotuner
// chooses from.  They are compiled in several translation units
// (pstd_variants.hip, one per group of lengths), which build side by side.
#pragma once
#include "pstd_kernels.hpp"

namespace pstd {

constexpr int NT = 256;

// Tuning knobs (the autotuner picks one value of each per context): the
// column-tile width of the y and z kernels and the threads per block of the
// two update kernels.
using VelFn = void (*)(dim3, hipStream_t, Geo, Mat, Pml, const float2*, float*, float2*, Rec, float*, const int*,
                       int*, int, int);
using StrFn = void (*)(dim3, hipStream_t, Geo, Mat, Pml, const float2*, float*, float2*, Rec, Inj, float*,
                       const int*, int, int);
struct XFns {
    void (*xfwd)(dim3, hipStream_t, Geo, const float2*, const float*, long, float2*, long, SumDesc);
    void (*xinv)(dim3, hipStream_t, Geo, const float2*, const float2*, float*);
    int rows;
};
struct VelVar {
    VelFn fn;
    int nt;
};
struct StrVar {
    StrFn fn;
    StrFn visc;   // the Kelvin-Voigt variant
    int nt;
};
struct YFns {
    void (*fwd)(dim3, hipStream_t, Geo, const float2*, float2*, int, int);
    void (*inv)(dim3, hipStream_t, Geo, const float2*, float2*, const ZDesc*, int, int);
    int tile;
};
struct ZFns {
    void (*op)(dim3, hipStream_t, Geo, const float2*, float2*, int, const ZDesc*, int, int);
    int tile;
    int nt;     // threads per block
};
constexpr int MAX_VARIANTS = 8;

// everything built for one length
struct Variants {
    XFns x;
    VelVar vel[3];
    StrVar str[3];
    int nx = 0;            // update kernel variants
    YFns y[MAX_VARIANTS];
    int ny = 0;
    ZFns z[MAX_VARIANTS];
    int nz = 0;
    const void* probe = nullptr;   // a kernel of the group
};

// the groups' tables (false: length not in the group)
bool variants_0(int n, Variants* v);
bool variants_1(int n, Variants* v);
bool variants_2(int n, Variants* v);
bool variants_3(int n, Variants* v);
bool variants_4(int n, Variants* v);
bool variants_5(int n, Variants* v);
bool variants_6(int n, Variants* v);
bool variants_7(int n, Variants* v);

// false: length not built
inline bool find_variants(int n, Variants* v)
{
    return variants_0(n, v) || variants_1(n, v) || variants_2(n, v) || variants_3(n, v) || variants_4(n, v) ||
           variants_5(n, v) || variants_6(n, v) || variants_7(n, v);
}

}  // namespace pstd
