// Variants of one group of grid lengths (PSTD_GROUP, 0 .. 7):
// compiled once per group.  All lengths factor into 2, 3 and 5.
#include "pstd_variants.hpp"

#if PSTD_GROUP == 0
#define PSTD_LENGTHS(X) X(20) X(24) X(128) X(144) X(512)
#elif PSTD_GROUP == 1
#define PSTD_LENGTHS(X) X(16) X(30) X(125) X(150) X(480)
#elif PSTD_GROUP == 2
#define PSTD_LENGTHS(X) X(32) X(120) X(160) X(400)
#elif PSTD_GROUP == 3
#define PSTD_LENGTHS(X) X(40) X(100) X(180) X(384)
#elif PSTD_GROUP == 4
#define PSTD_LENGTHS(X) X(48) X(96) X(192) X(360)
#elif PSTD_GROUP == 5
#define PSTD_LENGTHS(X) X(60) X(90) X(200) X(320)
#elif PSTD_GROUP == 6
#define PSTD_LENGTHS(X) X(64) X(80) X(240) X(300)
#elif PSTD_GROUP == 7
#define PSTD_LENGTHS(X) X(72) X(75) X(256) X(288)
#endif

namespace pstd {

namespace {

constexpr int N_TILES = 4;
constexpr int TILE_CANDIDATES[N_TILES] = {8, 16, 32, 64};

// Threads per block of the update kernels of length N: 128, 256 and 512, none
// above the cells of a block; up to length 48, whose blocks were halved
// (rows_for), none above the cells of twice the rows: a shape that a caller
// measured and kept with the taller blocks can still be forced
// (pstd3d_set_tuning).  There the largest count leaves up to half of its
// threads without a cell.
constexpr int nt_candidate(int n, int i)
{
    const int cells = (n <= 48 ? 2 : 1) * rows_for(n) * n;
    const int c[3] = {128, 256, 512};
    const int v = c[i];
    if (v > cells || v % 64 || v > 1024) return 0;
    for (int j = 0; j < i; ++j)
        if (c[j] == v) return 0;
    return v;
}

template <int N>
struct Launch {
    static void xfwd(dim3 gr, hipStream_t st, Geo g, const float2* tw, const float* in, long is, float2* out,
                     long os, SumDesc sd)
    {
        hipLaunchKernelGGL((k_xfwd<N, NT>), gr, dim3(NT), 0, st, g, tw, in, is, out, os, sd);
    }
    static void xinv(dim3 gr, hipStream_t st, Geo g, const float2* tw, const float2* in, float* out)
    {
        hipLaunchKernelGGL((k_xinv<N, NT>), gr, dim3(NT), 0, st, g, tw, in, out);
    }
};

template <int N, int T>
struct LaunchX {
    static void vel(dim3 gr, hipStream_t st, Geo g, Mat m, Pml p, const float2* tw, float* f, float2* s, Rec r,
                    float* tr, const int* sp, int* sn, int n0, int ldt)
    {
        const auto fn = g.stream ? k_vel<N, T, true> : k_vel<N, T, false>;
        hipLaunchKernelGGL(fn, gr, dim3(T), 0, st, g, m, p, tw, f, s, r, tr, sp, sn, n0, ldt);
    }
    template <bool VISC>
    static void str(dim3 gr, hipStream_t st, Geo g, Mat m, Pml p, const float2* tw, float* f, float2* s, Rec r,
                    Inj in, float* tr, const int* sp, int n0, int ldt)
    {
        const auto fn = g.stream ? k_str<N, T, VISC, true> : k_str<N, T, VISC, false>;
        hipLaunchKernelGGL(fn, gr, dim3(T), 0, st, g, m, p, tw, f, s, r, in, tr, sp, n0, ldt);
    }
};

template <int N, int I = 0>
void x_variants(VelVar* v, StrVar* s, int& n)
{
    if constexpr (I < 3) {
        constexpr int T = nt_candidate(N, I);
        if constexpr (T > 0) {
            v[n] = VelVar{LaunchX<N, T>::vel, T};
            s[n] = StrVar{LaunchX<N, T>::template str<false>, LaunchX<N, T>::template str<true>, T};
            ++n;
        }
        x_variants<N, I + 1>(v, s, n);
    }
}

template <int N, int TX>
struct LaunchYZ {
    static void yf(dim3 gr, hipStream_t st, Geo g, const float2* tw, float2* s, int f0, int nf)
    {
        hipLaunchKernelGGL((k_y<N, y_threads(N, TX), TX>), gr, dim3(y_threads(N, TX)), 0, st, g, tw, s, f0, nf);
    }
    static void yi(dim3 gr, hipStream_t st, Geo g, const float2* tw, float2* s, const ZDesc* zd, int ph, int nsrc)
    {
        hipLaunchKernelGGL((k_yinv<N, y_threads(N, TX), TX>), gr, dim3(y_threads(N, TX)), 0, st, g, tw, s, zd, ph, nsrc);
    }
    static void z(dim3 gr, hipStream_t st, Geo g, const float2* tw, float2* s, int in0, const ZDesc* zd, int ph,
                  int fpb)
    {
        hipLaunchKernelGGL((k_z<N, NT, TX>), gr, dim3(NT), 0, st, g, tw, s, in0, zd, ph, fpb);
    }
    static void z512(dim3 gr, hipStream_t st, Geo g, const float2* tw, float2* s, int in0, const ZDesc* zd, int ph,
                     int fpb)
    {
        hipLaunchKernelGGL((k_z<N, 512, TX, z_maxr(N, TX, 512)>), gr, dim3(512), 0, st, g, tw, s, in0, zd, ph, fpb);
    }
};

// the variants of length N: y tiles and z tiles (counts returned)
template <int N, int I = 0>
void yz_variants(YFns* y, int& ny, ZFns* z, int& nz)
{
    if constexpr (I < N_TILES) {
        constexpr int TX = TILE_CANDIDATES[I];
        if constexpr (y_tile_built(N, TX)) y[ny++] = YFns{LaunchYZ<N, TX>::yf, LaunchYZ<N, TX>::yi, TX};
        if constexpr (z_tile_built(N, TX)) z[nz++] = ZFns{LaunchYZ<N, TX>::z, TX, NT};
        if constexpr (z512_ok(N, TX)) z[nz++] = ZFns{LaunchYZ<N, TX>::z512, TX, 512};
        yz_variants<N, I + 1>(y, ny, z, nz);
    }
}

template <int N>
void fill(Variants* v)
{
    v->x = XFns{Launch<N>::xfwd, Launch<N>::xinv, rows_for(N)};
    v->nx = v->ny = v->nz = 0;
    x_variants<N>(v->vel, v->str, v->nx);
    yz_variants<N>(v->y, v->ny, v->z, v->nz);
    v->probe = reinterpret_cast<const void*>(&k_xfwd<N, NT>);
}

}  // namespace

#define CAT2(a, b) a##b
#define CAT(a, b) CAT2(a, b)
bool CAT(variants_, PSTD_GROUP)(int n, Variants* v)
{
    switch (n) {
#define CASE(N)          \
    case N:              \
        fill<N>(v);      \
        return true;
        PSTD_LENGTHS(CASE)
#undef CASE
    default:
        return false;
    }
}

}  // namespace pstd
