// Device kernels of one leapfrog step of the pseudo-spectral elastic solver.
//
// One step (Sec. II-A: FFT-based spatial derivatives, staggered leapfrog):
//   V phase: 6 summed stresses --x FFT (fused in the previous S kernel)-->
//            y FFT --> z FFT * operator * inverse z FFT (9 derivatives) -->
//            inverse y FFT --> [inverse x FFT + velocity update + receivers +
//            x FFT of the 3 summed velocities]
//   S phase: y FFT --> z operator --> inverse y FFT --> [inverse x FFT +
//            stress update + source injection + receivers + x FFT of the 6
//            summed stresses]
// Real fields are [nz][ny][nx].  An x-transformed spectrum (kx = 0 .. nx/2)
// is stored as a main block [nz][ny][ldx] holding kx < nxm (nxm = nx/2 for
// even nx, (nx+1)/2 for odd nx; ldx = nxm rounded up to 16, i.e. 128-byte
// rows) followed, for even nx, by the Nyquist plane kx = nx/2 as [nz][ny].
// The y and z transforms work on 16-column tiles of the main block plus
// tiles of 16 Nyquist pencils, so no tile is left almost empty.
#pragma once
#include "fft_lds.hpp"

namespace pstd {

struct Geo {
    int nx, ny, nz, nxh, ldx, nrows;   // nrows = ny * nz; nxh = nx/2 + 1
    int nxm, has_nyq;                  // main columns, Nyquist plane present
    long n;                            // cells
    long nqoff;                        // offset of the Nyquist plane in a spectrum
    long nspec;                        // complex values per spectrum
    long fstride;                      // floats per shot of split fields (24 n)
    long sstride;                      // complex values per shot of spectra (18 nspec)
    int shot_fast;                     // update kernels' grid is (shots, row blocks)
    int stream;                        // the update kernels pass the caches by (STREAM_BYTES)
};

// material coefficients pre-multiplied by dt (FP64 on the host, stored FP32)
struct Mat {
    const float* dtr[3];   // dt / rho at the vx, vy, vz nodes
    const float* dlam;     // dt * lambda at centres
    const float* dmu2;     // 2 dt * mu at centres
    const float* dmus[3];  // dt * mu at xy, xz, yz shear nodes
    // Kelvin-Voigt viscosity (eq. 1-2), only read by the viscous stress
    // update: chi and 2 eta at centres, eta at the shear nodes (not times dt:
    // they multiply the change of a velocity derivative over one step)
    const float* chi;
    const float* eta2;
    const float* etas[3];
};

// PML factors a = exp(-alpha dt / 2) per axis, at integer and half nodes, and
// the multi-axial factors b = a^p: a split part along axis d is damped by
// a_d times b_e of the two other axes e.
struct Pml {
    const float* ai[3];
    const float* ah[3];
    const float* bi[3];
    const float* bh[3];
    // per axis, the indices [flo, fhi] whose four factors are all exactly 1:
    // a cell inside all three ranges is undamped, and there each field keeps
    // its whole value in its first split part (the others stay zero)
    int flo[3] = {0, 0, 0}, fhi[3] = {-1, -1, -1};
};

__device__ __forceinline__ bool undamped(const Pml& pm, int x, int y, int z)
{
    return x >= pm.flo[0] && x <= pm.fhi[0] && y >= pm.flo[1] && y <= pm.fhi[1] && z >= pm.flo[2] &&
           z <= pm.fhi[2];
}

struct Rec {
    const int* ptr;     // [nrows + 1] receivers sorted by row
    const int4* ent;    // {x, row, id, 0}
    int n_rec;
};

struct Inj {
    const int* ptr;     // [n_shots][nrows + 1]
    const int4* ent;    // {row nx + x, split field 0..14, coef (float bits), wavelet row}
    const float* wav;   // [n_src_total][nt_w]
    int nt_w;
};

// How a phase's derivatives are formed.  D_d f = IFFT[i k_d e^{..} kappa FFT f]:
// kappa couples the axes and is applied where the full spectrum is at hand, in
// the z kernel; the symbol of one axis only needs that axis in the spectral
// domain.  The z kernel therefore writes at most two spectra per input, kappa f
// (which serves the x and the y derivative: the inverse y transform multiplies
// its input by the y or the x symbol) and, where the input has a z derivative,
// kappa times the z symbol: 8 instead of 9 spectra in the velocity phase, 6
// instead of 9 in the stress phase.
struct PhaseDesc {
    int nin, in0;       // input spectra, the first one
    int nz[6];          // z kernel outputs of each input
    int zslot[6][2];    // derivative slot each is stored in (below 0: its input's own spectrum)
    int zplus[6][2];    // -1: kappa alone, 0 / 1: times the D- / D+ z symbol
    int nsrc;           // spectra that the inverse y kernel reads
    int ysrc[8];        // their slots
    int yn[8];          // derivatives formed from each (one: in place)
    int yslot[8][2];
    int yaxis[8][2];    // symbol applied: 0 x, 1 y, 2 none
    int yplus[8][2];    // 1: D+, 0: D-
    int nders, dsrc[9], dord[9];   // the nine derivatives one by one: source and which of its derivatives
};

struct Ops {
    const float2* sym[3][2];   // per axis, [0] = D-, [1] = D+ : i k exp(-+ i k h/2)
    const float* kap;          // kappa(|k|) / (nx ny nz), main block [nz][ny][ldx]
    const float* kapn;         // the same on the Nyquist plane [nz][ny]
    // kappa evaluated in the kernel instead of read from the table (kpoly[phase]
    // = 1): s = (c_ref dt / 2)^2 |k|^2 from the per-axis squares k2[d] (x:
    // 0..nx/2), kappa / (nx ny nz) = sum_n kc[n] s^n, the series of sin(a)/a in
    // s = a^2
    int kpoly[2];
    const float* k2[3];
    float kc[8];
};

// device-resident descriptor of the two derivative phases (read with uniform
// loads; kept out of the kernel arguments so runtime indexing stays in memory)
struct ZDesc {
    PhaseDesc ph[2];   // [0] V phase, [1] S phase
    Ops ops;
};

// Rows per block of the update kernels.  Up to 32: 8 (16 left three quarters of
// the chip without a block at 32^3: 50.8 us a step, 48.8 with 8); up to 48: 4
// (48^3 65.8 with 8, 62.0); at 64 8 and 4 are even (64^3 72.9 and 71.7, 16 shots
// of it 536 and 544).
constexpr int rows_for(int nx) { return nx <= 32 ? 8 : nx <= 48 ? 4 : nx <= 64 ? 8 : nx <= 160 ? 4 : 2; }

// Load through a pointer that addresses global memory.  Pointers read from a
// device-resident descriptor are generic to the compiler, and a generic load
// also holds the LDS wait counter, so every LDS wait after it would wait for
// the memory load as well.
__device__ __forceinline__ float gld(const float* p)
{
    return *(const __attribute__((address_space(1))) float*)p;
}
__device__ __forceinline__ float2 gld(const float2* p)
{
    typedef float f2v __attribute__((ext_vector_type(2)));
    const f2v v = *(const __attribute__((address_space(1))) f2v*)p;
    return make_float2(v.x, v.y);
}

// Column-tile widths of the y and z kernels that the library is built with:
// a tile of TX pencils of length N stages N (TX + 1) complex values in LDS
// (at most 64 KB) and, in the z kernel, keeps N TX / NT of them per thread in
// registers twice (spectrum and one derivative), at most 16 each.  y: width 8
// only where 16 does not fit; z: width 8 always (half the LDS of 16, so twice
// the blocks per CU, against 64-byte instead of 128-byte row segments).
constexpr bool y_tile_ok(int n, int tx) { return (long)n * (tx + 1) * 8 + n * 8 <= 65536; }
constexpr bool z_tile_ok(int n, int tx) { return n * tx <= 16 * 256 && (long)n * (tx + 1) * 8 + 3L * n * 8 <= 65536; }
// threads per block of the y kernels: 512 where the tile's LDS leaves room for
// only two blocks per compute unit
constexpr int y_threads(int n, int tx) { return (long)n * (tx + 2) * 8 > 40960 ? 512 : 256; }
constexpr bool y_tile_built(int n, int tx) { return y_tile_ok(n, tx) && (tx != 8 || !y_tile_ok(n, 16)); }
constexpr bool z_tile_built(int n, int tx) { return z_tile_ok(n, tx); }


// index of spectrum element (row, kx) within one field's spectrum
__device__ __forceinline__ long spec_idx(const Geo& g, int row, int k)
{
    return k < g.nxm ? (long)row * g.ldx + k : g.nqoff + row;
}

// Loader for an inverse x transform: complex pencil q is the Hermitian
// extension of the half spectra of real pencils 2q and 2q+1 (Z = A + i B), so
// one complex inverse FFT gives both real rows (as real and imaginary parts;
// ROWS is even: both are rows of one field).  DC and Nyquist keep only their
// real parts.  Rows past the grid (only in the last block of a ragged row
// count) read the last row instead: their pencils are transformed on their own
// and never stored, and no branch separates the loads of a pass.
//
// fetch() loads the two half-spectrum values at k = min(i, NX - i), finish()
// combines them with w = sign(2 i - NX) (0 at DC and at the Nyquist bin):
// Z_i = (a.x + w b.y) + i (b.x - w a.y).  In a butterfly of even radix R the
// elements r < R / 2 lie below NX / 2 and the others above, and DC and Nyquist
// can only be r = 0 and r = R / 2 of j = 0: the sign is a constant, two
// addresses per row serve the butterfly with constant offsets, and only one
// element asks for the Nyquist plane.  (With the index, its half and the sign
// worked out per element the loads took some 20 instructions each.)
template <int NX, int ROWS>
struct HermLoader {
    const float2* __restrict__ src;
    Geo g;
    int row0;
    static constexpr bool TWO_PHASE = true;
    using Raw = float4;
    struct At {
        const float2 *a, *b;     // k = j of the two rows
        const float2 *ha, *hb;   // k = NX - j (even radix)
        long nyq;                // Nyquist value of the first row
        long nstep;              // to that of the second
    };
    template <int R>
    __device__ At begin(int q, int j) const
    {
        const int f = 2 * q / ROWS, r = 2 * q - f * ROWS;
        const int ra = min(row0 + r, g.nrows - 1), rb = min(row0 + r + 1, g.nrows - 1);
        const float2* p = src + (long)f * g.nspec;
        At t;
        t.a = p + (long)ra * g.ldx + j;
        t.b = t.a + (ra == rb ? 0 : g.ldx);
        t.ha = t.a + (NX - 2 * j);
        t.hb = t.b + (NX - 2 * j);
        t.nyq = (long)f * g.nspec + g.nqoff + ra;
        t.nstep = rb - ra;
        return t;
    }
    template <int R>
    __device__ float4 fetch(const At& t, int j, int r) const
    {
        constexpr int M = NX / R;
        const float2 *pa, *pb;
        if (R % 2 == 0) {
            pa = 2 * r < R ? t.a + r * M : t.ha - r * M;
            pb = 2 * r < R ? t.b + r * M : t.hb - r * M;
            if (2 * r == R && j == 0) {
                pa = src + t.nyq;
                pb = pa + t.nstep;
            }
        } else {
            // odd radix: NX is odd (no Nyquist plane)
            const int i = j + r * M, d = min(i, NX - i) - j;
            pa = t.a + d;
            pb = t.b + d;
        }
        const float2 a = *pa, b = *pb;
        return make_float4(a.x, a.y, b.x, b.y);
    }
    template <int R>
    __device__ float2 finish(float4 v, int j, int r) const
    {
        constexpr int M = NX / R;
        float w;
        if (R % 2 == 0) {
            w = 2 * r < R ? -1.f : 1.f;
            if ((r == 0 || 2 * r == R) && j == 0) w = 0.f;
        } else {
            const int i = j + r * M;
            w = i == 0 ? 0.f : 2 * i > NX ? 1.f : -1.f;
        }
        return make_float2(fmaf(w, v.w, v.x), fmaf(-w, v.y, v.z));
    }
};

// Unpack NPO complex forward transforms of paired real rows into half spectra.
template <int NX, int ROWS, int NT, int NPO, int PS>
__device__ __forceinline__ void unstage_r2c(const float2* s, float2* __restrict__ dst, const Geo& g, int row0)
{
    constexpr int NXH = NX / 2 + 1;
    for (int e = threadIdx.x; e < NPO * NXH; e += NT) {
        const int q = e / NXH, k = e - q * NXH;
        const float2 z = s[q * PS + lidx<true>(k)];
        const float2 zm = s[q * PS + lidx<true>(k == 0 ? 0 : NX - k)];
        const float2 A = make_float2(0.5f * (z.x + zm.x), 0.5f * (z.y - zm.y));
        const float2 B = make_float2(0.5f * (z.y + zm.y), -0.5f * (z.x - zm.x));
        const int f = 2 * q / ROWS, row = row0 + 2 * q - f * ROWS;
        float2* d = dst + (long)f * g.nspec + spec_idx(g, row, k);
        if (row < g.nrows) d[0] = A;
        if (row + 1 < g.nrows) d[k < g.nxm ? g.ldx : 1] = B;
    }
}

// real value of pencil p at x (pairs stored as re / im of one complex pencil)
template <int PS>
__device__ __forceinline__ float pencil_val(const float2* s, int p, int x)
{
    const float2 v = s[(p >> 1) * PS + lidx<true>(x)];
    return (p & 1) ? v.y : v.x;
}

template <int PS>
__device__ __forceinline__ void pencil_set(float2* s, int p, int x, float v)
{
    float* f = reinterpret_cast<float*>(s + (p >> 1) * PS + lidx<true>(x));
    f[p & 1] = v;
}

// Field values by a block-uniform base and a 32-bit byte offset (a field is at
// most 512^3 floats): the base stays in scalar registers and one vector
// register addresses a cell in every field, where 64-bit indices cost two or
// three vector instructions per access.  The empty asm keeps the base a value
// of its own; otherwise the compiler adds the cell to the first field's address
// and the field's distance to that, in vector registers.
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) char* scalar_base(T* p)
{
    const unsigned long long u = (unsigned long long)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)u);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(u >> 32));
    auto b = (__attribute__((address_space(1))) char*)((unsigned long long)hi << 32 | lo);
    asm("" : "+s"(b));
    return b;
}
// STREAM: non-temporal (a run whose arrays together exceed the last-level cache
// finds none of its split fields there a step later, and leaves more of it to
// the spectra when they pass it by; the coefficients, which the shots of a
// batch share, do not: 64 shots at 128^3 15.9 ms a step with them, 15.6 without).
template <bool STREAM>
__device__ __forceinline__ float ldf(const float* base, unsigned off)
{
    const auto p = (const __attribute__((address_space(1))) float*)(scalar_base(base) + off);
    return STREAM ? __builtin_nontemporal_load(p) : *p;
}
template <bool STREAM>
__device__ __forceinline__ void stf(float* base, unsigned off, float v)
{
    const auto p = (__attribute__((address_space(1))) float*)(scalar_base(base) + off);
    if (STREAM) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// Device bytes of the contexts that run together from which their update kernels
// stream: the 256 MB of the last-level cache.  Microseconds per step without and with: 180 MB (96^3)
// 154, 166; 225 MB 175, 184; 288 MB (120 x 96 x 120) 209, 204; 426 MB (128^3)
// 275, 257; 665 MB (160 x 160 x 128) 416, 390; 3.4 GB (256^3) 2026, 1961.
constexpr long STREAM_BYTES = 256L << 20;

// Row r of a block's rows as the thread knows it: where a wave's 64 cells lie in
// one row (NX a multiple of 64) it is made a scalar, and with it the row's y
// and z and everything read by them.
template <int NX>
__device__ __forceinline__ int wave_row(int r)
{
    return NX % 64 == 0 ? __builtin_amdgcn_readfirstlane(r) : r;
}

// Block -> (shot, first row) of the update kernels.  A batch of shots is
// launched on a grid of (shots, row blocks), so that consecutive blocks take
// consecutive shots of one row block and the shots read the model's material
// and PML tables at about the same time and share them in cache; one shot
// (or more row blocks than a grid's y extent holds) on (row blocks, shots).
// The choice is a scalar flag: no division, so shot and row stay scalar.
__device__ __forceinline__ void update_block(const Geo& g, int& shot, int& row0, int rows)
{
    if (g.shot_fast) {
        shot = blockIdx.x;
        row0 = blockIdx.y * rows;
    } else {
        shot = blockIdx.y;
        row0 = blockIdx.x * rows;
    }
}

// Occupancy hint for the velocity update: at power-of-two lengths up to 256
// with 256 or 512 threads (and 512 with 512) the compiler fits it in 96 VGPRs
// without spilling when asked for 5 waves per SIMD (4 otherwise), which
// measured faster; at other lengths the same request spills to scratch or
// cannot be met, so it is not made there.  (The stress update, asked the
// same, measured slightly slower.)
template <int NX, int NT>
constexpr int vel_waves()
{
    return (NX >= 32 && (NX & (NX - 1)) == 0 && NT >= 256 && (NX <= 256 || NT == 512)) ? 5 : 1;
}

// ---------------------------------------------------------------------------
// V phase tail: inverse x FFT of the 9 stress derivatives, velocity split-PML
// update (eq. 2 second line), receivers vx vy vz, x FFT of the summed v.
template <int NX, int NT, bool STREAM>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(vel_waves<NX, NT>()))) void k_vel(
    Geo g, Mat m, Pml pm, const float2* __restrict__ twx, float* __restrict__ fields, float2* __restrict__ spec,
    Rec rc, float* __restrict__ traces, const int* __restrict__ stepp, int* __restrict__ stepn, int n0, int ldt)
{
    constexpr int ROWS = rows_for(NX);
    constexpr int PS = padded_len(NX);
    constexpr int NPI = 9 * ROWS / 2;
    constexpr int NPO = 3 * ROWS / 2;
    constexpr int CPT = (ROWS * NX + NT - 1) / NT;
    __shared__ float2 s[NPI * PS];
    __shared__ float2 tw[NX];
    // step counters alternate between two words: this step reads one and
    // publishes the next step's index in the other (read by no kernel of
    // this step)
    const int step = *stepp;
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *stepn = step + 1;

    int shot, row0;
    update_block(g, shot, row0, ROWS);
    float* __restrict__ F = fields + (long)shot * g.fstride;
    const float2* __restrict__ D9 = spec + (long)shot * g.sstride + 9 * g.nspec;
    float2* __restrict__ S3 = spec + (long)shot * g.sstride + 6 * g.nspec;
    const int e0 = rc.ptr[row0], e1 = rc.ptr[min(row0 + ROWS, g.nrows)];   // receivers, needed last

    for (int i = threadIdx.x; i < NX; i += NT) tw[i] = twx[i];
    fft_ld<NX, NPI, NT, +1, PS, 1, false, false, HermLoader<NX, ROWS>, NoSt, true>(s, tw, HermLoader<NX, ROWS>{D9, g, row0}, NoSt{});

    // all loads of the update before any store: the split parts share one
    // base pointer, so interleaved stores would serialise later loads
    float vp[CPT][9], dtr[CPT][3], a[CPT][3][3];
    bool ok[CPT], in[CPT];
    unsigned cell[CPT];   // byte offset
    const int z0 = row0 / g.ny, y0 = row0 - z0 * g.ny;   // ROWS <= 16 <= ny: at most one step in z
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        const int c = threadIdx.x + i * NT;
        const int r = wave_row<NX>(c / NX), x = c - r * NX;
        ok[i] = c < ROWS * NX && row0 + r < g.nrows;
        const int rr = ok[i] ? r : 0;
        const bool up = y0 + rr >= g.ny;
        const int y = y0 + rr - (up ? g.ny : 0), z = z0 + (up ? 1 : 0);
        cell[i] = 4u * ((unsigned)(row0 + rr) * NX + x);
        in[i] = undamped(pm, x, y, z);
        const float axi = pm.ai[0][x], axh = pm.ah[0][x];
        const float ayi = pm.ai[1][y], ayh = pm.ah[1][y];
        const float azi = pm.ai[2][z], azh = pm.ah[2][z];
        const float bxi = pm.bi[0][x], bxh = pm.bh[0][x];
        const float byi = pm.bi[1][y], byh = pm.bh[1][y];
        const float bzi = pm.bi[2][z], bzh = pm.bh[2][z];
        // component c sits half a cell up along axis c; split part d is damped
        // by a_d and by b of the two other axes, all at the component's node
        a[i][0][0] = axh * byi * bzi; a[i][0][1] = ayi * bxh * bzi; a[i][0][2] = azi * bxh * byi;
        a[i][1][0] = axi * byh * bzi; a[i][1][1] = ayh * bxi * bzi; a[i][1][2] = azi * bxi * byh;
        a[i][2][0] = axi * byi * bzh; a[i][2][1] = ayi * bxi * bzh; a[i][2][2] = azh * bxi * byi;
        // an undamped cell reads only the first part of each component (cells
        // outside the grid read valid ones and store nothing)
#pragma unroll
        for (int comp = 0; comp < 3; ++comp) {
            vp[i][3 * comp] = ldf<STREAM>(F + 3 * comp * g.n, cell[i]);
            vp[i][3 * comp + 1] = vp[i][3 * comp + 2] = 0.f;
            dtr[i][comp] = ldf<false>(m.dtr[comp], cell[i]);
        }
        if (!in[i])
#pragma unroll
            for (int q = 0; q < 9; ++q)
                if (q % 3) vp[i][q] = ldf<STREAM>(F + q * g.n, cell[i]);
    }

    float vsum[CPT][3];
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        const int c = threadIdx.x + i * NT;
        const int r = c / NX, x = c - r * NX;
#pragma unroll
        for (int comp = 0; comp < 3; ++comp) {
            float acc = 0.f;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const int q = 3 * comp + d;
                const float dv = ok[i] ? pencil_val<PS>(s, q * ROWS + r, x) : 0.f;
                const float ad = a[i][comp][d];
                vp[i][q] = ad * (ad * vp[i][q] + dtr[i][comp] * dv);
                acc += vp[i][q];
            }
            vsum[i][comp] = acc;
            // undamped: the parts' factors are 1, their sum is the component
            if (in[i]) vp[i][3 * comp] = acc;
        }
        if (ok[i]) {
#pragma unroll
            for (int q = 0; q < 9; q += 3) stf<STREAM>(F + q * g.n, cell[i], vp[i][q]);
            if (!in[i])
#pragma unroll
                for (int q = 0; q < 9; ++q)
                    if (q % 3) stf<STREAM>(F + q * g.n, cell[i], vp[i][q]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        const int c = threadIdx.x + i * NT;
        if (c >= ROWS * NX) continue;
        const int r = c / NX, x = c - r * NX;
#pragma unroll
        for (int comp = 0; comp < 3; ++comp) pencil_set<PS>(s, comp * ROWS + r, x, ok[i] ? vsum[i][comp] : 0.f);
    }
    __syncthreads();
    // receivers (vx, vy, vz at their staggered nodes, time (n + 1/2) dt)
    {
        const int tn = step - n0;
        for (int e = e0 + threadIdx.x; e < e1; e += NT) {
            const int4 q = rc.ent[e];
            const int r = q.y - row0;
#pragma unroll
            for (int comp = 0; comp < 3; ++comp)
                traces[(((long)shot * 4 + 1 + comp) * rc.n_rec + q.z) * ldt + tn] =
                    pencil_val<PS>(s, comp * ROWS + r, q.x);
        }
    }
    lds_fft<NX, NPO, NT, -1, PS, 1, false, true>(s, tw);
    unstage_r2c<NX, ROWS, NT, NPO, PS>(s, S3, g, row0);
}

// ---------------------------------------------------------------------------
// the first split part of a stress component (parts 0-8: three per normal
// component, 9-14: two per shear component)
__host__ __device__ constexpr bool first_part(int q) { return q < 9 ? q % 3 == 0 : (q - 9) % 2 == 0; }

// slot of velocity derivative q (order of e[] in k_str) among the nine stored ones
__host__ __device__ constexpr int ep_slot(int q) { return q < 3 ? q : ((q - 3) ^ 1) + 3; }

// S phase tail: inverse x FFT of the 9 velocity derivatives, stress split-PML
// update (eq. 2 first line), source injection, receiver p (eq. 3), x FFT of
// the 6 summed stresses.  Bound by memory where the grid is large and by the
// vector pipe below: at 384 x 384 x 256 it moves 5.88 GB (5.74 without the
// lines fetched whole at the ends of the rows) in 1.23 ms, 4.8 TB/s, and of its
// instructions more than a third were addresses (2691 vector instructions per
// thread at 384 with 64-bit indices, a division per cell and a branch per
// element of the loads, 2120 without the injection loop now).  Velocity and
// stress update together at 128^3: 158 -> 137 us (126 since they stream); with a
// smoothed source at 125 x 75 x 300 the stress update went from 207 to 100 us.
template <int NX, int NT, bool VISC, bool STREAM>
__global__ __launch_bounds__(NT) void k_str(Geo g, Mat m, Pml pm, const float2* __restrict__ twx,
                                            float* __restrict__ fields, float2* __restrict__ spec,
                                            Rec rc, Inj inj, float* __restrict__ traces,
                                            const int* __restrict__ stepp, int n0, int ldt)
{
    constexpr int ROWS = rows_for(NX);
    constexpr int PS = padded_len(NX);
    constexpr int NPI = 9 * ROWS / 2;
    constexpr int NPO = 6 * ROWS / 2;
    constexpr int CPT = (ROWS * NX + NT - 1) / NT;
    __shared__ float2 s[NPI * PS];
    __shared__ float2 tw[NX];

    int shot, row0;
    update_block(g, shot, row0, ROWS);
    float* __restrict__ F = fields + (long)shot * g.fstride + 9 * g.n;   // 15 stress parts
    // viscous: the nine velocity derivatives of the previous step, after the 24
    // split parts, in the order D-x vx, D-y vy, D-z vz, Dx+ vy, Dy+ vx, Dx+ vz,
    // Dz+ vx, Dy+ vz, Dz+ vy (e[] below swaps each shear pair)
    float* __restrict__ EP = fields + (long)shot * g.fstride + 24 * g.n;
    const float2* __restrict__ D9 = spec + (long)shot * g.sstride + 9 * g.nspec;
    float2* __restrict__ S6 = spec + (long)shot * g.sstride;
    const int step = *stepp;
    const int* __restrict__ iptr = inj.ptr + (long)shot * (g.nrows + 1);
    const int e0 = rc.ptr[row0], e1 = rc.ptr[min(row0 + ROWS, g.nrows)];   // receivers, needed last

    for (int i = threadIdx.x; i < NX; i += NT) tw[i] = twx[i];
    fft_ld<NX, NPI, NT, +1, PS, 1, false, false, HermLoader<NX, ROWS>, NoSt, true>(s, tw, HermLoader<NX, ROWS>{D9, g, row0}, NoSt{});

    // every load of every cell of this thread before any arithmetic or store
    // (the split parts share one base pointer, so a store would serialise
    // later loads): split parts, materials, PML factors, source rows
    float sp[CPT][15], mt[CPT][5], fa[CPT][9];
    float ep[VISC ? CPT : 1][9], vm[VISC ? CPT : 1][5];
    int jr[CPT][2];
    bool ok[CPT], in[CPT];
    const int z0 = row0 / g.ny, y0 = row0 - z0 * g.ny;   // ROWS <= 16 <= ny: at most one step in z
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        const int c = threadIdx.x + i * NT;
        const int r = wave_row<NX>(c / NX), x = c - r * NX;
        ok[i] = c < ROWS * NX && row0 + r < g.nrows;
        // lanes past the block's or the grid's rows follow the last row (their
        // loads are valid, they store nothing), so a wave's rows never decrease
        const int rr = min(min(r, ROWS - 1), g.nrows - 1 - row0);
        const bool up = y0 + rr >= g.ny;
        const int y = y0 + rr - (up ? g.ny : 0), z = z0 + (up ? 1 : 0);
        const unsigned cell = 4u * ((unsigned)(row0 + rr) * NX + x);   // byte offset
        in[i] = undamped(pm, x, y, z);
        // an undamped cell reads only the first part of each component
#pragma unroll
        for (int q = 0; q < 15; ++q) sp[i][q] = first_part(q) ? ldf<STREAM>(F + q * g.n, cell) : 0.f;
        if (!in[i])
#pragma unroll
            for (int q = 0; q < 15; ++q)
                if (!first_part(q)) sp[i][q] = ldf<STREAM>(F + q * g.n, cell);
        mt[i][0] = ldf<false>(m.dlam, cell);
        mt[i][1] = ldf<false>(m.dmu2, cell);
        mt[i][2] = ldf<false>(m.dmus[0], cell);
        mt[i][3] = ldf<false>(m.dmus[1], cell);
        mt[i][4] = ldf<false>(m.dmus[2], cell);
        const float bxi = pm.bi[0][x], bxh = pm.bh[0][x];
        const float byi = pm.bi[1][y], byh = pm.bh[1][y];
        const float bzi = pm.bi[2][z], bzh = pm.bh[2][z];
        // normal parts (centre nodes): a_d times b of the other two axes
        fa[i][0] = pm.ai[0][x] * byi * bzi;
        fa[i][1] = pm.ai[1][y] * bxi * bzi;
        fa[i][2] = pm.ai[2][z] * bxi * byi;
        // shear parts at their nodes: xy (h,h,i), xz (h,i,h), yz (i,h,h)
        fa[i][3] = pm.ah[0][x] * byh * bzi;   // xy, x part
        fa[i][4] = pm.ah[1][y] * bxh * bzi;   // xy, y part
        fa[i][5] = pm.ah[0][x] * byi * bzh;   // xz, x part
        fa[i][6] = pm.ah[2][z] * bxh * byi;   // xz, z part
        fa[i][7] = pm.ah[1][y] * bxi * bzh;   // yz, y part
        fa[i][8] = pm.ah[2][z] * bxi * byh;   // yz, z part
        jr[i][0] = iptr[row0 + rr];
        jr[i][1] = iptr[row0 + rr + 1];
        if constexpr (VISC) {
#pragma unroll
            for (int q = 0; q < 9; ++q) ep[i][q] = ldf<STREAM>(EP + ep_slot(q) * g.n, cell);
            vm[i][0] = ldf<false>(m.chi, cell);
            vm[i][1] = ldf<false>(m.eta2, cell);
            vm[i][2] = ldf<false>(m.etas[0], cell);
            vm[i][3] = ldf<false>(m.etas[1], cell);
            vm[i][4] = ldf<false>(m.etas[2], cell);
        }
    }
    __builtin_amdgcn_sched_barrier(0);

    float ssum[CPT][6];
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        const int c = threadIdx.x + i * NT;
        const int r = wave_row<NX>(min(c / NX, ROWS - 1)), x = c - wave_row<NX>(c / NX) * NX;
        const int idx = min(row0 + r, g.nrows - 1) * NX + x;
        const unsigned cell = 4u * (unsigned)idx;
        const float dlam = mt[i][0], dmu2 = mt[i][1];
        const float mxy = mt[i][2], mxz = mt[i][3], myz = mt[i][4];
        const float ai[3] = {fa[i][0], fa[i][1], fa[i][2]};
        const float axy_x = fa[i][3], axy_y = fa[i][4], axz_x = fa[i][5], axz_z = fa[i][6];
        const float ayz_y = fa[i][7], ayz_z = fa[i][8];
        // derivatives: e0..e2 = D_d^- v_d, e3 = Dy+ vx, e4 = Dx+ vy, e5 = Dz+ vx,
        //              e6 = Dx+ vz, e7 = Dz+ vy, e8 = Dy+ vz
        float e[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) e[q] = pencil_val<PS>(s, q * ROWS + r, x);
        // viscous terms (eq. 2): chi delta_cd d/dt(div v) + eta d/dt(D v + (D v)^T),
        // d/dt as the change of each derivative over the step
        float de[9];
        if constexpr (VISC) {
#pragma unroll
            for (int q = 0; q < 9; ++q) de[q] = e[q] - ep[i][q];
        }
        // normal parts sp[i][3c + d] (component c, axis d)
#pragma unroll
        for (int cc = 0; cc < 3; ++cc)
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const float coef = cc == d ? dlam + dmu2 : dlam;
                float rhs = coef * e[d];
                if constexpr (VISC) rhs += (cc == d ? vm[i][0] + vm[i][1] : vm[i][0]) * de[d];
                sp[i][3 * cc + d] = ai[d] * (ai[d] * sp[i][3 * cc + d] + rhs);
            }
        // shear parts: 9 sxy(x) <- Dx+ vy, 10 sxy(y) <- Dy+ vx, 11 sxz(x) <- Dx+ vz,
        //              12 sxz(z) <- Dz+ vx, 13 syz(y) <- Dy+ vz, 14 syz(z) <- Dz+ vy
        float sh[6] = {mxy * e[4], mxy * e[3], mxz * e[6], mxz * e[5], myz * e[8], myz * e[7]};
        if constexpr (VISC) {
            sh[0] += vm[i][2] * de[4];
            sh[1] += vm[i][2] * de[3];
            sh[2] += vm[i][3] * de[6];
            sh[3] += vm[i][3] * de[5];
            sh[4] += vm[i][4] * de[8];
            sh[5] += vm[i][4] * de[7];
        }
        sp[i][9] = axy_x * (axy_x * sp[i][9] + sh[0]);
        sp[i][10] = axy_y * (axy_y * sp[i][10] + sh[1]);
        sp[i][11] = axz_x * (axz_x * sp[i][11] + sh[2]);
        sp[i][12] = axz_z * (axz_z * sp[i][12] + sh[3]);
        sp[i][13] = ayz_y * (ayz_y * sp[i][13] + sh[4]);
        sp[i][14] = ayz_z * (ayz_z * sp[i][14] + sh[5]);
        if constexpr (VISC) {
            if (ok[i])
#pragma unroll
                for (int q = 0; q < 9; ++q) stf<STREAM>(EP + ep_slot(q) * g.n, cell, e[q]);
        }
        // point sources: the entries of the wave's rows, 64 at a time, one load
        // per lane, then field by field through scalar registers.  (Read one by
        // one by every thread, the entries of a smoothed source held their block
        // 100 us after all others had ended, those of a point source 4.)
        const int ja = __builtin_amdgcn_readfirstlane(jr[i][0]), jb = __builtin_amdgcn_readlane(jr[i][1], 63);
        if (ja != jb && step < inj.nt_w) {
            const int lane = threadIdx.x & 63;
            for (int j = ja; j < jb; j += 64) {
                int4 q = make_int4(0, -1, 0, 0);
                float val = 0.f;
                if (j + lane < jb) {
                    q = inj.ent[j + lane];
                    val = __int_as_float(q.z) * inj.wav[(long)q.w * inj.nt_w + step];
                }
#pragma unroll
                for (int f = 0; f < 15; ++f)
                    for (unsigned long long of = __ballot(q.y == f); of; of &= of - 1) {
                        const int l = __builtin_ctzll(of);
                        const float v = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(val), l));
                        sp[i][f] += idx == __builtin_amdgcn_readlane(q.x, l) ? v : 0.f;
                    }
            }
        }
        ssum[i][0] = sp[i][0] + sp[i][1] + sp[i][2];
        ssum[i][1] = sp[i][3] + sp[i][4] + sp[i][5];
        ssum[i][2] = sp[i][6] + sp[i][7] + sp[i][8];
        ssum[i][3] = sp[i][9] + sp[i][10];
        ssum[i][4] = sp[i][11] + sp[i][12];
        ssum[i][5] = sp[i][13] + sp[i][14];
        if (in[i]) {
            // undamped: the parts' factors are 1, their sum is the component
            sp[i][0] = ssum[i][0];
            sp[i][3] = ssum[i][1];
            sp[i][6] = ssum[i][2];
            sp[i][9] = ssum[i][3];
            sp[i][11] = ssum[i][4];
            sp[i][13] = ssum[i][5];
        }
        if (ok[i]) {
#pragma unroll
            for (int q = 0; q < 15; ++q)
                if (first_part(q)) stf<STREAM>(F + q * g.n, cell, sp[i][q]);
            if (!in[i])
#pragma unroll
                for (int q = 0; q < 15; ++q)
                    if (!first_part(q)) stf<STREAM>(F + q * g.n, cell, sp[i][q]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        const int c = threadIdx.x + i * NT;
        if (c >= ROWS * NX) continue;
        const int r = c / NX, x = c - r * NX;
#pragma unroll
        for (int q = 0; q < 6; ++q) pencil_set<PS>(s, q * ROWS + r, x, ok[i] ? ssum[i][q] : 0.f);
    }
    __syncthreads();
    {
        const int tn = step - n0;
        for (int e = e0 + threadIdx.x; e < e1; e += NT) {
            const int4 q = rc.ent[e];
            const int r = q.y - row0;
            const float tr = pencil_val<PS>(s, 0 * ROWS + r, q.x) + pencil_val<PS>(s, 1 * ROWS + r, q.x) +
                             pencil_val<PS>(s, 2 * ROWS + r, q.x);
            traces[((long)shot * 4 * rc.n_rec + q.z) * ldt + tn] = -tr * (1.0f / 3.0f);
        }
    }
    lds_fft<NX, NPO, NT, -1, PS, 1, false, true>(s, tw);
    unstage_r2c<NX, ROWS, NT, NPO, PS>(s, S6, g, row0);
}

// ---------------------------------------------------------------------------
// x FFT of sums of consecutive split parts: output f = sum of `cnt[f]` real
// fields starting at in + first[f] * n.  Used to rebuild the stress spectra
// after a state restore and by the derivative test entry.
struct SumDesc {
    int nf;
    int first[9];
    int cnt[9];
};

template <int NX, int NT>
__global__ __launch_bounds__(NT) void k_xfwd(Geo g, const float2* __restrict__ twx, const float* __restrict__ in,
                                             long in_shot_stride, float2* __restrict__ out,
                                             long out_shot_stride, SumDesc sd)
{
    constexpr int ROWS = rows_for(NX);
    constexpr int PS = padded_len(NX);
    constexpr int NPMAX = 9 * ROWS / 2;
    __shared__ float2 s[NPMAX * PS];
    const int shot = blockIdx.y;
    const int row0 = blockIdx.x * ROWS;
    const float* __restrict__ I = in + (long)shot * in_shot_stride;
    float2* __restrict__ O = out + (long)shot * out_shot_stride;
    const int np = sd.nf * ROWS;
    for (int e = threadIdx.x; e < ((np + 1) / 2) * 2 * NX; e += NT) {
        const int p = e / NX, x = e - p * NX;
        float v = 0.f;
        if (p < np) {
            const int f = p / ROWS, r = p - f * ROWS;
            const int row = row0 + r;
            if (row < g.nrows)
                for (int q = 0; q < sd.cnt[f]; ++q) v += I[(long)(sd.first[f] + q) * g.n + (long)row * NX + x];
        }
        pencil_set<PS>(s, p, x, v);
    }
    __syncthreads();
    // np is a multiple of ROWS (even): np / 2 complex pencils
    if (sd.nf == 3) {
        lds_fft<NX, 3 * ROWS / 2, NT, -1, PS, 1, false, true>(s, twx);
        unstage_r2c<NX, ROWS, NT, 3 * ROWS / 2, PS>(s, O, g, row0);
    } else {
        lds_fft<NX, 6 * ROWS / 2, NT, -1, PS, 1, false, true>(s, twx);
        unstage_r2c<NX, ROWS, NT, 6 * ROWS / 2, PS>(s, O, g, row0);
    }
}

// inverse x FFT of 9 spectra to 9 real fields (test entry)
template <int NX, int NT>
__global__ __launch_bounds__(NT) void k_xinv(Geo g, const float2* __restrict__ twx, const float2* __restrict__ in,
                                             float* __restrict__ out)
{
    constexpr int ROWS = rows_for(NX);
    constexpr int PS = padded_len(NX);
    constexpr int NPI = 9 * ROWS / 2;
    __shared__ float2 s[NPI * PS];
    const int row0 = blockIdx.x * ROWS;
    fft_ld<NX, NPI, NT, +1, PS, 1, false, false, HermLoader<NX, ROWS>, NoSt, true>(s, twx, HermLoader<NX, ROWS>{in, g, row0}, NoSt{});
    for (int e = threadIdx.x; e < 9 * ROWS * NX; e += NT) {
        const int p = e / NX, x = e - p * NX;
        const int f = p / ROWS, r = p - f * ROWS;
        const int row = row0 + r;
        if (row < g.nrows) out[(long)f * g.n + (long)row * NX + x] = pencil_val<PS>(s, p, x);
    }
}

// ---------------------------------------------------------------------------
// Column tile of a y or z transform: element (column c, position i) is at
// base[c * cs + i * is]; columns c >= ncol are outside the array.
struct Tile {
    float2* base;
    long cs, is;
    int ncol;
    // columns past the array read the last column (unconditional load, no
    // branch between the loads of a pass) and give zero
    __device__ float2 operator()(int c, int i) const
    {
        const float2 v = base[min(c, ncol - 1) * cs + i * is];
        return c < ncol ? v : make_float2(0.f, 0.f);
    }
    __device__ void operator()(int c, int i, float2 v) const
    {
        if (c < ncol) base[c * cs + i * is] = v;
    }
};

// Column tile of plane z (main tiles) or of the Nyquist pencils; false: none
template <int NY, int TX>
__device__ __forceinline__ bool y_tile(const Geo& g, long& off, long& cs, long& is, int& ncol)
{
    const int tmain = (g.nxm + TX - 1) / TX;
    if ((int)blockIdx.x < tmain) {
        const int kx0 = blockIdx.x * TX;
        off = (long)blockIdx.y * NY * g.ldx + kx0;
        cs = 1;
        is = g.ldx;
        ncol = min(TX, g.nxm - kx0);
        return true;
    }
    const int z0 = blockIdx.y * TX;
    off = g.nqoff + (long)z0 * NY;
    cs = NY;
    is = 1;
    ncol = min(TX, g.nz - z0);
    return z0 < g.nz;
}

// forward y FFT of `nf` spectra starting at field f0, in place.
// grid: (main tiles + Nyquist tile, nz, shots * nf).  Main tile bx covers
// columns [TX bx, TX bx + TX) of plane z = by; the Nyquist tile covers the
// Nyquist pencils of planes [TX by, TX by + TX).
template <int NY, int NT, int TX>
__global__ __launch_bounds__(NT) void k_y(Geo g, const float2* __restrict__ twy, float2* __restrict__ spec,
                                          int f0, int nf)
{
    constexpr int IS = TX + 1;
    __shared__ float2 s[NY * IS];
    __shared__ float2 tw[NY];
    const int shot = blockIdx.z / nf, f = f0 + blockIdx.z % nf;
    long off, cs, is;
    int ncol;
    if (!y_tile<NY, TX>(g, off, cs, is, ncol)) return;
    const Tile t{spec + (long)shot * g.sstride + (long)f * g.nspec + off, cs, is, ncol};
    for (int i = threadIdx.x; i < NY; i += NT) tw[i] = twy[i];
    fft_ld<NY, TX, NT, -1, 1, IS, true, true>(s, tw, t, t);
}

// Loader of the inverse y transform: a column tile times the y symbol (ysym;
// from LDS, or global memory if it does not fit) or a value per column
template <bool LDS>
struct TileSym {
    Tile t;
    const float2* sy;
    float2 k;
    float sgn;
    bool ysym;
    __device__ float2 operator()(int c, int i) const
    {
        const float2 v = t(c, i);
        const float2 y = LDS ? sy[i] : gld(sy + i);
        return c_mul(ysym ? make_float2(sgn * y.x, y.y) : k, v);
    }
};

// inverse y FFTs of one phase, forming the x and y derivatives: a block takes a
// tile of one of the phase's nsrc spectra and, for each derivative formed from
// it, loads the first pass's butterflies, multiplies them by the y symbol, the
// x symbol (one value per column) or nothing and transforms.  A second
// derivative finds the tile in the L2 (kept in registers through the first
// transform it took 256 of them at length 384 and 600 us).  At 384 x 384 x 256:
// 550 and 517 us for 17 and 15 spectra read or written, against 511 and 523 for
// 18 when the z kernel wrote all nine derivatives; the z kernel's part is
// 515 -> 488 and 420 -> 298 us.
// A source of one derivative is transformed in place (every element is read
// before the first store); one of two lies outside the derivatives' slots, so
// that its derivatives can also be formed by two blocks (nsrc = 9: grid z runs
// over the derivatives), which shortens the launch where the chip is not full.
// grid: (main tiles + Nyquist tile, nz, shots * nsrc).
template <int NY, int NT, int TX>
__global__ __launch_bounds__(NT) void k_yinv(Geo g, const float2* __restrict__ twy, float2* spec,
                                             const ZDesc* __restrict__ zd, int phase, int nsrc)
{
    constexpr int IS = TX + 1;
    // the y symbol goes to LDS where it fits beside the tile
    constexpr bool SYL = (long)NY * (IS + 2) * 8 <= 65536;
    static_assert(NT % TX == 0, "a thread keeps its column");
    __shared__ float2 s[NY * IS];
    __shared__ float2 tw[NY];
    __shared__ float2 sy[SYL ? NY : 1];
    const PhaseDesc& ph = zd->ph[phase];
    const bool single = nsrc == 9;   // a block per derivative
    const int shot = blockIdx.z / nsrc, item = blockIdx.z % nsrc;
    const int src = single ? ph.dsrc[item] : item;
    long off, cs, is;
    int ncol;
    if (!y_tile<NY, TX>(g, off, cs, is, ncol)) return;
    float2* D9 = spec + (long)shot * g.sstride + 9 * g.nspec + off;
    for (int i = threadIdx.x; i < NY; i += NT) {
        tw[i] = twy[i];
        if constexpr (SYL) sy[i] = gld(zd->ops.sym[1][1] + i);
    }
    // x symbol of this thread's column (the Nyquist pencils: that of nx / 2)
    const int kx = cs == 1 ? blockIdx.x * TX + min((int)threadIdx.x % TX, ncol - 1) : g.nx / 2;
    const float2 sx = gld(zd->ops.sym[0][1] + kx);
    const int o0 = single ? ph.dord[item] : 0, o1 = single ? o0 + 1 : ph.yn[src];
    for (int o = o0; o < o1; ++o) {
        // an offset the compiler cannot see through: without it the addresses
        // of every element are worked out before the loop and kept
        long zero = 0;
        asm volatile("" : "+s"(zero));
        const Tile in{D9 + ph.ysrc[src] * g.nspec + zero, cs, is + zero, ncol};
        const Tile out{D9 + ph.yslot[src][o] * g.nspec, cs, is + zero, ncol};
        const int axis = ph.yaxis[src][o];
        // D- is D+ with the real part negated: i k e^{-i k h/2} = (k sin, k cos)
        const float sgn = ph.yplus[src][o] ? 1.f : -1.f;
        const float2 k = axis == 0 ? make_float2(sgn * sx.x, sx.y) : make_float2(1.f, 0.f);
        __syncthreads();   // tw and sy staged; s was read by the previous last pass
        fft_ld<NY, TX, NT, +1, 1, IS, true, true>(s, tw, TileSym<SYL>{in, SYL ? sy : zd->ops.sym[1][1] + zero, k, sgn, axis == 1}, out);
    }
}

// z FFT, multiply by kappa and, for the z derivatives, the staggered symbol,
// inverse z FFT.  grid: (main tiles + Nyquist tile, ny, shots * groups).  Main tile bx
// covers columns [TX bx, +TX) of row ky = by; the Nyquist tile covers the
// Nyquist pencils of rows [TX by, +TX).  A block takes the input spectra
// [fpb g, fpb g + fpb) of its shot (g = blockIdx.z % groups), so that with
// fpb >= the phase's inputs one block applies its tile's kappa and symbols
// (loaded once) to every input field in turn.  For each input it reads
// spectrum `in0 + input` and writes one or two spectra (9 + slot, see
// PhaseDesc): the forward spectrum stays in registers, each output is
// multiplied there and inverted with the reversed radix plan.  MR caps the radix of the plan
// (16, or 8 for the 512-thread variants, whose threads then all take a
// butterfly of the first pass).
template <int NZ, int NT, int TX, int MR = 16>
__global__ __launch_bounds__(NT) void k_z(Geo g, const float2* __restrict__ twz, float2* __restrict__ spec,
                                          int in0, const ZDesc* __restrict__ zd, int phase, int fpb)
{
    const PhaseDesc& ph = zd->ph[phase];
    const Ops& ops = zd->ops;
    constexpr int IS = TX + 1;
    using RS = RegShape<NZ, TX, NT, MR>;
    constexpr int RL = RS::RL, QL = RS::QL;
    // LDS: the tile, the twiddles, and the D+ symbol along z (D- is D+ with the
    // real part negated: i k e^{-i k h/2} = (k sin, k cos) against
    // (-k sin, k cos)); kept under 40 KB at length 256 so that four blocks
    // share a CU
    __shared__ float2 s[NZ * IS];
    __shared__ float2 tw[NZ];
    __shared__ float2 symz[NZ];
    __shared__ float kxy2[TX];
    // the forward spectrum is reused by every output of the input field; kept
    // in registers it stays live through the inverse transforms (about a
    // quarter of the kernel's VGPRs), so where it takes at most 16 KB it is
    // parked in thread-private LDS slots instead
    constexpr bool STASH = QL * RL * NT * (int)sizeof(float2) <= 16384;
    __shared__ float2 xs[STASH ? QL * RL * NT : 1];
    const int tmain = (g.nxm + TX - 1) / TX;
    const int groups = (ph.nin + fpb - 1) / fpb;
    const int shot = blockIdx.z / groups, fg = blockIdx.z % groups;
    const int f0 = fg * fpb, f1 = min(ph.nin, f0 + fpb);
    long off, zs;
    const float* kap;
    int ncol, kx0, kxc, ky0, kyc;
    if ((int)blockIdx.x < tmain) {
        kx0 = blockIdx.x * TX;
        kxc = 1;
        ky0 = blockIdx.y;
        kyc = 0;
        off = (long)ky0 * g.ldx + kx0;
        zs = (long)g.ny * g.ldx;
        ncol = min(TX, g.nxm - kx0);
        kap = ops.kap + off;
    } else {
        ky0 = blockIdx.y * TX;
        if (ky0 >= g.ny) return;
        kyc = 1;
        kx0 = g.nx / 2;
        kxc = 0;
        off = g.nqoff + ky0;
        zs = g.ny;
        ncol = min(TX, g.ny - ky0);
        kap = ops.kapn + ky0;
    }
    const bool kpoly = ops.kpoly[phase] != 0;
    for (int i = threadIdx.x; i < NZ; i += NT) {
        tw[i] = twz[i];
        symz[i] = gld(ops.sym[2][1] + i);
    }
    if (kpoly)
        for (int i = threadIdx.x; i < TX; i += NT) {
            const int c = min(i, ncol - 1);
            kxy2[i] = gld(ops.k2[0] + kx0 + kxc * c) + gld(ops.k2[1] + ky0 + kyc * c);
        }
    __syncthreads();
    // kappa of the elements this thread multiplies, once for all the block's inputs
    float kr[QL][RL];
#pragma unroll
    for (int q = 0; q < QL; ++q)
#pragma unroll
        for (int r = 0; r < RL; ++r) {
            int c, z;
            const bool ok = reg_coords<NZ, RL, TX, NT, true>(q, r, c, z);
            float kv;
            if (kpoly) {
                const float sv = kxy2[min(c, TX - 1)] + gld(ops.k2[2] + (ok ? z : 0));
                kv = ops.kc[7];
#pragma unroll
                for (int t = 6; t >= 0; --t) kv = fmaf(kv, sv, ops.kc[t]);
            } else {
                // unconditional load (no branch between the loads) at a valid
                // element: slots past the last butterfly (ok false) carry z >= NZ
                kv = gld(kap + (ok ? z : 0) * zs + min(c, ncol - 1));
            }
            kr[q][r] = (ok && c < ncol) ? kv : 0.f;
        }
    float2* __restrict__ sb = spec + (long)shot * g.sstride;
    for (int fi = f0; fi < f1; ++fi) {
        if (fi > f0) __syncthreads();   // s was read by the previous input's last pass
        const Tile in{sb + (long)(in0 + fi) * g.nspec + off, 1, zs, ncol};
        float2 X[QL][RL];
        fft_g2r<NZ, TX, NT, -1, 1, IS, true, Tile, float2[QL][RL], MR>(s, tw, in, X);
        if constexpr (STASH) {
#pragma unroll
            for (int q = 0; q < QL; ++q)
#pragma unroll
                for (int r = 0; r < RL; ++r) xs[(q * RL + r) * NT + threadIdx.x] = X[q][r];
        }
        for (int o = 0; o < ph.nz[fi]; ++o) {
            const int plus = ph.zplus[fi][o];
            const float sgn = plus ? 1.f : -1.f;
            float2 Y[QL][RL];
#pragma unroll
            for (int q = 0; q < QL; ++q)
#pragma unroll
                for (int r = 0; r < RL; ++r) {
                    int c, z;
                    reg_coords<NZ, RL, TX, NT, true>(q, r, c, z);
                    float2 xv = STASH ? xs[(q * RL + r) * NT + threadIdx.x] : X[q][r];
                    if (plus >= 0) {   // the same for the whole block
                        const float2 s1 = symz[z];
                        xv = c_mul(make_float2(sgn * s1.x, s1.y), xv);
                    }
                    Y[q][r] = c_scale(xv, kr[q][r]);
                }
            __syncthreads();   // s was read by the previous pass
            const Tile out{sb + (long)(9 + ph.zslot[fi][o]) * g.nspec + off, 1, zs, ncol};
            fft_r2g<NZ, TX, NT, +1, 1, IS, true, float2[QL][RL], Tile, MR>(s, tw, Y, out);
        }
    }
}

// The 512-thread z variants: the largest radix (16 or 8) whose first pass
// still gives every thread a butterfly
constexpr int z_maxr(int n, int tx, int nt) { return tx * (n / 16) >= nt ? 16 : 8; }
// at least four values per thread and a radix-8 (or 16) first pass
constexpr bool z512_ok(int n, int tx) { return z_tile_ok(n, tx) && n * tx >= 4 * 512 && n % 8 == 0 && tx * (n / 8) >= 512; }

}  // namespace pstd
