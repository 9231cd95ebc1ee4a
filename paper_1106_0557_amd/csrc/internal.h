// internal.h -- data structures shared by the HIP kernels and the host runtime.
//
// Workspace layout of one in-flight solve (complex values of the precision):
//   W  : [z / B][ky < 2ny][z % B][kx < nx]   main part in tiles of B z planes
//                                            (rows of nx values, aligned)
//   Wn : [z < nz][ky < 2ny]                  the kx = nx (Nyquist) column, split
//                                            off so that every row of W is aligned
// B (DevPlan::zb, a power of two up to 16 that divides nz; 1 but for planes of 4 MB
// or more, half-length z lines: 1 MB) keeps the z lines of the z pass
// within nz/B regions of B rows instead of nz planes far apart, which the address
// translation caches cannot hold for large meshes.  Row (z, ky) starts at element
// ((z/B)*2ny + ky)*B*nx + (z%B)*nx.  Whole solves of large meshes keep W in slabs of kx, each
// laid out like that with its own width in place of nx (w_slab below).
// The x pass writes rows ky = y < ny of every z plane; the y pass fills all 2ny
// rows; the z pass works in place on z < nz; the inverse y pass leaves rows
// y < ny; the inverse x pass reads them.  The upper z half of the doubled mesh
// is never stored: it is zero on input and discarded on output.
//
// Green's-function spectrum (plan precision), octant kx <= nx, ky <= ny, kz <= nz,
// by DevPlan::gz:
//   0  G : [kz][ky][kx < nx]                  Gn : [kz][ky]   (kx = nx)
//   1  G : [ky][kx][kz]                       Gn : [ky][kz]
//   2  G : [ky][kx / kGroup][kz'][kx % kGroup]  Gn : [ky][kz']
// with kz' the even kz first, then the odd ones (a z pass by half-length lines reads
// one parity at a time).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace pspfft {

// Adjacent kx that a blocked spectrum keeps together.
constexpr int kGroup = 8;

constexpr int kMaxStages = 10;
constexpr int kMaxProblems = 32;  // problems per grouped launch

// One transform line along one axis, split into stages of radix R[s].
// y and z lines have length L = 2n (the doubled mesh).  x lines use the packed
// real-to-complex form: the 2n real values of a zero-padded row become n
// complex values, so L = n there, plus a split step with exp(-i pi k / n).
// A line is handled by NB = L / E threads, each owning the E positions
// t + NB*m (m < E) before the first and after the last stage; the upper half of
// the input (m >= E/2) is the zero padding and the upper half of the output is
// never needed, so both are known at compile time.
//
// Lengths outside the families (E = 0, NB = 0) run on the generic line kernel
// (line_generic.hip) with stages of radix 8, 4 or 2, then 5, 9 and 3.
struct AxisPlan {
    int n;        // mesh cells along the axis
    int L;        // transform length (2n for y and z, n for x)
    int E;        // elements per thread (radix family: 16, 20, 24 or 36; 0: generic kernel)
    int NB;       // threads per line (0: generic kernel)
    int nst;      // number of stages
    int ntw;      // entries in the twiddle table
    int R[kMaxStages];          // radix of stage s
    int Ns[kMaxStages];         // product of the radices before stage s
    uint32_t magic[kMaxStages]; // floor(2^32 / Ns) + 1, for b / Ns
    int twoff[kMaxStages];      // offset of stage s in the twiddle table
    const void *tw;             // twiddles exp(-2 pi i r k / (Ns R)), k < Ns, 1 <= r < R
    const void *post;           // x only: exp(-i pi k / n), k < n
    // stage twiddles of the half-length lines of mix_lines.h (null: another
    // kernel takes the axis): for s = 0, 1 and each stage past the first,
    // exp(-2 pi i r (k + s/2) / (Ns R)) at [(r - 1)*Ns + k]
    const void *mtw;
};

struct DevPlan {
    int nx, ny, nz, prec;  // prec: 0 = FP32, 1 = FP64
    int zb;                // z planes per tile of the workspace
    int ks;                // log2 of the kx per slab of the workspace (w_slab; kNoSlabs: one slab)
    int gz;                // spectrum layout (above)
    AxisPlan ax[3];        // x, y, z
    const void *G;         // spectrum, main part
    const void *Gn;        // spectrum, kx = nx
};

// One problem inside a grouped launch.
struct ProbArg {
    const DevPlan *plan;
    const void *S;    // source (x forward pass)
    void *Phi;        // potential (x inverse pass)
    void *W;          // workspace main part
    void *Wn;         // workspace Nyquist column
};

// A run of `group` consecutive problems p[first .. first+group) with the same
// plan.  Its workgroups are numbered tile-major (tile, member), so the members
// that read the same spectrum slice are neighbours in the launch; those of the
// half-length x and y passes problem by problem (mix_job).
struct Segment {
    int wg_begin;     // first workgroup of the segment
    int first;        // index of its first problem in LaunchArgs::p
    int group;        // problems in the segment
    int wg_main;      // tiles of main lines per problem; the rest are Nyquist lines
};

// Workspace bytes of a launch above which family kernels stream their line data with
// nontemporal accesses and half-length x and y passes take the chunked tile order: about
// the device's Infinity Cache (256 MB), which a
// smaller launch's workspaces can stay in between passes.  Half-length lines take no nontemporal accesses.
constexpr size_t kStreamBytes = size_t(256) << 20;

struct LaunchArgs {
    int count;        // problems in this launch
    int nseg;         // segments
    int nwg;          // workgroups doing work (the grid may be padded to a multiple of 8)
    int xcd_remap;    // renumber workgroups so each XCD gets a contiguous range (half-length lines: 1 or 0)
    int wave_z;       // z pass: spectra kz-fastest, lines kept within one wavefront
    int gtile;        // generic line kernel: lines per workgroup (a power of two)
    int rounds;       // half-length x rows: tiles that a workgroup takes one after the other (0: one)
    int glmax;        // generic line kernel: longest line of the launch
    int gtw;          // generic line kernel: stage twiddles copied into LDS after the two buffers
    int nt;           // streaming launch (workspaces beyond kStreamBytes): its line data takes
                      // nontemporal loads and stores where the kernel says so
    static constexpr int kProblems = kMaxProblems;
    Segment seg[kMaxProblems];
    ProbArg p[kMaxProblems];
};

// The same for the planes of one problem: copying the arguments is a third of what a launch costs the
// host (2.8 us with these, 4.2 us with LaunchArgs), which is what a sequence of small solves waits for.
struct SoloArgs {
    static constexpr int kProblems = 1;
    int nwg;
    ProbArg p[1];
};

enum PassMode { X_FWD = 0, Y_FWD = 1, Z_CONV = 2, Y_INV = 3, X_INV = 4 };

// Start (in elements) of workspace row (z, ky).
__host__ __device__ inline size_t w_row(int z, int ky, int ny, int nx, int zb) {
    const int sh = __builtin_ctz(static_cast<unsigned>(zb));  // zb is a power of two
    return ((static_cast<size_t>(z >> sh) * 2 * ny + ky) * zb + (z & (zb - 1))) * static_cast<size_t>(nx);
}

// Slabs of kx: the workspace main part of a large mesh is split along kx into slabs of kSlab values
// (the last one may hold fewer), one after the other, each with the layout of w_row for rows of its
// own width.  A y or z line then lies within one slab: without them, the lines of a z pass step
// through the whole workspace, and beyond about 4 GB a CU's translation cache has lost a page when the
// next tile comes back to it.  Measured, misses per z tile of 640, 768 and 1024 points (FP32 n^3): 49,
// 96 and 139, and none at 576; one solve without and with slabs, ms: FP32 576^3 5.5 and 5.4, 640^3 8.1
// and 7.1, 1024^3 36.6 and 28.7, 1152^3 57.9 and 49.2, FP64 640^3 17.3 and 15.5; no gain below
// kSlabBytes (FP64 432^3 4.1 and 4.1, where x passes write 512-byte pieces for nothing).  Widths 16, 32, 64 and
// 128 differ by 2 to 4 % (32 best); whole numbers of tiles fill each.
constexpr int kSlabShift = 5, kSlab = 1 << kSlabShift, kNoSlabs = 30;
constexpr size_t kSlabBytes = size_t(5) << 29;
struct Slab {
    int kx0, w;     // its first kx and width
    size_t start;   // elements before it
};
__host__ __device__ inline Slab w_slab(int s, int ks, int nx, int ny, int nz) {
    const int kx0 = s << ks, rest = nx - kx0;
    const int w = rest < (1 << ks) ? rest : 1 << ks;
    return Slab{kx0, w, static_cast<size_t>(kx0) * 2 * ny * nz};
}

// LDS layout of a workgroup (complex elements), identical on host and device.
// Column passes keep element (line c, position P) at P*col_stride + c; row passes
// at c*S + P + P/16, with S chosen so that the NB-lane chunks of consecutive
// rows fall on different banks.
__host__ __device__ constexpr int row_stride(int L, int NB, int csz) {
    int S = L + (L >> 4);
    const int chunk = NB * csz;
    if (chunk < 256) {
        const int want = chunk % 256;
        while ((S * csz) % 256 != want) ++S;
    }
    return S;
}
// Row stride (complex values) of a line in the wavefront-owned z convolution:
// the row layout's P + P/16, plus one so that the rows of neighbouring lines
// start on different banks (the tile is transposed through these rows).
__host__ __device__ constexpr int wave_line_stride(int L) { return L + L / 16 + 1; }

// Column passes: position stride of the LDS tile, tile + 1 (the extra column
// staggers the positions of a wavefront's lines over the banks), or tile where
// the LDS limits a CU to fewer than four workgroups (tile data plus the L - 1
// stage twiddles in 160 KB) and dropping that column lets one more fit:
// measured on 384-point lines, 3 workgroups per CU instead of 2 beat the bank
// staggering by 8 % per solve.
__host__ __device__ constexpr int col_stride(int L, int tile, int csz) {
    const long cap = 160 * 1024;
    const long padded = (static_cast<long>(L) * (tile + 1) + L - 1) * csz;
    const long packed = (static_cast<long>(L) * tile + L - 1) * csz;
    return cap / padded < 4 && cap / packed > cap / padded ? tile : tile + 1;
}

__host__ __device__ constexpr int data_elems(bool row, int L, int NB, int block, int csz) {
    const int tile = block / NB;
    return row ? tile * row_stride(L, NB, csz) : L * col_stride(L, tile, csz);
}

inline int pass_axis(int mode) { return mode == X_FWD || mode == X_INV ? 0 : (mode == Z_CONV ? 2 : 1); }

// Largest workgroup per (precision, radix family), chosen so that the E
// registers per thread fit without spilling.
// Default lines per workgroup: column passes take 128-byte row segments of
// complex values, row passes enough rows for 256-thread groups.
__host__ __device__ constexpr int default_tile(int prec, bool row) {
    return row ? (prec == 0 ? 32 : 16) : (prec == 0 ? 16 : 8);
}

// Lines per workgroup of pass `mode` (lines of nb threads): the default tile.
// Measured, smaller z-pass tiles (more workgroups per CU, 64- or 32-byte row
// segments) lose at every size.
__host__ __device__ constexpr int fix_tile(int prec, int mode, int /*nb*/) {
    return default_tile(prec, mode == X_FWD || mode == X_INV);
}

__host__ __device__ constexpr int max_block_for(int prec, int E) {
    return prec == 0 ? (E == 16 ? 1024 : (E <= 24 ? 512 : 256)) : (E == 16 ? 512 : 256);
}

// Line forms of the line-pass instances (template parameter FIX): FIX & 7 is
// the number of compile-time stages (0: run-time geometry; 2, 3 or 4: radices
// E, K / E, M, K / E, M, M, K with M the power-of-two part of E), FIX & 8 marks
// 64-bit addresses (some array of the launch reaches 4 GB; else 32-bit lane
// offsets).  fix_nb: threads per line.
__host__ __device__ constexpr int fix_stages(int fix) { return fix & 7; }
__host__ __device__ constexpr bool fix_off32(int fix) { return (fix & 7) != 0 && (fix & 8) == 0; }
__host__ __device__ constexpr int fix_nb(int fix, int E, int K) {
    return (fix & 7) == 2 ? K : ((fix & 7) == 3 ? (E & -E) * K : ((fix & 7) == 4 ? (E & -E) * (E & -E) * K : 0));
}
constexpr int kFixWide = 8;

// Lines per workgroup of a line-pass launch (pass_kernel) for lines of nb
// threads in radix family E: the default tile, halved while the workgroup
// exceeds the family's largest or its LDS (data, stage twiddles and, for rows,
// the split factors) exceeds 160 KB.  Long lines thus keep compile-time geometry
// with a smaller tile.
__host__ __device__ constexpr int pass_tile(int prec, int mode, int E, int nb) {
    const bool row = mode == X_FWD || mode == X_INV;
    const int L = E * nb, csz = prec == 0 ? 8 : 16;
    int t = default_tile(prec, row);
    if (nb <= 0) return t;  // run-time geometry
    while (t > 1) {
        const long elems = static_cast<long>(data_elems(row, L, nb, t * nb, csz)) + (L - 1) + (row ? L : 0);
        if (static_cast<long>(t) * nb <= max_block_for(prec, E) && elems * csz <= 160 * 1024) break;
        t /= 2;
    }
    return t;
}

// Row passes (X_FWD, X_INV) of compile-time lines of NB threads keep their
// stage twiddles and split factors in global memory (a table the L1 holds)
// where their pass_tile() rows alone let two workgroups share a CU and rows
// plus those 2L - 1 values let only one.
__host__ __device__ constexpr bool row_tables_global(int prec, int E, int NB) {
    const int L = E * NB, csz = prec == 0 ? 8 : 16;
    const long cap = 160 * 1024;
    const long data = static_cast<long>(data_elems(true, L, NB, pass_tile(prec, X_FWD, E, NB) * NB, csz)) * csz;
    return cap / data >= 2 && cap / (data + static_cast<long>(2 * L - 1) * csz) == 1;
}

// Column y passes (Y_FWD, Y_INV) of compile-time lines of NB threads keep their
// stage twiddles in global memory and pack the tile's positions (LDS stride =
// tile) where that lets two workgroups of pass_tile() lines share a CU and the
// layout with the twiddles in LDS lets only one.  col_ldsw: the LDS position
// stride of such a launch; col_default_lds: its bytes with the twiddles in LDS.
__host__ __device__ constexpr size_t col_default_lds(int prec, int mode, int E, int NB) {
    const int L = E * NB, csz = prec == 0 ? 8 : 16;
    const int tile = pass_tile(prec, mode, E, NB);
    return (static_cast<size_t>(L) * col_stride(L, tile, csz) + L - 1) * csz;
}
__host__ __device__ constexpr bool col_tables_global(int prec, int mode, int E, int NB) {
    if (mode != Y_FWD && mode != Y_INV) return false;
    const long L = static_cast<long>(E) * NB, csz = prec == 0 ? 8 : 16, cap = 160 * 1024;
    const long packed = L * pass_tile(prec, mode, E, NB) * csz;
    return cap / packed >= 2 && cap / static_cast<long>(col_default_lds(prec, mode, E, NB)) == 1;
}
__host__ __device__ constexpr int col_ldsw(int prec, int mode, int E, int NB) {
    const int tile = pass_tile(prec, mode, E, NB);
    return col_tables_global(prec, mode, E, NB) ? tile : col_stride(E * NB, tile, prec == 0 ? 8 : 16);
}

// The wavefront-owned z kernel: FP32 lines of kWaveE*NB points, NB = 32 or 64 threads, in four stages with
// radices 36, 4, 4 and K (1152 and 2304 points).  Threads per line:
constexpr int kWaveE = 36;
__host__ __device__ constexpr int wave_nb(int K) { return 16 * K; }

// Its lines per workgroup: the default tile, halved while the workgroup exceeds
// the family's largest or the tile's rows and the stage twiddles exceed the LDS.
__host__ __device__ constexpr int wave_tile(int NB) {
    int t = fix_tile(0, Z_CONV, NB);
    const long L = static_cast<long>(kWaveE) * NB, csz = 8;
    while (t > 1 && (static_cast<long>(t) * NB > max_block_for(0, kWaveE) ||
                     (t * static_cast<long>(wave_line_stride(static_cast<int>(L))) + L - 1) * csz > 160 * 1024))
        t /= 2;
    return t;
}

// Whether it keeps the stage twiddles in LDS after the tile's rows: unless
// leaving them in global memory (a table the L1 holds) lets one more
// workgroup share a CU.
__host__ __device__ constexpr bool wave_tw_lds(int NB) {
    const long L = static_cast<long>(kWaveE) * NB, csz = 8, cap = 160 * 1024;
    const long rows = wave_tile(NB) * static_cast<long>(wave_line_stride(static_cast<int>(L))) * csz;
    return cap / rows <= cap / (rows + (L - 1) * csz);
}

// Its LDS bytes: one row per line of the tile, then the stage twiddles (when
// they are kept in LDS).
__host__ __device__ constexpr size_t wave_lds_bytes(int NB) {
    const int L = kWaveE * NB;
    return static_cast<size_t>(wave_tile(NB) * wave_line_stride(L) + (wave_tw_lds(NB) ? L - 1 : 0)) * 8;
}

// Wavefronts per SIMD it is compiled for: as many as its workgroups that fit a
// CU's LDS bring (so that the register allocation does not keep a second
// workgroup out), at least one.
__host__ __device__ constexpr int wave_waves_per_simd(int NB) {
    const long per_cu = 160L * 1024 / static_cast<long>(wave_lds_bytes(NB));
    const long w = per_cu * wave_tile(NB) * NB / 64 / 4;
    return w < 1 ? 1 : (w > 8 ? 8 : static_cast<int>(w));
}

// Lines of L points of a radix family that pass `mode` still runs on the family's kernels: half-length lines have
// the mesh sizes 80, 96 and 144 to 1152 (128: FP64 x and y), but for z lines of meshes whose planes are too large for
// their 32-bit addresses (more than 2^32 bytes in a block of up to 128 positions: no planes of up to 4096 x 2048 values
// with fewer than 512 cells along z in FP32, 256 in FP64).  Those have 64-bit addresses (wide).
__host__ __device__ constexpr bool family_line(int prec, int mode, int L, bool wide) {
    const bool row = mode == X_FWD || mode == X_INV;
    const int n = row ? L : L / 2;
    if (n > (row ? 2 : 1) * (prec == 0 ? 2048 : 1152)) return false;
    if (mode == Z_CONV && wide && n >= (prec == 0 ? 512 : 256)) return true;
    const bool half = n == 80 || n == 96 || (n >= 144 && n <= 1152) || (n == 128 && prec == 1 && mode != Z_CONV);
    return !half;
}
// Some line of family E whose last stage has radix K does.
__host__ __device__ constexpr bool family_last(int prec, int mode, int E, int K) {
    for (int nb = 1; nb <= 4096 / E; nb *= 2) {
        int last = nb;
        while (last > (E & -E)) last /= E & -E;
        if (last == K && (family_line(prec, mode, E * nb, false) || family_line(prec, mode, E * nb, true))) return true;
    }
    return false;
}

// Fused plane kernels (x and y transforms of one z plane per workgroup) for
// nx == ny = n = E*K above 64 (mix_plane): n*K threads, the LDS plane (n rows of row_stride(n, K))
// followed by the n - 1 stage twiddles, the n split factors and 2n values of
// column 0.
__host__ __device__ constexpr size_t plane_lds_bytes(int prec, int E, int K) {
    const int n = E * K, csz = prec == 0 ? 8 : 16;
    return static_cast<size_t>(n * row_stride(n, K, csz) + 4 * n - 1) * csz;
}
// FP64 workgroups stay at 256 threads or fewer, where the two line transforms
// each thread holds fit in registers.
__host__ __device__ constexpr bool plane_fits(int prec, int E, int K) {
    return K >= 1 && K <= (E & -E) && E * K > 64 && E * K * K <= (prec == 0 ? 1024 : 256) &&
           plane_lds_bytes(prec, E, K) <= 160 * 1024;
}

// Launchers: one per (precision, family), defined in pass_<prec>_e<E>.hip.
// K is the radix of the last stage of the pass axis (1 for a single stage).
// The plane launchers run the forward (fwd) or inverse fused kernel with n*K threads.
#define PSPFFT_DECLARE_FAMILY(NAME, PLANE)                                                          \
    hipError_t NAME(int mode, int K, int fix, const LaunchArgs &args, int grid, int block,          \
                    size_t lds, hipStream_t stream);                                                \
    hipError_t PLANE(bool fwd, int K, const LaunchArgs &args, int grid, size_t lds, hipStream_t stream);
PSPFFT_DECLARE_FAMILY(launch_f32_e16, plane_f32_e16)
PSPFFT_DECLARE_FAMILY(launch_f32_e20, plane_f32_e20)
PSPFFT_DECLARE_FAMILY(launch_f32_e24, plane_f32_e24)
PSPFFT_DECLARE_FAMILY(launch_f32_e36, plane_f32_e36)
PSPFFT_DECLARE_FAMILY(launch_f64_e16, plane_f64_e16)
PSPFFT_DECLARE_FAMILY(launch_f64_e20, plane_f64_e20)
PSPFFT_DECLARE_FAMILY(launch_f64_e24, plane_f64_e24)
PSPFFT_DECLARE_FAMILY(launch_f64_e36, plane_f64_e36)
#undef PSPFFT_DECLARE_FAMILY
inline hipError_t launch_pass(int mode, int prec, int E, int K, int fix, const LaunchArgs &args, int grid,
                              int block, size_t lds, hipStream_t stream) {
    if (grid <= 0) return hipSuccess;
    switch (prec * 100 + E) {
        case 16: return launch_f32_e16(mode, K, fix, args, grid, block, lds, stream);
        case 20: return launch_f32_e20(mode, K, fix, args, grid, block, lds, stream);
        case 24: return launch_f32_e24(mode, K, fix, args, grid, block, lds, stream);
        case 36: return launch_f32_e36(mode, K, fix, args, grid, block, lds, stream);
        case 116: return launch_f64_e16(mode, K, fix, args, grid, block, lds, stream);
        case 120: return launch_f64_e20(mode, K, fix, args, grid, block, lds, stream);
        case 124: return launch_f64_e24(mode, K, fix, args, grid, block, lds, stream);
        case 136: return launch_f64_e36(mode, K, fix, args, grid, block, lds, stream);
        default: return hipErrorInvalidValue;
    }
}

inline hipError_t launch_plane(bool fwd, int prec, int E, int K, const LaunchArgs &args, int grid, size_t lds,
                               hipStream_t stream) {
    if (grid <= 0) return hipSuccess;
    switch (prec * 100 + E) {
        case 16: return plane_f32_e16(fwd, K, args, grid, lds, stream);
        case 20: return plane_f32_e20(fwd, K, args, grid, lds, stream);
        case 24: return plane_f32_e24(fwd, K, args, grid, lds, stream);
        case 36: return plane_f32_e36(fwd, K, args, grid, lds, stream);
        case 116: return plane_f64_e16(fwd, K, args, grid, lds, stream);
        case 120: return plane_f64_e20(fwd, K, args, grid, lds, stream);
        case 124: return plane_f64_e24(fwd, K, args, grid, lds, stream);
        case 136: return plane_f64_e36(fwd, K, args, grid, lds, stream);
        default: return hipErrorInvalidValue;
    }
}

// Generic line kernel (any 2^a 3^b 5^c length): `grid` workgroups of 256
// threads, each owning args.gtile lines, with `lds` bytes of LDS (two buffers of
// gtile * (glmax + 1) complex values, then, with args.gtw, the stage twiddles).
hipError_t launch_generic(int mode, int prec, const LaunchArgs &args, int grid, size_t lds, hipStream_t stream);


// Spectrum layout of a plan whose z lines of n cells are half-length lines: blocked, but kx-fastest for the lengths
// for which pspfft_plan_spectrum_kz_fastest has always answered 0.  That answer is what the list keeps, not
// speed: measured, z passes with the blocked layout take 0.95 of the time at 96 (thirteen FP32 96^3), 144 and 160
// (sixteen), 0.93 at 192 (nine), 0.97 in FP32 288 x 144 x 144, and in FP64 0.92 at 144 and 192 (eight), 0.88 at 320
// (two), 0.83 at 576, 0.94 at 640, 0.88 at 1024 and 1152 (512 x 512 planes); 80 and single small solves within 1 %.
__host__ __device__ constexpr int mix_spectrum(int prec, int n) {
    const bool fp32_only = n == 320 || n == 576 || n == 640 || n == 1024 || n == 1152;
    return n == 80 || n == 96 || n == 144 || n == 160 || n == 192 || (prec != 0 && fp32_only) ? 0 : 2;
}

// Stage radices of length n on the half-length line kernels (radix[2] = 1: two
// stages), threads per line, and the z lines, y lines and rows of a workgroup;
// false if they do not take the length.
struct MixInfo {
    int radix[3];
    int nb, tile_z, tile_y, rows;
};
bool mix_info(int prec, int n, MixInfo &info);
// The same for the plane kernels on these line transforms (mix_plane.h): the
// x and y transforms of planes with nx = ny = n.
bool mix_plane_info(int prec, int n, MixInfo &info);
// Pass `mode` by half-length lines of n cells (x rows of n) for the problems of
// args, whose segments count mix_info() tiles or rows.
hipError_t launch_mix_lines(int mode, int prec, int n, const LaunchArgs &args, hipStream_t stream);

// Plane kernels (mix_plane.h) for the planes of args (one workgroup each).
hipError_t launch_mix_plane(bool fwd, int prec, int n, const LaunchArgs &args, hipStream_t stream);

// Green's-function spectrum in FP64: fills the octant (nz+1)(ny+1)(nx+1) of G
// into `a`, applies the even-extension cosine transform along each axis (using
// `b` as scratch) and writes the scaled result in plan precision into G / Gn.
// gz: the layout of G and Gn (above).
hipError_t green_spectrum(int nx, int ny, int nz, const double h[3], int prec, int gz, double *a, double *b,
                          const double *cos_x, const double *cos_y, const double *cos_z, void *G, void *Gn,
                          hipStream_t stream);

// Copy the spectrum out as a dense (nz+1)(ny+1)(nx+1) octant, kx fastest,
// whichever layout it is kept in.
hipError_t green_export(int nx, int ny, int nz, int prec, int gz, const void *G, const void *Gn, void *dst,
                        hipStream_t stream);

}  // namespace pspfft
