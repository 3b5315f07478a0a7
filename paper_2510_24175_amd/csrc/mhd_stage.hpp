// Fused Runge-Kutta stage kernel: ghost fill (index remap), conservative ->
// primitive, reconstruction (PLM or WENO-Z), GLM + Riemann fluxes on every
// face, flux divergence and the stage combine, in one pass over the grid.
//
// Work decomposition (gfx950, wave64):
//   * a workgroup owns a tile of TX = 64 (x) by TY (y) columns and marches
//     along z over a chunk of planes [k0, k1);
//   * one wave per tile row, one lane per column; the primitive state of
//     the current plane, with an x/y halo of the stencil's half width (2
//     cells PLM, 3 WENO-Z), sits in LDS;
//   * z-faces come from a per-lane register window slid along the march
//     (PLM: U(k+1) and the limited slope of V(k), with V(k) in LDS; WENO-Z:
//     V(k-1) .. V(k+2) and the upper face value of cell k), so every z-face
//     flux is computed once per chunk plus one warm-up face;
//   * x- and y-faces of the plane are a flat work list of
//     TY(TX+1) + (TY+1)TX items spread over the workgroup; their fluxes
//     go through LDS to the cells on both sides, so each face is solved
//     once per tile.  WENO-Z first reconstructs every cell the faces need
//     once per direction (both of its face values) into LDS;
//   * ghost cells are never stored: out-of-range coordinates are mapped to
//     interior cells by the boundary rule when addresses are formed.
// Stage kinds (KIND): 1 writes U1 = Un + dt L(Un); 2 the SSP-RK2 result
// (Un + U1 + dt L(U1)) / 2; 3 the SSP-RK3 stage 3/4 Un + 1/4 (U1 + dt L(U1));
// 4 the SSP-RK3 result 1/3 Un + 2/3 (U2 + dt L(U2)).  The last stage of
// either integrator damps psi and reduces on its output the CFL maxima and
// the FP64 conservation sums into per-block partials (with helper waves,
// the helpers take these reductions off the column owners).
#pragma once

#include <type_traits>

#include "mhd_physics.hpp"

namespace mhd {

constexpr int TX = 64;
// partial layout: [NPART][nblocks]; 0: max (|v|+cf)/dx, 1: max (|v|+cf),
// 2..10: sums of the 9 conserved components
constexpr int NPART = 11;

// grid of a marching kernel: TX x TY column tiles and z chunks of kz planes
struct Launch {
    int tiles_x, tiles_y, chunks, kz, nblocks;
};

template <typename T> struct StageArgs {
    const T *uin;   // state the fluxes are built from (Un or U1); with
                    // constrained transport its components 9..11 are the
                    // face field on each cell's lower x, y, z face
    T *flx;         // constrained transport with the mean edge EMF: [6][ncell]
                    // transverse field fluxes of each cell's lower faces
                    // (x: By, Bz; y: Bx, Bz; z: Bx, By); null with the
                    // upwind EMF, which does not use them
    const T *un;    // Un (later stages' combine); equals uin in stage 1
    T *uout;        // this stage's output (U1, U2 or U_next)
    double *part;   // last stage: NPART x nblocks partials
    int *flag;      // non-physical flag
    int nx, ny, nz; // interior cells
    long long nxy;  // nx*ny
    long long ncell;
    int per[3];     // periodic per axis
    int kz;         // planes per chunk
    int tiles_x, tiles_y, chunks;
    int nblocks;
    T dt;
    T idx[3];       // 1/dx per axis
    T damp;
    double gamma_d; // FP64 copies for the reductions
    double idx_d[3];
    Phys<T> ph;
};

// Logical block id from the hardware id.  Consecutive hardware ids are
// dispatched round-robin over the 8 XCDs; giving each XCD a contiguous
// range of logical ids keeps neighbouring tiles (shared halos) in one L2.
__device__ __forceinline__ int logical_block(int hw, int nblocks)
{
    if ((nblocks & 7) != 0) return hw;
    return (hw & 7) * (nblocks >> 3) + (hw >> 3);
}

// FP64 signal speeds of one conserved cell state (any T), for the CFL
// reduction: smax = max_d (|v_d| + c_f,d)/dx_d, cmax = max_d (|v_d| + c_f,d).
template <typename T, int NDIM>
__device__ __forceinline__ bool cell_speeds(const T *u, double gamma, const double *idx,
                                            double &smax, double &cmax)
{
    const double rho = (double)u[RHO];
    const double ir = 1.0 / rho;
    const double m[3] = {(double)u[MX], (double)u[MY], (double)u[MZ]};
    const double b[3] = {(double)u[BX], (double)u[BY], (double)u[BZ]};
    const double bsq = b[0] * b[0] + b[1] * b[1] + b[2] * b[2];
    const double kin = 0.5 * (m[0] * m[0] + m[1] * m[1] + m[2] * m[2]) * ir;
    const double p = (gamma - 1.0) * ((double)u[ENG] - kin - 0.5 * bsq);
    bool ok = (rho > 0.0) & (rho < 1e300) & (p > 0.0) & (p < 1e300);
#pragma unroll
    for (int d = 0; d < NDIM; ++d) {
        const double lam = __builtin_fabs(m[d] * ir) + fast_speed(p, bsq, b[d] * b[d], gamma, ir);
        smax = __builtin_fmax(smax, lam * idx[d]);
        cmax = __builtin_fmax(cmax, lam);
    }
    return ok;
}

// FP32 signal speeds of one FP32 cell state, used only to pick the cell
// whose FP64 speeds a thread reports: ls = max_d (|v_d| + c_f,d)/dx_d,
// lc = max_d (|v_d| + c_f,d).  The discriminant is formed from the
// transverse field, (a^2 - b^2)^2 + 4 a^2 b_t^2, a sum of non-negative terms;
// the estimate carries rounding of the order of ten FP32 ulps plus the FP32
// pressure's cancellation, which reaches |v| + c_f only through the sound
// speed (about gamma M / 4 ulps at Mach M).
// Returns false for rho <= 0, p <= 0 or non-finite values.
template <int NDIM>
__device__ __forceinline__ bool cell_speeds_f32(const float *u, float gamma, const float *idx, float &ls,
                                                float &lc)
{
    const float rho = u[RHO];
    const float ir = __builtin_amdgcn_rcpf(rho);
    const float m[3] = {u[MX], u[MY], u[MZ]};
    const float b[3] = {u[BX], u[BY], u[BZ]};
    const float bb[3] = {b[0] * b[0], b[1] * b[1], b[2] * b[2]};
    const float bsq = bb[0] + bb[1] + bb[2];
    const float kin = 0.5f * (m[0] * m[0] + m[1] * m[1] + m[2] * m[2]) * ir;
    const float p = (gamma - 1.0f) * (u[ENG] - kin - 0.5f * bsq);
    const bool ok = (rho > 0.0f) & (rho < 1e30f) & (p > 0.0f) & (p < 1e30f);
    const float a2 = gamma * p * ir;
    const float b2 = bsq * ir;
    const float dab = a2 - b2;
    ls = 0.0f;
    lc = 0.0f;
#pragma unroll
    for (int d = 0; d < NDIM; ++d) {
        const float bt2 = (bb[(d + 1) % 3] + bb[(d + 2) % 3]) * ir;
        const float disc = dab * dab + 4.0f * a2 * bt2;
        const float cf = __builtin_amdgcn_sqrtf(0.5f * (a2 + b2 + __builtin_amdgcn_sqrtf(disc)));
        const float lam = __builtin_fabsf(m[d] * ir) + cf;
        ls = __builtin_fmaxf(ls, lam * idx[d]);
        lc = __builtin_fmaxf(lc, lam);
    }
    return ok;
}

template <typename T>
__device__ __forceinline__ void load_cell(const T *__restrict__ U, long long ncell, long long c, T *u)
{
#pragma unroll
    for (int q = 0; q < NQ; ++q) u[q] = U[q * ncell + c];
}

// Wave64 sum / max of a double.
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ double wave_max(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = __builtin_fmax(v, __shfl_xor(v, o, 64));
    return v;
}

// Waves per SIMD the kernels are compiled for.  FP32 PLM in 8-row tiles: 4, a
// budget of 128 registers (the first stage needs 106, the last 128), two
// 8-wave workgroups per compute unit; a spilled register in the plane loop
// costs more than the wave it buys (a last stage with 21 spilled: 8.3 ms at
// 512^3 against 5.8 without).  FP32 PLM in 2D: 3.  FP32 WENO-Z: 2 (256
// registers; its 8-row workgroups take 155 KB of LDS, one per compute unit).
// FP64 PLM: 2 (256 registers, none spilled; one 8-wave workgroup of 154 KB per
// compute unit).  FP64 WENO-Z: 2 (140 KB of LDS, the fluxes laid over the
// primitive plane, allows one workgroup per compute unit: 4 rows with two
// waves each, the helper waves below).
template <typename T, int LIM, int TY> constexpr int stage_min_waves()
{
    return sizeof(T) == 4 ? (LIM == LIM_WENOZ ? 2 : (TY == 8 ? 4 : 3)) : 2;
}

// Waves per tile row.  FP64 WENO-Z's arrays leave room for one workgroup per
// compute unit; a second wave per row (a helper that owns no column) shares
// the halo conversions, the WENO-Z reconstructions and the x/y face fluxes
// of the plane, so that those phases run two waves per SIMD instead of one.
// The z march (register window, z faces) and the update stay with the
// column owners.
template <typename T, int LIM> constexpr int stage_row_waves()
{
    return (sizeof(T) == 8 && LIM == LIM_WENOZ) ? 2 : 1;
}

// Stage kinds of the Runge-Kutta integrators (KIND): 1 U1 = Un + dt L(Un)
// (first stage of both); 2 SSP-RK2 second and last stage
// (Un + U1 + dt L(U1))/2; 3 SSP-RK3 second stage 3/4 Un + 1/4 (U1 + dt L(U1));
// 4 SSP-RK3 last stage 1/3 Un + 2/3 (U2 + dt L(U2)).  The last stage damps
// psi and reduces the CFL maxima and the conservation sums.
constexpr bool last_stage(int kind) { return kind == 2 || kind == 4; }

template <typename T, int SOLVER, int LIM, int NDIM, int KIND, int TY, bool CT = false>
__global__ void __launch_bounds__(TX *TY *(stage_row_waves<T, LIM>()), (stage_min_waves<T, LIM, TY>()))
stage_kernel(const StageArgs<T> a)
{
    constexpr bool WENO = LIM == LIM_WENOZ;
    // with constrained transport the cell field is final only after the
    // face update, which therefore takes the last stage's reductions
    constexpr bool LAST = last_stage(KIND) && !CT;
    static_assert(!CT || NDIM == 3, "constrained transport is three-dimensional");
    constexpr int H = WENO ? 3 : 2;        // stencil half width (ghost layers)
    constexpr int NW = TY * stage_row_waves<T, LIM>();  // waves: TY column owners, then helpers
    constexpr int NT = TX * NW;
    constexpr int HY = NDIM >= 2 ? H : 0;  // y halo width in LDS
    constexpr int PX = TX + 2 * H;         // LDS row pitch
    constexpr int PY = TY + 2 * HY;        // LDS rows
    constexpr int PLANE = PX * PY;         // LDS elements per component
    constexpr int NFX = TY * (TX + 1);     // x-face items
    constexpr int NFY = NDIM >= 2 ? (TY + 1) * TX : 0;
    constexpr int NCHX = (NFX + TX - 1) / TX;       // 64-wide chunks of x items
    constexpr int NCHUNK = NCHX + NFY / TX;          // NFY is a multiple of TX
    constexpr int NHX = 2 * H * TY;        // x-halo cells
    constexpr int NH = NHX + (NDIM >= 2 ? 2 * H * TX : 0);
    // WENO-Z reconstructs every cell once per direction (both of its face
    // values) before the face fluxes: x for cells -1 .. TX of each row, y for
    // rows -1 .. TY of each column; the values go to LDS edge arrays
    // E[2][NQ][rows][cells] (right/upper face first).
    constexpr int NXE = TX + 2;                          // cells per row with an x edge
    constexpr int NYE = TY + 2;                          // rows with a y edge
    constexpr int NRX = WENO ? TY * NXE : 0;             // x reconstruction items
    constexpr int NRY = (WENO && NDIM >= 2) ? NYE * TX : 0;
    constexpr int NRCH = (NRX + NRY + TX - 1) / TX;      // their 64-wide chunks
    // LDS: [P][FX][FY] and, for WENO-Z, [EX][EY]; when that exceeds the 160 KB
    // of a compute unit (FP64), FX and FY go over P once P is used, and the
    // next plane's loads wait for the update (one more barrier per plane)
    constexpr int SZP = NQ * PLANE;
    constexpr int SZFX = NQ * TY * (TX + 1);
    constexpr int SZFY = NDIM >= 2 ? NQ * (TY + 1) * TX : 0;
    constexpr int SZEX = WENO ? 2 * NQ * TY * NXE : 0;
    constexpr int SZEY = (WENO && NDIM >= 2) ? 2 * NQ * NYE * TX : 0;
    constexpr bool ALIAS = WENO && (SZP + SZFX + SZFY + SZEX + SZEY) * (int)sizeof(T) > 160 * 1024;
    constexpr int OFX = ALIAS ? 0 : SZP;
    constexpr int OFY = OFX + SZFX;
    constexpr int OEX = ALIAS ? (SZP > SZFX + SZFY ? SZP : SZFX + SZFY) : OFY + SZFY;
    constexpr int OEY = OEX + SZEX;
    constexpr int SZL0 = OEY + SZEY;
    // Last stage with helper waves: the column owners leave each plane's
    // results in LDS (OUTS[NQ][TY * TX]) and the helpers take their FP64
    // sums and signal speeds during the next plane's z-face phase, which
    // is the owners' alone; the owners then carry no reduction state
    // through the march.
    constexpr bool HELP_RED = LAST && stage_row_waves<T, LIM>() > 1;
    static_assert(!HELP_RED || sizeof(T) == 8, "helper reductions keep FP64 sums in T registers");
    constexpr int OOUT = SZL0;
    // PLM in 8-row tiles: two workgroups leave room for the momentum and
    // energy of U(k) (ME), four registers that the last stage lacks
    constexpr bool ME_LDS = !WENO && NDIM == 3 && TY == 8;
    constexpr int SZL = OOUT + (HELP_RED ? NQ * TY * TX : 0) + (ME_LDS ? 4 * TY * TX : 0);
    static_assert(SZL * (int)sizeof(T) <= 160 * 1024, "LDS of one compute unit");

    __shared__ T lds[SZL];
    // With helper waves (FP64 WENO-Z) the reconstruction chunks of a plane
    // are handed out through this counter, one more barrier after the plane
    // load letting the helpers start on them while the column owners form the
    // plane's z faces (the owners take what is left): 416^3 SSP-RK3 step
    // 47.8 -> 46.2 ms.  The chunk order changes no arithmetic.
    constexpr bool OVERLAP = WENO && stage_row_waves<T, LIM>() > 1 && NDIM == 3;
    __shared__ int chunk_next;
    T *const P = lds;
    T *const FXs = lds + OFX;
    T *const FYs = lds + OFY;
    T *const EX = lds + OEX;
    T *const EY = lds + OEY;
    T *const OUTS = lds + OOUT;
    T *const ME = lds + OOUT;

    const int t = threadIdx.x;
    const int tx = t & (TX - 1);
    const int ty = t / TX;  // tile row of a column owner (>= TY: helper)
    const int wave = __builtin_amdgcn_readfirstlane(ty);
    // With one wave per tile row every wave owns its row.
    constexpr bool ALL_OWN = stage_row_waves<T, LIM>() == 1;
    const bool owner = ALL_OWN || wave < TY;  // wave-uniform
    const int lb = logical_block(blockIdx.x, a.nblocks);
    const int tile_x = lb % a.tiles_x;
    const int rest = lb / a.tiles_x;
    // 3D: planes [k0, k1) of one column tile.  In two dimensions the march is
    // over the tiles [k0, k1) of a strip along y (in one, a single tile).
    const int tile_y = NDIM == 3 ? rest % a.tiles_y : 0;
    const int chunk = rest / a.tiles_y;
    const int i0 = tile_x * TX;
    const int k0 = chunk * a.kz;
    const int k1 = min(k0 + a.kz, NDIM == 3 ? a.nz : (a.ny + TY - 1) / TY);
    const int i = i0 + tx;
    int j0 = 0;
    bool active = false;
    // own column (remapped so that columns just past the grid edge hold the
    // ghost values their active neighbours need)
    auto own_of = [&](int row0) -> long long {
        return (long long)remap_index(row0 + ty, a.ny, a.per[1]) * a.nx + remap_index(i, a.nx, a.per[0]);
    };
    long long own = 0;
    // halo cells of this thread: LDS slot and offset
    constexpr int HPT = (NH + NT - 1) / NT;  // halo cells per thread
    int h_slot[HPT];
    long long h_off[HPT];
    // the tile whose first row is row0
    auto set_tile = [&](int row0) {
        j0 = row0;
        active = owner & (i < a.nx) & (j0 + ty < a.ny);
        own = own_of(j0);
#pragma unroll
        for (int m = 0; m < HPT; ++m) {
            const int h = t + m * NT;
            h_slot[m] = 0;
            h_off[m] = 0;
            if (h < NH) {
                int lx, ly;
                if (h < NHX) {
                    const int r = h / (2 * H), s = h % (2 * H);
                    lx = s < H ? s : TX + s;
                    ly = r + HY;
                } else {
                    const int hy = h - NHX;
                    const int rh = hy / TX, c = hy % TX;
                    lx = c + H;
                    ly = rh < H ? rh : TY + rh;
                }
                h_slot[m] = ly * PX + lx;
                const int gi = remap_index(i0 + lx - H, a.nx, a.per[0]);
                const int gj = remap_index(j0 + ly - HY, a.ny, a.per[1]);
                h_off[m] = (long long)gj * a.nx + gi;
            }
        }
    };
    set_tile((NDIM == 3 ? tile_y : k0) * TY);
    const int own_slot = (ty + HY) * PX + tx + H;
    bool ok = true;

    auto zoff = [&](int k) -> long long {
        return NDIM == 3 ? (long long)remap_index(k, a.nz, a.per[2]) * a.nxy : 0;
    };
    auto prim_at = [&](long long c, T *v) {
        T u[NQ];
        load_cell(a.uin, a.ncell, c, u);
        ok &= cons_to_prim(u, a.ph, v);
    };
    // the same, keeping the conserved momentum and energy
    auto prim_at_keep = [&](long long c, T *v, T *me) {
        T u[NQ];
        load_cell(a.uin, a.ncell, c, u);
        ok &= cons_to_prim(u, a.ph, v);
#pragma unroll
        for (int q = 0; q < 4; ++q) me[q] = u[MX + q];
    };
    auto slope9 = [&](const T *vm, const T *v0, const T *vp, T *s) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) s[q] = limited_slope<LIM>(v0[q] - vm[q], vp[q] - v0[q]);
    };

    // Constrained transport: the cell (plane offset) whose lower face item tx
    // of chunk ch is, and that face's value, the normal field of its Riemann
    // problem.  Loaded one chunk ahead (the first before the plane's
    // reconstructions): a load at the face itself exposes its latency.
    auto face_cell = [&](int ch) -> long long {
        int x, y;
        if (ch < NCHX) {
            const int it = min(ch * TX + tx, NFX - 1);
            y = it / (TX + 1);
            x = it - y * (TX + 1);
        } else {
            x = tx;
            y = ch - NCHX;
        }
        return (long long)remap_index(j0 + y, a.ny, a.per[1]) * a.nx + remap_index(i0 + x, a.nx, a.per[0]);
    };
    auto face_field = [&](int ch, long long zk) -> T {
        return a.uin[(ch < NCHX ? 9 : 10) * a.ncell + zk + face_cell(ch)];
    };
    T bn_next = T(0);
    // Flux through a face of chunk ch of the plane (offset zk) from its two
    // states, stored in LDS.  (x, y) is the tile cell whose lower face this
    // is.  Constrained transport: for the tile's own faces (mine) of grid
    // cells, the two transverse field fluxes go to flx.
    auto flux_item = [&](auto dir, const T *VL, const T *VR, T *dst, int fstride, long long zk, int ch, int x,
                         int y, bool mine) {
        constexpr int D = decltype(dir)::value;
        T F[NQ];
        if constexpr (CT) {
            const T bn = bn_next;
            if (ch + NW < NCHUNK) bn_next = face_field(ch + NW, zk);
            face_flux<T, SOLVER, true>(VL, VR, D, a.ph, F, bn);
            if (mine && (i0 + x < a.nx) & (j0 + y < a.ny) && a.flx) {
                const long long fc = zk + face_cell(ch);
                a.flx[(2 * D) * a.ncell + fc] = F[D == 0 ? BY : BX];
                a.flx[(2 * D + 1) * a.ncell + fc] = F[BZ];
            }
        } else {
            face_flux<T, SOLVER>(VL, VR, D, a.ph, F);
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) dst[q * fstride] = F[q];
    };
    // PLM face from the LDS stencil w0..w3 (stride apart; the face lies
    // between w1 and w2): limited slopes of w1 and w2, face states, flux.
    auto face_item = [&](auto dir, const T *base, int stride, T *dst, int fstride, long long zk, int ch, int x,
                         int y, bool mine) {
        T VL[NQ], VR[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const T *pq = base + q * PLANE;
            const T w0 = pq[0], w1 = pq[stride], w2 = pq[2 * stride], w3 = pq[3 * stride];
            const T s1 = limited_slope<LIM>(w1 - w0, w2 - w1);
            const T s2 = limited_slope<LIM>(w2 - w1, w3 - w2);
            VL[q] = w1 + T(0.5) * s1;
            VR[q] = w2 - T(0.5) * s2;
        }
        flux_item(dir, VL, VR, dst, fstride, zk, ch, x, y, mine);
    };

    // z window.  PLM: the conserved U(k+1), the limited slope D0 of V(k) and the
    // momentum and energy of U(k); V(k) itself is the own cell of the LDS
    // plane, and density, field and psi are the same in U and V, so the
    // combine needs no second read of the state.  WENO-Z: V(k-1) .. V(k+2) and
    // ZT, the upper face value of cell k.  Fzm is the flux through face k-1/2.
    constexpr int ZW = WENO ? 4 : 1;
    constexpr int ZC = WENO ? 1 : 0;       // window slot of plane k (WENO-Z)
    T Wz[ZW][NQ], D0[NQ], ZT[NQ], Fzm[NQ], me0[4], un1[NQ];
    // A helper wave keeps its running FP64 sums of the cells its row's owner
    // left in OUTS (same column) in Fzm and its maxima of the signal speeds
    // in ZT[0..1]: registers the owners hold through the march anyway and
    // the helpers have no other use for.  Cells outside the grid count
    // nothing.
    int j0_out = j0;  // first row of the tile whose results are in OUTS
    auto helper_fold = [&]() {
        const int row = wave - TY;
        if ((i < a.nx) & (j0_out + row < a.ny)) {
            T u[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                u[q] = OUTS[q * TY * TX + row * TX + tx];
                Fzm[q] += u[q];
            }
            double smx = ZT[0], cmx = ZT[1];
            ok &= cell_speeds<T, NDIM>(u, a.gamma_d, a.idx_d, smx, cmx);
            ZT[0] = smx;
            ZT[1] = cmx;
        }
    };
    if (HELP_RED && !owner) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) Fzm[q] = ZT[q] = T(0);
    }
    if (NDIM == 3 && owner) {
        T VL[NQ], VR[NQ];
        if constexpr (WENO) {
            // cell k0-1 gives the lower state of face k0-1/2, cell k0 the
            // upper one and its own upper face value
            T Vm3[NQ], Vm2[NQ];
            prim_at(zoff(k0 - 3) + own, Vm3);
            prim_at(zoff(k0 - 2) + own, Vm2);
#pragma unroll
            for (int m = 0; m < 4; ++m) prim_at(zoff(k0 - 1 + m) + own, Wz[m]);
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                T lo;
                wenoz_pair(Vm3[q], Vm2[q], Wz[0][q], Wz[1][q], Wz[2][q], VL[q], lo);
                wenoz_pair(Vm2[q], Wz[0][q], Wz[1][q], Wz[2][q], Wz[3][q], ZT[q], VR[q]);
            }
        } else {
            T Vm2[NQ], Vm1[NQ], V0[NQ], Dm1[NQ];
            prim_at(zoff(k0 - 2) + own, Vm2);
            prim_at(zoff(k0 - 1) + own, Vm1);
            prim_at_keep(zoff(k0) + own, V0, me0);
            load_cell(a.uin, a.ncell, zoff(k0 + 1) + own, un1);
            T V1[NQ];
            ok &= cons_to_prim(un1, a.ph, V1);
            slope9(Vm2, Vm1, V0, Dm1);
            slope9(Vm1, V0, V1, D0);
            if (ME_LDS) {
#pragma unroll
                for (int q = 0; q < 4; ++q) ME[q * TY * TX + t] = me0[q];
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                VL[q] = Vm1[q] + T(0.5) * Dm1[q];
                VR[q] = V0[q] - T(0.5) * D0[q];
                P[q * PLANE + own_slot] = V0[q];
            }
        }
        if constexpr (CT)
            face_flux<T, SOLVER, true>(VL, VR, 2, a.ph, Fzm, a.uin[11 * a.ncell + zoff(k0) + own]);
        else
            face_flux<T, SOLVER>(VL, VR, 2, a.ph, Fzm);
    }

    double smax = 0.0, cmax = 0.0;
    // FP64 speeds of every cell; in 3D FP32 only of the planes of this thread's
    // column with the largest FP32 estimates of the two maxima, taken at the end
    // (in 1D its one cell)
    constexpr bool ALL_SPEEDS = sizeof(T) == 8 || NDIM == 2;
    float best_s = -1.0f, best_c = -1.0f;
    int k_s = -1, k_c = -1;
    double sum[HELP_RED ? 1 : NQ];
#pragma unroll
    for (int q = 0; q < (HELP_RED ? 1 : NQ); ++q) sum[q] = 0.0;

    // divergence and stage combine of the own cell of plane k from its
    // conserved input state cin, the plane's x and y fluxes in LDS and the z
    // fluxes Fzm and Fzp
    auto update = [&](int k, long long c, const T *cin, const T *cun, const T *Fzp) {
        T L[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const T *fx = &FXs[q * TY * (TX + 1) + ty * (TX + 1) + tx];
            T l = (fx[0] - fx[1]) * a.idx[0];
            if (NDIM >= 2) {
                const T *fy = &FYs[q * (TY + 1) * TX + ty * TX + tx];
                l += (fy[0] - fy[TX]) * a.idx[1];
            }
            if (NDIM == 3) l += (Fzm[q] - Fzp[q]) * a.idx[2];
            L[q] = l;
        }
        T out[NQ];
        if (KIND == 1) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) out[q] = cin[q] + a.dt * L[q];
        } else if (KIND == 2) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) out[q] = T(0.5) * ((cun[q] + cin[q]) + a.dt * L[q]);
        } else if (KIND == 3) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) out[q] = T(0.75) * cun[q] + T(0.25) * (cin[q] + a.dt * L[q]);
        } else {
#pragma unroll
            for (int q = 0; q < NQ; ++q) out[q] = cun[q] * T(1.0 / 3.0) + T(2.0 / 3.0) * (cin[q] + a.dt * L[q]);
        }
        if (LAST) out[PSI] *= a.damp;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            // constrained transport: the face update writes the cell field
            if (CT && q >= BX && q <= BZ) continue;
            __builtin_nontemporal_store(out[q], &a.uout[q * a.ncell + c]);  // not read again here
        }
        if (CT && a.flx) {
            // transverse field fluxes of this cell's lower z face
            a.flx[4 * a.ncell + c] = Fzm[BX];
            a.flx[5 * a.ncell + c] = Fzm[BY];
        }
        if constexpr (HELP_RED) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) OUTS[q * TY * TX + t] = out[q];
        } else if (LAST) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) sum[q] += (double)out[q];
            if constexpr (ALL_SPEEDS) {
                ok &= cell_speeds<T, NDIM>(out, a.gamma_d, a.idx_d, smax, cmax);
            } else {
                float ls, lc;
                ok &= cell_speeds_f32<NDIM>(out, a.ph.gamma, a.idx, ls, lc);
                k_s = ls > best_s ? k : k_s;
                best_s = __builtin_fmaxf(best_s, ls);
                k_c = lc > best_c ? k : k_c;
                best_c = __builtin_fmaxf(best_c, lc);
            }
        }
    };

    // PLM.  Per plane: the x and y faces from the LDS plane, then the z face,
    // the update and the next plane's primitives.  The own cells of plane k+2
    // are loaded before the x and y faces and used after them, so that their
    // latency hides behind the faces; the halo cells of plane k+1 are loaded
    // before the z face in FP32, with Un, and after it in FP64, before the update
    // (128^3 step 333 -> 317 us against after the update, where they wait for its
    // stores; before the z face 256^3 stages 1.26 + 1.39 ms against 1.23 + 1.36).
    // Each cell is
    // read once as an own cell and once per halo that holds it: 512^3 FP32
    // fetches 7.9 GB in the first stage (4.8 compulsory) against 11.8 when the
    // combine re-read the state, and the stages take 3.83 + 4.55 ms against
    // 4.30 + 5.42 with the z face first, the re-read and 4-row tiles (256^3
    // FP64 1.23 + 1.36 against 1.37 + 1.64).  About 70% of the time is VALU
    // issue (3.2 face rounds of ~270 instructions per 64 cells), the rest
    // waits for LDS, barriers and memory.
    if constexpr (!WENO) {
        constexpr bool EARLY = sizeof(T) == 4;
        auto load_halo = [&](long long z, T (*h)[NQ]) {
#pragma unroll
            for (int m = 0; m < HPT; ++m)
                if (t + m * NT < NH) load_cell(a.uin, a.ncell, z + h_off[m], h[m]);
        };
        auto put_halo = [&](T (*h)[NQ]) {
#pragma unroll
            for (int m = 0; m < HPT; ++m) {
                if (t + m * NT < NH) {
                    T hv[NQ];
                    ok &= cons_to_prim(h[m], a.ph, hv);
#pragma unroll
                    for (int q = 0; q < NQ; ++q) P[q * PLANE + h_slot[m]] = hv[q];
                }
            }
        };
        // x and y faces of plane k.  Items go out in 64-wide chunks, one
        // chunk per wave at a time; x items are padded to whole chunks so
        // every chunk is a single direction and the solver is inlined with a
        // compile-time frame.
        auto plane_faces = [&](int k) {
            // no y faces past those of the grid's last row (256 x 2 x 256 FP64 step
            // 75.5 -> 60.2 us)
            const int nch = NDIM == 3 ? NCHX + min(TY, a.ny - j0) + 1 : NCHUNK;
            for (int ch = wave; ch < nch; ch += NW) {
                if (ch < NCHX) {
                    // lanes past the last item repeat it (same values, same slot)
                    const int it = min(ch * TX + tx, NFX - 1);
                    const int r = it / (TX + 1), f = it - r * (TX + 1);
                    // cells f-2 .. f+1 of row r
                    face_item(std::integral_constant<int, 0>{}, &P[(r + HY) * PX + f], 1, &FXs[it],
                              TY * (TX + 1), zoff(k), ch, f, r, f < TX);
                } else {
                    const int it = (ch - NCHX) * TX + tx;
                    const int r = it / TX, f = it - r * TX;
                    // rows r-2 .. r+1 of column f
                    face_item(std::integral_constant<int, 1>{}, &P[r * PX + f + H], PX, &FYs[it],
                              (TY + 1) * TX, zoff(k), ch, f, r, r < TY);
                }
            }
        };
        T hu[HPT][NQ];
        load_halo(zoff(k0), hu);
        if constexpr (NDIM < 3) {
            // a strip of tiles; the next tile's cells are loaded before the
            // faces of one and used after them
            T uo[NQ];
            load_cell(a.uin, a.ncell, own, uo);
            for (int k = k0; k < k1; ++k) {
                const long long c = own;
                const bool mine = active;
                T cin[NQ], cun[NQ], V0[NQ];
#pragma unroll
                for (int q = 0; q < NQ; ++q) cin[q] = uo[q];
                ok &= cons_to_prim(cin, a.ph, V0);
#pragma unroll
                for (int q = 0; q < NQ; ++q) P[q * PLANE + own_slot] = V0[q];
                put_halo(hu);
                __syncthreads();
                if (KIND != 1) load_cell(a.un, a.ncell, c, cun);
                if (k + 1 < k1) {
                    set_tile((k + 1) * TY);
                    load_cell(a.uin, a.ncell, own, uo);
                    load_halo(0, hu);
                }
                plane_faces(k);
                __syncthreads();
                if (mine) update(k, c, cin, cun, cun);
            }
        } else {
            put_halo(hu);
            __syncthreads();
            for (int k = k0; k < k1; ++k) {
                const long long c = zoff(k) + own;
                T un2[NQ], bnz = T(0);
                if (CT && wave < NCHUNK) bn_next = face_field(wave, zoff(k));
                load_cell(a.uin, a.ncell, zoff(k + 2) + own, un2);
                if (CT) bnz = a.uin[11 * a.ncell + zoff(k + 1) + own];
                plane_faces(k);
                __syncthreads();
                if (EARLY && k + 1 < k1) load_halo(zoff(k + 1), hu);
                T V0[NQ], V1[NQ], D1[NQ], Fzp[NQ], cun[NQ];
                if (EARLY && KIND != 1) load_cell(a.un, a.ncell, c, cun);
#pragma unroll
                for (int q = 0; q < NQ; ++q) V0[q] = P[q * PLANE + own_slot];
                {
                    T V2[NQ], VL[NQ], VR[NQ];
                    cons_to_prim(un1, a.ph, V1);
                    ok &= cons_to_prim(un2, a.ph, V2);
                    slope9(V0, V1, V2, D1);
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        VL[q] = V0[q] + T(0.5) * D0[q];
                        VR[q] = V1[q] - T(0.5) * D1[q];
                    }
                    if constexpr (CT)
                        face_flux<T, SOLVER, true>(VL, VR, 2, a.ph, Fzp, bnz);
                    else
                        face_flux<T, SOLVER>(VL, VR, 2, a.ph, Fzp);
                }
                if (!EARLY && k + 1 < k1) load_halo(zoff(k + 1), hu);
                if (active) {
                    if (!EARLY && KIND != 1) load_cell(a.un, a.ncell, c, cun);
                    if (ME_LDS) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) me0[q] = ME[q * TY * TX + t];
                    }
                    const T cin[NQ] = {V0[RHO], me0[0], me0[1], me0[2], me0[3], V0[BX], V0[BY], V0[BZ], V0[PSI]};
                    update(k, c, cin, cun, Fzp);
                }
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    P[q * PLANE + own_slot] = V1[q];
                    D0[q] = D1[q];
                    Fzm[q] = Fzp[q];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (ME_LDS) ME[q * TY * TX + t] = un1[MX + q];
                    else me0[q] = un1[MX + q];
                }
#pragma unroll
                for (int q = 0; q < NQ; ++q) un1[q] = un2[q];
                if (k + 1 < k1) put_halo(hu);
                __syncthreads();
            }
        }
    }

    // WENO-Z.  In 3D the halo cells of plane k+1 are loaded before the face
    // fluxes of plane k and converted at its start: a load issued there waits
    // for its own latency and for the update's stores before it.  256^3 stages
    // FP64 2.54, 2.66 and 2.79 -> 2.40, 2.57 and 2.68 ms; loaded before the
    // reconstructions 2.45, 2.60 and 2.65, before the z faces no gain.  FP32
    // also loads the input state of the combine there, 1.50, 1.53 and 1.61 ->
    // 1.44, 1.50 and 1.55 ms (FP64 spills with it, and either type with Un or
    // the own cells of plane k+4 as well).  Not with constrained transport:
    // its FP64 stages spill 22 registers then (352^3 step 28.5 -> 33.9 ms), its
    // FP32 ones gain nothing (176^3 2.40 -> 2.42 ms).
    if constexpr (WENO) {
        constexpr bool AHEAD = NDIM == 3 && !CT;
        constexpr bool EARLY_IN = AHEAD && sizeof(T) == 4;
        T hu[HPT][NQ];
        auto load_halo = [&](int k) {
#pragma unroll
            for (int m = 0; m < HPT; ++m)
                if (t + m * NT < NH) load_cell(a.uin, a.ncell, zoff(k) + h_off[m], hu[m]);
        };
        if (AHEAD) load_halo(k0);
        for (int k = k0; k < k1; ++k) {
            const long long zk = zoff(k);
            if constexpr (NDIM < 3) {
                // the next tile of the strip
                if (k > k0) set_tile(k * TY);
                if (owner) prim_at(own, Wz[ZC]);
            }
            T bnz = T(0);
            if (CT && wave < NCHUNK) bn_next = face_field(wave, zk);
            if (CT && owner) bnz = a.uin[11 * a.ncell + zoff(k + 1) + own];
            // the fluxes of the previous plane sit where P goes; the helpers
            // read the previous plane's results
            if ((ALIAS || HELP_RED) && k > k0) __syncthreads();
            // (a) primitives of plane k into LDS: own column and halo cell
            if (owner) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) P[q * PLANE + own_slot] = Wz[ZC][q];
            }
#pragma unroll
            for (int m = 0; m < HPT; ++m) {
                if (t + m * NT < NH) {
                    T hv[NQ];
                    if (AHEAD)
                        ok &= cons_to_prim(hu[m], a.ph, hv);
                    else
                        prim_at(zk + h_off[m], hv);
#pragma unroll
                    for (int q = 0; q < NQ; ++q) P[q * PLANE + h_slot[m]] = hv[q];
                }
            }
            if constexpr (OVERLAP) {
                // the plane is in LDS: the reconstructions may start
                if (t == 0) chunk_next = 0;
                __syncthreads();
            }
            // (the previous plane's results stay until this plane's update,
            // several barriers on)
            if (HELP_RED && !owner && k > k0) helper_fold();
            // (b) z-face k+1/2 from the register window
            T Fzp[NQ];
            if (NDIM == 3 && owner) {
                T Vn[NQ], VL[NQ], VR[NQ];
                prim_at(zoff(k + ZW - ZC) + own, Vn);  // V(k+3)
                // cell k+1: its lower face value closes face k+1/2, its upper
                // one is carried to the next plane
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    VL[q] = ZT[q];
                    wenoz_pair(Wz[0][q], Wz[1][q], Wz[2][q], Wz[3][q], Vn[q], ZT[q], VR[q]);
                }
                if constexpr (CT)
                    face_flux<T, SOLVER, true>(VL, VR, 2, a.ph, Fzp, bnz);
                else
                    face_flux<T, SOLVER>(VL, VR, 2, a.ph, Fzp);
                // The flux is used after the x/y faces: without a use here the
                // compiler moves half of the z face past them and keeps its
                // intermediates (about 40 registers) live across them.
#pragma unroll
                for (int q = 0; q < NQ; ++q) asm volatile("" : "+v"(Fzp[q]));
                // slide the window by one plane
#pragma unroll
                for (int m = 0; m + 1 < ZW; ++m) {
#pragma unroll
                    for (int q = 0; q < NQ; ++q) Wz[m][q] = Wz[m + 1][q];
                }
#pragma unroll
                for (int q = 0; q < NQ; ++q) Wz[ZW - 1][q] = Vn[q];
            }
            if constexpr (!OVERLAP) __syncthreads();
            // (c0) WENO-Z face values of every cell the plane's faces need,
            // each from the five cells centred on it: x items for cells
            // -1 .. TX of each row, y items for rows -1 .. TY of each column.
            // Direction only changes addresses, so chunks mix the two.
            auto next_chunk = [&](int ch) -> int {
                if constexpr (OVERLAP) {
                    int c = 0;
                    if (tx == 0) c = atomicAdd(&chunk_next, 1);
                    return __builtin_amdgcn_readfirstlane(c);
                } else {
                    return ch + NW;
                }
            };
            for (int ch = OVERLAP ? next_chunk(0) : wave; ch < NRCH; ch = next_chunk(ch)) {
                const int it = ch * TX + tx;
                if (it < NRX + NRY) {
                    const T *src;
                    int stride;
                    T *dst;
                    int esize;
                    if (it < NRX) {
                        const int r = it / NXE, c = it - r * NXE;
                        src = &P[(r + HY) * PX + c];
                        stride = 1;
                        dst = &EX[r * NXE + c];
                        esize = NQ * TY * NXE;
                    } else {
                        const int iy = it - NRX;
                        const int r = iy / TX, c = iy - r * TX;
                        src = &P[r * PX + c + H];
                        stride = PX;
                        dst = &EY[r * TX + c];
                        esize = NQ * NYE * TX;
                    }
                    const int qs = esize / NQ;
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        const T *pq = src + q * PLANE;
                        T hi, lo;
                        wenoz_pair(pq[0], pq[stride], pq[2 * stride], pq[3 * stride], pq[4 * stride], hi, lo);
                        dst[q * qs] = hi;
                        dst[esize + q * qs] = lo;
                    }
                }
            }
            __syncthreads();
            T cin[NQ];
            if (EARLY_IN) load_cell(a.uin, a.ncell, zk + own, cin);
            if (AHEAD && k + 1 < k1) load_halo(k + 1);
            // (c1) face fluxes from the edge values: x face f of row r between
            // cells f-1 and f, y face r of column c between rows r-1 and r;
            // (the fluxes overwrite P when the LDS is aliased)
            for (int ch = wave; ch < NCHUNK; ch += NW) {
                T VL[NQ], VR[NQ];
                if (ch < NCHX) {
                    const int it = min(ch * TX + tx, NFX - 1);  // lanes past the last item repeat it
                    const int r = it / (TX + 1), f = it - r * (TX + 1);
                    constexpr int QS = TY * NXE;
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        VL[q] = EX[q * QS + r * NXE + f];
                        VR[q] = EX[NQ * QS + q * QS + r * NXE + f + 1];
                    }
                    flux_item(std::integral_constant<int, 0>{}, VL, VR, &FXs[it], TY * (TX + 1), zk, ch, f, r, f < TX);
                } else {
                    const int it = (ch - NCHX) * TX + tx;
                    const int r = it / TX, c = it - r * TX;
                    constexpr int QS = NYE * TX;
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        VL[q] = EY[q * QS + r * TX + c];
                        VR[q] = EY[NQ * QS + q * QS + (r + 1) * TX + c];
                    }
                    flux_item(std::integral_constant<int, 1>{}, VL, VR, &FYs[it], (TY + 1) * TX, zk, ch, c, r, r < TY);
                }
            }
            __syncthreads();
            // (d) divergence and stage combine
            if (active) {
                const long long c = zk + own;
                T cun[NQ];
                if (!EARLY_IN) load_cell(a.uin, a.ncell, c, cin);
                if (KIND != 1) load_cell(a.un, a.ncell, c, cun);
                update(k, c, cin, cun, Fzp);
            }
            j0_out = j0;
            if (NDIM == 3 && owner) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) Fzm[q] = Fzp[q];
            }
        }
    }

    if constexpr (LAST && !ALL_SPEEDS) {
        // FP64 speeds of the selected cells, re-read from this thread's own
        // output (it stored them above)
        if (k_s >= 0) {
            T u[NQ];
            load_cell(a.uout, a.ncell, zoff(k_s) + own, u);
            ok &= cell_speeds<T, NDIM>(u, a.gamma_d, a.idx_d, smax, cmax);
        }
        if (k_c >= 0 && k_c != k_s) {
            T u[NQ];
            load_cell(a.uout, a.ncell, zoff(k_c) + own, u);
            ok &= cell_speeds<T, NDIM>(u, a.gamma_d, a.idx_d, smax, cmax);
        }
    }
    if (LAST) {
        // block reduction of the partials in a fixed order: every column's
        // values to LDS, then wave w takes the quantities w, w + NW, ..., folds
        // the rows per lane and the lanes by a wave reduction (two or three of
        // the eleven a wave; all eleven in every wave made the last stage of a
        // 1024^2 grid, with one tile per workgroup, 62 us against 34 for the
        // first)
        constexpr int COLS = TX * TY;
        static_assert(NPART * COLS * 8 <= SZL * (int)sizeof(T) || NDIM == 1, "LDS for the partials");
        __syncthreads();
        double *red = reinterpret_cast<double *>(P);  // LDS reuse
        double vals[NPART];
        if constexpr (HELP_RED) {
            if (!owner) helper_fold();  // the chunk's last plane
            vals[0] = ZT[0];
            vals[1] = ZT[1];
#pragma unroll
            for (int q = 0; q < NQ; ++q) vals[2 + q] = Fzm[q];
        } else {
            vals[0] = smax;
            vals[1] = cmax;
#pragma unroll
            for (int q = 0; q < NQ; ++q) vals[2 + q] = sum[q];
        }
        if constexpr (NDIM == 1) {
            // a single row: its reducing wave takes all
            if (HELP_RED ? !owner : owner) {
#pragma unroll
                for (int e = 0; e < NPART; ++e) {
                    const double r = e < 2 ? wave_max(vals[e]) : wave_sum(vals[e]);
                    if (tx == 0) a.part[(long long)e * a.nblocks + lb] = r;
                }
            }
        } else {
            // the row's reducing wave: its helper, or its owner
            if (HELP_RED ? !owner : owner) {
                const int row = HELP_RED ? wave - TY : ty;
#pragma unroll
                for (int e = 0; e < NPART; ++e) red[e * COLS + row * TX + tx] = vals[e];
            }
            __syncthreads();
            for (int e = wave; e < NPART; e += NW) {
                double r = red[e * COLS + tx];
                for (int w = 1; w < TY; ++w) {
                    const double x = red[e * COLS + w * TX + tx];
                    r = e < 2 ? __builtin_fmax(r, x) : r + x;
                }
                r = e < 2 ? wave_max(r) : wave_sum(r);
                if (tx == 0) a.part[(long long)e * a.nblocks + lb] = r;
            }
        }
    }
    if (!ok) *a.flag = 1;
}

} // namespace mhd
