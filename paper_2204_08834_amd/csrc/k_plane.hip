// k_plane.hip -- transforms along x and y of one z-plane by one workgroup
// (steps 1-3 and 7-9 of the solve sequence in FluTAS Section 3.3.1), for
// planes whose spectrum fits the LDS of one compute unit.
//
// Separately, the x pass writes the half spectrum of every row to HBM and the
// y pass reads it back: 2 s bytes per point (s = 4 or 8) and one launch more
// in each direction.  Here the last x pass leaves the rows in LDS and the y
// transform runs down their columns, so a plane is read once and written
// once: FP64 forward + inverse 64 -> 32 bytes per point, FP32 (first solve)
// 36 -> 20.  What bounds it: HBM for batches (many planes in flight), the
// latency of one workgroup's passes for a single small box.  Whole solves,
// separate passes -> planes: 32^3 FP64 27.2 -> 21.2 us, 64^3 periodic 53.3 ->
// 46.9, 128x128x64 FP64 64.8 -> 61.1, 96x96x48 FP32 + refinement 125.5 ->
// 113.1, batch of 64 boxes FP32 + refinement 1016 -> 954, and 896 with the
// tables fetched ahead of the field and the lists split by plane size.  Few
// large planes keep the separate passes (plane_pays).
//
// The arithmetic is that of k_xpass.hip and k_ypass.hip (same radix plans,
// tables and pair formulas).  The length along x is a compile-time constant,
// the number of rows is not: with radices 8, 4, 2 before the 3s every
// sub-transform length that a pass splits off is a power of two, so the y
// passes need no division by it.
//
// Compiled once per precision with PK_REAL = float or double.
#include <type_traits>

#include "fft_core.hpp"
#include "lengths.hpp"
#include "plane_lists.hpp"
#include "stencil.hpp"

#ifndef PK_REAL
#error "PK_REAL must be defined"
#endif

namespace pk {
namespace PK_NS {

using R = PK_REAL;

#include "xpair.hpp"

// Values per thread, EPT: 8 complex values keep a pass's inputs in registers
// across the barrier between its reads and its writes at about 64 (FP32) or
// 90 (FP64) VGPRs; planes of more than 8 * 1024 values (FP32 only: 128 KB of
// the 160 KB of LDS) take 16.
constexpr int PL_MAXT = 1024;
constexpr int pl_ept(int elems) { return elems <= 8 * PL_MAXT ? 8 : 16; }
constexpr int PL_ELEMS = (sizeof(R) == 4 ? 16 : 8) * PL_MAXT;

// A plane in LDS: row n of M complex values at n * PITCH.  Within a row,
// value m sits at m ^ ((m >> 3) & 7): the first x pass of radix 8 stores at
// stride 8, which without the swizzle puts eight lanes on the same banks.
// Both the x passes (consecutive lanes along a row) and the y passes
// (consecutive lanes across m) read aligned groups of eight, permuted.
template <int M> struct PlaneTile {
    static constexpr int PITCH = (M + 7) / 8 * 8 + 1;
    Cx<R> *base;
    __device__ __forceinline__ Cx<R> &at(int row, int m) const
    {
        return base[row * PITCH + (m ^ ((m >> 3) & 7))];
    }
};

// One Stockham pass over `nbf` butterflies, spread over nt threads:
// loc(u, line, j) gives butterfly u's line and index, kof(j) = j mod ns, ld
// and st move its values.  MIDSYNC: st overwrites what ld reads, so every
// value is read before the barrier and written after it.
// `loaded` runs once the loads are issued.
struct Nothing {
    __device__ __forceinline__ void operator()() const {}
};
template <int EPT, int RAD, bool MIDSYNC, class Loc, class Kof, class Ld, class St, class Hook>
__device__ __forceinline__ void plane_pass(int nbf, int nt, const Cx<R> *tw, int tws, int nj,
                                           int ns, Loc &&loc, Kof &&kof, Ld &&ld, St &&st,
                                           Hook &&loaded)
{
    constexpr int PER = (EPT + RAD - 1) / RAD;
    Cx<R> v[PER][RAD];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int u = threadIdx.x + q * nt;
        if (u < nbf) {
            int b, j;
            loc(u, b, j);
#pragma unroll
            for (int r = 0; r < RAD; ++r) v[q][r] = ld(b, j + r * nj);
        }
    }
    loaded();
    if (MIDSYNC) __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int u = threadIdx.x + q * nt;
        if (u < nbf) {
            int b, j;
            loc(u, b, j);
            const int k = ns > 1 ? kof(j) : 0;
            if (ns > 1) {
#pragma unroll
                for (int r = 1; r < RAD; ++r) v[q][r] = cmul(v[q][r], tw[r * k * tws]);
            }
            Bfly<R, RAD>::run(v[q]);
            const int base = (j - k) * RAD + k;
#pragma unroll
            for (int r = 0; r < RAD; ++r) st(b, base + r * ns, v[q][r]);
        }
    }
}

// The transform of length n (run time) down the M columns of the tile:
// pass 0 reads through gl, the last pass writes through gs, the others work
// in place.  GL_TILE: gl reads the tile; GS_TILE: gs writes it.  Each pass
// ends with a barrier unless it is the last.
template <int M, int EPT, bool GL_TILE, bool GS_TILE, class GL, class GS, class Hook>
__device__ __forceinline__ void plane_columns(int n, int nt, const Cx<R> *tw, PlaneTile<M> tile,
                                              GL &&gl, GS &&gs, Hook &&loaded)
{
    int n8, n4, n2, n3;
    plane_radices(n, n8, n4, n2, n3);
    const int passes = n8 + n4 + n2 + n3;
    auto loc = [&](int u, int &b, int &j) {
        b = u % M;
        j = u / M;
    };
    auto tl = [&](int b, int i) -> Cx<R> { return tile.at(i, b); };
    auto ts = [&](int b, int i, Cx<R> v) { tile.at(i, b) = v; };
    int ns = 1, p = 0;
    auto kof = [&](int j) { return j & (ns - 1); };  // ns is a power of two
    auto run = [&](auto radc) {
        constexpr int RAD = decltype(radc)::value;
        const int nj = n / RAD, nbf = M * nj, tws = n / (ns * RAD);
        const bool first = p == 0, last = p == passes - 1;
        if (first && last)
            plane_pass<EPT, RAD, true>(nbf, nt, tw, tws, nj, ns, loc, kof, gl, gs, loaded);
        else if (first)
            plane_pass<EPT, RAD, GL_TILE>(nbf, nt, tw, tws, nj, ns, loc, kof, gl, ts, loaded);
        else if (last)
            plane_pass<EPT, RAD, GS_TILE>(nbf, nt, tw, tws, nj, ns, loc, kof, tl, gs, Nothing{});
        else
            plane_pass<EPT, RAD, true>(nbf, nt, tw, tws, nj, ns, loc, kof, tl, ts, Nothing{});
        if (!last) __syncthreads();
        ns *= RAD;
        ++p;
    };
    for (int i = 0; i < n8; ++i) run(std::integral_constant<int, 8>{});
    for (int i = 0; i < n4; ++i) run(std::integral_constant<int, 4>{});
    for (int i = 0; i < n2; ++i) run(std::integral_constant<int, 2>{});
    for (int i = 0; i < n3; ++i) run(std::integral_constant<int, 3>{});
}

// The tables of both transforms, x entries then y entries.  A pass 0 needs
// neither, so the first entries of each thread go to registers, ahead of the
// field's loads, and to LDS while those are in flight (loaded and stored
// first, the tables' latency came before the field's).
template <int M> struct PlaneTables {
    const Cx<R> *x, *y;
    int n, nt;
    Cx<R> v[2];
    __device__ __forceinline__ Cx<R> entry(int i) const { return i < 2 * M ? x[i] : y[i - 2 * M]; }
    __device__ __forceinline__ void fetch()
    {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int i = threadIdx.x + k * nt;
            v[k] = entry(i < n ? i : 0);
        }
    }
    __device__ __forceinline__ void store(Cx<R> *lds) const
    {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int i = threadIdx.x + k * nt;
            if (i < n) lds[i] = v[k];
        }
        for (int i = threadIdx.x + 2 * nt; i < n; i += nt) lds[i] = entry(i);
    }
};

// LDS of a plane of ny rows: the tile (also the scratch of the partial sums)
// and the tables of both transforms
template <int M> constexpr size_t plane_tile_bytes(int ny)
{
    return ((sizeof(Cx<R>) * PlaneTile<M>::PITCH * ny + 511) / 512) * 512;
}
template <int M> constexpr size_t plane_lds_bytes(int ny)
{
    return plane_tile_bytes<M>(ny) + sizeof(Cx<R>) * (2 * M + ny);
}
template <int M> constexpr int plane_threads(int ny)
{
    const int e = 64 * pl_ept(M * ny);
    return (M * ny + e - 1) / e * 64;
}

// Forward: plane vb.x of problem vb.y.
template <int M, int EPT> struct PFBody {
    static __device__ __forceinline__ void run(const PlaneFwd &p0, VBlock vb, int nt, char *lds)
    {
        XFwdArgs a = p0.x;
        if (gated_off(a.batch, a.gate, vb.y)) return;
        if (a.batch) {
            const ProbPtrs &q = a.batch[vb.y];
            a.f = q.f;
            a.S = q.S;
            if (a.partials) a.partials = q.partials;
        }
        constexpr int NX = 2 * M;
        const int ny = a.ny, k = vb.x;
        PlaneTile<M> tile{(Cx<R> *)lds};
        Cx<R> *s_twx = (Cx<R> *)(lds + plane_tile_bytes<M>(ny));
        Cx<R> *s_twy = s_twx + NX;
        PlaneTables<M> tab{(const Cx<R> *)a.tw, (const Cx<R> *)p0.twy, NX + ny, nt, {}};
        tab.fetch();
        auto tables = [&]() { tab.store(s_twx); };

        const PK_GLOBAL double *gf = gbl(a.f) + (size_t)k * ny * NX;
        PK_GLOBAL Cx<R> *S = gbl((Cx<R> *)a.S) + (size_t)k * ny * M;
        double acc0 = 0.0;
        constexpr RPlan pl = make_rplan(M);
        static_assert(pl.count >= 2, "two passes or more along x");
        auto tl = [&](int b, int n) -> Cx<R> { return tile.at(b, n); };
        auto ts = [&](int b, int n, Cx<R> v) { tile.at(b, n) = v; };
        // ---- x: all passes but the last in the tile
        {
            constexpr int RAD = pl.r[0], NJ = M / RAD;
            auto loc = [&](int u, int &b, int &j) {
                b = u / NJ;
                j = u % NJ;
            };
            auto gl = [&](int b, int n) -> Cx<R> {
                const double2 fv = ld_stream(gf + (size_t)b * NX + 2 * n);
                acc0 += fv.x + fv.y;
                return {R(fv.x), R(fv.y)};
            };
            auto k0 = [](int) { return 0; };
            plane_pass<EPT, RAD, false>(ny * NJ, nt, s_twx, 0, NJ, 1, loc, k0, gl, ts, tables);
            __syncthreads();
        }
        auto mid = [&](auto pc) {
            constexpr int P = decltype(pc)::value;
            constexpr int RAD = pl.r[P], NJ = M / RAD, NS = rplan_ns(pl, P);
            auto loc = [&](int u, int &b, int &j) {
                b = u / NJ;
                j = u % NJ;
            };
            auto kof = [](int j) { return j % NS; };
            plane_pass<EPT, RAD, true>(ny * NJ, nt, s_twx, 2 * (M / (NS * RAD)), NJ, NS, loc, kof, tl, ts, Nothing{});
            __syncthreads();
        };
        static_assert(pl.count <= 4, "");
        if constexpr (pl.count > 2) mid(std::integral_constant<int, 1>{});
        if constexpr (pl.count > 3) mid(std::integral_constant<int, 2>{});
        // ---- x: last pass with the real-to-complex split, back into the tile
        {
            constexpr int RAD = pl.r[pl.count - 1], NJ = M / RAD, U = NJ / 2;
            static_assert(NJ == rplan_ns(pl, pl.count - 1) && NJ % 2 == 0, "pairing needs even NJ");
            constexpr int PER = (EPT + 2 * RAD - 1) / (2 * RAD);
            const int nu = ny * U;
            Cx<R> v1[PER][RAD], v2[PER][RAD];
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int u = threadIdx.x + q * nt;
                if (u < nu) {
                    const int b = u / U, pp = u % U;
                    int j1, j2;
                    pair_of<NJ>(pp, j1, j2);
#pragma unroll
                    for (int r = 0; r < RAD; ++r) {
                        v1[q][r] = tile.at(b, j1 + r * NJ);
                        v2[q][r] = tile.at(b, j2 + r * NJ);
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int u = threadIdx.x + q * nt;
                if (u < nu) {
                    const int b = u / U, pp = u % U;
                    int j1, j2;
                    pair_of<NJ>(pp, j1, j2);
#pragma unroll
                    for (int r = 1; r < RAD; ++r) {
                        v1[q][r] = cmul(v1[q][r], s_twx[2 * r * j1]);
                        v2[q][r] = cmul(v2[q][r], s_twx[2 * r * j2]);
                    }
                    Bfly<R, RAD>::run(v1[q]);
                    Bfly<R, RAD>::run(v2[q]);
                    auto emit = [&](int m, Cx<R> zm, Cx<R> zc) {
                        Cx<R> xm, xc;
                        split_pair(zm, zc, s_twx[m], xm, xc);
                        tile.at(b, m) = xm;
                        if (2 * m != M) tile.at(b, M - m) = xc;
                    };
                    if (pp == 0) {
                        tile.at(b, 0) = {v1[q][0].re + v1[q][0].im, v1[q][0].re - v1[q][0].im};
#pragma unroll
                        for (int r = 1; r < RAD; ++r)
                            if (r <= RAD - r) emit(r * NJ, v1[q][r], v1[q][RAD - r]);
#pragma unroll
                        for (int r = 0; r < RAD; ++r)
                            if (r <= RAD - 1 - r) emit(NJ / 2 + r * NJ, v2[q][r], v2[q][RAD - 1 - r]);
                    } else {
#pragma unroll
                        for (int r = 0; r < RAD; ++r) emit(j1 + r * NJ, v1[q][r], v2[q][RAD - 1 - r]);
                    }
                }
            }
            __syncthreads();
        }
        // ---- y: down the columns, the last pass to HBM
        auto cl = [&](int b, int i) -> Cx<R> { return tile.at(i, b); };
        auto gs = [&](int b, int i, Cx<R> v) { put(S + i * M + b, v); };
        plane_columns<M, EPT, true, false>(ny, nt, s_twy, tile, cl, gs, Nothing{});

        if (a.partials) {
            double z1 = 0.0, z2 = 0.0;
            if (a.hz) acc0 *= a.hz[k];
            __syncthreads();
            block_sum3(acc0, z1, z2, (double *)lds, nt);
            if (threadIdx.x == 0) {
                a.partials[4 * k] = acc0;
                a.partials[4 * k + 1] = 0.0;
                a.partials[4 * k + 2] = 0.0;
            }
        }
    }
};

// Inverse: plane vb.x of problem vb.y, stored to p (or to the FP32 first
// iterate, P32) or, ACC, added to the previous iterate with its mean removed
// (as XIBody in k_xpass.hip).
template <int M, int EPT, bool ACC, bool P32> struct PIBody {
    static __device__ __forceinline__ void run(const PlaneInv &p0, VBlock vb, int nt, char *lds)
    {
        const XInvArgs &a0 = p0.x;
        bool widen_only = false;
        if constexpr (P32 && ACC) {
            if (a0.batch && a0.gate) {
                const int *c = a0.batch[vb.y].ctrl;
                if (c[C_CORRECT] == 0) {
                    if (c[C_COPY] == 0) return;
                    widen_only = true;
                }
            }
        } else {
            if (gated_off(a0.batch, a0.gate, vb.y)) return;
        }
        XInvArgs a = a0;
        if (a.batch) {
            const ProbPtrs &q = a.batch[vb.y];
            a.S = q.S;
            a.p = q.p;
            a.p32 = q.p32;
            if (ACC && a.sum_p) a.sum_p = q.scal + 4;
        }
        constexpr int NX = 2 * M;
        const int ny = a.ny, k = vb.x;
        PK_GLOBAL double *gp = gbl(a.p) + (size_t)k * ny * NX;
        PK_GLOBAL float *gp32 = P32 ? gbl(a.p32) + (size_t)k * ny * NX : nullptr;
        if (widen_only) {  // uniform over the workgroup
            for (int e = threadIdx.x; e < ny * M; e += nt)
                st_stream(gp + 2 * (size_t)e, ld_stream(gp32 + 2 * (size_t)e));
            return;
        }
        const double pmean = (ACC && a.sum_p && !a.regular) ? (*a.sum_p) * a.inv_n : 0.0;
        PlaneTile<M> tile{(Cx<R> *)lds};
        Cx<R> *s_twx = (Cx<R> *)(lds + plane_tile_bytes<M>(ny));
        Cx<R> *s_twy = s_twx + NX;
        PlaneTables<M> tab{(const Cx<R> *)a.tw, (const Cx<R> *)p0.twy, NX + ny, nt, {}};
        tab.fetch();
        auto tables = [&]() { tab.store(s_twx); };
        const PK_GLOBAL Cx<R> *S = gbl((const Cx<R> *)a.S) + (size_t)k * ny * M;
        // ---- y: conj(FFT(conj)) down the columns, into the tile
        auto gl = [&](int b, int i) -> Cx<R> {
            const PK_GLOBAL Cx<R> &v = S[i * M + b];
            return {v.re, -v.im};
        };
        auto cs = [&](int b, int i, Cx<R> v) { tile.at(i, b) = cconj(v); };
        plane_columns<M, EPT, false, true>(ny, nt, s_twy, tile, gl, cs, tables);
        __syncthreads();

        // the FP32 first iterate, in the coalesced order of the final loop, in
        // flight during the x passes (an FP64 iterate, from the second
        // correction on, would spill: it is read in the loop)
        constexpr bool PRE = ACC && P32;
        pk_f2v pre[PRE ? EPT : 1];
        if constexpr (PRE) {
#pragma unroll
            for (int q = 0; q < EPT; ++q) {
                const int e = threadIdx.x + q * nt;
                pre[q] = pk_f2v{0, 0};
                if (e < ny * M)
                    pre[q] = __builtin_nontemporal_load((const PK_GLOBAL pk_f2v *)(gp32 + 2 * (size_t)e));
            }
        }
        constexpr RPlan pl = get_rplan(M, 1);
        // ---- x: first pass with the merge fused
        {
            constexpr int RAD = pl.r[0], NJ = M / RAD, U = NJ / 2;
            static_assert(pl.count >= 2 && NJ % 2 == 0, "pairing needs even NJ");
            constexpr int PER = (EPT + 2 * RAD - 1) / (2 * RAD);
            const int nu = ny * U;
            Cx<R> v1[PER][RAD], v2[PER][RAD];
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int u = threadIdx.x + q * nt;
                if (u < nu) {
                    const int b = u / U, pp = u % U;
                    int j1, j2;
                    pair_of<NJ>(pp, j1, j2);
#pragma unroll
                    for (int r = 0; r < RAD; ++r) {
                        v1[q][r] = tile.at(b, j1 + r * NJ);
                        v2[q][r] = tile.at(b, j2 + r * NJ);
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int u = threadIdx.x + q * nt;
                if (u < nu) {
                    const int b = u / U, pp = u % U;
                    int j1, j2;
                    pair_of<NJ>(pp, j1, j2);
                    Cx<R> *z1 = v1[q], *z2 = v2[q];  // merged in place
                    if (pp == 0) {
                        z1[0] = {z1[0].re + z1[0].im, -(z1[0].re - z1[0].im)};
#pragma unroll
                        for (int r = 1; r < RAD; ++r)
                            if (r <= RAD - r)
                                merge_pair(z1[r], z1[RAD - r], s_twx[r * NJ], z1[r], z1[RAD - r]);
#pragma unroll
                        for (int r = 0; r < RAD; ++r)
                            if (r <= RAD - 1 - r)
                                merge_pair(z2[r], z2[RAD - 1 - r], s_twx[NJ / 2 + r * NJ], z2[r],
                                           z2[RAD - 1 - r]);
                    } else {
#pragma unroll
                        for (int r = 0; r < RAD; ++r)
                            merge_pair(z1[r], z2[RAD - 1 - r], s_twx[j1 + r * NJ], z1[r],
                                       z2[RAD - 1 - r]);
                    }
                    Bfly<R, RAD>::run(z1);
                    Bfly<R, RAD>::run(z2);
#pragma unroll
                    for (int r = 0; r < RAD; ++r) {
                        tile.at(b, j1 * RAD + r) = z1[r];
                        tile.at(b, j2 * RAD + r) = z2[r];
                    }
                }
            }
            __syncthreads();
        }
        auto tl = [&](int b, int n) -> Cx<R> { return tile.at(b, n); };
        auto ts = [&](int b, int n, Cx<R> v) { tile.at(b, n) = v; };
        auto gs = [&](int b, int n, Cx<R> v) {
            const size_t di = (size_t)b * NX + 2 * n;
            const double2 o = {double(v.re), -double(v.im)};
            if constexpr (P32)
                st_stream(gp32 + di, o);
            else
                st_stream(gp + di, o);
        };
        auto step = [&](auto pc, auto &&st, bool sync_after) {
            constexpr int P = decltype(pc)::value;
            constexpr int RAD = pl.r[P], NJ = M / RAD, NS = rplan_ns(pl, P);
            auto loc = [&](int u, int &b, int &j) {
                b = u / NJ;
                j = u % NJ;
            };
            auto kof = [](int j) { return j % NS; };
            plane_pass<EPT, RAD, true>(ny * NJ, nt, s_twx, 2 * (M / (NS * RAD)), NJ, NS, loc, kof, tl, st, Nothing{});
            if (sync_after) __syncthreads();
        };
        constexpr int LAST = pl.count - 1;
        static_assert(pl.count <= 4, "");
        if constexpr (LAST > 1) step(std::integral_constant<int, 1>{}, ts, true);
        if constexpr (LAST > 2) step(std::integral_constant<int, 2>{}, ts, true);
        if constexpr (ACC) {
            step(std::integral_constant<int, LAST>{}, ts, true);
#pragma unroll
            for (int q = 0; q < EPT; ++q) {
                const int e = threadIdx.x + q * nt;
                if (e < ny * M) {
                    const Cx<R> v = tile.at(e / M, e % M);
                    double2 old;
                    if constexpr (PRE)
                        old = double2{double(pre[q].x), double(pre[q].y)};
                    else
                        old = ld_stream(gp + 2 * (size_t)e);
                    const double2 o = {double(v.re) + (old.x - pmean), -double(v.im) + (old.y - pmean)};
                    st_stream(gp + 2 * (size_t)e, o);
                }
            }
        } else {
            step(std::integral_constant<int, LAST>{}, gs, false);
        }
    }
};

template <int M, int EPT> __global__ __launch_bounds__(PL_MAXT) void k_plane_fwd(PlaneFwd a)
{
    extern __shared__ __align__(16) char s_dyn[];
    PFBody<M, EPT>::run(a, VBlock{(int)blockIdx.x, (int)blockIdx.y, (int)gridDim.x}, (int)blockDim.x,
                   s_dyn);
}

template <int M, int EPT, bool ACC, bool P32>
__global__ __launch_bounds__(PL_MAXT) void k_plane_inv(PlaneInv a)
{
    extern __shared__ __align__(16) char s_dyn[];
    PIBody<M, EPT, ACC, P32>::run(a, VBlock{(int)blockIdx.x, (int)blockIdx.y, (int)gridDim.x},
                             (int)blockDim.x, s_dyn);
}

template <int M> static bool fits(int ny)
{
    return M * ny <= PL_ELEMS && plane_lds_bytes<M>(ny) <= (size_t)160 * 1024;
}

template <int M, int EPT> static int run_fwd(const PlaneFwd &a, hipStream_t s)
{
    const XFwdArgs &x = a.x;
    hipLaunchKernelGGL((k_plane_fwd<M, EPT>), dim3(x.nz, x.batch ? x.nbatch : 1),
                       dim3(plane_threads<M>(x.ny)), plane_lds_bytes<M>(x.ny), s, a);
    return (int)hipGetLastError();
}

template <int M, int EPT> static int run_inv(const PlaneInv &a, hipStream_t s)
{
    const XInvArgs &x = a.x;
    const dim3 grid(x.nz, x.batch ? x.nbatch : 1), nt(plane_threads<M>(x.ny));
    const size_t lds = plane_lds_bytes<M>(x.ny);
    if constexpr (sizeof(R) == 4) {
        if (x.accumulate && x.p_in32)
            hipLaunchKernelGGL((k_plane_inv<M, EPT, true, true>), grid, nt, lds, s, a);
        else if (x.accumulate)
            hipLaunchKernelGGL((k_plane_inv<M, EPT, true, false>), grid, nt, lds, s, a);
        else if (x.p_in32)
            hipLaunchKernelGGL((k_plane_inv<M, EPT, false, true>), grid, nt, lds, s, a);
        else
            hipLaunchKernelGGL((k_plane_inv<M, EPT, false, false>), grid, nt, lds, s, a);
    } else {
        if (x.accumulate || x.p_in32) return -1;  // the refinement transforms in FP32
        hipLaunchKernelGGL((k_plane_inv<M, EPT, false, false>), grid, nt, lds, s, a);
    }
    return (int)hipGetLastError();
}

// f(values per thread) for planes of ny rows
template <int M, class F> static int by_size(int ny, F &&f)
{
    if (ny < 2 || !fits<M>(ny)) return -1;
    if constexpr (sizeof(R) == 4)
        if (pl_ept(M * ny) == 16) return f(std::integral_constant<int, 16>{});
    return f(std::integral_constant<int, 8>{});
}

// ---------------------------------------------------------------------------
// Work lists: the planes of problems of different shapes in one launch.
// Class: the half row length M (inverse: 4 M + 2 accumulate + FP32 iterate);
// planes that take 16 values per thread get launches of their own.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(PL_MAXT) void k_plane_fwd_list(ListArgs<PlaneFwd>)
{
    extern __shared__ __align__(16) char s_dyn[];
    const PK_KARG ListArgs<PlaneFwd> *L = list_args<PlaneFwd>();
    int g;
    VBlock vb;
    if (!list_find(L, g, vb)) return;
    const PlaneFwd arg = L->a[g];
    const int nt = L->nt[g];
    switch (L->cls[g]) {
#define PK_PF_CASE(N) case N: PFBody<N, 8>::run(arg, vb, nt, s_dyn); break;
        PK_PLANE_LENGTHS(PK_PF_CASE)
#undef PK_PF_CASE
    default: break;
    }
}

__global__ __launch_bounds__(PL_MAXT) void k_plane_inv_list(ListArgs<PlaneInv>)
{
    extern __shared__ __align__(16) char s_dyn[];
    const PK_KARG ListArgs<PlaneInv> *L = list_args<PlaneInv>();
    int g;
    VBlock vb;
    if (!list_find(L, g, vb)) return;
    const PlaneInv arg = L->a[g];
    const int nt = L->nt[g];
    switch (L->cls[g]) {
#define PK_PI_CASE(N)                                                                        \
    case 4 * N: PIBody<N, 8, false, false>::run(arg, vb, nt, s_dyn); break;                     \
    case 4 * N + 1:                                                                          \
        if constexpr (sizeof(R) == 4) PIBody<N, 8, false, true>::run(arg, vb, nt, s_dyn);       \
        break;                                                                               \
    case 4 * N + 2:                                                                          \
        if constexpr (sizeof(R) == 4) PIBody<N, 8, true, false>::run(arg, vb, nt, s_dyn);       \
        break;                                                                               \
    case 4 * N + 3:                                                                          \
        if constexpr (sizeof(R) == 4) PIBody<N, 8, true, true>::run(arg, vb, nt, s_dyn);        \
        break;
        PK_PLANE_LENGTHS(PK_PI_CASE)
#undef PK_PI_CASE
    default: break;
    }
}

// threads and LDS of a plane (false: it has no class or does not fit)
static bool plane_shape(int nx, int ny, int &nt, size_t &lds)
{
    if (ny < 2) return false;
    switch (nx / 2) {
#define PK_PL_INFO(N)                    \
    case N:                              \
        if (!fits<N>(ny)) return false;  \
        nt = plane_threads<N>(ny);       \
        lds = plane_lds_bytes<N>(ny);    \
        return true;
        PK_PLANE_LENGTHS(PK_PL_INFO)
#undef PK_PL_INFO
    default: return false;
    }
}

template <class A, class Cls, class Launch, class Own>
static int run_planes(const A *a, int n, Cls cls_of, Launch launch, Own own)
{
    std::vector<PlaneSeg> segs;
    std::vector<int> of;  // record of a segment
    for (int i = 0; i < n; ++i) {
        const auto &x = a[i].x;
        int t = 0;
        size_t b = 0;
        if (!plane_shape(x.nx, x.ny, t, b)) return -1;
        if (pl_ept(x.nx / 2 * x.ny) != 8) {
            const int e = own(a[i]);
            if (e) return e;
            continue;
        }
        segs.push_back(PlaneSeg{b, t, (long)x.nz * (x.batch ? x.nbatch : 1)});
        of.push_back(i);
    }
    for (const std::vector<int> &one : plane_launches(segs, LIST_MAX_SEG)) {
        // one shape alone: its own kernel, compiled for one length (FP32
        // inverse: 72 VGPRs against the list's 109)
        int e = 0;
        if (one.size() == 1) {
            e = own(a[of[one[0]]]);
        } else {
            ListArgs<A> L{};
            size_t lds = 0;
            int total = 0, nt = 0;
            for (int k : one) {
                const A &r = a[of[k]];
                const int g = L.nseg++;
                L.start[g] = total;
                L.gx[g] = r.x.nz;
                L.cls[g] = cls_of(r.x);
                L.nt[g] = segs[k].threads;
                L.a[g] = r;
                total += (int)segs[k].planes;
                lds = std::max(lds, segs[k].lds);
                nt = std::max(nt, segs[k].threads);
            }
            L.start[L.nseg] = total;
            launch(L, total, nt, lds);
            e = (int)hipGetLastError();
        }
        if (e) return e;
    }
    return 0;
}

}  // namespace PK_NS
using namespace PK_NS;

// A launch lasts as long as one workgroup takes for its plane, however few
// planes there are, and for the largest planes that is longer than both
// separate passes, which spread a plane over many workgroups.  Solves, us,
// separate passes -> planes, by the planes in flight:
//   FP32, 16 values per thread: 256x128 1 32 -> 41, 32 44 -> 48, 64 52 -> 54,
//     96 70 -> 59; 192x96 1 1.07x, 48 1.00x, 64 0.96x; 64x384 48 1.09x, 96 0.95x
//   FP64, more than 6144 values: 256x64 4 25 -> 28, 24 1.03x, 48 0.95x;
//     128x128 12 29 -> 31, 48 0.98x
//   FP64, 6144 values: 0.92x to 1.09x below 24 planes, 0.77x to 0.85x from 96;
//   smaller planes: 0.63x to 1.00x at every count (FP32 to 0.92x).
// 32x512 in FP64 is level from one plane on and has no line.  Where the routes
// round differently (plane_rounds_apart) the planes of one problem count, else
// those of all problems of the shape.
bool PK_SUFFIX(plane_pays)(int nx, int ny, int nz, long n)
{
    int nt = 0;
    size_t lds = 0;
    if (!plane_shape(nx, ny, nt, lds)) return false;
    constexpr int prec = sizeof(R) == 4 ? P_F32 : P_F64;
    const int values = nx / 2 * ny;
    const long planes = plane_rounds_apart(prec, nx, ny) ? nz : nz * n;
    if (prec == P_F32) return planes >= (pl_ept(values) == 16 ? 64 : 1);
    return planes >= (values > 6144 && nx != 32 ? 48 : 1);
}

#define PK_CASE_PF(N) \
    case N: return by_size<N>(a.x.ny, [&](auto e) { return run_fwd<N, decltype(e)::value>(a, s); });
#define PK_CASE_PI(N) \
    case N: return by_size<N>(a.x.ny, [&](auto e) { return run_inv<N, decltype(e)::value>(a, s); });

int PK_SUFFIX(launch_plane_fwd)(const PlaneFwd &a, hipStream_t s)
{
    switch (a.x.nx / 2) { PK_PLANE_LENGTHS(PK_CASE_PF) default: return -1; }
}

int PK_SUFFIX(launch_plane_inv)(const PlaneInv &a, hipStream_t s)
{
    switch (a.x.nx / 2) { PK_PLANE_LENGTHS(PK_CASE_PI) default: return -1; }
}

int PK_SUFFIX(launch_plane_fwd_list)(const PlaneFwd *a, int n, hipStream_t s)
{
    return run_planes(
        a, n, [](const XFwdArgs &x) { return x.nx / 2; },
        [&](const ListArgs<PlaneFwd> &L, int total, int nt, size_t lds) {
            hipLaunchKernelGGL(k_plane_fwd_list, dim3(total), dim3(nt), lds, s, L);
        },
        [&](const PlaneFwd &r) { return PK_SUFFIX(launch_plane_fwd)(r, s); });
}

int PK_SUFFIX(launch_plane_inv_list)(const PlaneInv *a, int n, hipStream_t s)
{
    return run_planes(
        a, n,
        [](const XInvArgs &x) { return 2 * x.nx + 2 * (x.accumulate ? 1 : 0) + (x.p_in32 ? 1 : 0); },
        [&](const ListArgs<PlaneInv> &L, int total, int nt, size_t lds) {
            hipLaunchKernelGGL(k_plane_inv_list, dim3(total), dim3(nt), lds, s, L);
        },
        [&](const PlaneInv &r) { return PK_SUFFIX(launch_plane_inv)(r, s); });
}

}  // namespace pk
