// What the kernels that take several steps per launch on tiles share (lbm_tile.hip,
// lbm_adjoint.hip).
#pragma once

#include "lbm_kernels.h"

namespace lbm {

// The launch constants as a kernel of several steps uses them: read again by scalar loads in
// every step.  Kept across the loop they, and the products the compiler forms of them ahead
// of it, take vector registers.
using KConst = const __attribute__((address_space(4))) KParams *;

__device__ __forceinline__ KConst fresh(KConst p)
{
    asm volatile("" : "+s"(p));
    return p;
}

template <typename T, typename U>
__device__ __forceinline__ void copy_consts(T *d, const __attribute__((address_space(4))) U *q)
{
    static_assert(sizeof(T) % sizeof(U) == 0, "a struct of U only");
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / sizeof(U)); ++i) reinterpret_cast<U *>(d)[i] = q[i];
}
__device__ __forceinline__ void load_consts(KConst p, Cst<float> &k)
{
    copy_consts(&k, (const __attribute__((address_space(4))) float *)&p->cf);
}
__device__ __forceinline__ void load_consts(KConst p, Cst<double> &k)
{
    copy_consts(&k, (const __attribute__((address_space(4))) double *)&p->cd);
}
__device__ __forceinline__ void load_eps(KConst p, EpsC<float> &e)
{
    e.epsd = p->eps; e.c0 = p->c0; e.c1 = p->c1;
    e.eps = p->ef.eps; e.ieps = p->ef.ieps; e.dlin = p->ef.dlin; e.dquad = p->ef.dquad; e.bM = p->ef.bM;
}
__device__ __forceinline__ void load_eps(KConst p, EpsC<double> &e)
{
    e.epsd = p->eps; e.c0 = p->c0; e.c1 = p->c1;
    e.eps = p->ed.eps; e.ieps = p->ed.ieps; e.dlin = p->ed.dlin; e.dquad = p->ed.dquad; e.bM = p->ed.bM;
}

// Tiles of at most tw x th nodes (of equal size to within one node).
inline TileGrid tile_grid(const KParams &P, int tw, int th)
{
    TileGrid g;
    g.nbx = (P.nx + tw - 1) / tw;
    g.nby = (P.ny + th - 1) / th;
    g.tw = P.nx / g.nbx; g.rx = P.nx % g.nbx;
    g.th = P.ny / g.nby; g.ry = P.ny % g.nby;
    g.magic = g.nbx > 1 ? (unsigned)(0x100000000ull / g.nbx + 1) : 0;
    return g;
}

// Row of tiles that tile b belongs to (b / nbx).  magic exceeds 2^32 / nbx by at most 1, so the
// product is b / nbx plus less than 1/2: its whole part is the row or, in the last tiles of rows
// of more than 65,000 tiles, the next one.
__host__ __device__ __forceinline__ int tile_row(const TileGrid &g, int b)
{
    if (g.nbx == 1) return b;
    const unsigned q = (unsigned)(((unsigned long long)(unsigned)b * g.magic) >> 32);
    return (int)(q * (unsigned)g.nbx > (unsigned)b ? q - 1 : q);
}

}  // namespace lbm
