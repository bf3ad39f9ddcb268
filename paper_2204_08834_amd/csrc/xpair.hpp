// xpair.hpp -- the real-to-complex split and the complex-to-real merge of a row
// (formulas in k_xpass.hip), on the butterfly pairs in which their operands
// meet.  Included inside namespace pk::PK_NS of a precision-templated source.
#pragma once

// The split of the M-point spectrum (forward) and its merge (inverse) couple
// the values at m and M - m.  In the last Stockham pass (forward) and the
// first one (inverse) the butterfly j handles indices j + r NJ, r < RAD,
// NJ = M/RAD, and the partner of j + r NJ is (NJ - j) + (RAD-1-r) NJ for
// j > 0, while butterflies 0 and NJ/2 are their own partners (r <-> RAD-r and
// r <-> RAD-1-r).  A thread therefore takes the butterfly pair (p, NJ - p)
// for p in [1, NJ/2), or (0, NJ/2) for p = 0, and both values of every
// coupled pair meet in its registers: no extra LDS round trip in the forward
// pass, and every spectrum element is read once in the inverse pass.
template <int NJ>
__device__ __forceinline__ void pair_of(int p, int &j1, int &j2)
{
    j1 = p;
    j2 = (p == 0) ? NJ / 2 : NJ - p;
}

// forward split of one coupled pair: zm = Z[m], zc = Z[M-m], w = exp(-2 pi i m/nx)
//   X[m] = A + w B,  X[M-m] = conj(A - w B),
//   A = (zm + conj zc)/2,  B = -i (zm - conj zc)/2
template <typename T>
__device__ __forceinline__ void split_pair(Cx<T> zm, Cx<T> zc, Cx<T> w, Cx<T> &xm, Cx<T> &xc)
{
    const Cx<T> A = cscale(cadd(zm, cconj(zc)), T(0.5));
    const Cx<T> B = cscale(cmul_mi(csub(zm, cconj(zc))), T(0.5));
    const Cx<T> wB = cmul(w, B);
    xm = cadd(A, wB);
    xc = cconj(csub(A, wB));
}

// inverse merge of one coupled pair: xm = X[m], xc = X[M-m], w = exp(-2 pi i m/nx)
//   Z'[m] = A + T,  Z'[M-m] = conj(A - T),
//   A = xm + conj xc,  T = i conj(w) (xm - conj xc);
// returned conjugated (the inverse runs as conj(FFT(conj))).
template <typename T>
__device__ __forceinline__ void merge_pair(Cx<T> xm, Cx<T> xc, Cx<T> w, Cx<T> &zm, Cx<T> &zc)
{
    const Cx<T> A = cadd(xm, cconj(xc));
    const Cx<T> Tt = cmul_pi(cmul(cconj(w), csub(xm, cconj(xc))));
    zm = cconj(cadd(A, Tt));
    zc = csub(A, Tt);
}
