// One element of the weight pre-segregation (Section 3.2), for the kernels that do it.
#pragma once
#include "kst_internal.h"

namespace kst {

struct SegGeom {
    int Cin, Cout, n;
    int group;             // channels side by side: 1 (fp32) or 8 (16 bits)
    unsigned off[5];       // element offset of class p; off[4] = total
    int Tb[4];             // columns of sub-kernel p
    int T[4];              // taps of sub-kernel p
};

inline SegGeom seg_geom(int Cin, int Cout, int n, kst_dtype dt)
{
    SegGeom g;
    g.Cin = Cin;
    g.Cout = Cout;
    g.n = n;
    g.group = is16(dt) ? 8 : 1;
    for (int p = 0; p < 4; ++p) {
        g.off[p] = (unsigned)seg_offset(Cin, Cout, n, p, dt);
        g.Tb[p] = taps_for_parity(n, p & 1);
        g.T[p] = class_taps(n, p);
    }
    g.off[4] = (unsigned)seg_elems(Cin, Cout, n, dt);
    return g;
}

// Element e of the segregated buffer (past the last: nothing).
template <typename T>
__device__ __forceinline__ void segregate_one(const T *__restrict__ w, T *__restrict__ w_seg, const SegGeom &g, unsigned e)
{
    if (e >= g.off[4]) return;
    int p = 0;
    while (p < 3 && e >= g.off[p + 1]) ++p;
    const int Tp = g.T[p];
    if (Tp == 0) return;   // empty class (n = 1): occupies no elements, unreachable
    unsigned ep = e - g.off[p];
    const int c_lo = (int)(ep % (unsigned)g.group);
    ep /= (unsigned)g.group;
    const int co = (int)(ep % (unsigned)g.Cout);
    ep /= (unsigned)g.Cout;
    const int t = (int)(ep % (unsigned)Tp);
    const int c_hi = (int)(ep / (unsigned)Tp);
    const int ci = c_hi * g.group + c_lo;
    const int a = t / g.Tb[p], b = t % g.Tb[p];
    const int u = 2 * a + (p >> 1), v = 2 * b + (p & 1);
    T val = T(0);
    if (ci < g.Cin) val = w[(((size_t)co * g.Cin + ci) * g.n + u) * g.n + v];
    w_seg[e] = val;
}

}  // namespace kst
