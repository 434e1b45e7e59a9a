// Radix plans of the streamed transforms and the layout of their twiddle
// tables, shared by the kernels and by the plan that fills the tables.
#pragma once

namespace mf {

// Transform lengths: 2^a 3^b with a >= 1 (even sides).
constexpr bool is_pow2(int L) { return L > 0 && (L & (L - 1)) == 0; }

// Radix plan: radix-16 passes while 16 divides what is left, then one
// radix-8/4/2 pass for the rest of the power of two, then radix-3 passes.
constexpr int radix_of(int rem) {
    return rem % 16 == 0 ? 16 : rem % 8 == 0 ? 8 : rem % 4 == 0 ? 4 : rem % 2 == 0 ? 2 : 3;
}
template <int REM>
constexpr int next_radix() { return radix_of(REM); }
// Transform plan of the fused streamed kernels: a radix-16 pass at one end,
// a radix-RL pass at the other, radix-RM passes between them.  L = 256 uses
// 16 x 4 x 4, so that its RL pass has enough butterflies for every lane and
// holds few values per thread; longer transforms use radix 16 and the
// remainder (2048 = 16 x 16 x 8).
constexpr int last_radix_of(int L) {
    if (L == 256) return 4;
    int r = L;
    while (r > 16) r /= 16;
    return r;
}
constexpr int middle_radix_of(int L) { return L == 256 ? 4 : 16; }

// Twiddles of the streamed transforms, one table per pass: a radix-R pass
// after NS points multiplies input r of butterfly j by W_{R NS}^{r k},
// k = j mod NS, and finds it at [(r - 1) NS + k].  Neighbouring lanes then
// read neighbouring entries.  Read as tw[r k L / (R NS)] from one table
// W_L^r, the 64 lanes of a load touch up to 4 r cache lines (or collide in
// r's LDS banks), and this, not the arithmetic or HBM, bounded the streamed
// kernels.  The values are the same.
struct PassPlan {
    int n, R[24], NS[24], off[24];  // passes with NS > 1 by rising NS, and each table's place (128-byte lines)
    int size;
};
constexpr PassPlan pass_plan(int L) {
    PassPlan p{};
    const auto add = [&p](int R, int NS) {
        if (NS == 1) return;
        int at = p.n;
        for (int i = p.n - 1; i >= 0; --i) {
            if (p.R[i] == R && p.NS[i] == NS) return;
            if (p.NS[i] > NS) at = i;
        }
        for (int i = p.n++; i > at; --i) {
            p.R[i] = p.R[i - 1];
            p.NS[i] = p.NS[i - 1];
        }
        p.R[at] = R;
        p.NS[at] = NS;
    };
    for (int NS = 1; NS < L;) {
        const int R = radix_of(L / NS);
        add(R, NS);
        NS *= R;
    }
    if (is_pow2(L) && L >= 256) {
        const int RL = last_radix_of(L), RM = middle_radix_of(L);
        for (int NS = 16; NS * RL < L; NS *= RM) add(RM, NS);
        add(RL, L / RL);
        for (int NS = RL; NS * 16 < L; NS *= RM) add(RM, NS);
        add(16, L / 16);
    }
    for (int i = 0; i < p.n; ++i) {
        p.off[i] = p.size;
        p.size += ((p.R[i] - 1) * p.NS[i] + 15) / 16 * 16;
    }
    return p;
}
constexpr int pass_tw(int L, int R, int NS) {
    const PassPlan p = pass_plan(L);
    for (int i = 0; i < p.n; ++i)
        if (p.R[i] == R && p.NS[i] == NS) return p.off[i];
    return -1;
}
// Entries of the tables with NS <= lim, the first of all.
constexpr int pass_prefix(int L, int lim) {
    const PassPlan p = pass_plan(L);
    for (int i = 0; i < p.n; ++i)
        if (p.NS[i] > lim) return p.off[i];
    return p.size;
}

}  // namespace mf
