// The Sturm sequence of a symmetric tridiagonal, free of HIP so that the
// device, the host and a host-compiled test use the same recurrence.
#pragma once

namespace wc {

// Whether the k x k tridiagonal with diagonal a and off-diagonal b has an
// eigenvalue below x (or at it): a pivot d_i = (a_i - x) - b_{i-1}^2 / d_{i-1} of
// T - x I that is not positive.  The first one settles it: what follows a zero
// or an infinite pivot is not looked at.  Eight entries are read ahead of their
// divisions, which are a chain.
template <class P>
constexpr bool eigenvalue_below(P a, P b, int k, double x) {
    bool below = false;
    double d = 1.0;
    for (int i0 = 0; i0 < k; i0 += 8) {
        double p[8] = {}, bb[8] = {};
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u < k ? i0 + u : k - 1;
            p[u] = a[i] - x;
            bb[u] = i > 0 ? b[i - 1] * b[i - 1] : 0.0;
        }
        for (int u = 0; u < 8; ++u) {
            d = p[u] - bb[u] / d;
            below = below || (i0 + u < k && d <= 0.0);
        }
        if (below) break;
    }
    return below;
}

}  // namespace wc
