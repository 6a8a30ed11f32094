// Transforms in registers.
//
// A row (column) of N points belongs to G = N/E lanes, and lane l holds the E
// elements congruent to l modulo G: in the x-pass lanes of one wavefront, 64/G
// rows per wavefront side by side; in the column passes lanes of one workgroup,
// whose consecutive threads hold consecutive columns.  That set is the same before the first butterfly stage and after the last
// one, of the inverse as of the forward transform, so a row's fields pass from
// the inverse transforms through the pointwise source into the forward
// transforms without leaving their registers; LDS only carries the exchange
// between two stages, and no workgroup barrier is needed.
#pragma once
#include "fft.hpp"

namespace flusi {

// Radix plans: E values per lane, every radix divides E.
// Row plans (PLAN 0): 3 fields of E values per lane fit the registers also in
// FP64; few values per lane (4, 6) on small grids, which then have more
// wavefronts to spread over the chip (64^3 FP32 insect x-pass: 14.8 us with 8,
// 13.6 with 4; 48^3: 17.4 with 12, 14.8 with 6).  0: no plan (1152 points, whose
// 32 lanes would hold 36 values per field).
// Column plans (PLAN 1): one field per thread, so as few exchanges as the
// radices allow.  (The z-pass, which keeps three fields of kept modes, takes row
// plans but for 512 points in FP32.)
__host__ __device__ constexpr int xr_E(int N, int PLAN = 0) {
    if (PLAN == 1) {
        switch (N) {
            case 16: return 4;
            case 24: return 6;
            case 32: case 64: return 8;
            case 48: case 192: return 12;
            case 128: case 256: case 512: return 16;
            case 96: case 384: case 768: return 24;
            default: return 0;
        }
    }
    switch (N) {
        case 16: case 32: case 64: return 4;
        case 24: case 48: return 6;
        case 128: case 256: case 512: return 8;
        case 96: case 192: case 384: return 12;
        default: return 0;
    }
}
__host__ __device__ constexpr int xr_radix(int N, int s, int PLAN = 0) {
    if (PLAN == 1) {
        switch (N) {
            case 16: return s < 2 ? 4 : 1;
            case 24: return s < 2 ? 2 : (s == 2 ? 6 : 1);
            case 32: return s == 0 ? 8 : (s == 1 ? 4 : 1);
            case 48: return s == 0 ? 4 : (s == 1 ? 12 : 1);
            case 64: return s < 2 ? 8 : 1;
            case 96: return s == 0 ? 8 : (s == 1 ? 12 : 1);
            case 128: return s == 0 ? 8 : (s == 1 ? 16 : 1);
            case 192: return s < 2 ? 4 : (s == 2 ? 12 : 1);
            case 256: return s < 2 ? 16 : 1;
            case 384: return s < 2 ? 8 : (s == 2 ? 6 : 1);
            case 512: return s == 0 ? 16 : (s == 1 ? 8 : (s == 2 ? 4 : 1));
            case 768: return s < 2 ? 8 : (s == 2 ? 12 : 1);
            default: return 1;
        }
    }
    switch (N) {
        case 16: return s < 2 ? 4 : 1;
        case 24: return s < 2 ? 2 : (s == 2 ? 6 : 1);
        case 32: return s < 2 ? 4 : (s == 2 ? 2 : 1);
        case 48: return s < 3 ? 2 : (s == 3 ? 6 : 1);
        case 64: return s < 3 ? 4 : 1;
        case 96: return s == 0 ? 4 : (s == 1 ? 2 : (s == 2 ? 12 : 1));
        case 128: return s == 0 ? 8 : (s < 3 ? 4 : 1);
        case 192: return s < 2 ? 4 : (s == 2 ? 12 : 1);
        case 256: return s < 2 ? 8 : (s == 2 ? 4 : 1);
        case 384: return s < 2 ? 4 : (s == 2 ? 2 : (s == 3 ? 12 : 1));
        case 512: return s < 3 ? 8 : 1;
        default: return 1;
    }
}
__host__ __device__ constexpr int xr_prefix(int N, int s, int PLAN = 0) {
    int p = 1;
    for (int i = 0; i < s; ++i) p *= xr_radix(N, i, PLAN);
    return p;
}
__host__ __device__ constexpr int xr_stages(int N, int PLAN = 0) {
    int s = 0;
    while (xr_radix(N, s, PLAN) > 1) ++s;
    return s;
}

// The exchange after stage s (butterflies of R inputs, Ns = product of the
// radices before): element n at n + Ns * (n / (Ns R)).  A lane's R outputs then
// lie at one base plus constants, and its E inputs of the next stage as well
// where G and Ns R divide one another (the plans' radix order sees to it), so
// the places cost two address registers; and the writes of consecutive lanes,
// runs of Ns elements Ns R apart, fall on different banks.
__host__ __device__ constexpr bool xr_plan_ok(int N, int PLAN = 0) {
    const int E = xr_E(N, PLAN);
    if (E == 0 || N % E != 0) return false;
    const int G = N / E, S = xr_stages(N, PLAN);
    if (64 % G != 0 || xr_prefix(N, S, PLAN) != N) return false;
    for (int s = 0; s < S; ++s) {
        const int B = xr_prefix(N, s + 1, PLAN);
        if (E % xr_radix(N, s, PLAN) != 0) return false;
        if (s + 1 < S && G % B != 0 && B % G != 0) return false;
    }
    return true;
}
// Elements of a row in its exchange buffer.
__host__ __device__ constexpr int xr_padded(int N, int PLAN = 0) {
    int m = N;
    for (int s = 0; s + 1 < xr_stages(N, PLAN); ++s)
        if (N + N / xr_radix(N, s, PLAN) > m) m = N + N / xr_radix(N, s, PLAN);
    return m;
}
// Stride of the exchange buffers of a wavefront's rows: to a whole turn of the
// banks (32 FP32 complex values) plus G, so that the rows start one after
// another's lanes.
__host__ __device__ constexpr int xr_stride(int N) {
    const int G = N / xr_E(N);
    return (xr_padded(N) + 31) / 32 * 32 + (G < 32 ? G : 0);
}

// Twiddles of the transforms in the order the lanes read them, one run of
// Ns values k for every stage and output r: (r, k) of stage S holds
// exp(-2 pi i k r / (Ns R)).  N - R_0 values, staged in LDS once per workgroup of
// nthreads: read from memory they would be two thirds of the x-pass's vector
// loads, whose issue then bounds it (65536 FP32 rows of 256 points: 181 us with
// them from memory, 123 us from LDS).
template <typename T, int N, int PLAN = 0>
__device__ __forceinline__ void xr_twiddles(cx<T>* tws, const cx<T>* __restrict__ tw, int nthreads) {
    constexpr int R0 = xr_radix(N, 0, PLAN);
    for (int e = threadIdx.x; e < N - R0; e += nthreads) {
        int i = 0;
        static_for<xr_stages(N, PLAN) - 1>([&](auto sc) {
            constexpr int S = decltype(sc)::value + 1;
            constexpr int R = xr_radix(N, S, PLAN), Ns = xr_prefix(N, S, PLAN);
            const int q = e - (Ns - R0);
            if (q >= 0 && q < (R - 1) * Ns) i = (q % Ns) * (q / Ns + 1) * (N / (Ns * R));
        });
        tws[e] = tw[i];
    }
}

// The lane index as a value of its own: what is derived from it (LDS places,
// twiddles) is formed again where it is used, not kept in registers across
// transforms.
template <int G>
__device__ __forceinline__ int xr_lane(int l) {
    __asm__ volatile("" : "+v"(l));
    return l & (G - 1);
}
// Transform of one row or column by its G lanes: v[t] is element l + G t on entry
// and on return (natural order).  col: its exchange buffer, elements CS apart;
// tws: xr_twiddles.  WG: the lanes lie in several wavefronts of the workgroup,
// all of whose threads call this together; else in one.  The buffer is free on
// entry, and every lane has read what it needs of it when its call returns.
template <typename T, int N, int DIR, int PLAN = 0, int CS = 1, bool WG = false>
__device__ __forceinline__ void xr_fft(cx<T> (&v)[xr_E(N, PLAN)], cx<T>* col, int lane, const cx<T>* tws) {
    constexpr int E = xr_E(N, PLAN), G = N / E, NS = xr_stages(N, PLAN);
    static_assert(xr_plan_ok(N, PLAN), "radix plan");
    const int l = xr_lane<G>(lane);
    static_for<NS>([&](auto sc) {
        constexpr int S = decltype(sc)::value;
        constexpr int R = xr_radix(N, S, PLAN), Ns = xr_prefix(N, S, PLAN), J = E / R;
        if constexpr (S > 0) {
            // exchange of the stage before: its blocks are Ns long, padded by Np
            constexpr int Np = xr_prefix(N, S - 1, PLAN);
            const cx<T>* rd = col + CS * (l + (G % Ns == 0 ? Np * (l / Ns) : 0));
            static_for<E>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                v[t] = rd[CS * (G * t + Np * (G * t / Ns))];
            });
            if constexpr (!WG) wave_sync();
            else if constexpr (S + 1 < NS) __syncthreads();
        }
        static_for<J>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            cx<T> a[R];
            static_for<R>([&](auto rc) { a[decltype(rc)::value] = v[j + decltype(rc)::value * J]; });
            if constexpr (Ns > 1) {
                // stage S's twiddles start at Ns - R_0 in the table
                const cx<T>* wt = tws + (Ns - xr_radix(N, 0, PLAN)) + (l + j * G) % Ns;
                static_for<R - 1>([&](auto rc) {
                    constexpr int r = decltype(rc)::value + 1;
                    const cx<T> wv = wt[(r - 1) * Ns];
                    a[r] = (DIR < 0) ? cmul(a[r], wv) : cmulc(a[r], wv);
                });
            }
            Dft<R, DIR, T>::run(a);
            static_for<R>([&](auto rc) { v[j + decltype(rc)::value * J] = a[decltype(rc)::value]; });
        });
        if constexpr (S + 1 < NS) {
            static_for<J>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                const int b = l + j * G;
                cx<T>* wr = col + CS * ((b / Ns) * (Ns * R + Ns) + b % Ns);
                static_for<R>([&](auto rc) {
                    constexpr int r = decltype(rc)::value;
                    wr[CS * r * Ns] = v[j + r * J];
                });
            });
            if constexpr (WG) __syncthreads();
            else wave_sync();
        }
    });
}

// Which of the kept modes (|j| <= K) element l + G t can be, over all lanes:
// 0 none, 1 k = l + G t on every lane, 2 the same on the lanes with k <= K,
// 3 the conjugate mode k = N - l - G t on every lane, 4 the same on the lanes
// with k <= K.
__host__ __device__ constexpr int xr_mode(int N, int K, int t, int PLAN = 0) {
    const int G = N / xr_E(N, PLAN), lo = G * t, hi = G * t + G - 1;
    if (hi <= K) return 1;
    if (lo <= K) return 2;
    if (lo >= N - K) return 3;
    if (hi >= N - K) return 4;
    return 0;
}

// The next t after t that holds a kept mode on some lane (E: none).
__host__ __device__ constexpr int xr_next(int N, int K, int t, int PLAN = 0) {
    for (++t; t < xr_E(N, PLAN) && xr_mode(N, K, t, PLAN) == 0;) ++t;
    return t;
}

}  // namespace flusi
