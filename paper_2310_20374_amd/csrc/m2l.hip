// Interaction tensors (Eq. 25) for every well-separated pair found by the walk.
//
// Target-major: one wave per target cell A, lanes over A's sources B (in the order the
// walk listed them, fixed by the tree), each lane accumulating
//   C^(m)_a(s_A) += sum_{n=0, n!=1}^{p-m} (-1)^n sum_{|b|=n} D_{a+b}(R) Mt_b(B),
// with R = s_A - s_B, D_g = d^g (1/|R|) and Mt_b = M_b / b! (the n! of Eq. 25 and
// the multinomial weights of the symmetric inner product cancel into 1/b!).  The
// wave then sums its 64 partial tensors by exchanges between lanes.  Both directions of a
// pair are separate entries of the list, so every target's sum has a fixed order and the
// result does not depend on scheduling.  D and the contraction are in expansion.h.
//
// Bound by FP64 (FP32) operations at the two to four waves per SIMD that D leaves room
// for, and by the lines of the sources' rows: a lane reads its own source's row, so a row
// is loaded at once, while its lines are in L1 (4e6 clumped moonlets, FP32, p = 6: 865 us
// with loads where they are used, 820 so).  The two highest orders take part with the
// monopole alone (there is no n = 1 term): where their sums don't fit the registers, D of
// a batch of 64 sources, times the masses, is summed over the lanes as it stands.  FP64
// at p = 6 computed D three times before, once per group of orders, and every sum over
// the wave read 64 rows of LDS: N = 1e6, s = 52: 381 -> 222 us; 1e5: 86 -> 57 us; p = 3,
// 262144: 99 -> 94 us; FP32, p = 4, 64 disks of 12324: 43 -> 38 us; p = 6, 1e6: 101 us
// both ways (92 with the highest orders summed per batch there too, but clumps 885).
#include "ncorp_internal.h"
#include "expansion.h"

namespace ncorp {

constexpr int kM2LBlock = 64;     // one wave per block, one target per wave

// Waves per SIMD that the registers are cut for.
template <int P, typename T> constexpr int m2l_waves() {
    return sizeof(T) == 8 ? (P >= 5 ? 2 : (P == 4 ? 3 : 4)) : (P >= 6 ? 2 : 4);
}

// Orders whose sums a lane keeps over a long list: all of them, but without the last two
// in FP64 from p = 5 on.
template <int P, typename T> constexpr int m2l_orders() {
    return sizeof(T) == 8 && P >= 5 ? P - 2 : P;
}

// ---------------------------------------------------------------- sums over the wave
// v[0..N) of every lane, summed over the wave: in each step a lane pairs with the lane
// across one bit of the lane index, the lower one keeps the sums of the first half of the
// values and the upper one those of the second, so 64 lanes share the N results after six
// steps and some 2 N additions.
constexpr int halved(int n) { return (n + 1) / 2; }
constexpr int folded(int n) {
    return halved(halved(halved(halved(halved(halved(n))))));
}
__device__ __forceinline__ double join(unsigned lo, unsigned hi) {
    return __hiloint2double((int)hi, (int)lo);
}
template <int N, int BIT> __device__ __forceinline__ void fold_step(double *v) {
    constexpr int H = halved(N);
    const bool upper = (threadIdx.x & BIT) != 0;
#pragma unroll
    for (int k = 0; k < H; k++) {
        const double a = v[k], b = k + H < N ? v[k + H] : 0.0;
        const unsigned al = (unsigned)__double2loint(a), ah = (unsigned)__double2hiint(a);
        const unsigned bl = (unsigned)__double2loint(b), bh = (unsigned)__double2hiint(b);
        if constexpr (BIT == 32) {
            const auto l = __builtin_amdgcn_permlane32_swap(al, bl, false, false);
            const auto h = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
            v[k] = join(l[0], h[0]) + join(l[1], h[1]);
        } else if constexpr (BIT == 16) {
            const auto l = __builtin_amdgcn_permlane16_swap(al, bl, false, false);
            const auto h = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
            v[k] = join(l[0], h[0]) + join(l[1], h[1]);
        } else {
            // rotation by 8 in rows of 16, mirror in rows of 8, quad permutations
            constexpr int ctl = BIT == 8 ? 0x128 : (BIT == 4 ? 0x141 : (BIT == 2 ? 0x4e : 0xb1));
            const double keep = upper ? b : a, send = upper ? a : b;
            const unsigned l = (unsigned)__builtin_amdgcn_mov_dpp(__double2loint(send), ctl, 0xf,
                                                                  0xf, true);
            const unsigned h = (unsigned)__builtin_amdgcn_mov_dpp(__double2hiint(send), ctl, 0xf,
                                                                  0xf, true);
            v[k] = keep + join(l, h);
        }
    }
}
template <int N> __device__ __forceinline__ void fold(double *v) {
    constexpr int N2 = halved(N), N3 = halved(N2), N4 = halved(N3), N5 = halved(N4),
                  N6 = halved(N5);
    fold_step<N, 32>(v);
    fold_step<N2, 16>(v);
    fold_step<N3, 8>(v);
    fold_step<N4, 4>(v);
    fold_step<N5, 2>(v);
    fold_step<N6, 1>(v);
}
// which of the N values the lane's k-th result is the sum of, or -1 (a lane left over)
template <int N> __device__ __forceinline__ int fold_index(int k) {
    constexpr int N2 = halved(N), N3 = halved(N2), N4 = halved(N3), N5 = halved(N4),
                  N6 = halved(N5), N7 = halved(N6);
    const int l = threadIdx.x;
    int i = k + ((l & 1) ? N7 : 0);
    bool ok = i < N6;
    i += (l & 2) ? N6 : 0;
    ok = ok && i < N5;
    i += (l & 4) ? N5 : 0;
    ok = ok && i < N4;
    i += (l & 8) ? N4 : 0;
    ok = ok && i < N3;
    i += (l & 16) ? N3 : 0;
    ok = ok && i < N2;
    i += (l & 32) ? N2 : 0;
    return ok && i < N ? i : -1;
}

template <int P, typename T>
__global__ void __launch_bounds__(kM2LBlock, (m2l_waves<P, T>()))
k_m2l(const DevState *__restrict__ st, const double4 *__restrict__ gcell,
      const T *__restrict__ mult, const int32_t *__restrict__ cnt,
      const int32_t *__restrict__ seg, int stride, double *__restrict__ local) {
    constexpr int NL = n_local(P), NM = n_mult(P), ND = off_order(P + 1);
    // orders 1 .. M1 have sums in registers; M2 .. P, where they don't fit, are summed over
    // the lanes after every batch
    constexpr int M1 = m2l_orders<P, T>(), M2 = M1 + 1;
    constexpr int BL = cidx(1, 0, 0), BH = cidx(M2, 0, 0);
    constexpr int NLO = BH - BL, NHI = NL - BH;
    if (st->status & kSkipMask) return;
    const int nc = st->ncells;
    const int lane = threadIdx.x;
    for (int A = blockIdx.x; A < nc; A += gridDim.x) {
        const int len = cnt[A];
        double *out = local + (int64_t)A * NL;
        if (len == 0) {
            for (int k = lane; k < NL; k += kWave) out[k] = 0.0;
            continue;
        }
        const int32_t *srcs = seg + (int64_t)A * stride;
        const double4 gA = gcell[A];
        T acc[NLO];
#pragma unroll
        for (int k = 0; k < NLO; k++) acc[k] = (T)0;
        double sum[folded(NHI) + 1];
#pragma unroll
        for (int k = 0; k < folded(NHI); k++) sum[k] = 0.0;
        for (int i0 = 0; i0 < len; i0 += kWave) {
            double hi[NHI + 1];
#pragma unroll
            for (int k = 0; k < NHI; k++) hi[k] = 0.0;
            if (i0 + lane < len) {
                const int B = srcs[i0 + lane];
                const double4 gB = gcell[B];
                const T *mb = mult + (int64_t)B * NM;
                const T x = (T)(gA.x - gB.x), y = (T)(gA.y - gB.y), z = (T)(gA.z - gB.z);
                const T r2 = x * x + y * y + z * z;
                T D[ND], M[NM];
                // FP32: the whole row at once, while its lines are in L1
#pragma unroll
                for (int k = 0; k < NM; k++) M[k] = mb[k];
                if constexpr (sizeof(T) == 4) {
#pragma unroll
                    for (int k = 0; k < NM; k++) asm volatile("" : "+v"(M[k]));
                }
                green_derivs<P, T>(x, y, z, rsqrt_t<T>(r2), D);
                m2l_contract<P, 1, M1, T>(D, M, acc);
                const T m0 = M[0];
#pragma unroll
                for (int m = M2; m <= P; m++)
#pragma unroll
                    for (int b = 0; b <= m; b++)
#pragma unroll
                        for (int c = 0; c <= m - b; c++)
                            hi[cidx(m - b - c, b, c) - BH] = (double)(D[sidx(m - b - c, b, c)] * m0);
            }
            if constexpr (NHI > 0) fold<NHI>(hi);
#pragma unroll
            for (int k = 0; k < folded(NHI); k++) sum[k] += hi[k];
        }
#pragma unroll
        for (int k = 0; k < folded(NHI); k++) {
            const int at = fold_index<(NHI > 0 ? NHI : 1)>(k);
            if (at >= 0) out[BH + at] = sum[k];
        }
        double lo[NLO];
#pragma unroll
        for (int k = 0; k < NLO; k++) lo[k] = (double)acc[k];
        fold<NLO>(lo);
#pragma unroll
        for (int k = 0; k < folded(NLO); k++) {
            const int at = fold_index<NLO>(k);
            if (at >= 0) out[BL + at] = lo[k];
        }
    }
}

template <int P, typename T>
static void launch_m2l_t(const Workspace &ws, const T *mult, hipStream_t s) {
    int g = (int)(ws.cell_cap < 16384 ? ws.cell_cap : 16384);
    if (g < 1) g = 1;
    k_m2l<P, T><<<g, kM2LBlock, 0, s>>>(ws.st, ws.gcell, mult, ws.m2l_cnt, ws.m2l_seg,
                                        ws.m2l_stride, ws.local);
}

template <int P>
static void launch_m2l_p(const Workspace &ws, int precision, hipStream_t s) {
    if (precision == NCORP_FP32_BULK) launch_m2l_t<P, float>(ws, ws.mult32, s);
    else launch_m2l_t<P, double>(ws, ws.mult, s);
}

hipError_t launch_m2l(const Workspace &ws, int p, int precision, hipStream_t s) {
    switch (p) {
        case 1: launch_m2l_p<1>(ws, precision, s); break;
        case 2: launch_m2l_p<2>(ws, precision, s); break;
        case 3: launch_m2l_p<3>(ws, precision, s); break;
        case 4: launch_m2l_p<4>(ws, precision, s); break;
        case 5: launch_m2l_p<5>(ws, precision, s); break;
        case 6: launch_m2l_p<6>(ws, precision, s); break;
        default: break;
    }
    return hipGetLastError();
}

}  // namespace ncorp
