// K3 for the lengths with compile-time plans: forward z transforms, tensor multiply and inverse z
// transforms of whole (kx, ky) columns, all three components of a column in the same lanes.
//
// A line of length L has T lanes, one per butterfly of its last (widest) pass, and a wave takes
// CPW = 64 / T columns.  The three component lines of a column run through the same lanes one
// after another, so
//   * a lane ends the forward passes with the three components at its own frequencies in registers
//     and multiplies by the tensor without an exchange,
//   * the twiddles of a pass are formed once for three butterflies,
//   * a line never leaves its wave: no block barrier after the tensor columns are staged, and one
//     LDS line per column serves all components (a wave's LDS accesses complete in order, so the
//     next component is written while the last one's reads are still on their way).
// The bound is neither memory nor one unit: at L = 512 (two vectors, fp64, 14.5 GB) the vector unit
// is busy 55 % of the time (2045 instructions per wave and column, 1732 of them fp64 arithmetic), LDS
// 48 %, and memory runs at 3.9 TB/s of the 5.1 TB/s a copy reaches; the registers hold two waves per
// SIMD (three where noted below).  Measured per pass against one component per wave with the block
// exchanging components through LDS (the kernel k_zmul, which the lengths planned at run time
// keep), two vectors in fp64, spheres of L / 2 cells, m = 1.3:
//   L      32   48   64   72   96  120  128  160  192  200  256   320   384   512
//   was    16   16   21   39   54   94   92  206  336  396  649  1292  2040  4439 us
//   is     10   13   15   24   36   64   63  141  209  276  457   998  1588  3718 us
// In fp32 (one vector) 64: 12 -> 11, 192: 105 -> 61, 320: 432 -> 284, 512: 1154 -> 875 us.
#pragma once

#include "fft.hpp"

namespace dda {

// Plans of a line and its place in a wave: T lanes, at least one per butterfly of the widest pass.
// The inverse plan is the forward plan reversed, so that the multiply sits between two passes of
// the same radix RL and butterfly indices.
template <int L> struct ZCol {
    static constexpr bool SORTED = zmul_multi(make_plan(L, 8, 0));
    static constexpr FftPlan F = make_plan(L, 8, SORTED ? 2 : 0), I = make_plan(L, 8, SORTED ? 3 : 1);
    static constexpr int NP = F.npass, RL = F.radix[NP - 1];
    static constexpr int CPW = 64 / F.tpl, T = 64 / CPW;
    static constexpr int S = lds_line_stride(L);
    static constexpr int HZ1 = L / 2 + 1;
    static constexpr bool TW8 = all_radix8(L, 8);
    static constexpr int NTW = TW8 ? L / 8 : L;
    static constexpr int NB(int R) { return (L / R + T - 1) / T; }  // butterflies per lane in a pass
};
// most elements of one line that a lane holds in any pass
constexpr int zcol_maxe(const FftPlan &p, int T) {
    int m = 0;
    for (int i = 0; i < p.npass; ++i) {
        const int e = (p.L / p.radix[i] + T - 1) / T * p.radix[i];
        m = m > e ? m : e;
    }
    return m;
}

// Complex products with their fused multiply-adds spelled out, so that their roundings do not change with
// how the compiler arranges the kernel around them (the additions of the butterflies are left to it; one
// instantiation serves every batch, so a vector's product does not depend on the others).  The imaginary
// part rounds a.x b.y (cmul1) or a.y b.x (cmul2) first; either would do, but an iterate of a slowly
// converging solve depends on the choice, which therefore stays.
template <typename R> __device__ __forceinline__ R fmar(R a, R b, R c) {
    if constexpr (sizeof(R) == 8) return __builtin_fma(a, b, c);
    else return __builtin_fmaf(a, b, c);
}
template <typename C> __device__ __forceinline__ C cmul1(C a, C b) {
    return mk<C>(fmar(a.x, b.x, -(a.y * b.y)), fmar(a.y, b.x, a.x * b.y));
}
template <typename C> __device__ __forceinline__ C cmul2(C a, C b) {
    return mk<C>(fmar(a.x, b.x, -(a.y * b.y)), fmar(a.x, b.y, a.y * b.x));
}
template <typename C> __device__ __forceinline__ C csqr(C a) {
    const auto t = a.x * a.y;
    return mk<C>(fmar(a.x, a.x, -(a.y * a.y)), t + t);
}
// whether twiddle r of a radix-R pass is a product of table entries
constexpr bool tw_derived(bool tw8, int R, int r) { return R == 8 && (tw8 ? r > 1 : r == 3 || r > 4); }

// w[r] = exp(-DIR 2 pi i r k step / L), r = 1..R-1
template <int DIR, int R, bool TW8, typename C>
__device__ __forceinline__ void zcol_tw(C *w, int k, int step, const C *tw) {
    if constexpr (R == 8) {
        C w1, w2, w4;
        if constexpr (TW8) {
            w1 = tw[k * step];
            w2 = csqr(w1);
            w4 = csqr(w2);
        } else {
            w1 = tw[k * step];
            w2 = tw[2 * k * step];
            w4 = tw[4 * k * step];
        }
        w[1] = w1;
        w[2] = w2;
        w[3] = TW8 ? cmul2(w1, w2) : cmul1(w1, w2);
        w[4] = w4;
        w[5] = TW8 ? cmul2(w1, w4) : cmul1(w1, w4);
        w[6] = TW8 ? cmul2(w2, w4) : cmul1(w2, w4);
        w[7] = cmul2(w[3], w4);
    } else {
#pragma unroll
        for (int r = 1; r < R; ++r) w[r] = tw[r * k * step];
    }
    if (DIR > 0) {
#pragma unroll
        for (int r = 1; r < R; ++r) w[r] = cconj(w[r]);
    }
}

// waves per SIMD that the registers are budgeted for: a third wave in fp64 where the kernel fits 168
// registers with at most a few spilled (two vectors, 2 against 3 waves: 192 215 -> 208 us, 320 and 384 even;
// but 160 141 -> 183 us, 512 3.72 -> 4.51 ms)
template <typename R> constexpr int zcol_waves_per_simd(int L) {
    return sizeof(R) == 4 ? 4 : L == 192 || L == 320 || L == 384 ? 3 : 2;
}
// lengths whose budget holds only if the tensor loads of one frequency are not hoisted over the
// products of the one before (192: 229 -> 208 us per two-vector fp64 pass, 384 1612 -> 1597, 320 even; fp32
// within 2 % either way)
template <typename R> constexpr bool zcol_fence(int L) {
    return sizeof(R) == 4 ? L > 128 : zcol_waves_per_simd<R>(L) == 3;
}

// lengths that load the first columns before the tensor is staged: there a block has one round and the
// pass is a chain of latencies (32: 10.5 -> 10.0 us; 48 and 64: no change)
constexpr bool zcol_ahead(int L) { return L <= 32; }

template <typename R, int LC>
__global__ void __launch_bounds__(256, zcol_waves_per_simd<R>(LC))
    k_zcol(cplx<R> *__restrict__ B2, const cplx<R> *__restrict__ Gh, int nz, int Lx, int Ly, int nrhs, int opb,
           const cplx<R> *__restrict__ twz, const int *__restrict__ done) {
    using C = cplx<R>;
    using Z = ZCol<LC>;
    constexpr int T = Z::T, CPW = Z::CPW, NP = Z::NP, HZ1 = Z::HZ1;
    constexpr int ME = zcol_maxe(Z::F, T);
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C *gsh = reinterpret_cast<C *>(smem_raw);
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63, W = blockDim.x >> 6;
    const int hx1 = Lx / 2 + 1, noct = hx1 * (Ly / 2 + 1);
    const int per_xcd = gridDim.x >> 3;
    const int blk = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    const int oct0 = blk * opb;
    if (oct0 >= noct) return;
    const int nocc = min(opb, noct - oct0);
    C *lines = gsh + opb * 6 * HZ1;
    C *tw = lines + W * CPW * Z::S;
    const int slot = lane / T, j0 = lane % T;
    C *ln = lines + (wave * CPW + slot) * Z::S;
    const int nzp = row_pitch(nz);
    const size_t cstride = (size_t)Ly * nzp;
    const int items = nocc * nrhs * 4;
    struct Item {
        C *col;
        int mir, o, rhs;
        bool ok;
    };
    auto item_at = [&](int it) {
        Item m;
        const int q = it >> 2, rhs = q % nrhs;
        m.mir = it & 3;
        m.o = q / nrhs < nocc ? q / nrhs : 0;
        const int oct = oct0 + m.o, kxo = oct % hx1, kyo = oct / hx1;
        const bool mxs = m.mir & 1, mys = m.mir & 2;
        m.ok = slot < CPW && it < items && (!mxs || (kxo != 0 && 2 * kxo != Lx)) &&
               (!mys || (kyo != 0 && 2 * kyo != Ly));
        m.rhs = rhs < nrhs ? rhs : 0;
        const int kx = m.ok && mxs ? Lx - kxo : kxo, ky = m.ok && mys ? Ly - kyo : kyo;
        m.col = B2 + (((size_t)kx * (3 * nrhs) + rhs * 3) * Ly + ky) * nzp;
        return m;
    };
    C v[3][ME];
    // first pass inputs: the lower half of the line from memory, the rest is padding
    auto load_column = [&](const Item &m, int j) {
        constexpr int R0 = Z::F.radix[0], NB = Z::NB(R0), nb = LC / R0;
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int r = 0; r < R0; ++r) {
                    if (2 * r >= R0 && R0 > 1) continue;
                    const int i = ((b + 1) * T <= nb ? j + b * T : min(j + b * T, nb - 1)) + r * nb;
                    v[c][b * R0 + r] = m.ok && i < nz ? ld_stream(&m.col[c * cstride + i]) : czero<C>();
                }
    };
    // short lines: the first columns are on their way while the block stages the tensor (they do not
    // wait for done either)
    Item m = item_at(wave * CPW + slot);
    if constexpr (zcol_ahead(LC)) load_column(m, j0);
    {   // the tensor columns and the twiddles of the block.  fp32 keeps eight loads of a thread in
        // flight (L = 256: 118 -> 114 us, 512: 1010 -> 891 us); fp64, with half the waves, is 0-2 %
        // faster loading one by one
        const C *gcol = Gh + (size_t)oct0 * 6 * HZ1;
        const int ng = nocc * 6 * HZ1;
        constexpr int U = sizeof(R) == 4 ? 8 : 1;
        for (int e0 = t; e0 < ng; e0 += U * blockDim.x) {
            C q[U];
#pragma unroll
            for (int u = 0; u < U; ++u) q[u] = gcol[min(e0 + u * (int)blockDim.x, ng - 1)];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (e0 + u * (int)blockDim.x < ng) gsh[e0 + u * blockDim.x] = q[u];
        }
        for (int e = t; e < Z::NTW; e += blockDim.x) tw[e] = twz[e];
    }
    __syncthreads();
    if (slot >= CPW) return;
    for (int it0 = wave * CPW; it0 < items; it0 += W * CPW) {
        const bool ahead = zcol_ahead(LC) && it0 == wave * CPW;
        if (!ahead) m = item_at(it0 + slot);
        m.ok = m.ok && !(done && done[m.rhs]);
        if (!__any(m.ok)) continue;
        // opaque from round to round: the LDS addresses are formed inside each round instead of being
        // held in registers across rounds
        int j = j0;
        __asm__ volatile("" : "+v"(j));
        // butterfly b of a pass with nb of them; lanes past the last one repeat it (same values to
        // the same places), so that no pass needs a branch
        auto bidx = [&](int b, int nb) { return (b + 1) * T <= nb ? j + b * T : min(j + b * T, nb - 1); };
        const R sg[3] = {m.mir & 1 ? (R)-1 : (R)1, m.mir & 2 ? (R)-1 : (R)1, (R)1};
        const C *g = gsh + m.o * 6 * HZ1;
        const bool ok = m.ok;
        C *col = m.col;
        if (!ahead) load_column(m, j);
        // forward passes
        static_for<0, NP>([&](auto pc) {
            constexpr int p = decltype(pc)::value, Rp = Z::F.radix[p], Ns = Z::F.ns[p], NB = Z::NB(Rp), nb = LC / Rp;
            C w[NB][Rp];
            if constexpr (Ns > 1) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const int jb = bidx(b, nb);
                    zcol_tw<-1, Rp, Z::TW8>(w[b], jb % Ns, nb / Ns, tw);
                }
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    C *a = v[c] + b * Rp;
                    if constexpr (p == 0) {
#pragma unroll
                        for (int r = 0; r < Rp; ++r) a[r] = (2 * r >= Rp && Rp > 1) ? czero<C>() : cscale(a[r], sg[c]);
                    }
                    if constexpr (Ns > 1) {
#pragma unroll
                        for (int r = 1; r < Rp; ++r) a[r] = tw_derived(Z::TW8, Rp, r) ? cmul2(a[r], w[b][r]) : cmul1(a[r], w[b][r]);
                    }
                    dftR<-1, Rp>(a);
                }
                if constexpr (p + 1 < NP) {
                    lds_sync<true>();
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        bfly_store<Rp>(v[c] + b * Rp, bidx(b, nb), Ns, [&](int i, C x) { ln[pidx(i)] = x; });
                    lds_sync<true>();
                    constexpr int Rn = Z::F.radix[p + 1], NBn = Z::NB(Rn), nbn = LC / Rn;
#pragma unroll
                    for (int b = 0; b < NBn; ++b) {
                        const int jb = bidx(b, nbn);
#pragma unroll
                        for (int r = 0; r < Rn; ++r) v[c][b * Rn + r] = ln[pidx(jb + r * nbn)];
                    }
                }
            }
        });
        // Ghat X at the frequencies that this lane's last forward pass left in its registers
        {
            constexpr int RL = Z::RL, NB = Z::NB(RL), nb = LC / RL;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int jb = bidx(b, nb);
#pragma unroll
                for (int r = 0; r < RL; ++r) {
                    const int kz = jb + r * nb, e = b * RL + r;
                    // the octant holds kz <= L/2; xz and yz are odd along z
                    bool lo;
                    if constexpr (RL % 2 == 0) lo = 2 * r < RL || (2 * r == RL && jb == 0);
                    else lo = 2 * kz <= LC;
                    const C *gp = g + (RL % 2 == 0 ? (2 * r < RL ? kz : LC - kz) : (lo ? kz : LC - kz));
                    const C xx = gp[0], xy = gp[HZ1], yy = gp[3 * HZ1], zz = gp[5 * HZ1];
                    const R sz = lo ? (R)1 : (R)-1;
                    const C xz = cscale(gp[2 * HZ1], sz), yz = cscale(gp[4 * HZ1], sz);
                    const C X = v[0][e], Y = v[1][e], W3 = v[2][e];
                    v[0][e] = cadd(cadd(cmul1(xx, X), cmul1(xy, Y)), cmul1(xz, W3));
                    v[1][e] = cadd(cadd(cmul1(xy, X), cmul1(yy, Y)), cmul1(yz, W3));
                    v[2][e] = cadd(cadd(cmul1(xz, X), cmul1(yz, Y)), cmul1(zz, W3));
                    if (zcol_fence<R>(LC)) __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        // inverse passes
        static_for<0, NP>([&](auto pc) {
            constexpr int p = decltype(pc)::value, Rp = Z::I.radix[p], Ns = Z::I.ns[p], NB = Z::NB(Rp), nb = LC / Rp;
            C w[NB][Rp];
            if constexpr (Ns > 1) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const int jb = bidx(b, nb);
                    zcol_tw<+1, Rp, Z::TW8>(w[b], jb % Ns, nb / Ns, tw);
                }
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    C *a = v[c] + b * Rp;
                    if constexpr (Ns > 1) {
#pragma unroll
                        for (int r = 1; r < Rp; ++r) a[r] = cmul1(a[r], w[b][r]);
                    }
                    dftR<+1, Rp>(a);
                }
                if constexpr (p + 1 < NP) {
                    lds_sync<true>();
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        bfly_store<Rp>(v[c] + b * Rp, bidx(b, nb), Ns, [&](int i, C x) { ln[pidx(i)] = x; });
                    lds_sync<true>();
                    constexpr int Rn = Z::I.radix[p + 1], NBn = Z::NB(Rn), nbn = LC / Rn;
#pragma unroll
                    for (int b = 0; b < NBn; ++b) {
                        const int jb = bidx(b, nbn);
#pragma unroll
                        for (int r = 0; r < Rn; ++r) v[c][b * Rn + r] = ln[pidx(jb + r * nbn)];
                    }
                } else {
#pragma unroll
                    for (int b = 0; b < NB; ++b)
#pragma unroll
                        for (int r = 0; r < Rp; ++r) {
                            if (2 * r >= Rp && Rp > 1) continue;
                            const int i = j + b * T + r * nb;
                            if (ok && i < nz && ((b + 1) * T <= nb || j + b * T < nb))
                                st_stream(&col[c * cstride + i], cscale(v[c][b * Rp + r], sg[c]));
                        }
                }
            }
        });
    }
}

// dynamic LDS bytes of a block of W waves over opb octant columns
template <typename R, int LC> constexpr size_t zcol_lds(int opb, int W) {
    using Z = ZCol<LC>;
    return ((size_t)opb * 6 * Z::HZ1 + (size_t)W * Z::CPW * Z::S + Z::NTW) * sizeof(cplx<R>);
}

}  // namespace dda
