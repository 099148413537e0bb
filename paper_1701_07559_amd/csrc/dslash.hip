// Wilson hop on every fifth-dimension slice, fused with the fifth-dimension
// operators of the Moebius domain-wall operator (arXiv:1701.07559, Sec. II).
//
// Thread mapping: the L5 slices of one 4D site sit in L5 consecutive lanes of
// one wavefront (64 / L5 sites per wave; the remaining lanes idle).  All lanes
// of a site read the same eight links, so a link is fetched once per site and
// reused across the fifth dimension, and the fifth-dimension couplings (B, C,
// K5 and B K5^-1) become exchanges inside that lane group:
// ds_bpermute for the nearest-slice terms, a recurrence through an LDS tile for
// the inverses (five_lanes).  Spinors are read 16 bytes per lane from the
// structure-of-arrays layout, so a wave's loads of one block are contiguous.
#include "hop_device.h"

namespace mdwf {

// Waves per SIMD the hop kernels are compiled for.  FP16 with staged links: five
// (96 VGPRs, no spills); left free, the scheduler takes 130 registers for
// kernels A / A^+ and they run 20 % slower, at six kernel B of S spills.  The
// other link modes of FP16 are left free: held to five they spill where B is
// applied before the hop (D5 at L5 = 5: 81 us for 53), and of the others kernels
// A, A^+ and B of K5^-1 S take 76 to 78 registers (six waves) by themselves,
// kernel B of S B^-1 96 (five; held to six it spills 64 bytes and S B^-1 takes
// 18 to 30 % longer at L5 = 4 to 7).  FP32 takes what its loads in flight need:
// held to four waves it spills and runs 18 % slower.
template <Prec P, int LM> constexpr int hop_waves_per_eu() { return (P == P16 && LM == 1) ? 5 : 1; }
// FP64 kernels are scheduled for two: at the three that their 146 to 168 registers
// would allow, fewer loads are in flight.  24^3 x 64, L5 = 8, staged links: bare
// hop 564 -> 480 us, S^+ 1146 -> 1072, S B^-1 1144 -> 1069, S 1170 -> 1147;
// 24^3 x 32, L5 = 4, links by every lane: bare hop 190 -> 169, D5 474 -> 380, S B^-1
// 387 -> 361.
template <Prec P> constexpr int hop_waves_at_most() { return P == P64 ? 2 : 8; }
template <int K> constexpr bool hop_five() {
    return HopTraits<K>::epi == 1 || HopTraits<K>::epi == 2 || HopTraits<K>::cen >= 4;
}

template <Prec P, int K, int LM>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(hop_waves_per_eu<P, LM>(), hop_waves_at_most<P>()))) k_hop(const Geo g, const HopDev a) {
    using R = typename Real<P>::T;
    using TR = HopTraits<K>;
    const int L5 = g.L5;
    const int spw = 64 / L5;
    // RHS groups of rg follow each other; within one, every XCD sweeps its own
    // range of tiles, the group's RHS fastest (they share each tile's links in
    // L2, and its neighbour reuse spans rg RHS, not all of them)
    int rhs, tile;
    {
        const int rg = (g.rhs_group[P] > 0 && g.rhs_group[P] < a.nrhs) ? g.rhs_group[P] : a.nrhs;
        const int grp = int(blockIdx.x) / (a.nblk * rg);
        const int base = grp * rg;
        const int gs = min(rg, a.nrhs - base);
        int off = int(blockIdx.x) - grp * a.nblk * rg;
        if (g.xcd_remap[P]) off = xcd_logical_block(off, a.nblk * gs);
        tile = off / gs;
        rhs = base + (off - tile * gs);
    }
    if (a.active && !a.active[rhs]) return;   // uniform over the block
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int sw = lane / L5;
    const int s = lane - sw * L5;
    const int pos = (tile * kWaves + wave) * spw + sw;   // traversal position
    const bool valid = (sw < spw) && (pos < g.Vh4);
    const int gbase = lane - s;
    // traversal position -> tile and place inside it (see Trav) ->
    // coordinates and the parity-compressed index i of the output site
    int xh, y, z, t, i;
    {
        const Trav& tr = g.trav[P];
        const uint32_t p = uint32_t(pos);
        const uint32_t q = tr.fTv.div(p);               // tile number
        const uint32_t r = p - q * uint32_t(tr.b[0] * tr.b[1] * tr.b[2] * tr.b[3]);
        const uint32_t r1 = tr.fBx.div(r), r2 = tr.fBy.div(r1), r3 = tr.fBz.div(r2);   // in-tile
        const uint32_t q1 = tr.fNt.div(q), q2 = tr.fNx.div(q1), q3 = tr.fNy.div(q2);   // tile grid
        const uint32_t nt = tr.fNt.d, nx = tr.fNx.d, ny = tr.fNy.d;
        xh = int(q1 - q2 * nx) * tr.b[0] + int(r - r1 * uint32_t(tr.b[0]));
        y = int(q2 - q3 * ny) * tr.b[1] + int(r1 - r2 * uint32_t(tr.b[1]));
        z = int(q3) * tr.b[2] + int(r2 - r3 * uint32_t(tr.b[2]));
        t = int(q - q1 * nt) * tr.b[3] + int(r3);
        i = xh + g.Xh * (y + g.Y * (z + g.Z * t));
    }
    if constexpr (LM == 3) {   // every lane takes part in the matrix products: idle ones read site 0
        if (!valid) xh = y = z = t = i = 0;
    }

    const RhsCoef& cf = a.coef[rhs];
    const R mq = R(cf.mq), b5 = R(cf.b5), c5 = R(cf.c5);
    Nbr5<R> nb;
    nb.am1 = (gbase + (s == 0 ? L5 - 1 : s - 1)) << 2;
    nb.ap1 = (gbase + (s == L5 - 1 ? 0 : s + 1)) << 2;
    nb.fm1 = (s == 0) ? -mq : R(1);
    nb.fp1 = (s == L5 - 1) ? -mq : R(1);

    const void* in = at_rhs(a.in, a.stride, rhs);
    cx<R> res[12];

    // neighbours of the output site (used only by valid lanes)
    const int x = 2 * xh + ((y + z + t + a.out_parity) & 1);
    const int row = i - xh;
    const int sy = g.Xh, sz = g.Xh * g.Y, st = sz * g.Z;
    const int n_xp = row + ((x + 1 == g.X ? 0 : x + 1) >> 1);
    const int n_xm = row + ((x == 0 ? g.X - 1 : x - 1) >> 1);
    const int n_yp = i + (y == g.Y - 1 ? -(g.Y - 1) * sy : sy);
    const int n_ym = i + (y == 0 ? (g.Y - 1) * sy : -sy);
    const int n_zp = i + (z == g.Z - 1 ? -(g.Z - 1) * sz : sz);
    const int n_zm = i + (z == 0 ? (g.Z - 1) * sz : -sz);
    const int n_tp = i + (t == g.T - 1 ? -(g.T - 1) * st : st);
    const int n_tm = i + (t == 0 ? (g.T - 1) * st : -st);

    // links: segment mu of the output parity at i (forward) and of the input
    // parity at the backward neighbour
    const size_t ls = a.lseg;
    const size_t lblk = size_t(g.Vh4) * 16;
    const size_t sblk = size_t(g.Vh) * 16;
    const char* lo = a.links_out;
    const char* lk = a.links_in;
    const char* src = static_cast<const char*>(in);
    constexpr bool D = TR::dag, PB = TR::preB;
    const uint32_t ui = uint32_t(i);
    const char* seg[8] = {lo, lk, lo + ls, lk + ls, lo + 2 * ls, lk + 2 * ls, lo + 3 * ls, lk + 3 * ls};
    const uint32_t lidx[8] = {ui, uint32_t(n_xm), ui, uint32_t(n_ym), ui, uint32_t(n_zm), ui, uint32_t(n_tm)};
    const uint32_t jn[8] = {uint32_t(n_xp * L5 + s), uint32_t(n_xm * L5 + s), uint32_t(n_yp * L5 + s),
                            uint32_t(n_ym * L5 + s), uint32_t(n_zp * L5 + s), uint32_t(n_zm * L5 + s),
                            uint32_t(n_tp * L5 + s), uint32_t(n_tm * L5 + s)};

    // LDS, per wave: the staged links and, once the hop is done, the tile of
    // five_lanes in the same bytes
    constexpr int kLinkBytes = LM == 1 ? stage_bytes<P>() : 0;
    constexpr bool kFive = hop_five<K>();
    constexpr int kFiveBytes = kFive ? (five_bytes<P, LM != 1>() + 15) / 16 * 16 : 0;
    constexpr int kSmem = kLinkBytes > kFiveBytes ? kLinkBytes : kFiveBytes;
    __shared__ __align__(16) unsigned char smem[kWaves][kSmem > 0 ? kSmem : 16];
    unsigned char* const lw = smem[wave];
    cx<R>* const ftile = reinterpret_cast<cx<R>*>(lw);
    const int a0 = gbase << 2;

    if constexpr (LM == 3) {
        // FP16 on the matrix cores: lane s of the site group holds row s & 3
        // of each link; the neighbour norms are gathered first so that every
        // direction enters one accumulator at a common scale
        const char* rseg[8] = {a.rows_out, a.rows_in, a.rows_out + a.rseg, a.rows_in + a.rseg,
                               a.rows_out + 2 * a.rseg, a.rows_in + 2 * a.rseg, a.rows_out + 3 * a.rseg,
                               a.rows_in + 3 * a.rseg};
        const size_t roff = size_t(s & 3) * lblk;   // this lane's row block
        const char* nsrc = src + align256(3 * sblk);
        float nrm[8];
#pragma unroll
        for (int d = 0; d < 8; ++d) nrm[d] = ldu<float>(nsrc, jn[d] * 4u);
        float S = 1.17549435e-38f;
#pragma unroll
        for (int d = 0; d < 8; ++d) S = fmaxf(S, nrm[d]);
        const float inv = __builtin_amdgcn_rcpf(S);
        f4 acc[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[q] = f4{0.f, 0.f, 0.f, 0.f};
        nu4 sp0[3], sp1[3];
        nu4 lr0, lr1;
        auto load = [&](int d, nu4 sp[3], nu4& lr) {
#pragma unroll
            for (int k = 0; k < 3; ++k) sp[k] = ldu<nu4>(src + k * sblk, jn[d] * 16u);
            lr = ldu<nu4>(rseg[d] + roff, lidx[d] * 16u);
        };
        load(0, sp0, lr0);
#define MDWF_MMA(d, spc, lrc, spn, lrn)                                                  \
    if ((d) < 7) load((d) + 1, spn, lrn);                                                \
    {                                                                                    \
        RowA A;                                                                          \
        A.set(lrc);                                                                      \
        mma_term<(d) / 2, (((d) % 2 == 0) != D) ? 1 : -1>(acc, A, spc, nrm[d] * inv);   \
    }
        MDWF_MMA(0, sp0, lr0, sp1, lr1) MDWF_MMA(1, sp1, lr1, sp0, lr0) MDWF_MMA(2, sp0, lr0, sp1, lr1)
        MDWF_MMA(3, sp1, lr1, sp0, lr0) MDWF_MMA(4, sp0, lr0, sp1, lr1) MDWF_MMA(5, sp1, lr1, sp0, lr0)
        MDWF_MMA(6, sp0, lr0, sp1, lr1) MDWF_MMA(7, sp1, lr1, sp0, lr0)
#undef MDWF_MMA
#pragma unroll
        for (int sp = 0; sp < 4; ++sp)
#pragma unroll
            for (int c = 0; c < 3; ++c) res[sp * 3 + c] = {S * acc[2 * sp][c], S * acc[2 * sp + 1][c]};
    } else if (valid) {
        // LM == 1: this lane's direction of the links
        LinkStage<P> stg;
        if constexpr (LM == 1) {
            const int d = s & 7, mu = d >> 1;
            const uint32_t nm = uint32_t(mu == 0 ? n_xm : mu == 1 ? n_ym : mu == 2 ? n_zm : n_tm);
            if (s < 8) stg.load(((d & 1) ? lk : lo) + mu * ls, lblk, (d & 1) ? nm : ui);
        }
        auto stage = [&]() {
            if constexpr (LM == 1) {
                if (s < 8) stg.put(lw, s, sw);
                wave_sync();
            }
        };
        if constexpr (P == P64) {
            // FP64: one direction in flight (two would exceed the register file)
            Raw<P> r;
            stage();
#define MDWF_DIR(d)                                                                 \
    r.load(seg[d], lidx[d], lblk, src, jn[d], sblk, LM == 0);                      \
    dir_term<P, D, PB, d, LM>(res, r, lw, sw, a0, nb, b5, c5);
            MDWF_DIR(0) MDWF_DIR(1) MDWF_DIR(2) MDWF_DIR(3) MDWF_DIR(4) MDWF_DIR(5) MDWF_DIR(6) MDWF_DIR(7)
#undef MDWF_DIR
        } else {
            // two directions in flight: load d + 1 before computing d
            Raw<P> r0, r1;
            r0.load(seg[0], lidx[0], lblk, src, jn[0], sblk, LM == 0);
            if constexpr (LM == 2) r0.load_part(seg[0], lidx[0], lblk, s);
            stage();
#define MDWF_STEP(d, rc, rn)                                                          \
    rn.load(seg[(d) + 1], lidx[(d) + 1], lblk, src, jn[(d) + 1], sblk, LM == 0);     \
    if constexpr (LM == 2) rn.load_part(seg[(d) + 1], lidx[(d) + 1], lblk, s);        \
    dir_term<P, D, PB, d, LM>(res, rc, lw, sw, a0, nb, b5, c5);
            MDWF_STEP(0, r0, r1) MDWF_STEP(1, r1, r0) MDWF_STEP(2, r0, r1) MDWF_STEP(3, r1, r0)
            MDWF_STEP(4, r0, r1) MDWF_STEP(5, r1, r0) MDWF_STEP(6, r0, r1)
#undef MDWF_STEP
            dir_term<P, D, PB, 7, LM>(res, r1, lw, sw, a0, nb, b5, c5);
        }
    }

    // ---- epilogue on the hop result
    if constexpr (TR::epi == 1 || TR::epi == 2) {
        // B K5^-1 (or its adjoint) across the L5 lanes
        five_lanes<P, TR::epi == 2, LM != 1>(res, ftile, cf.rm, cf.mq, lane, L5, spw);
    } else if constexpr (TR::epi == 3) {
        if (valid) {   // B^+ = b5 + c5 C^+
            cx<R> cr[12];
            apply_C_lanes<R, true>(nb, res, cr);
#pragma unroll
            for (int c = 0; c < 12; ++c) res[c] = b5 * res[c] + c5 * cr[c];
        }
    }

    // K5 B^-1 (or its adjoint) on the centre field
    cx<R> cd[12];
    if constexpr (TR::cen == 4 || TR::cen == 5) {
        // lanes past the lattice load site 0 (in bounds; no valid lane reads them)
        Field<P>::load(at_rhs(a.centre, a.stride, rhs), g.Vh, valid ? i * L5 + s : 0, cd);
        five_lanes<P, TR::cen == 5, LM != 1>(cd, ftile, cf.rw, cf.mq, lane, L5, spw);
    }

    double n2 = 0.0;
    if (valid) {
        const int j = i * L5 + s;
        const R hc = R(TR::coef);
        if constexpr (TR::cen == 4 || TR::cen == 5) {
#pragma unroll
            for (int c = 0; c < 12; ++c) res[c] = cd[c] + hc * res[c];
        } else if constexpr (TR::cen != 0) {
            cx<R> cv[12];
            Field<P>::load(at_rhs(a.centre, a.stride, rhs), g.Vh, j, cv);
            if constexpr (TR::cen == 1 || TR::cen == 2) {
                cx<R> cc[12];
                apply_C_lanes<R, TR::cen == 2>(nb, cv, cc);
                const R ka = R(cf.k5[0]), kb = R(cf.k5[1]);
#pragma unroll
                for (int c = 0; c < 12; ++c) res[c] = ka * cv[c] + kb * cc[c] + hc * res[c];
            } else {
#pragma unroll
                for (int c = 0; c < 12; ++c) res[c] = cv[c] + hc * res[c];
            }
        } else if constexpr (TR::coef != 1.0) {
#pragma unroll
            for (int c = 0; c < 12; ++c) res[c] = hc * res[c];
        }
        void* out = at_rhs(a.out, a.stride, rhs);
        if constexpr (TR::norm && P == P16) {   // the norm from the stored halves
            n2 = g.nt_store[P] ? Field<P>::template store_norm2<true>(out, g.Vh, j, res)
                               : Field<P>::template store_norm2<false>(out, g.Vh, j, res);
        } else {
            if (g.nt_store[P]) Field<P>::template store<true>(out, g.Vh, j, res);
            else Field<P>::store(out, g.Vh, j, res);
            if (TR::norm && a.partials) {
                R acc = R(0);
#pragma unroll
                for (int c = 0; c < 12; ++c) acc += res[c].re * res[c].re + res[c].im * res[c].im;
                n2 = double(acc);
            }
        }
    }
    if (TR::norm && a.partials) {
        // fixed-order reduction: wave (xor butterfly), then the 4 waves
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) n2 += __shfl_xor(n2, off, 64);
        __shared__ double wsum[kWaves];
        if (lane == 0) wsum[wave] = n2;
        __syncthreads();
        if (tid == 0) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) t += wsum[w];
            a.partials[size_t(rhs) * a.nblk + tile] = t;
        }
    }
}

int hop_blocks_per_rhs(const Geo& g) {
    const int spw = 64 / g.L5;
    const int sites_per_block = kWaves * spw;
    return (g.Vh4 + sites_per_block - 1) / sites_per_block;
}

// FP32 lattices of few waves wait for the staging instead of gaining by it; with
// the bits the same, links are staged above this many workgroups a right-hand
// side.  The line lies on the lattice alone, so that a right-hand side takes the
// same kernel alone and in any batch.  Staged over unstaged time at one right-hand
// side (L5 = 8 to 16; at four, each crosses 1 earlier):
//   bare hops       128 workgroups: 1.12, 216: 1.09, 432: 1.01, 1080: 0.96, 3000: 0.85
//                   (four right-hand sides: 1.01, 0.96, 0.93, 0.88, 0.91)
//   D5 and adjoint  1080: 1.02 and 1.18, 2304: 1.01 and 1.07, 2560: 0.97 and 1.00, 3000: 0.96
//   S B^-1          432: 1.05, 1792: 1.01, 2304: 1.00, 2560: 0.99, 3000: 0.96, 3600: 0.92
//   S, S^+          1080: 1.15 and 1.12, 2304: 1.11, 3000: 1.04, 3755: 1.04, 4096: 1.04 and
//                   1.00, 4320: 0.98 and 0.96 (kernels A, B and B^+ of it; A^+ is S B^-1's)
// (FP64, with three times the link loads to save, is staged everywhere: below 500
// workgroups S is up to 3 % slower and S B^-1 4 to 9 % faster.  FP16 too: 0 to 6 %
// slower below 4000, faster above.)
template <int K> constexpr int stage_blocks_f32() {
    if (K == HOP_BARE || K == HOP_BARE_DAG) return 350;
    return K == HOP_SCHUR_A || K == HOP_SCHUR_B || K == HOP_SCHUR_B_DAG ? 4000 : 2500;
}

template <Prec P, int K>
static void launch_hop_t(const Geo& g, const GaugeSet& gs, HopLaunch& L, hipStream_t st) {
    HopDev a;
    a.nblk = hop_blocks_per_rhs(g);
    int lm = g.link_mode[P];
    if (lm == 1 && 64 / g.L5 > kStageSites) lm = 0;
    if (lm == 1 && P == P32 && a.nblk <= stage_blocks_f32<K>()) lm = 0;
    if (lm == 2 && (P == P64 || g.L5 < link_parts<P>())) lm = 0;
    // matrix cores: FP16, blocks of four slices of one site, no B pre-hop
    if (lm == 3 && (P != P16 || g.L5 % 4 != 0 || HopTraits<K>::preB || !gs.mrow)) lm = 0;
    a.out = L.out;
    a.in = L.in;
    a.centre = L.centre;
    const size_t seg = gs.seg_bytes[P];
    a.lseg = seg;
    a.links_out = gs.seg[P] + size_t(L.out_parity) * 4 * seg;
    a.links_in = gs.seg[P] + size_t(1 - L.out_parity) * 4 * seg;
    a.rseg = gs.mrow_bytes;
    a.rows_out = gs.mrow ? gs.mrow + size_t(L.out_parity) * 4 * gs.mrow_bytes : nullptr;
    a.rows_in = gs.mrow ? gs.mrow + size_t(8 + (1 - L.out_parity) * 4) * gs.mrow_bytes : nullptr;
    a.stride = L.stride;
    a.nrhs = L.nrhs;
    a.out_parity = L.out_parity;
    a.coef = L.coef;
    a.active = L.active;
    a.partials = L.partials;
    L.nblocks_per_rhs = a.nblk;
    dim3 grid(a.nblk * L.nrhs);
    if (lm == 1) {
        hipLaunchKernelGGL((k_hop<P, K, 1>), grid, dim3(kBlock), 0, st, g, a);
    } else if (lm == 2) {
        if constexpr (P != P64) hipLaunchKernelGGL((k_hop<P, K, 2>), grid, dim3(kBlock), 0, st, g, a);
    } else if (lm == 3) {
        if constexpr (P == P16 && !HopTraits<K>::preB)
            hipLaunchKernelGGL((k_hop<P, K, 3>), grid, dim3(kBlock), 0, st, g, a);
    } else {
        hipLaunchKernelGGL((k_hop<P, K, 0>), grid, dim3(kBlock), 0, st, g, a);
    }
}

template <Prec P>
static void launch_hop_p(const Geo& g, const GaugeSet& gs, HopLaunch& L, hipStream_t st) {
    switch (L.kind) {
        case HOP_BARE: launch_hop_t<P, HOP_BARE>(g, gs, L, st); break;
        case HOP_BARE_DAG: launch_hop_t<P, HOP_BARE_DAG>(g, gs, L, st); break;
        case HOP_D5: launch_hop_t<P, HOP_D5>(g, gs, L, st); break;
        case HOP_D5_DAG: launch_hop_t<P, HOP_D5_DAG>(g, gs, L, st); break;
        case HOP_SCHUR_A: launch_hop_t<P, HOP_SCHUR_A>(g, gs, L, st); break;
        case HOP_SCHUR_B: launch_hop_t<P, HOP_SCHUR_B>(g, gs, L, st); break;
        case HOP_SCHUR_A_DAG: launch_hop_t<P, HOP_SCHUR_A_DAG>(g, gs, L, st); break;
        case HOP_SCHUR_B_DAG: launch_hop_t<P, HOP_SCHUR_B_DAG>(g, gs, L, st); break;
        case HOP_PREP: launch_hop_t<P, HOP_PREP>(g, gs, L, st); break;
        case HOP_SCHUR_B_SYM: launch_hop_t<P, HOP_SCHUR_B_SYM>(g, gs, L, st); break;
        case HOP_SCHUR_A_RP: launch_hop_t<P, HOP_SCHUR_A_RP>(g, gs, L, st); break;
        case HOP_SCHUR_B_RP: launch_hop_t<P, HOP_SCHUR_B_RP>(g, gs, L, st); break;
        case HOP_SCHUR_B_DAG_RP: launch_hop_t<P, HOP_SCHUR_B_DAG_RP>(g, gs, L, st); break;
    }
}

void launch_hop(const Geo& g, const GaugeSet& gs, HopLaunch& L, hipStream_t st) {
    if (launch_hop_plane(g, gs, L, st)) return;
    switch (L.prec) {
        case P64: launch_hop_p<P64>(g, gs, L, st); break;
        case P32: launch_hop_p<P32>(g, gs, L, st); break;
        case P16: launch_hop_p<P16>(g, gs, L, st); break;
    }
}

// ------------------------------------------------- site-local 5th dimension
// out = sum_k c_k C^k in (or with C^+), for K5, K5^-1 and B.
template <Prec P>
__global__ void __launch_bounds__(kBlock) k_fifth(const Geo g, int kind, int dag, const void* in, void* out,
                                                   size_t stride, int nrhs, int nblk, const RhsCoef* coef,
                                                   const int* active) {
    using R = typename Real<P>::T;
    const int L5 = g.L5;
    const int spw = 64 / L5;
    const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
    const int rhs = lb % nrhs;
    const int tile = lb / nrhs;
    if (active && !active[rhs]) return;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int sw = lane / L5;
    const int s = lane - sw * L5;
    const int i = (tile * kWaves + wave) * spw + sw;
    const bool valid = (sw < spw) && (i < g.Vh4);
    const int j = i * L5 + s;
    const RhsCoef& cf = coef[rhs];
    const R mq = R(cf.mq);

    __shared__ cx<R> sh[12 * kBlock];
    cx<R> v[12];
    if (valid) Field<P>::load(at_rhs(in, stride, rhs), g.Vh, j, v);
#pragma unroll
    for (int c = 0; c < 12; ++c) sh[c * kBlock + tid] = valid ? v[c] : cx<R>{R(0), R(0)};
    __syncthreads();
    if (!valid) return;

    // K5 = k5[0] + k5[1] C, B = b5 + c5 C, K5^-1 = sum_k kinv[k] C^k,
    // B^-1 = sum_k binv[k] C^k
    double two[2];
    const double* ck;
    if (kind == FIFTH_K5) { two[0] = cf.k5[0]; two[1] = cf.k5[1]; ck = two; }
    else if (kind == FIFTH_B) { two[0] = cf.b5; two[1] = cf.c5; ck = two; }
    else if (kind == FIFTH_BINV) { ck = cf.binv; }
    else { ck = cf.kinv; }
    cx<R> o[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) o[c] = {R(0), R(0)};
    const int tbase = tid - s;
    const int nterms = (kind == FIFTH_K5INV || kind == FIFTH_BINV) ? L5 : 2;
    for (int k = 0; k < nterms; ++k) {
        const R mk = R(ck[k]);
        int su = dag ? s + k : s - k;
        int sd = dag ? s - k : s + k;
        R fu = mk, fd = mk;
        // k may reach L5 only when L5 = 1 (then C^1 = -m_q on the single slice)
        while (su < 0) { su += L5; fu = -mq * fu; }
        while (su >= L5) { su -= L5; fu = -mq * fu; }
        while (sd < 0) { sd += L5; fd = -mq * fd; }
        while (sd >= L5) { sd -= L5; fd = -mq * fd; }
#pragma unroll
        for (int c = 0; c < 6; ++c) o[c] = o[c] + fu * sh[c * kBlock + tbase + su];
#pragma unroll
        for (int c = 6; c < 12; ++c) o[c] = o[c] + fd * sh[c * kBlock + tbase + sd];
    }
    Field<P>::store(at_rhs(out, stride, rhs), g.Vh, j, o);
}

void launch_fifth(const Geo& g, Prec p, FifthKind kind, int dag, const void* in, void* out, size_t stride,
                  int nrhs, const RhsCoef* coef, const int* active, hipStream_t st) {
    const int nblk = hop_blocks_per_rhs(g);
    dim3 grid(nblk * nrhs);
    switch (p) {
        case P64: hipLaunchKernelGGL(k_fifth<P64>, grid, dim3(kBlock), 0, st, g, int(kind), dag, in, out, stride, nrhs, nblk, coef, active); break;
        case P32: hipLaunchKernelGGL(k_fifth<P32>, grid, dim3(kBlock), 0, st, g, int(kind), dag, in, out, stride, nrhs, nblk, coef, active); break;
        case P16: hipLaunchKernelGGL(k_fifth<P16>, grid, dim3(kBlock), 0, st, g, int(kind), dag, in, out, stride, nrhs, nblk, coef, active); break;
    }
}

}  // namespace mdwf
