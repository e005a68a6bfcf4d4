// The row kernel: both horizontal path directions, the sum over the
// directions (Eq. 4) and the winner-take-all in one pass over a row.
//
// The aggregation stores the horizontal directions' values only where they
// enter a segment of kRowSegment columns (1/8 or 1/16 of a plane).  Here every
// segment is independent: 16 lanes walk it left to right from its entering
// state, keep the values in registers, walk it right to left from the other
// side's state, add the stored planes of the other directions at each step and
// take the winners.  Both walks use the same costs, loaded once.  So the two
// horizontal planes are never written nor read (4 of the 3P + 1 passes over a
// volume that one plane per direction takes, for two reads of the costs), at
// the price of running these two directions' arithmetic twice.
//
// The right view (D_R(x') = argmin_d S(x' + d, d)) is a systolic array: lane
// q, register i holds the smallest key offered so far to column x - d, with
// d = CPL q + i and x the current column; moving to column x - 1 shifts it
// down by one disparity, and what leaves at d = 0 is the segment's result for
// column x.  At the segment's left end the rest goes to the row's keys in LDS
// by atomic minima: Dp + SEG of them per segment instead of Dp SEG.
#pragma once

#include "sgm_device.h"

namespace sgm {
namespace dev {

struct RowArgs {
    const uint8_t* cost;  // C u8 [H][W][Dp]
    const void* planes;   // this SGM's planes of E = L - C: left-to-right (checkpoints), right-to-left
                          // (checkpoints; not in the 2-path set), then the other directions
    const uint8_t* img;   // base image (adaptive P2)
    uint16_t* dl;         // left disparity (raw, or the final output)
    uint16_t* dr;         // right-view disparity or nullptr
    int W, H, D, P1, P2, n_paths, adaptive;
    int subpixel;  // sub-pixel output of this SGM (its kernel is the SUB variant)
};

// Bytes of LDS of a row's right-view keys; its table of P2 by intensity change
// (256 u16) lies beside them.
static_assert(4 * (kMaxWidth + kWtaGuard) + 512 <= 64 * 1024, "a row's LDS at the largest width");
__host__ __device__ inline size_t row_smem_bytes(int W, bool right) { return right ? 4 * (size_t)(W + kWtaGuard) : 0; }

// One step of Eq. 3 for groups of G lanes: E = min(R - m, P2), L = C + E,
// then R and m of the next step.
template <int G, int NP, bool F16>
struct RowPath {
    u16x2 R[NP], mm;
    // R and m after a step that left L
    __device__ void after(const u16x2 (&L)[NP], u16x2 P1v, uint32_t edge_lo, uint32_t edge_hi) {
        u16x2 lp[NP];
#pragma unroll
        for (int k = 0; k < NP; ++k) lp[k] = F16 ? L[k] + P1v : vadds(L[k], P1v);
        const uint32_t prev = from_lower<G>(as1(lp[NP - 1])) | edge_lo;
        const uint32_t next = from_upper<G>(as1(lp[0])) | edge_hi;
        const u16x2 lo0 = as2(__builtin_amdgcn_alignbit(as1(lp[NP - 1]), prev, 16));
        const u16x2 hiN = as2(__builtin_amdgcn_alignbit(next, as1(lp[0]), 16));
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const u16x2 lo = k == 0 ? lo0 : lp[k - 1];
            const u16x2 hi = k == NP - 1 ? hiN : lp[k + 1];
            R[k] = F16 ? vmin3h(lo, hi, L[k]) : vmin(vmin(lo, hi), L[k]);
        }
        u16x2 t = L[0];
        if constexpr (F16 && NP >= 4) {
            t = vmin3h(L[0], L[1], L[2]);
#pragma unroll
            for (int k = 3; k + 1 < NP; k += 2) t = vmin3h(t, L[k], L[k + 1]);
            t = vmin(t, L[NP - 1]);
        } else {
#pragma unroll
            for (int k = 1; k < NP; ++k) t = vmin(t, L[k]);
        }
        mm = as2(group_min<G>(as1(vmin(t, t.yx))));
    }
    __device__ void step(const u16x2 (&c)[NP], u16x2 p2v, u16x2 P1v, uint32_t edge_lo, uint32_t edge_hi, u16x2 (&E)[NP]) {
        u16x2 L[NP];
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            E[k] = vmin(R[k] - mm, p2v);
            L[k] = F16 ? E[k] + c[k] : vadds(E[k], c[k]);
        }
        after(L, P1v, edge_lo, edge_hi);
    }
};

// One lane's values of one pixel in a plane: CPL bytes or u16.
template <int CPL, typename LT>
struct RowValues {
    static constexpr int NW = CPL * (int)sizeof(LT) / 4;  // dwords
    uint32_t w[NW];
};

template <int CPL, typename LT, int AUX>
__device__ inline RowValues<CPL, LT> row_load(__amdgpu_buffer_rsrc_t r, uint32_t ofs) {
    RowValues<CPL, LT> v;
    constexpr int NW = RowValues<CPL, LT>::NW;
    if constexpr (NW == 1) {
        v.w[0] = __builtin_amdgcn_raw_buffer_load_b32(r, ofs, 0, AUX);
    } else if constexpr (NW == 2) {
        const auto t = __builtin_amdgcn_raw_buffer_load_b64(r, ofs, 0, AUX);
        v.w[0] = t[0];
        v.w[1] = t[1];
    } else {
#pragma unroll
        for (int i = 0; i < NW / 4; ++i) {
            const auto t = __builtin_amdgcn_raw_buffer_load_b128(r, ofs + 16 * i, 0, AUX);
#pragma unroll
            for (int k = 0; k < 4; ++k) v.w[4 * i + k] = t[k];
        }
    }
    return v;
}

// Pair k of the split layout: values k and k + CPL / 2.
template <int CPL, typename LT>
__device__ inline u16x2 row_pair(const RowValues<CPL, LT>& v, int k) {
    constexpr int NP = CPL / 2;
    if constexpr (sizeof(LT) == 1) {
        const int a = k, b = k + NP;
        const uint32_t sel = (uint32_t)(a & 3) | 0x0C00u | ((uint32_t)(4 + (b & 3)) << 16) | 0x0C000000u;
        return as2(__builtin_amdgcn_perm(v.w[b >> 2], v.w[a >> 2], sel));
    } else {
        const int a = k, b = k + NP;
        const uint32_t sel = ((a & 1) ? 0x0302u : 0x0100u) | (((b & 1) ? 0x0706u : 0x0504u) << 16);
        return as2(__builtin_amdgcn_perm(v.w[b >> 1], v.w[a >> 1], sel));
    }
}

// Costs of pair k; `sel` as unpack_selector.
template <int CPL>
__device__ inline void row_costs(const RowValues<CPL, uint8_t>& v, const uint32_t (&sel)[CPL / 2], u16x2 (&c)[CPL / 2]) {
    if constexpr (CPL == 4) {
        unpack_costs<4>(v.w[0], sel, c);
    } else if constexpr (CPL == 8) {
        unpack_costs<8>(make_uint2(v.w[0], v.w[1]), sel, c);
    } else {
        unpack_costs<16>(make_uint4(v.w[0], v.w[1], v.w[2], v.w[3]), sel, c);
    }
}

template <int CPL, typename LT>
__device__ inline RowValues<CPL, LT> row_pack(const u16x2 (&e)[CPL / 2]) {
    RowValues<CPL, LT> v;
    if constexpr (sizeof(LT) == 1) {
        const auto p = pack_u8<CPL>(e);
        if constexpr (CPL == 4) {
            v.w[0] = p;
        } else if constexpr (CPL == 8) {
            v.w[0] = p.x;
            v.w[1] = p.y;
        } else {
            v.w[0] = p.x;
            v.w[1] = p.y;
            v.w[2] = p.z;
            v.w[3] = p.w;
        }
    } else {
        constexpr int NP = CPL / 2;
#pragma unroll
        for (int i = 0; i < NP / 2; ++i) {
            v.w[i] = __builtin_amdgcn_perm(as1(e[2 * i + 1]), as1(e[2 * i]), 0x05040100u);
            v.w[NP / 2 + i] = __builtin_amdgcn_perm(as1(e[2 * i + 1]), as1(e[2 * i]), 0x07060302u);
        }
    }
    return v;
}

// NV: directions with stored planes (1: the 2-path set, which has no
// right-to-left direction; 2, 6: 4 and 8 paths).  NT: the planes are loaded
// non-temporally.  PAIR: two values fit a byte together (2 P2 <= 255), so
// planes are added two at a time in bytes before they are widened.  SUB:
// sub-pixel output.
template <int Dp, int NV, typename LT, bool NT, bool PAIR, bool SUB>
__device__ inline void row_block(const RowArgs& a, int y, uint32_t* keyR_smem, const uint16_t* p2lut) {
    // lanes per segment: 8 levels a lane at most, which leaves registers for
    // three or four wavefronts per SIMD
    constexpr int G = Dp == 256 ? 32 : 16, S = 64 / G;
    constexpr int CPL = Dp / G, NP = CPL / 2;
    constexpr bool F16 = sizeof(LT) == 1;
    constexpr bool HB = NV != 1;  // a right-to-left direction
    constexpr int SEG = RowSegment<Dp, LT>::N;
    constexpr int A = NT ? 2 : 0;
    constexpr int UW = S * SEG;  // columns a wavefront takes at a time
    // plane values in flight: steps ahead of the one that adds them
    constexpr int PD = NV * CPL * (int)sizeof(LT) >= 48 ? 3 : (NV * CPL * (int)sizeof(LT) >= 16 ? 4 : 8);
    static_assert(PD <= SEG, "lookahead within a segment");
    using V = RowValues<CPL, LT>;

    const int W = a.W;
    const bool right = a.dr != nullptr;
    uint32_t* keyR = keyR_smem + kWtaGuard;  // keyR[t], t in [-kWtaGuard, W)
    if (right) {
        for (int i = threadIdx.x; i < W + kWtaGuard; i += blockDim.x) keyR_smem[i] = ~0u;
        __syncthreads();
    }
    const int lane = threadIdx.x & 63, grp = lane / G, q = lane % G;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), nwaves = blockDim.x >> 6;

    uint32_t sel[NP], dpair[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        sel[k] = unpack_selector<CPL>(k, q * CPL, a.D, F16);
        dpair[k] = (uint32_t)(q * CPL + k) | ((uint32_t)(q * CPL + k + NP) << 8);
    }
    const uint32_t inf = F16 ? 0x0FFFu : 0xFFFFu;
    const uint32_t edge_lo = q == 0 ? inf << 16 : 0u, edge_hi = q == G - 1 ? inf : 0u;
    const uint32_t edge_col = q == G - 1 ? ~0u : 0u;
    const uint32_t P1c = F16 && !a.adaptive ? (uint32_t)min(a.P1, a.P2) : (uint32_t)a.P1;
    const u16x2 P1v = as2(P1c * 0x10001u);
    const u16x2 nn = as2((uint32_t)a.n_paths * 0x10001u);

    // Buffers of this row alone: columns outside it load as zeros, and zero
    // costs and states keep a path at its start (R = 0, m = 0 on every real
    // level), so the row's ends need no code of their own.
    const size_t plane = (size_t)W * a.H * Dp, row0 = (size_t)y * W * Dp;
    const uint32_t rowb = (uint32_t)W * (uint32_t)Dp;
    const __amdgpu_buffer_rsrc_t rc = buffer_rsrc(a.cost + row0, rowb);
    const LT* pl = reinterpret_cast<const LT*>(a.planes) + row0;
    const __amdgpu_buffer_rsrc_t rf = buffer_rsrc(pl, rowb * (uint32_t)sizeof(LT));
    const __amdgpu_buffer_rsrc_t rb = buffer_rsrc(pl + (HB ? plane : 0), rowb * (uint32_t)sizeof(LT));
    __amdgpu_buffer_rsrc_t rv[NV];
#pragma unroll
    for (int p = 0; p < NV; ++p) rv[p] = buffer_rsrc(pl + plane * (p + (HB ? 2 : 1)), rowb * (uint32_t)sizeof(LT));

    const __amdgpu_buffer_rsrc_t rd = buffer_rsrc(a.dl + (size_t)y * W, 2u * (uint32_t)W);
    const __amdgpu_buffer_rsrc_t ri = buffer_rsrc(a.img + (size_t)y * W, (uint32_t)W);

    // The loads run ahead of the walks and across units, so that a unit
    // starts with its data at hand: the costs in the order they are used
    // (columns 0 .. SEG - 1, then back), RC of them in flight; a plane value
    // PD steps ahead; entering states and intensities a walk ahead.  The
    // right-to-left walk loads the costs again (from L2) rather than keep
    // them, which leaves registers for another wavefront per SIMD.
    constexpr int RC = 8;
    using C = RowValues<CPL, uint8_t>;
    C ring[RC];
    V ef, eb, vp[PD][NV];
    C cf, cb;
    uint32_t inten[3];
    const uint32_t ustep = (uint32_t)(nwaves * UW * Dp);
    // byte offset of the lane's costs at its segment's first column
    uint32_t at = (uint32_t)((wave * UW + grp * SEG) * Dp + q * CPL);
    auto load_cost = [&](int s) {  // place s of the unit's 2 SEG uses; past them the next unit's
        const uint32_t base = s < 2 * SEG ? at : at + ustep;
        const int t = s % (2 * SEG), j = t < SEG ? t : 2 * SEG - 1 - t;
        ring[s % RC] = row_load<CPL, uint8_t, 0>(rc, base + j * Dp);
    };
    auto load_planes = [&](int j, V (&v)[NV]) {
#pragma unroll
        for (int p = 0; p < NV; ++p) v[p] = row_load<CPL, LT, A>(rv[p], (at + j * Dp) * (uint32_t)sizeof(LT));
    };
    auto load_left_state = [&](uint32_t base) {
        ef = row_load<CPL, LT, 0>(rf, (base - Dp) * (uint32_t)sizeof(LT));
        cf = row_load<CPL, uint8_t, 0>(rc, base - Dp);
        // intensities of the lane's column and its neighbours (adaptive P2)
        const int x = (int)(base / (uint32_t)Dp) + (q & (SEG - 1));
#pragma unroll
        for (int i = 0; i < 3; ++i)
            inten[i] = __builtin_amdgcn_raw_buffer_load_b8(ri, (uint32_t)clampi(x + i - 1, 0, W - 1), 0, 0);
    };
    load_left_state(at);
#pragma unroll
    for (int s = 0; s < RC; ++s) load_cost(s);
    for (int u = wave; u * UW < W; u += nwaves) {
        const int x0 = u * UW + grp * SEG;
        RowPath<G, NP, F16> path;
        // state after column x0 - 1 (or x0 + SEG) from its stored values
        auto enter = [&](const V& e, const C& cv) {
            u16x2 c[NP], L[NP];
            row_costs<CPL>(cv, sel, c);
#pragma unroll
            for (int k = 0; k < NP; ++k) L[k] = F16 ? row_pair<CPL, LT>(e, k) + c[k] : vadds(row_pair<CPL, LT>(e, k), c[k]);
            path.after(L, P1v, edge_lo, edge_hi);
        };
        // P2 of the segment's steps, one per lane of a row of 16 (the table
        // holds P2 alone without the adaptive option)
        const int i0 = (int)inten[1];
        const uint32_t p2f = p2lut[abs(i0 - (int)inten[0])] * 0x10001u, p2b = p2lut[abs(i0 - (int)inten[2])] * 0x10001u;
        enter(ef, cf);
        if constexpr (HB) {
            eb = row_load<CPL, LT, 0>(rb, (at + SEG * Dp) * (uint32_t)sizeof(LT));
            cb = row_load<CPL, uint8_t, 0>(rc, at + SEG * Dp);
        }
        V fwd[SEG];
#pragma unroll
        for (int j = 0; j < SEG; ++j) {
            __builtin_amdgcn_sched_barrier(0);
            u16x2 c[NP], e[NP];
            row_costs<CPL>(ring[j % RC], sel, c);
            load_cost(j + RC);
            if (j >= SEG - PD) load_planes(j, vp[j % PD]);
            path.step(c, as2(row_broadcast(p2f, j)), P1v, edge_lo, edge_hi, e);
            fwd[j] = row_pack<CPL, LT>(e);
        }
        __builtin_amdgcn_sched_barrier(0);
        load_left_state(at + ustep);
        if constexpr (HB) enter(eb, cb);
        uint32_t col[CPL];  // right view: smallest keys of columns x - d
#pragma unroll
        for (int i = 0; i < CPL; ++i) col[i] = ~0u;
        uint32_t outl = 0, outn = 0, outr = 0;  // lane j: results of column x0 + j
#pragma unroll
        for (int j = SEG - 1; j >= 0; --j) {
            __builtin_amdgcn_sched_barrier(0);
            u16x2 c[NP], S[NP];
            row_costs<CPL>(ring[(2 * SEG - 1 - j) % RC], sel, c);
            load_cost(2 * SEG - 1 - j + RC);
            if constexpr (HB)
                path.step(c, as2(row_broadcast(p2b, j)), P1v, edge_lo, edge_hi, S);
            V(&v)[NV] = vp[j % PD];
            if constexpr (PAIR && !HB) {  // E of both directions in bytes
#pragma unroll
                for (int i = 0; i < V::NW; ++i) v[0].w[i] += fwd[j].w[i];
#pragma unroll
                for (int k = 0; k < NP; ++k) S[k] = c[k] * nn + row_pair<CPL, LT>(v[0], k);
            } else {
#pragma unroll
                for (int k = 0; k < NP; ++k) {
                    const u16x2 f = row_pair<CPL, LT>(fwd[j], k);
                    S[k] = HB ? c[k] * nn + (S[k] + f) : c[k] * nn + f;
                }
                if constexpr (PAIR) {
#pragma unroll
                    for (int p = 0; p < NV; p += 2)
#pragma unroll
                        for (int i = 0; i < V::NW; ++i) v[p].w[i] += v[p + 1].w[i];
                }
#pragma unroll
                for (int p = 0; p < NV; p += PAIR ? 2 : 1)
#pragma unroll
                    for (int k = 0; k < NP; ++k) S[k] = S[k] + row_pair<CPL, LT>(v[p], k);
            }
            if (j >= PD) load_planes(j - PD, vp[j % PD]);
            // padded levels lose: with byte planes they sum to more than
            // 1023 per path; 16-bit ones are set to the maximum (a real level
            // there has the smaller d)
            if constexpr (!F16) {
#pragma unroll
                for (int k = 0; k < NP; ++k) {
                    const uint32_t lo = q * CPL + k < a.D ? 0u : 0xFFFFu, hi = q * CPL + k + NP < a.D ? 0u : 0xFFFF0000u;
                    S[k] = as2(as1(S[k]) | lo | hi);
                }
            }
            // keys (S << 8) | d: the smallest wins, ties to the smaller d
            uint32_t key[CPL];
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                key[k] = __builtin_amdgcn_perm(as1(S[k]), dpair[k], 0x0C050400u);
                key[k + NP] = __builtin_amdgcn_perm(as1(S[k]), dpair[k], 0x0C070601u);
            }
            uint32_t best = key[0];
#pragma unroll
            for (int i = 1; i < CPL; ++i) best = min(best, key[i]);
            best = group_min<G>(best);
            // results enter at lane 0 and move up as the walk goes left
            if constexpr (SUB) {
                // the winner's key, and S(d - 1) | S(d + 1) << 16 from the
                // lanes that hold them; the vertex (a division) is taken once
                // a unit, by the lane the column ends in (640x480, D = 128, 4
                // paths: a call 99 us, 111 with the vertex in every step)
                const int t = (int)(best & 0xFFu) - q * CPL;
                uint32_t va = 0, vc = 0;
#pragma unroll
                for (int i = 0; i < CPL; ++i) {
                    if (t == i + 1) va = key[i];
                    if (t == i - 1) vc = key[i];
                }
                const uint32_t nb = group_or<G>(__builtin_amdgcn_perm(vc, va, 0x06050201u));
                outl = (uint32_t)__builtin_amdgcn_update_dpp((int)best, (int)outl, kDppRowShr1, 0xF, 0xF, false);
                outn = (uint32_t)__builtin_amdgcn_update_dpp((int)nb, (int)outn, kDppRowShr1, 0xF, 0xF, false);
            } else {
                outl = (uint32_t)__builtin_amdgcn_update_dpp((int)(best & 0xFFu), (int)outl, kDppRowShr1, 0xF, 0xF, false);
            }
            // the columns take the smaller key; past the row's end (off = ~0)
            // the median leaves them at ~0
            const uint32_t up = from_upper<G>(col[0]) | edge_col;
            const uint32_t off = (uint32_t)((W - 1 - x0 - j) >> 31);
#pragma unroll
            for (int i = 0; i < CPL; ++i) {
                const uint32_t o = i + 1 < CPL ? col[i + 1] : up;
                col[i] = max(min(o, key[i]), min(max(o, key[i]), off));
            }
            outr = (uint32_t)__builtin_amdgcn_update_dpp((int)col[0], (int)outr, kDppRowShr1, 0xF, 0xF, false);
        }
        if constexpr (SUB) outl = a.subpixel ? subpixel_q4(outl, outn & 0xFFFFu, outn >> 16, a.D) : outl & 0xFFu;
        const bool mine = q < SEG && x0 + q < W;
        // (lanes beyond the segment or the row store outside the buffer)
        __builtin_amdgcn_raw_buffer_store_b16((uint16_t)outl, rd, q < SEG ? 2u * (uint32_t)(x0 + q) : ~1u, 0, 0);
        if (right && x0 < W) {
            if (mine) atomicMin(&keyR[x0 + q], outr);
            // columns left of the segment (down to x0 - 255 in the guard)
#pragma unroll
            for (int i = 0; i < CPL; ++i) atomicMin(&keyR[x0 - (q * CPL + i)], col[i]);
        }
        at += ustep;
    }
    if (right) {
        __syncthreads();
        for (int i = threadIdx.x; i < W; i += blockDim.x) a.dr[(size_t)y * W + i] = (uint16_t)(keyR[i] & 0xFF);
    }
}

}  // namespace dev
}  // namespace sgm
