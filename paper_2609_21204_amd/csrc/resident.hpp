// Small systems on one workgroup, with their state on the chip.
//
// A system of at most kResMaxN particles gives every particle a thread (two
// threads where the workgroup has them), which keeps the particle's position,
// velocity, build position and bond words in registers for the whole launch.
// Positions of all particles live in LDS in two buffers (read one, write the
// other: one barrier per step), neighbour lists, cell lists and the matching's
// keys in LDS as well.  A launch takes the lists as they were last built, and
// builds where the grid kernels would: the same builds are counted, and the
// same lists and cells checked against their limits.  A step then touches global memory only for image
// counters (a particle that crosses the box) and in the sweeps, for the bond
// slots.  What bounds a step here is the latency of one particle's chain of
// work and, with 16 waves on a CU, the issue of its instructions.
//
// Every sum is exact and every decision is keyed by tag, so the trajectory is
// bit for bit that of db_step's grid kernels.
#pragma once

#include "kernels.hpp"

namespace dyb {

constexpr uint32_t kResMaxN = 1024;        // particles: a thread each
constexpr uint32_t kResMaxCells = 5000;    // cells of the list grid that fit the LDS layout
constexpr uint32_t kResList1 = 24, kResList2 = 16;   // list entries per thread in LDS, with 1 and 2 threads per particle

__host__ __device__ constexpr uint32_t res_list(uint32_t tpp) { return (tpp == 2u ? kResList2 : kResList1) * tpp; }

// Dynamic LDS of a resident system, in this order: positions (2 n float4),
// matching keys (2 n words of 8 bytes), cell offsets (ncell + 1), claims (n),
// lists (res_list n words of 2 bytes), particles in cell order (n words of 2
// bytes), occupancies (n bytes).
__host__ __device__ constexpr uint32_t res_lds_bytes(uint32_t n, uint32_t ncell, uint32_t tpp) {
    return 32u * n + 16u * n + 4u * (ncell + 1u) + 4u * n + 2u * res_list(tpp) * n + 2u * n + n + 16u;
}

// Where a system's run stands: read at the start of a launch, written back
// at its end, so consecutive launches of a batch chain without the host.
struct BatchState {
    unsigned long long t;    // step of the system
    int cur_x, cur_list;     // current position buffer and cell list
    uint32_t err[4];         // the system's device error words after the launch
    uint32_t listed;         // entries of all its neighbour lists
};

// Neighbour entries of one thread: the first KL in LDS, further ones in the
// system's list in memory (slot-major rows of nlmax, not used otherwise
// during a run): entry q >= KL in row q, or with two threads per particle,
// for the second of them, in row top - (q - KL), so that the pair's entries
// meet from both ends and fit together wherever their sum fits nlmax.
template <int TPP>
struct ResList {
    static constexpr uint32_t KL = TPP == 2 ? kResList2 : kResList1;
    static_assert(KL <= 32, "one bit per entry");
    uint16_t* lst;           // entry q < KL at lst[q * stride]
    uint32_t* far;           // the particle's column of the list in memory
    uint32_t stride, n, m, sub, top;
    __device__ __forceinline__ uint32_t row(uint32_t q) const { return TPP == 2 && sub ? top - (q - KL) : q; }
    __device__ __forceinline__ uint32_t near_at(uint32_t q) const { return lst[q * stride]; }
    __device__ __forceinline__ uint32_t far_at(uint32_t q) const { return far[(size_t)row(q) * n]; }
    __device__ __forceinline__ uint32_t at(uint32_t q) const { return q < KL ? near_at(q) : far_at(q); }
};

template <int TPP>
__device__ __forceinline__ long long res_sum(long long v) {
    if (TPP == 1) return v;
    // the other thread of the pair: DPP quad permutation [1, 0, 3, 2]
    const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)v, 0xB1, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)((unsigned long long)v >> 32), 0xB1, 0xF, 0xF, true);
    return v + (long long)(((unsigned long long)(uint32_t)hi << 32) | (uint32_t)lo);
}

// nsteps of the system from state st (see k_batch for the step's contents).
// flag and more: three LDS words each, zero on entry.
template <bool EXT, int TPP>
__device__ __forceinline__ void resident_steps(const Params& P, const Dev& D, const StepTabs& T, unsigned char* lds,
                                               const BatchState& st, uint32_t nsteps, uint32_t* flag, uint32_t* more,
                                               BatchState* out) {
    constexpr uint32_t KL = ResList<TPP>::KL;
    constexpr int BW = 4;                          // bond words held in registers per thread
    const uint32_t tid = threadIdx.x, bs = blockDim.x, n = P.n;
    const uint32_t i = tid / TPP, sub = tid % TPP;
    const bool live = i < n, own = live && sub == 0u;
    const int nc = (int)P.nc;
    const uint32_t ncell = P.ncell;
    float4* const xs = reinterpret_cast<float4*>(lds);
    unsigned long long* const B0 = reinterpret_cast<unsigned long long*>(xs + 2 * n);
    unsigned long long* const B1 = B0 + n;
    uint32_t* const cst = reinterpret_cast<uint32_t*>(B1 + n);
    uint32_t* const claimed = cst + ncell + 1;
    uint16_t* const lst = reinterpret_cast<uint16_t*>(claimed + n);
    uint16_t* const order = lst + KL * TPP * n;
    uint8_t* const occs = reinterpret_cast<uint8_t*>(order + n);
    const unsigned long long t0 = st.t;
    const int xin0 = st.cur_x;

    float4 p = make_float4(0.f, 0.f, 0.f, 0.f), u = p;
    float3 ref = make_float3(0.f, 0.f, 0.f);       // build position, on the packed grid
    uint32_t listed = 0;
    if (live) {
        p = D.x[xin0][i];
        u = D.u[i];
        ref = xref_point(P, D.xref[i]);
        listed = D.nl_cnt[i];
    }
    const uint32_t ti = type_of(p), tag = __float_as_uint(u.w);
    const uint32_t nstat = P.stat_max, nslot = live ? nstat + T.cap[ti] : 0u;
    uint32_t bw[BW];
    auto load_bonds = [&]() {
#pragma unroll
        for (int q = 0; q < BW; ++q) {
            const uint32_t b = sub + (uint32_t)q * TPP;
            bw[q] = b < nslot ? (b < nstat ? D.stat[(size_t)b * n + i] : D.dyn[(size_t)(b - nstat) * n + i]) : kEmpty;
        }
    };
    load_bonds();
    const uint32_t at = live ? i : 0u;
    // the lists as they were last built: the second thread of a pair takes the
    // last half, from the end
    ResList<TPP> L{lst + sub * n + at, D.nl + at, TPP * n, n, TPP == 2 ? (listed + 1u - sub) / 2u : listed, sub,
                   listed - 1u - KL};
    for (uint32_t q0 = 0, lim = min(L.m, KL); q0 < lim; q0 += 4) {
        uint32_t j[4];
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e) {
            const uint32_t q = min(q0 + e, lim - 1u);
            j[e] = L.far[(size_t)(sub ? listed - 1u - q : q) * n];
        }
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e)
            if (q0 + e < lim) L.lst[(q0 + e) * L.stride] = (uint16_t)j[e];
    }
    bool built = false;                            // since the launch began (the same for the whole workgroup)

    // Lists at the positions X (p: this thread's own): a counting sort of the
    // particles by cell, then each thread scans the 9 (5 and 4 with two
    // threads per particle) rows of 3 cells around its particle, 4 candidates
    // at a time.  An over-full cell or list is the error it is for db_step.
    auto build = [&](const float4* X) {
        for (uint32_t c = tid; c < ncell; c += bs) cst[c] = 0u;
        __syncthreads();
        const int cx = cell_coord(p.x, P), cy = cell_coord(p.y, P), cz = cell_coord(p.z, P);
        const uint32_t c = (uint32_t)((cz * nc + cy) * nc + cx);
        uint32_t slot = 0;
        if (own) {
            slot = atomicAdd(&cst[c], 1u);
            if (slot >= P.cellcap) atomicOr(&D.err[0], kErrOverflow);
        }
        __syncthreads();
        const uint32_t per = (ncell + bs - 1) / bs, c0 = min(tid * per, ncell), c1 = min(c0 + per, ncell);
        uint32_t sum = 0, total;
        for (uint32_t k = c0; k < c1; ++k) sum += cst[k];
        uint32_t run = block_exclusive_scan(sum, &total);
        for (uint32_t k = c0; k < c1; ++k) {
            const uint32_t v = cst[k];
            cst[k] = run;
            run += v;
        }
        if (tid == 0) cst[ncell] = n;
        __syncthreads();
        if (own) order[cst[c] + slot] = (uint16_t)i;
        __syncthreads();
        uint32_t m = 0;
        L.top = P.nlmax - 1u;
        if (live) {
            const float* rrow = T.rl2 + pair_index(P, ti, 0u);
            for (uint32_t r = sub; r < 9u; r += TPP) {
                const uint32_t rz = r / 3u, ry = r - 3u * rz;
                const int row = (wrapc(cz + (int)rz - 1, nc) * nc + wrapc(cy + (int)ry - 1, nc)) * nc;
                // the row's cells cx - 1 .. cx + 1: one run, or two where it wraps
                const int xa = cx == 0 ? nc - 1 : cx - 1, xb = cx == nc - 1 ? nc : (cx == 0 ? nc : cx + 2);
                const uint32_t s0 = cst[row + xa], n0 = cst[row + xb] - s0;
                const bool wraps = cx == 0 || cx == nc - 1;
                const uint32_t s1 = cst[row], n1 = wraps ? cst[row + (cx == 0 ? 2 : 1)] - s1 : 0u;
                const uint32_t len = n0 + n1;
                for (uint32_t k0 = 0; k0 < len; k0 += 4) {
                    uint32_t j[4];
                    float4 q[4];
#pragma unroll
                    for (uint32_t e = 0; e < 4; ++e) {
                        const uint32_t k = min(k0 + e, len - 1u);
                        j[e] = order[k < n0 ? s0 + k : s1 + (k - n0)];
                    }
#pragma unroll
                    for (uint32_t e = 0; e < 4; ++e) q[e] = X[j[e]];
#pragma unroll
                    for (uint32_t e = 0; e < 4; ++e) {
                        const float dx = mi_delta_list(p.x, q[e].x, P), dy = mi_delta_list(p.y, q[e].y, P),
                                    dz = mi_delta_list(p.z, q[e].z, P);
                        if (k0 + e < len && j[e] != i && dx * dx + dy * dy + dz * dz < rrow[type_of(q[e])]) {
                            if (m < KL) L.lst[m * L.stride] = (uint16_t)j[e];
                            else if (L.row(m) < P.nlmax) L.far[(size_t)L.row(m) * n] = j[e];
                            ++m;
                        }
                    }
                }
            }
        }
        const uint32_t both = TPP == 2 ? m + (uint32_t)__shfl_xor((int)m, 1, 64) : m;
        if (own && both > P.nlmax) atomicOr(&D.err[0], kErrNlist);
        L.m = min(m, max(KL, P.nlmax));            // (beyond it only after that error)
        ref = xref_point(P, xref_pack(P, p));
        built = true;
    };

    if (own) xs[i] = p;
    __syncthreads();
    for (uint32_t k = 0; k < nsteps; ++k) {
        const unsigned long long s = t0 + k + 1ull;
        const bool sweep = P.nrx > 0 && (s % P.period) == 0;
        const int ake = (sweep && P.kt_kinetic) ? 1 : 0;
        if (tid == 0) flag[(k + 1) % 3] = 0u;      // last read two steps ago
        const float4* const X = xs + (k & 1u) * n;
        float4* const Xn = xs + ((k & 1u) ^ 1u) * n;
        unsigned long long ke = 0ull;
        long long fx = 0, fy = 0, fz = 0;
        if (live) {
            // pairs: screen the thread's entries 2 at a time, then evaluate
            // those inside the cutoff, FP32 ones first, so that a wave runs
            // as many evaluations as its busiest lane needs.  Entries beyond
            // the LDS slots follow in rounds, brought into words that only the
            // sweep uses (a load from either place, chosen per entry, cost
            // every step 2.5 %, a loop of its own for them 9 %).
            const uint16_t* cur = L.lst;
            uint32_t q0 = 0, cnt = min(L.m, KL);
            for (;;) {
                uint32_t near = 0u, exact = 0u;
                for (uint32_t q1 = 0; q1 < cnt; q1 += 2) {
                    uint32_t j[2];
                    float4 pj[2];
#pragma unroll
                    for (uint32_t e = 0; e < 2; ++e) j[e] = cur[min(q1 + e, cnt - 1u) * L.stride];
#pragma unroll
                    for (uint32_t e = 0; e < 2; ++e) pj[e] = X[j[e]];
#pragma unroll
                    for (uint32_t e = 0; e < 2; ++e) {
                        const uint32_t w = pair_screen(P, T, p, pj[e], ti);
                        const uint32_t bit = q1 + e < cnt ? 1u << (q1 + e) : 0u;
                        near |= w == kPairNear ? bit : 0u;
                        exact |= w == kPairExact ? bit : 0u;
                    }
                }
                while (near) {
                    const uint32_t q = (uint32_t)__builtin_ctz(near);
                    near &= near - 1u;
                    pair_force_near(P, T, D.err, p, X[cur[q * L.stride]], ti, fx, fy, fz);
                }
                while (exact) {
                    const uint32_t q = (uint32_t)__builtin_ctz(exact);
                    exact &= exact - 1u;
                    pair_force_f64(P, T, D.err, p, X[cur[q * L.stride]], ti, fx, fy, fz);
                }
                q0 += cnt;
                if (q0 >= L.m) break;
                constexpr uint32_t kRound = 8 / TPP;         // 16 bytes of keys per particle
                uint16_t* const spare = reinterpret_cast<uint16_t*>(B0) + sub * n + i;
                uint32_t far[kRound];
                cnt = min(L.m - q0, kRound);
#pragma unroll
                for (uint32_t e = 0; e < kRound; ++e) far[e] = L.far_at(q0 + min(e, cnt - 1u));
#pragma unroll
                for (uint32_t e = 0; e < kRound; ++e) spare[e * L.stride] = (uint16_t)far[e];
                cur = spare;
            }
            auto bond = [&](uint32_t b, uint32_t w) {
                const uint32_t j = w & kIdxMask;
                bond_force_tab<EXT>(P, T, D, p, X[j], b < nstat ? w >> 24 : T.rbt[(w >> 24) & 0x7Fu], i, j, fx, fy, fz);
            };
#pragma unroll
            for (int q = 0; q < BW; ++q)
                if (bw[q] != kEmpty) bond(sub + (uint32_t)q * TPP, bw[q]);
            for (uint32_t b = sub + BW * TPP; b < nslot; b += TPP) {
                const uint32_t w = b < nstat ? D.stat[(size_t)b * n + i] : D.dyn[(size_t)(b - nstat) * n + i];
                if (w != kEmpty) bond(b, w);
            }
        }
        fx = res_sum<TPP>(fx);
        fy = res_sum<TPP>(fy);
        fz = res_sum<TPP>(fz);
        if (live) {
            int ix, iy, iz;
            float4 po, v;
            ke = advance_state(P, T, p, ti, fix_to_force(D, fx, fy, fz), u, tag, s, ake, po, v, ix, iy, iz);
            p = po;
            u = v;
            if (own) {
                Xn[i] = po;
                if (ix | iy | iz) {
                    D.img[i] += ix;
                    D.img[n + i] += iy;
                    D.img[2 * (size_t)n + i] += iz;
                }
                const float dx = mi_delta_list(ref.x, p.x, P), dy = mi_delta_list(ref.y, p.y, P),
                            dz = mi_delta_list(ref.z, p.z, P);
                if (dx * dx + dy * dy + dz * dz > P.disp2) flag[k % 3] = 1u;
            }
        }
        if (ake) {
            ke = own ? ke : 0ull;
            for (int off = 32; off >= 1; off >>= 1) ke += __shfl_xor(ke, off, 64);
            if (__lane_id() == 0 && ke)
                __hip_atomic_fetch_add(&D.ke_fix[ke_slot(P, s)], ke, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        __syncthreads();
        if (flag[k % 3]) {
            if (tid == 0) ++D.rflag[4];            // builds so far, on the grid kernels' schedule
            build(Xn);
            __syncthreads();
        }
        if (!sweep) continue;
        for (int slot = 0; slot < (int)P.nrx; ++slot) {
            const int a = reaction_at(P.seed, s, (int)P.nrx, slot);
            if (own) {
                B0[i] = kNoKey;
                B1[i] = kNoKey;
                claimed[i] = 0u;
                occs[i] = D.occ[i];
            }
            if (tid < 3) more[tid] = 0u;
            if (slot == 0 && tid == 0) {           // a new sweep: its event lists start empty
                // and the next sweep's energy slot, with barriers between this
                // and the adds of the next step (a sweep may follow every step)
                D.ke_fix[ke_slot(P, s) ^ 1u] = 0ull;
                D.evc[0] = 0u;
                D.evc[1] = 0u;
                D.evc[2] = (uint32_t)s;
                D.evc[3] = (uint32_t)(s >> 32);
            }
            __syncthreads();
            int j = -1;
            if (live && (ti == P.ra[a] || ti == P.rb[a]) && occs[i] < T.cap[ti]) {
                ProposeScan<TPP> scan;
                scan.begin(P, D, a, i, p, ti);
                for (uint32_t q = 0; q < L.m; ++q) {
                    const uint32_t c = L.at(q);
                    scan.consider(P, D, c, Xn[c], occs[c], scan.avoid ? D.mol[c] : 0u);
                }
                j = scan.finish(D);
            }
            unsigned long long key = 0;
            bool open = own && j >= 0;
            if (open) {
                key = match_key(P, a, s, tag);
                atomicMin(&B0[i], key);
                atomicMin(&B0[(uint32_t)j], key);
            }
            uint32_t att = 0, form = 0;
            for (uint32_t r = 0;; ++r) {
                unsigned long long* const Bc = (r & 1u) ? B1 : B0;
                unsigned long long* const Bn = (r & 1u) ? B0 : B1;
                if (tid == 0) more[(r + 1) % 3] = 0u;
                __syncthreads();
                if (open && Bc[i] == key && Bc[(uint32_t)j] == key) {
                    open = false;
                    claimed[i] = 1u;
                    claimed[(uint32_t)j] = 1u;
                    ++att;
                    form += accept_pair<EXT>(P, D, a, s, Xn, i, (uint32_t)j) ? 1u : 0u;
                }
                __syncthreads();
                if (own) Bc[i] = kNoKey;
                if (open) {
                    if (claimed[i] || claimed[(uint32_t)j]) {
                        open = false;
                    } else {
                        atomicMin(&Bn[i], key);
                        atomicMin(&Bn[(uint32_t)j], key);
                        more[r % 3] = 1u;
                    }
                }
                __syncthreads();
                if (!more[r % 3]) break;
            }
            count_add(D, a, kCtrAttempt, att);
            count_add(D, a, kCtrForm, form);
            const uint32_t broke = own ? break_site<EXT>(P, D, a, s, i, Xn) : 0u;
            count_add(D, a, kCtrBreak, broke);
            __syncthreads();
        }
        load_bonds();
    }
    // hand the state back in the form db_step leaves it: positions, velocities,
    // lists, step slots, no list rebuild pending
    const int xin = xin0 ^ (int)(nsteps & 1u);
    if (own) {
        D.x[xin][i] = p;
        D.u[i] = u;
    }
    uint32_t entries = live ? L.m : 0u;
    for (int off = 32; off >= 1; off >>= 1) entries += __shfl_xor(entries, off, 64);
    if (tid == 0) more[0] = 0u;
    __syncthreads();
    if (__lane_id() == 0) atomicAdd(&more[0], entries);
    // lists built during the launch: the pair's one after the other in D.nl.
    // Rows from KL on are the first thread's already, the second's further
    // entries move down from the end (to rows no higher than their own, lowest
    // first).
    const uint32_t m_other = TPP == 2 ? (uint32_t)__shfl_xor((int)L.m, 1, 64) : 0u;
    if (live && built) {
        const uint32_t r0 = sub ? m_other : 0u;
        for (uint32_t q = 0; q < min(L.m, KL); ++q)
            if (r0 + q < P.nlmax) L.far[(size_t)(r0 + q) * n] = L.near_at(q);
        if (TPP == 2 && sub && L.m > KL)
            for (uint32_t e = L.m - KL; e-- > 0u;) {
                const uint32_t r = r0 + L.m - 1u - e;
                if (r < P.nlmax) L.far[(size_t)r * n] = L.far_at(KL + e);
            }
        if (own) {
            D.nl_cnt[i] = min(L.m + m_other, P.nlmax);
            D.xref[i] = xref_pack(P, make_float4(ref.x, ref.y, ref.z, 0.f));
        }
    }
    __syncthreads();
    if (tid == 0) {
        // the flag of step t0, if it was still set, is retired as k_step would
        // (its list build filled cell list rflag[3] and cleared the other)
        if (D.rflag[t0 % 3]) D.rflag[3] ^= 1u;
        D.rflag[0] = D.rflag[1] = D.rflag[2] = 0u;
        D.stepv[0] = D.stepv[1] = t0 + nsteps;
        BatchState e;
        e.t = t0 + nsteps;
        e.cur_x = xin;
        e.cur_list = (int)((unsigned)(st.cur_list + nsteps % 3u) % 3u);
        for (int w = 0; w < 4; ++w) e.err[w] = __hip_atomic_load(&D.err[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        e.listed = more[0];
        *out = e;
    }
}

}  // namespace dyb
