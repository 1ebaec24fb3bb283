// Potentials and gradients of whole systems: groups of ions as the targets of one shared
// traversal.  Included by bhmc_eval.hip inside its per-order namespace.
//
// The ions, in the order of the build's key sort (a space-filling curve), are cut into
// groups of gt <= 16; a workgroup takes a group.  A frontier entry is an opened cell's first
// child with four 16-bit target masks: targets for which the cell is open, targets summing
// every source below it directly (the N_0 rule), targets whose own image, and whose own ion,
// lies inside.  Thread j of a chunk classifies child j mod 8 of entry j / 8.  Each target
// takes exactly the decisions its own traversal would take (Sec. 3.2): a cell that passes or
// fails the MAC for the group's bounding sphere, with a margin far above rounding, does so
// for every target, and only the cells between are tested target by target.
// Far cells go to a list with their target masks, near leaves likewise; the lists are
// evaluated when they fill up and at the end.
//
// What bounds it: the far rows' way through the CU's L1 and the FP64 issue of their
// evaluation, so a row is read once for four targets.  Energy of 10^5 ions + images
// (theta = 0.5, p = 6): 2.88 -> 0.90 ms against groups of four key positions whose targets
// each had frontier entries and lane-per-(cell, target) rows of their own; 199,999 ions at
// p = 8: 13.8 -> 2.0 ms; 10^4 ions (theta = 0.4, p = 5): 0.25 -> 0.14 ms.
constexpr int kGT = 16;
constexpr int kGroupBlock = 256;
constexpr int kStage = 256;     // near sources staged in LDS at a time
// Targets a lane evaluates from one row; 2 instead of 4 measured 1.68 -> 1.88 ms at 10^5 ions,
// theta = 0.3, p = 5 and 2.00 -> 2.13 ms at 199,999 ions, p = 8.
constexpr int kFT = 4, kFTLog = 2;

struct GroupShared {
    static constexpr int FCAP = 512;   // opened cells of a level on chip (4096 children); more continue in HBM
    static constexpr int FARCAP = 768 + kGroupBlock;
    static constexpr int NEARCAP = 256 + kGroupBlock;
    static constexpr int NW = kGroupBlock / 64;
    uint64_t pm[2][FCAP];          // masks: open | direct << 16 | image inside << 32 | ion inside << 48
    int pl[2][FCAP];               // first child
    int farc[FARCAP];
    uint16_t farm[FARCAP];
    uint16_t nearm[NEARCAP];
    int near_base[NEARCAP], near_pre[NEARCAP + 1];
    double4 ns[kStage];            // staged near sources, their indices and target masks
    int nsid[kStage];
    uint16_t nsm[kStage];
    double tx[kGT], ty[kGT], tz[kGT], tq[kGT];
    int ion[kGT];
    uint64_t kimg[kGT], kion[kGT];
    int flag_cell[kGT];
    double ctr[4];                 // the group's bounding sphere
    double red[NW][kGT][2];
    int nt, near_tot, err;
    uint64_t wcnt[2][NW];
    uint64_t wsum[NW + 1];
};

// Targets of a mask for which the cell holds at least k more sources than none: k of its
// count after the targets' own ion (in io) and image (in im) are left out.
__device__ __forceinline__ uint32_t left_mask(int k, uint32_t io, uint32_t im) {
    return k >= 2 ? 0xFFFFu : (k == 1 ? ~(io & im) & 0xFFFFu : (k == 0 ? ~(io | im) & 0xFFFFu : 0u));
}

// Near sources [base, base + cnt) of the flattened near leaves into LDS.
__device__ __forceinline__ void stage_near(const RepU& R, GroupShared& S, int near_n, int base, int cnt) {
    const int f = base + (int)threadIdx.x;
    if ((int)threadIdx.x < cnt) {
        const int j = near_search(S.near_pre, near_n, f);
        const int slot = S.near_base[j] + (f - S.near_pre[j]);
        S.ns[threadIdx.x] = gload(R.pool4 + slot);
        S.nsid[threadIdx.x] = gload(R.pidx + slot);
        S.nsm[threadIdx.x] = S.nearm[j];
    }
}

// Exclusive scan of the near leaves' slot counts in near_pre; returns their total.
__device__ __forceinline__ int group_near_scan(GroupShared& S, int near_n) {
    int carry = 0;
    for (int base = 0; base < near_n; base += kGroupBlock) {
        const int j = base + threadIdx.x;
        const int v = j < near_n ? S.near_pre[j] : 0;
        uint64_t tot;
        const uint64_t ex = block_exscan<kGroupBlock>((uint64_t)v, S.wsum, tot);
        if (j < near_n) S.near_pre[j] = carry + (int)ex;
        carry += (int)tot;
        __syncthreads();
    }
    return carry;
}

// The lists' far part for energies: a lane reads a row once for kFT of the group's targets,
// so a cell takes gt / kFT lanes.  far: this lane's sums of its targets.
template <bool F32>
__device__ __forceinline__ void energy_far(const RepU& R, GroupShared& S, int far_n, int lq, double (&far)[kFT]) {
    const int q = (int)threadIdx.x & ((1 << lq) - 1);
    double tx[kFT], ty[kFT], tz[kFT];
#pragma unroll
    for (int u = 0; u < kFT; ++u) { tx[u] = S.tx[kFT * q + u]; ty[u] = S.ty[kFT * q + u]; tz[u] = S.tz[kFT * q + u]; }
    for (int j = (int)threadIdx.x >> lq; j < far_n; j += kGroupBlock >> lq) {
        const uint32_t m = ((uint32_t)S.farm[j] >> (kFT * q)) & ((1u << kFT) - 1u);
        if (!m) continue;
        const int c = S.farc[j];
        if (F32 && R.M32) {
            const double4 g = gload(R.cgeo + c);
#pragma unroll
            for (int u = 0; u < kFT; ++u) {
                if ((m >> u) & 1u) far[u] += far_eval_f(g.x - tx[u], g.y - ty[u], g.z - tz[u], R.M32 + (size_t)c * MSTR);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            double v[kFT];
            far_rows<kFT>(grow(R.H + (size_t)c * HSTR), tx, ty, tz, v);
#pragma unroll
            for (int u = 0; u < kFT; ++u) far[u] += ((m >> u) & 1u) ? v[u] : 0.0;
        }
    }
}

// The near part: the leaves' sources staged in LDS 256 at a time; thread (row, k) takes every
// (256 / gt)-th of them for target k.
__device__ __forceinline__ void energy_near(const RepU& R, GroupShared& S, int near_n, int lg, double& near) {
    const int total = group_near_scan(S, near_n);
    const int k = (int)threadIdx.x & ((1 << lg) - 1), rows = kGroupBlock >> lg;
    const double x = S.tx[k], y = S.ty[k], z = S.tz[k];
    const int ion = S.ion[k], img = R.images ? R.n + ion : -1;
    for (int base = 0; base < total; base += kStage) {
        const int cnt = min(kStage, total - base);
        stage_near(R, S, near_n, base, cnt);
        __syncthreads();
        for (int s = (int)threadIdx.x >> lg; s < cnt; s += rows) {
            const double4 p = S.ns[s];
            const int sid = S.nsid[s];
            const double dx = x - p.x, dy = y - p.y, dz = z - p.z;
            const double d2 = dx * dx + dy * dy + dz * dz;
            if (((S.nsm[s] >> k) & 1u) && sid != ion && sid != img && d2 != 0.0) near += p.w * rsqrt_nr(d2);
        }
        __syncthreads();
    }
}

// The group's traversal.  run_lists(far_n, near_n): evaluates the lists (called by every
// thread, with barriers around it).  flag_far: keep the (cell, target) pairs of far cells that
// hold the target's own image out of the far list (their cell is in flag_cell either way).
template <class Lists>
__device__ __forceinline__ void group_traverse(const RepU& R, GroupShared& S, bool flag_apart, Lists&& run_lists) {
    using GS = GroupShared;
    constexpr int NW = GS::NW;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const bool imgs = R.images != 0;
    // levels past the LDS capacity go to this workgroup's HBM region: first children, then masks
    uint32_t* const gfr = spill_region(R);
    const int gcap = gfr ? (int)((R.spill_words - 2) / 6 < 0x7FFFFFFF ? (R.spill_words - 2) / 6 : 0x7FFFFFFF) : 0;
    int* const gpl = (int*)gfr;
    uint64_t* const gpm = gfr ? (uint64_t*)(gfr + 2 * (size_t)gcap) : nullptr;
    const int lcap = R.fcap / 8 < GS::FCAP ? R.fcap / 8 : GS::FCAP;
    const uint32_t all = (1u << S.nt) - 1u;
    const double bx = S.ctr[0], by = S.ctr[1], bz = S.ctr[2], br = S.ctr[3];
    // a cell of half side h passes the MAC beyond sqrt(3) h / theta of its centre
    const double rmac = R.theta2 > 0.0 ? sqrt(3.0 / R.theta2) : __builtin_huge_val();
    int cur = 0, np = 1, far_n = 0, near_n = 0, buf = 0;
    bool failed = false, frontier_full = false, rg = false, wg = false;
    for (int level = 0; np > 0 && !failed; ++level) {
        int next = 0;
        const int fs = level == 0 ? 1 : 8 * np;
        for (int base = 0; base < fs; base += kGroupBlock) {
            if (far_n > GS::FARCAP - kGroupBlock || near_n > GS::NEARCAP - kGroupBlock) {
                __syncthreads();
                run_lists(far_n, near_n);
                far_n = 0; near_n = 0;
                __syncthreads();
            }
            const int j = base + tid;
            const bool valid = j < fs;
            int c = 0, digit = -1;
            uint64_t pm = 0;
            uint32_t im = 0, io = 0;
            if (level == 0) {
                if (valid) { pm = (uint64_t)all | (imgs ? (uint64_t)all << 32 : 0ull) | ((uint64_t)all << 48); }
                im = (uint32_t)(pm >> 32) & 0xFFFFu; io = (uint32_t)(pm >> 48);
            } else if (valid) {
                const int e = j >> 3;
                digit = j & 7;
                c = (rg ? gpl[(size_t)cur * gcap + e] : S.pl[cur][e]) + digit;
                pm = rg ? gpm[(size_t)cur * gcap + e] : S.pm[cur][e];
                // the targets whose own image and ion lie in this child
                for (uint32_t rest = (uint32_t)(pm >> 32) & 0xFFFFu; rest; rest &= rest - 1u) {
                    const int t = __builtin_ctz(rest);
                    if (key_digit(S.kimg[t], level) == digit) im |= 1u << t;
                }
                for (uint32_t rest = (uint32_t)(pm >> 48); rest; rest &= rest - 1u) {
                    const int t = __builtin_ctz(rest);
                    if (key_digit(S.kion[t], level) == digit) io |= 1u << t;
                }
            }
            uint32_t farb = 0, nearb = 0, copen = 0, cdir = 0;
            int4 m = make_int4(0, -1, 0, 0);
            if (valid && (c < 0 || c >= R.ncell)) {
                S.err = kErrFrontCell;
            } else if (valid) {
                m = gload(R.cm + c);
                const double4 g = gload(R.cgeo + c);
                if (m.y >= 0 && m.y + 8 > R.ncell) {
                    S.err = kErrChildLink;
                } else if (m.x > 0) {
                    const uint32_t left = left_mask(m.x - 1, io, im);
                    const uint32_t open = (uint32_t)(pm & 0xFFFFu) & left, dir = (uint32_t)((pm >> 16) & 0xFFFFu) & left;
                    uint32_t mac = 0;
                    if (open) {
                        const double dx = g.x - bx, dy = g.y - by, dz = g.z - bz;
                        const double d2 = dx * dx + dy * dy + dz * dz, rm = rmac * g.w;
                        const double hi = rm * (1.0 + 1e-9) + br, lo = rm * (1.0 - 1e-9) - br;
                        if (d2 > hi * hi) mac = 0xFFFFu;
                        else if (!(lo > 0.0 && d2 < lo * lo))
                            for (uint32_t rest = open; rest; rest &= rest - 1u) {
                                const int t = __builtin_ctz(rest);
                                const double tx = g.x - S.tx[t], ty = g.y - S.ty[t], tz = g.z - S.tz[t];
                                const double t2 = tx * tx + ty * ty + tz * tz;
                                if (3.0 * (g.w * g.w) <= R.theta2 * t2) mac |= 1u << t;
                            }
                    }
                    const bool internal = m.y >= 0;
                    farb = open & mac & left_mask(m.x - R.n0, io, im);
                    const uint32_t rest = open & ~farb;
                    copen = internal ? rest & left_mask(m.x - R.n0 - 1, io, im) : 0u;
                    nearb = internal ? 0u : rest | dir;
                    cdir = internal ? (rest & ~copen) | dir : 0u;
                    if (farb & im) {
                        for (uint32_t fl = farb & im; fl; fl &= fl - 1u) S.flag_cell[__builtin_ctz(fl)] = c;
                        if (flag_apart) farb &= ~im;
                    }
                }
            }
            const bool kf = farb != 0, kn = nearb != 0, ks = (copen | cdir) != 0;
            const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
            const uint64_t bf = __ballot(kf), bn = __ballot(kn), bs = __ballot(ks);
            if (lane == 0)
                S.wcnt[buf][w] = (uint64_t)__popcll(bf) | ((uint64_t)__popcll(bn) << 16) | ((uint64_t)__popcll(bs) << 32);
            __syncthreads();
            uint64_t before = 0, tot = 0;
#pragma unroll
            for (int ww = 0; ww < NW; ++ww) {
                const uint64_t v = S.wcnt[buf][ww];
                before += ww < w ? v : 0ull;
                tot += v;
            }
            buf ^= 1;
            const int tf = (int)(tot & 0xffff), tn = (int)((tot >> 16) & 0xffff), ts = (int)(tot >> 32);
            if (next + ts > (wg ? gcap : lcap)) {  // uniform
                if (wg || next + ts > gcap) {
                    failed = frontier_full = true;
                    break;
                }
                // the next level moves to HBM: what this level wrote so far first
                for (int k = tid; k < next; k += kGroupBlock) {
                    gpl[(size_t)(cur ^ 1) * gcap + k] = S.pl[cur ^ 1][k];
                    gpm[(size_t)(cur ^ 1) * gcap + k] = S.pm[cur ^ 1][k];
                }
                wg = true;
            }
            if (kf) {
                const int o = far_n + (int)(before & 0xffff) + __popcll(bf & lt);
                S.farc[o] = c;
                S.farm[o] = (uint16_t)farb;
            }
            if (kn) {
                const int o = near_n + (int)((before >> 16) & 0xffff) + __popcll(bn & lt);
                S.nearm[o] = (uint16_t)nearb;
                S.near_base[o] = m.z;
                S.near_pre[o] = m.x;
                if (m.z < 0 || m.z + m.x > R.pool) { S.near_pre[o] = 0; S.err = kErrNearSlots; }
            }
            if (ks) {
                const int o = next + (int)(before >> 32) + __popcll(bs & lt);
                const uint32_t live = copen | cdir;
                const uint64_t mk = (uint64_t)copen | ((uint64_t)cdir << 16) | ((uint64_t)(im & live) << 32) |
                                    ((uint64_t)(io & live) << 48);
                if (wg) {
                    gpl[(size_t)(cur ^ 1) * gcap + o] = m.y;
                    gpm[(size_t)(cur ^ 1) * gcap + o] = mk;
                } else {
                    S.pl[cur ^ 1][o] = m.y;
                    S.pm[cur ^ 1][o] = mk;
                }
            }
            far_n += tf; near_n += tn; next += ts;
        }
        __syncthreads();  // the next level reads what this one wrote
        cur ^= 1;
        np = next;
        rg = wg;
    }
    if (failed && tid == 0) S.err = frontier_full ? kErrFrontier : kErrStack;
    __syncthreads();
    if (!failed) run_lists(far_n, near_n);
    __syncthreads();
}

// Targets of group grp (ions order[grp gt] ..), their bounding sphere, and empty results.
__device__ __forceinline__ void group_targets(const RepU& R, GroupShared& S, const int* order, int grp, int gt) {
    const int tid = threadIdx.x, g0 = grp * gt, nt = min(gt, R.n - g0);
    if (tid == 0) { S.nt = nt; S.err = 0; }
    if (tid < kGT) {
        // threads past the group's end repeat its last ion (their targets are in no mask)
        const int ion = order[g0 + min(tid, nt - 1)];
        const bool ok = (unsigned)ion < (unsigned)R.n;
        const double4 p = ok ? gload(R.src + ion) : make_double4(0, 0, 0, 0);
        const double4 k = ok && R.images ? gload(R.src + R.n + ion) : make_double4(0, 0, 0, 0);
        S.ion[tid] = ok ? ion : 0;
        S.tx[tid] = p.x; S.ty[tid] = p.y; S.tz[tid] = p.z; S.tq[tid] = p.w;
        S.kion[tid] = morton_key(R, p.x, p.y, p.z);
        S.kimg[tid] = R.images ? morton_key(R, k.x, k.y, k.z) : 0;
        S.flag_cell[tid] = -1;
        double lx = p.x, hx = p.x, ly = p.y, hy = p.y, lz = p.z, hz = p.z;
#pragma unroll
        for (int off = 1; off < kGT; off <<= 1) {
            lx = fmin(lx, __shfl_xor(lx, off, kGT)); hx = fmax(hx, __shfl_xor(hx, off, kGT));
            ly = fmin(ly, __shfl_xor(ly, off, kGT)); hy = fmax(hy, __shfl_xor(hy, off, kGT));
            lz = fmin(lz, __shfl_xor(lz, off, kGT)); hz = fmax(hz, __shfl_xor(hz, off, kGT));
        }
        if (tid == 0) {
            const double ex = 0.5 * (hx - lx), ey = 0.5 * (hy - ly), ez = 0.5 * (hz - lz);
            S.ctr[0] = 0.5 * (lx + hx); S.ctr[1] = 0.5 * (ly + hy); S.ctr[2] = 0.5 * (lz + hz);
            S.ctr[3] = sqrt(ex * ex + ey * ey + ez * ez) * (1.0 + 1e-9);
        }
        if (!ok) S.err = kErrBuildPerm;
    }
    __syncthreads();
}

// Term of ion i in E / l_B given its potential.
__device__ __forceinline__ double ion_term(const RepU& R, double x, double y, double z, double q, double ph) {
    double e = 0.5 * q * ph;
    if (R.geom == 1) {
        const double r2 = x * x + y * y + z * z;
        if (R.images) e += 0.5 * R.gamma * R.a * q * q / (r2 - R.a2);
        if (R.Qc != 0.0) e += R.Qc * q / sqrt(r2);
    }
    return e;
}

// Potential at every ion, with the ion and its image excluded, and each ion's term of
//   E / l_B = 1/2 q phi + 1/2 gamma a q^2 / (r^2 - a^2) + Q q / r.
// The ion itself is never in a far cell of its own traversal (theta < 1); its image may be,
// and is then taken back out through that cell's expansion (flagged_value where the far
// cells are taken in single precision).
template <bool F32>
__global__ void __launch_bounds__(kGroupBlock) __attribute__((amdgpu_waves_per_eu(2))) k_energy(Rep* reps, int r, int lg, double* phi, double* eterm) {
    __shared__ GroupShared S;
    __shared__ Rep Rs;
    load_rep(Rs, reps + r);
    __syncthreads();
    const RepU R(Rs);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int gt = 1 << lg, lq = lg - kFTLog;
    const bool apart = F32 && R.M32;
    const int ngroups = (R.n + gt - 1) / gt;
    // one group per workgroup, or several when the grid is bounded (HBM frontier regions)
    for (int grp = blockIdx.x; grp < ngroups; grp += gridDim.x) {
        group_targets(R, S, Rs.iord, grp, gt);
        double far[kFT] = {}, near = 0.0;
        group_traverse(R, S, apart, [&](int far_n, int near_n) {
            energy_far<F32>(R, S, far_n, lq, far);
            energy_near(R, S, near_n, lg, near);
        });
        // the lanes of a wave that share targets, then the waves
        for (int off = 1 << lq; off < 64; off <<= 1)
#pragma unroll
            for (int u = 0; u < kFT; ++u) far[u] += __shfl_xor(far[u], off, 64);
        for (int off = gt; off < 64; off <<= 1) near += __shfl_xor(near, off, 64);
        if (lane < (1 << lq))
#pragma unroll
            for (int u = 0; u < kFT; ++u) S.red[w][kFT * lane + u][0] = far[u];
        if (lane < gt) S.red[w][lane][1] = near;
        __syncthreads();
        if (tid < S.nt) {
            const int ion = S.ion[tid];
            const double x = S.tx[tid], y = S.ty[tid], z = S.tz[tid];
            double ph = 0.0;
            for (int ww = 0; ww < GroupShared::NW; ++ww) ph += S.red[ww][tid][0];
            for (int ww = 0; ww < GroupShared::NW; ++ww) ph += S.red[ww][tid][1];
            const int c = S.flag_cell[tid];
            if (c >= 0) {
                const double4 k = gload(R.src + R.n + ion);
                if (apart) {
                    ph += flagged_value<F32>(R, c, x, y, z, false, k, true, k);
                } else {
                    const double4 g = gload(R.cgeo + c);
                    ph -= k.w * point_expansion(g.x - x, g.y - y, g.z - z, k.x - g.x, k.y - g.y, k.z - g.z);
                }
            }
            if (S.err) {
                ph = __builtin_nan("");
                if (tid == 0) reps[r].err_detail = S.err;
            }
            if (phi) phi[ion] = ph;
            eterm[ion] = ion_term(R, x, y, z, S.tq[tid], ph);
        }
        __syncthreads();  // the next group reuses the traversal state
    }
}
