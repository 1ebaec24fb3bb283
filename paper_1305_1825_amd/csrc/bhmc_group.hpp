// Potentials and gradients of whole systems: groups of ions as the targets of one shared
// traversal.  Included by bhmc_eval.hip inside its per-order namespace.
//
// The ions, in the order of the build's key sort (a space-filling curve), are cut into
// groups of gt <= 16; a workgroup takes a group.  A frontier entry is an opened cell's first
// child with four 16-bit target masks: targets for which the cell is open, targets summing
// every source below it directly (the N_0 rule), targets whose own image, and whose own ion,
// lies inside.  Thread j of a chunk classifies child j mod 8 of entry j / 8.  Each target
// takes exactly the decisions its own traversal would take (Sec. 3.2): a cell that passes or
// fails the MAC for the group's bounding sphere, widened by more than the rounding of the
// sphere and of the test, does so for every target, and only the cells between are tested
// target by target.
// Far cells go to a list with their target masks, near leaves likewise; the lists are
// evaluated when they fill up and at the end.
//
// What bounds it: latencies at two waves a SIMD, by the counters of 10^5 ions + images (theta =
// 0.5, p = 6): waves wait 56 % of their cycles, vector instructions (69 % of them FP64 arithmetic)
// issue in 47 % of the time, LDS bank conflicts cost 2 % of its accesses.  A row read once for four
// targets has more arithmetic between its loads: that system 2.88 -> 0.90 ms against groups of four key
// positions whose targets each had frontier entries and lane-per-(cell, target) rows of their own
// (0.81 with the level loop's later changes); 199,999 ions at p = 8: 13.8 -> 2.0 ms; 10^4 ions
// (theta = 0.4, p = 5): 0.25 -> 0.13 ms.
constexpr int kGT = 16;
constexpr int kGroupBlock = 256;
constexpr int kStage = 256;     // near sources staged in LDS at a time
// Targets a lane evaluates from one row; 2 instead of 4 measured 1.68 -> 1.88 ms at 10^5 ions,
// theta = 0.3, p = 5 and 2.00 -> 2.13 ms at 199,999 ions, p = 8.
constexpr int kFT = 4, kFTLog = 2;

constexpr int kND = (NH + 3) / 4;
// row stride in LDS: 2 mod 4 doubles puts the 16 rows' words k in distinct quads of banks
constexpr int kLst = ((NH + 3 + 1) / 4) * 4 + 2;
static_assert(kLst >= NH + 3 && kLst >= HSTR, "a staged row holds the expansion row");

template <bool GRAD>
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
    union {
        struct {
            double4 ns[kStage];            // staged near sources, their indices and target masks
            int nsid[kStage];
            uint16_t nsm[kStage];
        };
        double rows[GRAD ? NW * 16 * kLst : 1];  // gradient: 16 expansion rows a wave
    };
    double tx[kGT], ty[kGT], tz[kGT], tq[kGT];
    int ion[kGT];
    uint64_t kimg[kGT], kion[kGT];
    int flag_cell[kGT];
    double ctr[4];                 // the group's bounding sphere
    double red[NW][kGT][2];
    int nt, err;
    uint64_t wcnt[2][NW];
    uint64_t wsum[NW + 1];
};

// Targets of a mask for which the cell holds at least k more sources than none: k of its
// count after the targets' own ion (in io) and image (in im) are left out.
__device__ __forceinline__ uint32_t left_mask(int k, uint32_t io, uint32_t im) {
    return k >= 2 ? 0xFFFFu : (k == 1 ? ~(io & im) & 0xFFFFu : (k == 0 ? ~(io | im) & 0xFFFFu : 0u));
}

// Near sources [base, base + cnt) of the flattened near leaves into LDS.
template <class GS>
__device__ __forceinline__ void stage_near(const RepU& R, GS& S, int near_n, int base, int cnt) {
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
template <class GS>
__device__ __forceinline__ int group_near_scan(GS& S, int near_n) {
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
// so a cell takes gt / kFT lanes.  far: this lane's sums of its targets.  In single precision
// (apart) the targets of a row are evaluated one after the other, so there a cell takes gt
// lanes, one a target, and far[0] is the lane's sum: small systems' few far cells otherwise
// left lanes idle (300 ions, p = 8: 38.9 us with four targets a lane, 31.1 with one a workgroup).
template <bool F32>
__device__ __forceinline__ void energy_far(const RepU& R, GroupShared<false>& S, int far_n, int lq, double (&far)[kFT]) {
    if constexpr (F32) {  // a far_fp32 replica: M32 is there
        const int lg = lq + kFTLog, k = (int)threadIdx.x & ((1 << lg) - 1);
        const double x = S.tx[k], y = S.ty[k], z = S.tz[k];
        for (int j = (int)threadIdx.x >> lg; j < far_n; j += kGroupBlock >> lg) {
            if (!((S.farm[j] >> k) & 1u)) continue;
            const int c = S.farc[j];
            const double4 g = gload(R.cgeo + c);
            far[0] += far_eval_f(g.x - x, g.y - y, g.z - z, R.M32 + (size_t)c * MSTR);
        }
        return;
    }
    const int q = (int)threadIdx.x & ((1 << lq) - 1);
    double tx[kFT], ty[kFT], tz[kFT];
#pragma unroll
    for (int u = 0; u < kFT; ++u) { tx[u] = S.tx[kFT * q + u]; ty[u] = S.ty[kFT * q + u]; tz[u] = S.tz[kFT * q + u]; }
    for (int j = (int)threadIdx.x >> lq; j < far_n; j += kGroupBlock >> lq) {
        const uint32_t m = ((uint32_t)S.farm[j] >> (kFT * q)) & ((1u << kFT) - 1u);
        if (!m) continue;
        const int c = S.farc[j];
        double v[kFT];
        far_rows<kFT>(grow(R.H + (size_t)c * HSTR), tx, ty, tz, v);
#pragma unroll
        for (int u = 0; u < kFT; ++u) far[u] += ((m >> u) & 1u) ? v[u] : 0.0;
    }
}

// The near part: the leaves' sources staged in LDS 256 at a time; thread (row, k) takes every
// (256 / gt)-th of them for target k.
__device__ __forceinline__ void energy_near(const RepU& R, GroupShared<false>& S, int near_n, int lg, double& near) {
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
template <class GS, class Lists>
__device__ __forceinline__ void group_traverse(const RepU& R, GS& S, bool flag_apart, Lists&& run_lists) {
    constexpr int NW = GS::NW;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const bool imgs = R.images != 0;
    // levels past the LDS capacity go to this workgroup's HBM region: first children, then masks
    const long long gw = uni(R.d.gspill_words);
    uint32_t* const gfr = spill_region(R.spill, uni(R.d.gspill_regions), gw);
    const int gcap = gfr ? (int)((gw - 2) / 6 < 0x7FFFFFFF ? (gw - 2) / 6 : 0x7FFFFFFF) : 0;
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
            const uint64_t bf = __ballot(kf), bn = __ballot(kn), bs = __ballot(ks);
            if (lane == 0)
                S.wcnt[buf][w] = (uint64_t)__popcll(bf) | ((uint64_t)__popcll(bn) << 16) | ((uint64_t)__popcll(bs) << 32);
            __syncthreads();
            const ChunkScan<NW> scan(S.wcnt[buf]);
            const uint64_t before = scan.before(uni(w)), tot = scan.before(NW);
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
                const int o = rank_below(bf, far_n + (int)(before & 0xffff));
                S.farc[o] = c;
                S.farm[o] = (uint16_t)farb;
            }
            if (kn) {
                const int o = rank_below(bn, near_n + (int)((before >> 16) & 0xffff));
                S.nearm[o] = (uint16_t)nearb;
                S.near_base[o] = m.z;
                S.near_pre[o] = m.x;
                if (m.z < 0 || m.z + m.x > R.pool) { S.near_pre[o] = 0; S.err = kErrNearSlots; }
            }
            if (ks) {
                const int o = rank_below(bs, next + (int)(before >> 32));
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
template <class GS>
__device__ __forceinline__ void group_targets(const RepU& R, GS& S, const int* order, int grp, int gt) {
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
            // the midpoints round in the coordinates' own last place, which far from the origin is
            // large against a deep cell: at most 2^-53 of the coordinate an axis
            const double m = fmax(fabs(lx), fabs(hx)) + fmax(fabs(ly), fabs(hy)) + fmax(fabs(lz), fabs(hz));
            S.ctr[3] = sqrt(ex * ex + ey * ey + ez * ez) * (1.0 + 1e-9) + 0x1p-52 * m;
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
// and is then taken back out through that cell's expansion (with that cell's value in FP64 from
// the moments where the far cells are taken in single precision).
//
// Workgroups a CU that the registers leave room for, a wave of each to a SIMD: in single precision 4
// up to order 4 (127 registers) and 3 at order 5 (146), in FP64 4 at order 0, 3 at 1 and 2 (158), 2
// from order 4 on (190).  Small systems are bound by latencies, which they share.  At orders 3 and 4
// the FP64 form is there twice, W = 2 and held to W = 3 waves a SIMD (172 registers cut to 168, 190 to
// 168 with 17 spilled): at order 3 from 2,049 ions on, at order 4 from 4,097, where groups of 8 no
// longer all run two to a CU (p = 4, theta = 0.8, leaf 16: 6,000 ions 61 -> 48 us; 2,000 ions 35 ->
// 38).  (Holding orders 2 and 3 of the single-precision form to 4 waves cost up to 8 %.)
constexpr int energy_groups_per_cu(bool f32) {
    return f32 ? (P > 5 ? 2 : (P > 4 ? 3 : 4)) : (P > 3 ? 2 : (P > 0 ? 3 : 4));
}
constexpr bool kEnergyTwice = P == 3 || P == 4;
constexpr int kEnergyW3Min = P == 3 ? 2049 : 4097;
template <bool F32, int W = 2>
__global__ void __launch_bounds__(kGroupBlock) __attribute__((amdgpu_waves_per_eu(W))) k_energy(Rep* reps, int r, int lg, double* phi, double* eterm) {
    __shared__ GroupShared<false> S;
    __shared__ Rep Rs;
    load_rep(Rs, reps + r);
    __syncthreads();
    const RepU R(Rs);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int gt = 1 << lg, lq = lg - kFTLog;
    constexpr bool apart = F32;
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
        for (int off = apart ? gt : 1 << lq; off < 64; off <<= 1)
#pragma unroll
            for (int u = 0; u < kFT; ++u) far[u] += __shfl_xor(far[u], off, 64);
        for (int off = gt; off < 64; off <<= 1) near += __shfl_xor(near, off, 64);
        if (apart) {
            if (lane < gt) S.red[w][lane][0] = far[0];
        } else if (lane < (1 << lq))
#pragma unroll
            for (int u = 0; u < kFT; ++u) S.red[w][kFT * lane + u][0] = far[u];
        if (lane < gt) S.red[w][lane][1] = near;
        __syncthreads();
        if (tid < S.nt) {
            const int ion = S.ion[tid];
            const double x = S.tx[tid], y = S.ty[tid], z = S.tz[tid];
            double ph = 0.0;
            for (int ww = 0; ww < GroupShared<true>::NW; ++ww) ph += S.red[ww][tid][0];
            for (int ww = 0; ww < GroupShared<true>::NW; ++ww) ph += S.red[ww][tid][1];
            const int c = S.flag_cell[tid];
            if (c >= 0) {
                const double4 k = gload(R.src + R.n + ion);
                const double4 g = gload(R.cgeo + c);
                // (inline: as a call it set the kernel's registers, 214 for 127 at order 4; from order 6 on
                // two workgroups a CU fit either way)
                if (apart) ph += cart_eval<(P <= 5)>(g.x - x, g.y - y, g.z - z, grow(R.M + (size_t)c * MSTR));
                ph -= k.w * point_expansion(g.x - x, g.y - y, g.z - z, k.x - g.x, k.y - g.y, k.z - g.z);
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

// ------------------------------------------------------------ gradient
// Step 1, over the same groups (16 ions): each target's potential and its gradient, and the
// source side of every pair term: the adjoint coefficients L_lm = sum_t w_t J_lm(x_t - c) of
// each far cell, w_t = 1/2 l_B q_t, J_lm = A_lm(X) / |X|^(2l+1), and the near pairs' terms in G.
// Per target:  dE/dx_t += 1/2 l_B q_t grad phi_t,  dE/dq_t += 1/2 l_B phi_t.
//
// A wave takes 16 far cells at a time, lane (c, k) = (lane mod 16, lane / 16) cell c and the
// targets k, 4 + k, 8 + k, 12 + k one after the other, the cells' rows staged in LDS by
// coalesced loads.  The sum over targets is a contraction, taken by the matrix cores: with
// A = w_t J_lm in lane (c, k) and B one-hot in its column, a 4x4x4 FP64 MFMA adds the sum
// over the four lanes k into column j of D for all 16 cells, so four terms share a D register
// and the (p + 1)^2 terms of 16 cells and 16 targets end in (p + 1)^2 / 4 of them; they go
// through LDS to one atomic per cell and term, consecutive lanes on consecutive words.
// (Summing 16 terms at a time across 16-lane rows by DPP exchanges took 105 instructions per
// 16 terms, as much as the evaluation.)  Gradient of 10^5 ions + images (theta = 0.5, p = 6)
// 9.46 -> 2.39 ms against the Cartesian form with 84 adjoint terms a cell, 199,999 ions at p = 8
// 56.4 -> 6.95 ms, 10^4 ions (theta = 0.4, p = 5) 1.05 -> 0.40 ms.  By the counters (p = 6 / 8)
// vector instructions issue in 52 / 50 % of the time and the matrix cores are busy in 14 / 15 %, waves
// wait 42 / 43 % of their cycles at two a SIMD, and bank conflicts add 43 / 46 % to the LDS's cycles.
struct GradTerms { double phi, gx, gy, gz; };
// phi and grad phi at X of a row: with the sums S = sum (.) zeta^m, E = sum (l + 1) (.) zeta^m over
// the terms H_lm a_lm and U = dS/du (da_lm/du = (l - m) a_{l,m+1}, from the Gegenbauer form of a_lm),
//   phi = S / |X|,  grad phi = w / |X| [ (Re S_zeta, -Im S_zeta, U) - X (E + u U + Re(zeta S_zeta)) ]
// (each term is homogeneous of degree l in the scale of 1 / X).  wt J_lm joins D.
// The columns go upwards, m = 0 .. p, each a_lm used as it comes: by the sums of its own column
// and, as da_{l,m-1}/du, by U through the coefficients of the column below.  Neither the a_lm of
// a column nor the powers of zeta are kept, so at order 8 only 29 of 256 registers spill (112 B a
// lane; downwards with Horner's rule so many that 199,999 ions took 14.9 ms for 7.1).
// The column below in registers; above order 6 its words are read again, for registers
// (10^5 ions, p = 6: 2.49 ms kept, 2.64 read again).
constexpr bool kKeepColumn = P <= 6;
struct GradSums { double S, E, U, d0, d1, zr, zi, pr, pi; };

template <int M, class HP>
__device__ __forceinline__ void grad_columns(HP h, double u, double w, double zx, double zy, double wt,
                                             const double (&hot)[4], double (&D)[kND], GradSums& g,
                                             double (&below)[2 * (P + 1)]) {
    if constexpr (M <= P) {
        double own[2 * (P + 1)];
        constexpr int st = M ? 2 : 1, stb = M > 1 ? 2 : 1;
        double qc = 0.0, qs = 0.0, ec = 0.0, es = 0.0, uc = 0.0, us = 0.0;
        double a0 = 0.0, a1 = 1.0;
        const double wr = wt * g.zr, wi = wt * g.zi;
#pragma unroll
        for (int l = M; l <= P; ++l) {
            if (l == M + 1) { a0 = 1.0; a1 = u; }
            if (l > M + 1) {
                const double a2 = fma(u, a1, -(hbeta(l, M) * w) * a0);
                a0 = a1; a1 = a2;
            }
            const int pl = hplace(M, M) + st * (l - M);
            const double hc = h[pl], e = (double)(l + 1) * a1;
            own[2 * l] = hc;
            qc = fma(hc, a1, qc); ec = fma(hc, e, ec);
            if (M) {
                const double hs = h[pl + 1];
                own[2 * l + 1] = hs;
                qs = fma(hs, a1, qs); es = fma(hs, e, es);
                // the column below, whose derivative in u this is
                const int pb = hplace(M - 1, M - 1) + stb * (l - M + 1);
                const double v = (double)(l - M + 1) * a1;
                uc = fma(kKeepColumn ? below[2 * l] : h[pb], v, uc);
                if (M > 1) us = fma(kKeepColumn ? below[2 * l + 1] : h[pb + 1], v, us);
            }
            // (a scheduling boundary every four terms: the compiler otherwise forms a whole column's
            // products ahead of the sums, at 80 more registers)
            if ((l - M) % 4 == 3) __builtin_amdgcn_sched_barrier(0);
            D[pl >> 2] = __builtin_amdgcn_mfma_f64_4x4x4f64(a1 * wr, hot[pl & 3], D[pl >> 2], 0, 0, 0);
            if (M) D[(pl + 1) >> 2] = __builtin_amdgcn_mfma_f64_4x4x4f64(a1 * wi, hot[(pl + 1) & 3], D[(pl + 1) >> 2], 0, 0, 0);
        }
        if (M == 0) {
            g.S = qc; g.E = ec;
        } else {
            g.S = fma(qc, g.zr, fma(qs, g.zi, g.S));
            g.E = fma(ec, g.zr, fma(es, g.zi, g.E));
            g.U = fma(uc, g.pr, fma(us, g.pi, g.U));
            g.d0 = fma((double)M * qc, g.pr, fma((double)M * qs, g.pi, g.d0));
            g.d1 = fma((double)M * qs, g.pr, fma(-((double)M * qc), g.pi, g.d1));
        }
        g.pr = g.zr; g.pi = g.zi;
        g.zr = fma(g.pr, zx, -(g.pi * zy));
        g.zi = fma(g.pr, zy, g.pi * zx);
        __builtin_amdgcn_sched_barrier(0);
        grad_columns<M + 1>(h, u, w, zx, zy, wt, hot, D, g, own);
    }
}

template <class HP>
__device__ __forceinline__ GradTerms grad_pair(HP h, double x, double y, double z, double wt, const double (&hot)[4],
                                               double (&D)[kND]) {
    const double ir = rsqrt_nr(x * x + y * y + z * z);
    const double w = ir * ir, u = z * w, zx = x * w, zy = y * w;
    GradSums s{0.0, 0.0, 0.0, 0.0, 0.0, 1.0, 0.0, 0.0, 0.0};
    double none[2 * (P + 1)];
    grad_columns<0>(h, u, w, zx, zy, wt * ir, hot, D, s, none);
    GradTerms g;
    g.phi = ir * s.S;
    const double k = ir * w, rad = s.E + u * s.U + (zx * s.d0 + zy * s.d1);
    g.gx = k * (s.d0 - x * rad);
    g.gy = k * (s.d1 - y * rad);
    g.gz = k * (s.U - z * rad);
    return g;
}

// LDS written by some lanes of a wave and read by others: the hardware keeps a wave's LDS
// accesses in order, this keeps the compiler to it.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// acc[4 pass + k']: this lane's sums for target 4 pass + lane / 16: phi, -grad phi.
__device__ __forceinline__ void grad_far(const RepU& R, GroupShared<true>& S, double* rows, int far_n, double half_lB,
                                         double* L, double (&acc)[16]) {
    const int lane = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6;
    const int c16 = lane & 15, k = lane >> 4;
    double hot[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) hot[j] = (lane & 3) == j ? 1.0 : 0.0;
    for (int b0 = 16 * w; b0 < far_n; b0 += 16 * GroupShared<true>::NW) {  // uniform in a wave
        const int nb = min(16, far_n - b0);
        for (int it = lane; it < nb * (HSTR / 2); it += 64) {
            const int f = it / (HSTR / 2), d = it - f * (HSTR / 2);
            const GRow src = grow(R.H + (size_t)S.farc[b0 + f] * HSTR + 2 * d);
            rows[f * kLst + 2 * d] = src[0];
            rows[f * kLst + 2 * d + 1] = src[1];
        }
        wave_lds_sync();
        const int row = min(c16, nb - 1) * kLst;
        const uint32_t mask = c16 < nb ? S.farm[b0 + c16] : 0u;
        double D[kND];
#pragma unroll
        for (int j = 0; j < kND; ++j) D[j] = 0.0;
#pragma unroll 1
        for (int pass = 0; pass < 4; ++pass) {
            const int t = 4 * pass + k;
            const bool act = (mask >> t) & 1u;
            if (__ballot(act) == 0) continue;  // uniform
            // the row's place as new in every pass, or its words would be held across all four
            int at = row;
            asm volatile("" : "+v"(at));
            const LRow h = lrow(rows) + at;
            const double cx = h[HCEN], cy = h[HCEN + 1], cz = h[HCEN + 2];
            // a lane whose target does not take the cell as far stands at a harmless place with weight zero
            const double x = act ? S.tx[t] - cx : 1.0, y = act ? S.ty[t] - cy : 0.0, z = act ? S.tz[t] - cz : 0.0;
            const GradTerms g = grad_pair(h, x, y, z, act ? half_lB * S.tq[t] : 0.0, hot, D);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const double on = act && q == pass ? 1.0 : 0.0;  // weights, not branches, keep the sums in place
                acc[4 * q] = fma(on, g.phi, acc[4 * q]);
                acc[4 * q + 1] = fma(-on, g.gx, acc[4 * q + 1]);
                acc[4 * q + 2] = fma(-on, g.gy, acc[4 * q + 2]);
                acc[4 * q + 3] = fma(-on, g.gz, acc[4 * q + 3]);
            }
        }
        wave_lds_sync();
        // D[r] of lane j + 4 b + 16 i: cell i + 4 b, term 4 r + j
        {
            const int cell = (lane >> 4) + (lane & 12), j = lane & 3;
#pragma unroll
            for (int r = 0; r < kND; ++r)
                if (4 * r + 3 < NH || 4 * r + j < NH) rows[cell * kLst + 4 * r + j] = D[r];
        }
        wave_lds_sync();
        for (int it = lane; it < nb * NH; it += 64) {
            const int f = it / NH, n = it - f * NH;
            gatomic_add(L + (size_t)S.farc[b0 + f] * HSTR + n, rows[f * kLst + n]);
        }
        wave_lds_sync();
    }
}

// Near leaves, 16-lane rows with lane k = target k; the leaves' sources staged in LDS, each
// source's side summed across its row before it is added to G.
__device__ __forceinline__ void grad_near(const RepU& R, GroupShared<true>& S, int near_n, double half_lB, double4* G,
                                          double (&acc)[4]) {
    const int total = group_near_scan(S, near_n);
    const int row = (int)threadIdx.x >> 4, k = (int)threadIdx.x & 15;
    const double x = S.tx[k], y = S.ty[k], z = S.tz[k], wk = half_lB * S.tq[k];
    const int ion = S.ion[k], img = R.images ? R.n + ion : -1;
    for (int base = 0; base < total; base += kStage) {
        const int cnt = min(kStage, total - base);
        stage_near(R, S, near_n, base, cnt);
        __syncthreads();
        for (int s = row; s < cnt; s += kGroupBlock / 16) {
            const double4 p = S.ns[s];
            const int sid = S.nsid[s];
            if (sid < 0 || sid >= R.nsrc) { S.err = kErrNearSlots; break; }  // uniform in the row
            const double dx = x - p.x, dy = y - p.y, dz = z - p.z;
            const double d2 = dx * dx + dy * dy + dz * dz;
            double sx = 0.0, sy = 0.0, sz = 0.0, sq = 0.0;
            if (((S.nsm[s] >> k) & 1u) && sid != ion && sid != img && d2 != 0.0) {
                const double ir = rsqrt_nr(d2);
                const double qi3 = p.w * (ir * ir * ir);
                acc[0] += p.w * ir; acc[1] += qi3 * dx; acc[2] += qi3 * dy; acc[3] += qi3 * dz;
                sx = wk * qi3 * dx; sy = wk * qi3 * dy; sz = wk * qi3 * dz; sq = wk * ir;
            }
            const double sv = row_sum4_scatter(sx, sy, sz, sq, k);
            if ((k & 6) == 0) gatomic_add(&G[sid].x + (((k >> 3) << 1) | (k & 1)), sv);
        }
        __syncthreads();
    }
}

__global__ void __launch_bounds__(kGroupBlock) __attribute__((amdgpu_waves_per_eu(2)))
k_grad(Rep* reps, int r, double* L, double4* G, double4* Gt, double* eterm, int* fcell) {
    constexpr int NW = GroupShared<true>::NW;
    __shared__ GroupShared<true> S;
    __shared__ double red[2][NW][kGT][4];
    __shared__ Rep Rs;
    load_rep(Rs, reps + r);
    __syncthreads();
    const RepU R(Rs);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const double half_lB = 0.5 * R.l_B;
    const int ngroups = (R.n + kGT - 1) / kGT;
    for (int grp = blockIdx.x; grp < ngroups; grp += gridDim.x) {
        group_targets(R, S, Rs.iord, grp, kGT);
        double fa[16], na[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int j = 0; j < 16; ++j) fa[j] = 0.0;
        group_traverse(R, S, false, [&](int far_n, int near_n) {
            grad_far(R, S, S.rows + w * 16 * kLst, far_n, half_lB, L, fa);
            __syncthreads();  // the rows' space takes the near sources next
            grad_near(R, S, near_n, half_lB, G, na);
        });
        // far sums: over the 16 cells of a lane row, leaving one (pass, component) a lane; near sums
        // over the wave's four rows
        const double fs = row_reduce_scatter16(fa, lane & 15);
        const int idx = rs_index(lane & 15);
        red[0][w][4 * (idx >> 2) + (lane >> 4)][idx & 3] = fs;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            na[j] += __shfl_xor(na[j], 16, 64);
            na[j] += __shfl_xor(na[j], 32, 64);
            if (lane < 16) red[1][w][lane][j] = na[j];
        }
        __syncthreads();
        if (tid < S.nt) {
            double a[4] = {0.0, 0.0, 0.0, 0.0};
            for (int part = 0; part < 2; ++part)
                for (int ww = 0; ww < NW; ++ww)
#pragma unroll
                    for (int j = 0; j < 4; ++j) a[j] += red[part][ww][tid][j];
            const int ion = S.ion[tid];
            const double q = S.tq[tid], wq = half_lB * q;
            const bool bad = S.err != 0;
            if (bad && tid == 0) reps[r].err_detail = S.err;
            const double ph = bad ? __builtin_nan("") : a[0];
            eterm[ion] = ion_term(R, S.tx[tid], S.ty[tid], S.tz[tid], q, ph);
            Gt[ion] = make_double4(-wq * a[1], -wq * a[2], -wq * a[3], half_lB * ph);
            fcell[ion] = S.flag_cell[tid];  // (the image's terms in that cell are k_gflag's)
        }
        __syncthreads();
    }
}

// One cell's adjoint row at a source, d = y - c: V = sum_lm N_lm L_lm A_lm(d) and its gradient,
// with da_lm/dz = (l - m) a_{l,m+1} and da_lm/d|d|^2 = -(l - m)(l - m - 1) / (2 (2l - 1)) a_{l-1,m+1}.
template <int M>
__device__ __forceinline__ void adj_columns(GRow L, double x, double y, double z, double s, double (&pc)[P + 1],
                                            double (&V)[2], double (&dV)[2], double (&Z)[2], double (&Q)[2]) {
    if constexpr (M >= 0) {
        constexpr int st = M ? 2 : 1;
        double gc = 0.0, gs = 0.0, zc = 0.0, zs = 0.0, qc = 0.0, qs = 0.0;
        double a0 = 0.0, a1 = 1.0;
        double col[P + 1];
#pragma unroll
        for (int l = M; l <= P; ++l) {
            if (l == M + 1) { a0 = 1.0; a1 = z; }
            if (l > M + 1) {
                const double a2 = fma(z, a1, -(hbeta(l, M) * s) * a0);
                a0 = a1; a1 = a2;
            }
            col[l] = a1;
            const int pl = hplace(M, M) + st * (l - M);
            const double lc = L[pl], ls = M ? L[pl + 1] : 0.0;
            const double v = hnorm(l, M) * a1;
            gc = fma(lc, v, gc);
            if (M) gs = fma(ls, v, gs);
            if (l > M) {
                const double g = hnorm(l, M) * (double)(l - M) * pc[l];
                zc = fma(lc, g, zc);
                if (M) zs = fma(ls, g, zs);
            }
            if (l > M + 1) {
                const double k = -(hnorm(l, M) * (double)((l - M) * (l - M - 1)) / (double)(2 * (2 * l - 1))) * pc[l - 1];
                qc = fma(lc, k, qc);
                if (M) qs = fma(ls, k, qs);
            }
        }
#pragma unroll
        for (int l = M; l <= P; ++l) pc[l] = col[l];
        double t;
        t = fma(dV[1], y, fma(dV[0], x, V[0])); dV[1] = fma(dV[1], x, fma(-dV[0], y, V[1])); dV[0] = t;
        t = fma(V[1], y, fma(V[0], x, gc)); V[1] = fma(V[1], x, fma(-V[0], y, gs)); V[0] = t;
        t = fma(Z[1], y, fma(Z[0], x, zc)); Z[1] = fma(Z[1], x, fma(-Z[0], y, zs)); Z[0] = t;
        t = fma(Q[1], y, fma(Q[0], x, qc)); Q[1] = fma(Q[1], x, fma(-Q[0], y, qs)); Q[0] = t;
        adj_columns<M - 1>(L, x, y, z, s, pc, V, dV, Z, Q);
    }
}

// Step 2, one thread per source in key order (neighbours share their ancestors' rows): the
// source side of every far cell holding it, summed over its ancestors and differentiated in
// the source's position (times its charge) and charge.
__global__ void __launch_bounds__(256) k_adj_down(const Rep* reps, int r, const double* L, double4* G) {
    const Rep& R = reps[r];
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= R.nsrc) return;
    const int s = R.perm[k];
    if ((unsigned)s >= (unsigned)R.nsrc) return;
    const double4 y = R.src[s];
    int c = R.track[s].x;
    double v = 0.0, gx = 0.0, gy = 0.0, gz = 0.0;
    for (int guard = 0; c >= 0 && guard < kMaxLevels; ++guard) {
        if (c >= R.ncell) { v = __builtin_nan(""); break; }
        const double4 g = R.cgeo[c];
        const double dx = y.x - g.x, dy = y.y - g.y, dz = y.z - g.z;
        double pc[P + 1], V[2] = {0.0, 0.0}, dV[2] = {0.0, 0.0}, Z[2] = {0.0, 0.0}, Q[2] = {0.0, 0.0};
        adj_columns<P>(grow(L + (size_t)c * HSTR), dx, dy, dz, dx * dx + dy * dy + dz * dz, pc, V, dV, Z, Q);
        v += V[0];
        gx += dV[0] + 2.0 * dx * Q[0];
        gy += dV[1] + 2.0 * dy * Q[0];
        gz += Z[0] + 2.0 * dz * Q[0];
        c = R.cparent[c];
    }
    double4 o = G[s];
    o.x += y.w * gx; o.y += y.w * gy; o.z += y.w * gz; o.w += v;
    G[s] = o;
}
