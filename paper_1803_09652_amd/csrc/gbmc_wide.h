// gbmc_wide.h -- the three all-pairs passes with one workgroup per tile, for
// launches that leave most of the chip idle (included by gbmc_kernels.hip).
//
// With one wavefront per tile such a launch takes as long as one wavefront
// needs for its 64 steps: it issues alone on its SIMD, at about four cycles an
// instruction (15 us in the energy pass of a 256-atom system, whose tiles have
// two rows, and 26 us in its chain pass).  Here the wavefronts of a workgroup share the steps of
// one work item.  The results stay bitwise those of the one-wavefront walk,
// whose FP32 sums run over the steps in order: the wavefronts write the terms
// of a chunk of steps to LDS, and then each takes some of the sums (the i side
// or the j side of one output) and adds the chunk's terms to them in step order,
// with the same fused operations as the walk.  No sum rotates from lane to
// lane, so the instructions per pair are about the same; what grows is the LDS
// traffic (about 25 words per pair and lane in the energy pass), which is why
// a launch that fills the chip keeps the walk (wide_items in gbmc_host.cpp).
// 256 atoms: descreening 13.5 -> 8.4 us, energy 15.0 -> 9.1, chain 25.9 -> 12.4.

// Two launches of an evaluation drop out as well: the energy pass of gb_evaluate forms
// the Born radii of its atoms itself (radius_state, once per workgroup and block;
// 3.1 us for the launch, under 1 us here), and the chain pass writes the
// outputs.  256 atoms, a whole evaluation: 41.5 -> 37.9 -> 36.7 us; 3,001 atoms
// (only the chain pass runs wide): 72.3 -> 71.7.  A launch that fills the
// chip keeps both kernels: there forming a radius in every item costs more
// FP64 issue (a tanh and four divisions per lane) than the launch.

// Wavefronts per workgroup.  The energy pass has most sums to share out and
// runs wide only where every workgroup has a CU of its own: there 16 took 9.5 us
// and 8 took 12.5 on 16 systems of 237 atoms.  In the other passes 16 gained
// less than 1 us there and lost 3 to 9 on a 3,001-atom system.
constexpr int kWide = 8;
constexpr int kWideEnergy = 16;
constexpr int kWindow = kWide * kTile;  // marked pairs evaluated per round

// (row, step) pairs of a chunk: 32 in FP32 and 16 in FP64, so that three or more
// workgroups fit into a CU's LDS
template <typename T>
constexpr int kChunk = sizeof(T) == 4 ? 32 : 16;

// One chunk walk: pair(s, r, k) evaluates row r at walk step k and stores its terms as
// number s * R + r of the chunk; then sum(s0, k0, n) adds the n steps from k0 on.
// The first step of a diagonal tile is k = 1, the last k = 32 (lanes 0..31).
template <typename T, int R, int W, class Pair, class Sum>
__device__ __forceinline__ void wide_walk(int wave, bool diagonal, Pair&& pair, Sum&& sum)
{
    constexpr int C = kChunk<T> / R, U = C / W;
    const int n = diagonal ? kTile / 2 : kTile, d = diagonal ? 1 : 0;
    for (int c = 0; c < n; c += C) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = wave * U + u;
#pragma unroll
            for (int r = 0; r < R; ++r) pair(s, r, c + s + d);
        }
        __syncthreads();
        sum(c + d);
        __syncthreads();
    }
}

// Marks of the overlapping pairs of a tile (see chain_item) evaluated by the
// workgroup, kWindow to a round: mask[r][lane] holds the marked
// steps, eval(t, il, ir, k) evaluates list entry t, and add(r, t, n) adds n of its
// lane's entries of row r, from t on, to the i side of this wavefront's sums.
template <int R, class Eval, class Add>
__device__ __forceinline__ bool wide_deferred(int wave, int lane, const unsigned long long* mask,
                                              int* slist, Eval&& eval, Add&& add)
{
    unsigned long long m[R];
    int cnt = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        m[r] = mask[r * kTile + lane];
        cnt += __builtin_popcountll(m[r]);
    }
    if (__builtin_amdgcn_ballot_w64(cnt != 0) == 0ull) return false;
    const int incl = wave_scan(cnt, lane);
    const int total = __builtin_amdgcn_readlane(incl, kTile - 1);
    for (int w0 = 0; w0 < total; w0 += kWindow) {
        const int o0 = max(incl - cnt, w0) - w0;
        const int n = max(min(incl, w0 + kWindow) - w0 - o0, 0);
        const int n0 = min(n, (int)__builtin_popcountll(m[0]));
        for (int t = o0; t < o0 + n; ++t) {
            const int ir = (R == 1 || m[0] != 0ull) ? 0 : 1;
            unsigned long long& q = m[R == 1 ? 0 : ir];
            if (wave == 0) slist[t] = (lane << 8) | (ir << 7) | __builtin_ctzll(q);
            q &= q - 1ull;
        }
        __syncthreads();
        const int t = wave * kTile + lane;
        if (w0 + t < total) {
            const int e = slist[t];
            eval(t, e >> 8, (e >> 7) & 1, e & 0x7f);
        }
        __syncthreads();
        add(0, o0, n0);
        if constexpr (R == 2) add(1, o0 + n0, n - n0);
    }
    return true;
}

// -------------------------------------------------------------- descreening

template <typename T>
struct RadiiWide {
    T term[4][kChunk<T>][kTile];        // H_ij as a product of two factors, H_ji
    T j[5][2 * kTile];                  // x, y, z, rt, S, twice
    T i[5][kTile];
    unsigned long long mask[kTile];
    unsigned long long def[kTile];      // j side of the marked pairs
    int list[kWindow];
};

// Item data of one atom block, one lane per atom, with the stand-ins of lanes
// past the end (dummy atoms that contribute nothing).
template <typename T>
__device__ __forceinline__ void radii_atom(const WorkItem& w, int a, const Q4<T>* __restrict__ P,
                                           const Q4<T>* __restrict__ Gx, T (&v)[5])
{
    if (a < w.n) {
        const Q4<T> p = P[w.base + a], g = Gx[w.base + a];
        v[0] = p.x; v[1] = p.y; v[2] = p.z; v[3] = g.x; v[4] = g.y;
    } else {
        dummy_pos(a, v[0], v[1], v[2]);
        v[3] = T(1); v[4] = T(0);
    }
}

template <typename T, int TIER>
__device__ __forceinline__ void radii_wide_walk(RadiiWide<T>& L, int wave, int lane, bool diagonal,
                                                bool vi, T& sum)
{
    constexpr bool SEP = TIER != 0;
    constexpr int FIT = sizeof(T) == 4 && SEP ? 1 : TIER;
    T me[5];
#pragma unroll
    for (int a = 0; a < 5; ++a) me[a] = L.i[a][lane];
    unsigned long long marks = 0ull;
    auto pair = [&](int s, int, int k) {
        const bool act = !(diagonal && k == kTile / 2 && lane >= kTile / 2);
        const T x = L.j[0][lane + k], y = L.j[1][lane + k], z = L.j[2][lane + k];
        const T rt = L.j[3][lane + k], S = L.j[4][lane + k];
        if constexpr (SEP) {
            // the walk adds the products x^3 / r * P in one fused operation
            const T dx = me[0] - x, dy = me[1] - y, dz = me[2] - z;
            T invr;
            if constexpr (sizeof(T) == 4) {
                invr = rsq(fma(dx, dx, fma(dy, dy, dz * dz)));
            } else {
                T r;
                dist64(me[0], me[1], me[2], x, y, z, r, invr);
            }
            const T xij = S * invr, yij = xij * xij;
            const T xji = me[4] * invr, yji = xji * xji;
            L.term[0][s][lane] = xij * yij * invr;
            L.term[1][s][lane] = tier_p<FIT>(yij);
            L.term[2][s][lane] = xji * yji * invr;
            L.term[3][s][lane] = tier_p<FIT>(yji);
        } else {
            T hij, hji;
            radii_pair_fast<0>(me[0], me[1], me[2], x, y, z, me[3], me[4], rt, S, act && vi,
                                  1ull << k, hij, hji, marks);
            L.term[0][s][lane] = act ? hij : T(0);
            L.term[2][s][lane] = act ? hji : T(0);
        }
    };
    auto add = [&](int k0) {
        if (wave == 0) {
#pragma unroll 8
            for (int s = 0; s < kChunk<T>; ++s) {
                if constexpr (SEP) sum = fma(L.term[0][s][lane], L.term[1][s][lane], sum);
                else sum += L.term[0][s][lane];
            }
        } else if (wave == 1) {
#pragma unroll 8
            for (int s = 0; s < kChunk<T>; ++s) {
                const int l = (lane - k0 - s) & (kTile - 1);
                if constexpr (SEP) sum = fma(L.term[2][s][l], L.term[3][s][l], sum);
                else sum += L.term[2][s][l];
            }
        }
    };
    wide_walk<T, 1, kWide>(wave, diagonal, pair, add);
    if (!SEP && marks != 0ull) atomicOr(&L.mask[lane], marks);
}

template <typename T>
__global__ __launch_bounds__(kWide * kTile) void k_radii_wide(
    const WorkItem* __restrict__ items, const Q4<T>* __restrict__ P, const Q4<T>* __restrict__ Gx,
    unsigned long long* __restrict__ I_fx, int* __restrict__ ovf, const Q4<float>* __restrict__ box)
{
    __shared__ RadiiWide<T> L;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kTile), lane = threadIdx.x % kTile;
    const WorkItem w = items[blockIdx.x];
    const int J = w.J0, i = w.I * kTile + lane, j = J * kTile + lane;
    const bool diagonal = J == w.I;
    const int tier = diagonal ? 0 : tile_tier<1>(box, w.blk0 + w.I, w.blk0 + J);
    if (wave < 2) {
        T v[5];
        radii_atom<T>(w, wave == 0 ? j : i, P, Gx, v);
#pragma unroll
        for (int a = 0; a < 5; ++a) {
            if (wave == 0) L.j[a][lane] = L.j[a][lane + kTile] = v[a];
            else L.i[a][lane] = v[a];
        }
    } else if (wave == 2) {
        L.mask[lane] = 0ull;
        L.def[lane] = 0ull;
    }
    __syncthreads();
    T sum = T(0);
    bool bad = false, deferred = false;
    if (tier == 2) {
        radii_wide_walk<T, 2>(L, wave, lane, false, true, sum);
    } else if (tier == 1) {
        radii_wide_walk<T, 1>(L, wave, lane, false, true, sum);
    } else {
        radii_wide_walk<T, 0>(L, wave, lane, diagonal, i < w.n, sum);
        __syncthreads();
        T* siv = &L.term[0][0][0];
        deferred = wide_deferred<1>(
            wave, lane, L.mask, L.list,
            [&](int t, int il, int, int k) {
                const int jl = il + k;
                const T dx = L.i[0][il] - L.j[0][jl], dy = L.i[1][il] - L.j[1][jl];
                const T dz = L.i[2][il] - L.j[2][jl];
                const T r2 = dist2(dx, dy, dz);
                const T invr = rsq(r2);
                const T rr = r2 * invr;
                siv[t] = slow_H(rr, invr, L.i[3][il], L.j[4][jl]);
                const T hv = slow_H(rr, invr, L.j[3][jl], L.i[4][il]);
                atomicAdd(&L.def[jl & (kTile - 1)], (unsigned long long)to_fixed(hv, kScaleI, bad));
            },
            [&](int, int t, int n) {
                if (wave == 0)
                    for (int u = 0; u < n; ++u) sum += siv[t + u];
            });
    }
    if (wave == 0 && i < w.n) fx_add(&I_fx[w.base + i], to_fixed(sum, kScaleI, bad));
    if (wave == 1 && j < w.n) {
        long long v = to_fixed(sum, kScaleI, bad);
        if (deferred) v += (long long)L.def[lane];
        fx_add(&I_fx[w.base + j], v);
    }
    if (bad) *ovf = 1;
}

// ------------------------------------------------ energies, explicit forces

template <typename T, int NT>
struct EnergyWide {
    T term[NT][kChunk<T>][kTile];       // qq, 1/r, 1/f, (dE/dr)/r, G term, (salt) GB factor
    T j[6][2 * kTile];                  // x, y, z, q, R, a, twice
    T i[2][6][kTile];
};

template <typename T, bool GRAD, int R, bool SALT, int NT>
__device__ __forceinline__ void energy_wide(EnergyWide<T, NT>& L, const WorkItem& w, int wave,
                                            int lane, const Q4<T>* __restrict__ P, T kC, T kT,
                                            const SaltK<T>& sk, const Work<T>& wk, bool finalize,
                                            const GBConst& gc, T* __restrict__ born_R)
{
    constexpr int FR = GRAD ? 3 : 0, CG = GRAD ? 4 : 0;     // terms of the gradients
    const int J = w.J0, j = J * kTile + lane;
    const bool diagonal = R == 1 && J == w.I;
    const EnergyK<T, SALT> ek(kC, kT);
    if (wave <= R) {
        const int a = wave == 0 ? j : (w.I + wave - 1) * kTile + lane;
        T v[6];
        if (a < w.n) {
            const int g = w.base + a;
            const Q4<T> p = P[g];
            v[0] = p.x; v[1] = p.y; v[2] = p.z; v[3] = p.w * ek.sq;
            // (finalize: the radii are formed here, and stored by the diagonal item)
            if (finalize) {
                const RadiusState st = radius_state(wk.I_fx[g], (double)wk.Gx[g].w, gc);
                v[4] = (T)st.R; v[5] = (T)(kAScale / st.R);
                if (diagonal && wave == 0) radius_store<T, false>(g, wk.perm[g], st, p, wk, born_R);
            } else {
                v[4] = wk.R_t[g]; v[5] = wk.a_t[g];
            }
        } else {
            dummy_pos(a, v[0], v[1], v[2]);
            v[3] = T(0); v[4] = T(1); v[5] = T(kAScale);
        }
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            if (wave == 0) L.j[c][lane] = L.j[c][lane + kTile] = v[c];
            else L.i[wave - 1][c][lane] = v[c];
        }
    }
    __syncthreads();
    T me[R][6];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < 6; ++c) me[r][c] = L.i[r][c][lane];
    auto pair = [&](int s, int r, int k) {
        const bool act = !(diagonal && k == kTile / 2 && lane >= kTile / 2);
        const int q = s * R + r, l = lane + k;
        const EnergyTerms<T> e = energy_terms<T, GRAD, SALT, false>(
            me[r][0], me[r][1], me[r][2], me[r][3], me[r][4], me[r][5], L.j[0][l], L.j[1][l],
            L.j[2][l], L.j[3][l], L.j[4][l], L.j[5][l], act, energy_xfirst(diagonal, k), kC, kT, ek,
            sk, T(0));
        L.term[0][q][lane] = e.qq;
        L.term[1][q][lane] = act ? e.invr : T(0);
        L.term[2][q][lane] = act ? e.invf : T(0);
        if constexpr (GRAD) {
            L.term[FR][q][lane] = e.fr;
            L.term[CG][q][lane] = e.cg;
        }
        if constexpr (SALT) L.term[NT - 1][q][lane] = e.kd;
    };
    constexpr int C = kChunk<T> / R;
    // The sums: of each row's i side the energies, the three force components,
    // G and phi (task 6 row + kind), then of the j side the three force
    // components, and G with phi; shared out over the wavefronts.
    constexpr int NTASK = GRAD ? 6 * R + 4 : R, PER = (NTASK + kWideEnergy - 1) / kWideEnergy;
    auto weight = [&](int q, int l) {
        return energy_weight<T, SALT>(L.term[1][q][l], L.term[2][q][l], kC,
                                      SALT ? L.term[NT - 1][q][l] : T(0), ek);
    };
    auto run_task = [&](int task, T (&sum)[2], int k0) {
        const int row = GRAD ? task / 6 : task, kind = GRAD ? task % 6 : 0, jt = task - 6 * R;
        if (row < R && kind == 0) {
#pragma unroll 8
            for (int s = 0; s < C; ++s) {
                const int q = s * R + row;
                const T qq = L.term[0][q][lane];
                sum[0] = fma(qq, L.term[1][q][lane], sum[0]);
                const T g = SALT ? qq * L.term[NT - 1][q][lane] : qq;
                sum[1] = fma(g, L.term[2][q][lane], sum[1]);
            }
        }
        if constexpr (GRAD) {
            if (row < R) {
                if (kind >= 1 && kind <= 3) {
                    const T x = L.i[row][kind - 1][lane];
#pragma unroll 8
                    for (int s = 0; s < C; ++s)
                        sum[0] = fma(-L.term[FR][s * R + row][lane], x - L.j[kind - 1][lane + k0 + s],
                                     sum[0]);
                } else if (kind == 4) {
#pragma unroll 8
                    for (int s = 0; s < C; ++s)
                        sum[0] = fma(L.term[CG][s * R + row][lane], L.j[4][lane + k0 + s], sum[0]);
                } else if (kind == 5) {
#pragma unroll 8
                    for (int s = 0; s < C; ++s)
                        sum[0] = fma(weight(s * R + row, lane), L.j[3][lane + k0 + s], sum[0]);
                }
            } else if (jt < 3) {
                const T xj = L.j[jt][lane];
#pragma unroll 8
                for (int s = 0; s < C; ++s) {
                    const int l = (lane - k0 - s) & (kTile - 1);
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        sum[0] = fma(L.term[FR][s * R + r][l], L.i[r][jt][l] - xj, sum[0]);
                }
            } else if (jt == 3) {
#pragma unroll 8
                for (int s = 0; s < C; ++s) {
                    const int l = (lane - k0 - s) & (kTile - 1);
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const int q = s * R + r;
                        sum[0] = fma(L.term[CG][q][l], L.i[r][4][l], sum[0]);
                        sum[1] = fma(weight(q, l), L.i[r][3][l], sum[1]);
                    }
                }
            }
        }
    };
    T sums[PER][2];
#pragma unroll
    for (int u = 0; u < PER; ++u) sums[u][0] = sums[u][1] = T(0);
    auto task_of = [&](int u) { return wave + u * kWideEnergy; };
    wide_walk<T, R, kWideEnergy>(wave, diagonal, pair, [&](int k0) {
#pragma unroll
        for (int u = 0; u < PER; ++u)
            if (task_of(u) < NTASK) run_task(task_of(u), sums[u], k0);
    });
    bool bad = false;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int task = task_of(u);
        if (task >= NTASK) break;
        const int row = GRAD ? task / 6 : task, kind = GRAD ? task % 6 : 0, jt = task - 6 * R;
        T(&sum)[2] = sums[u];
        if (row < R) {
            if (diagonal) {
                T eG = sum[1], phii = sum[0], Gi = sum[0];
                energy_self<T, SALT>(me[0][3], me[0][4], kC, ek, sk, eG, phii, Gi);
                sum[1] = eG;
                if (kind == 4) sum[0] = Gi;
                if (kind == 5) sum[0] = phii;
            }
            const int i = (w.I + row) * kTile + lane;
            if (kind == 0) {
                const long long e0 = to_fixed(T((SALT ? kC : T(1)) * sum[0]), kScaleE, bad);
                const long long e1 = to_fixed(T(-(SALT ? T(1) : ek.tau) * sum[1]), kScaleE, bad);
                if (i < w.n) {
                    fx_add(&wk.EA_fx[w.base + i], e0);
                    fx_add(&wk.EA_fx[wk.n_atoms + w.base + i], e1);
                }
            } else if constexpr (GRAD) {
                const T v = kind == 4 ? T(sum[0] * ek.sG) : kind == 5 ? T(sum[0] * ek.sPhi) : sum[0];
                const long long f = to_fixed(v, kScaleF, bad);
                unsigned long long* out = kind == 4   ? wk.G_fx
                                          : kind == 5 ? wk.phi_fx
                                                      : wk.F_fx + (kind - 1) * wk.n_atoms;
                if (i < w.n) fx_add(&out[w.base + i], f);
            }
        } else if constexpr (GRAD) {
            const T v = jt == 3 ? T(sum[0] * ek.sG) : sum[0];
            const long long f0 = to_fixed(v, kScaleF, bad);
            const long long f1 = to_fixed(T(sum[1] * ek.sPhi), kScaleF, bad);
            if (j < w.n) {
                fx_add(&(jt == 3 ? wk.G_fx : wk.F_fx + jt * wk.n_atoms)[w.base + j], f0);
                if (jt == 3) fx_add(&wk.phi_fx[w.base + j], f1);
            }
        }
    }
    if (bad) *wk.ovf = 1;
}

template <typename T, bool GRAD, bool SALT>
__global__ __launch_bounds__(kWideEnergy * kTile) void k_energy_wide(const WorkItem* __restrict__ items,
                                                              const Q4<T>* __restrict__ P, T kC,
                                                              T kT, SaltK<T> sk, Work<T> wk,
                                                              bool finalize, GBConst gc,
                                                              T* __restrict__ born_R)
{
    constexpr int NT = (GRAD ? 5 : 3) + (SALT ? 1 : 0);
    __shared__ EnergyWide<T, NT> L;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kTile), lane = threadIdx.x % kTile;
    const WorkItem w = items[blockIdx.x];
    if (sizeof(T) == 4 && w.rows == 2)
        energy_wide<T, GRAD, sizeof(T) == 4 ? 2 : 1, SALT, NT>(L, w, wave, lane, P, kC, kT, sk, wk, finalize,
                                                               gc, born_R);
    else
        energy_wide<T, GRAD, 1, SALT, NT>(L, w, wave, lane, P, kC, kT, sk, wk, finalize,
                                                               gc, born_R);
}

// -------------------------------------------------------- Born-radius chain

template <typename T>
struct ChainWide {
    T term[3][kChunk<T>][kTile];        // (dE/dr)/r, dH_ij/dS, dH_ji/dS
    T j[7][2 * kTile];                  // x, y, z, rt, S, B rt, screen, twice
    T i[2][7][kTile];
    unsigned long long mask[2 * kTile];
    unsigned long long def[4][kTile];   // j side of the marked pairs
    int list[kWindow];
};

// The sums of the chain pass: of each row's i side the three force components
// and dE/drho (task 4 row + component), then of the j side.
template <int R>
constexpr int chain_tasks_per = (4 * R + 4 + kWide - 1) / kWide;

template <typename T, int R, int TIER>
__device__ __forceinline__ void chain_wide_walk(ChainWide<T>& L, int wave, int lane, bool diagonal,
                                                const bool (&vi)[R],
                                                T (&sum)[chain_tasks_per<R>])
{
    T me[R][7];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int c = 0; c < 7; ++c) me[r][c] = L.i[r][c][lane];
    unsigned long long marks[R];
#pragma unroll
    for (int r = 0; r < R; ++r) marks[r] = 0ull;
    auto pair = [&](int s, int r, int k) {
        const bool act = !(diagonal && k == kTile / 2 && lane >= kTile / 2);
        const int q = s * R + r, l = lane + k;
        const T dx = me[r][0] - L.j[0][l], dy = me[r][1] - L.j[1][l], dz = me[r][2] - L.j[2][l];
        const T r2 = dist2(dx, dy, dz);
        const T invr = rsq(r2);
        const T rr = r2 * invr;
        T dEdr, gij, gji;
        chain_pair_fast<TIER>(rr, invr, me[r][3], me[r][4], L.j[3][l], L.j[4][l], me[r][5], L.j[5][l],
                              act && vi[r], 1ull << k, dEdr, gij, gji, marks[r]);
        L.term[0][q][lane] = act ? T(dEdr * invr) : T(0);
        L.term[1][q][lane] = act ? gij : T(0);
        L.term[2][q][lane] = act ? gji : T(0);
    };
    constexpr int C = kChunk<T> / R;
    auto run_task = [&](int task, T& sum, int k0) {
        const int row = task / 4, comp = task % 4;
        if (row < R) {
            if (comp < 3) {
                const T x = L.i[row][comp][lane];
#pragma unroll 8
                for (int s = 0; s < C; ++s)
                    sum = fma(-L.term[0][s * R + row][lane], x - L.j[comp][lane + k0 + s], sum);
            } else {
                const T sc = L.i[row][6][lane];
#pragma unroll 8
                for (int s = 0; s < C; ++s)
                    sum = fma(sc * L.j[5][lane + k0 + s], L.term[2][s * R + row][lane], sum);
            }
        } else if (comp < 3) {
            const T xj = L.j[comp][lane];
#pragma unroll 8
            for (int s = 0; s < C; ++s) {
                const int l = (lane - k0 - s) & (kTile - 1);
#pragma unroll
                for (int r = 0; r < R; ++r)
                    sum = fma(L.term[0][s * R + r][l], L.i[r][comp][l] - xj, sum);
            }
        } else {
            const T sc = L.j[6][lane];
#pragma unroll 8
            for (int s = 0; s < C; ++s) {
                const int l = (lane - k0 - s) & (kTile - 1);
#pragma unroll
                for (int r = 0; r < R; ++r)
                    sum = fma(sc * L.i[r][5][l], L.term[1][s * R + r][l], sum);
            }
        }
    };
    wide_walk<T, R, kWide>(wave, diagonal, pair, [&](int k0) {
#pragma unroll
        for (int u = 0; u < chain_tasks_per<R>; ++u)
            if (wave + u * kWide < 4 * R + 4) run_task(wave + u * kWide, sum[u], k0);
    });
    if constexpr (TIER == 0)
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (marks[r] != 0ull) atomicOr(&L.mask[r * kTile + lane], marks[r]);
}

template <typename T, int R>
__device__ __forceinline__ void chain_wide(ChainWide<T>& L, const WorkItem& w, int wave, int lane,
                                           const Q4<T>* __restrict__ P, const Q4<T>* __restrict__ Gx,
                                           const Work<T>& wk, const PostOut<T>& po,
                                           const int* __restrict__ total, int* __restrict__ cnt)
{
    const int J = w.J0, j = J * kTile + lane;
    const bool diagonal = R == 1 && J == w.I;
    const int tier = diagonal ? 0 : tile_tier<R>(wk.box, w.blk0 + w.I, w.blk0 + J);
    if (wave <= R) {
        const int a = wave == 0 ? j : (w.I + wave - 1) * kTile + lane;
        T v[7];
        if (a < w.n) {
            const int g = w.base + a;
            const Q4<T> p = P[g], gx = Gx[g];
            v[0] = p.x; v[1] = p.y; v[2] = p.z; v[3] = gx.x; v[4] = gx.y;
            v[5] = brt_from<T>(wk.G_fx[g], wk.dRdPsi_p[g], gx.x);
            v[6] = gx.z;
        } else {
            dummy_pos(a, v[0], v[1], v[2]);
            v[3] = T(1); v[4] = v[5] = v[6] = T(0);
        }
#pragma unroll
        for (int c = 0; c < 7; ++c) {
            if (wave == 0) L.j[c][lane] = L.j[c][lane + kTile] = v[c];
            else L.i[wave - 1][c][lane] = v[c];
        }
    } else if (wave == 3) {
        L.mask[lane] = L.mask[lane + kTile] = 0ull;
    } else if (wave >= 4 && wave < 8) {
        L.def[wave - 4][lane] = 0ull;
    }
    __syncthreads();
    constexpr int PER = chain_tasks_per<R>;
    T sum[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) sum[u] = T(0);
    bool vi[R];
#pragma unroll
    for (int r = 0; r < R; ++r) vi[r] = (w.I + r) * kTile + lane < w.n;
    bool bad = false, deferred = false;
    if (tier == 2) {
        chain_wide_walk<T, R, 2>(L, wave, lane, false, vi, sum);
    } else if (tier == 1) {
        chain_wide_walk<T, R, 1>(L, wave, lane, false, vi, sum);
    } else {
        chain_wide_walk<T, R, 0>(L, wave, lane, diagonal, vi, sum);
        __syncthreads();
        T* siv = &L.term[0][0][0];              // [4][kWindow]
        static_assert(sizeof(L.term) >= 4 * kWindow * sizeof(T), "room for a round's terms");
        deferred = wide_deferred<R>(
            wave, lane, L.mask, L.list,
            [&](int t, int il, int ir, int k) {
                const int jl = il + k;
                const T(&q)[7][kTile] = L.i[R == 1 ? 0 : ir];
                const T dx = q[0][il] - L.j[0][jl], dy = q[1][il] - L.j[1][jl];
                const T dz = q[2][il] - L.j[2][jl];
                const T r2 = dist2(dx, dy, dz);
                const T invr = rsq(r2);
                const T rr = r2 * invr;
                T iv[4], jv[4];
                chain_deferred(rr, invr, dx, dy, dz, q[3][il], q[4][il], q[5][il], q[6][il],
                               L.j[3][jl], L.j[4][jl], L.j[5][jl], L.j[6][jl], iv, jv);
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    siv[a * kWindow + t] = iv[a];
                    atomicAdd(&L.def[a][jl & (kTile - 1)],
                              (unsigned long long)to_fixed(jv[a], kScaleF, bad));
                }
            },
            [&](int r, int t, int n) {
#pragma unroll
                for (int u = 0; u < PER; ++u) {
                    const int task = wave + u * kWide;
                    if (task / 4 == r)
                        for (int v = 0; v < n; ++v) sum[u] += siv[(task % 4) * kWindow + t + v];
                }
            });
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int task = wave + u * kWide, row = task / 4, comp = task % 4;
        if (row > R) break;
        unsigned long long* out = comp < 3 ? wk.F_fx + comp * wk.n_atoms : wk.drho_fx;
        long long f = to_fixed(sum[u], kScaleF, bad);
        if (row == R && deferred) f += (long long)L.def[comp][lane];
        const int a = (row == R ? J : w.I + row) * kTile + lane;
        if (a < w.n) fx_add(&out[w.base + a], f);
    }
    if (bad) *wk.ovf = 1;
    // The workgroup whose sums are a block's last writes that block's outputs (a
    // launch of their own took 3.8 us of a 38 us evaluation of 256 atoms).  vmcnt(0):
    // every sum of the workgroup is added before it is counted.
    __builtin_amdgcn_s_waitcnt(0x0f70);
    __syncthreads();
    const int X = wave == 0 ? J : w.I + wave - 1;
    if (wave > R || (diagonal && wave == 1)) return;
    int before = 0;
    if (lane == 0) before = atomicAdd(cnt + w.blk0 + X, 1);
    if (__builtin_amdgcn_readfirstlane(before) != total[w.blk0 + X] - 1) return;
    if (X * kTile + lane < w.n) post_atom<T, true>(w.base + X * kTile + lane, po, wk);
}

// Workgroups [0, n_items) take one work item each; the following ones sum the
// energy shares, final before this pass begins.  total: the items that touch each
// block; cnt: those counted so far (cleared by the staging kernel).
template <typename T>
__global__ __launch_bounds__(kWide * kTile) void k_chain_wide(const WorkItem* __restrict__ items,
                                                             int n_items, const Q4<T>* __restrict__ P,
                                                             const Q4<T>* __restrict__ Gx, Work<T> wk,
                                                             PostOut<T> po,
                                                             const int* __restrict__ total,
                                                             int* __restrict__ cnt)
{
    __shared__ ChainWide<T> L;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kTile), lane = threadIdx.x % kTile;
    if ((int)blockIdx.x >= n_items) {
        sum_energies<T>(po.sums, blockIdx.x - n_items, wk, po.e_coul, po.e_gb);
        return;
    }
    const WorkItem w = items[blockIdx.x];
    if (sizeof(T) == 4 && w.rows == 2)
        chain_wide<T, sizeof(T) == 4 ? 2 : 1>(L, w, wave, lane, P, Gx, wk, po, total, cnt);
    else
        chain_wide<T, 1>(L, w, wave, lane, P, Gx, wk, po, total, cnt);
}
