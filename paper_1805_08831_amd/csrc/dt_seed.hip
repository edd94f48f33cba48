// The first insertions of a cloud, in the LDS of one block.
//
// The rounds of dt_insert.hip gain a few percent of the mesh's vertices each, whatever the
// mesh's size, and a round on a small mesh lasts 60 to 85 us: the latency of its dependent
// accesses to memory and of its launches.  From the four points of the initial tetrahedron to
// 576 vertices that is about 100 rounds, 5 to 8 ms of every triangulation.  Here one block per
// cloud takes the first 572 points of the insertion order (Sec. 2.3) with coordinates,
// tetrahedra and claims in LDS, where a barrier ends a round, and writes the mesh to the pool
// once: about 85 rounds of 18 us (half of it the slowest of the 16 attempts of a round), 1.6 ms.
// 1000 points 7.1 -> 4.0 ms, 2e4 points 15.1 -> 11.2 ms a pass when it came in.  Limits of 320,
// 448, 576 and 768 vertices: 1000 points 3.99, 3.80, 3.73, 3.78 ms, 2e4 points 9.93, 9.73, 9.64,
// 9.75, 64 clouds of 1000 to 2e5 points 71.9, 71.0, 70.8, 72.6.
//
// Only the fp64 filters run; an attempt they leave undecided, a cavity beyond the group's
// lists, or a point still open when the tetrahedra no longer fit, stays a candidate of the
// rounds.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dt_internal.h"
#include "dt_predicates.h"

namespace dtk {

namespace {

// 16 attempts at a time, 32 lanes each (two attempts per wavefront).  Measured on 1000 points,
// a pass: 16 x 32 lanes 4.0 ms, 16 x 64 4.0, 8 x 64 4.4, 8 x 32 4.7, 16 x 16 4.7, 32 x 32 4.1.
// With the exact predicates in the kernel (256 registers and spills) 16 x 32 took 4.3.
constexpr int SEED_THREADS = 512;
constexpr int SEED_LANES = 32;  // lanes per insertion
constexpr int SEED_GROUPS = SEED_THREADS / SEED_LANES;
// LDS: 34 bytes per vertex, 20 per tetrahedron and 480 per group, 112 KB in all
constexpr uint32_t SEED_VERTS = 576;
constexpr uint32_t SEED_TETS = 4224;  // uniform clouds have about 6.6 per vertex at this size
constexpr uint32_t SEED_CAV = 48, SEED_BND = 64;
constexpr uint32_t SEED_ROUNDS = 8 * SEED_VERTS;  // far more than a run takes
constexpr uint32_t SEED_WALK = 64;  // steps of a walk in one round; it goes on in the next

constexpr uint32_t LGHOST = 0xFFFFu, LDEAD = 0xFFFEu;  // GHOST and DEAD among 16-bit vertices
constexpr int UNSURE = 2;                               // a sign the filter leaves open
constexpr uint32_t LBOUND = 0x8000u;                   // marks a boundary facet among codes 4 t + f
static_assert(4 * SEED_TETS < LBOUND, "codes leave the mark's bit free");
// claims: round (lower later), vertex, kind (0 cavity, 1 outer)
constexpr int SEED_VBITS = 10;
static_assert(SEED_VERTS <= 1u << SEED_VBITS, "a vertex fits a claim");

// read as one 16-byte and one 8-byte word
struct alignas(16) SeedVert {
    double x, y, z;
    uint32_t pos;  // vertex record
    uint32_t pad;
};

struct SeedLds {
    SeedVert p[SEED_VERTS];
    ushort4 v[SEED_TETS];
    ushort4 n[SEED_TETS];  // neighbour codes
    uint32_t claim[SEED_TETS];
    uint16_t hint[SEED_VERTS];  // a live tetrahedron of an inserted vertex, LGHOST before
    uint16_t cav[SEED_GROUPS][SEED_CAV];
    uint16_t bnd[SEED_GROUPS][SEED_BND];   // boundary facets, codes in the cavity
    uint16_t outer[SEED_GROUPS][SEED_BND];  // codes of their outer side
    uint16_t slot[SEED_GROUPS][SEED_BND];  // new tetrahedra
    uint32_t wave[SEED_THREADS / 64];
    uint32_t count, ntets, next, full, base;
    uint32_t won, lost, att, walk, ncav, nbnd;
};
static_assert(sizeof(SeedLds) <= 160 * 1024, "the block's LDS");

__device__ __forceinline__ P3 seed_pt(const SeedLds &s, uint32_t v) { return {s.p[v].x, s.p[v].y, s.p[v].z}; }

// vertex or neighbour code number k of four
__device__ __forceinline__ uint32_t at4(ushort4 q, int k) {
    return k == 0 ? q.x : (k == 1 ? q.y : (k == 2 ? q.z : q.w));
}
// entry 4 t + f of the vertices or neighbours, by its code
__device__ __forceinline__ uint16_t &entry4(ushort4 *a, uint32_t cd) { return reinterpret_cast<uint16_t *>(a)[cd]; }

// -1: P is strictly inside the circumsphere of a, b, c, d (positive); 1 outside; UNSURE
__device__ __forceinline__ int seed_insphere(const SeedLds &s, const uint32_t q[4], P3 P, PredStats &st) {
    st.insphere++;
    const int r = insphere_filter(seed_pt(s, q[0]), seed_pt(s, q[1]), seed_pt(s, q[2]), seed_pt(s, q[3]), P);
    return r == 0 ? UNSURE : r;
}

__device__ __forceinline__ int seed_orient(P3 a, P3 b, P3 c, P3 d, PredStats &st) {
    st.orient++;
    const int r = orient3d_filter(a, b, c, d);
    return r == 0 ? UNSURE : r;
}

// exclusive count of `ok` over the block's threads, *total over all of them
__device__ __forceinline__ uint32_t seed_count(SeedLds &s, bool ok, uint32_t *total) {
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    const unsigned long long m = __ballot(ok);
    if (lane == 0) s.wave[wid] = (uint32_t)__popcll(m);
    __syncthreads();
    uint32_t before = 0, all = 0;
    for (uint32_t w = 0; w < SEED_THREADS / 64; ++w) {
        if (w < wid) before += s.wave[w];
        all += s.wave[w];
    }
    __syncthreads();
    *total = all;
    return before + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
}

// first position in the ascending list a[0 .. n) whose entry is at least x
__device__ __forceinline__ uint32_t seed_lower(const uint32_t *__restrict__ a, uint32_t n, uint32_t x) {
    uint32_t lo = 0, hi = n;
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (a[mid] < x) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ uint32_t &seed_nref(Tet *T, uint32_t t, uint32_t f) {
    return reinterpret_cast<uint32_t *>(&T[t].n)[f];
}
__device__ __forceinline__ unsigned long long &seed_nref(TetW *T, uint32_t t, uint32_t f) { return T[t].n.c[f]; }

}  // namespace

// One block per cloud.  lord: the first level's records, ascending; the cloud's part of them is
// taken in bit-reversed order, which spreads any prefix over the cloud.  Slots first_slot + 5 c
// .. + 4 hold the cloud's initial tetrahedron and its ghosts.
template <class K>
__global__ __launch_bounds__(SEED_THREADS) void k_seed(const Vert *__restrict__ V, Cloud *__restrict__ clouds,
                                                       uint32_t first_slot, const uint32_t *__restrict__ lord,
                                                       uint32_t nlord, const uint8_t *__restrict__ dup,
                                                       typename K::Rec *T, uint32_t tcap, uint32_t *vtet, Ctr *ctr,
                                                       SubD *subd, unsigned long long *stat, uint32_t *log_att,
                                                       uint32_t vlo) {
    using code = typename K::code;
    __shared__ SeedLds s;
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t gl = tid % SEED_LANES, gi = tid / SEED_LANES;
    const uint32_t gbase = lane & ~(uint32_t)(SEED_LANES - 1);
    const unsigned long long gmask = ((1ull << SEED_LANES) - 1ull) << gbase;
    const unsigned long long below = gmask & ((1ull << lane) - 1ull);
    const uint32_t c0 = first_slot + 5 * blockIdx.x;
    Cloud *const cl = &clouds[blockIdx.x];
    PredStats st;

    // the initial mesh: vertices 0 .. 3 of tetrahedron 0, ghosts 1 .. 4
    for (uint32_t t = tid; t < SEED_TETS; t += SEED_THREADS) {
        s.claim[t] = ~0u;
        s.v[t].x = (uint16_t)LDEAD;
    }
    for (uint32_t v = tid; v < SEED_VERTS; v += SEED_THREADS) s.hint[v] = v < 4 ? 0u : (uint16_t)LGHOST;
    if (tid == 0) {
        s.count = 4;
        s.ntets = 5;
        s.next = 4;
        s.full = 0;
        s.won = s.lost = s.att = s.walk = s.ncav = s.nbnd = 0;
    }
    __syncthreads();
    if (tid < 20) {
        const uint32_t t = tid >> 2, f = tid & 3u;
        const uint4 v0 = T[c0].v, vt = T[c0 + t].v;
        const uint32_t g = comp(vt, (int)f);
        uint32_t l = LGHOST;
        for (int k = 0; k < 4; ++k)
            if (g != GHOST && comp(v0, k) == g) l = (uint32_t)k;
        entry4(s.v, tid) = (uint16_t)l;
        entry4(s.n, tid) = (uint16_t)(comp(T[c0 + t].n, (int)f) - 4 * (code)c0);
    }
    if (tid < 4) {
        const uint32_t p = comp(T[c0].v, (int)tid);
        const Vert r = V[p];
        s.p[tid] = SeedVert{r.x, r.y, r.z, p, 0u};
    }
    __syncthreads();

    // the points: vertices 4, 5, ...
    {
        const uint32_t a = seed_lower(lord, nlord, cl->lo), m = seed_lower(lord, nlord, cl->hi) - a;
        uint32_t bits = 0;
        while ((1u << bits) < m) ++bits;
        uint32_t have = 4;
        for (uint32_t r0 = 0; r0 < (1u << bits) && have < SEED_VERTS; r0 += SEED_THREADS) {
            const uint32_t r = r0 + tid, q = bits ? __brev(r) >> (32 - bits) : 0u;
            bool ok = r < (1u << bits) && q < m;
            uint32_t p = 0;
            if (ok) {
                p = lord[a + q];
                ok = !dup[p] && vtet[p] == NONE;
            }
            uint32_t total;
            const uint32_t at = have + seed_count(s, ok, &total);
            if (ok && at < SEED_VERTS) {
                const Vert rec = V[p];
                s.p[at] = SeedVert{rec.x, rec.y, rec.z, p, 0u};
            }
            have = min(have + total, SEED_VERTS);
        }
        if (tid == 0) s.count = have;
        __syncthreads();
    }
    const uint32_t nverts = s.count;

    // Rounds: a group keeps its point until it is inserted (or left out), then takes the next;
    // the earliest point in hand always wins its round.
    uint32_t mine = 0, start = LGHOST;  // 0: no point in hand
    unsigned walk = 0, tries = 0, tries_all = 0, ncav_all = 0, nbnd_all = 0, won = 0, lost = 0;
    bool more = true;
    for (uint32_t round = 0; round < SEED_ROUNDS; ++round) {
        if (mine == 0 && more) {
            uint32_t got = 0;
            if (gl == 0) got = atomicAdd(&s.next, 1u);
            got = __shfl(got, (int)gbase);
            more = got < nverts;
            mine = more ? got : 0u;
            start = LGHOST;
            tries = 0;
        }
        if (!__syncthreads_or(mine != 0) || s.full) break;
        const uint32_t S = ((SEED_ROUNDS - round) << (SEED_VBITS + 1)) | (mine << 1);
        bool cand = false, drop = false, later = false;
        uint32_t ncav = 0, nbnd = 0;
        if (mine) {
            ++tries;
            const P3 P = seed_pt(s, mine);
            // start: the tetrahedron found before if it is live, else at the nearest of 64
            // vertices spread over those before this one, as far as they are inserted
            if (start == LGHOST || s.v[start].x == LDEAD) {
                double best = INFINITY;
                uint32_t bt = 0;
                for (int k = 0; k < 2; ++k) {
                    const uint32_t v = (gl + SEED_LANES * k) * (mine - 1) / (2 * SEED_LANES - 1);
                    const uint32_t h = s.hint[v];
                    if (h == LGHOST) continue;
                    const P3 Q = seed_pt(s, v);
                    const double d = (Q.x - P.x) * (Q.x - P.x) + (Q.y - P.y) * (Q.y - P.y) + (Q.z - P.z) * (Q.z - P.z);
                    if (d < best) {
                        best = d;
                        bt = h;
                    }
                }
                for (int o = SEED_LANES / 2; o > 0; o >>= 1) {
                    const double d = __shfl_xor(best, o, 64);
                    const uint32_t t = __shfl_xor(bt, o, 64);
                    if (d < best || (d == best && t < bt)) {
                        best = d;
                        bt = t;
                    }
                }
                start = bt;
            }
            uint32_t t = start;
            if (s.v[t].w == LGHOST) t = s.n[t].w >> 2;
            // walk: lane j < 4 tests facet j
            int entry = -1;
            const int jl = (int)(gl & 3u);
            bool in_ghost = false;
            for (unsigned ws = 0;; ++ws) {
                int o = 1;
                const ushort4 tn = s.n[t];
                if (gl < 4 && jl != entry) {
                    const ushort4 tv = s.v[t];
                    P3 q[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) q[k] = k == jl ? P : seed_pt(s, at4(tv, k));
                    o = seed_orient(q[0], q[1], q[2], q[3], st);
                }
                const unsigned out = (unsigned)((__ballot(o < 0) & gmask) >> gbase) & 0xFu;
                if (!out) {
                    drop = (__ballot(o == UNSURE) & gmask) != 0;  // on a facet's plane, or close
                    break;
                }
                if (ws >= SEED_WALK) {
                    later = true;
                    break;
                }
                ++walk;
                const unsigned rot = (mine + ws) & 3u;
                const unsigned rb = ((out >> rot) | (out << (4u - rot))) & 0xFu;
                const uint32_t cd = at4(tn, (int)(((unsigned)__ffs(rb) - 1u + rot) & 3u));
                t = cd >> 2;
                entry = (int)(cd & 3u);
                if (s.v[t].w == LGHOST) {
                    in_ghost = true;
                    break;
                }
            }
            start = t;
            if (!drop && !later && !in_ghost) {
                bool same = false;
                if (gl < 4) {
                    const P3 Q = seed_pt(s, at4(s.v[t], jl));
                    same = Q.x == P.x && Q.y == P.y && Q.z == P.z;
                }
                drop = (__ballot(same) & gmask) != 0;  // a duplicate is for the rounds to find
            }
            // cavity: four tetrahedra per step, lane (entry, facet)
            bool beaten = false;
            if (!drop && !later) {
                uint32_t found = ~0u;
                if (gl == 0) {
                    found = atomicMin(&s.claim[t], S);
                    s.cav[gi][0] = (uint16_t)(4 * t);
                }
                beaten = (__ballot(gl == 0 && found < S) & gmask) != 0;
                ncav = 1;
                __asm__ volatile("" ::: "memory");
                for (uint32_t k0 = 0, np = 0; k0 < ncav && !beaten && !drop; k0 += np) {
                    np = min((uint32_t)SEED_LANES / 4, ncav - k0);
                    const uint32_t e = k0 + (gl >> 2);
                    const int f = jl;
                    const uint32_t cd = e < k0 + np ? s.cav[gi][e] : 0u;
                    const uint32_t c = cd >> 2;
                    const bool act = e < k0 + np && (e == 0 || f != (int)(cd & 3u));
                    const ushort4 cv = s.v[c];
                    const uint32_t ncode = entry4(s.n, 4 * c + f), u = ncode >> 2;
                    const uint32_t word = act ? s.claim[u] : S;
                    bool inside = false, outside = act && word == S + 1, unsure = false;
                    if (act && word != S && word != S + 1) {
                        // One orient3d and one insphere for all cases (lanes of different
                        // cases would run one after the other):
                        //   c finite, u finite: insphere of facet f of c and the apex across
                        //     it (negatively oriented: the sign turned)
                        //   c finite, u ghost: inside iff P is beyond facet f
                        //   c ghost, u ghost: inside iff P is beyond u's finite facet
                        //   c ghost, u finite: insphere of u
                        const bool cghost = cv.w == LGHOST;
                        const ushort4 uv = s.v[u];
                        const uint32_t apex = at4(uv, (int)(ncode & 3u));
                        const bool plane = cghost ? uv.w == LGHOST : apex == LGHOST;
                        const bool swapped = !cghost && !plane;  // negatively oriented as it stands
                        uint32_t q[4];
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            q[k] = cghost ? at4(uv, k) : (k == f && !plane ? apex : at4(cv, k));
                        int side = 0;
                        if (plane) {
                            P3 r[4];
#pragma unroll
                            for (int k = 0; k < 4; ++k) r[k] = k == (cghost ? 3 : f) ? P : seed_pt(s, q[k]);
                            const int o = seed_orient(r[0], r[1], r[2], r[3], st);
                            side = o == UNSURE || !cghost ? o : -o;
                        }
                        if (!plane) {
                            side = seed_insphere(s, q, P, st);
                            if (swapped && side != UNSURE) side = -side;
                        }
                        inside = side < 0;
                        unsure = side == UNSURE;
                        const uint32_t old = unsure ? ~0u : atomicMin(&s.claim[u], inside ? S : S + 1);
                        // a lower claim this one cannot share; another lane of the group may
                        // have entered u through another facet (old == S)
                        beaten = old < S && (inside || !(old & 1u));
                        outside = !inside;
                        inside = inside && old != S;
                    }
                    const unsigned long long mi = __ballot(inside) & gmask, mo = __ballot(outside) & gmask;
                    beaten = (__ballot(beaten) & gmask) != 0;
                    const uint32_t ni = (uint32_t)__popcll(mi), no = (uint32_t)__popcll(mo);
                    drop = ncav + ni > SEED_CAV || nbnd + no > SEED_BND;
                    drop = drop || (__ballot(unsure) & gmask) != 0;
                    if (!drop && inside) s.cav[gi][ncav + (uint32_t)__popcll(mi & below)] = (uint16_t)ncode;
                    if (!drop && outside) {
                        const uint32_t b = nbnd + (uint32_t)__popcll(mo & below);
                        s.bnd[gi][b] = (uint16_t)(4 * c + f);
                        s.outer[gi][b] = (uint16_t)ncode;
                    }
                    ncav += ni;
                    nbnd += no;
                    __asm__ volatile("" ::: "memory");
                }
                cand = !beaten && !drop;
            }
        }
        __syncthreads();
        // winners hold every claim of their cavity, and no earlier point's cavity is next to it
        bool ok = cand;
        if (cand) {
            for (uint32_t k = gl; k < ncav; k += SEED_LANES) ok &= s.claim[s.cav[gi][k] >> 2] == S;
            for (uint32_t k = gl; k < nbnd; k += SEED_LANES) ok &= (s.claim[s.outer[gi][k] >> 2] & 1u) != 0;
        }
        const bool win = cand && (__ballot(!ok) & gmask) == 0;
        uint32_t fresh = 0;
        if (win) {
            // slots: the cavity's own, and more from the end
            if (gl == 0 && nbnd > ncav) {
                fresh = atomicAdd(&s.ntets, nbnd - ncav);
                if (fresh + (nbnd - ncav) > SEED_TETS) {
                    s.full = 1;
                    fresh = ~0u;
                }
            }
            fresh = __shfl(fresh, (int)gbase);
        }
        if (win && fresh != ~0u) {
            // the ball, as in the rounds; siblings by pivoting around each edge through the
            // cavity, whose records are all read before the first is overwritten
            constexpr int NB = (int)SEED_BND / SEED_LANES;
            for (uint32_t b = gl; b < nbnd; b += SEED_LANES) {
                s.slot[gi][b] = (uint16_t)(b < ncav ? s.cav[gi][b] >> 2 : fresh + (b - ncav));
                entry4(s.n, s.bnd[gi][b]) = (uint16_t)(LBOUND | b);
            }
            __asm__ volatile("" ::: "memory");
            uint32_t w[NB][4], nn[NB][4];
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const uint32_t b = gl + (uint32_t)(SEED_LANES * k);
                if (b < nbnd) {
                    const uint32_t cd = s.bnd[gi][b];
                    const int f = (int)(cd & 3u);
                    const ushort4 cv = s.v[cd >> 2];
#pragma unroll
                    for (int r = 0; r < 4; ++r) w[k][r] = r == f ? mine : at4(cv, r);
                    // the three pivots run side by side
                    uint32_t t[4], in[4], e0[4], e1[4];
                    unsigned open = 0xFu & ~(1u << f);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        nn[k][q] = s.outer[gi][b];
                        t[q] = cd >> 2;
                        in[q] = (uint32_t)f;
                        e0[q] = e1[q] = LGHOST;
                        bool first = true;
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (r != q && r != f) {
                                if (first) e0[q] = w[k][r];
                                else e1[q] = w[k][r];
                                first = false;
                            }
                    }
                    for (uint32_t guard = 0; open && guard <= SEED_CAV; ++guard) {
                        ushort4 tv[4], tn[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (open >> q & 1u) {
                                tv[q] = s.v[t[q]];
                                tn[q] = s.n[t[q]];
                            }
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (open >> q & 1u) {
                                uint32_t lc = tn[q].x;
#pragma unroll
                                for (uint32_t m = 0; m < 4; ++m) {
                                    const uint32_t x = at4(tv[q], (int)m);
                                    if (m != in[q] && x != e0[q] && x != e1[q]) lc = at4(tn[q], (int)m);
                                }
                                if (lc & LBOUND) {
                                    nn[k][q] = 4u * s.slot[gi][lc & (SEED_BND - 1)] + in[q];
                                    open &= ~(1u << q);
                                } else {
                                    t[q] = lc >> 2;
                                    in[q] = lc & 3u;
                                }
                            }
                    }
                    if (open) atomicOr(&ctr->error, ERR_WALK);  // a pivot without an end: never expected
                }
            }
            __asm__ volatile("" ::: "memory");
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const uint32_t b = gl + (uint32_t)(SEED_LANES * k);
                if (b < nbnd) {
                    const uint32_t slot = s.slot[gi][b];
                    entry4(s.n, s.outer[gi][b]) = (uint16_t)(4 * slot + (s.bnd[gi][b] & 3u));
                    s.v[slot] = make_ushort4((uint16_t)w[k][0], (uint16_t)w[k][1], (uint16_t)w[k][2], (uint16_t)w[k][3]);
                    s.n[slot] = make_ushort4((uint16_t)nn[k][0], (uint16_t)nn[k][1], (uint16_t)nn[k][2], (uint16_t)nn[k][3]);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (w[k][r] != LGHOST) s.hint[w[k][r]] = (uint16_t)slot;
                    }
                }
            }
            for (uint32_t k = nbnd + gl; k < ncav; k += SEED_LANES) s.v[s.cav[gi][k] >> 2].x = (uint16_t)LDEAD;
            ++won;
            ncav_all += ncav;
            nbnd_all += nbnd;
        } else if (mine) {
            ++lost;
        }
        const bool done = mine && (drop || (win && fresh != ~0u));
        if (done) {
            tries_all += tries;
            if (log_att && gl == 0) atomicAdd(&log_att[s.p[mine].pos - vlo], tries);
            mine = 0;
        }
    }
    if (mine) {
        tries_all += tries;
        if (log_att && gl == 0) atomicAdd(&log_att[s.p[mine].pos - vlo], tries);
    }
    if (gl == 0) {
        atomicAdd(&s.won, won);
        atomicAdd(&s.lost, lost);
        atomicAdd(&s.att, tries_all);
        atomicAdd(&s.walk, walk);
        atomicAdd(&s.ncav, ncav_all);
        atomicAdd(&s.nbnd, nbnd_all);
    }
    __syncthreads();

    // the mesh into the pool: the initial slots, then one range reserved for the rest.  Where
    // the pool has no room the cloud keeps its initial tetrahedron.
    const uint32_t nt = min(s.ntets, SEED_TETS);
    uint32_t live = 0;
    for (uint32_t t0 = 5; t0 < nt; t0 += SEED_THREADS) {
        const uint32_t t = t0 + tid;
        const bool ok = t < nt && s.v[t].x != LDEAD;
        uint32_t total;
        const uint32_t at = seed_count(s, ok, &total);
        if (t < nt) s.claim[t] = live + at;
        live += total;
    }
    if (tid == 0) {
        uint32_t cur = atomicAdd(&ctr->tet_count, 0u);
        s.base = NONE;
        while ((uint64_t)cur + live <= tcap) {
            const uint32_t was = atomicCAS(&ctr->tet_count, cur, cur + live);
            if (was == cur) {
                s.base = cur;
                break;
            }
            cur = was;
        }
    }
    __syncthreads();
    const uint32_t base = s.base;
    if (base == NONE) return;
    auto place = [&](uint32_t t) { return t < 5 ? c0 + t : base + s.claim[t]; };
    for (uint32_t t = tid; t < nt; t += SEED_THREADS) {
        uint32_t w[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] = at4(s.v[t], r);
        if (w[0] == LDEAD) {
            if (t < 5) T[c0 + t].v.x = DEAD;
            continue;
        }
        const uint32_t g = place(t);
        typename K::Rec *const rec = &T[g];
        rec->v = make_uint4(s.p[w[0]].pos, s.p[w[1]].pos, s.p[w[2]].pos, w[3] == LGHOST ? GHOST : s.p[w[3]].pos);
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            const uint32_t cd = at4(s.n[t], f);
            seed_nref(T, g, (uint32_t)f) = ((code)place(cd >> 2) << 2) | (code)(cd & 3u);
        }
        rec->claim = ~0ull;
        rec->spare[0] = 0;
        if (subd && w[3] != LGHOST)
            subd[g] = subdets(seed_pt(s, w[0]), seed_pt(s, w[1]), seed_pt(s, w[2]), seed_pt(s, w[3]));
    }
    for (uint32_t v = tid; v < nverts; v += SEED_THREADS)
        if (s.hint[v] != LGHOST) vtet[s.p[v].pos] = place(s.hint[v]);
    // statistics
    auto add = [&](int id, unsigned long long x) {
        if (x) atomicAdd(&stat[((size_t)id * STAT_SPREAD + (blockIdx.x % STAT_SPREAD)) * STAT_PAD], x);
    };
    uint32_t orient = st.orient, insphere = st.insphere;
    for (int o = 32; o > 0; o >>= 1) {
        orient += __shfl_xor(orient, o, 64);
        insphere += __shfl_xor(insphere, o, 64);
    }
    if (lane == 0) {
        add(STAT_ORIENT, orient);
        add(STAT_INSPHERE, insphere);
    }
    if (tid == 0) {
        cl->any_live = place(s.hint[0]);
        atomicAdd(&ctr->won, s.won);
        add(STAT_WON, s.won);
        atomicAdd(&ctr->conflicts, s.lost);
        add(STAT_ATTEMPTS, s.att);
        add(STAT_WALK, s.walk);
        add(STAT_CAV_TETS, s.ncav);
        add(STAT_BND_FACETS, s.nbnd);
    }
}

hipError_t launch_seed(const Vert *V, Cloud *clouds, uint32_t nclouds, uint32_t first_slot, const uint32_t *lord,
                       uint32_t nlord, const uint8_t *dup, void *T, bool wide, uint32_t tcap, uint32_t *vtet,
                       Ctr *ctr, void *subd, unsigned long long *stat, uint32_t *log_att, uint32_t vlo,
                       hipStream_t s) {
    if (nclouds == 0) return hipSuccess;
    if (wide)
        k_seed<Wide><<<nclouds, SEED_THREADS, 0, s>>>(V, clouds, first_slot, lord, nlord, dup, (TetW *)T, tcap, vtet,
                                                      ctr, (SubD *)subd, stat, log_att, vlo);
    else
        k_seed<Narrow><<<nclouds, SEED_THREADS, 0, s>>>(V, clouds, first_slot, lord, nlord, dup, (Tet *)T, tcap, vtet,
                                                        ctr, (SubD *)subd, stat, log_att, vlo);
    return hipGetLastError();
}

}  // namespace dtk
