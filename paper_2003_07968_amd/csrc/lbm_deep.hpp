#pragma once
// lbm_deep.hpp -- the deep pass: T time steps of a lattice or a batch in one
// launch, each step computed by waves of its own.
//
// A workgroup of T x BX threads owns a strip of columns and walks a segment
// of rows.  Its first BX lanes (four waves at BX = 256) compute step t from
// the populations in memory, the next BX lanes step t + 1 from what the first
// hand them through LDS, and so on; the last store step t + T - 1's result.
// The populations are read once and written once for T updates, so a pass
// needs 1/T of the memory traffic of single steps.  At every hand-over the
// values are rounded to the storage type, and every step calls the single
// step's routines (lbm_kernels.hpp) in the same order, so the result is
// bitwise that of single steps, the first domain error included.
//
// Why a step per wave: the two-step pass holds both steps in one thread (186
// registers in FP64); a third step would not fit, and its two steps wait for
// each other at three barriers a row.  Here a thread holds one step's rows
// (125 registers in FP64, 64 in FP32 and FP16, 73 per cell), all steps of a row
// run at once, and one barrier per row is enough: in iteration m a step pulls
// what the previous step wrote in iteration m - 1 and writes what the next
// step pulls in iteration m + 1.
//
// Iteration m of step j (a = m - lag is a row of its walk):
//   collides row a - 2: the force from the psi rows a - 3 .. a - 1 (own column
//   in registers, x-neighbours of row a - 1 from LDS), then hands the row to
//   the next step, or stores it;
//   pulls the nine populations of the previous step's newest row w from LDS
//   (the first step: takes the row loaded an iteration ago and loads the
//   next): those pulled from the walk's next row complete row w - 1 = a, those
//   of the row itself belong to row w, those pulled from the previous row to
//   row w + 1, and are held in registers until then;
//   turns row a into rho and psi and publishes psi.
// T is kDeepSteps, or one less for the three steps that a call may leave.
// A step's lag is 4 rows behind the previous step's; a tile needs 2T - 1
// halo columns and rows on each side, and n rows take n + 6T - 3 iterations.
//
// What bounds it (T = 4, 2048 x 8192, one MI355X; the two-step pass on the
// same lattice in parentheses): FP64 140 G cell updates/s (74), FP32 242
// (134), FP16 255 (185), per-cell FP16 186 (144).  A row update is 129
// (FP64), 125 (FP32), 139 (FP16) or 192 (per-cell) VALU instructions per wave.
// FP32 and the FP16 modes are at their issue rate (0.94 to 1.11 of one
// instruction per four cycles of every SIMD at 2.4 GHz).  FP64, with 16 waves
// per CU, issues at 0.54 of it, at a clock that FP64 arithmetic on all CUs
// holds at 1.96 GHz, and waits 25% of its wave-cycles; its HBM traffic, 1.02
// times one read and one write of the populations per launch, runs at 5.05
// TB/s, near a plain copy's rate (5.2).
//
// The MRT collision: FP64 117, FP32 197, FP16 210, per-cell 152.  It needs more
// registers than there are: four steps spill 9 to 12 vector registers in FP64
// (up to 44 bytes of scratch a lane, reloaded in the row loop) and 7 in FP32
// and FP16, and 22 to 82 scalar ones.  BGK spills no vector registers; scalar
// ones, into vector lanes, 2 (FP64; batched 7) and 11 (FP32, FP16; batched
// 28).  The per-cell mode, compiled for 128 registers, spills none.
//
// What the issue rate needed, each measured on that lattice in FP64:
//   LDS addressed by byte offset from four registers (the compiler kept an
//   address register per row and spilled them: 247 us per step, 148 after);
//   the coefficients as kernel arguments, so that they sit in scalar
//   registers (formed in the kernel they occupied 26 vector registers);
//   one barrier per row instead of two (per-cell FP16 115 -> 101 us);
//   wave priorities (144 -> 128 us): waves collide at high priority and turn
//   their next row into psi at low priority, so that at the end of an
//   iteration all four waves of a SIMD still have independent work; left to
//   the oldest-first order, the last wave ran its whole iteration alone.  The
//   waves that load and store come first, so that their accesses are issued
//   while the others compute.
#include "lbm_kernels.hpp"

namespace lbmk {

// Halo columns (and rows) of a tile on each side: a step depends on the cells
// within two of a cell, but the first step's own pull is made by its loads.
template <int T>
constexpr int kHaloT = 2 * T - 1;

// LDS of a tile, in rows of BX elements: one region per step, holding two
// rows of its psi and two rows of what it hands to the next step, its nine
// post-collision populations (rounded to the storage type) and, in the
// per-cell mode, the new reference.  A row is written in one iteration and
// read in the next.  Accessed by byte offset (lds_at), so that one register
// per lane and the instructions' immediate offsets address everything.
template <class R, int BX, int T, bool LOC>
struct DeepLds {
    static constexpr int kRow = BX * (int)sizeof(R);
    static constexpr int kPsi = 0, kPops = 2 * kRow, kRef = 20 * kRow,
                         kRegion = kRef + (LOC ? 2 * BX * 4 : 0);
    // FP32: the first step keeps six rows of psi
    static constexpr bool kRing = sizeof(R) == 4;
    static constexpr int kLead = kRing ? 4 * kRow : 0;
    char bytes[kLead + (T - 1) * kRegion + 2 * kRow];
};

template <class V>
__device__ __forceinline__ __attribute__((address_space(3))) V &lds_at(uint32_t addr)
{
    return *(__attribute__((address_space(3))) V *)(uintptr_t)addr;
}

// Waves per SIMD the deep pass is compiled for: two workgroups of 256 columns
// per CU with FP32 and FP16 storage (64 registers; one per CU, 83 registers:
// FP32 74 us per step instead of 68), one in FP64 (128 registers) and in the
// per-cell mode (75; at 64 it spills and takes 120 us instead of 96).
template <int ST>
constexpr int kDeepWaves =
    ST == LBM_STORE_F32_SHIFTED || ST == LBM_STORE_F16_SHIFTED ? 8 : 4;

enum Role { kFirst, kMid, kLast };

// Calls f(integral_constant<int, J>) for J = 0 .. N-1 while it returns true.
template <class F, int... J>
__device__ __forceinline__ bool unroll_while(F &&f, std::integer_sequence<int, J...>)
{
    return (f(std::integral_constant<int, J>{}) && ...);
}

// Makes an address register unknown to the compiler here, in place: what is
// added to it below goes into the instructions' immediate offsets instead of
// being formed once in registers of its own.
__device__ __forceinline__ void opaque(uint32_t &v) { asm("" : "+v"(v)); }

// Coefficients formed by vector instructions, moved to scalar registers.  The
// empty asm statement makes the value look divergent: a readfirstlane of a
// value known to be uniform is dropped, and the value stays in vector
// registers of every wave.
template <class V>
__device__ __forceinline__ V in_scalar_registers(const V &v)
{
    static_assert(sizeof(V) % 4 == 0);
    struct Words {
        int w[sizeof(V) / 4];
    };
    Words a = __builtin_bit_cast(Words, v);
#pragma unroll
    for (int &w : a.w) {
        asm("" : "+v"(w));
        w = __builtin_amdgcn_readfirstlane(w);
    }
    return __builtin_bit_cast(V, a);
}

// The stored values that load_pulled pulls, unconverted (a conversion would
// wait for the load), with the three lattice rows given (r - 1, r, r + 1).
template <int ST, class E = typename Store<ST>::E>
__device__ __forceinline__ void load_rows(const E *__restrict__ src, const Coeffs &c, int rm, int r,
                                          int rp, const Cols &x, E d[kQ])
{
    const size_t P = c.plane;
    const E *row_r = src + (size_t)r * c.pitch;
    const E *row_m = src + (size_t)rm * c.pitch;
    const E *row_p = src + (size_t)rp * c.pitch;
    d[0] = ld<E, E>(row_r, x.o);
    d[1] = ld<E, E>(row_r + 1 * P, x.m);
    d[2] = ld<E, E>(row_m + 2 * P, x.o);
    d[3] = ld<E, E>(row_r + 3 * P, x.p);
    d[4] = ld<E, E>(row_p + 4 * P, x.o);
    d[5] = ld<E, E>(row_m + 5 * P, x.m);
    d[6] = ld<E, E>(row_m + 6 * P, x.p);
    d[7] = ld<E, E>(row_p + 7 * P, x.p);
    d[8] = ld<E, E>(row_p + 8 * P, x.m);
}

// Step j of a tile's walk (role: the first step loads, the last stores).
// `checked` lanes hold columns whose psi is one of the tile's at this step,
// `interior` ones output columns; `bad` receives the lowest cell index outside
// the EOS domain.
template <int BX, int T, int ROLE, int ST, int COLL, int DIR>
__device__ __forceinline__ void deep_stage(
    const typename Store<ST>::E *__restrict__ src, typename Store<ST>::E *__restrict__ dst,
    const Coeffs &c, const Phys<typename Store<ST>::R> &P, int j, int y0, int n, int x,
    const Cols &cols, bool checked, bool interior, uint32_t lds, uint32_t &bad)
{
    using E = typename Store<ST>::E;
    using R = typename Store<ST>::R;
    constexpr bool LOC = Store<ST>::local;
    constexpr int H = kHaloT<T>;
    constexpr bool fwd = DIR > 0;
    const R gref = (R)c.rho_ref;
    using L = DeepLds<R, BX, T, LOC>;
    const uint32_t tx = threadIdx.x & (BX - 1);
    const uint32_t txm = (tx + BX - 1) & (BX - 1), txp = (tx + 1) & (BX - 1);
    // byte addresses of the own lane's and its neighbours' elements: of this
    // step's region to write (w), of the previous step's to pull from (po, pm,
    // pp; the first step's own)
    constexpr bool RING = L::kRing && ROLE == kFirst;
    const uint32_t own = lds + (ROLE == kFirst ? 0 : L::kLead + j * L::kRegion),
                   prev = ROLE == kFirst ? own : own - L::kRegion;
    constexpr int kOut = RING ? L::kLead : 0;  // own region from w
    uint32_t w = own + tx * (uint32_t)sizeof(R), po = prev + tx * (uint32_t)sizeof(R),
             pm = prev + txm * (uint32_t)sizeof(R), pp = prev + txp * (uint32_t)sizeof(R);
    // (FP32: the own region is within reach of the immediate offsets from po)
    constexpr bool kFromPo = ROLE == kMid && sizeof(R) == 4;
    constexpr int kOwn = kFromPo ? L::kRegion : 0;
    constexpr int kPsiOff = ROLE == kFirst ? 0 : L::kRegion;  // own psi rows from pm, pp
    // populations pulled from the walk's previous row (back) and next row:
    // the vertical one, the diagonal one that moves right (read from lane
    // txm), the one that moves left (from txp)
    constexpr int kB0 = fwd ? 2 : 4, kBr = fwd ? 5 : 8, kBl = fwd ? 6 : 7;
    constexpr int kA0 = fwd ? 4 : 2, kAr = fwd ? 8 : 5, kAl = fwd ? 7 : 6;
    auto lrow = [&](int s) {
        const int r = (y0 + DIR * s) % c.ny;
        return r < 0 ? r + c.ny : r;
    };
    auto step_row = [&](int r) {
        if (fwd) return r + 1 == c.ny ? 0 : r + 1;
        return r - 1 + ((r - 1) >> 31 & c.ny);
    };
    auto recon = [&](R g[kQ], const Tri<R> &back, const Tri<R> &cur, const Tri<R> &ahead) {
        if constexpr (fwd)
            reconstruct<R>(g, back, cur, ahead);
        else
            reconstruct<R>(g, ahead, cur, back);
    };
    auto load_tri = [&](int r) {
        const float *row = ref_row(src, c, r);
        return Tri<R>{ld<float, R>(row, 2 * cols.m), ld<float, R>(row, 2 * cols.o),
                      ld<float, R>(row, 2 * cols.p)};
    };

    // Iteration m collides row a - 2 and turns row a = m - lag into psi.  Rows
    // lo .. hi of psi are the rows whose update this step's successors or
    // outputs need, and one more on each side.
    R f[2][kQ];              // rows a - 2, a - 1
    E raw[2][kQ];            // first step: row a as loaded, row a + 1 in flight
    R here[3], back[2][3];   // pulled ahead of time: 1 and 2 iterations
    Row<R> rw[3];            // psi of rows a - 3, a - 2, a - 1
    Tri<R> tr[3], tn;        // per-cell mode: R of rows a - 1, a, a + 1
    R refs[2];               // and of the rows in f
    const int lag = H + 4 * j;
    const int lo = -H + 2 * j, hi = n - 1 + H - 2 * j;
    const int a0 = ROLE == kFirst ? lo : lo - 2;
    int rpsi = lrow(a0);                    // lattice row turned into psi
    [[maybe_unused]] int rstore = lrow(0);  // lattice row stored next
    // the row loaded next and its neighbours in the walk
    [[maybe_unused]] int rback = lrow(lo), rload = lrow(lo + 1), rahead = lrow(lo + 2);

    if constexpr (ROLE == kFirst) {
        load_rows<ST>(src, c, fwd ? lrow(lo - 1) : rload, rback, fwd ? rload : lrow(lo - 1), cols,
                      raw[0]);
        if constexpr (LOC) {
            tr[1] = load_tri(lrow(lo - 1));
            tr[2] = load_tri(rback);
            tn = load_tri(rload);
        }
    }

    auto body = [&](auto Jc, int m) {
        constexpr int J = decltype(Jc)::value;  // m % 6
        constexpr int cur = J % 2;
        const int a = m - lag;
        // Values that an iteration outside a0 .. hi + 2 leaves unset are not used.
        R g[kQ], nhere[3], nback[3], nref;
        Row<R> last = rw[(J + 2) % 3], lead;
        Tri<R> nt;
        if (a >= a0 && a <= hi + 2) {
            __builtin_amdgcn_s_setprio(ROLE == kLast ? 3 : (ROLE == kFirst ? 2 : 1));
            if constexpr (!kFromPo) opaque(w);
            opaque(po);
            opaque(pm);
            opaque(pp);
            constexpr int in = (J + 1) % 2, out = J % 2;  // LDS rows of the last and this iteration
            if constexpr (!RING) {
                last.l = lds_at<R>(pm + kPsiOff + in * L::kRow);
                last.r = lds_at<R>(pp + kPsiOff + in * L::kRow);
            }
            // collision of row a - 2
            const Row<R> &C = rw[(J + 1) % 3];
            R sv[kQ], Fx, Fy, ux, uy, Jx, Jy;
            if constexpr (RING) {
                // the first step, which holds a third row of populations, has
                // no registers for the window (64 with two workgroups per CU)
                auto row = [&](int k) {
                    const int o = (J + 6 - k) % 6 * L::kRow;
                    return Row<R>{lds_at<R>(pm + o), lds_at<R>(po + o), lds_at<R>(pp + o), R(0)};
                };
                stencil<DIR, R>(row(3), row(2), row(1), sv);
            } else {
                stencil<DIR, R>(rw[J % 3], C, last, sv);
            }
            force<R>(sv, P, Fx, Fy);
            R h[kQ];
#pragma unroll
            for (int i = 0; i < kQ; ++i)
                h[i] = f[cur][i];
            const R ref = LOC ? refs[J % 2] : gref;
            velocity<R>(h, C.rho, Fx, Fy, ux, uy, Jx, Jy);
            if constexpr (COLL == LBM_COLL_MRT)
                collide_mrt<R>(h, C.rho, ux, uy, Jx, Jy, Fx, Fy, P);
            else
                collide<R>(h, ref, C.rho, ux, uy, Jx, Jy, Fx, Fy, P);
            E X[kQ];
            float newref = 0.0f;
            if constexpr (LOC) {
                const R sd =
                    (((h[0] + h[1]) + (h[2] + h[3])) + ((h[4] + h[5]) + (h[6] + h[7]))) + h[8];
                R err = R(0);
#pragma unroll
                for (int i = 0; i < kQ; ++i) {
                    const R wt = i == 0 ? R(4.0 / 9.0) : (i < 5 ? R(1.0 / 9.0) : R(1.0 / 36.0));
                    h[i] = fma(-wt, sd, h[i]);
                }
                to_stored<E, R>(h, X);
#pragma unroll
                for (int i = 0; i < kQ; ++i)
                    err += h[i] - (R)X[i];
                newref = (float)(ref + (sd + err));
            } else {
                to_stored<E, R>(h, X);
            }
            if constexpr (ROLE == kLast) {
                if (interior && a >= 2 && a < n + 2) {
                    store_pops<E>(dst, c, rstore, cols.o, X);
                    if constexpr (LOC)
                        __builtin_nontemporal_store(
                            newref,
                            (float *)((char *)ref_row(dst, c, rstore) + col_offset(2 * cols.o)));
                }
                if (a >= 2) rstore = step_row(rstore);
            } else {
                constexpr int q = kOut + kOwn + L::kPops + out * 9 * L::kRow;
                const uint32_t to = kFromPo ? po : w;
                lds_at<R>(to + q) = (R)X[kA0];
                lds_at<R>(to + q + L::kRow) = (R)X[kAr];
                lds_at<R>(to + q + 2 * L::kRow) = (R)X[kAl];
                lds_at<R>(to + q + 3 * L::kRow) = (R)X[0];
                lds_at<R>(to + q + 4 * L::kRow) = (R)X[1];
                lds_at<R>(to + q + 5 * L::kRow) = (R)X[3];
                lds_at<R>(to + q + 6 * L::kRow) = (R)X[kB0];
                lds_at<R>(to + q + 7 * L::kRow) = (R)X[kBr];
                lds_at<R>(to + q + 8 * L::kRow) = (R)X[kBl];
                if constexpr (LOC)
                    lds_at<float>(own + kOut + L::kRef + out * BX * 4 + 4 * tx) = newref;
            }
            if constexpr (ROLE == kFirst) {
                // row a + 1 into the registers of the row that is done, ahead
                // of row a's arithmetic; past the last row it is loaded again,
                // from cache
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (LOC) nt = tn;
                load_rows<ST>(src, c, fwd ? rback : rahead, rload, fwd ? rahead : rback, cols,
                              raw[(J + 1) % 2]);
                if constexpr (LOC) tn = load_tri(rahead);
                if (a + 1 < hi) {
                    rback = rload;
                    rload = rahead;
                    rahead = step_row(rahead);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            R next[3];
            if constexpr (ROLE != kFirst) {
                // pulled only now: before the collision there are no registers
                // for nine more values
                __builtin_amdgcn_sched_barrier(0);
                opaque(po);
                opaque(pm);
                opaque(pp);
                constexpr int q = L::kPops + in * 9 * L::kRow;
                next[0] = lds_at<R>(po + q);
                next[1] = lds_at<R>(pm + q + L::kRow);
                next[2] = lds_at<R>(pp + q + 2 * L::kRow);
                nhere[0] = lds_at<R>(po + q + 3 * L::kRow);
                nhere[1] = lds_at<R>(pm + q + 4 * L::kRow);
                nhere[2] = lds_at<R>(pp + q + 5 * L::kRow);
                nback[0] = lds_at<R>(po + q + 6 * L::kRow);
                nback[1] = lds_at<R>(pm + q + 7 * L::kRow);
                nback[2] = lds_at<R>(pp + q + 8 * L::kRow);
                if constexpr (LOC) {
                    const uint32_t r = prev + L::kRef + in * BX * 4;
                    nt = Tri<R>{(R)lds_at<float>(r + 4 * txm), (R)lds_at<float>(r + 4 * tx),
                                (R)lds_at<float>(r + 4 * txp)};
                }
            }
            __builtin_amdgcn_s_setprio(0);
            // row a: rho and psi
            if constexpr (ROLE == kFirst) {
#pragma unroll
                for (int i = 0; i < kQ; ++i)
                    g[i] = (R)raw[J % 2][i];
            } else {
                g[kA0] = next[0];
                g[kAr] = next[1];
                g[kAl] = next[2];
                g[0] = here[0];
                g[1] = here[1];
                g[3] = here[2];
                g[kB0] = back[J % 2][0];
                g[kBr] = back[J % 2][1];
                g[kBl] = back[J % 2][2];
            }
            nref = gref;
            if constexpr (LOC) {
                recon(g, tr[(J + 1) % 3], tr[(J + 2) % 3], nt);
                nref = tr[(J + 2) % 3].o;
            }
            const bool ok = rho_psi<1, R>(g, nref, P, lead.rho, lead.o);
            if (!ok && checked && a >= lo && a <= hi)
                bad = min(bad, (uint32_t)rpsi * (uint32_t)c.nx + (uint32_t)x);
            rpsi = step_row(rpsi);
            lds_at<R>((kFromPo ? po : w) + kOwn + (RING ? J : out) * L::kRow) = lead.o;
        }
#pragma unroll
        for (int i = 0; i < kQ; ++i)
            f[cur][i] = g[i];
        if constexpr (ROLE != kFirst) {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                here[i] = nhere[i];
                back[J % 2][i] = nback[i];
            }
        }
        rw[(J + 2) % 3] = last;
        rw[J % 3] = lead;
        if constexpr (LOC) {
            tr[J % 3] = nt;
            refs[J % 2] = nref;
        }
        __syncthreads();
    };

    // the same count for every step: the barriers are the workgroup's
    const int total = n + 6 * T - 3;
    for (int m = 0;; m += 6)
        if (!unroll_while([&](auto J) {
                constexpr int k = decltype(J)::value;
                body(J, m + k);
                return m + k + 1 < total;
            }, std::make_integer_sequence<int, 6>{}))
            break;
}

// A tile's walk: columns [xs, xe), n rows from y0 in direction DIR.
template <int BX, int T, int ST, int COLL, int DIR>
__device__ __forceinline__ void deep_walk(const void *__restrict__ src_v, void *__restrict__ dst_v,
                                          const Coeffs &c, const Phys<typename Store<ST>::R> &P,
                                          int xs, int xe, int y0, int n, uint32_t lds, long long t,
                                          unsigned long long *__restrict__ err)
{
    using E = typename Store<ST>::E;
    constexpr int H = kHaloT<T>;
    const int j = __builtin_amdgcn_readfirstlane((int)threadIdx.x / BX);
    // lane tx holds column xs - H + pos: the output columns in lanes 0 ..
    // width - 1, the right halo after them and the left halo in the last H
    const int pos = (int)(((threadIdx.x & (BX - 1)) + H) & (BX - 1));
    const int width = xe - xs;
    const bool checked = pos >= 2 * j && pos < width + 2 * H - 2 * j;
    const bool interior = pos >= H && pos < width + H;
    int x = (xs - H + (pos < width + 2 * H ? pos : H)) % c.nx;
    x = x < 0 ? x + c.nx : x;
    const int xm = wrap_lo(x - 1, c.nx), xp = wrap_hi(x + 1, c.nx);
    constexpr uint32_t es = sizeof(E);
    const Cols cols{(uint32_t)x * es, (uint32_t)xm * es, (uint32_t)xp * es};
    uint32_t bad = ~0u;
    if (j == 0)
        deep_stage<BX, T, kFirst, ST, COLL, DIR>((const E *)src_v, (E *)dst_v, c, P, 0, y0, n, x,
                                                 cols, checked, interior, lds, bad);
    else if (j == T - 1)
        deep_stage<BX, T, kLast, ST, COLL, DIR>((const E *)src_v, (E *)dst_v, c, P, T - 1, y0, n, x,
                                                cols, checked, interior, lds, bad);
    else
        deep_stage<BX, T, kMid, ST, COLL, DIR>((const E *)src_v, (E *)dst_v, c, P, j, y0, n, x, cols,
                                               checked, interior, lds, bad);
    if (bad != ~0u) atomicMin(err, ((unsigned long long)(t + j) << 32) | bad);
}

// One tile of the deep pass: output strip `strip` of row band `seg`; odd
// bands walk down the lattice, as in the other passes.
template <int BX, int T, int ST, int COLL>
__device__ __forceinline__ void deep_tile(const void *__restrict__ src, void *__restrict__ dst,
                                          const Coeffs &c, const Phys<typename Store<ST>::R> &P,
                                          const Tiles &tl, int tile, long long t,
                                          unsigned long long *__restrict__ err)
{
    static_assert((BX & (BX - 1)) == 0, "ring of lanes needs a power-of-two width");
    __shared__ __align__(16) DeepLds<typename Store<ST>::R, BX, T, Store<ST>::local> lds_mem;
    const uint32_t lds =
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds_mem.bytes;
    const int seg = tile / tl.nstrips;
    const int strip = tile - seg * tl.nstrips;
    const int xs = strip * tl.width;
    const int xe = min(c.nx, xs + tl.width);
    const int ys = (int)((long long)seg * c.ny / tl.nseg);
    const int ye = (int)((long long)(seg + 1) * c.ny / tl.nseg);
    if (seg & 1)
        deep_walk<BX, T, ST, COLL, -1>(src, dst, c, P, xs, xe, ye - 1, ye - ys, lds, t, err);
    else
        deep_walk<BX, T, ST, COLL, 1>(src, dst, c, P, xs, xe, ys, ye - ys, lds, t, err);
}

// The deep pass over one lattice.
template <int BX, int T, int ST, int COLL>
__global__ __launch_bounds__(BX *T, (kDeepWaves<ST>)) void deep_kernel(const void *__restrict__ src,
                                                     void *__restrict__ dst, Coeffs c,
                                                     Phys<typename Store<ST>::R> P, Tiles tl,
                                                     long long t,
                                                     unsigned long long *__restrict__ err)
{
    deep_tile<BX, T, ST, COLL>(src, dst, c, P, tl, xcd_tile(blockIdx.x, tl.ntiles), t, err);
}

// The deep pass over every lattice of a batch, `steps` steps after the table was
// written, from the buffers of this parity.
template <int BX, int T, int ST, int COLL>
__global__ __launch_bounds__(BX *T, (kDeepWaves<ST>)) void batch_deep_kernel(
    const BatchEntry *__restrict__ table, int nlat, long long steps, int parity)
{
    const BatchTile k = batch_tile<&BatchEntry::tile0_4, &BatchEntry::tl4>(
        table, nlat, xcd_tile(blockIdx.x, gridDim.x), steps, parity);
    const auto P = in_scalar_registers(Phys<typename Store<ST>::R>(k.c));
    deep_tile<BX, T, ST, COLL>(k.src, k.dst, k.c, P, k.tl, k.tile, k.t, k.err);
}

#define LBM_WIDTHSD(X) X(64) X(128) X(256)

template <int T, int ST, int COLL>
hipError_t deep_launch_bx(const SweepArgs &a)
{
    const dim3 grid((unsigned)a.tl.ntiles);
    switch (a.bx) {
#define LBM_CASE(BX)                                                                          \
    case BX:                                                                                  \
        hipLaunchKernelGGL((deep_kernel<BX, T, ST, COLL>), grid, dim3(BX *T), 0, a.stream, a.src, a.dst, a.c,              \
                           Phys<typename Store<ST>::R>(a.c), a.tl, a.t, a.err);                                                            \
        break;
        LBM_WIDTHSD(LBM_CASE)
#undef LBM_CASE
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int ST, int T>
hipError_t launch_deep(const SweepArgs &a)
{
    return a.c.coll == LBM_COLL_MRT ? deep_launch_bx<T, ST, LBM_COLL_MRT>(a)
                                    : deep_launch_bx<T, ST, LBM_COLL_BGK>(a);
}

template <int T, int ST, int COLL>
hipError_t batch_deep_launch_bx(const BatchArgs &a)
{
    switch (a.bx) {
#define LBM_CASE(BX)                                                                          \
    case BX:                                                                                  \
        hipLaunchKernelGGL((batch_deep_kernel<BX, T, ST, COLL>), dim3(a.grid), dim3(BX *T),    \
                           0, a.stream, a.table, a.nlat, a.steps_add, a.launches_add & 1);    \
        break;
        LBM_WIDTHSD(LBM_CASE)
#undef LBM_CASE
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int ST, int T>
hipError_t launch_batch_deep(const BatchArgs &a)
{
    return a.coll == LBM_COLL_MRT ? batch_deep_launch_bx<T, ST, LBM_COLL_MRT>(a)
                                  : batch_deep_launch_bx<T, ST, LBM_COLL_BGK>(a);
}

}  // namespace lbmk
