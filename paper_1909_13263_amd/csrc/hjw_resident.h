// hjw_resident.h - many RK3 steps of one grid in a single launch, with phi held on the chip.
//
// A grid whose tiles all fit on the GPU at once needs neither a launch per stage nor a round
// trip of phi, phi_2 and the flux records through memory: each workgroup keeps its tile in
// LDS (the stage input) and registers (phi^n) from step to step, and only the three outermost
// layers of a tile go to its neighbours, through mailboxes in memory.  One step is
//   sweeps of phi^n; flux records of the tile's border to the neighbours; the derivative
//   box reduced over all workgroups; every workgroup plans the step;
//   phi_1 on the tile and, from the received records, on its halo; sweeps; phi_2 border;
//   sweeps; phi^{n+1} border.
//
// Mailboxes.  Every 8-byte word carries its own tag (the step's number), written and read
// with relaxed device-scope atomics, so a received word is known to be the current one by
// itself: no flags, no fences, one store and one load between two tiles.  A word is
// overwritten one step later at the earliest, and by then its reader has passed a later
// exchange with (or a reduction that includes) the writer: flux, phi_2 and phi^{n+1} have
// mailboxes of their own, so between two uses of one the neighbour has answered on another.
//
// All workgroups must be on the GPU together.  The launch starts with a rendezvous that
// either all of them pass or none: the last to arrive opens it, and one that waits longer
// than kJoinTicks closes it, whereupon every workgroup (also one that starts later) leaves
// without having changed anything and the host steps with the launches per stage.  Once all
// have arrived every later wait ends; the waits are bounded all the same.
// What bounds it.  On small grids a step is a chain of latencies: 256^2 (256 tiles of 64 x 4, FP32
// stencil) takes 14.3 us a step = sweeps 1.9, finishes and phi_1 2.8, the box reduced over all tiles
// and the plan 5.1, two border exchanges 3.0, barriers and the rest 1.5.  At 1024^2 (four 64 x 16
// tiles a compute unit) it is the issue of vector instructions: a wave instruction takes 4 cycles
// of its SIMD here (the counters give 1.04 quad-cycles each), and they keep the vector units busy
// for 0.88 of the launch; the launches per stage take 38 us a step, this one 30.  Whole solves,
// launches per stage -> this launch: Burgers 1024^2 8.1 -> 6.6 ms (FP32 stencil), 1-D N = 160
// 0.92 -> 0.26 ms, Dirichlet 80^2 FP64 7.9 -> 3.0 ms, level set 512^2 FP64 8.7 -> 7.2 ms.
// Nodes' results and phi^n stay in LDS, not in registers, from sweep to finish: with them in
// registers the unrolled finishes of three stages and all families were 118 KB of code with
// scratch traffic, and a 1024^2 step took 50 us.  Borders are sent from LDS in the mailboxes'
// order, whole lines a wave; sent node by node from the finish they made it 64 us.
#pragma once

#include "hjw_kernels.h"

namespace hjw {

// n nodes over nb tiles whose sizes differ by one at most, so that no tile of a split axis is
// narrower than the three layers it sends.
struct Split {
    int nb, base, extra;
    __host__ __device__ int start(int i) const { return i * base + (i < extra ? i : extra); }
    __host__ __device__ int size(int i) const { return base + (i < extra ? 1 : 0); }
};
inline Split split_axis(int64_t n, int most) {
    const int nb = int((n + most - 1) / most);
    return Split{nb, int(n / nb), int(n % nb)};
}

constexpr int kResidentTX1 = 255, kResidentThreads1 = 256;   // 1-D: nodes and threads of a tile
constexpr int kGroup = 64;          // workgroups whose ranges one leader reduces
constexpr int kMaxResident = 1024;  // workgroups of a launch (16 groups)
enum { kWest = 0, kEast, kSouth, kNorth };

struct ResidentCtl {
    unsigned int arrived;   // workgroups at the rendezvous
    unsigned int go;        // 0 waiting, 1 all arrived, 2 given up
    unsigned int fail;      // a wait ran out after the rendezvous
    unsigned int pad;
};

struct ResidentArgs {
    Split sx, sy;
    unsigned long long* flux_mail;   // [tile][word][element]
    unsigned long long* mid_mail;    // phi_2
    unsigned long long* last_mail;   // phi^{n+1}
    unsigned long long* ranges;      // [step parity][quantity, half][workgroup]
    unsigned long long* groups;      // [step parity][copy][quantity, half][group]
    ResidentCtl* ctl;
    DevState* state;                 // the grid's step records
    unsigned int epoch;              // the tag of the launch's first step; never 0
    int max_steps;
    int count;                       // workgroups
    int remap;
    int meet;                        // workgroups the rendezvous waits for
    int looks;                       // of a wait, before it gives up
};

// One tile of the launch: its nodes and, per side, whether a neighbouring tile sends the halo
// (else it comes from the tile itself: wrapped, or extrapolated at the grid's edge).
struct Spot {
    int tile, x0, y0, w, h;
    int sides;        // bit `side`: a neighbour sends that side
    bool any_local;
    int west, east, south, north;   // the neighbouring tiles
    __host__ __device__ bool remote(int side) const { return (sides >> side) & 1; }
    __host__ __device__ int nbr(int side) const {   // (an array indexed by side would live in scratch)
        const int x = side == kWest ? west : east, y = side == kSouth ? south : north;
        return side < kSouth ? x : y;
    }
};
__host__ __device__ inline Spot make_spot(const ResidentArgs& r, int tile, int dim, int bcx,
                                          int bcy) {
    Spot s;
    s.tile = tile;
    const int nbx = r.sx.nb, nby = r.sy.nb;
    const int ix = tile % nbx, iy = tile / nbx;
    s.x0 = r.sx.start(ix);
    s.y0 = r.sy.start(iy);
    s.w = r.sx.size(ix);
    s.h = r.sy.size(iy);
    const bool px = bcx == kBcPeriodic, py = bcy == kBcPeriodic;
    s.sides = (nbx > 1 && (ix > 0 || px) ? 1 << kWest : 0) |
              (nbx > 1 && (ix < nbx - 1 || px) ? 1 << kEast : 0) |
              (nby > 1 && (iy > 0 || py) ? 1 << kSouth : 0) |
              (nby > 1 && (iy < nby - 1 || py) ? 1 << kNorth : 0);
    s.any_local = s.sides != (dim == 2 ? 15 : 3);
    s.west = iy * nbx + (ix > 0 ? ix - 1 : nbx - 1);
    s.east = iy * nbx + (ix < nbx - 1 ? ix + 1 : 0);
    s.south = (iy > 0 ? iy - 1 : nby - 1) * nbx + ix;
    s.north = (iy < nby - 1 ? iy + 1 : 0) * nbx + ix;
    return s;
}

// ------------------------------------------------------------------ tagged words
__device__ inline void put_word(unsigned long long* p, unsigned long long w) {
    __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__host__ inline void put_word(unsigned long long* p, unsigned long long w) { *p = w; }
__device__ inline unsigned long long get_word(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__host__ inline unsigned long long get_word(const unsigned long long* p) { return *p; }

using u64 = unsigned long long;
__host__ __device__ inline u64 bits_of(double x) { return __builtin_bit_cast(u64, x); }
__host__ __device__ inline u64 bits_of(float x) { return __builtin_bit_cast(uint32_t, x); }

// A value in words of 32 data bits and a 32-bit tag.
template <typename V>
struct Tagged {
    static constexpr int kWords = sizeof(V) / 4;
    u64 w[kWords];
    __host__ __device__ static Tagged make(V v, unsigned int tag) {
        Tagged t;
        const u64 b = bits_of(v), hi = u64(tag) << 32;
        t.w[0] = (b & 0xffffffffull) | hi;
        if (kWords == 2) t.w[kWords - 1] = (b >> 32) | hi;
        return t;
    }
    __host__ __device__ bool is(unsigned int tag) const {
        return uint32_t(w[0] >> 32) == tag && uint32_t(w[kWords - 1] >> 32) == tag;
    }
    __host__ __device__ V value() const {
        if constexpr (kWords == 2)
            return __builtin_bit_cast(V, (w[0] & 0xffffffffull) | (w[1] << 32));
        else
            return __builtin_bit_cast(V, uint32_t(w[0]));
    }
};
// A flux record in words of 48 data bits and a 16-bit tag: its three values' bits end to end.
template <typename T>
struct TaggedFlux {
    static constexpr int kWords = sizeof(T) == 8 ? 4 : 2;
    u64 w[kWords];
    __host__ __device__ static TaggedFlux make(const Flux3<T>& f, unsigned int tag) {
        TaggedFlux t;
        const u64 a = bits_of(f.h), b = bits_of(f.dx), c = bits_of(f.dy);
        const u64 top = u64(tag) << 48, low = 0xffffffffffffull;
        if constexpr (kWords == 4) {
            t.w[0] = (a & low) | top;
            t.w[1] = (b & low) | top;
            t.w[2] = (c & low) | top;
            t.w[3] = (a >> 48) | ((b >> 48) << 16) | ((c >> 48) << 32) | top;
        } else {
            t.w[0] = a | ((b & 0xffffull) << 32) | top;
            t.w[1] = c | ((b >> 16) << 32) | top;
        }
        return t;
    }
    __host__ __device__ bool is(unsigned int tag) const {
        bool ok = true;
        for (int q = 0; q < kWords; ++q) ok = ok && (w[q] >> 48) == (tag & 0xffffu);
        return ok;
    }
    __host__ __device__ Flux3<T> value() const {
        const u64 low = 0xffffffffffffull;
        Flux3<T> f;
        if constexpr (kWords == 4) {
            f.h = __builtin_bit_cast(T, (w[0] & low) | (w[3] << 48));
            f.dx = __builtin_bit_cast(T, (w[1] & low) | ((w[3] >> 16) << 48));
            f.dy = __builtin_bit_cast(T, (w[2] & low) | ((w[3] >> 32) << 48));
        } else {
            f.h = __builtin_bit_cast(T, uint32_t(w[0]));
            f.dx = __builtin_bit_cast(T, uint32_t((w[0] >> 32) & 0xffffu) |
                                             uint32_t((w[1] >> 32) & 0xffffu) << 16);
            f.dy = __builtin_bit_cast(T, uint32_t(w[1]));
        }
        return f;
    }
};

// ------------------------------------------------------------------ a tile's borders
// Geometry of the tile in LDS: own node (c, r) at phiL[(r + 3 HALO_Y) * PITCH + c + 3], where a
// 1-D tile has no rows around it.  A mailbox holds the halo's elements: three columns of TY
// on the west and the east, three rows of TX on the south and the north.
template <typename T, typename P, int TX, int TY, int PITCH, int DIM, int THREADS>
struct Border {
    static constexpr int kRow0 = DIM == 2 ? 3 : 0;
    static constexpr int kSouth0 = 6 * TY, kNorth0 = 6 * TY + 3 * TX;
    static constexpr int kElems = 6 * TY + (DIM == 2 ? 6 * TX : 0);
    static constexpr int kRounds = (kElems + THREADS - 1) / THREADS;

    __host__ __device__ static int own(int c, int r) { return (r + kRow0) * PITCH + c + 3; }

    // The border's elements in the order in which they are sent, so that a wave's stores fill
    // whole lines of a neighbour's mailbox: three columns to the west, three to the east, three
    // rows to the south, three to the north.
    struct Out {
        int side, c, r, el;   // own node, and its element of that neighbour's mailbox
    };
    __host__ __device__ static bool outgoing(const Spot& s, int o, Out& x) {
        if (o >= kElems) return false;
        if (o < kSouth0 || DIM == 1) {
            const int k = o / TY;
            x.r = o % TY;
            x.side = k < 3 ? kWest : kEast;
            x.c = k < 3 ? k : s.w - 6 + k;
            x.el = (k < 3 ? 3 + k : k - 3) * TY + x.r;
            return x.r < s.h && s.remote(x.side);
        }
        const int f = o - kSouth0, k = f / TX;
        x.c = f % TX;
        x.side = k < 3 ? kSouth : kNorth;
        x.r = k < 3 ? k : s.h - 6 + k;
        x.el = kSouth0 + (k < 3 ? 3 + k : k - 3) * TX + x.c;
        return x.c < s.w && s.remote(x.side);
    }
    template <class Rec>
    __host__ __device__ static void put(const Spot& s, const Out& x, const Rec& rec, u64* mail) {
        u64* p = mail + int64_t(s.nbr(x.side)) * (Rec::kWords * kElems) + x.el;
        for (int q = 0; q < Rec::kWords; ++q) put_word(p + q * kElems, rec.w[q]);
    }
    // Thread t's share (of `threads`) of the tile's border of phi.
    __host__ __device__ static void send_phi(int t, int threads, const Spot& s, const P* phiL,
                                             unsigned int tag, u64* mail) {
        for (int o = t; o < kElems; o += threads) {
            Out x;
            if (outgoing(s, o, x)) put(s, x, Tagged<P>::make(phiL[own(x.c, x.r)], tag), mail);
        }
    }
    // The same of its flux records, which lie in three arrays of one value a node: f(c, r).
    template <class At>
    __host__ __device__ static void send_flux(int t, int threads, const Spot& s, At f,
                                              unsigned int tag, u64* mail) {
        for (int o = t; o < kElems; o += threads) {
            Out x;
            if (outgoing(s, o, x)) put(s, x, TaggedFlux<T>::make(f(x.c, x.r), tag), mail);
        }
    }

    // The LDS element of mailbox element el, or -1 where no neighbour sends it.
    __host__ __device__ static int place(const Spot& s, int el) {
        if (el < kSouth0 || DIM == 1) {
            const int k = el / TY, r = el % TY;
            if (el >= kElems || r >= s.h || !s.remote(k < 3 ? kWest : kEast)) return -1;
            return (r + kRow0) * PITCH + (k < 3 ? k : s.w + k);
        }
        const int f = el - kSouth0, k = f / TX, c = f % TX;
        if (el >= kElems || c >= s.w || !s.remote(k < 3 ? kSouth : kNorth)) return -1;
        return (k < 3 ? k : s.h + k) * PITCH + c + 3;
    }

    // Halo sides that no neighbour sends, from the tile's own nodes: thread tid's share.
    __host__ __device__ static void fill_local(int tid, const Spot& s, const StageArgs<T, P>& a,
                                               P* phiL) {
        for (int el = tid; el < kElems; el += THREADS) {
            if (el < kSouth0 || DIM == 1) {
                const int k = el / TY, r = el % TY;
                if (r >= s.h || s.remote(k < 3 ? kWest : kEast)) continue;
                P v;
                if (a.bcx == kBcPeriodic) {
                    v = phiL[own(k < 3 ? s.w - 3 + k : k - 3, r)];
                } else {
                    const int e = k < 3 ? 0 : s.w - 1, in = k < 3 ? 1 : s.w - 2;
                    v = extrapolate(phiL[own(e, r)], phiL[own(in, r)], k < 3 ? 3 - k : k - 2);
                }
                phiL[(r + kRow0) * PITCH + (k < 3 ? k : s.w + k)] = v;
            } else {
                const int f = el - kSouth0, k = f / TX, c = f % TX;
                if (c >= s.w || s.remote(k < 3 ? kSouth : kNorth)) continue;
                P v;
                if (a.bcy == kBcPeriodic) {
                    v = phiL[own(c, k < 3 ? s.h - 3 + k : k - 3)];
                } else {
                    const int e = k < 3 ? 0 : s.h - 1, in = k < 3 ? 1 : s.h - 2;
                    v = extrapolate(phiL[own(c, e)], phiL[own(c, in)], k < 3 ? 3 - k : k - 2);
                }
                phiL[(k < 3 ? k : s.h + k) * PITCH + c + 3] = v;
            }
        }
    }

    // phi^n of the tile and its halo from memory (the launch's start); the rest of the tile,
    // which no node of the grid reads, is zero so that its marches stay on the short path.
    template <int LDS>
    __host__ __device__ static void load(int tid, const Spot& s, const StageArgs<T, P>& a,
                                         P* phiL) {
        for (int e = tid; e < LDS; e += THREADS) {
            const int r = e / PITCH - kRow0, c = e % PITCH - 3;
            const bool in_x = c >= 0 && c < s.w, in_y = r >= 0 && r < s.h;
            const bool halo_x = c >= -3 && c < s.w + 3, halo_y = DIM == 2 && r >= -3 && r < s.h + 3;
            P v = P(0);
            if ((halo_x && in_y) || (in_x && halo_y))
                v = stage_value<kStagePre>(a, int64_t(s.x0 + c), int64_t(s.y0 + r), 0.0, 0.0, 0.0);
            phiL[e] = v;
        }
    }

    // phi_1 at a node from phi^n and its flux record: node_value() of the second stage.
    __host__ __device__ static P phi1(P pn, const Flux3<T>& f, double dt, double ax, double ay) {
        const double rr = double(f.h) - (mul_rn(ax, double(f.dx)) + mul_rn(ay, double(f.dy)));
        return P(fma(-dt, rr, double(pn)));
    }

    // Thread t's share (of `threads`) of the halo that neighbours send, received whole before
    // any of it is used: the loads of a round trip are in flight together.
    template <class Rec, int ROUNDS>
    struct Received {
        Rec rec[ROUNDS];
        int at[ROUNDS];
        bool open[ROUNDS];   // expected and not here yet
    };
    template <class Rec, int ROUNDS>
    __host__ __device__ static void expect(int t, int threads, const Spot& s,
                                           Received<Rec, ROUNDS>& g) {
#pragma unroll
        for (int k = 0; k < ROUNDS; ++k) {
            g.at[k] = place(s, t + k * threads);
            g.open[k] = g.at[k] >= 0;
        }
    }
    // One look at the mailbox, at what has not come yet; whether everything has.
    template <class Rec, int ROUNDS>
    __host__ __device__ static bool look(int t, int threads, const Spot& s, unsigned int tag,
                                         const u64* mail, Received<Rec, ROUNDS>& g) {
        const u64* box = mail + int64_t(s.tile) * (Rec::kWords * kElems);
#pragma unroll
        for (int k = 0; k < ROUNDS; ++k) {
            const int el = t + k * threads;
            if (!g.open[k]) continue;
            for (int q = 0; q < Rec::kWords; ++q) g.rec[k].w[q] = get_word(box + q * kElems + el);
        }
        bool ok = true;
#pragma unroll
        for (int k = 0; k < ROUNDS; ++k) {
            if (g.open[k] && g.rec[k].is(tag)) g.open[k] = false;
            ok = ok && !g.open[k];
        }
        return ok;
    }
};

// The sweeps of a resident 2-D tile: as the stage kernels', but the columns' results go to LDS
// too, so that every node's four derivatives lie there, and a finish may take its nodes in any
// order, in a loop, with nothing of theirs in registers from stage to stage.
// S = 0: a thread per cell instead of a thread per segment (65 cells a row, TY + 1 a column):
// the march is one cell long.  On tiles of four rows that takes 640 threads, and no cell is
// computed twice.  Against two nodes a thread (three cells, 256 threads): 48^2 13.6 -> 12.1 us a
// step (FP64 17.7 -> 16.3), 128^2 12.8 -> 11.8, Dirichlet 80^2 FP64 19.3 -> 17.8; in 1-D, where a
// thread marched one node (two cells), N = 160 8.0 -> 6.0, N = 5000 11.2 -> 9.3.
constexpr int cell_waves_x(int ty) { return (ty * (kTX + 1) + 63) / 64; }
constexpr int resident_threads2d(int ty, int seg) {
    return seg == 0 ? 64 * (cell_waves_x(ty) + ty + 1) : threads2d(ty, seg);
}
template <typename T, typename P, int TY, int S>
struct ResidentTile {
    using TL = Tile<T, P, kTX, TY, S ? S : 2, S ? S : 2>;
    static constexpr int kThreads = resident_threads2d(TY, S);
    static constexpr int kNodes = kTX * TY;
    static constexpr int kVElems = 2 * kNodes;
    static_assert(kThreads <= 1024 && kNodes % 64 == 0, "one workgroup, rows are waves");

    template <int SEG, class Out>
    __host__ __device__ static void march(const P* line, int stride, const StageArgs<T, P>& a, P ih,
                                          T ihT, T eps, const Out& out) {
        if (a.scheme == kSchemeJP)
            sweep_emit<T, P, SEG, kSchemeJP>(line, stride, ih, ihT, eps, out);
        else
            sweep_emit<T, P, SEG, kSchemeL>(line, stride, ih, ihT, eps, out);
    }
    // Both sweeps, thread id's share.
    __host__ __device__ static void sweeps(int id, const StageArgs<T, P>& a, const P* phiL, T* uL,
                                           T* vL) {
        if constexpr (S == 0) {
            constexpr int kX = 64 * cell_waves_x(TY);
            // the cell's left side is the node before it, its right side the node at it
            struct Cell {
                T *m, *p;
                bool right, left;
                __host__ __device__ void minus(int, T v) const { if (right) *m = v; }
                __host__ __device__ void plus(int, T v) const { if (left) *p = v; }
            };
            if (id < kX) {
                const int q = id < TY * (kTX + 1) ? id : 0;   // idle threads repeat the first cell
                const int row = q / (kTX + 1), c = q % (kTX + 1);
                T* u = uL + row * TL::UW + c;
                march<0>(phiL + (row + 3) * TL::PW + c, 1, a, a.ihx, a.ihxT, a.epsx,
                         Cell{u, u + TY * TL::UW - 1, id == q && c < kTX, id == q && c > 0});
            } else {
                const int q = id - kX, it = q / kTX, col = q % kTX;
                T* v = vL + it * kTX + col;
                march<0>(phiL + it * TL::PW + col + 3, TL::PW, a, a.ihy, a.ihyT, a.epsy,
                         Cell{v, v + kNodes - kTX, it < TY, it > 0});
            }
        } else if (id < TL::kHalf) {
            TL::sweep_x(id, a, phiL, uL);
        } else {
            const int t = id - TL::kHalf, col = t % kTX, seg = t / kTX;
            struct ToLds {
                T* base;
                __host__ __device__ void minus(int k, T v) const { base[k * kTX] = v; }
                __host__ __device__ void plus(int k, T v) const { base[kNodes + k * kTX] = v; }
            };
            march<S>(phiL + seg * S * TL::PW + col + 3, TL::PW, a, a.ihy, a.ihyT, a.epsy,
                     ToLds{vL + seg * S * kTX + col});
        }
    }
    // The node's places in uL and vL; once its derivatives have been read, its flux record
    // takes three of the four.
    __host__ __device__ static int u_at(int c, int r) { return r * TL::UW + c; }
    __host__ __device__ static int v_at(int c, int r) { return r * kTX + c; }
    __host__ __device__ static void put_flux(T* uL, T* vL, int c, int r, const Flux3<T>& f) {
        uL[u_at(c, r)] = f.h;
        uL[TY * TL::UW + u_at(c, r)] = f.dx;
        vL[v_at(c, r)] = f.dy;
    }
    __host__ __device__ static Flux3<T> get_flux(const T* uL, const T* vL, int c, int r) {
        return Flux3<T>{uL[u_at(c, r)], uL[TY * TL::UW + u_at(c, r)], vL[v_at(c, r)]};
    }
    // One node's finish from LDS.
    template <int MODE, class Fin>
    __host__ __device__ static void node(Fin& fin, int c, int r, const T* uL, const T* vL, P ps,
                                         P pn) {
        fin.template node<MODE>(c, r, uL[u_at(c, r)], uL[TY * TL::UW + u_at(c, r)], vL[v_at(c, r)],
                                vL[kNodes + v_at(c, r)], ps, pn);
    }
};

// A 1-D tile: a thread a cell (one more than nodes), then a thread a node.
template <typename T, typename P>
struct ResidentTile1D {
    static constexpr int PW = kResidentTX1 + 7;   // 255 nodes and their halos, and one spare
    static constexpr int kPhiElems = PW;
    static constexpr int kUElems = 2 * kResidentThreads1;
    __host__ __device__ static void sweep(int t, const StageArgs<T, P>& a, const P* phiL, T* uL) {
        struct Cell {
            T* u;
            bool left;
            __host__ __device__ void minus(int, T v) const { u[0] = v; }
            __host__ __device__ void plus(int, T v) const { if (left) u[kUElems / 2 - 1] = v; }
        };
        const Cell out{uL + t, t > 0};
        if (a.scheme == kSchemeJP)
            sweep_emit<T, P, 0, kSchemeJP>(phiL + t, 1, a.ihx, a.ihxT, a.epsx, out);
        else
            sweep_emit<T, P, 0, kSchemeL>(phiL + t, 1, a.ihx, a.ihxT, a.epsx, out);
    }
};

// Keeps what a node's finish hands on instead of storing it.
template <typename T, typename P>
struct Kept {
    Flux3<T> f;
    P v;
    __host__ __device__ void flux(const StageArgs<T, P>&, int64_t, uint32_t, const Flux3<T>& rec) {
        f = rec;
    }
    __host__ __device__ void phi(const StageArgs<T, P>&, int64_t, uint32_t, P val) { v = val; }
};

// The kernel of a resident launch (hjw_resident.hip): tiles of 64 x ty nodes marched in segments
// of seg (ignored in 1-D); own: with the time-dependent family and the local dissipation.
const void* resident_kernel(int prec, int dim, int ty, int seg, bool own);

// Words of the reductions' areas and of one tile's mailboxes.
template <typename T>
constexpr int range_words() {
    return 4 * Tagged<T>::kWords;
}
template <typename T, typename P>
constexpr size_t mail_words(int elems) {
    return size_t(elems) * (TaggedFlux<T>::kWords + 2 * Tagged<P>::kWords);
}

#ifdef __HIPCC__
// ------------------------------------------------------------------ waits (device)
constexpr int64_t kJoinTicks = 50000;    // 0.5 ms of the 100 MHz wall clock
constexpr int kMaxLooks = 1 << 21;       // a second or more

template <int NW>
struct ResidentShared {
    DevState st;
    double red[NW][4];
    int red_bad[NW];
    int fail;
    int go;
    int active;
};

// Whether all workgroups of the launch are on the GPU (thread 0 of each).
__device__ inline int resident_join(const ResidentArgs& r) {
    const unsigned int before =
        __hip_atomic_fetch_add(&r.ctl->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    unsigned int want = 0;
    if (before + 1 == unsigned(r.meet))
        __hip_atomic_compare_exchange_strong(&r.ctl->go, &want, 1u, __ATOMIC_RELAXED,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const long long t0 = wall_clock64();
    for (int k = 0; k < kMaxLooks; ++k) {
        const unsigned int go =
            __hip_atomic_load(&r.ctl->go, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (go) return int(go);
        if (wall_clock64() - t0 > kJoinTicks) break;
        __builtin_amdgcn_s_sleep(2);
    }
    want = 0;
    __hip_atomic_compare_exchange_strong(&r.ctl->go, &want, 2u, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
    return int(__hip_atomic_load(&r.ctl->go, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// Calls look() until every lane of the wave has what it waits for; false when the wait ran
// out or another workgroup's did.
template <class Look>
__device__ inline bool wait_for(const ResidentArgs& r, Look look) {
    for (int k = 0;; ++k) {
        if (__all(look() ? 1 : 0)) return true;
        if ((k & 1023) == 1023 &&
            __hip_atomic_load(&r.ctl->fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u)
            return false;
        if (k >= r.looks) {
            __hip_atomic_store(&r.ctl->fail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

// The derivative box over n workgroups (or groups): lane l holds the l-th one's four values
// (a NaN in the first marks a non-finite node).
template <typename T>
struct Box {
    T v[4];
    bool bad;
};
template <typename T>
__device__ inline bool gather_box(const ResidentArgs& r, const u64* words, int pitch, int n,
                                  unsigned int tag, Box<T>& b) {
    const int lane = threadIdx.x % 64;
    constexpr int H = Tagged<T>::kWords;
    Tagged<T> w[4];
    const bool on = lane < n;
    const bool ok = wait_for(r, [&] {
        bool all = true;
        if (on) {
            for (int q = 0; q < 4; ++q)
                for (int h = 0; h < H; ++h) w[q].w[h] = get_word(words + (q * H + h) * pitch + lane);
            for (int q = 0; q < 4; ++q) all = all && w[q].is(tag);
        }
        return all;
    });
    for (int q = 0; q < 4; ++q)
        b.v[q] = on ? w[q].value() : (q & 1) ? T(-INFINITY) : T(INFINITY);
    b.bad = __any(b.v[0] != b.v[0]) != 0;
    b.v[0] = wave_min(b.v[0]);
    b.v[1] = wave_max(b.v[1]);
    b.v[2] = wave_min(b.v[2]);
    b.v[3] = wave_max(b.v[3]);
    return ok;
}
// Quantity q of a box as it is sent: a NaN in the first says that a node was not finite.
template <typename T>
__device__ inline T box_word(const Box<T>& b, int q) {
    const T v = q == 0 ? b.v[0] : q == 1 ? b.v[1] : q == 2 ? b.v[2] : b.v[3];
    return q == 0 && b.bad ? T(NAN) : v;
}
template <typename T>
__device__ inline void publish_box(u64* words, int pitch, int at, const Box<T>& b,
                                   unsigned int tag) {
    constexpr int H = Tagged<T>::kWords;
    const int q = threadIdx.x % 64;
    if (q < 4) {
        const Tagged<T> t = Tagged<T>::make(box_word(b, q), tag);
        for (int h = 0; h < H; ++h) put_word(words + (q * H + h) * pitch + at, t.w[h]);
    }
}

// The box over the whole grid, from this workgroup's own (first wave, all lanes).
template <typename T>
__device__ inline bool reduce_box(const ResidentArgs& r, int tile, int step, Box<T>& b) {
    if (r.count == 1) return true;
    const unsigned int tag = r.epoch + unsigned(step);
    // two sets by step parity: a workgroup that has passed this reduction may publish its next
    // range while one far away still reads this one, but not the one after that
    u64* ranges = r.ranges + (step & 1) * (range_words<T>() * r.count);
    publish_box(ranges, r.count, tile, b, tag);
    if (r.count <= kGroup) return gather_box(r, ranges, r.count, r.count, tag, b);
    // Every group has a copy of its own of all groups' boxes, so that at most kGroup workgroups
    // look at one line; a leader writes its box to all copies at once, a lane each.
    constexpr int H = Tagged<T>::kWords, kCopy = range_words<T>() * (kMaxResident / kGroup);
    const int ng = (r.count + kGroup - 1) / kGroup;
    u64* groups = r.groups + (step & 1) * (kCopy * (kMaxResident / kGroup));
    if (tile % kGroup == 0) {
        const int n = r.count - tile < kGroup ? r.count - tile : kGroup;
        if (!gather_box(r, ranges + tile, r.count, n, tag, b)) return false;
        const int lane = threadIdx.x % 64, copy = lane / 4;
        static_assert(kMaxResident / kGroup * 4 == 64, "a lane per copy and quantity");
        const Tagged<T> t = Tagged<T>::make(box_word(b, lane % 4), tag);
        if (copy < ng)
            for (int h = 0; h < H; ++h)
                put_word(groups + copy * kCopy + (lane % 4 * H + h) * ng + tile / kGroup, t.w[h]);
    }
    groups += tile / kGroup * kCopy;
    return gather_box(r, groups, ng, ng, tag, b);
}

// Step plan of this workgroup (first wave): the record in sh.st becomes the step's.
template <int NW, typename T, typename P>
__device__ inline void resident_plan(const StageArgs<T, P>& a, const ResidentArgs& r, int tile,
                                     int step, ResidentShared<NW>& sh) {
    Box<T> b;
    double v[4] = {sh.red[0][0], sh.red[0][1], sh.red[0][2], sh.red[0][3]};
    int bad = sh.red_bad[0];
    for (int k = 1; k < NW; ++k) {
        v[0] = fmin(v[0], sh.red[k][0]);
        v[1] = fmax(v[1], sh.red[k][1]);
        v[2] = fmin(v[2], sh.red[k][2]);
        v[3] = fmax(v[3], sh.red[k][3]);
        bad |= sh.red_bad[k];
    }
    for (int q = 0; q < 4; ++q) b.v[q] = T(v[q]);
    b.bad = bad != 0;
    const bool ok = reduce_box(r, tile, step, b);
    if (threadIdx.x == 0) {
        if (!ok) sh.fail = 1;
        const double box[4] = {double(b.v[0]), double(b.v[1]), double(b.v[2]), double(b.v[3])};
        if (b.bad ||
            !(finite_t(box[0]) && finite_t(box[1]) && finite_t(box[2]) && finite_t(box[3])))
            sh.st.bad = 1;
        else
            plan_step(sh.st, a.ham, a.hpD, a.dim, a.ihxD, a.ihyD, box);
        sh.active = sh.st.bad ? 0 : 1;
    }
}

// This workgroup's part of the derivative box into LDS.
template <int NW, typename T>
__device__ inline void resident_fold(ResidentShared<NW>& sh, T lu, T hu, T lv, T hv, bool bad) {
    lu = wave_min(lu);
    hu = wave_max(hu);
    lv = wave_min(lv);
    hv = wave_max(hv);
    const bool any = __any(bad) != 0;
    if (threadIdx.x % 64 == 0) {
        const int w = threadIdx.x / 64;
        sh.red[w][0] = double(lu);
        sh.red[w][1] = double(hu);
        sh.red[w][2] = double(lv);
        sh.red[w][3] = double(hv);
        sh.red_bad[w] = any ? 1 : 0;
    }
}

// The launch's end: the record of the last step and the non-finite flag.
template <typename T, typename P>
__device__ inline void resident_close(const StageArgs<T, P>& a, const ResidentArgs& r, int tile,
                                      const DevState& s, int fail, bool bad) {
    DevState& out = a.st[a.par];
    if (threadIdx.x == 0) {
        if (tile == 0) {
            out.t = s.t;
            out.dt = s.dt;
            out.alpha_x = s.alpha_x;
            out.alpha_y = s.alpha_y;
            for (int k = 0; k < 4; ++k) out.range[k] = s.range[k];
            out.steps = s.steps;
            out.steps_left = s.steps_left;
        }
        atomicMax(&out.pad[0], fail ? 2 : 1);
        if (s.bad) atomicOr(&out.bad, 1);
    }
    if (__any(bad) && threadIdx.x % 64 == 0) atomicOr(&out.bad, 1);
}

// Resets the rendezvous and the outcome; with set, also the step target.  With next, the launch
// follows another whose outcome the host has not seen: unless that one ran to its end, the
// rendezvous starts closed, and the launch leaves the outcome as it is.
static __global__ void k_resident_begin(DevState* st, ResidentCtl* ctl, int set, double t_final,
                                        double cfl, int64_t steps_left, int next) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        if (next && st->pad[0] != 1) {
            ctl->go = 2u;
            return;
        }
        ctl->arrived = 0u;
        ctl->go = 0u;
        ctl->fail = 0u;
        st->pad[0] = 0;
        if (set) {
            st->t_final = t_final;
            st->cfl = cfl;
            st->steps_left = steps_left;
            st->active = 0;
        }
    }
}

static __global__ void k_clear_words(unsigned long long* w, int64_t n) {
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += int64_t(gridDim.x) * blockDim.x)
        w[i] = 0ull;
}

// The thread's index, taken afresh: what is derived from it is formed where it is used, and
// not kept in registers across a loop over stages.
__device__ inline int fresh(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

// Waves per SIMD asked of the resident kernels.
constexpr int resident_waves(int elem, int ty, int seg) {
    return seg == 0 ? 3 : elem == 8 && ty == 16 ? 3 : 4;
}

template <typename T, typename P, int TY, int S, bool TIMED>
__global__ __launch_bounds__(resident_threads2d(TY, S), resident_waves(sizeof(T), TY, S)) void k_resident2d(
    StageArgs<T, P> a, ResidentArgs r) {
    using RT = ResidentTile<T, P, TY, S>;
    using TL = typename RT::TL;
    using BD = Border<T, P, kTX, TY, TL::PW, 2, RT::kThreads>;
    constexpr int NW = RT::kThreads / 64;
    __shared__ P phiL[TL::kPhiElems];
    __shared__ P pnL[RT::kNodes];   // phi^n of the tile's nodes
    __shared__ T uL[TL::kUElems];
    __shared__ T vL[RT::kVElems];
    __shared__ ResidentShared<NW> sh;
    __shared__ DevState sh_tn;   // t_n of the step, for the time-dependent family
    const int tid = threadIdx.x;
    __builtin_assume(tid >= 0 && tid < RT::kThreads);
    const Spot s = make_spot(r, tile_of_block(int(blockIdx.x), r.count, r.remap), 2, a.bcx, a.bcy);
    if (tid == 0) {
        sh.go = resident_join(r);
        sh.st = a.st[a.par];
        sh.fail = 0;
        sh.active = 0;
    }
    BD::template load<TL::kPhiElems>(tid, s, a, phiL);
    __syncthreads();
    if (sh.go != 1) return;   // uniform over the launch
    if (!(step_open(sh.st) && r.max_steps > 0)) {
        if (s.tile == 0 && tid == 0) atomicMax(&a.st[a.par].pad[0], 1);
        return;   // uniform over the launch too: every workgroup read the same record
    }
    if constexpr (TIMED) {   // the finishes read t_n of the step from LDS
        a.st = &sh_tn;
    }
    const int par = a.par;
    if constexpr (TIMED) a.par = 0;

    // Calls f(column, row) for the thread's nodes inside the grid.
    auto each_node = [&](auto f) {
        const int id = fresh(tid);
        const int c = id % kTX;
        if (c >= s.w) return;
        int row = uniform_int(id / kTX);
#pragma unroll 1
        for (; row < s.h; row += RT::kThreads / kTX) f(c, row);
    };
    for (int e = tid; e < RT::kNodes; e += RT::kThreads)
        pnL[e] = phiL[BD::own(e % kTX, e / kTX)];
    double dt = 0.0, ax = 0.0, ay = 0.0;
    bool bad = false;       // a non-finite phi^{n+1} of the last step taken, here
    int step = 0, stage = 0;

    // fin over the thread's nodes; hand(c, row, kept) for each
    auto finish = [&](auto& fin, auto hand) {
        fin.room_x = s.w;
        fin.room_y = s.h;
        const auto nodes = [&](auto mode) {
            each_node([&](int c, int row) {
                RT::template node<decltype(mode)::value>(fin, c, row, uL, vL,
                                                         phiL[BD::own(c, row)], pnL[row * kTX + c]);
                hand(c, row, fin.sink);
            });
        };
        const int mode = fin.mode();
        if constexpr (TIMED) {
            if (mode == kNodeTimed) {
                nodes(std::integral_constant<int, kNodeTimed>{});
                return;
            }
        }
        if (mode == kNodeExtended)
            nodes(std::integral_constant<int, kNodeExtended>{});
        else
            nodes(std::integral_constant<int, kNodePlain>{});
    };
    // the border of phi_2 or phi^{n+1} to the neighbours, and theirs
    auto exchange = [&](u64* mail, unsigned int tag) {
        __syncthreads();
        BD::send_phi(fresh(tid), RT::kThreads, s, phiL, tag, mail);
        typename BD::template Received<Tagged<P>, BD::kRounds> got;
        const int id = fresh(tid);
        BD::expect(id, RT::kThreads, s, got);
        if (!wait_for(r, [&] { return BD::look(id, RT::kThreads, s, tag, mail, got); }))
            sh.fail = 1;
#pragma unroll
        for (int k = 0; k < BD::kRounds; ++k)
            if (got.at[k] >= 0) phiL[got.at[k]] = got.rec[k].value();
    };
    auto settle = [&] {
        if (s.any_local) {
            __syncthreads();
            BD::fill_local(fresh(tid), s, a, phiL);
        }
        __syncthreads();
    };

#pragma unroll 1
    for (;;) {
        const unsigned int tag = r.epoch + unsigned(step);
        const int id = fresh(tid);
        __builtin_assume(id >= 0 && id < RT::kThreads);
        RT::sweeps(id, a, phiL, uL, vL);
        if (TIMED && stage == 0 && tid == 0) sh_tn.t = sh.st.t;
        __syncthreads();
        if (stage == 0) {
            Finisher<kStagePre, T, P, TIMED, Kept<T, P>> fin(a, s.x0, s.y0, 0.0, 0.0, 0.0, 2);
            finish(fin, [&](int c, int row, const Kept<T, P>& k) {
                RT::put_flux(uL, vL, c, row, k.f);
            });
            resident_fold(sh, fin.lo_u, fin.hi_u, fin.lo_v, fin.hi_v, fin.bad || bad);
            __syncthreads();
            // the first wave reduces the box and plans while the others exchange the records
            constexpr int kOthers = RT::kThreads - 64;
            constexpr int kFluxRounds = (BD::kElems + kOthers - 1) / kOthers;
            typename BD::template Received<TaggedFlux<T>, kFluxRounds> got;
            if (tid < 64) {
                resident_plan(a, r, s.tile, step, sh);
            } else {
                const int el = fresh(tid) - 64;
                BD::send_flux(el, kOthers, s, [&](int c, int row) {
                    return RT::get_flux(uL, vL, c, row);
                }, tag, r.flux_mail);
                BD::expect(el, kOthers, s, got);
                if (!wait_for(r, [&] {
                        return BD::look(el, kOthers, s, tag, r.flux_mail, got);
                    }))
                    sh.fail = 1;
            }
            __syncthreads();
            if (sh.fail || !sh.active) break;
            dt = sh.st.dt;
            ax = sh.st.alpha_x;
            ay = sh.st.alpha_y;
            if (tid >= 64) {
#pragma unroll
                for (int k = 0; k < kFluxRounds; ++k)
                    if (got.at[k] >= 0)
                        phiL[got.at[k]] =
                            BD::phi1(phiL[got.at[k]], got.rec[k].value(), dt, ax, ay);
            }
            each_node([&](int c, int row) {
                phiL[BD::own(c, row)] = BD::phi1(pnL[row * kTX + c],
                                                 RT::get_flux(uL, vL, c, row), dt, ax, ay);
            });
            settle();
            stage = 1;
        } else if (stage == 1) {
            Finisher<kStageMid, T, P, TIMED, Kept<T, P>> fin(a, s.x0, s.y0, dt, ax, ay, 2);
            finish(fin, [&](int c, int row, const Kept<T, P>& k) { phiL[BD::own(c, row)] = k.v; });
            exchange(r.mid_mail, tag);
            settle();
            if (sh.fail) break;
            stage = 2;
        } else {
            Finisher<kStageLast, T, P, TIMED, Kept<T, P>> fin(a, s.x0, s.y0, dt, ax, ay, 2);
            finish(fin, [&](int c, int row, const Kept<T, P>& k) {
                phiL[BD::own(c, row)] = k.v;
                pnL[row * kTX + c] = k.v;
            });
            bad = fin.bad;
            ++step;
            if (!(step_open(sh.st) && step < r.max_steps)) break;   // uniform over the launch
            exchange(r.last_mail, tag);
            settle();
            if (sh.fail) break;
            stage = 0;
        }
    }
    each_node([&](int c, int row) {
        const_cast<P*>(a.phi_n)[int64_t(s.y0 + row) * a.nx + s.x0 + c] = pnL[row * kTX + c];
    });
    if constexpr (TIMED) {
        a.st = r.state;
        a.par = par;
    }
    resident_close(a, r, s.tile, sh.st, sh.fail, bad);
}

template <typename T, typename P, bool TIMED>
__global__ __launch_bounds__(kResidentThreads1) void k_resident1d(StageArgs<T, P> a, ResidentArgs r) {
    using RT = ResidentTile1D<T, P>;
    using BD = Border<T, P, kResidentTX1, 1, RT::PW, 1, kResidentThreads1>;
    constexpr int NW = kResidentThreads1 / 64;
    __shared__ P phiL[RT::kPhiElems];
    __shared__ T uL[RT::kUElems];
    __shared__ Flux3<T> fluxL[kResidentTX1];
    __shared__ ResidentShared<NW> sh;
    __shared__ DevState sh_tn;
    const int tid = threadIdx.x;
    __builtin_assume(tid >= 0 && tid < kResidentThreads1);
    const Spot s = make_spot(r, int(blockIdx.x), 1, a.bcx, a.bcy);
    if (tid == 0) {
        sh.go = resident_join(r);
        sh.st = a.st[a.par];
        sh.fail = 0;
        sh.active = 0;
    }
    BD::template load<RT::kPhiElems>(tid, s, a, phiL);
    __syncthreads();
    if (sh.go != 1) return;
    if (!(step_open(sh.st) && r.max_steps > 0)) {
        if (s.tile == 0 && tid == 0) atomicMax(&a.st[a.par].pad[0], 1);
        return;
    }
    const int par = a.par;
    if constexpr (TIMED) {
        a.st = &sh_tn;
        a.par = 0;
    }
    const bool mine = tid < s.w;
    P pn = phiL[tid + 3];
    double dt = 0.0, ax = 0.0;
    bool bad = false;
    int step = 0, stage = 0;
    auto finish = [&](auto& fin) {
        fin.room_x = s.w;
        fin.room_y = 1;
        if (!mine) return;
        const T um = uL[tid], up = uL[RT::kUElems / 2 + tid];
        const int mode = fin.mode();
        if (TIMED && mode == kNodeTimed)
            fin.template node<TIMED ? kNodeTimed : kNodePlain>(tid, 0, um, up, T(0), T(0),
                                                              phiL[tid + 3], pn);
        else if (mode == kNodeExtended)
            fin.template node<kNodeExtended>(tid, 0, um, up, T(0), T(0), phiL[tid + 3], pn);
        else
            fin.template node<kNodePlain>(tid, 0, um, up, T(0), T(0), phiL[tid + 3], pn);
    };
    auto exchange = [&](u64* mail, unsigned int tag) {
        typename BD::template Received<Tagged<P>, 1> got;
        __syncthreads();
        if (tid < 64) {
            BD::send_phi(tid, kResidentThreads1, s, phiL, tag, mail);
            BD::expect(tid, kResidentThreads1, s, got);
            if (!wait_for(r, [&] { return BD::look(tid, kResidentThreads1, s, tag, mail, got); }))
                sh.fail = 1;
            if (got.at[0] >= 0) phiL[got.at[0]] = got.rec[0].value();
        }
    };
    auto settle = [&] {
        if (s.any_local) {
            __syncthreads();
            BD::fill_local(tid, s, a, phiL);
        }
        __syncthreads();
    };
#pragma unroll 1
    for (;;) {
        const unsigned int tag = r.epoch + unsigned(step);
        RT::sweep(tid, a, phiL, uL);
        if (TIMED && stage == 0 && tid == 0) sh_tn.t = sh.st.t;
        __syncthreads();
        if (stage == 0) {
            Finisher<kStagePre, T, P, TIMED, Kept<T, P>> fin(a, s.x0, 0, 0.0, 0.0, 0.0, 1);
            finish(fin);
            if (mine) fluxL[tid] = fin.sink.f;
            resident_fold(sh, fin.lo_u, fin.hi_u, T(0), T(0), fin.bad || bad);
            __syncthreads();
            typename BD::template Received<TaggedFlux<T>, 1> got;
            if (tid < 64) {
                resident_plan(a, r, s.tile, step, sh);
            } else if (tid < 128) {
                BD::send_flux(tid - 64, kResidentThreads1, s, [&](int c, int) { return fluxL[c]; }, tag,
                              r.flux_mail);
                BD::expect(tid - 64, kResidentThreads1, s, got);
                if (!wait_for(r, [&] {
                        return BD::look(tid - 64, kResidentThreads1, s, tag, r.flux_mail, got);
                    }))
                    sh.fail = 1;
            }
            __syncthreads();
            if (sh.fail || !sh.active) break;
            dt = sh.st.dt;
            ax = sh.st.alpha_x;
            if (tid >= 64 && tid < 128 && got.at[0] >= 0)
                phiL[got.at[0]] = BD::phi1(phiL[got.at[0]], got.rec[0].value(), dt, ax, 0.0);
            if (mine) phiL[tid + 3] = BD::phi1(pn, fin.sink.f, dt, ax, 0.0);
            settle();
            stage = 1;
        } else if (stage == 1) {
            Finisher<kStageMid, T, P, TIMED, Kept<T, P>> fin(a, s.x0, 0, dt, ax, 0.0, 1);
            finish(fin);
            if (mine) phiL[tid + 3] = fin.sink.v;
            exchange(r.mid_mail, tag);
            settle();
            if (sh.fail) break;
            stage = 2;
        } else {
            Finisher<kStageLast, T, P, TIMED, Kept<T, P>> fin(a, s.x0, 0, dt, ax, 0.0, 1);
            finish(fin);
            if (mine) pn = phiL[tid + 3] = fin.sink.v;
            bad = fin.bad;
            ++step;
            if (!(step_open(sh.st) && step < r.max_steps)) break;
            exchange(r.last_mail, tag);
            settle();
            if (sh.fail) break;
            stage = 0;
        }
    }
    if (mine) const_cast<P*>(a.phi_n)[s.x0 + tid] = pn;
    if constexpr (TIMED) {
        a.st = r.state;
        a.par = par;
    }
    resident_close(a, r, s.tile, sh.st, sh.fail, bad);
}
#endif

}  // namespace hjw
