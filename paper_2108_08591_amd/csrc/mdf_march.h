#pragma once
// mdf_march.h -- several time steps per pass over HBM on a 2D grid
// (temporal blocking along y), for the lattices with axis links.
//
// Included by mdf_kernels.h, whose node code (moments, collision, fields) it
// shares, so that every population is bitwise that of one-step launches.
//
// One wavefront owns a strip of 64 columns, one per lane, and a chunk of
// rows, and walks the rows upwards.  For every new row of f*(t) that it
// loads, it advances the row below it by step 1, the row below that by step
// 2, and so on up to step K, whose result goes back to HBM.  Between two
// steps only the values that the next one still needs are kept, all in
// registers: what a node pulls along y comes from the same lane one row
// earlier or later, what it pulls along x from the neighbouring lane by a
// wavefront rotation (one DPP move).  No LDS and no barrier: the loads of
// the next row are in flight while the K steps of the current one are
// computed, and every population crosses HBM once per K steps.  The price is
// the halo: each step makes one more column invalid at either end of the
// strip (at most 64 - 2K of its 64 columns are written, except where the
// strip ends at a wall or wraps onto itself), and every chunk of rows takes
// K (K - 1) / 2 extra node rows at either end.
// Bound in FP32 by vector issue and HBM at once (8192^2, five steps: 2.2 ms, 1.2
// wave instructions per CU and cycle, 6.1 GB read, 1.5 states, and 4.2 GB written:
// 4.7 TB/s, a plain copy's rate), in the 16-bit formats by vector issue (4000 x 2977
// FP16 with obstacles: 0.83 per CU and cycle, 2.3 TB/s).
namespace mdf {
namespace {

// Value of the lane one below / one above, the last lane's neighbour being
// the first: wave_ror:1 and wave_rol:1.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v)
{
    const int r = __builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, false);
    return __int_as_float(r);
}
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = uint32_t(__builtin_amdgcn_mov_dpp(int(uint32_t(b)), CTRL, 0xf, 0xf, false));
    const uint32_t hi = uint32_t(__builtin_amdgcn_mov_dpp(int(uint32_t(b >> 32)), CTRL, 0xf, 0xf, false));
    return __builtin_bit_cast(double, uint64_t(hi) << 32 | lo);
}
// (a 64-bit value as its two halves)
template <class C> __device__ __forceinline__ C lane_below(C v) { return dpp_move<0x13C>(v); }
template <class C> __device__ __forceinline__ C lane_above(C v) { return dpp_move<0x134>(v); }

// Index of the direction (cx, cy) of a 2D axis-link lattice.
template <class L>
constexpr int axis_dir(int cx, int cy)
{
    for (int i = 0; i < L::Q; ++i)
        if (L::cx[i] == cx && L::cy[i] == cy) return i;
    return -1;
}

// Wavefronts per block.
constexpr int kMarchWaves = 4;

// One value of a row of `bytes` bytes, written at byte offset `off`, or
// nowhere where off lies beyond the row: the bounds check of a buffer
// store.  The store is then the same instruction for every lane, without a
// branch around it.  (After a branch that may skip stores the compiler
// must assume they were skipped, and waits for them where it only means to
// wait for older loads.)
template <class T>
__device__ __forceinline__ void put_row(T *row, uint32_t bytes, uint32_t off, T v)
{
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(row, 0, int(bytes), 0x00020000);
    if constexpr (sizeof(T) == 2)
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, v), r, int(off), 0, 0);
    else if constexpr (sizeof(T) == 4)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, int(off), 0, 0);
    else {
        typedef unsigned int u2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, int(off), 0, 0);
    }
}

// The wall rule on a value leaving through a wall or a solid link.
template <class L, class C>
__device__ __forceinline__ C bounced(C v, int a, int i, C uw)
{
    if (a + L::A0 == 0) return v;
    const C w = C(L::w[i]);
    return -v + C(2) * w * uw;
}

// Velocity component of wall face f that set a's wall rule takes.
template <class L, class C>
__device__ __forceinline__ C wall_of(const KCase &p, int f, int a)
{
    const int b = a + L::A0 > 0 ? a + L::A0 - 1 : 0;
    return kpar<C>(p.wallu[f][b], p.walluf[f][b]);
}

// Between two steps, per lane: the values the pending row's nodes pull, all
// but the one from the row above (c_y = -1), whose slot holds the row's own
// +y population instead (what the row above pulls, and what bounces back
// from a wall or a solid node above).
template <class L, class C>
struct MarchStage {
    C f[L::NS][L::Q];
};

// Strip s writes columns [s * step, (s + 1) * step); its first lane holds
// column s * step - halo.  The last strip before a wall needs no halo there
// and goes on up to the wall; a row that fits one wavefront between walls, or
// divides it on a periodic axis (the wavefront rotation then wraps exactly),
// takes one strip without a halo.

// K steps on strip s, chunk c.
template <class L, int ST, int K, bool GEN, bool EMIT, bool MASK>
__device__ __forceinline__ void march_strip(const KCase &pc, const MarchGrid &g, int s, int c,
                                            const typename Store<ST>::T *__restrict__ src,
                                            typename Store<ST>::T *__restrict__ dst,
                                            const uint8_t *__restrict__ links, uint32_t fields,
                                            typename Store<ST>::C *__restrict__ out)
{
    static_assert(L::D == 2 && !L::DIAG, "2D axis-link lattices");
    static_assert(K <= 7, "eight rows of link bits in a 64-bit history");
    using S = Store<ST>;
    using T = typename S::T;
    using C = typename S::C;
    constexpr int XP = axis_dir<L>(1, 0), XM = axis_dir<L>(-1, 0), YP = axis_dir<L>(0, 1), YM = axis_dir<L>(0, -1);
    KCase p = pc;
    if (!GEN) {
        p.ffield = nullptr;
        p.forcing = MDF_FORCING_PLAIN;
        p.fmove = 1.0;
        p.fmovef = 1.0f;
    }
    const int lane = threadIdx.x & 63;
    const bool wallx = p.bc[0] == MDF_WALL, wally = p.bc[2] == MDF_WALL;
    // column of this lane: wrapped on a periodic axis, clamped to the row
    // between walls (lanes beyond the row compute values nothing reads)
    const int xu = s * g.step - g.halo + lane;
    int x = xu;
    if (wallx) {
        x = x < 0 ? 0 : (x < p.nx ? x : p.nx - 1);
    } else {
        x %= p.nx;
        if (x < 0) x += p.nx;
    }
    const int o0 = s * g.step, o1 = s + 1 == g.nx ? p.nx : o0 + g.step;
    const bool mine = xu >= o0 && xu < o1;
    const bool at_lo = wallx && xu == 0, at_hi = wallx && xu == p.nx - 1;
    const bool edge = wallx && (s == 0 || s + 1 >= g.nx);
    const int y0 = c * g.rows, y1 = (y0 + g.rows < p.ny) ? y0 + g.rows : p.ny;
    const Ix32 col{uint32_t(x)};
    const long long nodes = (long long)p.nx * p.ny;
    const uint32_t row_bytes = uint32_t(p.pitch) * uint32_t(sizeof(T));

    // row y of the grid that an unwrapped row r stands for
    auto wrapped = [&](int r) {
        r = __builtin_amdgcn_readfirstlane(r % p.ny);
        return r < 0 ? r + p.ny : r;
    };
    MarchStage<L, C> st[K] = {};
    T raw[L::NS][L::Q];            // row R + 1 of f*(t), on its way
    unsigned lbraw = 0;
    uint64_t hist = 0;              // byte j: link bits of row R - j
    auto fetch = [&](int y) __attribute__((always_inline)) {
        const T *row = src + (long long)y * p.pitch;
        // (opaque in every iteration: a 32-bit offset known in the block it
        // is used in takes the load's scalar-base form)
        uint32_t k = col.k;
        asm volatile("" : "+v"(k));
        if (MASK && (!GEN || links)) lbraw = *elem(links + (long long)y * p.pitch, Ix32{k});
#pragma unroll
        for (int i = 0; i < L::Q; ++i)
#pragma unroll
            for (int a = 0; a < L::NS; ++a) raw[a][i] = *elem(row + plane_of<L>(a, i) * p.dstride, Ix32{k});
    };
    // waits here for the loads in flight
    auto arrived = [&]() __attribute__((always_inline)) {
        if (MASK) asm volatile("" : "+v"(lbraw));
#pragma unroll
        for (int a = 0; a < L::NS; ++a)
#pragma unroll
            for (int i = 0; i < L::Q; ++i) asm volatile("" : "+v"(raw[a][i]));
    };
    // between walls the walk starts at row 0 at the earliest and loads up
    // to row ny - 1 at the latest
    const int rb = (wally && y0 < K) ? 0 : y0 - K;
    const int rload = wally ? (y1 + K < p.ny ? y1 + K : p.ny) : y1 + K;
    int ynext = wally ? rb : wrapped(rb);
    fetch(ynext);

    // One row: all K steps.  WARM: some step may not have its rows yet, or
    // a wall above or below is within reach.
    auto advance = [&](int R, auto warm) __attribute__((always_inline)) {
        constexpr bool WARM = decltype(warm)::value;
        C o[L::NS][L::Q] = {};
        if (!WARM || R < rload) {
            // row R of f*(t)
            if (MASK) hist = hist << 8 | lbraw;
#pragma unroll
            for (int a = 0; a < L::NS; ++a)
#pragma unroll
                for (int i = 0; i < L::Q; ++i) o[a][i] = S::decode(raw[a][i], rest_value<L, C>(p, a, i), p.scale);
        } else {
            if (MASK) hist = hist << 8;
        }
        const bool links_near = MASK && __builtin_amdgcn_ballot_w64(hist != 0) != 0;
#pragma unroll
        for (int j = 1; j <= K; ++j) {
            MarchStage<L, C> &g1 = st[j - 1];
            const int r = R - j;                       // row this step works on
            const unsigned lb = MASK ? unsigned(hist >> (8 * j)) & 0xffu : 0u;
            Node<L, C> n;
            // the pending row's values, completed by what comes from the row above
#pragma unroll
            for (int a = 0; a < L::NS; ++a)
#pragma unroll
                for (int i = 0; i < L::Q; ++i) n.f[a][i] = i == YM ? o[a][YM] : g1.f[a][i];
            if (WARM && wally && r + 1 >= p.ny) {
#pragma unroll
                for (int a = 0; a < L::NS; ++a)
                    n.f[a][YM] = bounced<L, C>(g1.f[a][YM], a, YM, wall_of<L, C>(p, 3, a));
            }
            if (MASK && links_near) {
                asm volatile("");
#pragma unroll
                for (int a = 0; a < L::NS; ++a)
                    if ((lb >> YM) & 1u) n.f[a][YM] = bounced<L, C>(g1.f[a][YM], a, YM, C(0));
            }
            // the row above becomes the pending row
#pragma unroll
            for (int a = 0; a < L::NS; ++a) {
                const C up = g1.f[a][YM];
#pragma unroll
                for (int i = 0; i < L::Q; ++i) {
                    if (i == XP) g1.f[a][i] = lane_below(o[a][i]);
                    else if (i == XM) g1.f[a][i] = lane_above(o[a][i]);
                    else if (i == YP) g1.f[a][i] = up;
                    else if (i == YM) g1.f[a][i] = o[a][YP];
                    else g1.f[a][i] = o[a][i];
                }
            }
            if (edge) {
#pragma unroll
                for (int a = 0; a < L::NS; ++a) {
                    C vm = o[a][XM], vp = o[a][XP];
                    asm volatile("" : "+v"(vm), "+v"(vp));     // keeps this a branch that interior strips skip
                    const C lo = bounced<L, C>(vm, a, XP, wall_of<L, C>(p, 0, a));
                    const C hi = bounced<L, C>(vp, a, XM, wall_of<L, C>(p, 1, a));
                    g1.f[a][XP] = at_lo ? lo : g1.f[a][XP];
                    g1.f[a][XM] = at_hi ? hi : g1.f[a][XM];
                }
            }
            if (WARM && wally && r + 1 == 0) {
#pragma unroll
                for (int a = 0; a < L::NS; ++a)
                    g1.f[a][YP] = bounced<L, C>(o[a][YM], a, YP, wall_of<L, C>(p, 2, a));
            }
            if (MASK && links_near) {
                asm volatile("");
                const unsigned lq = unsigned(hist >> (8 * (j - 1))) & 0xffu;
#pragma unroll
                for (int a = 0; a < L::NS; ++a) {
                    if ((lq >> XP) & 1u) g1.f[a][XP] = bounced<L, C>(o[a][XM], a, XP, C(0));
                    if ((lq >> XM) & 1u) g1.f[a][XM] = bounced<L, C>(o[a][XP], a, XM, C(0));
                    if ((lq >> YP) & 1u) g1.f[a][YP] = bounced<L, C>(o[a][YM], a, YP, C(0));
                }
            }
            if (j == 1) {
                // row R is taken over: its registers take the next one, whose
                // loads fly during the arithmetic of K steps
                // (after the last row that one is read again, unused)
                ynext = ynext + 1 < p.ny ? ynext + 1 : (wally ? ynext : 0);
                fetch(ynext);
            }
            // step j of row r, once its rows below and above went through step j - 1
            if (WARM && (r < y0 - (K - j) || (wally && (r < 0 || r >= p.ny)))) continue;
            if (GEN && p.ffield) {
                load_sources<L, C>(p, (long long)(wally ? r : wrapped(r)) * p.nx + x, n);
            } else {
#pragma unroll
                for (int pa = 0; pa <= L::D; ++pa) n.fb[pa] = kpar<C>(p.fbar[pa], p.fbarf[pa]);
            }
            Moments<L, C> m;
            moments<L, C>(p, n, m);
            if (j == K && EMIT) arrived();
            if (EMIT && mine && r >= y0 && r < y1 && (j == K || (fields & MDF_FIELD_ACCUMULATE))) {
                // (accumulated fields count every step)
                C *row = out + (long long)r * p.nx;
                if (MASK && (lb & 0x80u)) write_zero_fields<L, C>(fields, row, col, nodes);
                else write_fields<L, C>(p, n, m, fields, row, col, nodes);
            }
            const uint32_t off = (mine && !(MASK && (lb & 0x80u))) ? col.k * uint32_t(sizeof(T)) : ~0u;
#pragma unroll
            for (int a = 0; a < L::NS; ++a) {
                C fo[L::Q];
                collide_fused<L, C>(p, n, m, a, fo, m.fb[a + L::A0]);
#pragma unroll
                for (int i = 0; i < L::Q; ++i) {
                    const C rest = rest_value<L, C>(p, a, i);
                    if (j < K) {
                        o[a][i] = S::decode(S::encode(fo[i], rest, p.inv_scale), rest, p.scale);
                        // formed here: sunk to their uses, the sums f + d
                        // would keep both terms in registers until then
                        asm volatile("" : "+v"(o[a][i]));
                    } else {
                        put_row<T>(dst + (long long)r * p.pitch + plane_of<L>(a, i) * p.dstride, row_bytes, off,
                                   S::encode(fo[i], rest, p.inv_scale));
                    }
                }
            }
        }
    };
    // every step has its rows from R = y0 + K on, and rows of f*(t) to load
    // up to rload
    const int r1 = y0 + K < rload ? y0 + K : rload;
    int R = rb;
    for (;;) {
        const int lim = R < r1 ? r1 : y1 + K;
        for (; R < lim; ++R) advance(R, std::true_type{});
        // (on entry no load is left in flight: the loop's own wait counts then
        // allow for the stores issued after the loads)
        arrived();
        for (; R + 1 < rload; R += 2) {
            advance(R, std::false_type{});
            advance(R + 1, std::false_type{});
        }
        if (R >= y1 + K) break;
    }
}

// Several steps where strips do not pay: in FP64, whose rows between the
// steps do not fit the registers, and on grids inside the Infinity Cache,
// where a strip's rows, one after the other in one wavefront, leave the chip
// waiting for them.  A block owns a tile and its halo of 4 nodes, one or two
// nodes per thread, and takes all K <= 4 steps of it at once: populations along
// x pass between neighbouring lanes (DPP), those along y through LDS (or within
// the thread), in two buffers, so that one barrier per step is enough.  The
// halo is computed again by the neighbouring tiles.
// Tiles are 16 x 16 threads (8 x 8 nodes written) on small grids, where the
// latency of a step counts and not its arithmetic, and 32 x 32 nodes (24 x 24
// written) beyond.  There a thread takes two nodes of a column in FP64 and
// FP32: as many wavefronts fit a CU, with half the LDS and two independent
// chains each (FP64 1024^2 19.3 us per step with one node, 16.8 with tiles of
// 32 x 16, 13.4 with two nodes; FP32 8.1 and 7.5).  The 16-bit formats, which
// convert every value at every step, keep one (FP16 1024^2 9.4 us, 9.9 with two).
// Bound by vector issue and the waits of the barrier (FP32 1024^2, emitting: 0.67
// wave instructions per CU and cycle, 29 % of the wavefronts' time waiting), in FP64
// beyond the cache by HBM as well (60 grids of 64^2 to 512^2: 0.40, 3.8 TB/s).
// One and two steps per launch, before: 64^2 4.2 us in FP32 and 3.3 us in FP64
// per step (1.1 and 1.3 now), 1024^2 12.8 and 21.1 us.
constexpr int kTileHalo = 4;
template <int ST, bool LARGE>
struct TileShape {
    static constexpr int W = LARGE ? 32 : 16, H = LARGE ? 32 : 16;             // columns and rows
    static constexpr int R = LARGE && sizeof(typename Store<ST>::T) > 2 ? 2 : 1, NT = W * H / R;   // rows per thread, threads
    static constexpr int SX = W - 2 * kTileHalo, SY = H - 2 * kTileHalo;       // nodes written
    // Wavefronts per SIMD at least: two blocks of 16 fit a CU.  With a mask and
    // emitted fields 98 to 102 SGPRs would be taken, of which 7 wavefronts fit and
    // with them one block, and now 78 (21 steps, 2048^2: BF16 D2Q4 1049 and 792 us,
    // FP16 D2Q5 1004 and 782 us; in launches of two steps 864 and 969).
    static constexpr int WAVES = NT == 1024 ? 8 : 1;
};

template <class L, int ST, bool LARGE>
struct TileLds {
    typename Store<ST>::C v[2][L::NS][2][TileShape<ST, LARGE>::NT];
};

template <class L, int ST, bool LARGE, int K, bool GEN, bool EMIT, bool MASK>
__device__ __forceinline__ void tile_steps(const KCase &pc, int gx, int tile,
                                           const typename Store<ST>::T *__restrict__ src,
                                           typename Store<ST>::T *__restrict__ dst, const uint8_t *__restrict__ links,
                                           uint32_t fields, typename Store<ST>::C *__restrict__ out,
                                           TileLds<L, ST, LARGE> &lds)
{
    static_assert(L::D == 2 && !L::DIAG && K <= kTileHalo, "2D axis-link lattices");
    using S = Store<ST>;
    using C = typename S::C;
    constexpr int XP = axis_dir<L>(1, 0), XM = axis_dir<L>(-1, 0), YP = axis_dir<L>(0, 1), YM = axis_dir<L>(0, -1);
    KCase p = pc;
    if (!GEN) {
        p.ffield = nullptr;
        p.forcing = MDF_FORCING_PLAIN;
        p.fmove = 1.0;
        p.fmovef = 1.0f;
    }
    using TS = TileShape<ST, LARGE>;
    constexpr int R = TS::R;
    const int e = threadIdx.x, tx = e % TS::W, ty = e / TS::W * R;
    const bool wallx = p.bc[0] == MDF_WALL, wally = p.bc[2] == MDF_WALL;
    const int xu = (tile % gx) * TS::SX - kTileHalo + tx, yu = (tile / gx) * TS::SY - kTileHalo + ty;
    int x = xu;
    // wrapped on a periodic axis; clamped between walls (values beyond them are never used)
    if (wallx) x = x < 0 ? 0 : (x < p.nx ? x : p.nx - 1);
    else { x %= p.nx; x = x < 0 ? x + p.nx : x; }
    const bool minex = unsigned(tx - kTileHalo) < unsigned(TS::SX) && xu < p.nx;
    const bool at_x0 = wallx && xu == 0, at_x1 = wallx && xu == p.nx - 1;
    const long long nodes = (long long)p.nx * p.ny;
    int y[R];
    unsigned lb[R];
    bool mine[R], at_y0[R], at_y1[R];
    Node<L, C> n[R];
    C o[R][L::NS][L::Q];
    bool wall = at_x0 || at_x1;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        y[r] = yu + r;
        if (wally) y[r] = y[r] < 0 ? 0 : (y[r] < p.ny ? y[r] : p.ny - 1);
        else { y[r] %= p.ny; y[r] = y[r] < 0 ? y[r] + p.ny : y[r]; }
        mine[r] = minex && unsigned(ty + r - kTileHalo) < unsigned(TS::SY) && yu + r < p.ny;
        at_y0[r] = wally && yu + r == 0;
        at_y1[r] = wally && yu + r == p.ny - 1;
        const Ix32 own = grid_ix<false>(x, y[r], 0, p.ny, p.pitch);
        lb[r] = 0;
        if (MASK && (!GEN || links)) lb[r] = *elem(links, own);
        load_sources<L, C>(p, (long long)y[r] * p.nx + x, n[r]);
#pragma unroll
        for (int a = 0; a < L::NS; ++a)
#pragma unroll
            for (int i = 0; i < L::Q; ++i)
                o[r][a][i] = S::load(src + plane_of<L>(a, i) * p.dstride, own, rest_value<L, C>(p, a, i), p.scale);
        wall = wall || at_y0[r] || at_y1[r] || (lb[r] & 0x7fu);
    }
    const bool special = __builtin_amdgcn_ballot_w64(wall) != 0;
    const int below = ty > 0 ? e - TS::W : e, above = ty < TS::H - R ? e + TS::W : e;
#pragma unroll
    for (int j = 1; j <= K; ++j) {
        auto &ex = lds.v[j & 1];
#pragma unroll
        for (int a = 0; a < L::NS; ++a) {
            ex[a][0][e] = o[R - 1][a][YP];
            ex[a][1][e] = o[0][a][YM];
        }
        __syncthreads();
#pragma unroll
        for (int a = 0; a < L::NS; ++a)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (L::R == 1) n[r].f[a][0] = o[r][a][0];
                n[r].f[a][XP] = lane_below(o[r][a][XP]);
                n[r].f[a][XM] = lane_above(o[r][a][XM]);
                n[r].f[a][YP] = r > 0 ? o[r > 0 ? r - 1 : 0][a][YP] : ex[a][0][below];
                n[r].f[a][YM] = r + 1 < R ? o[r + 1 < R ? r + 1 : r][a][YM] : ex[a][1][above];
            }
        if (special) {
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int a = 0; a < L::NS; ++a) {
                    if (at_x0) n[r].f[a][XP] = bounced<L, C>(o[r][a][XM], a, XP, wall_of<L, C>(p, 0, a));
                    if (at_x1) n[r].f[a][XM] = bounced<L, C>(o[r][a][XP], a, XM, wall_of<L, C>(p, 1, a));
                    if (at_y0[r]) n[r].f[a][YP] = bounced<L, C>(o[r][a][YM], a, YP, wall_of<L, C>(p, 2, a));
                    if (at_y1[r]) n[r].f[a][YM] = bounced<L, C>(o[r][a][YP], a, YM, wall_of<L, C>(p, 3, a));
                    if (MASK) {
                        if ((lb[r] >> XP) & 1u) n[r].f[a][XP] = bounced<L, C>(o[r][a][XM], a, XP, C(0));
                        if ((lb[r] >> XM) & 1u) n[r].f[a][XM] = bounced<L, C>(o[r][a][XP], a, XM, C(0));
                        if ((lb[r] >> YP) & 1u) n[r].f[a][YP] = bounced<L, C>(o[r][a][YM], a, YP, C(0));
                        if ((lb[r] >> YM) & 1u) n[r].f[a][YM] = bounced<L, C>(o[r][a][YP], a, YM, C(0));
                    }
                }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            Moments<L, C> m;
            moments<L, C>(p, n[r], m);
            if (EMIT && mine[r] && fields && (j == K || (fields & MDF_FIELD_ACCUMULATE))) {
                const Ix32 node = grid_ix<false>(x, y[r], 0, p.ny, p.nx);
                if (MASK && (lb[r] & 0x80u)) write_zero_fields<L, C>(fields, out, node, nodes);
                else write_fields<L, C>(p, n[r], m, fields, out, node, nodes);
            }
            const Ix32 own = grid_ix<false>(x, y[r], 0, p.ny, p.pitch);
#pragma unroll
            for (int a = 0; a < L::NS; ++a) {
                C fo[L::Q];
                collide_fused<L, C>(p, n[r], m, a, fo, m.fb[a + L::A0]);
#pragma unroll
                for (int i = 0; i < L::Q; ++i) {
                    const C rest = rest_value<L, C>(p, a, i);
                    if (j < K) {
                        o[r][a][i] = S::decode(S::encode(fo[i], rest, p.inv_scale), rest, p.scale);
                        if (R > 1) asm volatile("" : "+v"(o[r][a][i]));       // (as in march_strip)
                    } else if (mine[r] && !(MASK && (lb[r] & 0x80u))) {
                        S::store(dst + plane_of<L>(a, i) * p.dstride, own, fo[i], rest, p.inv_scale);
                    }
                }
            }
        }
    }
}

template <class L, int ST, bool LARGE, int K, bool GEN, bool EMIT, bool MASK>
__global__ void __launch_bounds__((TileShape<ST, LARGE>::NT), (TileShape<ST, LARGE>::WAVES))
k_tile(KCase p, Tiling tl, const typename Store<ST>::T *__restrict__ src, typename Store<ST>::T *__restrict__ dst,
       const uint8_t *__restrict__ links, uint32_t fields, typename Store<ST>::C *__restrict__ out)
{
    __shared__ TileLds<L, ST, LARGE> lds;
    tile_steps<L, ST, LARGE, K, GEN, EMIT, MASK>(p, tl.gx, block_tile(tl), src, dst, links, fields, out, lds);
}

template <class L, int ST, int K, bool GEN, bool EMIT, bool MASK>
__global__ void __launch_bounds__(64 * kMarchWaves, 3)
k_march(KCase p, Tiling tl, MarchGrid g, const typename Store<ST>::T *__restrict__ src,
        typename Store<ST>::T *__restrict__ dst, const uint8_t *__restrict__ links, uint32_t fields,
        typename Store<ST>::C *__restrict__ out)
{
    const int w = __builtin_amdgcn_readfirstlane(block_tile(tl) * kMarchWaves + int(threadIdx.x >> 6));
    if (w >= g.nx * g.ny) return;
    // (quotients are formed in vector registers: say that they are uniform)
    const int c = __builtin_amdgcn_readfirstlane(w / g.nx);
    march_strip<L, ST, K, GEN, EMIT, MASK>(p, g, w - c * g.nx, c, src, dst, links, fields, out);
}

// k_tile over the flat list of the tiles of a batch's active cases (prefix
// offsets tile_start2, total meta[2]).
template <class L, int ST, bool LARGE, int K, bool GEN, bool EMIT, bool MASK>
__global__ void __launch_bounds__((TileShape<ST, LARGE>::NT), (TileShape<ST, LARGE>::WAVES))
k_tile_batch(const BatchEntry *__restrict__ tab, const int *__restrict__ meta, const int *__restrict__ tile_start2,
             const int *__restrict__ active, int parity, uint32_t fields, int groups)
{
    __shared__ TileLds<L, ST, LARGE> lds;
    const int nact = meta[0];
    Tiling tl;
    tl.nb = meta[2];
    tl.groups = groups;
    if ((int)blockIdx.x >= tl.nb) return;
    const int t = block_tile(tl);
    int lo = 0, hi = nact - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tile_start2[mid] <= t) lo = mid;
        else hi = mid - 1;
    }
    const BatchEntry &e = tab[active[lo]];
    const int sel = (e.cur + parity) & 1;
    using T = typename Store<ST>::T;
    using C = typename Store<ST>::C;
    tile_steps<L, ST, LARGE, K, GEN, EMIT, MASK>(e.p, e.march.nx, t - tile_start2[lo], static_cast<const T *>(e.pop[sel]),
                                          static_cast<T *>(e.pop[sel ^ 1]), e.links, fields, static_cast<C *>(e.out), lds);
}

// k_march over the flat list of the strips of a batch's active cases
// (prefix offsets tile_start2, total meta[2]): wavefront w of the list finds
// its case and works on one strip of one chunk there.  The grid covers the
// running cases' units and may be larger (march_grid).
template <class L, int ST, int K, bool GEN, bool EMIT, bool MASK>
__global__ void __launch_bounds__(64 * kMarchWaves, 3)
k_march_batch(const BatchEntry *__restrict__ tab, const int *__restrict__ meta, const int *__restrict__ tile_start2,
              const int *__restrict__ active, int parity, uint32_t fields, int groups)
{
    const int nact = meta[0], total = meta[2];
    Tiling tl;
    tl.nb = (total + kMarchWaves - 1) / kMarchWaves;
    tl.groups = groups;
    if ((int)blockIdx.x >= tl.nb) return;
    const int w = __builtin_amdgcn_readfirstlane(block_tile(tl) * kMarchWaves + int(threadIdx.x >> 6));
    if (w >= total) return;
    int lo = 0, hi = nact - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tile_start2[mid] <= w) lo = mid;
        else hi = mid - 1;
    }
    lo = __builtin_amdgcn_readfirstlane(lo);
    const BatchEntry &e = tab[active[lo]];
    const int sel = (e.cur + parity) & 1, t = w - tile_start2[lo];
    const int c = __builtin_amdgcn_readfirstlane(t / e.march.nx);
    using T = typename Store<ST>::T;
    using C = typename Store<ST>::C;
    march_strip<L, ST, K, GEN, EMIT, MASK>(e.p, e.march, t - c * e.march.nx, c, static_cast<const T *>(e.pop[sel]),
                                           static_cast<T *>(e.pop[sel ^ 1]), e.links, fields, static_cast<C *>(e.out));
}

}  // namespace
}  // namespace mdf
