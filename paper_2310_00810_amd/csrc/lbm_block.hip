// Time-blocked D2Q9 kernels (gfx950): one launch takes several time steps of
// a rectangle of nodes in LDS.
//
// A block loads the populations of an EX x EY region of the lattice, i.e. a
// tile with a halo of T.ms nodes on every side, into LDS and takes n <= T.ms
// steps there.  Step s = 0 .. n - 1 is computed for the nodes at distance at
// most n - 1 - s from the tile, so every value it reads was computed (or
// loaded) by this block and the tile is exact after n steps; neighbouring
// blocks repeat each other's halo work instead of exchanging it.  The
// arithmetic per node is that of k_step / k_adj_step (the same functions on
// the same operands), so the states are bit for bit theirs, whatever the
// grouping of steps.
//
// A tile's nodes come from a list built once per handle (k_build_tiles):
// fluid nodes only, ordered by distance from the tile, so that the nodes of
// every step are a prefix of the list and no lane idles on a solid node or
// in the part of the halo that is done.
//
// What bounds a launch of a small lattice is latency: about 4 us pass before
// the first step and after the last (launch, list, populations, store), then
// about 0.5 us per step with two wavefronts or fewer on each SIMD; a
// single-step launch takes 4 - 6 us for one step.  The arguments that the
// first loads need lead the argument list, where the build has them preloaded
// into scalar registers (without: 1.5 us more per launch).  Per step, 64 x 32
// empty channel: forward 4.5 -> 1.55 us, adjoint 5.4 -> 1.84 us; 512 x 256
// grains: 6.6 -> 3.0 and 7.1 -> 4.6 us.  Large lattices gain from the memory
// traffic, about (1.7 read + 1 written) / 5 states per step instead of 2: a
// batch of 2.6 M fluid nodes 32.8 -> 23 us per step.  One LDS copy of the
// region, written after a barrier, keeps two 64 x 32 blocks on a CU.  The
// stores keep the default cache policy: a tile's rows end inside a cache
// line, and non-temporal stores of such rows halved the speed.
#include "lbm_device.hpp"
#include "lbm_kernels.hpp"

namespace lbm {

// List entry: .x = fluid id; .y = region node p = ey EX + ex (bits 0-15), wall
// links k = 1 .. 8 (bits 16-23: halfway bounce-back, see Links), inlet face
// (bit 24), outlet face (bit 25).
constexpr int E_WALL = 16, E_IN = 24, E_OUT = 25;

// Lattice coordinate v of a region node wrapped around a periodic axis of n.
__device__ inline int wrap(int v, int n) { return v >= 0 && v < n ? v : ((v % n) + n) % n; }

// One block per tile: the list of its fluid nodes by distance d = 0 .. ms from
// the tile, and the number of nodes within each distance.
template <int EX, int EY>
__global__ void __launch_bounds__(256) k_build_tiles(Geo G, BlockGeo T, MTileDesc *__restrict__ tiles,
                                                     uint2 *__restrict__ list) {
    using V = Vel<9>;
    constexpr int P = EX * EY;
    __shared__ int wcount[4];
    MTileDesc &e = tiles[blockIdx.x];
    const InstDev &I = G.inst[e.b];
    const int ms = T.ms, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int x1 = min(e.x0 + EX - 2 * ms, I.nx), y1 = min(e.y0 + EY - 2 * ms, I.ny);
    const bool xper = G.bcx == BC_PERIODIC, yper = G.bcy == BC_PERIODIC, faces = density_faces(G.bcx);
    auto fluid = [&](int x, int y) {
        if ((!xper && (x < 0 || x >= I.nx)) || (!yper && (y < 0 || y >= I.ny))) return false;
        x = wrap(x, I.nx);
        return !solid_bit(row_word(G, I, x, wrap(y, I.ny), 0), x);
    };
    int n = 0;
    for (int d = 0; d <= ms; ++d) {
        for (int p0 = 0; p0 < P; p0 += 256) {
            const int p = p0 + (int)threadIdx.x;
            const int x = e.x0 - ms + p % EX, y = e.y0 - ms + p / EX;
            const int dx = x < e.x0 ? e.x0 - x : max(x - (x1 - 1), 0), dy = y < e.y0 ? e.y0 - y : max(y - (y1 - 1), 0);
            const bool on = p < P && max(dx, dy) == d && fluid(x, y);
            const unsigned long long m = __builtin_amdgcn_ballot_w64(on);
            if (lane == 0) wcount[wave] = __popcll(m);
            __syncthreads();
            int at = n;
            for (int w = 0; w < 4; ++w) {
                if (w < wave) at += wcount[w];
                n += wcount[w];
            }
            if (on) {
                const int xw = wrap(x, I.nx), yw = wrap(y, I.ny);
                uint2 v = make_uint2((unsigned)fluid_id(row_word(G, I, xw, yw, 0), xw), (unsigned)p);
                if (faces && x == 0) v.y |= 1u << E_IN;
                if (faces && x == I.nx - 1) v.y |= 1u << E_OUT;
#pragma unroll
                for (int k = 1; k < 9; ++k) {
                    const int xs = x + V::cx(k);
                    const bool open = faces && (xs < 0 || xs >= I.nx);
                    if (!open && !fluid(xs, y + V::cy(k))) v.y |= 1u << (E_WALL + k - 1);
                }
                list[e.list + at + __popcll(m & ((1ull << lane) - 1ull))] = v;
            }
            __syncthreads();
        }
        if (threadIdx.x == 0) e.cnt[d] = n;
    }
}

// LDS word (forward: populations, see gather_fwd; adjoint: see gather_adj)
// that feeds each direction of a node: its own word or a neighbour's, or the
// zero word behind the planes.
template <int BCX, int EX, int P, bool ADJ>
__device__ inline void sources(uint2 v, int (&from)[9]) {
    using V = Vel<9>;
    constexpr int ZERO = 9 * P;
    const int p = (int)(v.y & 0xffffu);
    const bool in = density_faces(BCX) && ((v.y >> E_IN) & 1u), out = density_faces(BCX) && ((v.y >> E_OUT) & 1u);
    from[0] = p;
#pragma unroll
    for (int k = 1; k < 9; ++k) {
        const int i = V::opp(k), q = p + V::cy(k) * EX + V::cx(k);
        const bool open = V::cx(k) != 0 && (V::cx(k) < 0 ? in : out);
        const bool wall = (v.y >> (E_WALL + k - 1)) & 1u;
        if (ADJ) from[k] = open ? ZERO : (wall ? i * P + p : k * P + q);
        else from[i] = wall || (BCX == BC_ABB && open) ? k * P + p : (open ? ZERO : i * P + q);
    }
}

template <int BCX, int EX, int EY, int NT>
__global__ void __launch_bounds__(NT) k_steps(const uint2 *__restrict__ lists, const MTileDesc *__restrict__ tiles,
                                              const float *__restrict__ src, const InstDev *__restrict__ insts,
                                              int ms, int n_inst, int n_steps, Geo G, StepRun st,
                                              const float *__restrict__ face_in,
                                              const float *__restrict__ face_out) {
    constexpr int P = EX * EY, NPT = P / NT;
    __shared__ float B[9 * P + 1];
    const int tile = xcd_tile(blockIdx.x, gridDim.x), t = (int)threadIdx.x;
    const MTileDesc &e = tiles[tile];
    const uint2 *list = lists + e.list;
    uint2 v[NPT];            // beyond the tile's entries: loaded (the table is padded), never followed
#pragma unroll
    for (int j = 0; j < NPT; ++j) v[j] = list[t + j * NT];
    const int n_load = e.cnt[n_steps], owned = e.cnt[0];
    const InstDev &I = insts[n_inst == 1 ? 0 : e.b];
    const int plane = (int)I.plane;
    {
        const __amdgpu_buffer_rsrc_t rs = planes_rsrc(src + I.st_off, 9, I.plane);
        float f[NPT][9];
#pragma unroll
        for (int j = 0; j < NPT; ++j)
            if (t + j * NT < n_load)
#pragma unroll
                for (int i = 0; i < 9; ++i) f[j][i] = bload(rs, v[j].x * 4u + (unsigned)plane_off(i, plane));
#pragma unroll
        for (int j = 0; j < NPT; ++j)
            if (t + j * NT < n_load)
#pragma unroll
                for (int i = 0; i < 9; ++i) B[i * P + (int)(v[j].y & 0xffffu)] = f[j][i];
    }
    int from[NPT][9];
    float drho_b[NPT];
#pragma unroll
    for (int j = 0; j < NPT; ++j) {
        sources<BCX, EX, P, false>(v[j], from[j]);
        drho_b[j] = 0.f;
        if (density_faces(BCX) && t + j * NT < n_load && (v[j].y >> E_IN)) {
            const int y = wrap(e.y0 - ms + (int)(v[j].y & 0xffffu) / EX, I.ny);
            drho_b[j] = (v[j].y >> E_IN) & 1u ? face_in[I.face_off + y] : face_out[I.face_off + y];
        }
    }
    if (t == 0) B[9 * P] = 0.f;
    __syncthreads();
    // the step's destination and node count are loaded one step ahead
    float *dst = st.dst[0], *dst_next;
    int lim = e.cnt[n_steps - 1], lim_next;
    for (int s = 0; s < n_steps; ++s, dst = dst_next, lim = lim_next) {
        const int sn = min(s + 1, n_steps - 1);
        dst_next = st.dst[sn];
        lim_next = e.cnt[n_steps - 1 - sn];
        float f[NPT][9];
#pragma unroll
        for (int j = 0; j < NPT; ++j) {
            if (t + j * NT >= lim) continue;
            const bool in = density_faces(BCX) && ((v[j].y >> E_IN) & 1u), out = density_faces(BCX) && ((v[j].y >> E_OUT) & 1u);
            float g[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) g[i] = B[from[j][i]];
            if (zouhe_faces(BCX) && wave_has_face(in || out)) zouhe<9>(g, in, out, drho_b[j], BCX == BC_VELOCITY);
            if (BCX == BC_ABB) {
                float uF[3] = {0.f, 0.f, 0.f};
                if (in || out) {
                    float own[9];
#pragma unroll
                    for (int i = 0; i < 9; ++i) own[i] = B[i * P + from[j][0]];
                    const Moments mo = moments<9>(own);
                    uF[0] = mo.ux; uF[1] = mo.uy; uF[2] = mo.uz;
                }
                abb<9>(g, in, out, drho_b[j], uF);
            }
            const Moments m = moments<9>(g);
            collide(G, I.omega, m, g, f[j]);
        }
        if (s + 1 < n_steps) {
            __syncthreads();
#pragma unroll
            for (int j = 0; j < NPT; ++j)
                if (t + j * NT < lim)
#pragma unroll
                    for (int i = 0; i < 9; ++i) B[i * P + from[j][0]] = f[j][i];
        }
        if (dst) {
            const __amdgpu_buffer_rsrc_t rd = planes_rsrc(dst + I.st_off, 9, I.plane);
#pragma unroll
            for (int j = 0; j < NPT; ++j)
                if (t + j * NT < owned)
#pragma unroll
                    for (int i = 0; i < 9; ++i) bstore(rd, f[j][i], v[j].x * 4u, plane_off(i, plane));
        }
        if (s + 1 < n_steps) __syncthreads();
        else if (st.check) {
            const unsigned *ref = (const unsigned *)(st.check + I.st_off);
            bool bad = false;
#pragma unroll
            for (int j = 0; j < NPT; ++j)
                if (t + j * NT < owned)
#pragma unroll
                    for (int i = 0; i < 9; ++i)
                        bad |= __builtin_bit_cast(unsigned, f[j][i]) != ref[(long long)i * plane + v[j].x];
            if (bad) *st.flag = 1u;
        }
    }
}

// part[fluid tile] += the tile's dL/dtau of n <= MS_MAX adjoint steps (values
// per node in v[s]), each step's nodes summed as block_sum sums them; by the
// 256 threads t of one tile, all threads of the block calling.
__device__ inline void dtau_sums(const Geo &G, int tile, int t, const float *const (&v)[MS_MAX], int n,
                                 double (*lds)[4], double *__restrict__ part) {
    const bool on = tile < G.n_ftiles;
    if (on) {
        const FTileDesc e = G.fblk[tile];
        const InstDev &I = G.inst[e.b];
        const int id = (tile - I.ftile_begin) * FT + t;
#pragma unroll
        for (int s = 0; s < MS_MAX; ++s) {
            if (s >= n) break;
            const double w = wave_sum(id < I.n_fluid ? (double)v[s][I.poff + id] : 0.0);
            if ((t & 63) == 0) lds[s][t >> 6] = w;
        }
    }
    __syncthreads();
    if (on && t == 0) {
        double acc = part[tile];
        for (int s = 0; s < n; ++s) acc += (lds[s][0] + lds[s][1]) + (lds[s][2] + lds[s][3]);
        part[tile] = acc;
    }
}

__global__ void __launch_bounds__(FT) k_dtau_sums(Geo G, AdjRun st, double *__restrict__ part) {
    __shared__ double lds[MS_MAX][4];
    dtau_sums(G, (int)blockIdx.x, (int)threadIdx.x, st.prev, st.n_prev, lds, part);
}

// Adjoint steps (see k_adj_step): nu in LDS, F^{k-1} gathered from the tape one
// step ahead of its use.  dL/d(face density) is added per node in time order.
// A node's dL/dtau of each step is stored, and the blocks behind the tiles of
// the next launch (after the last one k_dtau_sums) add it in k_adj_step's
// order, so that neither sum depends on the grouping of steps, nor on which
// kernel takes them.
template <int BCX, int EX, int EY, int NT, bool SEED>
__global__ void __launch_bounds__(NT) k_adj_steps(const uint2 *__restrict__ lists, const MTileDesc *__restrict__ tiles,
                                                  const float *__restrict__ nu_in, const InstDev *__restrict__ insts,
                                                  int ms, int n_inst, int n_steps, int n_tiles, Geo G, AdjRun st,
                                                  float *__restrict__ nu_out, const float *__restrict__ face_in,
                                                  const float *__restrict__ face_out, double *__restrict__ grad_in,
                                                  double *__restrict__ grad_out, double *__restrict__ dtau_part,
                                                  const float *__restrict__ roi, int kind) {
    using V = Vel<9>;
    constexpr int P = EX * EY, NPT = P / NT;
    __shared__ float B[9 * P + 1];
    __shared__ int ids[P];
    __shared__ double sums[NT / FT][MS_MAX][4];
    const int t = (int)threadIdx.x;
    if ((int)blockIdx.x >= n_tiles) {
        const int w = t / FT;
        dtau_sums(G, ((int)blockIdx.x - n_tiles) * (NT / FT) + w, t % FT, st.prev, st.n_prev, sums[w], dtau_part);
        return;
    }
    const int tile = xcd_tile(blockIdx.x, n_tiles);
    const MTileDesc &e = tiles[tile];
    const uint2 *list = lists + e.list;
    uint2 v[NPT];            // beyond the tile's entries: loaded (the table is padded), never followed
#pragma unroll
    for (int j = 0; j < NPT; ++j) v[j] = list[t + j * NT];
    const int n_load = e.cnt[n_steps], owned = e.cnt[0], n_first = e.cnt[n_steps - 1];
    const InstDev &I = insts[n_inst == 1 ? 0 : e.b];
    const int plane = (int)I.plane;
    {
        const __amdgpu_buffer_rsrc_t rs = planes_rsrc(nu_in + I.st_off, 9, I.plane);
        float f[NPT][9];
#pragma unroll
        for (int j = 0; j < NPT; ++j)
            if (t + j * NT < n_load)
#pragma unroll
                for (int i = 0; i < 9; ++i) f[j][i] = bload(rs, v[j].x * 4u + (unsigned)plane_off(i, plane));
#pragma unroll
        for (int j = 0; j < NPT; ++j)
            if (t + j * NT < n_load) {
                ids[v[j].y & 0xffffu] = (int)v[j].x;
#pragma unroll
                for (int i = 0; i < 9; ++i) B[i * P + (int)(v[j].y & 0xffffu)] = f[j][i];
            }
    }
    int from[NPT][9];
    unsigned foff[NPT][9];       // byte offset of each population's source (see gather_fwd)
    float drho_b[NPT], gn[NPT][9];
    double gface[NPT];
    int face[NPT];
#pragma unroll
    for (int j = 0; j < NPT; ++j) {
        sources<BCX, EX, P, true>(v[j], from[j]);
        drho_b[j] = 0.f;
        gface[j] = 0.0;
        face[j] = 0;
        if (density_faces(BCX) && t + j * NT < n_load && (v[j].y >> E_IN)) {
            const bool in = (v[j].y >> E_IN) & 1u;
            face[j] = wrap(e.y0 - ms + (int)(v[j].y & 0xffffu) / EX, I.ny);
            drho_b[j] = in ? face_in[I.face_off + face[j]] : face_out[I.face_off + face[j]];
            if (t + j * NT < owned) gface[j] = in ? grad_in[I.face_off + face[j]] : grad_out[I.face_off + face[j]];
        }
    }
    if (t == 0) B[9 * P] = 0.f;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NPT; ++j) {
        if (t + j * NT >= n_first) continue;
        const unsigned own = v[j].x * 4u;
        const bool in = density_faces(BCX) && ((v[j].y >> E_IN) & 1u), out = density_faces(BCX) && ((v[j].y >> E_OUT) & 1u);
        foff[j][0] = own;
#pragma unroll
        for (int k = 1; k < 9; ++k) {
            const int i = V::opp(k), q = from[j][0] + V::cy(k) * EX + V::cx(k);
            const bool open = V::cx(k) != 0 && (V::cx(k) < 0 ? in : out);
            const bool wall = (v[j].y >> (E_WALL + k - 1)) & 1u;
            const unsigned off = wall || open ? own + (unsigned)plane_off(k, plane)
                                              : (unsigned)ids[q] * 4u + (unsigned)plane_off(i, plane);
            foff[j][i] = zouhe_faces(BCX) && open ? OOB : off;
        }
    }
    auto fetch = [&](const float *F, int lim) {
        const __amdgpu_buffer_rsrc_t rs = planes_rsrc(F + I.st_off, 9, I.plane);
#pragma unroll
        for (int j = 0; j < NPT; ++j)
            if (t + j * NT < lim)
#pragma unroll
                for (int i = 0; i < 9; ++i) gn[j][i] = bload(rs, foff[j][i]);
    };
    const float *F = st.Fprev[0], *F_next;
    int lim = n_first, lim_next;
    fetch(F, lim);
    for (int s = 0; s < n_steps; ++s, F = F_next, lim = lim_next) {
        const int sn = min(s + 1, n_steps - 1);
        F_next = st.Fprev[sn];
        lim_next = e.cnt[n_steps - 1 - sn];
        float g[NPT][9], a[NPT][9];
#pragma unroll
        for (int j = 0; j < NPT; ++j)
#pragma unroll
            for (int i = 0; i < 9; ++i) g[j][i] = gn[j][i];
        const __amdgpu_buffer_rsrc_t rs = planes_rsrc(F + I.st_off, 9, I.plane);
        if (s + 1 < n_steps) fetch(F_next, lim_next);
#pragma unroll
        for (int j = 0; j < NPT; ++j) {
            if (t + j * NT >= lim) continue;
            const bool in = density_faces(BCX) && ((v[j].y >> E_IN) & 1u), out = density_faces(BCX) && ((v[j].y >> E_OUT) & 1u);
            float lam[9], nuo[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) lam[i] = B[from[j][i]];
            float uF[3] = {0.f, 0.f, 0.f}, rhoF = 1.0f;
            if (BCX == BC_ABB) {
#pragma unroll
                for (int i = 0; i < 9; ++i) nuo[i] = 0.f;
                if (in || out) {
                    own_velocity<9>(rs, plane, v[j].x * 4u, rhoF, uF);
#pragma unroll
                    for (int i = 1; i < 9; ++i)
                        if (V::cx(i) != 0 && (V::cx(i) > 0 ? in : out)) nuo[i] = B[i * P + from[j][0]];
                }
            }
            if (zouhe_faces(BCX)) zouhe<9>(g[j], in, out, drho_b[j], BCX == BC_VELOCITY);
            if (BCX == BC_ABB) abb<9>(g[j], in, out, drho_b[j], uF, fmaf(uF[1], uF[1], uF[0] * uF[0]));
            const Moments m = moments<9>(g[j]);
            if (BCX == BC_ABB) {
                const float um[3] = {m.ux, m.uy, m.uz};
                const float jb = abb_adj<9>(lam, in, out, drho_b[j], m.rho, um, nuo);
                if (in || out) gface[j] += (double)jb;
            }
            const float dt = collide_adj<lam_first(BCX, SEED)>(G, I.omega, I.inv_tau2, m, g[j], lam, a[j]);
            if (t + j * NT < owned) st.dtau[s][I.poff + v[j].x] = dt;
            if constexpr (SEED)
                seed_adj<9>(st.target + I.poff * 2 + v[j].x, I.plane, roi[I.poff + v[j].x] * I.loss_scale, kind, m, a[j]);
            if (zouhe_faces(BCX)) {
                const float jb = zouhe_adj<9>(a[j], in, out, g[j], drho_b[j], BCX == BC_VELOCITY);
                if (in || out) gface[j] += (double)jb;
            }
        }
        if (s + 1 < n_steps) {
            __syncthreads();
#pragma unroll
            for (int j = 0; j < NPT; ++j)
                if (t + j * NT < lim)
#pragma unroll
                    for (int i = 0; i < 9; ++i) B[i * P + from[j][0]] = a[j][i];
            __syncthreads();
        } else {
            const __amdgpu_buffer_rsrc_t rd = planes_rsrc(nu_out + I.st_off, 9, I.plane);
#pragma unroll
            for (int j = 0; j < NPT; ++j)
                if (t + j * NT < owned)
#pragma unroll
                    for (int i = 0; i < 9; ++i) bstore(rd, a[j][i], v[j].x * 4u, plane_off(i, plane));
        }
    }
#pragma unroll
    for (int j = 0; j < NPT; ++j) {
        if (t + j * NT >= owned) continue;
        if (density_faces(BCX) && ((v[j].y >> E_IN) & 1u)) grad_in[I.face_off + face[j]] = gface[j];
        else if (density_faces(BCX) && (v[j].y >> E_OUT)) grad_out[I.face_off + face[j]] = gface[j];
    }
}

#define DISPATCH9(bcx, CALL)                                                               \
    do {                                                                                   \
        if (bcx == BC_PRESSURE) CALL(BC_PRESSURE);                                         \
        else if (bcx == BC_PERIODIC) CALL(BC_PERIODIC);                                    \
        else if (bcx == BC_WALL) CALL(BC_WALL);                                            \
        else if (bcx == BC_ABB) CALL(BC_ABB);                                              \
        else CALL(BC_VELOCITY);                                                            \
    } while (0)

hipError_t launch_build_tiles(const Geo &G, const BlockGeo &T, MTileDesc *tiles, uint2 *list, hipStream_t s) {
    if (T.n_tiles == 0) return hipSuccess;
    const dim3 grid((unsigned)T.n_tiles), blk(256);
    if (T.big) hipLaunchKernelGGL((k_build_tiles<64, 32>), grid, blk, 0, s, G, T, tiles, list);
    else hipLaunchKernelGGL((k_build_tiles<32, 16>), grid, blk, 0, s, G, T, tiles, list);
    return hipGetLastError();
}

hipError_t launch_steps(const Geo &G, const BlockGeo &T, const float *src, const StepRun &st, const float *fin,
                        const float *fout, hipStream_t s) {
    if (T.n_tiles == 0) return hipSuccess;
    const dim3 grid((unsigned)T.n_tiles), blk(512);
#define LAUNCH(B, EX, EY)                                                                                          \
    hipLaunchKernelGGL((k_steps<B, EX, EY, 512>), grid, blk, 0, s, T.list, T.tile, src, G.inst, T.ms, G.n_inst, \
                       st.n, G, st, fin, fout)
#define CALL(B)                                            \
    do {                                                   \
        if (T.big) LAUNCH(B, 64, 32);                      \
        else LAUNCH(B, 32, 16);                            \
    } while (0)
    DISPATCH9(G.bcx, CALL);
#undef CALL
#undef LAUNCH
    return hipGetLastError();
}

hipError_t launch_adj_steps(const Geo &G, const BlockGeo &T, const AdjRun &st, const float *nu_in, float *nu_out,
                            const float *fin, const float *fout, double *gin, double *gout, double *dtau_part,
                            const float *roi, int kind, hipStream_t s) {
    if (T.n_tiles == 0) return hipSuccess;
    const dim3 grid((unsigned)(T.n_tiles + (st.n_prev ? (G.n_ftiles + 1) / 2 : 0))), blk(2 * FT);
#define LAUNCH(B, SEED)                                                                                            \
    hipLaunchKernelGGL((k_adj_steps<B, 32, 16, 2 * FT, SEED>), grid, blk, 0, s, T.list, T.tile, nu_in, G.inst, T.ms, \
                       G.n_inst, st.n, T.n_tiles, G, st, nu_out, fin, fout, gin, gout, dtau_part, roi, kind)
#define CALL(B)                                            \
    do {                                                   \
        if (st.target) LAUNCH(B, true);                    \
        else LAUNCH(B, false);                             \
    } while (0)
    DISPATCH9(G.bcx, CALL);
#undef CALL
#undef LAUNCH
    return hipGetLastError();
}

hipError_t launch_dtau_sums(const Geo &G, const AdjRun &st, double *dtau_part, hipStream_t s) {
    if (G.n_ftiles == 0 || st.n_prev == 0) return hipSuccess;
    hipLaunchKernelGGL(k_dtau_sums, dim3((unsigned)G.n_ftiles), dim3(FT), 0, s, G, st, dtau_part);
    return hipGetLastError();
}

}  // namespace lbm
