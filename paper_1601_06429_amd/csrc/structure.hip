// structure.hip -- the full tessellation structure of the owned cells: every cell's vertices and
// its faces as vertex loops (the full structure output the paper mentions in section 3's
// memory figures and section 4's summary).  Output is CSR in output-row order:
//   vertices  vert_off[row] .. vert_off[row + 1], absolute coordinates (seed + offset);
//   faces     face_off[row] .. face_off[row + 1], ascending by the id across the face: the
//             neighbour's global id, or -1 .. -6 for the walls -x, +x, -y, +y, -z, +z of a
//             bounded item; a particle's face is kept if the particle is in the cell's facet
//             list (the faces of area > area_eps V^(2/3), the neighbour list), a wall if its
//             area is above that threshold;
//   loops     loop_off[f] .. loop_off[f + 1], vertex indices local to the cell, counter-clockwise
//             seen from outside, starting at the face's smallest index.
// Two passes over the cells: the first counts (vertices, faces, loop entries) per row, the host
// scans the counts, and the second writes.
//
// Nearly every cell has a topology record whose faces are all in its facet list.  Such a cell (of a
// bounded world only if no face is small enough to be of rounding's making: k_structure_count) is
// counted by one thread (its vertices, its faces, three loop entries per vertex), and written by
// k_structure_fast from the record alone: no face is dropped, the record's vertex triples are
// counter-clockwise seen from outside, so a loop needs no area to know its direction, and the faces'
// order is the rank of their ids.  A cell of the large clip kernel with F = V / 2 + 2 facets (a simple
// polytope has that many faces), none of them that small, is counted alike.  The others (faces dropped,
// walls, no record) are counted and written by k_structure: rebuilt, their face loops walked
// lane-parallel for area and direction, one face per lane, and sorted by id with a wave bitonic sort;
// cells with more than 64 vertices by its large variant with four vertex slots per lane.
//
// Bound by the latency of dependent loads (cell -> seed -> row -> offsets, tags -> positions) and of
// LDS.  400k clustered cells: the write pass 2.39 -> 0.42 ms (1.1 TB/s written; 79 vector registers
// and 4.6 KB of LDS a wavefront, six per SIMD, the scalars of 16 cells loaded by the lanes together),
// the count pass 0.48 -> 0.04 ms, the call with its sizing call 4.12 -> 0.98 ms.
#include "rebuild.h"

template <int VPL>
struct StructMem {
    double vp[64 * VPL][3];  // vertices, seed-relative
    uint32_t vt[64 * VPL];   // vertex triples (face slots)
    int32_t vidx[64 * VPL];  // local vertex index: rank among the cell's vertices
    int32_t flen[64 * VPL];  // loop length of each kept face slot, 0 otherwise
    int32_t frev[64 * VPL];  // 1: the walk runs clockwise seen from outside and is written reversed
    int32_t fl[64 * VPL];    // the cell's facet list (sorted indices of its neighbours)
    PolyMem<double, VPL> P;
};

struct StructArgs {
    CellSrc src;
    const DevItem *items;
    int n_items;
    const int32_t *cells;     // cell slot -> sorted index of its seed
    int64_t ncells;
    const int32_t *srow;      // sorted index -> output row
    const int32_t *sgid;      // sorted index -> global id
    const uint8_t *cstat;
    const double *cvol;
    const int32_t *queue;     // the clip's retry queue (cells with more than 64 vertices)
    int64_t queue_cap;
    int32_t *squeue;          // cells the normal kernel could not hold, for the large kernel
    int64_t squeue_cap;
    int32_t *slow;            // cells for the normal kernel
    uint8_t *smark;           // per cell slot: who writes it (MARK_*)
    uint32_t *counters;
    float area_eps;
    int write;                // 0: count, 1: write
    int64_t *nvert, *nface, *nloop;                  // counts per row (count pass)
    const int64_t *vert_off, *face_off, *loop_base;  // row offsets (write pass)
    double *verts;
    int32_t *face_nbr;
    int64_t *loop_off;
    int32_t *loop_vert;
};

// which kernel writes a cell: from its record, the normal kernel, the large kernel (counted already
// or by that kernel), or none (a failed cell)
enum { MARK_FAST = 0, MARK_SLOW = 1, MARK_LARGE = 2, MARK_LARGE_COUNTED = 3, MARK_NONE = 4 };

__device__ __forceinline__ int item_of(const DevItem *items, int n_items, int64_t p) {
    int lo = 0, hi = n_items - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (items[mid].start <= p) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// the vertex after u on face f walking the face's loop: u's triple names the face that shares
// the edge leaving u along f; the next vertex is the other vertex on both faces
template <int VPL>
__device__ __forceinline__ int loop_next(const PolyMem<double, VPL> &SP, const uint32_t *vt, int f, const uint64_t *mf,
                                         int u) {
    const uint32_t t = vt[u];
    const int t0 = t & 0xFF, t1 = (t >> 8) & 0xFF, t2 = (t >> 16) & 0xFF;
    const int cf = (t0 == f) ? t2 : (t1 == f) ? t0 : t1;
    int nx = -1;
#pragma unroll
    for (int ww = 0; ww < VPL; ++ww) {
        uint64_t x = mf[ww] & SP.fm[cf][ww];
        if (ww == (u >> 6)) x &= ~(1ull << (u & 63));
        if (nx < 0 && x) nx = ww * 64 + __builtin_ctzll(x);
    }
    return nx;
}

template <typename PT4, int VPL, bool RETRY>
__global__ void __launch_bounds__(256) k_structure(StructArgs A) {
    using M = StructMem<VPL>;
    extern __shared__ char smem[];
    M &S = *reinterpret_cast<M *>(smem + (size_t)(threadIdx.x >> 6) * sizeof(M));
    const int lane = lane_id();
    const uint64_t lt = lanemask_lt();
    const int64_t nq = RETRY ? (int64_t)min((uint64_t)A.counters[CTR_QUEUE], (uint64_t)A.queue_cap) : 0;
    const int64_t ntodo = RETRY ? nq + (int64_t)min((uint64_t)A.counters[CTR_STRUCT_Q], (uint64_t)A.squeue_cap)
                                : (int64_t)A.counters[CTR_STRUCT_SLOW];
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x >> 6);
    for (int64_t w = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); w < ntodo; w += nwaves) {
        const int32_t c = RETRY ? (w < nq ? A.queue[w] : A.squeue[w - nq]) : A.slow[w];
        const uint8_t mark = A.smark[c];
        // the write pass skips cells that the count pass handed to the large kernel
        if (mark == MARK_NONE || (!RETRY && mark != MARK_SLOW) || (RETRY && !A.write && mark == MARK_LARGE_COUNTED)) continue;
        const int32_t j0 = A.cells[c];
        const int64_t row = A.srow[j0];
        const DevItem it = uniform_item(A.items[item_of(A.items, A.n_items, j0)]);
        double xs[3];
        gpos<PT4>(A.src.spos, j0, xs[0], xs[1], xs[2]);
        double blo[3], bhi[3];
        for (int a = 0; a < 3; ++a) {
            if (it.periodic) {
                blo[a] = -0.5 * it.L[a];
                bhi[a] = 0.5 * it.L[a];
            } else {
                blo[a] = it.lo[a] - xs[a];
                bhi[a] = it.lo[a] + it.L[a] - xs[a];
            }
        }
        Poly<double, VPL> P;
        const int rb = rebuild_cell<PT4, VPL, RETRY>(A.src, it, S.P, P, c, xs[0], xs[1], xs[2], blo, bhi);
        if (rb == REBUILD_OVERFLOW) {
            if (lane == 0) {
                if (!A.write) {
                    A.smark[c] = MARK_LARGE;
                    const uint32_t qi = atomicAdd(&A.counters[CTR_STRUCT_Q], 1u);
                    if ((int64_t)qi < A.squeue_cap) A.squeue[qi] = c;
                    else atomicOr(&A.counters[CTR_STATUS], VT_DEV_CAPACITY);
                } else {
                    // counted from its record, but rebuilt from its facets here: no room was
                    // counted for what this pass would write
                    atomicOr(&A.counters[CTR_STATUS], VT_DEV_TOPOLOGY);
                }
            }
            continue;
        }
        bool failed = rb == REBUILD_FAILED;
        // ---- vertices: positions, triples and local indices in LDS
        int nv = 0;
#pragma unroll
        for (int s = 0; s < VPL; ++s) {
            const uint64_t am = P.alive[s];
            const int u = s * 64 + lane;
            if (am & (1ull << lane)) {
                S.vp[u][0] = P.vx[s];
                S.vp[u][1] = P.vy[s];
                S.vp[u][2] = P.vz[s];
                S.vt[u] = P.vt[s];
                S.vidx[u] = nv + __popcll(am & lt);
            }
            nv += __popcll(am);
        }
        wave_sync();
        // ---- the cell's facet list in LDS
        const int32_t fcnt = min(A.src.ccnt[c], 64 * VPL);
        const int64_t frow = A.src.crow[c];
        for (int t = lane; t < fcnt; t += 64) S.fl[t] = A.src.stage_ids[frow + t];
        wave_sync();
        // ---- faces: walk each loop once (one face slot per lane) for its length, area and
        // orientation; a particle's face is kept if the particle is in the facet list, a wall
        // if its area is above the facet threshold (as the clip kernel takes it)
        const double amin = (double)(A.area_eps * exp2f(log2f((float)fabs(A.cvol[c])) * (2.0f / 3.0f)));
        uint64_t key[VPL];
        bool open_loop = false;
#pragma unroll
        for (int r = 0; r < VPL; ++r) {
            const int f = r * 64 + lane;
            key[r] = ~0ull;
            int keep_len = 0, rev = 0;
            if (P.fa[r] & (1ull << lane)) {
                uint64_t mf[VPL];
                int u0 = -1, m = 0;
#pragma unroll
                for (int ww = 0; ww < VPL; ++ww) {
                    mf[ww] = S.P.fm[f][ww];
                    m += __popcll(mf[ww]);
                    if (u0 < 0 && mf[ww]) u0 = ww * 64 + __builtin_ctzll(mf[ww]);
                }
                // Newell's normal: N = sum of v_k x v_k+1 over the loop (twice the vector area)
                double nx = 0.0, ny = 0.0, nz = 0.0;
                int u = u0, k = 0;
                for (; k < m && u >= 0; ++k) {
                    const int un = loop_next<VPL>(S.P, S.vt, f, mf, u);
                    if (un < 0) {
                        u = -1;
                        break;
                    }
                    const double *p = S.vp[u], *q = S.vp[un];
                    nx += p[1] * q[2] - p[2] * q[1];
                    ny += p[2] * q[0] - p[0] * q[2];
                    nz += p[0] * q[1] - p[1] * q[0];
                    u = un;
                }
                if (m > 0 && (k != m || u != u0)) open_loop = true;
                // the area along the face's outward unit normal: negative if the walk runs
                // clockwise seen from outside
                const P4<double> &pl = S.P.pl64[f];
                const double sa = 0.5 * (nx * pl.x + ny * pl.y + nz * pl.z) / sqrt(pl.x * pl.x + pl.y * pl.y + pl.z * pl.z);
                const int32_t tag = S.P.ptag[f];
                bool keep = false;
                if (tag >= 0) {
                    for (int t = 0; t < fcnt; ++t) keep = keep || S.fl[t] == tag;
                } else {
                    keep = fabs(sa) > amin;
                }
                if (m >= 3 && keep) {
                    rev = sa < 0.0 ? 1 : 0;
                    keep_len = m;
                    const int64_t g = tag >= 0 ? (int64_t)A.sgid[tag] : (int64_t)tag;
                    key[r] = ((uint64_t)(g + 16) << 32) | (uint64_t)f;
                }
            }
            S.flen[f] = keep_len;
            S.frev[f] = rev;
        }
        wave_sync();
        if (__ballot(open_loop) != 0ull) failed = true;
        if (failed) {
            if (lane == 0) {
                atomicOr(&A.counters[CTR_STATUS], VT_DEV_TOPOLOGY);
                if (!A.write) A.nvert[row] = A.nface[row] = A.nloop[row] = 0;
            }
            continue;
        }
        // kept faces in ascending order of the id across them
        bitonic_u64<VPL>(key);
        int nkept = 0, nloop = 0;
#pragma unroll
        for (int r = 0; r < VPL; ++r) {
            const bool k = key[r] != ~0ull;
            nkept += __popcll(__ballot(k));
            nloop += uni_i(wave_sum_i(k ? S.flen[(int)(key[r] & 0xFFFFull)] : 0));
        }
        if (!A.write) {
            if (lane == 0) {
                A.nvert[row] = nv;
                A.nface[row] = nkept;
                A.nloop[row] = nloop;
            }
            continue;
        }
        // ---- write pass: only into the room the count pass made for this row
        const int64_t vb = A.vert_off[row], fb = A.face_off[row], lb = A.loop_base[row];
        if (A.vert_off[row + 1] - vb != nv || A.face_off[row + 1] - fb != nkept || A.loop_base[row + 1] - lb != nloop) {
            if (lane == 0) atomicOr(&A.counters[CTR_STATUS], VT_DEV_TOPOLOGY);
            continue;
        }
#pragma unroll
        for (int s = 0; s < VPL; ++s) {
            const int u = s * 64 + lane;
            if (P.alive[s] & (1ull << lane)) {
                const int64_t o = 3 * (vb + S.vidx[u]);
                A.verts[o + 0] = xs[0] + S.vp[u][0];
                A.verts[o + 1] = xs[1] + S.vp[u][1];
                A.verts[o + 2] = xs[2] + S.vp[u][2];
            }
        }
        int64_t carry = 0;
#pragma unroll
        for (int r = 0; r < VPL; ++r) {
            const int e = r * 64 + lane;
            const bool k = e < nkept;
            const int f = k ? (int)(key[r] & 0xFFFFull) : 0;
            const int m = k ? S.flen[f] : 0;
            int tot;
            const int pre = wave_excl_scan(m, &tot);
            if (k) {
                const int64_t lo = lb + carry + pre;
                A.face_nbr[fb + e] = (int32_t)((int64_t)(key[r] >> 32) - 16);
                A.loop_off[fb + e] = lo;
                uint64_t mf[VPL];
                int u0 = -1;
#pragma unroll
                for (int ww = 0; ww < VPL; ++ww) {
                    mf[ww] = S.P.fm[f][ww];
                    if (u0 < 0 && mf[ww]) u0 = ww * 64 + __builtin_ctzll(mf[ww]);
                }
                const bool rv = S.frev[f] != 0;
                int u = u0;
                for (int t = 0; t < m; ++t) {
                    // reversed: the start vertex stays first, the rest run backwards
                    const int pos = (rv && t > 0) ? m - t : t;
                    A.loop_vert[lo + pos] = S.vidx[u];
                    u = loop_next<VPL>(S.P, S.vt, f, mf, u);
                }
            }
            carry += tot;
        }
    }
}

// The count pass, one thread per cell: the counts that follow without rebuilding the cell, and who
// writes it.
__global__ void __launch_bounds__(256) k_structure_count(StructArgs A) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool slow = false;
    if (c < A.ncells) {
        const uint8_t st = A.cstat[c];
        const int64_t row = A.srow[A.cells[c]];
        const int nf = A.src.cnf[c], nv = A.src.cnv[c], fc = A.src.ccnt[c];
        int64_t v = 0, f = 0;
        uint8_t mark = MARK_SLOW;
        // Counted without being rebuilt, a cell whose loops do not close has room but nothing to put
        // there.  A facet threshold from 1e-12 on keeps no face that rounding could make or move.
        const bool sure = A.area_eps >= 1e-12f;
        if (st & VT_CELL_FAILED) {
            mark = MARK_NONE;
        } else if (st & VT_CELL_RETRIED) {
            mark = sure && nv >= 4 && 2 * fc == nv + 4 ? MARK_LARGE_COUNTED : MARK_LARGE;
        } else if (nf >= 4 && nf <= VT_TOPO_FACES && nv >= 4 && nv <= 64 && fc == nf &&
                   (sure || A.items[item_of(A.items, A.n_items, A.cells[c])].periodic)) {
            mark = MARK_FAST;
        }
        if (mark == MARK_FAST || mark == MARK_LARGE_COUNTED) {
            v = nv;
            f = fc;
        }
        A.smark[c] = mark;
        A.nvert[row] = v;
        A.nface[row] = f;
        A.nloop[row] = 3 * v;
        slow = mark == MARK_SLOW;
    }
    const uint64_t m = __ballot(slow);
    if (m != 0ull) {
        uint32_t base = 0;
        if (lane_id() == 0) base = atomicAdd(&A.counters[CTR_STRUCT_SLOW], (uint32_t)__popcll(m));
        base = readlane_u32(base, 0);
        if (slow) A.slow[base + rank_in(m)] = (int32_t)c;
    }
}

// The write pass for cells written from their records.
struct FastMem {
    P4<double> pl[VT_TOPO_FACES];
    uint64_t fm[VT_TOPO_FACES];            // vertices on each face
    uint8_t next[VT_TOPO_FACES][64];       // next[f][u]: the vertex after u on face f
    int32_t order[64];                     // the faces by ascending id
    uint8_t loop[3 * 64];                  // the cell's loop entries
};
#define STRUCT_BATCH 16

template <typename PT4>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) k_structure_fast(StructArgs A) {
    __shared__ FastMem Ms[4];
    FastMem &S = Ms[threadIdx.x >> 6];
    const int lane = lane_id();
    // each XCD (blocks are dealt to them in turn) takes one contiguous eighth of the Morton order
    const int seg = (int)(blockIdx.x % VT_XCD_SEGMENTS);
    const int64_t c_end = A.ncells * (seg + 1) / VT_XCD_SEGMENTS;
    const int64_t step = (int64_t)(gridDim.x / VT_XCD_SEGMENTS) * 4 * STRUCT_BATCH;
    for (int64_t c0 = A.ncells * seg / VT_XCD_SEGMENTS + ((int64_t)(blockIdx.x / VT_XCD_SEGMENTS) * 4 + (threadIdx.x >> 6)) * STRUCT_BATCH;
         c0 < c_end; c0 += step) {
        // the batch's scalars, a cell per lane
        const int64_t cl = c0 + lane;
        bool todo = lane < STRUCT_BATCH && cl < c_end;
        if (todo) todo = A.smark[cl] == MARK_FAST;
        int nf_l = 0, nv_l = 0, item_l = 0;
        int64_t vb_l = 0, fb_l = 0, lb_l = 0;
        double x_l = 0.0, y_l = 0.0, z_l = 0.0;
        if (todo) {
            const int32_t j0 = A.cells[cl];
            nf_l = A.src.cnf[cl];
            nv_l = A.src.cnv[cl];
            const int64_t row = A.srow[j0];
            gpos<PT4>(A.src.spos, j0, x_l, y_l, z_l);
            item_l = item_of(A.items, A.n_items, j0);
            vb_l = A.vert_off[row];
            fb_l = A.face_off[row];
            lb_l = A.loop_base[row];
        }
        for (uint64_t m = __ballot(todo); m; m &= m - 1) {
            const int i = uni_i(__builtin_ctzll(m));
            const int64_t c = c0 + i;
            const int nf = (int)readlane_u32((uint32_t)nf_l, i), nv = (int)readlane_u32((uint32_t)nv_l, i);
            const double sx = readlane_dbl(x_l, i), sy = readlane_dbl(y_l, i), sz = readlane_dbl(z_l, i);
            const DevItem &it = A.items[(int)readlane_u32((uint32_t)item_l, i)];
            auto readlane_i64 = [&](int64_t v) {
                return (int64_t)(((uint64_t)readlane_u32((uint32_t)((uint64_t)v >> 32), i) << 32) |
                                 readlane_u32((uint32_t)(uint64_t)v, i));
            };
            const int64_t vb = readlane_i64(vb_l), fb = readlane_i64(fb_l), lb = readlane_i64(lb_l);
            const int32_t *rec = A.src.ctopo + c * VT_TOPO_STRIDE;
            int32_t tag = -1, gid = 0;
            uint32_t t = 0;
            if (lane < nf) tag = rec[lane];
            if (lane < nv) t = (uint32_t)rec[VT_TOPO_FACES + lane];
            const int k[3] = {(int)(t & 0xFFu), (int)((t >> 8) & 0xFFu), (int)((t >> 16) & 0xFFu)};
            // a record that fails a check can only come from a fault of the clip kernel (rebuild.h)
            bool ok = true;
            if (lane < nf) ok = tag >= 0 && (int64_t)tag < A.src.npos;
            if (lane < nv) ok = ok && (t >> 24) == 0 && k[0] < nf && k[1] < nf && k[2] < nf && k[0] != k[1] && k[1] != k[2] && k[0] != k[2];
            bool bad = __ballot(!ok) != 0ull;
            double x = 0.0, y = 0.0, z = 0.0;
            if (!bad) {
                if (lane < nf) {
                    double qx, qy, qz;
                    gpos<PT4>(A.src.spos, tag, qx, qy, qz);
                    gid = A.sgid[tag];
                    // the expressions of rebuild.h, so the vertices are the clip kernel's own
                    qx -= sx;
                    qy -= sy;
                    qz -= sz;
                    if (it.periodic) {
                        qx -= it.L[0] * rint(qx * (1.0 / it.L[0]));
                        qy -= it.L[1] * rint(qy * (1.0 / it.L[1]));
                        qz -= it.L[2] * rint(qz * (1.0 / it.L[2]));
                    }
                    S.pl[lane] = P4<double>{qx, qy, qz, 0.5 * (qx * qx + qy * qy + qz * qz)};
                    S.fm[lane] = 0ull;
                }
                wave_sync();
                if (lane < nv) {
                    intersect3<double>(S.pl[k[0]], S.pl[k[1]], S.pl[k[2]], x, y, z);
                    for (int e = 0; e < 3; ++e) atomicOr((unsigned long long *)&S.fm[k[e]], 1ull << lane);
                }
                bad = __ballot(!(isfinite(x) && isfinite(y) && isfinite(z))) != 0ull;
                wave_sync();
                // on face k[e] the next vertex also lies on the face before k[e] in the triple
                if (lane < nv) {
                    for (int e = 0; e < 3; ++e) {
                        const uint64_t w = S.fm[k[e]] & S.fm[k[(e + 2) % 3]] & ~(1ull << lane);
                        S.next[k[e]][lane] = (uint8_t)(w ? __builtin_ctzll(w) : 255);
                    }
                }
            }
            if (bad) {
                if (lane == 0) {
                    atomicAdd(&A.counters[CTR_REC_REJECT], 1u);
                    atomicOr(&A.counters[CTR_STATUS], VT_DEV_TOPOLOGY);
                }
                continue;
            }
            // the faces by ascending id, then slot (k_structure's key)
            int rank = 0;
            const uint32_t key = (uint32_t)gid + 16u;
            for (int q = 0; q < nf; ++q) {
                const uint32_t g = readlane_u32(key, q);
                rank += g < key || (g == key && q < lane) ? 1 : 0;
            }
            if (lane < nf) S.order[rank] = lane;
            wave_sync();
            const int f = lane < nf ? S.order[lane] : 0;
            const uint64_t mf = S.fm[f];
            const int len = lane < nf ? __popcll(mf) : 0;
            const int32_t fid = __shfl(gid, f);
            int total;
            const int pre = wave_excl_scan(len, &total);
            bool open_loop = total != 3 * nv;
            if (lane < nf && !open_loop) {
                const int u0 = __builtin_ctzll(mf);
                int u = u0;
                for (int q = 0; q < len; ++q) {
                    S.loop[pre + q] = (uint8_t)u;
                    u = S.next[f][u & 63];
                }
                open_loop = len < 3 || u != u0;
            }
            if (__ballot(open_loop) != 0ull) {
                if (lane == 0) atomicOr(&A.counters[CTR_STATUS], VT_DEV_TOPOLOGY);
                continue;
            }
            wave_sync();
            if (lane < nf) {
                A.face_nbr[fb + lane] = fid;
                A.loop_off[fb + lane] = lb + pre;
            }
            if (lane < nv) {
                double *v = A.verts + 3 * (vb + lane);
                v[0] = sx + x;
                v[1] = sy + y;
                v[2] = sz + z;
            }
            for (int q = lane; q < total; q += 64) A.loop_vert[lb + q] = S.loop[q];
            wave_sync();
        }
    }
}

// after the scans: the totals in one place for the host
__global__ void k_structure_totals(const int64_t *vert_off, const int64_t *face_off, const int64_t *lbase, int64_t n,
                                   int64_t *tot) {
    if (threadIdx.x == 0) {
        tot[0] = vert_off[n];
        tot[1] = face_off[n];
        tot[2] = lbase[n];
    }
}

__global__ void k_store_last(int64_t *dst, const int64_t *src) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *dst = *src;
}

template <typename PT4, int VPL, bool RETRY>
static hipError_t launch_structure_one(vt_ctx *c, StructArgs &a, int wpb) {
    const size_t lds = sizeof(StructMem<VPL>) * (size_t)wpb;
    auto kern = k_structure<PT4, VPL, RETRY>;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    int ncu = 0;
    hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, c->device);
    if (ncu <= 0) ncu = 256;
    const int64_t blocks = RETRY ? (int64_t)ncu : (int64_t)ncu * 16 / wpb;
    kern<<<dim3((unsigned)blocks), dim3(64 * wpb), lds, c->stream>>>(a);
    return hipGetLastError();
}

static hipError_t structure_pass(vt_ctx *c, StructArgs &a) {
    hipError_t e;
    if (c->dtype == VT_F32) {
        e = launch_structure_one<float4, 1, false>(c, a, 4);
        if (e == hipSuccess) e = launch_structure_one<float4, 4, true>(c, a, 1);
    } else {
        e = launch_structure_one<double4, 1, false>(c, a, 4);
        if (e == hipSuccess) e = launch_structure_one<double4, 4, true>(c, a, 1);
    }
    return e;
}

void vt_struct_free(vt_ctx *c) {
    (void)hipFree(c->st_cnt);
    (void)hipFree(c->st_lbase);
    (void)hipFree(c->st_tmp);
    (void)hipFree(c->st_slow);
    (void)hipFree(c->smark);
    (void)hipFree(c->squeue);
    c->st_cnt = c->st_lbase = c->st_tmp = nullptr;
    c->st_slow = nullptr;
    c->smark = nullptr;
    c->squeue = nullptr;
    c->cap_struct = c->cap_squeue = 0;
}

static hipError_t reserve_structure(vt_ctx *c) {
    const int64_t n = c->n_owned;
    if (c->cap_struct >= n && c->cap_squeue >= c->cap_retry && c->st_cnt) return hipSuccess;
    vt_struct_free(c);
    hipError_t e = hipMalloc(&c->st_cnt, sizeof(int64_t) * 3 * (size_t)n);
    if (e == hipSuccess) e = hipMalloc(&c->st_lbase, sizeof(int64_t) * (size_t)(n + 1));
    if (e == hipSuccess) e = hipMalloc(&c->st_tmp, sizeof(int64_t) * 3 * (size_t)(1 + vt_scan_tmp_elems(n)));
    if (e == hipSuccess) e = hipMalloc(&c->st_slow, sizeof(int32_t) * (size_t)n);
    if (e == hipSuccess) e = hipMalloc(&c->smark, (size_t)n);
    if (e == hipSuccess) e = hipMalloc(&c->squeue, sizeof(int32_t) * (size_t)c->cap_retry);
    if (e == hipSuccess) {
        c->cap_struct = n;
        c->cap_squeue = c->cap_retry;
    } else {
        vt_struct_free(c);
    }
    return e;
}

// Count, scan, and (if the capacities suffice) write.  sizes[] gets the totals of vertices,
// faces and loop entries; *fits is false when one of them exceeds its capacity (then only the
// offsets are written).  Synchronizes the stream to read the totals.
hipError_t vt_launch_structure(vt_ctx *c, int64_t *vert_off, double *verts, int64_t vert_cap, int64_t *face_off,
                               int32_t *face_nbr, int64_t face_cap, int64_t *loop_off, int32_t *loop_vert,
                               int64_t loop_cap, int64_t sizes[3], bool *fits) {
    const int64_t n = c->n_owned;
    hipError_t e = reserve_structure(c);
    if (e != hipSuccess) return e;
    StructArgs a;
    a.src = CellSrc{c->spos, c->ctopo, c->cnf, c->cnv, c->n_total, c->crow, c->ccnt, c->stage_ids, c->counters};
    a.items = c->items;
    a.n_items = c->n_items;
    a.cells = c->cells;
    a.ncells = n;
    a.srow = c->srow;
    a.sgid = c->sgid;
    a.cstat = c->cstat;
    a.cvol = c->cvol;
    a.queue = c->queue;
    a.queue_cap = c->cap_retry;
    a.squeue = c->squeue;
    a.squeue_cap = c->cap_retry;
    a.slow = c->st_slow;
    a.smark = c->smark;
    a.counters = c->counters;
    a.area_eps = c->opts.area_eps > 0 ? c->opts.area_eps : 1e-12f;
    a.write = 0;
    a.nvert = c->st_cnt;
    a.nface = c->st_cnt + n;
    a.nloop = c->st_cnt + 2 * n;
    a.vert_off = vert_off;
    a.face_off = face_off;
    a.loop_base = c->st_lbase;
    a.verts = verts;
    a.face_nbr = face_nbr;
    a.loop_off = loop_off;
    a.loop_vert = loop_vert;
    int64_t *totals = c->st_tmp + 3 * vt_scan_tmp_elems(n);
    e = vt_launch_zero_u32(c->counters + CTR_STRUCT_SLOW, 1, c->stream);
    if (e == hipSuccess) e = vt_launch_zero_u32(c->counters + CTR_STRUCT_Q, 1, c->stream);
    if (e != hipSuccess) return e;
    k_structure_count<<<(unsigned)((n + 255) / 256), 256, 0, c->stream>>>(a);
    e = hipGetLastError();
    if (e == hipSuccess) e = structure_pass(c, a);
    if (e == hipSuccess) e = vt_launch_scan3_i64(a.nvert, vert_off, face_off, c->st_lbase, n, c->st_tmp, c->stream);
    if (e != hipSuccess) return e;
    k_structure_totals<<<1, 64, 0, c->stream>>>(vert_off, face_off, c->st_lbase, n, totals);
    int64_t tot[3];
    e = hipMemcpyAsync(tot, totals, sizeof(tot), hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) return e;
    for (int k = 0; k < 3; ++k) sizes[k] = tot[k];
    *fits = tot[0] <= vert_cap && tot[1] <= face_cap && tot[2] <= loop_cap && verts && face_nbr && loop_off && loop_vert;
    if (!*fits) return hipSuccess;
    a.write = 1;
    int ncu = 0;
    hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, c->device);
    if (ncu <= 0) ncu = 256;
    // six blocks of four wavefronts per CU, a multiple of the XCDs
    const unsigned blocks = (unsigned)((ncu * 6 + VT_XCD_SEGMENTS - 1) / VT_XCD_SEGMENTS * VT_XCD_SEGMENTS);
    if (c->dtype == VT_F32) k_structure_fast<float4><<<blocks, 256, 0, c->stream>>>(a);
    else k_structure_fast<double4><<<blocks, 256, 0, c->stream>>>(a);
    e = hipGetLastError();
    if (e == hipSuccess) e = structure_pass(c, a);
    if (e == hipSuccess) {
        k_store_last<<<1, 64, 0, c->stream>>>(loop_off + tot[1], c->st_lbase + n);
        e = hipGetLastError();
    }
    return e;
}
