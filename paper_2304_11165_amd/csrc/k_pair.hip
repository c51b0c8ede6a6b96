// k_pair.hip -- two steps of 8^3 blocks in one launch, column form, block layout.
//
// One wave per block.  The second step of a block needs the first step's values of the
// block and of the six face layers around it, so the wave computes those itself from a
// halo of two layers: the block (8 planes), the layer across each face and the one behind
// it, and the 12 edge lines, 1376 values for 896 + 512 updates.  The first step's values
// of the faces are computed twice, here and in the neighbour, with the same operations and
// rounding, so the fields equal those of two launches bit for bit.
//
// A single step is bound by its traffic past the L2 (large lists) or by the launch and one
// chain of latencies (short ones); a pair has one of each for two steps, and the second
// layers and edges lie in cache lines that the first layers touch anyway.  What it adds is
// arithmetic (22 plane updates where two steps take 16), and it is bound by that and by the
// latency of its loads.  us per step, single and paired: one species FP32 packing 64^3 3.3 /
// 2.76, 160^3 8.7 / 6.95, soil 256^3 16.9 / 12.7; FP16 7.7 / 6.5 and 13.5 / 11.8 (160^3,
// 256^3); BF16 with stochastic rounding 9.0 / 7.7 and 16.1 / 14.0; two species FP32 17.9 /
// 11.7 and 30.2 / 21.2, BF16 with stochastic rounding 13.8 / 12.1 and 23.8 / 21.5.
// All 10^3 values of a wave sit in LDS at once (4 KB per species and wave), so a step needs
// no order among its planes.
#include <type_traits>

#include "rd_device.h"
#include "rd_diff.h"

namespace {
constexpr int PY = 10, PZ = 100;  // strides of the 10^3 tile of a wave
__device__ __forceinline__ int tpos(int x, int y, int z) { return (z + 1) * PZ + (y + 1) * PY + (x + 1); }

__device__ __forceinline__ void wave_sync()  // the wave's LDS writes before its reads of other lanes' words
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The value a store into T would hold, with the rounding of the step kernels.
template <typename T, bool SR>
__device__ __forceinline__ float stored(float v, uint32_t rnd)
{
    if constexpr (std::is_same<T, float>::value) return v;
    else if constexpr (!SR) return rd_round<T>(v);
    else if constexpr (std::is_same<T, bf16_t>::value) return __uint_as_float((uint32_t)bf16_sr(v, rnd) << 16);
    else return (float)f16_sr(v, rnd);
}

// MID: the first step's field is stored too (a.cmid).  FAC: with the diffusivity factor fe,
// the operations of k_step8e (FP32 rounds to nearest); its halo is the fields', and the face
// voxels' code bytes tell which of their neighbours are active.
template <typename T, int S, bool SR, bool MID, bool FAC>
__device__ __forceinline__ void pair8z(const StepArgs &a, const float *fe)
{
    constexpr bool DITHER = !FAC && SR && std::is_same<T, float>::value;
    __shared__ float tile[4][FAC ? S + 1 : S][1000];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int b = __builtin_amdgcn_readfirstlane(map_group(blockIdx.x, a.xcd_chunk) * 4 + wv);
    if (b >= a.nb) return;
    const int lx = lane & 7, ly = lane >> 3;
    const T *cin = (const T *)a.cin;
    const T *own[S];
    T *out[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
        own[s] = uniform_ptr(cin + s * a.sstride + (int64_t)b * 512);
        out[s] = uniform_ptr((T *)a.cout + s * a.sstride + (int64_t)b * 512);
    }
    const BlockInfo bi = a.info[b];
    const uint64_t *rec = a.mask + (int64_t)b * 16;
    uint64_t Wo[8], Wf[6];
#pragma unroll
    for (int z = 0; z < 8; ++z) Wo[z] = rec[z];
#pragma unroll
    for (int f = 0; f < 6; ++f) Wf[f] = rec[8 + f];
    typedef typename RawOf<T>::type R;
    R rc[S][8], r1[S][6], r2[S][6], re[S][2];
    float ec[8], e1[6], e2[6], ee[2];  // FAC: the factor
    const float *eown = FAC ? uniform_ptr(fe + (int64_t)b * 512) : nullptr;
    const uint32_t ncw = a.ncnt[(int64_t)b * 64 + lane];
    uint32_t fcw[6];
#pragma unroll
    for (int z = 0; z < 8; ++z) {
#pragma unroll
        for (int s = 0; s < S; ++s) rc[s][z] = (R)0;
        ec[z] = 0.0f;
        if (lane_bit(Wo[z])) {
            if (FAC) ec[z] = *at_byte(eown, (uint32_t)(z * 64 + lane) * 4u);
#pragma unroll
            for (int s = 0; s < S; ++s)
                rc[s][z] = ld_raw(at_byte(own[s], (uint32_t)(z * 64 + lane) * (uint32_t)sizeof(T)), 0);
        }
    }
    // the two layers across face f at face coordinates (u, v) = (lx, ly), and the count word
    // of the first (a voxel of the layer behind an inactive one is not needed)
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        int s1, s2, col;  // slots of the layers, lane of the count word
        switch (f) {
        case 0: s1 = lane * 8 + 7; s2 = s1 - 1; col = lx * 8 + 7; break;
        case 1: s1 = lane * 8; s2 = s1 + 1; col = lx * 8; break;
        case 2: s1 = ly * 64 + 56 + lx; s2 = s1 - 8; col = 56 + lx; break;
        case 3: s1 = ly * 64 + lx; s2 = s1 + 8; col = lx; break;
        case 4: s1 = 448 + lane; s2 = s1 - 64; col = lane; break;
        default: s1 = lane; s2 = s1 + 64; col = lane; break;
        }
        const int n = bi.nbr[f] >= 0 ? bi.nbr[f] : b;
#pragma unroll
        for (int s = 0; s < S; ++s) r1[s][f] = r2[s][f] = (R)0;
        // (the count word unconditionally: under the predicate its extraction would be folded
        // into the branch and wait there for the loads before it)
        if (FAC) fcw[f] = *at_byte(uniform_ptr(a.code + (int64_t)n * 512), (uint32_t)s1);
        else fcw[f] = *at_byte(uniform_ptr(a.ncnt + (int64_t)n * 64), (uint32_t)col * 4u);
        e1[f] = e2[f] = 0.0f;
        if (lane_bit(Wf[f])) {
            if (FAC) {
                const float *nb = uniform_ptr(fe + (int64_t)n * 512);
                e1[f] = *at_byte(nb, (uint32_t)s1 * 4u);
                e2[f] = *at_byte(nb, (uint32_t)s2 * 4u);
            }
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const T *nb = uniform_ptr(cin + s * a.sstride + (int64_t)n * 512);
                r1[s][f] = ld_raw(at_byte(nb, (uint32_t)s1 * (uint32_t)sizeof(T)), 0);
                r2[s][f] = ld_raw(at_byte(nb, (uint32_t)s2 * (uint32_t)sizeof(T)), 0);
            }
        }
    }
    // edge lines: the block across faces f and d through either face block that exists
    // (an edge without one has no active face voxel beside it)
    int en[12];
    {
        int32_t nn[6][6];
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            const BlockInfo ni = a.info[bi.nbr[f] >= 0 ? bi.nbr[f] : b];
#pragma unroll
            for (int d = 0; d < 6; ++d) nn[f][d] = bi.nbr[f] >= 0 ? ni.nbr[d] : -1;
        }
#pragma unroll
        for (int e = 0; e < 12; ++e) {  // xy, xz, yz; bit 0 and 1 of e the sides
            const int f = (e < 8 ? 0 : 2) + (e & 1), d = (e < 4 ? 2 : 4) + ((e >> 1) & 1);
            en[e] = nn[f][d] >= 0 ? nn[f][d] : nn[d][f];
        }
    }
    // lane 8 e + k holds value k of line e (xy and xz lines), then of line 8 + e (yz)
    const int sa = (lane >> 3) & 1, sb = (lane >> 4) & 1;
    const bool xy = lane < 32;
    int eb[2] = {-1, -1};
#pragma unroll
    for (int e = 0; e < 8; ++e) eb[0] = lane_bit(0xffull << (8 * e)) ? en[e] : eb[0];
#pragma unroll
    for (int e = 0; e < 4; ++e) eb[1] = lane_bit(0xffull << (8 * e)) ? en[8 + e] : eb[1];
    const int es0 = (xy ? lx * 64 + (sb ? 0 : 56) : (sb ? 0 : 448) + lx * 8) + (sa ? 0 : 7);
    const int es1 = (sb ? 0 : 448) + (sa ? 0 : 56) + lx;
    // without a predicate, the block's first slot where the edge block is missing (a select at
    // the use: a predicated value was copied, and waited for, between the two loads)
    const int64_t eo[2] = {eb[0] >= 0 ? (int64_t)eb[0] * 512 + es0 : (int64_t)b * 512,
                           eb[1] >= 0 ? (int64_t)eb[1] * 512 + es1 : (int64_t)b * 512};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
#pragma unroll
        for (int s = 0; s < S; ++s) re[s][k] = ld_raw(cin + s * a.sstride, eo[k]);
        ee[k] = FAC ? fe[eo[k]] : 0.0f;
    }

    // all loads are issued
    float c[S][8], h1[S][6], h2[S][6];
    const int fp[6] = {tpos(-1, lx, ly), tpos(8, lx, ly), tpos(lx, -1, ly),
                       tpos(lx, 8, ly),  tpos(lx, ly, -1), tpos(lx, ly, 8)};
    const int ep0 = xy ? tpos(sa ? 8 : -1, sb ? 8 : -1, lx) : tpos(sa ? 8 : -1, lx, sb ? 8 : -1);
#pragma unroll
    for (int s = 0; s < S; ++s) {
        float *t = tile[wv][s];
#pragma unroll
        for (int z = 0; z < 8; ++z) {
            c[s][z] = from_raw<T>(rc[s][z]);
            t[tpos(lx, ly, z)] = c[s][z];
        }
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            h1[s][f] = from_raw<T>(r1[s][f]);
            h2[s][f] = from_raw<T>(r2[s][f]);
            t[fp[f]] = h1[s][f];
        }
        t[ep0] = eb[0] >= 0 ? from_raw<T>(re[s][0]) : 0.0f;
        if (lane < 32) t[tpos(lx, sa ? 8 : -1, sb ? 8 : -1)] = eb[1] >= 0 ? from_raw<T>(re[s][1]) : 0.0f;
    }
    if constexpr (FAC) {
        float *t = tile[wv][S];
#pragma unroll
        for (int z = 0; z < 8; ++z) t[tpos(lx, ly, z)] = ec[z];
#pragma unroll
        for (int f = 0; f < 6; ++f) t[fp[f]] = e1[f];
        t[ep0] = eb[0] >= 0 ? ee[0] : 0.0f;
        if (lane < 32) t[tpos(lx, sa ? 8 : -1, sb ? 8 : -1)] = eb[1] >= 0 ? ee[1] : 0.0f;
    }
    wave_sync();

    int bx, by, bz, gid;
    block_pos(bi, &bx, &by, &bz, &gid);
    const GeomInfo g = a.geom[gid];
    const int gx = bx * 8 + lx, gy = by * 8 + ly;
    // some voxel of the block or of its face layers on a box face
    const bool bnd = bx == 0 || by == 0 || bz == 0 || bx * 8 + 9 >= g.nx || by * 8 + 9 >= g.ny || bz * 8 + 9 >= g.nz;
    const uint32_t ctr = SR ? *a.ctr + a.ctr_off : 0u;
    const uint32_t key = SR ? sr_key(ctr, a.seed) : 0u;
    const uint32_t colw = SR ? sr_column(g, gx, gy, key) : 0u;
    // per voxel: neighbours, walls (in-box neighbours that are not active), and per species the
    // lanes whose value changes (active, not on a held face: the others keep theirs, 0 where
    // inactive); the box faces come in for boundary blocks only
    float na[8], nw[8], fna[6], fnw[6];
    uint64_t Uo[S][8], Uf[S][6];
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        na[z] = (float)((ncw >> (3 * z)) & 7u);
        nw[z] = 6.0f - na[z];
#pragma unroll
        for (int s = 0; s < S; ++s) Uo[s][z] = Wo[z];
    }
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        fna[f] = FAC ? (float)__popc(fcw[f] & 63u) : (float)((fcw[f] >> (f == 4 ? 21 : f == 5 ? 0 : 3 * ly)) & 7u);
        fnw[f] = 6.0f - fna[f];
#pragma unroll
        for (int s = 0; s < S; ++s) Uf[s][f] = Wf[f];
    }
    auto face_xyz = [&](int f, int *x, int *y, int *z) {
        *x = f == 0 ? bx * 8 - 1 : f == 1 ? bx * 8 + 8 : gx;
        *y = f < 2 ? by * 8 + lx : f == 2 ? by * 8 - 1 : f == 3 ? by * 8 + 8 : gy;
        *z = f < 4 ? bz * 8 + ly : f == 4 ? bz * 8 - 1 : bz * 8 + 8;
    };
    if (bnd) {
#pragma unroll
        for (int z = 0; z < 8; ++z) {
            const unsigned onf = box_faces(g, gx, gy, bz * 8 + z);
            nw[z] -= (float)__popc(onf);
#pragma unroll
            for (int s = 0; s < S; ++s) Uo[s][z] &= ~__ballot((onf & a.coef[s].dir) != 0u);
        }
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            int x, y, z;
            face_xyz(f, &x, &y, &z);
            const unsigned onf = box_faces(g, x, y, z);
            fnw[f] -= (float)__popc(onf);
#pragma unroll
            for (int s = 0; s < S; ++s) Uf[s][f] &= ~__ballot((onf & a.coef[s].dir) != 0u);
        }
    }
    auto update = [&](int s, const float *cen, const float *nbv, const float *w, float nact, float nwall, uint64_t U,
                      uint32_t h) {
        if constexpr (FAC) {  // as k_step8e
            const SpeciesCoef &k = a.coef[s];
            const float uc = cen[s];
            float lap = 0.0f;
#pragma unroll
            for (int d = 0; d < 6; ++d) lap = fmaf(w[d], nbv[d] - uc, lap);
            float r = fmaf(k.alpha, lap, uc);
            r = fmaf(-fmaf(k.gamma, nwall, k.beta), uc, r);
#pragma unroll
            for (int q = 0; q < S; ++q) r = fmaf(k.K[q], cen[q], r);
            return lane_bit(U) ? r : uc;
        }
        const float dth = DITHER ? fp32_dither(cen[s], sr_species(h, s)) : 0.0f;
        const float r = rd_update_n<S, DITHER>(cen[s], nbv, nact, nwall, a.coef[s], cen, s, dth);
        return lane_bit(U) ? r : cen[s];
    };
    // step 1 of the face layers
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        float r[S];
#pragma unroll
        for (int s = 0; s < S; ++s) r[s] = 0.0f;
        if (Wf[f] != 0ull) {
            const int off[6] = {-1, 1, -PY, PY, -PZ, PZ};
            int x, y, z;
            face_xyz(f, &x, &y, &z);
            const uint32_t h = SR ? sr_combine(f < 4 ? sr_column(g, x, y, key) : colw, sr_plane(z, key)) : 0u;
            float cen[S];
#pragma unroll
            for (int s = 0; s < S; ++s) cen[s] = h1[s][f];
            float w[6];
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                w[q] = 0.0f;
                if (FAC) {
                    const float en_ = q == f ? e2[f] : tile[wv][FAC ? S : 0][fp[f] + (q == f ? 0 : off[q])];
                    w[q] = (fcw[f] >> q) & 1u ? 0.5f * (e1[f] + en_) : 0.0f;
                }
            }
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const float *p = tile[wv][s] + fp[f];
                float nbv[6];
#pragma unroll
                for (int d = 0; d < 6; ++d) nbv[d] = d == f ? h2[s][f] : p[d == f ? 0 : off[d]];
                r[s] = stored<T, SR>(update(s, cen, nbv, w, fna[f], fnw[f], Uf[s][f], h), sr_species(h, s));
            }
        }
#pragma unroll
        for (int s = 0; s < S; ++s) h2[s][f] = r[s];
    }
    BlockMasks M;  // FAC: which faces of the block's voxels join two active ones
    if constexpr (FAC) M.load(rec);
    auto weight = [](float ep, float eq, uint64_t both) { return lane_bit(both) ? 0.5f * (ep + eq) : 0.0f; };
    // one step of plane z, from the values v of the block's column, the layers below and above
    // and the tile
    auto plane = [&](int z, const float (*v)[8], const float (*hz)[6], uint32_t h, float *r) {
        float cen[S];
#pragma unroll
        for (int s = 0; s < S; ++s) cen[s] = v[s][z];
        float w[6];
        if constexpr (FAC) {
            const float *p = tile[wv][S] + tpos(lx, ly, z);
            const float en_[6] = {p[-1], p[1], p[-PY], p[PY], z == 0 ? e1[4] : ec[z > 0 ? z - 1 : 0],
                                  z == 7 ? e1[5] : ec[z < 7 ? z + 1 : 7]};
#pragma unroll
            for (int q = 0; q < 6; ++q) w[q] = weight(ec[z], en_[q], M.pair(z, q));
        }
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const float *p = tile[wv][s] + tpos(lx, ly, z);
            const float nbv[6] = {p[-1], p[1], p[-PY], p[PY], z == 0 ? hz[s][4] : v[s][z > 0 ? z - 1 : 0],
                                  z == 7 ? hz[s][5] : v[s][z < 7 ? z + 1 : 7]};
            r[s] = update(s, cen, nbv, w, na[z], nw[z], Uo[s][z], h);
        }
    };
    float u[S][8];
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        const uint32_t h = SR ? sr_combine(colw, sr_plane(bz * 8 + z, key)) : 0u;
        float r[S];
        plane(z, c, h1, h, r);
#pragma unroll
        for (int s = 0; s < S; ++s) u[s][z] = stored<T, SR>(r[s], sr_species(h, s));
    }
    if constexpr (MID) {  // (rounded already)
#pragma unroll
        for (int s = 0; s < S; ++s) {
            T *o = uniform_ptr((T *)a.cmid + s * a.sstride + (int64_t)b * 512);
#pragma unroll
            for (int z = 0; z < 8; ++z)
                if (lane_bit(sector_lanes<T>(Wo[z])))
                    rd_st(at_byte(o, (uint32_t)(z * 64 + lane) * (uint32_t)sizeof(T)), 0, u[s][z]);
        }
    }
    wave_sync();
#pragma unroll
    for (int s = 0; s < S; ++s) {
        float *t = tile[wv][s];
#pragma unroll
        for (int z = 0; z < 8; ++z) t[tpos(lx, ly, z)] = u[s][z];
#pragma unroll
        for (int f = 0; f < 4; ++f) t[fp[f]] = h2[s][f];
    }
    wave_sync();
    // step 2 of the block
    const uint32_t key2 = SR ? sr_key(ctr + 1u, a.seed) : 0u;
    const uint32_t colw2 = SR ? sr_column(g, gx, gy, key2) : 0u;
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        const uint32_t h = SR ? sr_combine(colw2, sr_plane(bz * 8 + z, key2)) : 0u;
        float r[S];
        plane(z, u, h2, h, r);
        // whole sectors only (an inactive slot of an active sector stores its 0 again)
        if (lane_bit(sector_lanes<T>(Wo[z]))) {
#pragma unroll
            for (int s = 0; s < S; ++s) {
                T *o = at_byte(out[s], (uint32_t)(z * 64 + lane) * (uint32_t)sizeof(T));
                if constexpr (SR) rd_st_sr(o, 0, r[s], sr_species(h, s));
                else rd_st(o, 0, r[s]);
            }
        }
    }
}

template <typename T, bool SR, bool MID>
__global__ __launch_bounds__(256) void k_pair8z(StepArgs a)
{
    pair8z<T, 1, SR, MID, false>(a, nullptr);
}
// two species: 32 KB of LDS per workgroup, five waves per SIMD
template <typename T, bool SR>
__global__ __launch_bounds__(256, 5) void k_pair8z2(StepArgs a)
{
    pair8z<T, 2, SR, false, false>(a, nullptr);
}
// One species with the factor: 32 KB of LDS per workgroup.  us per step, k_step8e without and
// with the x-face exchange / a pair: FP32 packing 64^3 5.1, 6.2 / 4.1, 160^3 14.8, 16.2 / 12.3,
// soil 256^3 25.1, 28.1 / 21.9; BF16 with stochastic rounding 160^3 14.4, 14.8 / 13.3.  Lists
// of 216, 1000, 2744 and 7996 blocks, without the exchange / a pair: FP32 5.1 / 4.0, 5.2 / 4.1, 7.2 /
// 5.4, 15.5 / 11.9; BF16 5.3 / 4.0, 5.3 / 4.1, 7.2 / 5.4, 13.1 / 11.1, with stochastic rounding
// 5.6 / 4.5, 5.6 / 4.6, 7.6 / 6.3, 14.2 / 12.7; FP16 as BF16, with it 6.0 / 5.1, 5.9 / 5.1, 8.1 /
// 7.0, 15.1 / 14.2.
template <typename T, bool SR, bool MID>
__global__ __launch_bounds__(256, 5) void k_pair8e(StepArgs a, const float *e)
{
    pair8z<T, 1, SR, MID, true>(a, e);
}

template <typename T>
void launch_pair_t(const StepArgs &a, int groups, hipStream_t st)
{
    if (a.cmid) hipLaunchKernelGGL((k_pair8z<T, false, true>), dim3(groups), dim3(256), 0, st, a);
    else if (a.S == 1 && a.sround) hipLaunchKernelGGL((k_pair8z<T, true, false>), dim3(groups), dim3(256), 0, st, a);
    else if (a.S == 1) hipLaunchKernelGGL((k_pair8z<T, false, false>), dim3(groups), dim3(256), 0, st, a);
    else if (a.sround) hipLaunchKernelGGL((k_pair8z2<T, true>), dim3(groups), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((k_pair8z2<T, false>), dim3(groups), dim3(256), 0, st, a);
}
template <typename T>
void launch_pair_e(const StepArgs &a, const float *e, int groups, hipStream_t st)
{
    // FP32 rounds to nearest with the factor
    const bool sr = a.sround && !std::is_same<T, float>::value;
    if (a.cmid) hipLaunchKernelGGL((k_pair8e<T, false, true>), dim3(groups), dim3(256), 0, st, a, e);
    else if (sr)
        hipLaunchKernelGGL((k_pair8e<T, !std::is_same<T, float>::value, false>), dim3(groups), dim3(256), 0, st, a, e);
    else hipLaunchKernelGGL((k_pair8e<T, false, false>), dim3(groups), dim3(256), 0, st, a, e);
}
}  // namespace

int rd_launch_step_pair_diff(int storage, const DiffArgs &d, void *stream)
{
    const StepArgs &a = d.s;
    if (a.nb <= 0) return 0;
    if (a.S != 1 || a.cbase || (a.cmid && a.sround)) return (int)hipErrorInvalidValue;
    const int groups = rd_xcd_grid((a.nb + 3) / 4, a.xcd_chunk);
    if (storage == 0) launch_pair_e<float>(a, d.e, groups, (hipStream_t)stream);
    else if (storage == 1) launch_pair_e<bf16_t>(a, d.e, groups, (hipStream_t)stream);
    else launch_pair_e<_Float16>(a, d.e, groups, (hipStream_t)stream);
    return (int)hipGetLastError();
}

int rd_launch_step_pair(int storage, const StepArgs &a, void *stream)
{
    if (a.nb <= 0) return 0;
    if (a.S < 1 || a.S > 2 || a.cbase || (a.cmid && (a.S != 1 || a.sround))) return (int)hipErrorInvalidValue;
    const int groups = rd_xcd_grid((a.nb + 3) / 4, a.xcd_chunk);
    if (storage == 0) launch_pair_t<float>(a, groups, (hipStream_t)stream);
    else if (storage == 1) launch_pair_t<bf16_t>(a, groups, (hipStream_t)stream);
    else launch_pair_t<_Float16>(a, groups, (hipStream_t)stream);
    return (int)hipGetLastError();
}
