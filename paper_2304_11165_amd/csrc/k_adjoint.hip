// k_adjoint.hip -- discrete adjoint of the FTCS step for one species.
//
// The forward step on free voxels is c^{n+1} = J c^n + g with
//   J = I + alpha * L_f - (beta + gamma * n_wall) I,
// L_f the graph Laplacian among active voxels (the mirror rule makes it symmetric)
// and g the Dirichlet contribution.  J is symmetric, so the adjoint recursion
// lambda^n = J^T lambda^{n+1} is the forward step applied to lambda with every
// Dirichlet value set to 0 (lambda is 0 on Dirichlet and inactive voxels).  The
// same per-voxel update (rd_update) is used, so the adjoint step rounds like the
// forward one.  Fused with it are the FP64 gradient partials
//   dL/dD += <lambda^{n+1}, dt/dx^2 * sum_q (c^n_q - c^n_p)>
//   dL/dk += <lambda^{n+1}, -dt * c^n>           (k: first-order decay rate).
#include "rd_device.h"
#include "rd_adjoint.h"

namespace {

template <typename T, int B>
__global__ __launch_bounds__(256) void k_adjoint(AdjArgs a)
{
    using K = Blk<B>;
    using C = Cfg<B>;
    __shared__ float tl[C::BPW][1][K::TL];
    __shared__ float tc[C::BPW][1][K::TL];
    __shared__ uint64_t srec[C::BPW][K::MW];
    __shared__ double wsum[4][2];
    const int sub = threadIdx.x / C::TPB, lt = threadIdx.x % C::TPB;
    const int b = blockIdx.x * C::BPW + sub;
    const bool valid = b < a.nb;
    BlockInfo bi = {};
    if (valid) {
        bi = a.info[b];
        if (lt < K::MW) srec[sub][lt] = a.mask[(int64_t)b * K::MW + lt];
    }
    stage_tile<float, B>(tl[sub], a.lam_in, 0, 1, b, bi, lt, valid);
    stage_tile<T, B>(tc[sub], (const T *)a.c, 0, 1, b, bi, lt, valid);
    __syncthreads();
    double gD = 0.0, gk = 0.0;
    if (valid) {
        int bx, by, bz, gid;
        block_pos(bi, &bx, &by, &bz, &gid);
        const GeomInfo g = a.geom[gid];
        const uint64_t *rec = srec[sub];
        for (int k = 0; k < C::VPT; ++k) {
            const int slot = lt + k * C::TPB;
            const int lx = slot % B, ly = (slot / B) % B, lz = slot / (B * B);
            const int gx = bx * B + lx, gy = by * B + ly, gz = bz * B + lz;
            const int64_t i = (int64_t)b * K::NS + slot;
            const int t = K::tidx(lx, ly, lz);
            const bool act = own_bit<B>(rec, slot);
            float out = 0.0f;
            if (act) {
                int nwall = 0;
                const unsigned nbm = nb_bits<B>(rec, lx, ly, lz, gx, gy, gz, g.nx, g.ny, g.nz, &nwall);
                const float lp = tl[sub][0][t];
                if (on_dirichlet(a.coef.dir, gx, gy, gz, g.nx, g.ny, g.nz)) {
                    out = lp;  // stays 0
                } else {
                    const float *ts = tl[sub][0];
                    const float nbv[6] = {ts[t - 1], ts[t + 1], ts[t - K::E], ts[t + K::E],
                                          ts[t - K::E * K::E], ts[t + K::E * K::E]};
                    const float cen[1] = {lp};
                    out = rd_update<1>(lp, nbv, nbm, nwall, a.coef, cen, 0);
                    // gradient partials with the forward state c^n
                    const float *tcs = tc[sub][0];
                    const float cc = tcs[t];
                    const float cnb[6] = {tcs[t - 1], tcs[t + 1], tcs[t - K::E], tcs[t + K::E],
                                          tcs[t - K::E * K::E], tcs[t + K::E * K::E]};
                    double lap = 0.0;
#pragma unroll
                    for (int d = 0; d < 6; ++d)
                        if ((nbm >> d) & 1u) lap += (double)cnb[d] - (double)cc;
                    gD += (double)lp * lap;
                    gk -= (double)lp * (double)cc;
                }
            }
            a.lam_out[i] = out;
        }
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const double s0 = wave_sum(gD), s1 = wave_sum(gk);
    if (lane == 0) {
        wsum[wave][0] = s0;
        wsum[wave][1] = s1;
    }
    __syncthreads();
    if (threadIdx.x < 2) {  // this workgroup's accumulator, in step order
        const int l = threadIdx.x;
        a.partial[(int64_t)blockIdx.x * 2 + l] += ((wsum[0][l] + wsum[1][l]) + wsum[2][l]) + wsum[3][l];
    }
}

// Slot, in the neighbour's block across face f, of lane (u, v)'s face voxel (8^3 blocks).
__device__ __forceinline__ uint32_t face_slot8(int f, int u, int v)
{
    switch (f) {
    case 0: return (uint32_t)((v * 8 + u) * 8 + 7);
    case 1: return (uint32_t)((v * 8 + u) * 8 + 0);
    case 2: return (uint32_t)((v * 8 + 7) * 8 + u);
    case 3: return (uint32_t)((v * 8 + 0) * 8 + u);
    case 4: return (uint32_t)((7 * 8 + v) * 8 + u);
    default: return (uint32_t)((0 * 8 + v) * 8 + u);
    }
}
// Plane z of one field and its four side halos (held by the lanes with ly == z) into a
// wave's 10 x 10 LDS tile.
__device__ __forceinline__ void tile_plane(float *t, int lx, int ly, int z, float c, const float side[6])
{
    t[(ly + 1) * 10 + (lx + 1)] = c;
    if (ly == z) {
        t[(lx + 1) * 10 + 0] = side[0];
        t[(lx + 1) * 10 + 9] = side[1];
        t[0 * 10 + (lx + 1)] = side[2];
        t[9 * 10 + (lx + 1)] = side[3];
    }
}
__device__ __forceinline__ void tile_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// Keeps a plane's FP64 sums in that plane: the compiler would otherwise form the terms of all
// eight planes after the last one and hold their inputs in registers until then (200 of them).
__device__ __forceinline__ void settle(double &x, double &y) { asm volatile("" : "+v"(x), "+v"(y)); }

// The adjoint step for 8^3 blocks in the column form of the forward step: one wave per
// block (four per workgroup), lane (lx, ly) walking its z-column; lambda^{n+1} and c^n
// of the block and of its face halos are loaded under the activity predicates, the
// +-x / +-y neighbours of both go through one-plane LDS tiles.  lambda^n on free
// voxels is rd_update on lambda (the forward step with zero Dirichlet data), 0
// elsewhere; the gradient terms of the block are added, in step order, to its own
// FP64 accumulators partial[b][0..1] (one wave owns a block, so there is no race):
//   dL/dD: lambda^{n+1}_p * (sum of the six c^n neighbours - n_active * c^n_p)
//   dL/dk: -lambda^{n+1}_p * c^n_p                      (scaled on the host)
// lambda is 0 off the free voxels, so every lane adds its terms; products of two FP32
// values are exact in FP64, so fused multiply-adds round like a product and a sum.
// On a 128^3 packing (4096 blocks, one round of waves: bound by one wave's chain of loads,
// planes and sums) 8.9 us, against 12.5 with code bits tested per neighbour, the
// accumulators read at the end and the wave sums through LDS permutes.
template <typename T>
__global__ __launch_bounds__(256) void k_adjoint8(AdjArgs a)
{
    __shared__ float tl[4][100], tc[4][100];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int b = __builtin_amdgcn_readfirstlane(map_group(blockIdx.x, a.order) * 4 + wv);
    if (b >= a.nb) return;
    const BlockInfo bi = a.info[b];
    const T *call = (const T *)a.c;
    const int64_t base = (int64_t)b * 512;
    const float *lin = uniform_ptr(a.lam_in + base);
    float *lout = uniform_ptr(a.lam_out + base);
    const T *cin = uniform_ptr(call + base);
    const int lx = lane & 7, ly = lane >> 3;
    const uint64_t *rec = a.mask + (int64_t)b * 16;
    uint64_t Wo[8], Wf[6];
#pragma unroll
    for (int z = 0; z < 8; ++z) Wo[z] = rec[z];
#pragma unroll
    for (int f = 0; f < 6; ++f) Wf[f] = rec[8 + f];
    typedef typename RawOf<T>::type R;
    float lc[8], lh[6];
    R cc[8], ch[6];
    const uint32_t ncw = a.ncnt[(int64_t)b * 64 + lane];
    const double p0 = a.partial[(int64_t)b * 2 + 0], p1 = a.partial[(int64_t)b * 2 + 1];
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        lc[z] = 0.0f;
        cc[z] = (R)0;
        if (lane_bit(Wo[z])) {
            const uint32_t o = (uint32_t)(z * 64 + lane);
            lc[z] = *at_byte(lin, o * 4u);
            cc[z] = ld_raw(at_byte(cin, o * (uint32_t)sizeof(T)), 0);
        }
    }
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const int n = bi.nbr[f];
        const int64_t nb0 = (int64_t)(n >= 0 ? n : b) * 512;
        const uint32_t o = face_slot8(f, lx, ly);
        lh[f] = 0.0f;
        ch[f] = (R)0;
        if (lane_bit(Wf[f])) {
            lh[f] = *at_byte(uniform_ptr(a.lam_in + nb0), o * 4u);
            ch[f] = ld_raw(at_byte(uniform_ptr(call + nb0), o * (uint32_t)sizeof(T)), 0);
        }
    }
    float c[8], cs[6];
#pragma unroll
    for (int z = 0; z < 8; ++z) c[z] = from_raw<T>(cc[z]);
#pragma unroll
    for (int f = 0; f < 6; ++f) cs[f] = from_raw<T>(ch[f]);

    int bx, by, bz, gid;
    block_pos(bi, &bx, &by, &bz, &gid);
    const GeomInfo g = a.geom[gid];
    const int gx = bx * 8 + lx, gy = by * 8 + ly;
    const bool bnd = bx == 0 || by == 0 || bz == 0 || bx * 8 + 8 >= g.nx || by * 8 + 8 >= g.ny ||
                     bz * 8 + 8 >= g.nz;
    float *TL = tl[wv], *TC = tc[wv];
    double gD = 0.0, gk = 0.0;
    double below = (double)cs[4], here = (double)c[0];  // the column in FP64
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        tile_plane(TL, lx, ly, z, lc[z], lh);
        tile_plane(TC, lx, ly, z, c[z], cs);
        tile_order();
        const float nact = (float)((ncw >> (3 * z)) & 7u);
        unsigned onf = 0u;
        if (bnd) onf = box_faces(g, gx, gy, bz * 8 + z);
        const float nwall = (6.0f - nact) - (float)__popc(onf);
        const int o = (ly + 1) * 10 + (lx + 1);
        const float lp = lc[z];
        const float nbl[6] = {TL[o - 1], TL[o + 1], TL[o - 10], TL[o + 10], z == 0 ? lh[4] : lc[z > 0 ? z - 1 : 0],
                              z == 7 ? lh[5] : lc[z < 7 ? z + 1 : 7]};
        const float cen[1] = {lp};
        float r = rd_update_n<1>(lp, nbl, nact, nwall, a.coef, cen, 0);
        if (bnd) {  // Dirichlet voxels lie on the box faces: boundary blocks only (uniform)
            if ((onf & a.coef.dir) != 0u) r = 0.0f;
        }
        const double above = (double)(z == 7 ? cs[5] : c[z < 7 ? z + 1 : 7]);
        const double sc = (((((double)TC[o - 1] + (double)TC[o + 1]) + (double)TC[o - 10]) + (double)TC[o + 10]) + below) +
                          above;
        const double lapc = fma(-(double)nact, here, sc);
        gD += (double)lp * lapc;
        gk = fma(-(double)lp, here, gk);
        settle(gD, gk);
        below = here;
        here = above;
        tile_order();
        // lambda is FP32 and read under activity predicates: whole 128-byte sectors
        if (lane_bit(sector_lanes<float>(Wo[z]))) *at_byte(lout, (uint32_t)(z * 64 + lane) * 4u) = lane_bit(Wo[z]) ? r : 0.0f;
    }
    gD = wave_sum(gD);
    gk = wave_sum(gk);
    if (lane == 0) {
        a.partial[(int64_t)b * 2 + 0] = p0 + gD;
        a.partial[(int64_t)b * 2 + 1] = p1 + gk;
    }
}

// lambda^N on free voxels: c^N - c* (mode 0, loss partial 1/2 (c^N - c*)^2) or the
// given dL/dc^N (mode 1); 0 on Dirichlet and inactive slots.
template <typename T, int B>
__global__ __launch_bounds__(256) void k_adj_seed(AdjArgs a, int mode)
{
    using K = Blk<B>;
    __shared__ double wsum[4];
    const int b = blockIdx.x;
    double loss = 0.0;
    if (b < a.nb) {
        const BlockInfo bi = a.info[b];
        int bx, by, bz, gid;
        block_pos(bi, &bx, &by, &bz, &gid);
        const GeomInfo g = a.geom[gid];
        const uint64_t *rec = a.mask + (int64_t)b * K::MW;
        for (int slot = threadIdx.x; slot < K::NS; slot += 256) {
            const int gx = bx * B + slot % B, gy = by * B + (slot / B) % B, gz = bz * B + slot / (B * B);
            const int64_t i = (int64_t)b * K::NS + slot;
            float l = 0.0f;
            if (own_bit<B>(rec, slot) && !on_dirichlet(a.coef.dir, gx, gy, gz, g.nx, g.ny, g.nz)) {
                if (mode == 0) {
                    const float d = rd_ld((const T *)a.c, i) - a.seed[i];
                    l = d;
                    loss += 0.5 * (double)d * (double)d;
                } else {
                    l = a.seed[i];
                }
            }
            a.lam_out[i] = l;
        }
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const double s = wave_sum(loss);
    if (lane == 0) wsum[wave] = s;
    __syncthreads();
    if (threadIdx.x == 0) a.partial[b] = ((wsum[0] + wsum[1]) + wsum[2]) + wsum[3];
}


// Adjoint step with a diffusivity factor, one thread per slot (see AdjEArgs).  The
// lambda update mirrors the inhomogeneous forward step in FP32; the gradient terms are
// FP64.  Rows as in k_adjoint: one per workgroup (B = 8: one block, B = 4: four).
template <typename T, int B>
__global__ __launch_bounds__(256) void k_adjoint_e(AdjEArgs x)
{
    using C = Cfg<B>;
    constexpr int NS = B * B * B;
    const AdjArgs &a = x.a;
    __shared__ double wsum[4][2];
    const int sub = threadIdx.x / C::TPB, lt = threadIdx.x % C::TPB;
    const int b = blockIdx.x * C::BPW + sub;
    double gD = 0.0, gk = 0.0;
    if (b < a.nb) {
        const BlockInfo bi = a.info[b];
        int bx, by, bz, gid;
        block_pos(bi, &bx, &by, &bz, &gid);
        const GeomInfo g = a.geom[gid];
        const T *c = (const T *)a.c;
        for (int k = 0; k < C::VPT; ++k) {
            const int slot = lt + k * C::TPB;
            const int64_t i = (int64_t)b * NS + slot;
            const unsigned code = a.code[i];
            float out = 0.0f;
            if (code & 64u) {
                const int lx = slot % B, ly = (slot / B) % B, lz = slot / (B * B);
                const int gx = bx * B + lx, gy = by * B + ly, gz = bz * B + lz;
                const unsigned onf = (gx == 0 ? 1u : 0u) | (gx == g.nx - 1 ? 2u : 0u) | (gy == 0 ? 4u : 0u) |
                                     (gy == g.ny - 1 ? 8u : 0u) | (gz == 0 ? 16u : 0u) |
                                     (gz == g.nz - 1 ? 32u : 0u);
                const unsigned m = code & 63u;
                const int nwall = __popc(~onf & ~m & 0x3fu);
                const float lp = a.lam_in[i], ep = x.e[i];
                const double cp = (double)rd_ld(c, i);
                float laml = 0.0f;
                double lapc = 0.0, gsum = 0.0;
                const int stride[3] = {1, B, B * B};
                for (int d = 0; d < 6; ++d) {
                    if (!((m >> d) & 1u)) continue;
                    const int ax = d >> 1, l = ax == 0 ? lx : ax == 1 ? ly : lz;
                    const bool up = d & 1;
                    int64_t q;
                    if (up ? l < B - 1 : l > 0) q = i + (up ? stride[ax] : -stride[ax]);
                    else q = (int64_t)bi.nbr[d] * NS + slot + (up ? -(B - 1) : (B - 1)) * stride[ax];
                    const float lq = a.lam_in[q], eq = x.e[q];
                    const double cq = (double)rd_ld(c, q);
                    laml = fmaf(0.5f * (ep + eq), lq - lp, laml);
                    lapc += 0.5 * ((double)ep + (double)eq) * (cq - cp);
                    gsum += (cq - cp) * ((double)lp - (double)lq);
                }
                x.ge[i] += 0.5 * x.alpha * gsum;  // lambda is 0 on Dirichlet voxels
                if (!(onf & a.coef.dir)) {
                    gD += (double)lp * lapc;
                    gk -= (double)lp * cp;
                    const float r = fmaf(a.coef.alpha, laml, lp);
                    out = fmaf(-fmaf(a.coef.gamma, (float)nwall, a.coef.beta), lp, r);
                }
            }
            a.lam_out[i] = out;
        }
    }
    const int wave = threadIdx.x >> 6;
    const double s0 = wave_sum(gD), s1 = wave_sum(gk);
    if ((threadIdx.x & 63) == 0) {
        wsum[wave][0] = s0;
        wsum[wave][1] = s1;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        a.partial[(int64_t)blockIdx.x * 2 + 0] += ((wsum[0][0] + wsum[1][0]) + wsum[2][0]) + wsum[3][0];
        a.partial[(int64_t)blockIdx.x * 2 + 1] += ((wsum[0][1] + wsum[1][1]) + wsum[2][1]) + wsum[3][1];
    }
}

// Column form of k_adjoint_e for 8^3 blocks: one wave per block, lane (lx, ly) walking
// z, lambda / c / e planes staged in LDS with their side halos, the z neighbours in
// registers.  Per voxel the same operations in the same order as k_adjoint_e (dL/de and
// lambda are bitwise equal; the dL/dD and dL/dk rows are summed in another order): a face
// toward an inactive neighbour adds 0 (weight 0 and no difference of c) instead of being
// branched over, and a z face's terms are formed once for the two voxels it joins (equal, or
// of opposite sign).  dL/de is read with the other inputs: read where it was added to, it
// made each of the eight planes wait for memory.  One row per block.
// On a 160^3 packing (8000 blocks, 32 bytes per voxel) 27.5 us, against 38.3.
template <typename T>
__global__ __launch_bounds__(256) void k_adjoint8e(AdjEArgs x)
{
    __shared__ float tl[4][100], tc[4][100], te[4][100];
    const AdjArgs &a = x.a;
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int b = __builtin_amdgcn_readfirstlane(map_group(blockIdx.x, a.order) * 4 + wv);
    if (b >= a.nb) return;
    const BlockInfo bi = a.info[b];
    const T *call = (const T *)a.c;
    const int64_t base = (int64_t)b * 512;
    const float *lin = uniform_ptr(a.lam_in + base), *ein = uniform_ptr(x.e + base);
    float *lout = uniform_ptr(a.lam_out + base);
    double *gep = uniform_ptr(x.ge + base);
    const T *cin = uniform_ptr(call + base);
    const int lx = lane & 7, ly = lane >> 3;
    BlockMasks M;
    M.load(a.mask + (int64_t)b * 16);
    typedef typename RawOf<T>::type R;
    float lc[8], lh[6], ec[8], eh[6];
    R cr[8], cg[6];
    double ge[8];
    const uint32_t ncw = a.ncnt[(int64_t)b * 64 + lane];
    const double p0 = a.partial[(int64_t)b * 2 + 0], p1 = a.partial[(int64_t)b * 2 + 1];
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        lc[z] = ec[z] = 0.0f;
        cr[z] = (R)0;
        if (lane_bit(M.Wo[z])) {
            const uint32_t o = (uint32_t)(z * 64 + lane);
            lc[z] = *at_byte(lin, o * 4u);
            cr[z] = ld_raw(at_byte(cin, o * (uint32_t)sizeof(T)), 0);
            ec[z] = *at_byte(ein, o * 4u);
        }
    }
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const int n = bi.nbr[f];
        const int64_t nb0 = (int64_t)(n >= 0 ? n : b) * 512;
        const uint32_t o = face_slot8(f, lx, ly);
        lh[f] = eh[f] = 0.0f;
        cg[f] = (R)0;
        if (lane_bit(M.Wf[f])) {
            lh[f] = *at_byte(uniform_ptr(a.lam_in + nb0), o * 4u);
            cg[f] = ld_raw(at_byte(uniform_ptr(call + nb0), o * (uint32_t)sizeof(T)), 0);
            eh[f] = *at_byte(uniform_ptr(x.e + nb0), o * 4u);
        }
    }
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        ge[z] = 0.0;
        if (lane_bit(M.Wo[z])) ge[z] = *at_byte(gep, (uint32_t)(z * 64 + lane) * 8u);
    }
    float cc[8], ch[6];
#pragma unroll
    for (int z = 0; z < 8; ++z) cc[z] = from_raw<T>(cr[z]);
#pragma unroll
    for (int f = 0; f < 6; ++f) ch[f] = from_raw<T>(cg[f]);
    int bx, by, bz, gid;
    block_pos(bi, &bx, &by, &bz, &gid);
    const GeomInfo g = a.geom[gid];
    const int gx = bx * 8 + lx, gy = by * 8 + ly;
    const bool bnd = bx == 0 || by == 0 || bz == 0 || bx * 8 + 8 >= g.nx || by * 8 + 8 >= g.ny ||
                     bz * 8 + 8 >= g.nz;
    // what a face adds to voxel p, whose neighbour across it is q
    struct Face {
        float w, dl;   // weight and lambda_q - lambda_p
        double lap, g; // (e_p + e_q) / 2 (c_q - c_p) and (c_q - c_p)(lambda_p - lambda_q)
    };
    auto face = [](float lp, float cp, float ep, float lq, float cq, float eq, uint64_t both) {
        Face t;
        t.w = lane_bit(both) ? 0.5f * (ep + eq) : 0.0f;
        t.dl = lq - lp;
        const double dc = (double)(lane_bit(both) ? cq : cp) - (double)cp;
        t.lap = 0.5 * ((double)ep + (double)eq) * dc;
        t.g = dc * ((double)lp - (double)lq);
        return t;
    };
    const int t = (ly + 1) * 10 + (lx + 1);
    const double half_alpha = 0.5 * x.alpha;
    double gD = 0.0, gk = 0.0;
    // the z face below plane 0, as seen from the voxel under it
    Face zf = face(lh[4], ch[4], eh[4], lc[0], cc[0], ec[0], M.pair(0, 4));
#pragma unroll
    for (int z = 0; z < 8; ++z) {
        tile_plane(tl[wv], lx, ly, z, lc[z], lh);
        tile_plane(tc[wv], lx, ly, z, cc[z], ch);
        tile_plane(te[wv], lx, ly, z, ec[z], eh);
        tile_order();
        const float lp = lc[z], cp = cc[z], ep = ec[z];
        float laml = 0.0f;
        double lapc = 0.0, gsum = 0.0;
        const int off[4] = {-1, 1, -10, 10};
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const Face f = face(lp, cp, ep, tl[wv][t + off[d]], tc[wv][t + off[d]], te[wv][t + off[d]], M.pair(z, d));
            laml = fmaf(f.w, f.dl, laml);
            lapc += f.lap;
            gsum += f.g;
        }
        laml = fmaf(zf.w, -zf.dl, laml);
        lapc -= zf.lap;
        gsum += zf.g;
        zf = face(lp, cp, ep, z == 7 ? lh[5] : lc[z < 7 ? z + 1 : 7], z == 7 ? ch[5] : cc[z < 7 ? z + 1 : 7],
                  z == 7 ? eh[5] : ec[z < 7 ? z + 1 : 7], M.pair(z, 5));
        laml = fmaf(zf.w, zf.dl, laml);
        lapc += zf.lap;
        gsum += zf.g;
        // lambda is 0 on Dirichlet and inactive voxels
        gD += (double)lp * lapc;
        gk = fma(-(double)lp, (double)cp, gk);
        settle(gD, gk);
        const float nact = (float)((ncw >> (3 * z)) & 7u);
        unsigned onf = 0u;
        if (bnd) onf = box_faces(g, gx, gy, bz * 8 + z);
        const float nwall = (6.0f - nact) - (float)__popc(onf);
        float out = fmaf(-fmaf(a.coef.gamma, nwall, a.coef.beta), lp, fmaf(a.coef.alpha, laml, lp));
        if (bnd) {
            if ((onf & a.coef.dir) != 0u) out = 0.0f;
        }
        tile_order();
        if (lane_bit(M.Wo[z])) *at_byte(gep, (uint32_t)(z * 64 + lane) * 8u) = ge[z] + half_alpha * gsum;
        if (lane_bit(sector_lanes<float>(M.Wo[z])))
            *at_byte(lout, (uint32_t)(z * 64 + lane) * 4u) = lane_bit(M.Wo[z]) ? out : 0.0f;
    }
    gD = wave_sum(gD);
    gk = wave_sum(gk);
    if (lane == 0) {
        a.partial[(int64_t)b * 2 + 0] = p0 + gD;
        a.partial[(int64_t)b * 2 + 1] = p1 + gk;
    }
}

template <int B>
__global__ __launch_bounds__(256) void k_dense_f64(const BlockInfo *info, const uint8_t *code, const GeomInfo *geom,
                                                   int nb, const double *v, double *dense)
{
    constexpr int NS = B * B * B;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)nb * NS || !(code[i] & 64u)) return;
    const int b = (int)(i / NS), slot = (int)(i % NS);
    int bx, by, bz, gid;
    block_pos(info[b], &bx, &by, &bz, &gid);
    const GeomInfo g = geom[gid];
    dense[voxel_id(g, bx * B + slot % B, by * B + (slot / B) % B, bz * B + slot / (B * B))] = v[i];
}

}  // namespace

#define ADJ_DISPATCH(storage, B, KERNEL, grid, stream, ...)                                        \
    do {                                                                                           \
        hipStream_t st_ = (hipStream_t)(stream);                                                   \
        if ((B) == 8) {                                                                            \
            if ((storage) == 0) hipLaunchKernelGGL((KERNEL<float, 8>), grid, dim3(256), 0, st_, __VA_ARGS__);      \
            else if ((storage) == 1) hipLaunchKernelGGL((KERNEL<bf16_t, 8>), grid, dim3(256), 0, st_, __VA_ARGS__); \
            else hipLaunchKernelGGL((KERNEL<_Float16, 8>), grid, dim3(256), 0, st_, __VA_ARGS__);                  \
        } else {                                                                                   \
            if ((storage) == 0) hipLaunchKernelGGL((KERNEL<float, 4>), grid, dim3(256), 0, st_, __VA_ARGS__);      \
            else if ((storage) == 1) hipLaunchKernelGGL((KERNEL<bf16_t, 4>), grid, dim3(256), 0, st_, __VA_ARGS__); \
            else hipLaunchKernelGGL((KERNEL<_Float16, 4>), grid, dim3(256), 0, st_, __VA_ARGS__);                  \
        }                                                                                          \
        return (int)hipGetLastError();                                                             \
    } while (0)

int adj_groups(int B, int nb) { return B == 8 ? nb : (nb + 3) / 4; }

int adj_launch_step(int storage, int B, const AdjArgs &a, void *stream)
{
    if (B == 8) {  // column form, four blocks per workgroup, per-block accumulators
        const dim3 grid((unsigned)rd_xcd_grid((a.nb + 3) / 4, a.order));
        hipStream_t st = (hipStream_t)stream;
        if (storage == 0) hipLaunchKernelGGL((k_adjoint8<float>), grid, dim3(256), 0, st, a);
        else if (storage == 1) hipLaunchKernelGGL((k_adjoint8<bf16_t>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((k_adjoint8<_Float16>), grid, dim3(256), 0, st, a);
        return (int)hipGetLastError();
    }
    ADJ_DISPATCH(storage, B, k_adjoint, dim3((unsigned)adj_groups(B, a.nb)), stream, a);
}

int adj_launch_seed(int storage, int B, const AdjArgs &a, int mode, void *stream)
{
    ADJ_DISPATCH(storage, B, k_adj_seed, dim3((unsigned)a.nb), stream, a, mode);
}

int adj_launch_step_e(int storage, int B, const AdjEArgs &x, int column, void *stream)
{
    if (x.a.nb <= 0) return 0;
    hipStream_t st = (hipStream_t)stream;
    const dim3 grid((unsigned)adj_groups(B, x.a.nb));
    if (B == 8 && column) {  // four blocks per workgroup, one row per block
        const dim3 g8((unsigned)rd_xcd_grid((x.a.nb + 3) / 4, x.a.order));
        if (storage == 0) hipLaunchKernelGGL((k_adjoint8e<float>), g8, dim3(256), 0, st, x);
        else if (storage == 1) hipLaunchKernelGGL((k_adjoint8e<bf16_t>), g8, dim3(256), 0, st, x);
        else hipLaunchKernelGGL((k_adjoint8e<_Float16>), g8, dim3(256), 0, st, x);
    } else if (B == 8) {
        if (storage == 0) hipLaunchKernelGGL((k_adjoint_e<float, 8>), grid, dim3(256), 0, st, x);
        else if (storage == 1) hipLaunchKernelGGL((k_adjoint_e<bf16_t, 8>), grid, dim3(256), 0, st, x);
        else hipLaunchKernelGGL((k_adjoint_e<_Float16, 8>), grid, dim3(256), 0, st, x);
    } else {
        if (storage == 0) hipLaunchKernelGGL((k_adjoint_e<float, 4>), grid, dim3(256), 0, st, x);
        else if (storage == 1) hipLaunchKernelGGL((k_adjoint_e<bf16_t, 4>), grid, dim3(256), 0, st, x);
        else hipLaunchKernelGGL((k_adjoint_e<_Float16, 4>), grid, dim3(256), 0, st, x);
    }
    return (int)hipGetLastError();
}

int adj_launch_dense_f64(int B, const BlockInfo *info, const uint8_t *code, const GeomInfo *geom, int nb,
                         const double *v, double *dense, int64_t ndense, void *stream)
{
    int rc = rd_launch_fill_u32(dense, 0u, 2 * ndense, stream);
    if (rc != 0 || nb <= 0) return rc;
    hipStream_t st = (hipStream_t)stream;
    const int64_t n = (int64_t)nb * B * B * B;
    const dim3 grid((unsigned)((n + 255) / 256));
    if (B == 8) hipLaunchKernelGGL((k_dense_f64<8>), grid, dim3(256), 0, st, info, code, geom, nb, v, dense);
    else hipLaunchKernelGGL((k_dense_f64<4>), grid, dim3(256), 0, st, info, code, geom, nb, v, dense);
    return (int)hipGetLastError();
}
