// Apply: v = FFM(w u), one descent over the plan's levels, then the leaf near field.
//
// Paper: Sec. 2.2.2 (v ~ L_X^T (T (L_Y u)), Lagrange levels), Sec. 2.2.3 (v ~ F_{s->X} (T_L (F_{Y->s} u)),
// Gegenbauer levels, eqs. gegenbauerQuadrature and the three products that follow it), Sec. 2.2.4 (dense
// remainder), remark closing Sec. 2.2.3 (transforms evaluated on the fly at every level, no upward pass).
//
// Every kernel reads its parameters from the level descriptor named by its work item (int4, .x =
// descriptor), so one launch serves one level of one plan or the same step of many plans (a batch).
// Every output element is owned by exactly one thread of each kernel and accumulated in a fixed order,
// so results are bitwise reproducible and independent of how work items are grouped into launches.
#include "common.h"

#include <algorithm>
#include <cmath>
#include <map>
#include <mutex>
#include <tuple>

namespace ffm {

namespace {

constexpr int kThreads = 256;

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
using gch4 = const __attribute__((address_space(1))) half4_t *;
using gch8 = const __attribute__((address_space(1))) half8_t *;

// sin(2 pi x), cos(2 pi x) for x in revolutions.  The hardware reduces its argument itself over
// |x| <= 256 revolutions; against an exact reduction to [0, 1) first it differs by at most 2.4e-7
// (measured over 1.6e7 arguments), below the FP32 rounding of a phase of even one revolution.  FP32
// phases are passed unreduced where the planner bounds them by 128 revolutions (FP64 phases are
// reduced exactly in FP64 before rounding to FP32).
__device__ __forceinline__ void sincos_rev(float x, float &s, float &c) {
    s = __builtin_amdgcn_sinf(x);
    c = __builtin_amdgcn_cosf(x);
}

// ------------------------------------------------------------------ permutations and scaling
// item (desc, first index): u[i] = wu[perm_y[i]] for i < ny, v[i] = 0 for i < nx (256 per block)
__global__ void __launch_bounds__(kThreads)
k_perm_in(const LDesc *__restrict__ descs, const IoEntry *__restrict__ io, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const IoEntry e = io[d.inst];
    const int64_t i = (int64_t)wk.y + threadIdx.x;
    if (i < d.ny) {
        const int64_t j = d.perm_y[i];
        float2 r;
        switch (e.dtype) {
            case FFM_C64: r = static_cast<const float2 *>(e.wu)[j]; break;
            case FFM_F32: r = make_float2(static_cast<const float *>(e.wu)[j], 0.f); break;
            case FFM_F64: r = make_float2((float)static_cast<const double *>(e.wu)[j], 0.f); break;
            default: {
                const double2 w = static_cast<const double2 *>(e.wu)[j];
                r = make_float2((float)w.x, (float)w.y);
            }
        }
        d.u[i] = r;
        if (d.ucomp) {
            // split double layer: the densities u n_c
            const float4 n = d.sn[i];
            d.ucomp[i] = make_float2(r.x * n.x, r.y * n.x);
            d.ucomp[d.ny + i] = make_float2(r.x * n.y, r.y * n.y);
            d.ucomp[2 * d.ny + i] = make_float2(r.x * n.z, r.y * n.z);
        }
    }
    if (i < d.nx) {
        for (int c = 0; c < d.ncomp; ++c) d.v[(int64_t)c * d.nx + i] = make_float2(0.f, 0.f);
        if (d.vtmp)
            for (int c = 0; c < 3; ++c) d.vtmp[(int64_t)c * d.nx + i] = make_float2(0.f, 0.f);
    }
}

// max over |Re u|, |Im u| (non-negative floats compare as their bit patterns); item (desc, first index),
// 4096 entries per block.  The maximum is zeroed by the stage before (k_zero_amax).
__global__ void __launch_bounds__(kThreads)
k_amax(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    float m = 0.f;
    const int64_t end = min<int64_t>(d.ny, (int64_t)wk.y + 16 * kThreads);
    for (int64_t i = (int64_t)wk.y + threadIdx.x; i < end; i += kThreads)
        m = fmaxf(m, fmaxf(fabsf(d.u[i].x), fabsf(d.u[i].y)));
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    if ((threadIdx.x & 63) == 0 && m > 0.f) atomicMax(reinterpret_cast<unsigned int *>(d.amax), __float_as_uint(m));
}

// item (desc, 0): zero the instance's max |u| (a kernel, not a memset, so the apply can be captured)
__global__ void k_zero_amax(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    if (threadIdx.x == 0) *descs[wk.x].amax = 0.f;
}

// v[i] = 0 (empty plans: no sources or no targets)
__global__ void __launch_bounds__(kThreads) k_zero_out(float2 *v, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < n) v[i] = make_float2(0.f, 0.f);
}

// item (desc, first index): vout[i] = 0 for i < nx ncomp (an instance without sources inside a batch)
__global__ void __launch_bounds__(kThreads)
k_zero_io(const LDesc *__restrict__ descs, const IoEntry *__restrict__ io, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int64_t i = (int64_t)wk.y + threadIdx.x;
    if (i < d.nx * d.ncomp) io[d.inst].vout[i] = make_float2(0.f, 0.f);
}

// item (desc, first index): vout[perm_x[i]] = v[i]; gradient plans: vout[3 perm_x[i] + c] = v[c nx + i]
__global__ void __launch_bounds__(kThreads)
k_perm_out(const LDesc *__restrict__ descs, const IoEntry *__restrict__ io, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int64_t i = (int64_t)wk.y + threadIdx.x;
    if (i >= d.nx) return;
    if (d.ncomp == 1) {
        io[d.inst].vout[d.perm_x[i]] = d.v[i];
        return;
    }
    const int64_t o = 3 * (int64_t)d.perm_x[i];
    for (int c = 0; c < 3; ++c) io[d.inst].vout[o + c] = d.v[(int64_t)c * d.nx + i];
}

// ------------------------------------------------------------------ Gegenbauer levels, direction pairs
// Forward transform u~_s(q) = sum_{j in s} e^{-ik s_q.(y_j - c_s)} u_j for an antipodal pair (q, -q): with
// S = sum cos(th) u, T = sum sin(th) u, u~(q) = S - iT and u~(-q) = S + iT.
// Item (desc, source box, tile of 256 PPT pairs); the box's points stream through LDS.
// With DL (the normal derivative at the sources), every direction's term is multiplied by -ik (s . n_j): with
// a_j = k (s_q . n_j) u_j and S, T now the sums of cos(th) a and sin(th) a, u~(q) = -i (S - iT) and
// u~(-q) = i (S + iT).
template <int PPT, int BS, bool P64, bool DL>
__device__ __forceinline__ void pw_forward_body(const LDesc &d, const int4 wk) {
    const int b = wk.y;
    const int tid = threadIdx.x;
    const int64_t npair = d.npair;
    const int64_t p0 = (int64_t)wk.z * BS * PPT + tid;
    typedef typename std::conditional<P64, double, float>::type real;
    real sx[PPT], sy[PPT], sz[PPT];
    float Sre[PPT], Sim[PPT], Tre[PPT], Tim[PPT];
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        const int64_t p = p0 + (int64_t)j * BS;
        const int64_t pc = p < npair ? p : npair - 1;
        if (P64) {
            sx[j] = d.dirs64[3 * pc]; sy[j] = d.dirs64[3 * pc + 1]; sz[j] = d.dirs64[3 * pc + 2];
        } else {
            const float4 q = d.dirs[pc];
            sx[j] = q.x; sy[j] = q.y; sz[j] = q.z;
        }
        Sre[j] = Sim[j] = Tre[j] = Tim[j] = 0.f;
    }
    const double cx = d.sctr[3 * b], cy = d.sctr[3 * b + 1], cz = d.sctr[3 * b + 2];
    __shared__ real px[BS], py[BS], pz[BS];
    __shared__ float2 us[BS];
    __shared__ float4 ns[DL ? BS : 1];
    const int i0 = d.sstart[b], i1 = d.sstart[b + 1];
    for (int s0 = i0; s0 < i1; s0 += BS) {
        const int cnt = min(BS, i1 - s0);
        __syncthreads();
        if (tid < cnt) {
            const int i = s0 + tid;
            px[tid] = (real)(d.sxs[i] - cx);
            py[tid] = (real)(d.sys[i] - cy);
            pz[tid] = (real)(d.szs[i] - cz);
            us[tid] = d.u[i];
            if (DL) ns[tid] = d.sn[i];
        }
        __syncthreads();
        for (int jj = 0; jj < cnt; ++jj) {
            const real x = px[jj], y = py[jj], z = pz[jj];
            const float2 uu = us[jj];
#pragma unroll
            for (int j = 0; j < PPT; ++j) {
                float f;
                if (P64) {
                    const double ph = fma((double)sx[j], (double)x, fma((double)sy[j], (double)y, (double)sz[j] * z));
                    f = (float)__builtin_amdgcn_fract(ph);
                } else {
                    const float ph = fmaf((float)sx[j], (float)x, fmaf((float)sy[j], (float)y, (float)sz[j] * (float)z));
                    f = ph;
                }
                float sn, cs;
                sincos_rev(f, sn, cs);
                float ax = uu.x, ay = uu.y;
                if (DL) {
                    // k (s . n) = 2 pi (s k / 2 pi) . n
                    const float4 n = ns[jj];
                    const float D = 6.2831853f * fmaf((float)sx[j], n.x, fmaf((float)sy[j], n.y, (float)sz[j] * n.z));
                    ax *= D;
                    ay *= D;
                }
                Sre[j] = fmaf(cs, ax, Sre[j]);
                Sim[j] = fmaf(cs, ay, Sim[j]);
                Tre[j] = fmaf(sn, ax, Tre[j]);
                Tim[j] = fmaf(sn, ay, Tim[j]);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        const int64_t p = p0 + (int64_t)j * BS;
        if (p < npair) {
            d.ut[(int64_t)b * npair + p] =
                DL ? make_float4(Sim[j] - Tre[j], -(Sre[j] + Tim[j]), -(Sim[j] + Tre[j]), Sre[j] - Tim[j])
                   : make_float4(Sre[j] + Tim[j], Sim[j] - Tre[j], Sre[j] - Tim[j], Sim[j] + Tre[j]);
        }
    }
}

template <int PPT, int BS, bool P64>
__global__ void __launch_bounds__(BS)
k_pw_forward(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    pw_forward_body<PPT, BS, P64, false>(descs[wk.x], wk);
}

template <int PPT, int BS, bool P64>
__global__ void __launch_bounds__(BS)
k_pw_forward_dl(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    pw_forward_body<PPT, BS, P64, true>(descs[wk.x], wk);
}

// Diagonal transfer v~_t(q) = sum_{s in far(t)} D_{c(t,s)}(q) u~_s(q) (both directions of a pair), for
// target t and the pairs p0 + j BS, j < PPT (t the same across the wave).
template <int PPT, int BS>
__device__ __forceinline__ void transfer_target(const LDesc &d, int t, int64_t p0) {
    const int64_t npair = d.npair;
    float4 acc[PPT];
#pragma unroll
    for (int j = 0; j < PPT; ++j) acc[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    const int e0 = __builtin_amdgcn_readfirstlane((int)d.far_ptr[t]);
    const int e1 = __builtin_amdgcn_readfirstlane((int)d.far_ptr[t + 1]);
    const float4 *__restrict__ D = d.D;
    const float4 *__restrict__ ut = d.ut;
    // the far list in chunks of 64 entries, one per lane (a single load and wait per chunk), then four far
    // pairs per step taken from the lanes' registers, their data loads issued together
    constexpr int U = 4;
    const int lane = threadIdx.x & 63;
    for (int c0 = e0; c0 < e1; c0 += 64) {
        const int nch = min(64, e1 - c0);
        int src_l = 0, cls_l = 0;
        if (lane < nch) {
            src_l = d.far_src[c0 + lane];
            cls_l = d.far_cls[c0 + lane];
        }
        int k0 = 0;
        for (; k0 + U <= nch; k0 += U) {
            int64_t sv[U], cv[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                sv[k] = __builtin_amdgcn_readlane(src_l, k0 + k);
                cv[k] = __builtin_amdgcn_readlane(cls_l, k0 + k);
            }
#pragma unroll
            for (int j = 0; j < PPT; ++j) {
                const int64_t p = p0 + (int64_t)j * BS;
                if (p < npair) {
                    float4 q[U], w[U];
#pragma unroll
                    for (int k = 0; k < U; ++k) {
                        q[k] = D[cv[k] * npair + p];
                        w[k] = ut[sv[k] * npair + p];
                    }
#pragma unroll
                    for (int k = 0; k < U; ++k) {
                        acc[j].x = fmaf(q[k].x, w[k].x, fmaf(-q[k].y, w[k].y, acc[j].x));
                        acc[j].y = fmaf(q[k].x, w[k].y, fmaf(q[k].y, w[k].x, acc[j].y));
                        acc[j].z = fmaf(q[k].z, w[k].z, fmaf(-q[k].w, w[k].w, acc[j].z));
                        acc[j].w = fmaf(q[k].z, w[k].w, fmaf(q[k].w, w[k].z, acc[j].w));
                    }
                }
            }
        }
        for (; k0 < nch; ++k0) {
            const int64_t s = __builtin_amdgcn_readlane(src_l, k0), c = __builtin_amdgcn_readlane(cls_l, k0);
#pragma unroll
            for (int j = 0; j < PPT; ++j) {
                const int64_t p = p0 + (int64_t)j * BS;
                if (p < npair) {
                    const float4 q = D[c * npair + p];
                    const float4 w = ut[s * npair + p];
                    acc[j].x = fmaf(q.x, w.x, fmaf(-q.y, w.y, acc[j].x));
                    acc[j].y = fmaf(q.x, w.y, fmaf(q.y, w.x, acc[j].y));
                    acc[j].z = fmaf(q.z, w.z, fmaf(-q.w, w.w, acc[j].z));
                    acc[j].w = fmaf(q.z, w.w, fmaf(q.w, w.z, acc[j].w));
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        const int64_t p = p0 + (int64_t)j * BS;
        if (p < npair) d.vt[(int64_t)t * npair + p] = acc[j];
    }
}

// Item (desc, target box, tile of BS PPT pairs).
template <int PPT, int BS>
__global__ void __launch_bounds__(BS)
k_pw_transfer(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    transfer_target<PPT, BS>(descs[wk.x], wk.y, (int64_t)wk.z * BS * PPT + threadIdx.x);
}

// Four consecutive target slots (Morton order) per block, one per wave, on the same tile of 64 pairs: a
// quarter of the blocks and work items of one target per block, for the same work per wave.  Item (desc,
// group of four slots, tile).
__global__ void __launch_bounds__(kThreads)
k_pw_transfer_grp(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int ti = __builtin_amdgcn_readfirstlane(wk.y * 4 + (int)(threadIdx.x >> 6));
    if (ti >= d.ntr) return;
    transfer_target<1, 64>(d, __builtin_amdgcn_readfirstlane(d.tr_tgt[ti]), (int64_t)wk.z * 64 + (threadIdx.x & 63));
}

// The transfer by sibling group (one tree): wave w of a block takes group 4 item.y + w, up to four targets of one
// parent box, on a tile of 64 pairs.  The group's far sources are visited once each (in position order): u~_s is read
// once and applied to every sibling whose far list holds s, with that pair's D.  Item (desc, block of four
// groups, tile).
__global__ void __launch_bounds__(kThreads)
k_pw_transfer_sib(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int g = __builtin_amdgcn_readfirstlane(wk.y * 4 + (int)(threadIdx.x >> 6));
    if (g >= d.nsibg) return;
    const int64_t npair = d.npair;
    const int64_t p0 = (int64_t)wk.z * 64 + (threadIdx.x & 63);
    const bool active = p0 < npair;
    const int64_t p = active ? p0 : npair - 1;       // idle lanes read a valid pair and store nothing
    const float4 *__restrict__ D = d.D;
    const float4 *__restrict__ ut = d.ut;
    float4 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    const int n = __builtin_amdgcn_readfirstlane(d.sib_cnt[g]);
    const int32_t *src = d.sib_src + (int64_t)216 * g;
    const uint2 *cls = d.sib_cls + (int64_t)216 * g;
    const int lane = threadIdx.x & 63;
    // the group's slots in chunks of 64, one per lane (one load and wait per chunk), then taken from the lanes'
    // registers slot by slot
    for (int c0 = 0; c0 < n; c0 += 64) {
        const int nch = min(64, n - c0);
        int src_l = 0;
        uint2 cls_l = make_uint2(0xFFFFFFFFu, 0xFFFFFFFFu);
        if (lane < nch) {
            src_l = src[c0 + lane];
            cls_l = cls[c0 + lane];
        }
        for (int k = 0; k < nch; ++k) {
            const int64_t sv = __builtin_amdgcn_readlane(src_l, k);
            const uint32_t wds[2] = {(uint32_t)__builtin_amdgcn_readlane((int)cls_l.x, k),
                                     (uint32_t)__builtin_amdgcn_readlane((int)cls_l.y, k)};
            const float4 w = ut[sv * npair + p];
            float4 q[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int c = (int)(int16_t)(wds[j >> 1] >> (16 * (j & 1)));
                if (c >= 0) q[j] = D[(int64_t)c * npair + p];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int c = (int)(int16_t)(wds[j >> 1] >> (16 * (j & 1)));
                if (c >= 0) {
                    acc[j].x = fmaf(q[j].x, w.x, fmaf(-q[j].y, w.y, acc[j].x));
                    acc[j].y = fmaf(q[j].x, w.y, fmaf(q[j].y, w.x, acc[j].y));
                    acc[j].z = fmaf(q[j].z, w.z, fmaf(-q[j].w, w.w, acc[j].z));
                    acc[j].w = fmaf(q[j].z, w.w, fmaf(q[j].w, w.z, acc[j].w));
                }
            }
        }
    }
    if (!active) return;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int t = __builtin_amdgcn_readfirstlane(d.sib_tgt[4 * g + j]);
        if (t >= 0) d.vt[(int64_t)t * npair + p0] = acc[j];
    }
}

// The same transfer for levels with many direction pairs per box.  Block: a
// tile of QT direction pairs for 256 / QT target boxes (consecutive in Morton order); the tile of every class's
// D is staged in LDS once per block, so each far pair reads D from LDS and only u~ from memory.  Four far pairs
// per step, their loads issued together.  Item (desc, group of target slots, tile).
template <int QT>
__global__ void __launch_bounds__(kThreads)
k_pw_transfer_lds(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    extern __shared__ float4 Ds[];            // [ncls][QT]
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int64_t npair = d.npair, q0 = (int64_t)wk.z * QT;
    const int ncls = d.ncls;
    for (int k = threadIdx.x; k < ncls * QT; k += kThreads) {
        const int c = k / QT, ql = k % QT;
        Ds[k] = q0 + ql < npair ? d.D[(int64_t)c * npair + q0 + ql] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();
    const int slot = threadIdx.x / QT, ql = threadIdx.x % QT;
    const int ti = wk.y * (kThreads / QT) + slot;
    const int64_t q = q0 + ql;
    if (ti >= d.ntr || q >= npair) return;
    const int t = d.tr_tgt[ti];
    const float4 *__restrict__ ut = d.ut;
    const float4 *Dq = Ds + ql;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    auto step = [&](const float4 &dq, const float4 &w) {
        acc.x = fmaf(dq.x, w.x, fmaf(-dq.y, w.y, acc.x));
        acc.y = fmaf(dq.x, w.y, fmaf(dq.y, w.x, acc.y));
        acc.z = fmaf(dq.z, w.z, fmaf(-dq.w, w.w, acc.z));
        acc.w = fmaf(dq.z, w.w, fmaf(dq.w, w.z, acc.w));
    };
    const int64_t e0 = d.far_ptr[t], e1 = d.far_ptr[t + 1];
    int64_t e = e0;
    // groups of four far pairs; the list entries of the next group are loaded while this group's u~ loads
    // are in flight
    int sn[4], cn[4];
    if (e + 4 <= e1) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            sn[k] = d.far_src[e + k];
            cn[k] = d.far_cls[e + k];
        }
    }
    for (; e + 4 <= e1; e += 4) {
        int64_t sv[4];
        int cv[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            sv[k] = sn[k];
            cv[k] = cn[k];
        }
        float4 w[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = ut[sv[k] * npair + q];
        if (e + 8 <= e1) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                sn[k] = d.far_src[e + 4 + k];
                cn[k] = d.far_cls[e + 4 + k];
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) step(Dq[cv[k] * QT], w[k]);
    }
    for (; e < e1; ++e) step(Dq[d.far_cls[e] * QT], ut[(int64_t)d.far_src[e] * npair + q]);
    d.vt[(int64_t)t * npair + q] = acc;
}

// Gradient plans: the target transform of component c is that of ik s_c v~, so the plain transforms (direct,
// ring or grid form) give the derivative along axis c.  For the pair (q, -q) (s(-q) = -s(q)):
// ik s_c v~(q) = f (-Im, Re) and -ik s_c v~(-q) = f (Im, -Re), f = k s_c = 2 pi (k s / 2 pi)_c.  Components 1 and 2
// go to the descriptor's vtx planes, component 0 replaces v~.  Item (desc, target box, tile of 256 pairs).
__global__ void __launch_bounds__(kThreads)
k_dir_scale(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int64_t p = (int64_t)wk.z * kThreads + threadIdx.x;
    if (p >= d.npair) return;
    const int64_t o = (int64_t)wk.y * d.npair + p;
    const float4 w = d.vt[o];
    const float4 s = d.dirs[p];
    auto sc = [&](float f) { return make_float4(-f * w.y, f * w.x, f * w.w, -f * w.z); };
    d.vtx[o] = sc(6.2831853f * s.y);
    d.vtx[d.vtstride + o] = sc(6.2831853f * s.z);
    d.vt[o] = sc(6.2831853f * s.x);
}

// Split double layer: u~(q) = -ik sum_c s_c u~_c(q) from the source transforms u~_c of the densities u n_c (in
// place of u~_0); for the pair (q, -q), with f_c = k s_c(q) = 2 pi (k s / 2 pi)_c:
// u~(q) = sum_c f_c (Im, -Re) u~_c(q) and u~(-q) = sum_c f_c (-Im, Re) u~_c(-q).  Item (desc, source box, tile of
// 256 pairs).
__global__ void __launch_bounds__(kThreads)
k_dl_combine(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int64_t p = (int64_t)wk.z * kThreads + threadIdx.x;
    if (p >= d.npair) return;
    const int64_t o = (int64_t)wk.y * d.npair + p;
    const float4 a = d.ut[o], b = d.utx[o], c = d.utx[d.utstride + o];
    const float4 s = d.dirs[p];
    const float fx = 6.2831853f * s.x, fy = 6.2831853f * s.y, fz = 6.2831853f * s.z;
    d.ut[o] = make_float4(fmaf(fx, a.y, fmaf(fy, b.y, fz * c.y)), -fmaf(fx, a.x, fmaf(fy, b.x, fz * c.x)),
                          -fmaf(fx, a.w, fmaf(fy, b.w, fz * c.w)), fmaf(fx, a.z, fmaf(fy, b.z, fz * c.z)));
}

// Split normal derivative at the targets: v_i += n_i . (T_0, T_1, T_2)_i over the axis planes of a level's
// target transforms, which are cleared for the next level.  Item (desc, target box, first point), 256 points.
__global__ void __launch_bounds__(kThreads)
k_dn_combine(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int i = wk.z + threadIdx.x;
    if (i >= d.tstart[wk.y + 1]) return;
    const float4 n = d.tn[i];
    float2 *t0 = d.vtmp + i, *t1 = t0 + d.nx, *t2 = t1 + d.nx;
    const float2 a = *t0, b = *t1, c = *t2;
    float2 o = d.v[i];
    o.x = fmaf(n.x, a.x, fmaf(n.y, b.x, fmaf(n.z, c.x, o.x)));
    o.y = fmaf(n.x, a.y, fmaf(n.y, b.y, fmaf(n.z, c.y, o.y)));
    d.v[i] = o;
    *t0 = *t1 = *t2 = make_float2(0.f, 0.f);
}

// Backward transform v_i += sum_q e^{ik s_q.(x_i - c_t)} v~_t(q): per pair, with A = v~(q) + v~(-q) and
// B = v~(q) - v~(-q), the pair contributes cos(th) A + i sin(th) B.  Item (desc, target box, first point);
// BS points per block (64 for levels of small boxes).
// With DN (the normal derivative at the target), every direction's term is multiplied by ik (s . n_i): the pair
// (q, -q) contributes ik (s_q . n) (e^{iP} v~(q) - e^{-iP} v~(-q)), with k s_q . n from the scaled directions.
template <int BS, bool P64, bool DN>
__device__ __forceinline__ void pw_backward_body(const LDesc &d, const int4 wk) {
    const int t = wk.y;
    const int tid = threadIdx.x;
    const int i = wk.z + tid;
    const bool valid = i < d.tstart[t + 1];
    const int64_t npair = d.npair;
    typedef typename std::conditional<P64, double, float>::type real;
    real x = 0, y = 0, z = 0;
    float nx = 0.f, ny = 0.f, nz = 0.f;
    if (valid) {
        x = (real)(d.txs[i] - d.tctr[3 * t]);
        y = (real)(d.tys[i] - d.tctr[3 * t + 1]);
        z = (real)(d.tzs[i] - d.tctr[3 * t + 2]);
        if (DN) {
            const float4 n = d.tn ? d.tn[i] : d.tnc;
            nx = n.x;
            ny = n.y;
            nz = n.z;
        }
    }
    float are = 0.f, aim = 0.f;
    __shared__ real sdx[BS], sdy[BS], sdz[BS];
    __shared__ float4 ab[BS];
    const float4 *vb = d.vt + (int64_t)t * npair;
    for (int64_t q0 = 0; q0 < npair; q0 += BS) {
        const int cnt = (int)min<int64_t>(BS, npair - q0);
        __syncthreads();
        if (tid < cnt) {
            const int64_t q = q0 + tid;
            if (P64) {
                sdx[tid] = d.dirs64[3 * q]; sdy[tid] = d.dirs64[3 * q + 1]; sdz[tid] = d.dirs64[3 * q + 2];
            } else {
                const float4 w = d.dirs[q];
                sdx[tid] = w.x; sdy[tid] = w.y; sdz[tid] = w.z;
            }
            const float4 w = vb[q];
            ab[tid] = DN ? make_float4(w.x - w.z, w.y - w.w, w.x + w.z, w.y + w.w)
                         : make_float4(w.x + w.z, w.y + w.w, w.x - w.z, w.y - w.w);
        }
        __syncthreads();
        for (int jj = 0; jj < cnt; ++jj) {
            float f;
            if (P64) {
                const double ph = fma((double)sdx[jj], (double)x, fma((double)sdy[jj], (double)y, (double)sdz[jj] * z));
                f = (float)__builtin_amdgcn_fract(ph);
            } else {
                const float ph = fmaf((float)sdx[jj], (float)x, fmaf((float)sdy[jj], (float)y, (float)sdz[jj] * (float)z));
                f = ph;
            }
            float sn, cs;
            sincos_rev(f, sn, cs);
            const float4 w = ab[jj];
            if (DN) {
                // k (s . n) = 2 pi (s k / 2 pi) . n; X + iY = e^{iP} v~(q) - e^{-iP} v~(-q); adds i k (s . n) (X + iY)
                const float D = 6.2831853f * fmaf((float)sdx[jj], nx, fmaf((float)sdy[jj], ny, (float)sdz[jj] * nz));
                const float X = fmaf(cs, w.x, -sn * w.w), Y = fmaf(cs, w.y, sn * w.z);
                are = fmaf(-D, Y, are);
                aim = fmaf(D, X, aim);
            } else {
                are = fmaf(cs, w.x, fmaf(-sn, w.w, are));
                aim = fmaf(cs, w.y, fmaf(sn, w.z, aim));
            }
        }
    }
    if (valid) {
        float2 o = d.v[i];
        o.x += are;
        o.y += aim;
        d.v[i] = o;
    }
}

template <int BS, bool P64>
__global__ void __launch_bounds__(BS)
k_pw_backward(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    pw_backward_body<BS, P64, false>(descs[wk.x], wk);
}

template <int BS, bool P64>
__global__ void __launch_bounds__(BS)
k_pw_backward_dn(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    pw_backward_body<BS, P64, true>(descs[wk.x], wk);
}

// ------------------------------------------------------------------ Gegenbauer levels, ring-pair form
// The quadrature's directions (sin t_m cos f_n, sin t_m sin f_n, cos t_m) of ring m and its antipodal
// ring L - m (cos t_{L-m} = -cos t_m) with f_n and f_n + pi give four directions whose phases against
// a box-centred point y are +-P +- C, P = (k/2pi) sin t_m (y_1 cos f_n + y_2 sin f_n) and
// C = (k/2pi) cos t_m y_3.  One sin/cos of P and the per-(point, ring) factors e^{-+iC} serve all four:
//   u~(m, n)        = sum e^{-iP} u',    u~(m, n+L)     = sum e^{+iP} u',    u' = u e^{-iC}
//   u~(L-m, n)      = sum e^{-iP} u'',   u~(L-m, n+L)   = sum e^{+iP} u'',   u'' = u e^{+iC}
// Storage keeps the direction-pair layout: pair (m, n) = (u~(m,n), u~(L-m,n+L)), pair (m, n+L) =
// (u~(m,n+L), u~(L-m,n)); the equator ring (m = L/2, L even) holds pair (m, n) = (u~(m,n), u~(m,n+L)).
// C is reduced in FP64 once per (point, ring); P is evaluated in FP32 or FP64 (P64).
constexpr int kRingChunk = 64;
constexpr int kMaxRings = 16;

// Item (desc, source box, ring chunk, point segment); Tr threads per ring, R rings per block.
template <int G, bool P64>
__global__ void __launch_bounds__(kThreads)
k_pw_forward_rings(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    typedef typename std::conditional<P64, double, float>::type real;
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int b = wk.y;
    const int L = d.L, nrp = d.nrp, Tr = d.Tr, R = d.R, nsplit = d.nsplit, seg = wk.w;
    const int64_t npair = d.npair;
    const int m0 = wk.z * R;
    const int tid = threadIdx.x;
    const int rl = tid / Tr, nloc = tid % Tr;
    const int m = m0 + rl;
    const int nr = min(R, nrp - m0);
    const bool active = rl < nr;
    real cf[G], sf[G];
    float acc[G][8];
#pragma unroll
    for (int j = 0; j < G; ++j) {
        const int n = min(nloc + j * Tr, L - 1);
        cf[j] = (real)d.phis[n].x;
        sf[j] = (real)d.phis[n].y;
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[j][q] = 0.f;
    }
    const double cx = d.sctr[3 * b], cy = d.sctr[3 * b + 1], cz = d.sctr[3 * b + 2];
    __shared__ real sA[kMaxRings][kRingChunk], sB[kMaxRings][kRingChunk];
    __shared__ float4 sU[kMaxRings][kRingChunk];
    // this block's segment of the box's points
    const int b0 = d.sstart[b], b1 = d.sstart[b + 1];
    const int per = (b1 - b0 + nsplit - 1) / nsplit;
    const int i0 = b0 + seg * per, i1 = min(b1, i0 + per);
    for (int s0 = i0; s0 < i1; s0 += kRingChunk) {
        const int cnt = min(kRingChunk, i1 - s0);
        __syncthreads();
        for (int it = tid; it < nr * cnt; it += kThreads) {
            const int r = it / cnt, j = it % cnt, i = s0 + j;
            const double2 rg = d.rings[m0 + r];
            const double xr = d.sxs[i] - cx, yr = d.sys[i] - cy, zr = d.szs[i] - cz;
            sA[r][j] = (real)(rg.x * xr);
            sB[r][j] = (real)(rg.x * yr);
            const double C = rg.y * zr;
            float sn, cs;
            sincos_rev((float)(C - floor(C)), sn, cs);
            const float2 uu = d.u[i];
            // explicit fused forms: the rounding must not depend on how the compiler contracts
            sU[r][j] = make_float4(fmaf(uu.x, cs, uu.y * sn), fmaf(uu.y, cs, -(uu.x * sn)),
                                   fmaf(uu.x, cs, -(uu.y * sn)), fmaf(uu.y, cs, uu.x * sn));
        }
        __syncthreads();
        if (active) {
            for (int jj = 0; jj < cnt; ++jj) {
                const real A = sA[rl][jj], B = sB[rl][jj];
                const float4 w = sU[rl][jj];
#pragma unroll
                for (int j = 0; j < G; ++j) {
                    float f;
                    if (P64) {
                        const double P = fma((double)A, (double)cf[j], (double)B * (double)sf[j]);
                        f = (float)__builtin_amdgcn_fract(P);
                    } else {
                        const float P = fmaf((float)A, (float)cf[j], (float)B * (float)sf[j]);
                        f = P;
                    }
                    float sn, cs;
                    sincos_rev(f, sn, cs);
                    acc[j][0] = fmaf(cs, w.x, acc[j][0]);
                    acc[j][1] = fmaf(cs, w.y, acc[j][1]);
                    acc[j][2] = fmaf(sn, w.x, acc[j][2]);
                    acc[j][3] = fmaf(sn, w.y, acc[j][3]);
                    acc[j][4] = fmaf(cs, w.z, acc[j][4]);
                    acc[j][5] = fmaf(cs, w.w, acc[j][5]);
                    acc[j][6] = fmaf(sn, w.z, acc[j][6]);
                    acc[j][7] = fmaf(sn, w.w, acc[j][7]);
                }
            }
        }
    }
    if (!active) return;
    const bool equator = 2 * m == L;
    float4 *o = (nsplit > 1 ? d.part + (int64_t)seg * d.part_stride : d.ut) + (int64_t)b * npair + (int64_t)m * 2 * L;
#pragma unroll
    for (int j = 0; j < G; ++j) {
        const int n = nloc + j * Tr;
        if (n >= L) continue;
        // S' = (0,1), T' = (2,3), S'' = (4,5), T'' = (6,7); S -+ iT
        const float2 k0 = make_float2(acc[j][0] + acc[j][3], acc[j][1] - acc[j][2]);
        const float2 k1 = make_float2(acc[j][0] - acc[j][3], acc[j][1] + acc[j][2]);
        const float2 k2 = make_float2(acc[j][4] + acc[j][7], acc[j][5] - acc[j][6]);
        const float2 k3 = make_float2(acc[j][4] - acc[j][7], acc[j][5] + acc[j][6]);
        if (equator) {
            o[n] = make_float4(k0.x, k0.y, k1.x, k1.y);
        } else {
            o[n] = make_float4(k0.x, k0.y, k3.x, k3.y);
            o[n + L] = make_float4(k1.x, k1.y, k2.x, k2.y);
        }
    }
}

// Sum the point-segment partials of the forward transform, or of the anterpolation, in segment order.  Item (desc, source box).
__global__ void __launch_bounds__(kThreads)
k_sum_segments(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int64_t npair = d.npair;
    for (int64_t p = threadIdx.x; p < npair; p += kThreads) {
        const int64_t o = (int64_t)wk.y * npair + p;
        float4 a = d.part[o];
        for (int s = 1; s < d.nsplit; ++s) {
            const float4 w = d.part[(int64_t)s * d.part_stride + o];
            a.x += w.x; a.y += w.y; a.z += w.z; a.w += w.w;
        }
        d.ut[o] = a;
    }
}

// Backward transform in ring-pair form: per target point and ring pair m,
//   v += e^{iC} sum_n [e^{iP} v~(m,n) + e^{-iP} v~(m,n+L)] + e^{-iC} sum_n [e^{iP} v~(L-m,n) + e^{-iP} v~(L-m,n+L)]
// PT target points per thread, BS threads per block; item (desc, target box, first point).  The staged entries of a ring pair are
// padded with zeros to a multiple of U (a zero term leaves every sum unchanged), so the inner loop runs in
// unrolled steps of U with immediate LDS offsets.  Where a ring's padded azimuths fit one block's worth, the
// entries of as many ring pairs as fit kBkStage go to LDS at once (one load round and one barrier pair for
// all of them); otherwise ring pair by ring pair in chunks of kThreads azimuths.  Either way each ring pair's
// sums run over the same terms in the same order.
constexpr int kBkStage = 512;

// entries of ring pair m, azimuth n: (v~(m,n) + v~(m,n+L), i-free difference) pairs as the inner sums use them
__device__ __forceinline__ void bk_stage_entry(const float4 *vb, int L, int m, int n, float4 &e01, float4 &e23) {
    const float4 p1 = vb[(int64_t)m * 2 * L + n];
    if (2 * m == L) {
        e01 = make_float4(p1.x + p1.z, p1.y + p1.w, p1.x - p1.z, p1.y - p1.w);
        e23 = make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
        const float4 p2 = vb[(int64_t)m * 2 * L + n + L];
        e01 = make_float4(p1.x + p2.x, p1.y + p2.y, p1.x - p2.x, p1.y - p2.y);
        e23 = make_float4(p2.z + p1.z, p2.w + p1.w, p2.z - p1.z, p2.w - p1.w);
    }
}

template <int PT, int U, bool P64, typename real>
__device__ __forceinline__ void bk_ring_terms(const float4 *s01, const float4 *s23, const real *scf, const real *ssf,
                                              int cnt4, const real *A, const real *B, float *xre, float *xim,
                                              float *yre, float *yim) {
    for (int j0 = 0; j0 < cnt4; j0 += U) {
#pragma unroll
        for (int ju = 0; ju < U; ++ju) {
            const int jj = j0 + ju;
            const real cfn = scf[jj], sfn = ssf[jj];
            const float4 a = s01[jj], c = s23[jj];
#pragma unroll
            for (int q = 0; q < PT; ++q) {
                float f;
                if (P64) {
                    const double P = fma((double)A[q], (double)cfn, (double)B[q] * (double)sfn);
                    f = (float)__builtin_amdgcn_fract(P);
                } else {
                    const float P = fmaf((float)A[q], (float)cfn, (float)B[q] * (float)sfn);
                    f = P;
                }
                float sn, cs;
                sincos_rev(f, sn, cs);
                xre[q] = fmaf(cs, a.x, fmaf(-sn, a.w, xre[q]));
                xim[q] = fmaf(cs, a.y, fmaf(sn, a.z, xim[q]));
                yre[q] = fmaf(cs, c.x, fmaf(-sn, c.w, yre[q]));
                yim[q] = fmaf(cs, c.y, fmaf(sn, c.z, yim[q]));
            }
        }
    }
}

template <int PT, int U, bool P64, int BS = kThreads>
__global__ void __launch_bounds__(BS)
k_pw_backward_rings(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    typedef typename std::conditional<P64, double, float>::type real;
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int t = wk.y;
    const int tid = threadIdx.x;
    const int L = d.L, nrp = d.nrp;
    const int64_t npair = d.npair;
    const int iend = d.tstart[t + 1];
    double xr[PT], yr[PT], zr[PT];
    bool valid[PT];
    float vr[PT], vi[PT];
#pragma unroll
    for (int q = 0; q < PT; ++q) {
        const int i = wk.z + tid + q * BS;
        valid[q] = i < iend;
        xr[q] = valid[q] ? d.txs[i] - d.tctr[3 * t] : 0.0;
        yr[q] = valid[q] ? d.tys[i] - d.tctr[3 * t + 1] : 0.0;
        zr[q] = valid[q] ? d.tzs[i] - d.tctr[3 * t + 2] : 0.0;
        vr[q] = vi[q] = 0.f;
    }
    __shared__ float4 s01[kBkStage], s23[kBkStage];
    __shared__ real scf[kThreads], ssf[kThreads];
    const float4 *vb = d.vt + (int64_t)t * npair;
    // this block's ring pairs (part wk.w of bsplit)
    const int mper = (nrp + d.bsplit - 1) / d.bsplit;
    const int mb = wk.w * mper, me = min(nrp, mb + mper);
    const int Lp = (L + U - 1) / U * U;
    // per ring pair: the point factors, then the sums over its azimuths (staged at e01, e23), then the
    // ring's contribution to v
    auto ring = [&](int m, const float4 *e01, const float4 *e23, int n0, int cnt4, bool first, bool last,
                    float *xre, float *xim, float *yre, float *yim, float *ecs, float *esn, real *A, real *B) {
        if (first) {
            const double2 rg = d.rings[m];
#pragma unroll
            for (int q = 0; q < PT; ++q) {
                A[q] = (real)(rg.x * xr[q]);
                B[q] = (real)(rg.x * yr[q]);
                const double C = rg.y * zr[q];
                sincos_rev((float)(C - floor(C)), esn[q], ecs[q]);
                xre[q] = xim[q] = yre[q] = yim[q] = 0.f;
            }
        }
        bk_ring_terms<PT, U, P64, real>(e01, e23, scf + n0, ssf + n0, cnt4, A, B, xre, xim, yre, yim);
        if (last) {
#pragma unroll
            for (int q = 0; q < PT; ++q) {
                // explicit fused forms, so every points-per-thread variant rounds identically
                vr[q] = fmaf(ecs[q], xre[q] + yre[q], fmaf(-esn[q], xim[q] - yim[q], vr[q]));
                vi[q] = fmaf(ecs[q], xim[q] + yim[q], fmaf(esn[q], xre[q] - yre[q], vi[q]));
            }
        }
    };
    real A[PT], B[PT];
    float ecs[PT], esn[PT], xre[PT], xim[PT], yre[PT], yim[PT];
    if (Lp <= kThreads) {
        // whole rings: the azimuth tables once, then groups of ring pairs
        for (int e = tid; e < Lp; e += BS) {
            scf[e] = e < L ? (real)d.phis[e].x : (real)0;
            ssf[e] = e < L ? (real)d.phis[e].y : (real)0;
        }
        const int rps = kBkStage / Lp;
        for (int g0 = mb; g0 < me; g0 += rps) {
            const int ng = min(rps, me - g0);
            __syncthreads();
            for (int e = tid; e < ng * Lp; e += BS) {
                const int r = e / Lp, n = e - r * Lp;
                if (n >= L) {
                    s01[e] = make_float4(0.f, 0.f, 0.f, 0.f);
                    s23[e] = make_float4(0.f, 0.f, 0.f, 0.f);
                } else {
                    bk_stage_entry(vb, L, g0 + r, n, s01[e], s23[e]);
                }
            }
            __syncthreads();
            for (int r = 0; r < ng; ++r)
                ring(g0 + r, s01 + r * Lp, s23 + r * Lp, 0, Lp, true, true, xre, xim, yre, yim, ecs, esn, A, B);
        }
    } else {
        for (int m = mb; m < me; ++m) {
            for (int n0 = 0; n0 < L; n0 += BS) {
                const int cnt = min(BS, L - n0);
                const int cnt4 = (cnt + U - 1) / U * U;
                __syncthreads();
                if (tid < cnt4) {
                    const int n = n0 + tid;
                    if (tid >= cnt) {
                        s01[tid] = make_float4(0.f, 0.f, 0.f, 0.f);
                        s23[tid] = make_float4(0.f, 0.f, 0.f, 0.f);
                        scf[tid] = (real)0;
                        ssf[tid] = (real)0;
                    } else {
                        bk_stage_entry(vb, L, m, n, s01[tid], s23[tid]);
                        scf[tid] = (real)d.phis[n].x;
                        ssf[tid] = (real)d.phis[n].y;
                    }
                }
                __syncthreads();
                ring(m, s01, s23, 0, cnt4, n0 == 0, n0 + BS >= L, xre, xim, yre, yim, ecs, esn, A, B);
            }
        }
    }
#pragma unroll
    for (int q = 0; q < PT; ++q) {
        if (!valid[q]) continue;
        const int i = wk.z + tid + q * BS;
        if (d.bsplit > 1) {
            d.bpart[(int64_t)wk.w * d.nx + i] = make_float2(vr[q], vi[q]);
        } else {
            float2 o = d.v[i];
            o.x += vr[q];
            o.y += vi[q];
            d.v[i] = o;
        }
    }
}

// v_i += sum over ring parts of the target-transform partials, in part order.  Item (desc, target box,
// first point), 256 points per block.
__global__ void __launch_bounds__(kThreads)
k_sum_parts(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int i = wk.z + threadIdx.x;
    if (i >= d.tstart[wk.y + 1]) return;
    float2 a = d.bpart[i];
    for (int s = 1; s < d.bsplit; ++s) {
        const float2 w = d.bpart[(int64_t)s * d.nx + i];
        a.x += w.x;
        a.y += w.y;
    }
    float2 o = d.v[i];
    o.x += a.x;
    o.y += a.y;
    d.v[i] = o;
}

// ------------------------------------------------------------------ Gegenbauer levels, grid form
// The transforms as sums over a uniform grid: with a smooth kernel phi of width w (grid units) and its
// Fourier transform phi^, e^{-ik s.y} ~ (1/Phi(s)) sum_g phi((x_g - y)/h) e^{-ik s.x_g} (per axis, aliasing
// negligible for kh <= pi / 1.9), Phi(s) = prod_d phi^(k s_d h).  Forward: spread u onto the grid, sum
// over z for every ring (cos t_m), then over the plane for every direction; backward: the mirror sums
// and an interpolation at the targets.  Phi is divided out (twice) in the transfer diagonal.  Grid nodes
// x_a = (a - (p-1)/2) h about the box centre; G [box][c][a][b] (c: z), H [ring][box][a][b].
// Rings m and L - m (cos t opposite) share Ex, Ey; azimuths n and n + L give the conjugate tables.

// phi(x) = exp(beta (sqrt(1 - (2x/w)^2) - 1)) for |x| < w/2, 0 outside (exponential of semicircle), with
// k1 = 2 / w and k2 = beta log2(e): the hardware square root and base-2 exponential (exponents in
// [-27, 0]), about 1e-7 relative.
__device__ __forceinline__ float es_phi(float x, float k1, float k2) {
    const float t = x * k1;
    const float s = fmaf(-t, t, 1.f);
    return s > 0.f ? __builtin_amdgcn_exp2f(k2 * (__builtin_amdgcn_sqrtf(s) - 1.f)) : 0.f;
}

constexpr int kGT = 64;      // spreading tile edge (grid nodes)

// A contribution t (|t| < 2^62) as 64-bit fixed point: hi = floor(t 2^-32) and lo = t - hi 2^32 in [0, 2^32),
// th = t 2^-32 given.  lo is rounded to FP32 and truncated (at most 2^32 - 256), so the value is within a few
// hundred units of t, far below the FP32 rounding of the sums; each contribution is converted once, which keeps the integer sums order-independent.
__device__ __forceinline__ unsigned long long fixed64(float t, float th) {
    const float hi = floorf(th);
    const float lo = fmaf(-hi, 4294967296.f, t);
    return ((unsigned long long)(unsigned)(int)hi << 32) | (unsigned long long)(unsigned)fminf(lo, 4294967040.f);
}

// Spread the source points of a box onto one z-plane of its grid (one tile of at most 64 x 64 nodes), kernel
// width W.  The points come ordered by z-plane floor(z_g) with their grid coordinates: the W planes below and
// at c + W/2 - 1 hold exactly the points whose support reaches plane c.  Every contribution is rounded once
// to 64-bit fixed point (u scaled by 2^(61-e), 2^e >= (points of the box) x max |Re u|, |Im u| >= any partial
// sum) and summed with integer LDS atomics: the sums are exact, so the result does not depend on the order of
// the points.  Lane l of a wave takes every R-th point from l R on, so that the lanes of one atomic
// instruction fall on distinct, distant nodes (points are in Morton order within a plane).  Item (desc, box,
// plane, tile).
template <int W>
__global__ void __launch_bounds__(kThreads)
k_grid_spread(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int sb = wk.y, c = wk.z;
    const int p = d.gp;
    const int nta = (p + kGT - 1) / kGT;
    const int a0 = (wk.w / nta) * kGT, b0 = (wk.w % nta) * kGT;
    const int na = min(kGT, p - a0), nb = min(kGT, p - b0), ncell = na * nb;
    extern __shared__ unsigned long long accs[];           // [part][(a - a0) nb + b - b0], dynamic: 2 ncell
    unsigned long long *acc0 = accs, *acc1 = accs + ncell;
    for (int i = threadIdx.x; i < ncell; i += kThreads) {
        acc0[i] = 0ull;
        acc1[i] = 0ull;
    }
    __syncthreads();
    const double bound = (double)(d.sstart[sb + 1] - d.sstart[sb]) * (double)(*d.amax);
    int e = 0;
    if (bound > 0.0) frexp(bound, &e);
    constexpr float hw = 0.5f * W, k1 = 2.f / W;
    const float k2 = d.gbeta * 1.44269504f;
    const int64_t zoff = (int64_t)sb * p;
    // points binned by plane (even W: floor(z), odd W: nearest plane) whose support reaches plane c
    constexpr int zlo = W / 2, zhi = (W - 1) / 2;
    const int j0 = d.gzs[zoff + max(0, c - zlo)], j1 = d.gzs[zoff + min(p - 1, c + zhi) + 1];
    const int R = (j1 - j0 + 63) / 64, lane = threadIdx.x & 63;
    for (int r = threadIdx.x >> 6; r < R; r += kThreads / 64) {
        const int j = j0 + lane * R + r;
        if (j >= j1) continue;
        const float4 g = d.gxyz[j];
        const int alo = min(max((int)floorf(g.x - hw) + 1, 0), p - W);
        const int blo = min(max((int)floorf(g.y - hw) + 1, 0), p - W);
        if (alo + W <= a0 || alo >= a0 + na || blo + W <= b0 || blo >= b0 + nb) continue;
        const float wz = es_phi((float)c - g.z, k1, k2);
        const float2 uu = d.u[d.gperm[j]];
        const float ur = ldexpf(uu.x * wz, 61 - e), ui = ldexpf(uu.y * wz, 61 - e);
        float wx[W], ry[W], iy[W], rh[W], ih[W];
        int col[W];
#pragma unroll
        for (int k = 0; k < W; ++k) {
            const int a = alo + k, b = blo + k;
            wx[k] = (a >= a0 && a < a0 + na) ? es_phi((float)a - g.x, k1, k2) : 0.f;
            const float wy = (b >= b0 && b < b0 + nb) ? es_phi((float)b - g.y, k1, k2) : 0.f;
            ry[k] = ur * wy;
            iy[k] = ui * wy;
            rh[k] = ry[k] * 2.3283064e-10f;    // 2^-32
            ih[k] = iy[k] * 2.3283064e-10f;
            col[k] = min(max(b - b0, 0), nb - 1);
        }
#pragma unroll
        for (int ka = 0; ka < W; ++ka) {
            const int row = min(max(alo + ka - a0, 0), na - 1) * nb;
#pragma unroll
            for (int q = 0; q < W; ++q) {
                atomicAdd(&acc0[row + col[q]], fixed64(ry[q] * wx[ka], rh[q] * wx[ka]));
                atomicAdd(&acc1[row + col[q]], fixed64(iy[q] * wx[ka], ih[q] * wx[ka]));
            }
        }
    }
    __syncthreads();
    const double inv_scale = ldexp(1.0, e - 61);
    float2 *G = d.G + ((int64_t)d.gslot_s[sb] * p + c) * p * p;
    for (int kk = threadIdx.x; kk < ncell; kk += kThreads) {
        const int al = kk / nb, bl = kk % nb;
        G[(int64_t)(a0 + al) * p + b0 + bl] = make_float2((float)((double)(long long)acc0[kk] * inv_scale),
                                                          (float)((double)(long long)acc1[kk] * inv_scale));
    }
}

// v_mfma_f32_16x16x4f32: A[i][k] from lane i + 16 k, B[k][j] from lane j + 16 k, D[4 (lane / 16) + r][lane % 16]
// in register r.  The four grid sums below are real products with the real and imaginary parts of each
// operand as separate rows or columns; LDS operand rows are padded (80 floats for 64 columns, 144 for 128) so
// that the four 16-lane groups of a wave, which read four consecutive rows, hit distinct banks.  Steps run in
// groups of four without per-step conditions, so that the LDS reads of a group are issued together.
__device__ __forceinline__ floatx4 mfma16(float a, float b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
constexpr int kRow64 = 80;
constexpr int kRow128 = 144;

// Global-memory views of device pointers: accesses through them compile to global instructions, which the
// LDS wait counter does not track (flat accesses are counted by both the memory and the LDS counters).
// Complex values are accessed as two-float vectors.
typedef float v2f __attribute__((ext_vector_type(2)));
using gc2 = const __attribute__((address_space(1))) v2f *;
using gm2 = __attribute__((address_space(1))) v2f *;
__device__ __forceinline__ gc2 gl(const float2 *p) { return (gc2)p; }
__device__ __forceinline__ gm2 gw(float2 *p) { return (gm2)p; }
using gcf = const __attribute__((address_space(1))) float *;
__device__ __forceinline__ gcf gfl(const float *p) { return (gcf)p; }
// Read-only views in the constant address space: wave-uniform loads through them are scalar loads.
using kc2 = const __attribute__((address_space(4))) v2f *;
__device__ __forceinline__ kc2 kcv(const float2 *p) { return (kc2)p; }

// Sums over z: C[(m, pe)][(ab, pg)] = sum_c Ez_pe[m][c] G_pg[c][ab]; H[m] = C_rr - C_ii + i (C_ri + C_ir) and
// H[L-m] = C_rr + C_ii + i (C_ri - C_ir) (rings m and L - m have conjugate z tables).  Block: 64 grid columns
// (16 per wave, held in registers) and a group of up to four 16-ring-pair blocks (grid_z_groups, their z
// tables staged through LDS); planes 64 at a time, MFMA step s and lane group g taking plane c0 + S g + s.
// Item (desc, box, column chunk, group).
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4)))
k_grid_z(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int sb = wk.y, p = d.gp, L = d.L, nrp = d.nrp, p2 = p * p;
    const int ab0 = wk.z * 64;
    int ngr, gsz;
    grid_z_groups(nrp, ngr, gsz);
    const int nmb = (nrp + 15) / 16, mb0 = wk.w * gsz, nmbg = min(gsz, nmb - mb0);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, li = lane & 15, lg = lane >> 4;
    __shared__ float As[64 * kRow128];       // [step s, group g][ring block, part, ring]
    floatx4 acc[4][2][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int k = 0; k < 2; ++k) acc[i][j][k] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int ab = ab0 + wv * 16 + li;
    const gc2 G = gl(d.G) + (int64_t)d.gslot_s[sb] * p * p2 + min(ab, p2 - 1);
    const gc2 Ez = gl(d.Ez);
    const float gkeep = ab < p2 ? 1.f : 0.f;
    for (int c0 = 0; c0 < p; c0 += 64) {
        const int nc = min(64, p - c0), S = nc / 4;
        float gr[16], gi[16];
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4)
            if (4 * s4 < S) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const v2f g = G[(int64_t)(c0 + S * lg + 4 * s4 + u) * p2];
                    gr[4 * s4 + u] = g.x * gkeep;
                    gi[4 * s4 + u] = g.y * gkeep;
                }
            }
        __syncthreads();
        for (int k = threadIdx.x; k < nc * 16 * nmbg; k += kThreads) {
            const int cl = k % nc, mr = k / nc, m = mb0 * 16 + mr;
            v2f e = {0.f, 0.f};
            if (m < nrp) e = Ez[(int64_t)m * p + c0 + cl];
            float *r = As + (4 * (cl % S) + cl / S) * kRow128 + (mr >> 4) * 32 + (mr & 15);
            r[0] = e.x;
            r[16] = e.y;
        }
        __syncthreads();
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) {
            if (mi < nmbg) {
#pragma unroll
                for (int s4 = 0; s4 < 4; ++s4)
                    if (4 * s4 < S) {
                        float er[4], ei[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const float *ar = As + (4 * (4 * s4 + u) + lg) * kRow128 + mi * 32 + li;
                            er[u] = ar[0];
                            ei[u] = ar[16];
                        }
                        __builtin_amdgcn_sched_barrier(0);   // the group's LDS reads are issued together
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int s = 4 * s4 + u;
                            acc[mi][0][0] = mfma16(er[u], gr[s], acc[mi][0][0]);
                            acc[mi][0][1] = mfma16(er[u], gi[s], acc[mi][0][1]);
                            acc[mi][1][0] = mfma16(ei[u], gr[s], acc[mi][1][0]);
                            acc[mi][1][1] = mfma16(ei[u], gi[s], acc[mi][1][1]);
                        }
                    }
            }
        }
    }
    if (ab >= p2) return;
    const gm2 H = gw(d.H);
    const int hslot = d.gslot_s[sb];
#pragma unroll
    for (int mi = 0; mi < 4; ++mi) {
        if (mi >= nmbg) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = (mb0 + mi) * 16 + 4 * lg + r;
            if (m >= nrp) continue;
            const float q1 = acc[mi][0][0][r], q3 = acc[mi][0][1][r], q4 = acc[mi][1][0][r], q2 = acc[mi][1][1][r];
            H[((int64_t)m * d.gnbox + hslot) * p2 + ab] = v2f{q1 - q2, q3 + q4};
            if (L - m != m) H[((int64_t)(L - m) * d.gnbox + hslot) * p2 + ab] = v2f{q1 + q2, q3 - q4};
        }
    }
}

// The MFMA steps of k_grid_phi: 4 S4 steps over the staged rows, NT column tiles, in groups of four steps
// whose LDS operands are read together before their products.
template <int S4, int NT>
__device__ __forceinline__ void phi_steps(const float *bl, const float (&hr)[16], const float (&hi)[16],
                                          floatx4 (&acc)[2][4]) {
#pragma unroll
    for (int g = 0; g < S4; ++g) {
        float bv[4][NT];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int t = 0; t < NT; ++t) bv[u][t] = bl[4 * (4 * g + u) * kRow64 + t * 16];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                acc[0][t] = mfma16(hr[4 * g + u], bv[u][t], acc[0][t]);
                acc[1][t] = mfma16(hi[4 * g + u], bv[u][t], acc[1][t]);
            }
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <int S4>
__device__ __forceinline__ void phi_steps_nt(int ntile, const float *bl, const float (&hr)[16], const float (&hi)[16],
                                             floatx4 (&acc)[2][4]) {
    switch (ntile) {
        case 1: phi_steps<S4, 1>(bl, hr, hi, acc); break;
        case 2: phi_steps<S4, 2>(bl, hr, hi, acc); break;
        case 3: phi_steps<S4, 3>(bl, hr, hi, acc); break;
        default: phi_steps<S4, 4>(bl, hr, hi, acc); break;
    }
}

// Sums over the plane to the directions of ring m: C[(a, pa)][(n, pe)] = sum_b H_pa[a][b] Ey_pe[b][n], whose
// four real products give z0 = C_rr + i C_ir and z1 = C_ri + i C_ii per (a, n); then u~(m, n) = sum_a Ex[a][n]
// (z0 + i z1) and u~(m, n + L) = sum_a conj(Ex[a][n]) (z0 - i z1) (azimuths n and n + L have conjugate
// in-plane tables).  Block: one ring of one box; waves take 16-row blocks of a (held in registers when the
// grid has at most 64 rows); azimuths in chunks of 32 (four column tiles of 8 azimuths, real parts in columns
// 0-7 and imaginary parts in 8-15), b staged through LDS 64 at a time (step s, lane group g: b = b0 + S g + s)
// with Ex beside it.  Each lane sums its four rows, the two parts are added across lanes, and the partial
// sums of the 16 row groups are added in order.  Item (desc, box, ring, 0).
__global__ void __launch_bounds__(kThreads)
k_grid_phi(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int sb = wk.y, m = wk.z;
    const int p = d.gp, L = d.L, mt = min(m, L - m);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, li = lane & 15, lg = lane >> 4;
    constexpr int kExRow = 68;               // 32 complex azimuths + pad, in floats
    __shared__ float Bs[64 * kRow64];
    __shared__ float Exs[64 * kExRow];
    __shared__ float4 red[4][4][32];         // [wave][lane group][azimuth]
    const gc2 H = gl(d.H) + ((int64_t)m * d.gnbox + d.gslot_s[sb]) * p * p;
    const gc2 Ey = gl(d.Ey) + (int64_t)mt * p * L;
    const gc2 Ex = gl(d.Ex) + (int64_t)mt * p * L;
    const int nab = p / 16, rounds = (nab + 3) / 4;
    const bool one = p <= 64;                // one round of row blocks and one chunk of b
    const gm2 ut = gw(reinterpret_cast<float2 *>(d.ut)) + (int64_t)sb * d.npair * 2;
    const int64_t twoL = 2 * (int64_t)L;
    float hr[16], hi[16];
    auto load_rows = [&](int blk, int b0, int S) {
        const gc2 hrow = H + (int64_t)(blk * 16 + li) * p + b0 + S * lg;
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4)
            if (4 * s4 < S) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const v2f h = hrow[4 * s4 + u];
                    hr[4 * s4 + u] = h.x;
                    hi[4 * s4 + u] = h.y;
                }
            }
    };
    if (one && wv < nab) load_rows(wv, 0, p / 4);
    const float *bl = Bs + lg * kRow64 + li;
    for (int n0 = 0; n0 < L; n0 += 32) {
        const int ntile = min(4, (L - n0 + 7) / 8);
        float4 tot[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) tot[t] = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int rd = 0; rd < rounds; ++rd) {
            const int blk = rd * 4 + wv;
            const bool act = blk < nab;
            floatx4 acc[2][4];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[i][t] = floatx4{0.f, 0.f, 0.f, 0.f};
            for (int b0 = 0; b0 < p; b0 += 64) {
                const int nb = min(64, p - b0), S = nb / 4;
                __syncthreads();
                {
                    // all loads of the chunk in flight at once: 8 per thread for Ey, 8 for Ex
                    const int nl = threadIdx.x % 32, n = n0 + nl, q0 = threadIdx.x / 32;
                    const int na = b0 == 0 ? min(64, p - rd * 64) : 0;
                    v2f ey[8], ex[8];
#pragma unroll
                    for (int it = 0; it < 8; ++it) {
                        const int q = q0 + 8 * it;
                        ey[it] = v2f{0.f, 0.f};
                        ex[it] = v2f{0.f, 0.f};
                        if (q < nb && n < L) ey[it] = Ey[(int64_t)(b0 + q) * L + n];
                        if (q < na && n < L) ex[it] = Ex[(int64_t)(rd * 64 + q) * L + n];
                    }
#pragma unroll
                    for (int it = 0; it < 8; ++it) {
                        const int q = q0 + 8 * it;
                        if (q < nb) {
                            float *r = Bs + (4 * (q % S) + q / S) * kRow64 + (nl >> 3) * 16 + (nl & 7);
                            r[0] = ey[it].x;
                            r[8] = ey[it].y;
                        }
                        if (q < na) reinterpret_cast<float2 *>(Exs + q * kExRow)[nl] = make_float2(ex[it].x, ex[it].y);
                    }
                }
                __syncthreads();
                if (act) {
                    if (!one) load_rows(blk, b0, S);
                    switch (S / 4) {
                        case 1: phi_steps_nt<1>(ntile, bl, hr, hi, acc); break;
                        case 2: phi_steps_nt<2>(ntile, bl, hr, hi, acc); break;
                        case 3: phi_steps_nt<3>(ntile, bl, hr, hi, acc); break;
                        default: phi_steps_nt<4>(ntile, bl, hr, hi, acc); break;
                    }
                }
            }
            if (act) {
                const bool im = li >= 8;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    if (t >= ntile) continue;
                    const int nl = 8 * t + (li & 7);
                    float fr = 0.f, fi = 0.f, gr = 0.f, gi = 0.f;   // sum Ex z, sum conj(Ex) z over this lane's rows
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float2 ex = reinterpret_cast<const float2 *>(Exs + (wv * 16 + 4 * lg + r) * kExRow)[nl];
                        const float x = acc[0][t][r], y = acc[1][t][r];
                        fr = fmaf(ex.x, x, fmaf(-ex.y, y, fr));
                        fi = fmaf(ex.x, y, fmaf(ex.y, x, fi));
                        gr = fmaf(ex.x, x, fmaf(ex.y, y, gr));
                        gi = fmaf(ex.x, y, fmaf(-ex.y, x, gi));
                    }
                    // the imaginary-part columns hold z1: contribute i F and -i G
                    float t0 = im ? -fi : fr, t1 = im ? fr : fi, t2 = im ? gi : gr, t3 = im ? -gr : gi;
                    t0 += __shfl_xor(t0, 8, 64);
                    t1 += __shfl_xor(t1, 8, 64);
                    t2 += __shfl_xor(t2, 8, 64);
                    t3 += __shfl_xor(t3, 8, 64);
                    tot[t].x += t0;
                    tot[t].y += t1;
                    tot[t].z += t2;
                    tot[t].w += t3;
                }
            }
        }
        if (li < 8) {
#pragma unroll
            for (int t = 0; t < 4; ++t) red[wv][lg][8 * t + li] = tot[t];
        }
        __syncthreads();
        const int nl = threadIdx.x, n = n0 + nl;
        if (nl < 32 && n < L) {
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
            for (int w = 0; w < min(4, nab); ++w)
                for (int g = 0; g < 4; ++g) {
                    const float4 b = red[w][g][nl];
                    a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
                }
            // a.xy = u~(m, n), a.zw = u~(m, n + L), into the antipodal-pair layout
            if (2 * m < L) {
                ut[(m * twoL + n) * 2] = v2f{a.x, a.y};
                ut[(m * twoL + n + L) * 2] = v2f{a.z, a.w};
            } else if (2 * m > L) {
                const int64_t m2 = L - m;
                ut[(m2 * twoL + n) * 2 + 1] = v2f{a.z, a.w};
                ut[(m2 * twoL + n + L) * 2 + 1] = v2f{a.x, a.y};
            } else {
                ut[(m * twoL + n) * 2] = v2f{a.x, a.y};
                ut[(m * twoL + n) * 2 + 1] = v2f{a.z, a.w};
            }
        }
    }
}

// The MFMA steps of k_grid_phi_r: 16 P16 steps over all staged rows (groups of four whose LDS operands are read
// together before their products), NT column tiles, the A operand (H rows) in registers.
template <int P16, int NT>
__device__ __forceinline__ void phi_steps_r(const float *bl, const float (&hr)[4 * P16], const float (&hi)[4 * P16],
                                            floatx4 (&acc)[2][4]) {
#pragma unroll
    for (int g = 0; g < P16; ++g) {
        float bv[4][NT];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int t = 0; t < NT; ++t) bv[u][t] = bl[4 * (4 * g + u) * kRow64 + t * 16];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                acc[0][t] = mfma16(hr[4 * g + u], bv[u][t], acc[0][t]);
                acc[1][t] = mfma16(hi[4 * g + u], bv[u][t], acc[1][t]);
            }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The sums of k_grid_phi for grids of P = 16 P16 nodes, 64 < P <= 128: rounds of four 16-row blocks of a on
// the outside, each wave's H rows over the whole of b loaded once per round into registers (4 P16 values per
// lane and part), and every chunk of 32 azimuths staged with all of Ey's P rows.  The partial sums of a round
// (over its rows, the two parts and the four lane groups, in that order) are added to u~ in round order by the
// thread that owns the azimuth.  Item (desc, box, ring, 0).
template <int P16>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2)))
k_grid_phi_r(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    constexpr int P = 16 * P16, S = 4 * P16;        // nodes; MFMA steps (b = S g + s for lane group g, step s)
    constexpr int kExRow = 68;                       // 32 complex azimuths + pad, in floats
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int sb = wk.y, m = wk.z;
    const int L = d.L, mt = min(m, L - m);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, li = lane & 15, lg = lane >> 4;
    __shared__ float Bs[P * kRow64];
    __shared__ float Exs[64 * kExRow];
    __shared__ float4 red[4][4][32];                 // [wave][lane group][azimuth]
    const gc2 H = gl(d.H) + ((int64_t)m * d.gnbox + d.gslot_s[sb]) * P * P;
    const gc2 Ey = gl(d.Ey) + (int64_t)mt * P * L;
    const gc2 Ex = gl(d.Ex) + (int64_t)mt * P * L;
    const gm2 ut = gw(reinterpret_cast<float2 *>(d.ut)) + (int64_t)sb * d.npair * 2;
    const int64_t twoL = 2 * (int64_t)L;
    const float *bl = Bs + lg * kRow64 + li;
    for (int rd = 0; rd < (P16 + 3) / 4; ++rd) {
        const int blk = rd * 4 + wv, nact = min(4, P16 - rd * 4), na = min(64, P - rd * 64);
        const bool act = blk < P16;
        float hr[S], hi[S];
        if (act) {
            const gc2 hrow = H + (int64_t)(blk * 16 + li) * P + S * lg;
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const v2f h = hrow[s];
                hr[s] = h.x;
                hi[s] = h.y;
            }
        }
        for (int n0 = 0; n0 < L; n0 += 32) {
            const int ntile = min(4, (L - n0 + 7) / 8);
            __syncthreads();
            {
                // Ey rows q < P and Ex rows q < na of this round, azimuth n0 + nl; loads in flight together
                const int nl = threadIdx.x % 32, n = n0 + nl, q0 = threadIdx.x / 32;
                v2f ey[P / 8], ex[8];
#pragma unroll
                for (int it = 0; it < P / 8; ++it) {
                    const int q = q0 + 8 * it;
                    ey[it] = n < L ? Ey[(int64_t)q * L + n] : v2f{0.f, 0.f};
                }
#pragma unroll
                for (int it = 0; it < 8; ++it) {
                    const int q = q0 + 8 * it;
                    ex[it] = (q < na && n < L) ? Ex[(int64_t)(rd * 64 + q) * L + n] : v2f{0.f, 0.f};
                }
#pragma unroll
                for (int it = 0; it < P / 8; ++it) {
                    const int q = q0 + 8 * it;
                    float *r = Bs + (4 * (q % S) + q / S) * kRow64 + (nl >> 3) * 16 + (nl & 7);
                    r[0] = ey[it].x;
                    r[8] = ey[it].y;
                }
#pragma unroll
                for (int it = 0; it < 8; ++it)
                    reinterpret_cast<float2 *>(Exs + (q0 + 8 * it) * kExRow)[nl] = make_float2(ex[it].x, ex[it].y);
            }
            __syncthreads();
            float4 tot[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) tot[t] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (act) {
                floatx4 acc[2][4];
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int t = 0; t < 4; ++t) acc[i][t] = floatx4{0.f, 0.f, 0.f, 0.f};
                switch (ntile) {
                    case 1: phi_steps_r<P16, 1>(bl, hr, hi, acc); break;
                    case 2: phi_steps_r<P16, 2>(bl, hr, hi, acc); break;
                    case 3: phi_steps_r<P16, 3>(bl, hr, hi, acc); break;
                    default: phi_steps_r<P16, 4>(bl, hr, hi, acc); break;
                }
                const bool im = li >= 8;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    if (t >= ntile) continue;
                    const int nl = 8 * t + (li & 7);
                    float fr = 0.f, fi = 0.f, gr = 0.f, gi = 0.f;   // sum Ex z, sum conj(Ex) z over this lane's rows
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float2 ex = reinterpret_cast<const float2 *>(Exs + (wv * 16 + 4 * lg + r) * kExRow)[nl];
                        const float x = acc[0][t][r], y = acc[1][t][r];
                        fr = fmaf(ex.x, x, fmaf(-ex.y, y, fr));
                        fi = fmaf(ex.x, y, fmaf(ex.y, x, fi));
                        gr = fmaf(ex.x, x, fmaf(ex.y, y, gr));
                        gi = fmaf(ex.x, y, fmaf(-ex.y, x, gi));
                    }
                    // the imaginary-part columns hold z1: contribute i F and -i G
                    float t0 = im ? -fi : fr, t1 = im ? fr : fi, t2 = im ? gi : gr, t3 = im ? -gr : gi;
                    t0 += __shfl_xor(t0, 8, 64);
                    t1 += __shfl_xor(t1, 8, 64);
                    t2 += __shfl_xor(t2, 8, 64);
                    t3 += __shfl_xor(t3, 8, 64);
                    tot[t] = make_float4(t0, t1, t2, t3);
                }
            }
            if (li < 8) {
#pragma unroll
                for (int t = 0; t < 4; ++t) red[wv][lg][8 * t + li] = tot[t];
            }
            __syncthreads();
            const int nl = threadIdx.x, n = n0 + nl;
            if (nl < 32 && n < L) {
                float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
                for (int w = 0; w < nact; ++w)
                    for (int g = 0; g < 4; ++g) {
                        const float4 b = red[w][g][nl];
                        a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
                    }
                // a.xy: u~(m, n), a.zw: u~(m, n + L), added to the earlier rounds' sums in the antipodal-pair layout
                int64_t i1, i2;
                if (2 * m < L) {
                    i1 = (m * twoL + n) * 2;
                    i2 = (m * twoL + n + L) * 2;
                } else if (2 * m > L) {
                    const int64_t m2 = L - m;
                    i1 = (m2 * twoL + n + L) * 2 + 1;
                    i2 = (m2 * twoL + n) * 2 + 1;
                } else {
                    i1 = (m * twoL + n) * 2;
                    i2 = (m * twoL + n) * 2 + 1;
                }
                if (rd > 0) {
                    const v2f o1 = ut[i1], o2 = ut[i2];
                    a.x = o1.x + a.x;
                    a.y = o1.y + a.y;
                    a.z = o2.x + a.z;
                    a.w = o2.y + a.w;
                }
                ut[i1] = v2f{a.x, a.y};
                ut[i2] = v2f{a.z, a.w};
            }
        }
    }
}

// Sums over the plane to the directions for grids of P = 16 P16 <= 64 nodes per axis: the products of
// k_grid_phi with H staged once in LDS as the A operand ([b][a block, part, a % 16], b = 4 s + g for step s and
// lane group g); each wave then runs on its own over its 8-azimuth column tiles (tiles w, w + 4, ...): the Ey
// values a lane needs come from memory straight into registers one tile ahead, Ex goes through a
// wave-private LDS slice, and the sums over a are completed inside the wave (its 4 rows per lane, then across
// the two parts and the four lane groups).  Steps go in groups of two (their LDS reads issued together), and
// the kernel keeps to 53 KB of LDS and the registers of three waves per SIMD, so that three blocks share a CU
// (64 nodes: 0.58 -> 0.53 ms on the 1M-point sphere's level 2 against groups of four steps at two blocks per
// CU).  Item (desc, box, ring, 0).
template <int P16>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3)))
k_grid_phi_s(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    constexpr int P = 16 * P16, S = 4 * P16, NX = P / 8;   // nodes, MFMA steps, Ex values per lane and tile
    constexpr int kExR = 16;                                // floats per Ex row: 8 complex azimuths
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int sb = wk.y, m = wk.z, L = d.L, mt = min(m, L - m);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, li = lane & 15, lg = lane >> 4;
    __shared__ float As[P * kRow128];
    __shared__ float Exw[4][P * kExR];
    {
        const gc2 H = gl(d.H) + ((int64_t)m * d.gnbox + d.gslot_s[sb]) * P * P;
        v2f hv[P16 * P16];
#pragma unroll
        for (int it = 0; it < P16 * P16; ++it) hv[it] = H[threadIdx.x + it * kThreads];
#pragma unroll
        for (int it = 0; it < P16 * P16; ++it) {
            const int idx = threadIdx.x + it * kThreads, a = idx / P, b = idx % P;
            float *r = As + b * kRow128 + (a >> 4) * 32 + (a & 15);
            r[0] = hv[it].x;
            r[16] = hv[it].y;
        }
    }
    __syncthreads();
    using gcf = const __attribute__((address_space(1))) float *;
    const gcf Eyf = (gcf)(d.Ey + (int64_t)mt * P * L);
    const gc2 Ex = gl(d.Ex) + (int64_t)mt * P * L;
    const int pe = li >> 3, ntiles = (L + 7) / 8;
    float *exw = Exw[wv];
    const gm2 ut = gw(reinterpret_cast<float2 *>(d.ut)) + (int64_t)sb * d.npair * 2;
    const int64_t twoL = 2 * (int64_t)L;
    float bnx[S];
    v2f xnx[NX];
    auto prefetch = [&](int t) {
        const int n = 8 * t + (li & 7);
        const bool ok = n < L;
        const int nc = ok ? n : 0;
#pragma unroll
        for (int s = 0; s < S; ++s) bnx[s] = ok ? Eyf[2 * ((int64_t)(4 * s + lg) * L + nc) + pe] : 0.f;
        const int nx = 8 * t + (lane & 7);
        const bool okx = nx < L;
#pragma unroll
        for (int j = 0; j < NX; ++j) xnx[j] = okx ? Ex[(int64_t)(lane / 8 + 8 * j) * L + nx] : v2f{0.f, 0.f};
    };
    if (wv < ntiles) prefetch(wv);
    for (int t = wv; t < ntiles; t += 4) {
        float bv[S];
#pragma unroll
        for (int s = 0; s < S; ++s) bv[s] = bnx[s];
#pragma unroll
        for (int j = 0; j < NX; ++j)
            reinterpret_cast<float2 *>(exw + (lane / 8 + 8 * j) * kExR)[lane & 7] = make_float2(xnx[j].x, xnx[j].y);
        if (t + 4 < ntiles) prefetch(t + 4);
        floatx4 acc[P16][2];
#pragma unroll
        for (int q = 0; q < P16; ++q) acc[q][0] = acc[q][1] = floatx4{0.f, 0.f, 0.f, 0.f};
        const float *al = As + lg * kRow128 + li;
#pragma unroll
        for (int g = 0; g < 2 * P16; ++g) {
            float av[2][P16][2];
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int q = 0; q < P16; ++q) {
                    av[u][q][0] = al[4 * (2 * g + u) * kRow128 + q * 32];
                    av[u][q][1] = al[4 * (2 * g + u) * kRow128 + q * 32 + 16];
                }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int q = 0; q < P16; ++q) {
                    acc[q][0] = mfma16(av[u][q][0], bv[2 * g + u], acc[q][0]);
                    acc[q][1] = mfma16(av[u][q][1], bv[2 * g + u], acc[q][1]);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        // sums over this lane's rows: F = sum Ex z, G = sum conj(Ex) z, z = (row of H_r, row of H_i) products
        float fr = 0.f, fi = 0.f, gr = 0.f, gi = 0.f;
#pragma unroll
        for (int q = 0; q < P16; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float2 ex = reinterpret_cast<const float2 *>(exw + (q * 16 + 4 * lg + r) * kExR)[li & 7];
                const float x = acc[q][0][r], y = acc[q][1][r];
                fr = fmaf(ex.x, x, fmaf(-ex.y, y, fr));
                fi = fmaf(ex.x, y, fmaf(ex.y, x, fi));
                gr = fmaf(ex.x, x, fmaf(ex.y, y, gr));
                gi = fmaf(ex.x, y, fmaf(-ex.y, x, gi));
            }
        // the imaginary-part columns hold z1: contribute i F and -i G
        float t0 = pe ? -fi : fr, t1 = pe ? fr : fi, t2 = pe ? gi : gr, t3 = pe ? -gr : gi;
#pragma unroll
        for (int o = 8; o < 64; o <<= 1) {
            t0 += __shfl_xor(t0, o, 64);
            t1 += __shfl_xor(t1, o, 64);
            t2 += __shfl_xor(t2, o, 64);
            t3 += __shfl_xor(t3, o, 64);
        }
        const int n = 8 * t + li;
        if (lane < 8 && n < L) {
            // (t0, t1) = u~(m, n), (t2, t3) = u~(m, n + L), into the antipodal-pair layout
            if (2 * m < L) {
                ut[(m * twoL + n) * 2] = v2f{t0, t1};
                ut[(m * twoL + n + L) * 2] = v2f{t2, t3};
            } else if (2 * m > L) {
                const int64_t m2 = L - m;
                ut[(m2 * twoL + n) * 2 + 1] = v2f{t2, t3};
                ut[(m2 * twoL + n + L) * 2 + 1] = v2f{t0, t1};
            } else {
                ut[(m * twoL + n) * 2] = v2f{t0, t1};
                ut[(m * twoL + n) * 2 + 1] = v2f{t2, t3};
            }
        }
    }
}

// The products of steps s_lo .. s_hi - 1 of one staged chunk of k_grid_phit for the 16-row block ab of a: QN
// column tiles of 16, in groups of four steps where the range allows (a group's LDS reads are all issued before
// its products; rows past the staged azimuths of a partial chunk are zero), with no conditions inside a step.
template <int QN, int RB, int QB>
__device__ __forceinline__ void phit_mma(const float *Ar, const float *Ai, const float *Bs, int ab, int li, int lg,
                                         int s_lo, int s_hi, floatx4 (&acc)[2][QB]) {
    int s0 = s_lo;
#pragma unroll 1
    for (; s0 + 4 <= s_hi; s0 += 4) {
        float ar[4], ai[4], bv[4][QN];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int row = (4 * (s0 + u) + lg) * kRow64;
            ar[u] = Ar[row + ab * 16 + li];
            ai[u] = Ai[row + ab * 16 + li];
#pragma unroll
            for (int q = 0; q < QN; ++q) bv[u][q] = Bs[(4 * (s0 + u) + lg) * RB + q * 16 + li];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int q = 0; q < QN; ++q) {
                acc[0][q] = mfma16(ar[u], bv[u][q], acc[0][q]);
                acc[1][q] = mfma16(ai[u], bv[u][q], acc[1][q]);
            }
    }
    {
        for (int s = s0; s < s_hi; ++s) {
            const int row = (4 * s + lg) * kRow64;
            const float ar = Ar[row + ab * 16 + li], ai = Ai[row + ab * 16 + li];
            float bv[QN];
#pragma unroll
            for (int q = 0; q < QN; ++q) bv[q] = Bs[(4 * s + lg) * RB + q * 16 + li];
#pragma unroll
            for (int q = 0; q < QN; ++q) {
                acc[0][q] = mfma16(ar, bv[q], acc[0][q]);
                acc[1][q] = mfma16(ai, bv[q], acc[1][q]);
            }
        }
    }
}

// v~ of ring m back to its plane: H'_pa[a][b] = sum over (n, pe) of A[(a, pa)][(n, pe)] E_pe[b][n] with
// A = (S_r, -D_i | S_i, D_r), S = conj(Ex) v~(n) + Ex v~(n + L), D = Ex v~(n + L) - conj(Ex) v~(n).  Block: one
// ring and a 64 x 64 tile of the plane; waves take 16-row blocks of a and all four 16-column blocks of b;
// azimuths staged through LDS 16 at a time from the transposed tables ([n][node]), step s and lane group g
// taking azimuth 2 s + g / 2 and part g % 2.  Where the tile has only one or two 16-row blocks of a (grids of
// 16 or 32 nodes, edge tiles), the otherwise idle waves take a share of each chunk's steps, and their partial
// sums are added to the first share's through LDS, in the order of the shares.  The next chunk's table values
// and v~ are loaded into registers while the current chunk's products run.  Grids of 80, 96 and 112 nodes take
// tiles of 64 rows of a by the whole of b (k_grid_phit_wide: up to eight 16-column blocks per wave), so that
// no tile is a sliver and each chunk's A operand is staged once per 64 rows.  Item (desc, box, ring, tile).
template <int BW>
__device__ __forceinline__ void grid_phit_body(const int4 wk, const LDesc &d) {
    constexpr int QB = BW / 16;                              // column blocks of 16 in a tile
    constexpr int RB = BW == 64 ? kRow64 : kRow128;          // floats per staged row of B
    constexpr int kStage = 2 * 32 * kRow64 + 32 * RB;        // A (two parts) and B
    constexpr int kRed = 3 * 2 * QB * 4 * 64;                // at most three shares of partial sums
    const int tb = wk.y, m = wk.z;
    const int p = d.gp, L = d.L, mt = min(m, L - m);
    const int nta = (p + 63) / 64;
    const int a0 = BW == 64 ? (wk.w / nta) * 64 : wk.w * 64, b0 = BW == 64 ? (wk.w % nta) * 64 : 0;
    const int qn = min(QB, (p - b0 + 15) / 16);   // column tiles of 16 inside the grid
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, li = lane & 15, lg = lane >> 4;
    __shared__ float lds[kStage > kRed ? kStage : kRed];
    float *const Ar = lds, *const Ai = lds + 32 * kRow64, *const Bs = lds + 2 * 32 * kRow64;
    floatx4 acc[2][QB];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int q = 0; q < QB; ++q) acc[i][q] = floatx4{0.f, 0.f, 0.f, 0.f};
    // row blocks of a in the tile, shares of the steps, this wave's row block and share
    const int nab = min(4, (p - a0 + 15) / 16);
    const int ks = nab == 1 ? 4 : (nab == 2 ? 2 : 1);
    const int ab = wv % nab, kp = wv / nab;
    const bool act = kp < ks;
    constexpr int kStepsPerChunk = 8;
    const int64_t twoL = 2 * (int64_t)L;
    const gc2 ExT = gl(d.ExT) + (int64_t)mt * L * p, EyT = gl(d.EyT) + (int64_t)mt * L * p;
    // v~(m, n) and v~(m, n + L) in the antipodal-pair layout
    int64_t o1, o2, dn;   // v1 at vt[o1 + dn n], v2 at vt[o2 + dn n]
    if (2 * m < L) {
        o1 = (int64_t)m * twoL * 2;
        o2 = ((int64_t)m * twoL + L) * 2;
    } else if (2 * m > L) {
        o1 = ((int64_t)(L - m) * twoL + L) * 2 + 1;
        o2 = (int64_t)(L - m) * twoL * 2 + 1;
    } else {
        o1 = (int64_t)m * twoL * 2;
        o2 = (int64_t)m * twoL * 2 + 1;
    }
    dn = 2;
    const int x = threadIdx.x % 64, nq = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    // v~ depends on the azimuth only, one per wave and step: scalar loads into scalar registers
    const kc2 vts = kcv(reinterpret_cast<const float2 *>(d.vt)) + (int64_t)tb * d.npair * 2;
    v2f exv[4], eyv[4], eyw[4], v1v[4], v2v[4];   // eyw: columns 64 .. 127 of wide tiles
    auto fetch = [&](int n0) {
        const int cnt = min(16, L - n0);
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int nl = nq + 4 * it, n = n0 + nl;
            const bool ok = nl < cnt;
            exv[it] = eyv[it] = eyw[it] = v1v[it] = v2v[it] = v2f{0.f, 0.f};
            if (ok) {
                v1v[it] = vts[o1 + dn * n];
                v2v[it] = vts[o2 + dn * n];
            }
            if (ok && a0 + x < p) exv[it] = ExT[(int64_t)n * p + a0 + x];
            if (ok && b0 + x < p) eyv[it] = EyT[(int64_t)n * p + b0 + x];
            if (BW > 64 && ok && b0 + 64 + x < p) eyw[it] = EyT[(int64_t)n * p + b0 + 64 + x];
        }
    };
    fetch(0);
    for (int n0 = 0; n0 < L; n0 += 16) {
        const int cnt = min(16, L - n0);
        __syncthreads();
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int nl = nq + 4 * it;
            const v2f ex = exv[it], v1 = v1v[it], v2 = v2v[it];
            const float y1r = fmaf(ex.x, v1.x, ex.y * v1.y), y1i = fmaf(ex.x, v1.y, -(ex.y * v1.x));   // conj(ex) v1
            const float y2r = fmaf(ex.x, v2.x, -(ex.y * v2.y)), y2i = fmaf(ex.x, v2.y, ex.y * v2.x);   // ex v2
            Ar[(2 * nl) * kRow64 + x] = y1r + y2r;          // S_r
            Ar[(2 * nl + 1) * kRow64 + x] = y1i - y2i;      // -D_i
            Ai[(2 * nl) * kRow64 + x] = y1i + y2i;          // S_i
            Ai[(2 * nl + 1) * kRow64 + x] = y2r - y1r;      // D_r
            Bs[(2 * nl) * RB + x] = eyv[it].x;
            Bs[(2 * nl + 1) * RB + x] = eyv[it].y;
            if (BW > 64) {
                Bs[(2 * nl) * RB + 64 + x] = eyw[it].x;
                Bs[(2 * nl + 1) * RB + 64 + x] = eyw[it].y;
            }
        }
        if (n0 + 16 < L) fetch(n0 + 16);
        __syncthreads();
        if (act) {
            // branch-free bodies for the common shapes, so that the LDS reads of later steps are issued
            // ahead of the products (rows past the chunk hold zeros in the partial last chunk)
            const int steps = (2 * cnt + 3) / 4;
            const int s_lo = kp * (kStepsPerChunk / ks), s_hi = min(steps, s_lo + kStepsPerChunk / ks);
            if (BW == 64) {
                switch (qn) {
                    case 4: phit_mma<4, RB, QB>(Ar, Ai, Bs, ab, li, lg, s_lo, s_hi, acc); break;
                    case 3: phit_mma<3, RB, QB>(Ar, Ai, Bs, ab, li, lg, s_lo, s_hi, acc); break;
                    case 2: phit_mma<2, RB, QB>(Ar, Ai, Bs, ab, li, lg, s_lo, s_hi, acc); break;
                    default: phit_mma<1, RB, QB>(Ar, Ai, Bs, ab, li, lg, s_lo, s_hi, acc); break;
                }
            } else {
                switch (qn) {   // wide tiles cover grids of 80 .. 128 nodes: 5 .. 8 column blocks
                    case 8: phit_mma<(QB < 8 ? QB : 8), RB, QB>(Ar, Ai, Bs, ab, li, lg, s_lo, s_hi, acc); break;
                    case 7: phit_mma<(QB < 7 ? QB : 7), RB, QB>(Ar, Ai, Bs, ab, li, lg, s_lo, s_hi, acc); break;
                    case 6: phit_mma<(QB < 6 ? QB : 6), RB, QB>(Ar, Ai, Bs, ab, li, lg, s_lo, s_hi, acc); break;
                    default: phit_mma<(QB < 5 ? QB : 5), RB, QB>(Ar, Ai, Bs, ab, li, lg, s_lo, s_hi, acc); break;
                }
            }
        }
    }
    if (ks > 1) {
        // shares 1 .. ks-1 through LDS (8 QB floats per lane and share: [part][column tile][row]), added to share
        // 0 in share order; (ks - 1) nab <= 3 shares, within the array
        constexpr int kShare = 2 * QB * 4 * 64;
        __syncthreads();
        if (act && kp > 0) {
            float *red = lds + ((kp - 1) * nab + ab) * kShare + lane;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int q = 0; q < QB; ++q)
#pragma unroll
                    for (int r = 0; r < 4; ++r) red[((i * QB + q) * 4 + r) * 64] = acc[i][q][r];
        }
        __syncthreads();
        if (act && kp == 0)
            for (int k = 1; k < ks; ++k) {
                const float *red = lds + ((k - 1) * nab + ab) * kShare + lane;
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int q = 0; q < QB; ++q)
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[i][q][r] += red[((i * QB + q) * 4 + r) * 64];
            }
    }
    if (!act || kp > 0) return;
    const gm2 Hb = gw(d.H) + ((int64_t)m * d.gnbox + d.gslot_t[tb]) * p * p;
#pragma unroll
    for (int q = 0; q < QB; ++q) {
        const int b = b0 + q * 16 + li;
        if (b >= p) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int a = a0 + ab * 16 + 4 * lg + r;
            Hb[(int64_t)a * p + b] = v2f{acc[0][q][r], acc[1][q][r]};
        }
    }
}

// The mirror plane sums for grids of at most 32 nodes, rings m and L - m together (they share the tables ExT and
// EyT; only v~ differs): the staged A operand holds both rings' 32 rows of a side by side (64 columns), B the
// shared 32 columns of Ey, and wave w takes ring w / 2 and row block w % 2, so every wave has two full column
// blocks of products.  Item (desc, box, ring m <= L / 2, 0).
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4)))
k_grid_phit_pair(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int tb = wk.y, m = wk.z;
    const int p = d.gp, L = d.L;                   // p <= 32, m <= L - m
    const int mr[2] = {m, L - m};
    const bool two = L - m != m;
    const int qn = (p + 15) / 16;                  // column blocks of b (1 or 2)
    const int nab = (p + 15) / 16;                 // row blocks of a per ring
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, li = lane & 15, lg = lane >> 4;
    const int rr = wv >> 1, ab = wv & 1;
    const bool act = ab < nab && (rr == 0 || two);
    __shared__ float Ar[32 * kRow64], Ai[32 * kRow64], Bs[32 * kRow64];
    floatx4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int q = 0; q < 2; ++q) acc[i][q] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int64_t twoL = 2 * (int64_t)L;
    const gc2 ExT = gl(d.ExT) + (int64_t)m * L * p, EyT = gl(d.EyT) + (int64_t)m * L * p;
    // v~(m', n) and v~(m', n + L) of both rings in the antipodal-pair layout: v1 at vt[o1 + 2 n], v2 at vt[o2 + 2 n]
    int64_t o1[2], o2[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int mm = mr[k];
        if (2 * mm < L) {
            o1[k] = (int64_t)mm * twoL * 2;
            o2[k] = ((int64_t)mm * twoL + L) * 2;
        } else if (2 * mm > L) {
            o1[k] = ((int64_t)(L - mm) * twoL + L) * 2 + 1;
            o2[k] = (int64_t)(L - mm) * twoL * 2 + 1;
        } else {
            o1[k] = (int64_t)mm * twoL * 2;
            o2[k] = (int64_t)mm * twoL * 2 + 1;
        }
    }
    // staging thread: column x of A is ring x / 32, row a = x % 32; columns x < 32 of B are b = x
    const int x = threadIdx.x % 64, xr = x >> 5, xa = x & 31, nq = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const kc2 vts = kcv(reinterpret_cast<const float2 *>(d.vt)) + (int64_t)tb * d.npair * 2;
    v2f exv[4], eyv[4], v1v[4], v2v[4];
    auto fetch = [&](int n0) {
        const int cnt = min(16, L - n0);
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int nl = nq + 4 * it, n = n0 + nl;
            const bool ok = nl < cnt;
            exv[it] = eyv[it] = v1v[it] = v2v[it] = v2f{0.f, 0.f};
            if (ok) {
                // both rings' values by scalar loads, each lane keeping its own ring's
                const v2f a1 = vts[o1[0] + 2 * n], a2 = vts[o2[0] + 2 * n];
                v2f b1 = a1, b2 = a2;
                if (two) {
                    b1 = vts[o1[1] + 2 * n];
                    b2 = vts[o2[1] + 2 * n];
                }
                v1v[it] = xr ? b1 : a1;
                v2v[it] = xr ? b2 : a2;
            }
            if (ok && xa < p) exv[it] = ExT[(int64_t)n * p + xa];
            if (ok && x < p) eyv[it] = EyT[(int64_t)n * p + x];
        }
    };
    fetch(0);
    for (int n0 = 0; n0 < L; n0 += 16) {
        const int cnt = min(16, L - n0);
        __syncthreads();
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int nl = nq + 4 * it;
            const v2f ex = exv[it], v1 = v1v[it], v2 = v2v[it];
            const float y1r = fmaf(ex.x, v1.x, ex.y * v1.y), y1i = fmaf(ex.x, v1.y, -(ex.y * v1.x));   // conj(ex) v1
            const float y2r = fmaf(ex.x, v2.x, -(ex.y * v2.y)), y2i = fmaf(ex.x, v2.y, ex.y * v2.x);   // ex v2
            Ar[(2 * nl) * kRow64 + x] = y1r + y2r;          // S_r
            Ar[(2 * nl + 1) * kRow64 + x] = y1i - y2i;      // -D_i
            Ai[(2 * nl) * kRow64 + x] = y1i + y2i;          // S_i
            Ai[(2 * nl + 1) * kRow64 + x] = y2r - y1r;      // D_r
            Bs[(2 * nl) * kRow64 + x] = eyv[it].x;
            Bs[(2 * nl + 1) * kRow64 + x] = eyv[it].y;
        }
        if (n0 + 16 < L) fetch(n0 + 16);
        __syncthreads();
        if (act) {
            const int steps = (2 * cnt + 3) / 4;
            // A's row block for this wave: ring rr's rows start at column 32 rr
            if (qn == 2)
                phit_mma<2, kRow64, 2>(Ar, Ai, Bs, 2 * rr + ab, li, lg, 0, steps, acc);
            else
                phit_mma<1, kRow64, 2>(Ar, Ai, Bs, 2 * rr + ab, li, lg, 0, steps, acc);
        }
    }
    if (!act) return;
    const gm2 Hb = gw(d.H) + ((int64_t)mr[rr] * d.gnbox + d.gslot_t[tb]) * p * p;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int b = q * 16 + li;
        if (q >= qn || b >= p) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int a = ab * 16 + 4 * lg + r;
            Hb[(int64_t)a * p + b] = v2f{acc[0][q][r], acc[1][q][r]};
        }
    }
}

__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4)))
k_grid_phit(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    grid_phit_body<64>(wk, descs[wk.x]);
}

__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2)))
k_grid_phit_wide(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    grid_phit_body<128>(wk, descs[wk.x]);
}

// Back over z: G'_pg[c][ab] = sum over (ring pair m, part pe) of A[c][(m, pe)] B[(m, pe)][(ab, pg)] with
// A = (Re Ez, Im Ez) and B = (S_r, S_i | -D_i, D_r), S = H'[m] + H'[L-m], D = H'[L-m] - H'[m].  Block: 64 grid
// columns and 64 planes (16 per wave); ring pairs staged through LDS 16 at a time, step s and lane group g
// taking ring pair 2 s + g / 2 and part g % 2.  Item (desc, box, column chunk, plane chunk).
__global__ void __launch_bounds__(kThreads)
k_grid_zt(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int tb = wk.y, p = d.gp, L = d.L, nrp = d.nrp, p2 = p * p;
    const int ab0 = wk.z * 64, c0 = wk.w * 64;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, li = lane & 15, lg = lane >> 4;
    __shared__ float As[32 * kRow64];
    __shared__ float Bs[32 * kRow128];
    floatx4 acc[4][2];
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q][0] = acc[q][1] = floatx4{0.f, 0.f, 0.f, 0.f};
    const bool act = c0 + wv * 16 < p;
    const gc2 H = gl(d.H), Ez = gl(d.Ez);
    const int hslot = d.gslot_t[tb];
    for (int mp0 = 0; mp0 < nrp; mp0 += 16) {
        const int mc = min(16, nrp - mp0);
        __syncthreads();
        {
            const int x = threadIdx.x % 64, mq = threadIdx.x / 64, ab = ab0 + x;
            v2f ev[4], h1v[4], h2v[4];
#pragma unroll
            for (int it = 0; it < 4; ++it) {     // all loads of the chunk in flight at once
                const int ml = mq + 4 * it, mp = mp0 + ml, m2 = L - mp;
                ev[it] = h1v[it] = h2v[it] = v2f{0.f, 0.f};
                if (ml < mc) {
                    if (c0 + x < p) ev[it] = Ez[(int64_t)mp * p + c0 + x];
                    if (ab < p2) {
                        h1v[it] = H[((int64_t)mp * d.gnbox + hslot) * p2 + ab];
                        if (m2 != mp) h2v[it] = H[((int64_t)m2 * d.gnbox + hslot) * p2 + ab];
                    }
                }
            }
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int ml = mq + 4 * it;
                const v2f h1 = h1v[it], h2 = h2v[it];
                const float Sx = h1.x + h2.x, Sy = h1.y + h2.y, Dx = h2.x - h1.x, Dy = h2.y - h1.y;
                As[(2 * ml) * kRow64 + x] = ev[it].x;
                As[(2 * ml + 1) * kRow64 + x] = ev[it].y;
                float *r0 = Bs + (2 * ml) * kRow128 + (x >> 4) * 32 + (x & 15);
                float *r1 = r0 + kRow128;
                r0[0] = Sx;
                r0[16] = Sy;
                r1[0] = -Dy;
                r1[16] = Dx;
            }
        }
        __syncthreads();
        if (act) {
            const int steps = (2 * mc + 3) / 4;
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                if (4 * g >= steps) break;
                float av[4], bv[4][8];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int s = 4 * g + u;
                    av[u] = As[(4 * s + lg) * kRow64 + wv * 16 + li];
                    const float *br = Bs + (4 * s + lg) * kRow128 + li;
#pragma unroll
                    for (int q = 0; q < 8; ++q) bv[u][q] = br[q * 16];
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        acc[q][0] = mfma16(av[u], bv[u][2 * q], acc[q][0]);
                        acc[q][1] = mfma16(av[u], bv[u][2 * q + 1], acc[q][1]);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    if (!act) return;
    const gm2 G = gw(d.G) + (int64_t)hslot * p * p2;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int ab = ab0 + q * 16 + li;
        if (ab >= p2) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int c = c0 + wv * 16 + 4 * lg + r;
            if (c < p) G[(int64_t)c * p2 + ab] = v2f{acc[q][0][r], acc[q][1][r]};
        }
    }
}

// v_i += sum over the W^3 grid nodes around x_i of phi phi phi G'.  Item (desc, target box, first point).
template <int W>
__global__ void __launch_bounds__(kThreads)
k_grid_interp(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int t = wk.y;
    const int i = wk.z + threadIdx.x;
    if (i >= d.tstart[t + 1]) return;
    const int p = d.gp;
    constexpr float hw = 0.5f * W, k1 = 2.f / W;
    const float half = 0.5f * (float)(p - 1), k2 = d.gbeta * 1.44269504f;
    const double ih = d.ginv_h;
    const float xg = (float)((d.txs[i] - d.tctr[3 * t]) * ih) + half;
    const float yg = (float)((d.tys[i] - d.tctr[3 * t + 1]) * ih) + half;
    const float zg = (float)((d.tzs[i] - d.tctr[3 * t + 2]) * ih) + half;
    const int alo = min(max((int)floorf(xg - hw) + 1, 0), p - W);
    const int blo = min(max((int)floorf(yg - hw) + 1, 0), p - W);
    const int clo = min(max((int)floorf(zg - hw) + 1, 0), p - W);
    float wx[W], wy[W], wz[W];
#pragma unroll
    for (int k = 0; k < W; ++k) {
        wx[k] = es_phi((float)(alo + k) - xg, k1, k2);
        wy[k] = es_phi((float)(blo + k) - yg, k1, k2);
        wz[k] = es_phi((float)(clo + k) - zg, k1, k2);
    }
    const gc2 G = gl(d.G) + (int64_t)d.gslot_t[t] * p * p * p + ((int64_t)clo * p + alo) * p + blo;
    float sr = 0.f, si = 0.f;
#pragma unroll
    for (int kc = 0; kc < W; ++kc) {
        float pr = 0.f, pi = 0.f;
#pragma unroll
        for (int ka = 0; ka < W; ++ka) {
            const gc2 row = G + ((int64_t)kc * p + ka) * p;
            float rr = 0.f, ri = 0.f;
#pragma unroll
            for (int q = 0; q < W; ++q) {
                const v2f g = row[q];
                rr = fmaf(wy[q], g.x, rr);
                ri = fmaf(wy[q], g.y, ri);
            }
            pr = fmaf(wx[ka], rr, pr);
            pi = fmaf(wx[ka], ri, pi);
        }
        sr = fmaf(wz[kc], pr, sr);
        si = fmaf(wz[kc], pi, si);
    }
    float2 o = d.v[i];
    o.x += sr;
    o.y += si;
    d.v[i] = o;
}

// ------------------------------------------------------------------ Lagrange levels
constexpr int kMaxR1 = 8;

// Orders a wave's LDS writes before its own later reads (and its reads before later writes): a wave's LDS
// operations complete in order, so only the compiler has to keep them in place.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One-dimensional Lagrange polynomials on the Chebyshev nodes at t (denominators precomputed).
__device__ __forceinline__ void lagrange_1d(float t, int r1, const float *nodes, const float *inv_den, float *ell) {
    for (int a = 0; a < r1; ++a) {
        float v = inv_den[a];
        for (int b = 0; b < r1; ++b)
            if (b != a) v *= (t - nodes[b]);
        ell[a] = v;
    }
}

// Their derivatives: l_a'(t) = inv_den_a sum_{m != a} prod_{b != a, m} (t - t_b).
__device__ __forceinline__ void lagrange_1d_deriv(float t, int r1, const float *nodes, const float *inv_den, float *dell) {
    for (int a = 0; a < r1; ++a) {
        float sum = 0.f;
        for (int m = 0; m < r1; ++m) {
            if (m == a) continue;
            float pr = 1.f;
            for (int b = 0; b < r1; ++b)
                if (b != a && b != m) pr *= (t - nodes[b]);
            sum += pr;
        }
        dell[a] = sum * inv_den[a];
    }
}

// u~_s = L_Y u_s: u~_s[(a r1 + b) r1 + c] = sum_j l_a(t_x) l_b(t_y) l_c(t_z) u_j, t = 2 (y - c_s) / d_l.
// With DL (the normal derivative at the sources) the weight of node (a, b, c) is n_j . grad_y of its polynomial:
// (2 / d_l) (n_x l'_a l_b l_c + n_y l_a l'_b l_c + n_z l_a l_b l'_c); the staged derivative tables carry the
// factors (2 / d_l) n.  Item (desc, source box, segment of its points).
//
// The sum over the points is a matrix product: rows (a, b), columns (c, part), one step of
// v_mfma_f32_16x16x4f32 per four points and 16 rows, with l_a l_b as the A and l_c u as the B operand (DL: two
// steps, A = l'_a l_b + l_a l'_b with B = l_c u, then A = l_a l_b with B = l'_c u).  Each wave takes every
// nw-th 64 points of the box: a lane evaluates one point's bases into the wave's own part of LDS, which the
// wave then reads as operands (an odd number of floats per point: the lanes' writes lie in distinct banks), without
// block barriers; the waves' tiles are added in wave order at the end.  MFMA issue bounds it (96 cycles per
// four points at r1 = 6 against about 50 for its LDS reads).  Sphere of 1M points, r1 = 6, levels 2 to 6: 974,
// 282, 96, 72, 82 us with one 256-thread block per box and a thread per node (three LDS reads and four VALU
// operations per point and node) -> 141, 46, 39, 38, 42 us; level 2 in 14 segments
// per box 52 us and 8 for their sums; with 25 floats per point instead of 24 43, 39, 32, 34, 34 us.
template <bool DL>
__host__ __device__ constexpr int anterp_floats(int r1) { return (DL ? 8 : 4) * r1 + 1; }   // LDS floats per point

template <bool DL, int R1>
__device__ __forceinline__ void lag_anterp_r1(const LDesc &d, const int4 wk, float *sm) {
    constexpr int R2 = R1 * R1, NT = (R2 + 15) / 16, W = 2 * R1, PT = anterp_floats<DL>(R1);
    const int b = wk.y;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nw = blockDim.x >> 6;
    const double two_over_dl = d.two_over_dl;
    float *my = sm + wv * 64 * PT;     // per point: l_x, l_y | l_z u (re, im) | DL: l'_x, l'_y | l'_z u
    const int li = lane & 15, lk = lane >> 4;
    int ia[NT], ib[NT];
    floatx4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int row = min(t * 16 + li, R2 - 1);
        ia[t] = row / R1;
        ib[t] = R1 + row % R1;
        acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    float nodes[R1], den[R1];
#pragma unroll
    for (int a = 0; a < R1; ++a) {
        nodes[a] = d.lnodes[a];
        den[a] = d.lden[a];
    }
    const double cx = d.sctr[3 * b], cy = d.sctr[3 * b + 1], cz = d.sctr[3 * b + 2];
    // this block's segment of the box's points: whole rounds of the block
    const int per = 64 * nw * ((d.sstart[b + 1] - d.sstart[b] + 64 * nw * d.nsplit - 1) / (64 * nw * d.nsplit));
    const int i0 = d.sstart[b] + wk.z * per, i1 = min(d.sstart[b + 1], i0 + per);
    for (int s0 = i0 + wv * 64; s0 < i1; s0 += nw * 64) {
        const int cnt = min(64, i1 - s0);
        {
            // lanes past the last point repeat it with u = 0
            const int j = min(s0 + lane, i1 - 1);
            float2 u = d.u[j];
            if (lane >= cnt) u = make_float2(0.f, 0.f);
            const float tx = (float)((d.sxs[j] - cx) * two_over_dl), ty = (float)((d.sys[j] - cy) * two_over_dl);
            const float tz = (float)((d.szs[j] - cz) * two_over_dl);
            float *q = my + lane * PT;
            float e[R1];
            lagrange_1d(tx, R1, nodes, den, e);
#pragma unroll
            for (int a = 0; a < R1; ++a) q[a] = e[a];
            lagrange_1d(ty, R1, nodes, den, e);
#pragma unroll
            for (int a = 0; a < R1; ++a) q[R1 + a] = e[a];
            lagrange_1d(tz, R1, nodes, den, e);
#pragma unroll
            for (int a = 0; a < R1; ++a) {
                q[W + 2 * a] = e[a] * u.x;
                q[W + 2 * a + 1] = e[a] * u.y;
            }
            if (DL) {
                const float4 n = d.sn[j];
                const float f = (float)two_over_dl;
                lagrange_1d_deriv(tx, R1, nodes, den, e);
#pragma unroll
                for (int a = 0; a < R1; ++a) q[2 * W + a] = e[a] * (f * n.x);
                lagrange_1d_deriv(ty, R1, nodes, den, e);
#pragma unroll
                for (int a = 0; a < R1; ++a) q[2 * W + R1 + a] = e[a] * (f * n.y);
                lagrange_1d_deriv(tz, R1, nodes, den, e);
#pragma unroll
                for (int a = 0; a < R1; ++a) {
                    q[3 * W + 2 * a] = e[a] * (f * n.z) * u.x;
                    q[3 * W + 2 * a + 1] = e[a] * (f * n.z) * u.y;
                }
            }
        }
        wave_lds_fence();
        // two steps per round, their operands loaded before the products (points past the last have u = 0)
        for (int p0 = 0; p0 < cnt; p0 += 8) {
            float a[2][NT], g[2][NT], bv[2], bg[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float *q = my + (p0 + 4 * h + lk) * PT;
                bv[h] = li < W ? q[W + li] : 0.f;
                bg[h] = DL && li < W ? q[3 * W + li] : 0.f;
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const float ex = q[ia[t]], ey = q[ib[t]];
                    a[h][t] = ex * ey;
                    if (DL) g[h][t] = fmaf(q[2 * W + ia[t]], ey, ex * q[2 * W + ib[t]]);
                }
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    if (DL) {
                        acc[t] = mfma16(g[h][t], bv[h], acc[t]);
                        acc[t] = mfma16(a[h][t], bg[h], acc[t]);
                    } else {
                        acc[t] = mfma16(a[h][t], bv[h], acc[t]);
                    }
                }
        }
        wave_lds_fence();
    }
    // entry (row, j) of the product is float row W + j of u~: lane (j, g) holds rows 4 g + v of each tile
    float *ut = reinterpret_cast<float *>((d.nsplit > 1 ? d.part + wk.z * d.part_stride : d.ut) + (int64_t)b * d.npair);
    if (nw == 1) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = t * 16 + 4 * lk + v;
                if (li < W && row < R2) ut[row * W + li] = acc[t][v];
            }
    } else {
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = t * 16 + 4 * lk + v;
                if (li < W && row < R2) sm[(wv * R2 + row) * W + li] = acc[t][v];
            }
        __syncthreads();
        for (int e = tid; e < R2 * W; e += blockDim.x) {
            float a = 0.f;
            for (int q = 0; q < nw; ++q) a += sm[q * R2 * W + e];
            ut[e] = a;
        }
    }
    for (int e = R2 * W + tid; e < 2 * d.rp; e += blockDim.x) ut[e] = 0.f;
}

template <bool DL>
__device__ __forceinline__ void lag_anterp_body(const LDesc &d, const int4 wk) {
    extern __shared__ float anterp_sm[];   // [waves][64][anterp_floats], then the waves' tiles
    // the node count as a compile-time constant: the basis loops unroll and the tiles per wave are fixed
    switch (d.r1) {
        case 1: lag_anterp_r1<DL, 1>(d, wk, anterp_sm); break;
        case 2: lag_anterp_r1<DL, 2>(d, wk, anterp_sm); break;
        case 3: lag_anterp_r1<DL, 3>(d, wk, anterp_sm); break;
        case 4: lag_anterp_r1<DL, 4>(d, wk, anterp_sm); break;
        case 5: lag_anterp_r1<DL, 5>(d, wk, anterp_sm); break;
        case 6: lag_anterp_r1<DL, 6>(d, wk, anterp_sm); break;
        case 7: lag_anterp_r1<DL, 7>(d, wk, anterp_sm); break;
        default: lag_anterp_r1<DL, 8>(d, wk, anterp_sm); break;
    }
}

__global__ void __launch_bounds__(1024)
k_lag_anterp(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    lag_anterp_body<false>(descs[wk.x], wk);
}

__global__ void __launch_bounds__(512)
k_lag_anterp_dl(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    lag_anterp_body<true>(descs[wk.x], wk);
}

// Transfers through the ACA factors of the classes (Sec. 2.2.2, eq. ffmACAmatvec: T_c ~ A_c B_c^T) in two kernels:
// k_lag_project forms Y_e = B_c^T u~_{s(e)} for every far pair e, by class groups; k_lag_expand forms v~_t = sum_e
// A_c(e) Y_e by target groups, so that only the rank's worth of values per pair goes through memory (128 B per 16
// ranks, against 1.7 KB for a transferred pair at r1 = 6), and the reductions per target need no buffer of pairs.
// Both are bound by what the L2s deliver (11 to 14 TB/s measured: the gathered sources, and the classes' tables once
// per group), the expansion by the memory behind them where the tables are larger (two sets, 665 complex classes: 5.9 GB of
// A_c in 1.07 ms).  Sphere of 1M points, Laplace, r1 = 6, level 6 (833,000 pairs): one kernel with both products
// through LDS and Z per pair 1570 us and its sum in the interpolation 326 -> 228 + 342 and 52 us; sphere of 300,000
// points, Helmholtz gradient, level 6: 1644 + 3 x 278 -> 294 + 602 + 3 x 50 us; workspaces of these plans 1.6 GB ->
// 0.3 and 0.46 GB.  Rank 4 u + g of a tile of 16 sits at position 4 g + u:
// a lane of k_lag_expand reads the positions of its g as one 16-byte load and uses them in steps u, so steps
// beyond the rank are left out.
//
// k_lag_project: one wave per class group of up to 16 pairs, products of v_mfma_f32_16x16x4f32 with the class's
// ranks as rows (tiles of 16) and the pairs as columns, the real and the imaginary parts of u~ in two products.
// Column m's lanes take their source's entries 16 jb + 4 g .. + 3 for the four steps of a block of 16 nodes, and
// B_c^T is stored in that fragment order ([class][plane][rank tile][jb][lane][4 steps]), so a lane's four A
// operands are one 16-byte load.  The sources go through the wave's own LDS, 32 nodes at a time, so that 16
// consecutive lanes read 256 consecutive bytes of one source (reading the columns straight from memory puts every
// lane of a load in another line, at a quarter of the rate).  The next step's loads are issued before a step's
// products.  Ranks above 16 (few classes) go over the sources once more per tile.
typedef float v4f __attribute__((ext_vector_type(4)));
typedef const v4f __attribute__((address_space(1))) *gc4;
typedef v4f __attribute__((address_space(1))) *gm4;
typedef const char __attribute__((address_space(1))) *gcb;

constexpr int kProjRow = 72;        // LDS floats per staged source: 32 nodes (64 floats) and a pad of two 16-byte slots

template <bool HELM>
__device__ __forceinline__ void lag_project_group(const LDesc &d, int grp, float *st, int *srcs, int lane) {
    const int g = lane >> 4, m = lane & 15, nb = d.aca_nb, kt = d.aca_kt;
    const int c = __builtin_amdgcn_readfirstlane(d.grp_cls[grp]);
    const int e = d.grp_pair[(int64_t)grp * 16 + m];
    // an empty slot computes some source's column and stores nothing
    if (lane < 16) srcs[lane] = d.far_src[max(e, 0)];
    wave_lds_fence();
    // staging: this lane moves 16 bytes (two nodes) of sources lane / 16 + 4 i
    gc4 U[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) U[i] = (gc4)(const v4f *)(d.ut2 + (int64_t)srcs[g + 4 * i] * d.rp) + m;
    float *sw = st + g * kProjRow + 4 * m;
    const float *sr = st + m * kProjRow + 8 * g;
    const int64_t tile = (int64_t)nb * 64, plane = tile * kt;
    const int ntile = (d.acaKp[c] + 15) >> 4;
    for (int rt = 0; rt < ntile; ++rt) {
        const gc4 B = (gc4)(d.acaB) + ((int64_t)c * (HELM ? 2 : 1) * kt + rt) * tile + lane;
        floatx4 yr = floatx4{0.f, 0.f, 0.f, 0.f}, yi = floatx4{0.f, 0.f, 0.f, 0.f};
        v4f u[4], br[2], bi[2];
        auto load = [&](int jb) {
#pragma unroll
            for (int i = 0; i < 4; ++i) u[i] = U[i][8 * jb];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                br[h] = B[(int64_t)(jb + h) * 64];
                if (HELM) bi[h] = B[plane + (int64_t)(jb + h) * 64];
            }
        };
        load(0);
        for (int jb = 0; jb < nb; jb += 2) {          // 32 nodes (nb is even)
#pragma unroll
            for (int i = 0; i < 4; ++i) *reinterpret_cast<v4f *>(sw + 4 * i * kProjRow) = u[i];
            const v4f cr[2] = {br[0], br[1]}, ci[2] = {bi[0], bi[1]};
            wave_lds_fence();
            v4f c0[2], c1[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const v4f *q = reinterpret_cast<const v4f *>(sr + 32 * h);
                c0[h] = q[0];
                c1[h] = q[1];
            }
            wave_lds_fence();
            if (jb + 2 < nb) load(jb + 2);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float ur[4] = {c0[h].x, c0[h].z, c1[h].x, c1[h].z}, ui[4] = {c0[h].y, c0[h].w, c1[h].y, c1[h].w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    yr = mfma16(cr[h][q], ur[q], yr);
                    yi = mfma16(cr[h][q], ui[q], yi);
                    if (HELM) {
                        yr = mfma16(-ci[h][q], ui[q], yr);
                        yi = mfma16(ci[h][q], ur[q], yi);
                    }
                }
            }
        }
        // Y_e: [tile][re, im][16]; lane (pair m, g) holds positions 4 g .. 4 g + 3 of the tile
        if (e >= 0) {
            const gm4 Y = (gm4)(v4f *)(d.Z) + ((int64_t)e * kt + rt) * 8 + g;
            Y[0] = v4f{yr[0], yr[1], yr[2], yr[3]};
            Y[4] = v4f{yi[0], yi[1], yi[2], yi[3]};
        }
    }
}

// Item (desc, first group, groups' end, 0): four class groups per block, one per wave.
template <bool HELM>
__global__ void __launch_bounds__(256)
k_lag_project(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    __shared__ float st[4][16 * kProjRow];
    __shared__ int srcs[4][16];
    const int4 wk = work[blockIdx.x];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), grp = wk.y + wv;
    if (grp < wk.z) lag_project_group<HELM>(descs[wk.x], grp, st[wv], srcs[wv], threadIdx.x & 63);
}

// k_lag_expand: v~ of a group of target boxes of the same octant of their parents, neighbours in Morton order, which
// share most of their translation classes: 16 columns (target, part) for eight targets, one unit of products per
// class that occurs in the group and rank tile (the plan lists them with each target's pair, k_expand_fill), 16
// rows and 4 ranks per v_mfma_f32_16x16x4f32.  A wave keeps RT row tiles of the group (the last block of a group the
// one or two that are left) in registers and walks its share of the group's units; A_c is stored in fragment order
// ([class][rank tile][row tile][plane][lane][4 steps]), so a unit is RT + 1 loads of 16 bytes per lane (twice that
// for the complex kernel), issued one or two units ahead (the unit list is staged in LDS, kExpandUnits at a time: read
// from memory unit by unit it put its misses into the chain, 335 -> 517 us at level 6).  A target without the class has
// a zero column: half of them on a sphere (a quarter in a volume), which still costs less than FMAs on the VALU
// with Y_e broadcast (LDS or scalar loads in a serial chain per pair).  The complex kernel, whose A_c is twice as
// long, takes two tiles of eight targets per group for each load of A_c, and leaves a tile out where none of its
// targets has the class.  The waves' tiles are added in wave order in LDS.  Item (desc, target group, first row tile).
// LONG: unit lists beyond kExpandUnits may occur (plan.hip asks for it by the longest list); the loop over pieces costs the
// others 1% (two sets, Helmholtz double layer, 200,000 targets).
template <bool HELM, int RT, bool LONG>
__device__ __forceinline__ void lag_expand_body(const LDesc &d, const int grp, const int rt0, float *sm) {
    constexpr int CT = HELM ? 2 : 1, NP = HELM ? 2 : 1;        // column tiles of eight targets, planes of A
    const int tid = threadIdx.x, lane = tid & 63, nw = blockDim.x >> 6;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, g = lane >> 4, part = col & 1;
    const int r = d.r1 * d.r1 * d.r1, nrt = (r + 15) >> 4, kt = d.aca_kt;
    const int off = __builtin_amdgcn_readfirstlane(d.exp_ptr[grp]), n = __builtin_amdgcn_readfirstlane(d.exp_cnt[grp]);
    const int cap = LONG ? min(n, kExpandUnits) : n;                   // units staged at a time
    int *se = reinterpret_cast<int *>(sm), *sc = se + 8 * CT * cap;    // [cap][8 CT] pairs, [cap] codes
    int q1 = 0;                                                        // end of the wave's share
    const uint32_t ustride = (uint32_t)nrt * NP * 1024;        // bytes of A per (class, rank tile)
    const gcb A0 = (gcb)(d.acaA) + (uint32_t)rt0 * NP * 1024;
    const gcb Y0 = (gcb)(d.Z);
    const uint32_t alane = 16 * lane, ylane = 16 * g + 64 * part, ystride = 128 * kt;
    const float sgn = part ? 1.f : -1.f;                       // (re, im) columns of i Y: (-Y_im, Y_re)
    floatx4 acc[RT][CT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int h = 0; h < CT; ++h) acc[t][h] = floatx4{0.f, 0.f, 0.f, 0.f};
    struct Unit {
        v4f a[RT][NP], y[CT][NP];
        int steps, e[CT];
    };
    // operands in flight: two units ahead, one for the complex kernel's four tiles (registers)
    constexpr int NB = HELM && RT == 4 ? 2 : 3;
    Unit buf[NB];
    auto load = [&](int q, Unit &u) {
        q = min(q, q1 - 1);
        const uint32_t code = __builtin_amdgcn_readfirstlane(sc[q]), kb = (code >> 2) & 7;
        u.steps = code & 3;
        const gcb A = A0 + (uint64_t)((code >> 5) * kt + kb) * ustride;
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int p = 0; p < NP; ++p) u.a[t][p] = *(gc4)(A + (t * NP + p) * 1024 + alane);
#pragma unroll
        for (int h = 0; h < CT; ++h) {
            u.e[h] = se[(8 * CT) * q + 8 * h + (col >> 1)];
            // a target without the class reads pair 0 instead (a branch here costs more: 335 -> 460 us at level 6); its
            // column is zeroed before the products
            const gcb Y = Y0 + (uint64_t)(uint32_t)max(u.e[h], 0) * ystride + (kb * 128 + ylane);
            u.y[h][0] = *(gc4)Y;
            if (HELM) u.y[h][NP - 1] = *(gc4)(Y + (64 - 128 * part));
        }
    };
    auto products = [&](const Unit &u) {
#pragma unroll
        for (int h = 0; h < CT; ++h) {
            if (CT > 1 && __ballot(u.e[h] >= 0) == 0) continue;    // none of these eight targets has the class
            v4f y0, y1;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                y0[k] = u.e[h] < 0 ? 0.f : u.y[h][0][k];
                if (HELM) y1[k] = u.e[h] < 0 ? 0.f : sgn * u.y[h][NP - 1][k];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (k > u.steps) break;
#pragma unroll
                for (int t = 0; t < RT; ++t) {
                    acc[t][h] = mfma16(u.a[t][0][k], y0[k], acc[t][h]);
                    if (HELM) acc[t][h] = mfma16(u.a[t][NP - 1][k], y1[k], acc[t][h]);
                }
            }
        }
    };
    int p0 = 0;
    do {
        // the units in LDS: addresses then depend on no load in flight
        const int cnt = LONG ? min(cap, n - p0) : n;
        if (LONG && p0) __syncthreads();
        for (int i = tid; i < 8 * CT * cnt; i += blockDim.x) se[i] = d.exp_e[(int64_t)(off + p0) * (8 * CT) + i];
        for (int i = tid; i < cnt; i += blockDim.x) sc[i] = d.exp_cls[off + p0 + i];
        __syncthreads();
        const int q0 = cnt * wv / nw;
        q1 = cnt * (wv + 1) / nw;
        if (q0 == q1) continue;
#pragma unroll
        for (int i = 0; i < NB - 1; ++i) load(q0 + i, buf[i]);
        for (int q = q0; q < q1; q += NB) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                load(q + i + NB - 1, buf[(i + NB - 1) % NB]);
                __builtin_amdgcn_sched_barrier(0);
                if (q + i < q1) products(buf[i]);
            }
        }
    } while (LONG && (p0 += cap) < n);
    // one column tile after the other, the waves' tiles added in wave order
#pragma unroll
    for (int h = 0; h < CT; ++h) {
        __syncthreads();                          // every wave is done with the unit list, or with the other tile
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) sm[((wv * RT + t) * 16 + 4 * g + v) * 16 + col] = acc[t][h][v];
        __syncthreads();
        for (int i = tid; i < 8 * 16 * RT; i += blockDim.x) {
            const int q = i / (16 * RT), row = i % (16 * RT), t = d.exp_tgt[((int64_t)grp * CT + h) * 8 + q];
            if (t < 0 || rt0 * 16 + row >= r) continue;
            float2 s = make_float2(0.f, 0.f);
            for (int w = 0; w < nw; ++w) {
                const float *p = sm + (w * RT * 16 + row) * 16 + 2 * q;
                s.x += p[0];
                s.y += p[1];
            }
            // over u~, which k_lag_project has read for the last time
            const int64_t at = d.exp_slot ? ((int64_t)grp * CT + h) * 8 + q : t;
            d.ut2[at * d.rp + rt0 * 16 + row] = s;
        }
    }
}

template <bool HELM, int RT, bool LONG>
__global__ void __launch_bounds__(RT == 1 ? 1024 : 512)
k_lag_expand(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    extern __shared__ float expand_sm[];      // the group's units, then [waves][RT][16][16]
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int left = ((d.r1 * d.r1 * d.r1 + 15) >> 4) - wk.z;        // row tiles from this block's first on
    if (RT == 4 && left < 4) {
        if (left > 1) lag_expand_body<HELM, 2, LONG>(d, wk.y, wk.z, expand_sm);
        else lag_expand_body<HELM, 1, LONG>(d, wk.y, wk.z, expand_sm);
    } else {
        lag_expand_body<HELM, RT, LONG>(d, wk.y, wk.z, expand_sm);
    }
}

// FP16 levels: the same u~ with every node's sum in the order of the points, one FMA per point.  u~ is rounded to FP16
// for the transfers, where a last-bit difference of a sum can move a value by a half unit of FP16, a thousand times
// more; in this order u~ does not depend on how the work is split.  v_mfma_f32_16x16x4f32 adds its four products
// as FMAs one after the other (checked on the device), so rows of nodes by two columns (re, im) give just that chain:
// l_a l_b l_c of the row's node is the A operand, formed from the chunk's bases in LDS, and every wave takes its own
// rows.  Bases are evaluated one chunk of 64 points ahead, an axis per wave.  Item (desc, source box, first row tile,
// waves of row tiles if four more stage, or 0: at least four waves that do both).  The serial chain (16 products
// of 32 cycles a chunk) and the barrier bound boxes of many points, LDS reads (four per 64 nodes and points) the rest.
// Ellipsoid, 137k points, r1 = 4, levels 2 to 6: 121, 55, 25, 13, 17 us.
template <int R1>
__device__ __forceinline__ void lag_anterp_ord_r1(const LDesc &d, const int4 wk, float (*e)[64 * 3 * kMaxR1],
                                                  float (*us)[128]) {
    constexpr int r = R1 * R1 * R1, NRT = (r + 15) / 16, W = 3 * R1;
    constexpr int MT = NRT > 16 ? 2 : 1;                           // row tiles per wave
    const int b = wk.y, tid = threadIdx.x, lane = tid & 63, nw = blockDim.x >> 6;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 15, lk = lane >> 4;
    const double two_over_dl = d.two_over_dl;
    float nodes[R1], den[R1];
#pragma unroll
    for (int a = 0; a < R1; ++a) {
        nodes[a] = d.lnodes[a];
        den[a] = d.lden[a];
    }
    const int xs = wv - wk.w;                                      // what the wave stages
    const int nc = wk.w ? wk.w : nw, t0 = wk.z + wv;                                      // first row tile of the wave
    int ia[MT], ib[MT], ic[MT];
    floatx4 acc[MT];
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        const int i = min(16 * (t0 + t * nc) + li, r - 1);
        ia[t] = i / (R1 * R1);
        ib[t] = R1 + (i / R1) % R1;
        ic[t] = 2 * R1 + i % R1;
        acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    const int i0 = d.sstart[b], i1 = d.sstart[b + 1];
    // wave wk.w + x, x < 3, evaluates axis x of a chunk and the next one lays down its inputs; the values are loaded a chunk earlier
    // (in every wave, whatever its part: a load under a condition would be waited for at once)
    const double *p = xs == 0 ? d.sxs : (xs == 1 ? d.sys : d.szs);
    const double ctr = d.sctr[3 * b + min(max(xs, 0), 2)];
    double pn = 0.0;
    float2 un{0.f, 0.f};
    auto fetch = [&](int s0) {
        const int j = min(s0 + lane, i1 - 1);
        pn = p[j];
        un = d.u[j];
    };
    auto stage = [&](int s0, int buf) {
        if (xs >= 0 && xs < 3) {
            float l[R1];
            lagrange_1d((float)((pn - ctr) * two_over_dl), R1, nodes, den, l);
#pragma unroll
            for (int a = 0; a < R1; ++a) e[buf][lane * W + xs * R1 + a] = l[a];
        } else if (xs == 3) {
            us[buf][2 * lane] = s0 + lane < i1 ? un.x : 0.f;
            us[buf][2 * lane + 1] = s0 + lane < i1 ? un.y : 0.f;
        }
    };
    fetch(i0);
    stage(i0, 0);
    fetch(i0 + 64);
    __syncthreads();
    for (int s0 = i0, buf = 0; s0 < i1; s0 += 64, buf ^= 1) {
        const int cnt = min(64, i1 - s0);
        if (s0 + 64 < i1) {
            stage(s0 + 64, buf ^ 1);
            fetch(s0 + 128);
        }
        // four steps per round (points past the last have u = 0 and leave every sum as it is)
        if (wv < nc) {
            for (int p0 = 0; p0 < cnt; p0 += 16) {
                float a[4][MT], bv[4];
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    const int pt = p0 + 4 * h + lk;
                    const float *q = e[buf] + pt * W;
                    bv[h] = us[buf][2 * pt + (li & 1)];
#pragma unroll
                    for (int t = 0; t < MT; ++t) a[h][t] = q[ia[t]] * q[ib[t]] * q[ic[t]];
                }
#pragma unroll
                for (int h = 0; h < 4; ++h)
#pragma unroll
                    for (int t = 0; t < MT; ++t)
                        if (t == 0 || t0 + t * nc < NRT) acc[t] = mfma16(a[h][t], bv[h], acc[t]);
            }
        }
        __syncthreads();
    }
    float *ut = reinterpret_cast<float *>(d.ut2 + (int64_t)b * d.rp);
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = 16 * (t0 + t * nc) + 4 * lk + v;
            if (li < 2 && i < r && wv < nc) ut[2 * i + li] = acc[t][v];
        }
    if (wk.z == 0)
        for (int x = 2 * r + tid; x < 2 * d.rp; x += blockDim.x) ut[x] = 0.f;
}

__global__ void __launch_bounds__(1024)
k_lag_anterp_ord(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    __shared__ float e[2][64 * 3 * kMaxR1], us[2][128];
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    switch (d.r1) {
        case 1: lag_anterp_ord_r1<1>(d, wk, e, us); break;
        case 2: lag_anterp_ord_r1<2>(d, wk, e, us); break;
        case 3: lag_anterp_ord_r1<3>(d, wk, e, us); break;
        case 4: lag_anterp_ord_r1<4>(d, wk, e, us); break;
        case 5: lag_anterp_ord_r1<5>(d, wk, e, us); break;
        case 6: lag_anterp_ord_r1<6>(d, wk, e, us); break;
        case 7: lag_anterp_ord_r1<7>(d, wk, e, us); break;
        default: lag_anterp_ord_r1<8>(d, wk, e, us); break;
    }
}

// Full transfer matrices: Z_e = T_c(e) u~_{s(e)} for every far pair, by class groups of 16 pairs (the columns, real and
// imaginary parts in two products), four groups of one class per block, one per wave.  T_c is stored in fragment
// order (rows and nodes of a product in one 16-byte load per lane) and goes through LDS once per block, two
// buffers, a barrier per step: at one group per load T_c is what the L2s deliver (16 KB per group at r1 = 4; 200 KB in
// FP16 and complex at r1 = 6) and the products waited for it.  The sources go through the wave's own LDS as in
// k_lag_project.  What the L2s deliver bounds it still: T_c once per 64 pairs, and the sources' u~.  FP32, r1 = 4: 137k
// points on an ellipsoid, level 6, 111 -> 63 us; 129k in a cube, 584k pairs, 155 us now.  32 problems of 2k to 137k
// points in one batch, against a wave per group and operands straight from memory: 9203 -> 4916 us FP32 with the
// kernels before and after it, FP16 8596 -> 5038 us.
struct GroupPairs {              // this lane's pair and its sources, one class group per wave
    int e = -1;
    gc4 U[4];
};

__device__ __forceinline__ void group_pairs(const LDesc &d, int grp, bool on, int *srcs, int lane, GroupPairs &p) {
    p.e = on ? d.grp_pair[(int64_t)grp * 16 + (lane & 15)] : -1;
    if (lane < 16) srcs[lane] = d.far_src[max(p.e, 0)];
    wave_lds_fence();
#pragma unroll
    for (int i = 0; i < 4; ++i)
        p.U[i] = (gc4)(const v4f *)(d.ut2 + (int64_t)srcs[(lane >> 4) + 4 * i] * d.rp) + (lane & 15);
}

// k_lag_mfma, FP32: v_mfma_f32_16x16x4f32, four row tiles at a time and 32 nodes per step.  T: [class][plane][row
// tile][block of 16 nodes][64 lanes][4 steps].  Item (desc, first group, groups, first row tile):
// a block takes four row tiles, for its few blocks are not enough to fill the chip where classes have few pairs, and its
// sources pass through LDS once per four tiles in any case.  (Node counts above r1 = 4, all row tiles in one block ->
// four, against one group per block and a row tile per wave: 4000 points on a sphere, Helmholtz, r1 = 6, 7, 8, the
// product with both levels 322, 671, 1218 -> 211, 379, 638 against 248, 467, 767 us; 200,000 points 1769, 3753, 6895 ->
// 1618, 3334, 6004 against 2371, 4558, 8168.)
template <bool HELM>
__global__ void __launch_bounds__(256)
k_lag_mfma(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    constexpr int P = HELM ? 2 : 1, RT = 4;
    __shared__ v4f sa[2][RT * 2 * P][64];
    __shared__ float st[4][16 * kProjRow];
    __shared__ int srcs[4][16];
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, m = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool on = wv < wk.z;
    const int c = __builtin_amdgcn_readfirstlane(d.grp_cls[wk.y]);
    const int rp = d.rp, nb = rp >> 4, nrt = (d.r1 * d.r1 * d.r1 + 15) >> 4;
    GroupPairs gp;
    group_pairs(d, wk.y + wv, on, srcs[wv], lane, gp);
    float *sw = st[wv] + g * kProjRow + 4 * m;
    const float *sr = st[wv] + m * kProjRow + 8 * g;
    const gc4 T = (gc4)(const v4f *)d.T + (int64_t)c * P * nrt * nb * 64 + lane;
    const int rt0 = wk.w;
    floatx4 zr[RT], zi[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) zr[t] = zi[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    v4f u[4], a[2 * P];
    auto load = [&](int jb) {
        if (on) {
#pragma unroll
            for (int i = 0; i < 4; ++i) u[i] = gp.U[i][8 * jb];
        }
        // this wave's share of the fragments: row tile wv, both blocks, both planes (tiles past the last repeat it)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int p = 0; p < P; ++p)
                a[h * P + p] = T[((int64_t)(p * nrt + min(rt0 + wv, nrt - 1)) * nb + jb + h) * 64];
    };
    load(0);
    for (int jb = 0; jb < nb; jb += 2) {
        const int buf = (jb >> 1) & 1;
#pragma unroll
        for (int q = 0; q < 2 * P; ++q) sa[buf][wv * 2 * P + q][lane] = a[q];
        if (on) {
            wave_lds_fence();                // (the step before has read its sources)
#pragma unroll
            for (int i = 0; i < 4; ++i) *reinterpret_cast<v4f *>(sw + 4 * i * kProjRow) = u[i];
        }
        __syncthreads();
        if (jb + 2 < nb) load(jb + 2);
        if (!on) continue;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const v4f c0 = *reinterpret_cast<const v4f *>(sr + 32 * h), c1 = *reinterpret_cast<const v4f *>(sr + 32 * h + 4);
            const float ur[4] = {c0.x, c0.z, c1.x, c1.z}, ui[4] = {c0.y, c0.w, c1.y, c1.w};
            v4f tr[RT], ti[RT];
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                tr[t] = sa[buf][t * 2 * P + h * P][lane];
                if (HELM) ti[t] = sa[buf][t * 2 * P + h * P + P - 1][lane];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int t = 0; t < RT; ++t) {
                    zr[t] = mfma16(tr[t][q], ur[q], zr[t]);
                    zi[t] = mfma16(tr[t][q], ui[q], zi[t]);
                    if (HELM) {
                        zr[t] = mfma16(-ti[t][q], ui[q], zr[t]);
                        zi[t] = mfma16(ti[t][q], ur[q], zi[t]);
                    }
                }
        }
    }
    // lane (pair m, g) holds rows 4 g .. 4 g + 3 of each tile
    if (gp.e >= 0) {
#pragma unroll
        for (int t = 0; t < RT; ++t)
            if (rt0 + t < nrt) {
                const gm4 Z = (gm4)(v4f *)(d.Z + (int64_t)gp.e * rp + 16 * (rt0 + t) + 4 * g);
                Z[0] = v4f{zr[t][0], zi[t][0], zr[t][1], zi[t][1]};
                Z[1] = v4f{zr[t][2], zi[t][2], zr[t][3], zi[t][3]};
            }
    }
}

// Mixed precision: the same products on FP16 MFMA (v_mfma_f32_16x16x32_f16: 16 rows, 32 nodes) with FP32
// accumulation.  T16 = T * sT (plan time); the sources are scaled by a power of two s_u derived on the device from
// max |u| so that |u~ s_u| < 6e4; Z = C / (sT s_u).
__device__ __forceinline__ float u_scale(float amax, int maxpts) {
    // |u~| <= (Lebesgue constant of the tensor grid, <= 8) * points * max|u|
    const float bound = 8.f * (float)maxpts * fmaxf(amax, 1e-30f);
    return exp2f(floorf(log2f(6.0e4f / bound)));
}

// k_lag_mfma16: the group's sources stay in registers as operands of all KB = rp / 32 blocks of 32 nodes, and T16 goes
// by RT row tiles per step, [class][row tile][block][plane][64 lanes][8 nodes].  Item (desc, first group, groups, 0).
template <bool HELM, int KB>
__global__ void __launch_bounds__(256)
k_lag_mfma16(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    constexpr int P = HELM ? 2 : 1, RT = KB == 1 ? 2 : (KB == 2 ? 4 : (KB == 4 ? 2 : 1)), NF = RT * KB * P;
    constexpr int NL = (NF + 3) / 4;         // fragments (1 KB each) a wave moves per step
    __shared__ half8_t sa[2][NF][64];
    __shared__ float st[4][16 * kProjRow];
    __shared__ int srcs[4][16];
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, m = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool on = wv < wk.z;
    const int c = __builtin_amdgcn_readfirstlane(d.grp_cls[wk.y]);
    const int rp = d.rp, nrt = (d.r1 * d.r1 * d.r1 + 15) >> 4;
    const float su = u_scale(*d.amax, d.maxpts), inv = 1.f / (d.sT * su);
    const gch8 T = (gch8)(const half8_t *)d.T16 + (int64_t)c * nrt * KB * P * 64 + lane;
    half8_t a[NL];
    auto load = [&](int rt0) {
        // (fragments past the last row tile's repeat the last fragment)
#pragma unroll
        for (int q = 0; q < NL; ++q)
            a[q] = T[(int64_t)min(rt0 * KB * P + min(wv + 4 * q, NF - 1), nrt * KB * P - 1) * 64];
    };
    load(0);
    GroupPairs gp;
    group_pairs(d, wk.y + wv, on, srcs[wv], lane, gp);
    half8_t ur[KB], ui[KB];
    if (on) {
        float *sw = st[wv] + g * kProjRow + 4 * m;
        const float *sr = st[wv] + m * kProjRow + 16 * g;
        v4f u[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) u[i] = gp.U[i][0];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
            for (int i = 0; i < 4; ++i) *reinterpret_cast<v4f *>(sw + 4 * i * kProjRow) = u[i];
            wave_lds_fence();
            if (kb + 1 < KB) {
#pragma unroll
                for (int i = 0; i < 4; ++i) u[i] = gp.U[i][16 * (kb + 1)];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v4f w = *reinterpret_cast<const v4f *>(sr + 4 * q);
                ur[kb][2 * q] = (_Float16)(w.x * su);
                ui[kb][2 * q] = (_Float16)(w.y * su);
                ur[kb][2 * q + 1] = (_Float16)(w.z * su);
                ui[kb][2 * q + 1] = (_Float16)(w.w * su);
            }
            wave_lds_fence();
        }
    }
    for (int rt0 = 0, step = 0; rt0 < nrt; rt0 += RT, ++step) {
        const int buf = step & 1;
#pragma unroll
        for (int q = 0; q < NL; ++q)
            if (wv + 4 * q < NF) sa[buf][wv + 4 * q][lane] = a[q];
        __syncthreads();
        if (rt0 + RT < nrt) load(rt0 + RT);
        if (!on) continue;
#pragma unroll
        for (int t = 0; t < RT; ++t) {
            floatx4 zr = floatx4{0.f, 0.f, 0.f, 0.f}, zi = zr, wr = zr, wi = zr;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                const half8_t tr = sa[buf][(t * KB + kb) * P][lane];
                zr = __builtin_amdgcn_mfma_f32_16x16x32_f16(tr, ur[kb], zr, 0, 0, 0);
                zi = __builtin_amdgcn_mfma_f32_16x16x32_f16(tr, ui[kb], zi, 0, 0, 0);
                if (HELM) {
                    const half8_t ti = sa[buf][(t * KB + kb) * P + P - 1][lane];
                    wr = __builtin_amdgcn_mfma_f32_16x16x32_f16(ti, ui[kb], wr, 0, 0, 0);
                    wi = __builtin_amdgcn_mfma_f32_16x16x32_f16(ti, ur[kb], wi, 0, 0, 0);
                }
            }
            if (gp.e >= 0 && rt0 + t < nrt) {
                float zx[4], zy[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    zx[v] = (HELM ? zr[v] - wr[v] : zr[v]) * inv;
                    zy[v] = (HELM ? zi[v] + wi[v] : zi[v]) * inv;
                }
                const gm4 Z = (gm4)(v4f *)(d.Z + (int64_t)gp.e * rp + 16 * (rt0 + t) + 4 * g);
                Z[0] = v4f{zx[0], zy[0], zx[1], zy[1]};
                Z[1] = v4f{zx[2], zy[2], zx[3], zy[3]};
            }
        }
    }
}

// R1 nodes per axis (a compile-time constant, so the basis arrays stay in registers with constant indices).
// v~_t = sum_{e in far(t)} Z_e in list order; the loads of eight entries are issued before their additions.
template <bool DN, int R1>
__device__ __forceinline__ void lag_interp_r1(const LDesc &d, const int4 wk, float2 *vt, const float *nodes,
                                              const float *den) {
    constexpr int r = R1 * R1 * R1;
    const int t = wk.y;
    const int tid = threadIdx.x;
    const int rp = d.rp;
    const double two_over_dl = d.two_over_dl;
    const int64_t e0 = d.far_ptr[t], e1 = d.far_ptr[t + 1];
    const gc2 Z = gl(d.Z);
    if (d.acaA) {
        // ACA levels: k_lag_expand has summed v~
        const gc2 V = gl(d.ut2) + (int64_t)(d.exp_slot ? d.exp_slot[t] : t) * rp;
        for (int i = tid; i < r; i += blockDim.x) {
            const v2f z = V[i];
            vt[i] = make_float2(z.x, z.y);
        }
    } else
    for (int i = tid; i < r; i += blockDim.x) {
        float ax = 0.f, ay = 0.f;
        int64_t e = e0;
        for (; e + 8 <= e1; e += 8) {
            v2f z[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) z[u] = Z[(e + u) * rp + i];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                ax += z[u].x;
                ay += z[u].y;
            }
        }
        for (; e < e1; ++e) {
            const v2f z = Z[e * rp + i];
            ax += z.x;
            ay += z.y;
        }
        vt[i] = make_float2(ax, ay);
    }
    __syncthreads();
    const double cx = d.tctr[3 * t], cy = d.tctr[3 * t + 1], cz = d.tctr[3 * t + 2];
    for (int i = wk.z + tid; i < wk.w; i += blockDim.x) {
        float lx[R1], ly[R1], lz[R1];
        const float tx = (float)((d.txs[i] - cx) * two_over_dl), ty = (float)((d.tys[i] - cy) * two_over_dl);
        const float tz = (float)((d.tzs[i] - cz) * two_over_dl);
        lagrange_1d(tx, R1, nodes, den, lx);
        lagrange_1d(ty, R1, nodes, den, ly);
        lagrange_1d(tz, R1, nodes, den, lz);
        float sre = 0.f, sim = 0.f;
        if (DN) {
            // n . grad of the interpolant: (2 / d_l) (n_x l'_a l_b l_c + n_y l_a l'_b l_c + n_z l_a l_b l'_c) v~
            float dx[R1], dy[R1], dz[R1];
            lagrange_1d_deriv(tx, R1, nodes, den, dx);
            lagrange_1d_deriv(ty, R1, nodes, den, dy);
            lagrange_1d_deriv(tz, R1, nodes, den, dz);
            const float4 n = d.tn ? d.tn[i] : d.tnc;
#pragma unroll
            for (int a = 0; a < R1; ++a) {
                float b0r = 0.f, b0i = 0.f, b1r = 0.f, b1i = 0.f;
#pragma unroll
                for (int bb = 0; bb < R1; ++bb) {
                    float c0r = 0.f, c0i = 0.f, c1r = 0.f, c1i = 0.f;
                    const float2 *row = vt + (a * R1 + bb) * R1;
#pragma unroll
                    for (int c = 0; c < R1; ++c) {
                        c0r = fmaf(lz[c], row[c].x, c0r);
                        c0i = fmaf(lz[c], row[c].y, c0i);
                        c1r = fmaf(dz[c], row[c].x, c1r);
                        c1i = fmaf(dz[c], row[c].y, c1i);
                    }
                    b0r = fmaf(ly[bb], c0r, b0r);      // l_b l_c
                    b0i = fmaf(ly[bb], c0i, b0i);
                    b1r = fmaf(n.y * dy[bb], c0r, fmaf(n.z * ly[bb], c1r, b1r));   // n_y l'_b l_c + n_z l_b l'_c
                    b1i = fmaf(n.y * dy[bb], c0i, fmaf(n.z * ly[bb], c1i, b1i));
                }
                sre = fmaf(n.x * dx[a], b0r, fmaf(lx[a], b1r, sre));
                sim = fmaf(n.x * dx[a], b0i, fmaf(lx[a], b1i, sim));
            }
            const float f = (float)two_over_dl;
            sre *= f;
            sim *= f;
        } else {
#pragma unroll
            for (int a = 0; a < R1; ++a) {
                float bre = 0.f, bim = 0.f;
#pragma unroll
                for (int bb = 0; bb < R1; ++bb) {
                    float cre = 0.f, cim = 0.f;
                    const float2 *row = vt + (a * R1 + bb) * R1;
#pragma unroll
                    for (int c = 0; c < R1; ++c) {
                        cre = fmaf(lz[c], row[c].x, cre);
                        cim = fmaf(lz[c], row[c].y, cim);
                    }
                    bre = fmaf(ly[bb], cre, bre);
                    bim = fmaf(ly[bb], cim, bim);
                }
                sre = fmaf(lx[a], bre, sre);
                sim = fmaf(lx[a], bim, sim);
            }
        }
        float2 o = d.v[i];
        o.x += sre;
        o.y += sim;
        d.v[i] = o;
    }
}

template <bool DN>
__device__ __forceinline__ void lag_interp_body(const LDesc &d, const int4 wk) {
    extern __shared__ float2 vt[];   // [r]
    __shared__ float nodes[kMaxR1], den[kMaxR1];
    const int tid = threadIdx.x;
    if (tid < d.r1) {
        nodes[tid] = d.lnodes[tid];
        den[tid] = d.lden[tid];
    }
    // (the reduction into vt below does not read nodes or den; the barrier after it orders their writes)
    switch (d.r1) {
        case 1: lag_interp_r1<DN, 1>(d, wk, vt, nodes, den); break;
        case 2: lag_interp_r1<DN, 2>(d, wk, vt, nodes, den); break;
        case 3: lag_interp_r1<DN, 3>(d, wk, vt, nodes, den); break;
        case 4: lag_interp_r1<DN, 4>(d, wk, vt, nodes, den); break;
        case 5: lag_interp_r1<DN, 5>(d, wk, vt, nodes, den); break;
        case 6: lag_interp_r1<DN, 6>(d, wk, vt, nodes, den); break;
        case 7: lag_interp_r1<DN, 7>(d, wk, vt, nodes, den); break;
        default: lag_interp_r1<DN, 8>(d, wk, vt, nodes, den); break;
    }
}

// v_i += L_X^T v~_t (or its normal derivative at x_i, k_lag_interp_dn) with v~_t = sum_{e in far(t)} Z_e (fixed
// order), t = 2 (x - c_t) / d_l.  Item (desc, target box, first point, end): boxes with many points are cut into
// ranges (plan.hip, kInterpBlocks), each forming v~_t anew (sphere of 1M points, r1 = 6: level 2 443 -> 41 us,
// level 3 135 -> 51).
__global__ void __launch_bounds__(kThreads)
k_lag_interp(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    lag_interp_body<false>(descs[wk.x], wk);
}

__global__ void __launch_bounds__(kThreads)
k_lag_interp_dn(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    lag_interp_body<true>(descs[wk.x], wk);
}

// ------------------------------------------------------------------ near field (leaf)
// v_i += sum_{s in near(t)} sum_{j in s, r_ij > 0} G(r_ij) u_j.  One block per target box, of one wave or, where boxes
// are too few to fill the chip, of two (in the symmetric pass of one set up to eight), which share the box's source
// chunks (plan.hip, near_waves).  A chunk
// whose list entry, range and points were fetched one after the other cost three memory latencies, more than its
// evaluation: with the list in LDS and the next chunk's points loaded ahead, and the waves, 23 -> 8.5 us for 4096 points
// (Laplace, 260 boxes), 236 -> 168 for 262,000 (4636), 525 -> 478 for 1M (18,354, one wave each), 4.4 -> 3.0 ms for 10M
// (Helmholtz, symmetric pass; times by rocprofv3).  Source points
// are staged through LDS in chunks of 64, in FP64 relative to the target centre, and every pair's difference is
// formed in FP64 and rounded once to FP32, so close pairs keep the full FP32 relative accuracy of r.  Helmholtz
// coordinates are scaled by k / 2 pi when staged (r then reads in revolutions, the phase of e^{ikr}), and the
// factors that scaling takes out of 1/r (and of the derivative's 1/r^3) go into the staged u.
//
// Targets go through the lanes in passes.  A pass of nt targets gives each lane T of them (T = 1, 2 or 4: g =
// ceil(nt / T) target groups, group gi holding targets gi, gi + g, ...) and gives each group R = 64 / g lanes;
// lane r of a group takes the contiguous range r * steps ... r * steps + steps - 1 of the chunk's staged sources
// (steps = ceil(cnt / R); staged slots past the chunk hold zero sources).  A lane evaluates every staged source
// against its T targets, so one set of LDS reads serves T pairs.  The R partial sums of a target are added in
// order of r.  The pass sizes come from the box's target count alone, so the summation order is fixed.
// Ranges of consecutive lanes start an odd number of 8-byte slots apart (slot r * (steps | 1) + q), so the R
// distinct addresses of one read fall in distinct banks.  The r > 0 test runs only where coincident points can
// occur: a box against itself when sources and targets are one set, every pair otherwise.
constexpr int kNearSlots = 128;

struct NearPass {
    int nt, T;
};

// Pass sizes for rem remaining targets: a full pass (64 m targets, m = 1, 2, 4, four per lane on 4 / m lanes
// each) is taken while it beats a single partial pass over everything left; cost = pairs per lane per staged
// source.  Equal costs go to four targets per lane, whose LDS reads serve four pairs.
__device__ __forceinline__ float near_pass_cost(int n, int T) {
    const int g = (n + T - 1) / T;
    return g > 64 ? 1e30f : (float)T / (float)(64 / g);
}

__device__ __forceinline__ NearPass near_next_pass(int rem) {
    float best = 1e30f;
    int bt = 1;
    for (int T = 1; T <= 4; T *= 2) {
        const float c = near_pass_cost(rem, T);
        if (c <= best) {
            best = c;
            bt = T;
        }
    }
    NearPass out{rem, bt};
    for (int m = 4; m >= 1; m /= 2) {
        const int full = 64 * m;
        if (rem <= full) continue;
        float rest = 1e30f;
        for (int T2 = 1; T2 <= 4; T2 *= 2) rest = fminf(rest, near_pass_cost(rem - full, T2));
        if (rest > 1e29f) rest = (float)((rem - full + 255) / 256) * 4.f;   // more full passes follow
        if ((float)m + rest < best) {
            best = (float)m + rest;
            out = NearPass{full, 4};
        }
    }
    return out;
}

struct NearSmem {
    double x[kNearSlots], y[kNearSlots], z[kNearSlots];   // part[] reuses x and y after the last chunk
    float2 u[kNearSlots];
    float2 sp[kNearSlots];                                 // source-side sums of a chunk (symmetric pairs)
};

// The chunks of a box's near list, numbered in list order, every chunk at most 64 sources of one box.  A wave reads
// the list's entries at once, one per lane, into its LDS, so finding a chunk's box and range takes no memory access,
// and a chunk's sources are loaded into registers while the chunk before is evaluated; the waves of a block take
// every nw-th chunk.
struct NearChunk {
    int s, c0, cnt, rel;          // source box, first source, sources, first source's position in its box
    int64_t off;                  // symmetric lists: the entry's near_off
};

struct NearRegs {                 // one source per lane
    double x, y, z;
    float2 u;
    float4 n;
};

struct NearList {                 // one entry per lane, in the wave's LDS
    int64_t off[64];
    int s[64], j0[64], j1[64], incl[64];      // incl: chunks up to and including the entry's
};

// SYM: lower neighbours with a reverse entry are left out (their own block evaluates the pair of boxes).  Returns the
// number of chunks.
template <bool SYM>
__device__ __forceinline__ int near_list(const LDesc &d, NearList &w, int t, int64_t e, int64_t e1) {
    const int lane = threadIdx.x & 63;
    const bool on = e + lane < e1;
    const int64_t el = on ? e + lane : e;
    const int s = d.near_src[el];
    const int64_t off = SYM ? d.near_off[el] : -1;
    const int j0 = d.sstart[s], j1 = d.sstart[s + 1];
    int n = !on || (SYM && s < t && off >= 0) ? 0 : (j1 - j0 + 63) >> 6;
    for (int k = 1; k < 64; k <<= 1) {
        const int v = __shfl_up(n, k, 64);
        if (lane >= k) n += v;
    }
    wave_lds_fence();
    w.s[lane] = s;
    w.j0[lane] = j0;
    w.j1[lane] = j1;
    w.incl[lane] = n;
    if (SYM) w.off[lane] = off;
    wave_lds_fence();
    return __builtin_amdgcn_readlane(n, 63);
}

template <bool SYM>
__device__ __forceinline__ NearChunk near_chunk(const NearList &w, int q) {
    const int e = __popcll(__ballot(w.incl[threadIdx.x & 63] <= q));
    NearChunk c;
    c.s = __builtin_amdgcn_readfirstlane(w.s[e]);
    c.rel = 64 * (q - (e ? __builtin_amdgcn_readfirstlane(w.incl[e - 1]) : 0));
    c.c0 = __builtin_amdgcn_readfirstlane(w.j0[e]) + c.rel;
    c.cnt = min(64, __builtin_amdgcn_readfirstlane(w.j1[e]) - c.c0);
    c.off = -1;
    if (SYM) {
        const int64_t o = w.off[e];
        c.off = ((int64_t)__builtin_amdgcn_readfirstlane((int)(o >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((int)o);
    }
    return c;
}

template <bool NRM>
__device__ __forceinline__ void near_load(const LDesc &d, const NearChunk &c, const float4 *nsrc, NearRegs &r) {
    const int j = c.c0 + min((int)(threadIdx.x & 63), c.cnt - 1);
    r.x = d.sxs[j];
    r.y = d.sys[j];
    r.z = d.szs[j];
    r.u = d.u[j];
    if (NRM) r.n = nsrc[j];
}

// Walk this wave's chunks of box t's near list: stage(chunk, registers), then compute(chunk).
template <bool SYM, bool NRM, class Stage, class Compute>
__device__ __forceinline__ void near_walk(const LDesc &d, NearList &w, int t, const float4 *nsrc, Stage &&stage,
                                          Compute &&compute) {
    const int nw = blockDim.x >> 6;
    const int64_t e1 = d.near_ptr[t + 1];
    for (int64_t e = d.near_ptr[t]; e < e1; e += 64) {
        const int total = near_list<SYM>(d, w, t, e, e1);
        int q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        if (q >= total) continue;
        NearChunk cur = near_chunk<SYM>(w, q);
        NearRegs r;
        near_load<NRM>(d, cur, nsrc, r);
        for (;;) {
            const NearChunk c = cur;
            stage(c, r);
            q += nw;
            const bool more = q < total;
            if (more) {
                cur = near_chunk<SYM>(w, q);
                near_load<NRM>(d, cur, nsrc, r);
            }
            compute(c);
            if (!more) break;
        }
    }
}

// Stage a chunk's sources (relative to the target centre, scaled) for R lane rows of `steps` sources each: source jj
// at slot (jj / steps) * so + jj % steps, zero sources in the slots of cnt <= jj < R * steps (at most 127).
// d.two_over_dl is 2 / d_l of the descriptor's level.  With snm, the source normals times nsign go to snm[slot] (the
// double layer stages the negated source normals: n_y . grad_y G(x - y) = (-n_y) . grad_x G(x - y)).
__device__ __forceinline__ void near_stage_chunk(const LDesc &d, NearSmem &sm, const NearRegs &r, int cnt, int R, int steps,
                                                 int so, double cx, double cy, double cz, double scale,
                                                 float uscale, float4 *snm, float nsign = -1.f) {
    const int lane = threadIdx.x & 63;
    // zero sources sit at (2, 2, 2) d_l from the target centre: no target is there (each lies within d_l / 2 of
    // its centre on every axis), so every pair with them has r > 0 and adds exactly zero, and their phases stay
    // within the bound of the level's near pairs
    const double pad = 4.0 / d.two_over_dl * scale;
    const uint32_t mul = (65536u + (uint32_t)steps - 1u) / (uint32_t)steps;   // jj / steps for jj < 128
    wave_lds_fence();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int jj = lane + 64 * h;
        if (jj < R * steps) {
            const int qd = (int)(((uint32_t)jj * mul) >> 16);
            const int slot = qd * so + (jj - qd * steps);
            if (jj < cnt) {
                sm.x[slot] = (r.x - cx) * scale;
                sm.y[slot] = (r.y - cy) * scale;
                sm.z[slot] = (r.z - cz) * scale;
                sm.u[slot] = make_float2(r.u.x * uscale, r.u.y * uscale);
                if (snm) snm[slot] = make_float4(nsign * r.n.x, nsign * r.n.y, nsign * r.n.z, 0.f);
            } else {
                sm.x[slot] = sm.y[slot] = sm.z[slot] = pad;   // padding: zero sources
                sm.u[slot] = make_float2(0.f, 0.f);
                if (snm) snm[slot] = make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
    }
    wave_lds_fence();
}

// A wave's LDS of the near-field kernels: the staged chunk, with normals (NRM 1, 2 of the kernels that stage them) or
// the source-side sums of a gradient's other two components.
template <int NRM, bool SYM>
struct NearWave {
    NearSmem sm;
    NearList list;
    float4 snm[(SYM ? NRM == 1 || NRM == 2 : NRM == 2) ? kNearSlots : 1];
    float2 sp12[SYM && NRM == 3 ? 2 : 1][SYM && NRM == 3 ? kNearSlots : 1];
};
extern __shared__ __align__(16) char near_raw[];

// Add a pass's sums to the output: every wave's partial sums a[k] of its lanes go to its LDS, and one thread per target
// adds the waves' R partial sums each in order, eight reads ahead of their sums.  (With the g lanes of the first wave
// going through all T targets of a lane, read by read, this was the larger part of a block with few sources: two waves
// per box then cost more than they gave, four of them 125 us for 64 boxes of 8 targets and 27 lists of 4 sources,
// gradient, against 62 with one.)
template <class W, int T>
__device__ __forceinline__ void near_reduce(W *waves, const float (&are)[T], const float (&aim)[T], int g, int R, int nt,
                                            float2 *out) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    float2 *part = reinterpret_cast<float2 *>(waves[wv].sm.x);   // [T][64], over x, y, z and u (T <= 5)
    __syncthreads();
#pragma unroll
    for (int k = 0; k < T; ++k) part[k * 64 + lane] = make_float2(are[k], aim[k]);
    __syncthreads();
    for (int ti = threadIdx.x; ti < nt; ti += blockDim.x) {
        const int k = ti / g, at = k * 64 + (ti - k * g);
        float2 a = make_float2(0.f, 0.f), o = out[ti];
        for (int w = 0; w < nw; ++w) {
            const float2 *pw = reinterpret_cast<const float2 *>(waves[w].sm.x) + at;
            for (int r0 = 0; r0 < R; r0 += 8) {
                float2 b[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) b[u] = pw[min(r0 + u, R - 1) * g];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (r0 + u < R) {
                        a.x += b[u].x;
                        a.y += b[u].y;
                    }
            }
        }
        o.x += a.x;
        o.y += a.y;
        out[ti] = o;
    }
    __syncthreads();
}

template <bool HELM, bool DN, bool BIG, bool CHK>
__device__ __forceinline__ void near_pair(double x, double y, double z, float nx, float ny, float nz, double sx,
                                          double sy, double sz, float2 uu, float &are, float &aim) {
    const float dx = (float)(x - sx), dy = (float)(y - sy), dz = (float)(z - sz);
    const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
    float inv = __builtin_amdgcn_rsqf(r2);
    if (CHK) inv = r2 > 0.f ? inv : 0.f;
    if (DN) {
        // n . grad_x G: (n . d) G'(r) / r with G' = -1 / r^2 (Laplace), (ikr - 1) e^{ikr} / r^2 (Helmholtz)
        const float i3 = inv * inv * inv * fmaf(nx, dx, fmaf(ny, dy, nz * dz));
        if (HELM) {
            const float rr = r2 * inv;
            float sn, cs;
            sincos_rev(BIG ? __builtin_amdgcn_fractf(rr) : rr, sn, cs);
            const float kr = 6.2831853f * rr;
            const float gr = i3 * fmaf(-kr, sn, -cs), gi = i3 * fmaf(kr, cs, -sn);
            are = fmaf(gr, uu.x, fmaf(-gi, uu.y, are));
            aim = fmaf(gr, uu.y, fmaf(gi, uu.x, aim));
        } else {
            are = fmaf(-i3, uu.x, are);
            aim = fmaf(-i3, uu.y, aim);
        }
    } else if (HELM) {
        const float rr = r2 * inv;
        float sn, cs;
        sincos_rev(BIG ? __builtin_amdgcn_fractf(rr) : rr, sn, cs);
        const float gr = cs * inv, gi = sn * inv;
        are = fmaf(gr, uu.x, fmaf(-gi, uu.y, are));
        aim = fmaf(gr, uu.y, fmaf(gi, uu.x, aim));
    } else {
        are = fmaf(inv, uu.x, are);
        aim = fmaf(inv, uu.y, aim);
    }
}

// One staged source against the lane's T targets.  NRM: 0 the kernel itself, 1 the normal derivative at the
// targets (their normals in nx, ny, nz), 2 at the sources (the staged negated normal of slot s).
template <bool HELM, int NRM, bool BIG, bool CHK, int T>
__device__ __forceinline__ void near_source(const NearSmem &sm, const float4 *snm, int s, const double (&x)[T],
                                            const double (&y)[T], const double (&z)[T], const float (&nx)[T],
                                            const float (&ny)[T], const float (&nz)[T], float (&are)[T],
                                            float (&aim)[T]) {
    const double sx = sm.x[s], sy = sm.y[s], sz = sm.z[s];
    const float2 uu = sm.u[s];
    if (NRM == 2) {
        const float4 n = snm[s];
#pragma unroll
        for (int t = 0; t < T; ++t)
            near_pair<HELM, true, BIG, CHK>(x[t], y[t], z[t], n.x, n.y, n.z, sx, sy, sz, uu, are[t], aim[t]);
    } else {
#pragma unroll
        for (int t = 0; t < T; ++t)
            near_pair<HELM, NRM == 1, BIG, CHK>(x[t], y[t], z[t], nx[t], ny[t], nz[t], sx, sy, sz, uu, are[t], aim[t]);
    }
}

// steps staged sources from slot base against the lane's T targets
template <bool HELM, int NRM, bool BIG, bool CHK, int T>
__device__ __forceinline__ void near_range(const NearSmem &sm, const float4 *snm, int base, int steps,
                                           const double (&x)[T], const double (&y)[T], const double (&z)[T],
                                           const float (&nx)[T], const float (&ny)[T], const float (&nz)[T],
                                           float (&are)[T], float (&aim)[T]) {
    constexpr int U = T >= 4 ? 1 : 4 / T;
    int q = 0;
    for (; q + U <= steps; q += U) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            near_source<HELM, NRM, BIG, CHK, T>(sm, snm, base + q + u, x, y, z, nx, ny, nz, are, aim);
    }
    for (; q < steps; ++q) near_source<HELM, NRM, BIG, CHK, T>(sm, snm, base + q, x, y, z, nx, ny, nz, are, aim);
}

// One pass: targets i0 ... i0 + nt - 1 of box t, T per lane.
template <bool HELM, int NRM, bool BIG, int T>
__device__ __forceinline__ void near_pass(const LDesc &d, NearWave<NRM, false> *waves, int t, int i0, int nt,
                                          double scale, float uscale) {
    const int lane = threadIdx.x & 63;
    NearSmem &sm = waves[threadIdx.x >> 6].sm;
    float4 *snm = waves[threadIdx.x >> 6].snm;
    const int g = __builtin_amdgcn_readfirstlane((nt + T - 1) / T), R = __builtin_amdgcn_readfirstlane(64 / g);
    const int r = lane / g, gi = lane - r * g;
    const bool valid = r < R;
    const double cx = d.tctr[3 * t], cy = d.tctr[3 * t + 1], cz = d.tctr[3 * t + 2];
    double x[T], y[T], z[T];
    float nx[T], ny[T], nz[T], are[T], aim[T];
#pragma unroll
    for (int k = 0; k < T; ++k) {
        const int ti = gi + g * k;
        x[k] = y[k] = z[k] = 0.0;
        nx[k] = ny[k] = nz[k] = 0.f;
        are[k] = aim[k] = 0.f;
        if (valid && ti < nt) {
            const int i = i0 + ti;
            x[k] = (d.txs[i] - cx) * scale;
            y[k] = (d.tys[i] - cy) * scale;
            z[k] = (d.tzs[i] - cz) * scale;
            if (NRM == 1) {
                const float4 n = d.tn ? d.tn[i] : d.tnc;
                nx[k] = n.x;
                ny[k] = n.y;
                nz[k] = n.z;
            }
        }
    }
    const bool same = d.same != 0;
    near_walk<false, NRM == 2>(
        d, waves[threadIdx.x >> 6].list, t, d.sn,
        [&](const NearChunk &c, const NearRegs &rg) {
            const int steps = (c.cnt + R - 1) / R;
            near_stage_chunk(d, sm, rg, c.cnt, R, steps, steps | 1, cx, cy, cz, scale, uscale, NRM == 2 ? snm : nullptr);
        },
        [&](const NearChunk &c) {
            const int steps = (c.cnt + R - 1) / R;
            const int base = valid ? r * (steps | 1) : 0;     // idle lanes read staged slots and discard their sums
            if (!same || c.s == t)
                near_range<HELM, NRM, BIG, true, T>(sm, snm, base, steps, x, y, z, nx, ny, nz, are, aim);
            else
                near_range<HELM, NRM, BIG, false, T>(sm, snm, base, steps, x, y, z, nx, ny, nz, are, aim);
        });
    near_reduce(waves, are, aim, g, R, nt, d.v + i0);
}

template <bool HELM, int NRM, bool BIG>
__device__ __forceinline__ void near_body(const LDesc &d, const int4 wk) {
    NearWave<NRM, false> *waves = reinterpret_cast<NearWave<NRM, false> *>(near_raw);
    const int t = wk.y;
    const int ta = d.tstart[t], tz = d.tstart[t + 1];
    // Helmholtz: coordinates in units of 2 pi / k; 1/r = (k / 2 pi) / r', 1/r^3 = (k / 2 pi)^3 / r'^3 and
    // n . d = (2 pi / k) n . d'
    const double kr = (double)d.k_rev;
    const double scale = HELM ? kr : 1.0;
    const float uscale = (float)((1.0 / (4.0 * M_PI)) * (HELM ? (NRM ? kr * kr : kr) : 1.0));
    for (int i0 = ta; i0 < tz;) {
        const NearPass ps = near_next_pass(tz - i0);
        if (ps.T == 1)
            near_pass<HELM, NRM, BIG, 1>(d, waves, t, i0, ps.nt, scale, uscale);
        else if (ps.T == 2)
            near_pass<HELM, NRM, BIG, 2>(d, waves, t, i0, ps.nt, scale, uscale);
        else
            near_pass<HELM, NRM, BIG, 4>(d, waves, t, i0, ps.nt, scale, uscale);
        i0 += ps.nt;
    }
}

template <bool HELM, bool BIG>
__global__ void __launch_bounds__(512, 4)
k_near(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    near_body<HELM, 0, BIG>(descs[wk.x], wk);
}

// The normal derivative at the target (the adjoint double-layer kernel), same blocks and lanes.
template <bool HELM, bool BIG>
__global__ void __launch_bounds__(512, 4)
k_near_dn(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    near_body<HELM, 1, BIG>(descs[wk.x], wk);
}

// The normal derivative at the source (the double-layer kernel), same blocks and lanes.
template <bool HELM, bool BIG>
__global__ void __launch_bounds__(512, 4)
k_near_dl(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    near_body<HELM, 2, BIG>(descs[wk.x], wk);
}

// The gradient at the targets: grad_x G(x - y) = d G'(r) / r, d = x - y.  The three components share r, 1/r^3
// and the phase; each component is formed as the normal derivative along its axis would form it (the same
// operations in the same order), so component c equals that pass with n = e_c.
template <bool HELM, bool BIG, bool CHK>
__device__ __forceinline__ void near_pair_grad(double x, double y, double z, double sx, double sy, double sz,
                                               float2 uu, float &ar0, float &ai0, float &ar1, float &ai1,
                                               float &ar2, float &ai2) {
    const float dx = (float)(x - sx), dy = (float)(y - sy), dz = (float)(z - sz);
    const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
    float inv = __builtin_amdgcn_rsqf(r2);
    if (CHK) inv = r2 > 0.f ? inv : 0.f;
    const float i3 = inv * inv * inv;
    const float f0 = i3 * dx, f1 = i3 * dy, f2 = i3 * dz;
    if (HELM) {
        const float rr = r2 * inv;
        float sn, cs;
        sincos_rev(BIG ? __builtin_amdgcn_fractf(rr) : rr, sn, cs);
        const float kr = 6.2831853f * rr;
        const float hr = fmaf(-kr, sn, -cs), hi = fmaf(kr, cs, -sn);
        float gr = f0 * hr, gi = f0 * hi;
        ar0 = fmaf(gr, uu.x, fmaf(-gi, uu.y, ar0));
        ai0 = fmaf(gr, uu.y, fmaf(gi, uu.x, ai0));
        gr = f1 * hr;
        gi = f1 * hi;
        ar1 = fmaf(gr, uu.x, fmaf(-gi, uu.y, ar1));
        ai1 = fmaf(gr, uu.y, fmaf(gi, uu.x, ai1));
        gr = f2 * hr;
        gi = f2 * hi;
        ar2 = fmaf(gr, uu.x, fmaf(-gi, uu.y, ar2));
        ai2 = fmaf(gr, uu.y, fmaf(gi, uu.x, ai2));
    } else {
        ar0 = fmaf(-f0, uu.x, ar0);
        ai0 = fmaf(-f0, uu.y, ai0);
        ar1 = fmaf(-f1, uu.x, ar1);
        ai1 = fmaf(-f1, uu.y, ai1);
        ar2 = fmaf(-f2, uu.x, ar2);
        ai2 = fmaf(-f2, uu.y, ai2);
    }
}

// steps staged sources from slot base against the lane's T targets, three components each
template <bool HELM, bool BIG, bool CHK, int T>
__device__ __forceinline__ void near_range_grad(const NearSmem &sm, int base, int steps, const double (&x)[T],
                                                const double (&y)[T], const double (&z)[T], float (&ar)[3][T],
                                                float (&ai)[3][T]) {
    for (int q = 0; q < steps; ++q) {
        const int s = base + q;
        const double sx = sm.x[s], sy = sm.y[s], sz = sm.z[s];
        const float2 uu = sm.u[s];
#pragma unroll
        for (int t = 0; t < T; ++t)
            near_pair_grad<HELM, BIG, CHK>(x[t], y[t], z[t], sx, sy, sz, uu, ar[0][t], ai[0][t], ar[1][t], ai[1][t],
                                           ar[2][t], ai[2][t]);
    }
}

// One pass of the gradient near field: the lanes and sources of near_pass; component c of target i is added
// to output plane c (d.v + c n_x).
template <bool HELM, bool BIG, int T>
__device__ __forceinline__ void near_pass_grad(const LDesc &d, NearWave<3, false> *waves, int t, int i0, int nt,
                                               double scale, float uscale) {
    const int lane = threadIdx.x & 63;
    NearSmem &sm = waves[threadIdx.x >> 6].sm;
    const int g = __builtin_amdgcn_readfirstlane((nt + T - 1) / T), R = __builtin_amdgcn_readfirstlane(64 / g);
    const int r = lane / g, gi = lane - r * g;
    const bool valid = r < R;
    const double cx = d.tctr[3 * t], cy = d.tctr[3 * t + 1], cz = d.tctr[3 * t + 2];
    double x[T], y[T], z[T];
    float ar[3][T], ai[3][T];
#pragma unroll
    for (int k = 0; k < T; ++k) {
        const int ti = gi + g * k;
        x[k] = y[k] = z[k] = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) ar[c][k] = ai[c][k] = 0.f;
        if (valid && ti < nt) {
            const int i = i0 + ti;
            x[k] = (d.txs[i] - cx) * scale;
            y[k] = (d.tys[i] - cy) * scale;
            z[k] = (d.tzs[i] - cz) * scale;
        }
    }
    const bool same = d.same != 0;
    near_walk<false, false>(
        d, waves[threadIdx.x >> 6].list, t, nullptr,
        [&](const NearChunk &c, const NearRegs &rg) {
            const int steps = (c.cnt + R - 1) / R;
            near_stage_chunk(d, sm, rg, c.cnt, R, steps, steps | 1, cx, cy, cz, scale, uscale, nullptr);
        },
        [&](const NearChunk &c) {
            const int steps = (c.cnt + R - 1) / R;
            const int base = valid ? r * (steps | 1) : 0;     // idle lanes read staged slots and discard their sums
            if (!same || c.s == t)
                near_range_grad<HELM, BIG, true, T>(sm, base, steps, x, y, z, ar, ai);
            else
                near_range_grad<HELM, BIG, false, T>(sm, base, steps, x, y, z, ar, ai);
        });
#pragma unroll
    for (int c = 0; c < 3; ++c) near_reduce(waves, ar[c], ai[c], g, R, nt, d.v + (int64_t)c * d.nx + i0);
}

// The gradient at the targets, all three components in one pass over the near pairs.  Item (desc, target box).
template <bool HELM, bool BIG>
__global__ void __launch_bounds__(512, 4)
k_near_grad(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    NearWave<3, false> *waves = reinterpret_cast<NearWave<3, false> *>(near_raw);
    const int t = wk.y;
    const int ta = d.tstart[t], tz = d.tstart[t + 1];
    const double kr = (double)d.k_rev;
    const double scale = HELM ? kr : 1.0;
    const float uscale = (float)((1.0 / (4.0 * M_PI)) * (HELM ? kr * kr : 1.0));
    for (int i0 = ta; i0 < tz;) {
        const NearPass ps = near_next_pass(tz - i0);
        if (ps.T == 1)
            near_pass_grad<HELM, BIG, 1>(d, waves, t, i0, ps.nt, scale, uscale);
        else if (ps.T == 2)
            near_pass_grad<HELM, BIG, 2>(d, waves, t, i0, ps.nt, scale, uscale);
        else
            near_pass_grad<HELM, BIG, 4>(d, waves, t, i0, ps.nt, scale, uscale);
        i0 += ps.nt;
    }
}

// ------------------------------------------------------------------ near field, one set (symmetric pairs)
// Sources and targets one set: G(x, y) = G(y, x), so an unordered pair of distinct neighbour boxes {t, s} is
// evaluated once, by the block of the lower box index: each pair's kernel value gives both v_i += G u_j (target
// side, in the lane's registers as above) and w_j += G u_i (source side).  The lanes form 4 rows of 16; a row
// holds 16 T targets (T = 1 ... 8 per lane, target slot gi + 16 k) and takes a contiguous range of the staged
// sources.  The source-side sums of a staged source over the row's 16 lanes are added in a fixed tree
// (data-parallel shifts within the row), and the chunk's sums are written, in order, to the entry's slice of a
// buffer (offset near_off[e]); passes after the first add to it.  The box itself (ordered, with the r > 0
// test) and lower neighbours without a reverse entry are evaluated as in k_near; lower neighbours with one are
// skipped here and added afterwards from the buffer by k_near_gather, in list order.  Passes hold up to 80
// targets (T <= 5: more targets per lane would cost registers, hence resident waves, more than they save).
template <int N>
__device__ __forceinline__ float dpp_row_shr(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x110 | N, 0xF, 0xF,
                                                                  true));
}

// inclusive sum over each 16-lane row: the row's total in its last lane
__device__ __forceinline__ float row_sum16(float v) {
    v += dpp_row_shr<1>(v);
    v += dpp_row_shr<2>(v);
    v += dpp_row_shr<4>(v);
    v += dpp_row_shr<8>(v);
    return v;
}

// nuy = -us.y and nty = -ut.y keep every product an FMA without a negation
template <bool HELM, bool BIG>
__device__ __forceinline__ void near_pair_sym(double x, double y, double z, float2 ut, float nty, double sx, double sy,
                                              double sz, float2 us, float nuy, float &are, float &aim, float &sre,
                                              float &sim) {
    const float dx = (float)(x - sx), dy = (float)(y - sy), dz = (float)(z - sz);
    const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
    const float inv = __builtin_amdgcn_rsqf(r2);   // distinct boxes of one set, padding far away: r > 0
    if (HELM) {
        const float rr = r2 * inv;
        float sn, cs;
        sincos_rev(BIG ? __builtin_amdgcn_fractf(rr) : rr, sn, cs);
        const float gr = cs * inv, gi = sn * inv;
        are = fmaf(gi, nuy, fmaf(gr, us.x, are));
        aim = fmaf(gi, us.x, fmaf(gr, us.y, aim));
        sre = fmaf(gi, nty, fmaf(gr, ut.x, sre));
        sim = fmaf(gi, ut.x, fmaf(gr, ut.y, sim));
    } else {
        are = fmaf(inv, us.x, are);
        aim = fmaf(inv, us.y, aim);
        sre = fmaf(inv, ut.x, sre);
        sim = fmaf(inv, ut.y, sim);
    }
}

template <bool HELM, bool BIG, int T>
__device__ __forceinline__ void near_pass_sym(const LDesc &d, NearWave<0, true> *waves, int t, int i0, int nt, bool first,
                                              double scale, float uscale) {
    constexpr int g = 16, R = 4;
    const int lane = threadIdx.x & 63;
    NearSmem &sm = waves[threadIdx.x >> 6].sm;
    const int r = lane >> 4, gi = lane & 15;
    const bool last = gi == g - 1;
    const double cx = d.tctr[3 * t], cy = d.tctr[3 * t + 1], cz = d.tctr[3 * t + 2];
    double x[T], y[T], z[T];
    float nx[T], ny[T], nz[T], are[T], aim[T], nty[T];
    float2 ut[T];
#pragma unroll
    for (int k = 0; k < T; ++k) {
        // a slot past nt repeats target 0 with zero input: its source-side terms are zero, its own sums discarded
        const int ti = gi + g * k;
        const int i = i0 + (ti < nt ? ti : 0);
        x[k] = (d.txs[i] - cx) * scale;
        y[k] = (d.tys[i] - cy) * scale;
        z[k] = (d.tzs[i] - cz) * scale;
        nx[k] = ny[k] = nz[k] = 0.f;
        are[k] = aim[k] = 0.f;
        const float2 uu = d.u[i];
        ut[k] = ti < nt ? make_float2(uu.x * uscale, uu.y * uscale) : make_float2(0.f, 0.f);
        nty[k] = -ut[k].y;
    }
    near_walk<true, false>(
        d, waves[threadIdx.x >> 6].list, t, nullptr,
        [&](const NearChunk &c, const NearRegs &rg) {
            const int steps = (c.cnt + R - 1) / R;
            near_stage_chunk(d, sm, rg, c.cnt, R, steps, steps | 1, cx, cy, cz, scale, uscale, nullptr);
        },
        [&](const NearChunk &c) {
            const int steps = (c.cnt + R - 1) / R, base = r * (steps | 1);
            if (c.s == t) {
                near_range<HELM, 0, BIG, true, T>(sm, nullptr, base, steps, x, y, z, nx, ny, nz, are, aim);
            } else if (c.s < t) {
                near_range<HELM, 0, BIG, false, T>(sm, nullptr, base, steps, x, y, z, nx, ny, nz, are, aim);
            } else {
                const int jb = r * steps;
                for (int q = 0; q < steps; ++q) {
                    const int sl = base + q;
                    const double sx = sm.x[sl], sy = sm.y[sl], sz = sm.z[sl];
                    const float2 us = sm.u[sl];
                    const float nuy = -us.y;
                    float sre = 0.f, sim = 0.f;
#pragma unroll
                    for (int k = 0; k < T; ++k)
                        near_pair_sym<HELM, BIG>(x[k], y[k], z[k], ut[k], nty[k], sx, sy, sz, us, nuy, are[k], aim[k],
                                                 sre, sim);
                    sre = row_sum16(sre);
                    sim = row_sum16(sim);
                    if (last) sm.sp[jb + q] = make_float2(sre, sim);   // slots past cnt are never read
                }
                wave_lds_fence();
                if (lane < c.cnt) {
                    // (the same wave takes this chunk in every pass)
                    float2 *o = d.nsym + c.off + c.rel + lane;
                    float2 a = sm.sp[lane];
                    if (!first) {
                        const float2 b = *o;
                        a.x += b.x;
                        a.y += b.y;
                    }
                    *o = a;
                }
            }
        });
    near_reduce(waves, are, aim, g, R, nt, d.v + i0);
}

template <bool HELM, bool BIG>
__global__ void __launch_bounds__(512, 4)
k_near_sym(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    NearWave<0, true> *waves = reinterpret_cast<NearWave<0, true> *>(near_raw);
    static_assert(offsetof(NearSmem, sp) >= 5 * 64 * sizeof(float2), "the partial sums must fit");
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int t = wk.y;
    const int ta = d.tstart[t], tz = d.tstart[t + 1];
    const double kr = (double)d.k_rev;
    const double scale = HELM ? kr : 1.0;
    const float uscale = (float)((1.0 / (4.0 * M_PI)) * (HELM ? kr : 1.0));
    for (int i0 = ta; i0 < tz;) {
        const int nt = min(80, tz - i0);
        const int T = (nt + 15) >> 4;
        const bool first = i0 == ta;
        switch (T) {
            case 1: near_pass_sym<HELM, BIG, 1>(d, waves, t, i0, nt, first, scale, uscale); break;
            case 2: near_pass_sym<HELM, BIG, 2>(d, waves, t, i0, nt, first, scale, uscale); break;
            case 3: near_pass_sym<HELM, BIG, 3>(d, waves, t, i0, nt, first, scale, uscale); break;
            case 4: near_pass_sym<HELM, BIG, 4>(d, waves, t, i0, nt, first, scale, uscale); break;
            default: near_pass_sym<HELM, BIG, 5>(d, waves, t, i0, nt, first, scale, uscale); break;
        }
        i0 += nt;
    }
}

// The symmetric pairs of the derivative kernels (one set), NRM 1: the normal derivative at the targets, 2: at the
// sources, 3: the gradient.  With d = x_i - x_j, grad_x G(x_i - x_j) = d h(r) and grad_x G(x_j - x_i) = -d h(r):
//   NRM 1: target i gets (n_i . d) h u_j, source j gets -(n_j . d) h u_i;
//   NRM 2: target i gets -(n_j . d) h u_j, source j gets (n_i . d) h u_i (the staged normals are -n_j);
//   NRM 3: target i gets d h u_j, source j gets -d h u_i (three components).
// h = -1 / r^3 (Laplace), (ikr - 1) e^{ikr} / r^3 (Helmholtz), in the scaled units of the ordered kernels.
template <bool HELM, bool BIG, int NRM, int NC>
__device__ __forceinline__ void near_pair_symd(double x, double y, double z, float tnx, float tny, float tnz,
                                               float2 ut, double sx, double sy, double sz, float4 sn, float2 us,
                                               float (&are)[NC], float (&aim)[NC], float (&sre)[NC],
                                               float (&sim)[NC]) {
    const float dx = (float)(x - sx), dy = (float)(y - sy), dz = (float)(z - sz);
    const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
    const float inv = __builtin_amdgcn_rsqf(r2);   // distinct boxes of one set, padding far away: r > 0
    const float i3 = inv * inv * inv;
    float hr = -1.f, hi = 0.f;
    if (HELM) {
        const float rr = r2 * inv;
        float sn_, cs;
        sincos_rev(BIG ? __builtin_amdgcn_fractf(rr) : rr, sn_, cs);
        const float kr = 6.2831853f * rr;
        hr = fmaf(-kr, sn_, -cs);
        hi = fmaf(kr, cs, -sn_);
    }
    if (NRM == 3) {
        const float dd[3] = {dx, dy, dz};
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const float f = i3 * dd[c];
            if (HELM) {
                const float gr = f * hr, gi = f * hi;
                are[c] = fmaf(gr, us.x, fmaf(-gi, us.y, are[c]));
                aim[c] = fmaf(gr, us.y, fmaf(gi, us.x, aim[c]));
                sre[c] = fmaf(-gr, ut.x, fmaf(gi, ut.y, sre[c]));
                sim[c] = fmaf(-gr, ut.y, fmaf(-gi, ut.x, sim[c]));
            } else {
                are[c] = fmaf(-f, us.x, are[c]);
                aim[c] = fmaf(-f, us.y, aim[c]);
                sre[c] = fmaf(f, ut.x, sre[c]);
                sim[c] = fmaf(f, ut.y, sim[c]);
            }
        }
    } else {
        const float a = fmaf(tnx, dx, fmaf(tny, dy, tnz * dz));       // n_i . d
        const float b = fmaf(sn.x, dx, fmaf(sn.y, dy, sn.z * dz));      // staged normal . d
        const float ft = NRM == 1 ? i3 * a : i3 * b, fs = NRM == 1 ? -(i3 * b) : i3 * a;
        if (HELM) {
            float gr = ft * hr, gi = ft * hi;
            are[0] = fmaf(gr, us.x, fmaf(-gi, us.y, are[0]));
            aim[0] = fmaf(gr, us.y, fmaf(gi, us.x, aim[0]));
            gr = fs * hr;
            gi = fs * hi;
            sre[0] = fmaf(gr, ut.x, fmaf(-gi, ut.y, sre[0]));
            sim[0] = fmaf(gr, ut.y, fmaf(gi, ut.x, sim[0]));
        } else {
            are[0] = fmaf(-ft, us.x, are[0]);
            aim[0] = fmaf(-ft, us.y, aim[0]);
            sre[0] = fmaf(-fs, ut.x, sre[0]);
            sim[0] = fmaf(-fs, ut.y, sim[0]);
        }
    }
}

// One pass of the symmetric derivative near field: the lanes, rows, lists and buffer of near_pass_sym; the
// sources' normals are staged beside them (NRM 1: n_j, NRM 2: -n_j), and a gradient's three components have
// their own accumulators, source-side sums, buffer planes (nsym + c nsymn) and output planes (v + c n_x).
template <bool HELM, bool BIG, int NRM, int T>
__device__ __forceinline__ void near_pass_symd(const LDesc &d, NearWave<NRM, true> *waves, int t, int i0, int nt,
                                               bool first, double scale, float uscale) {
    constexpr int g = 16, R = 4, NC = NRM == 3 ? 3 : 1;
    const int lane = threadIdx.x & 63;
    NearSmem &sm = waves[threadIdx.x >> 6].sm;
    float4 *snm = waves[threadIdx.x >> 6].snm;
    auto &sp12 = waves[threadIdx.x >> 6].sp12;
    const int r = lane >> 4, gi = lane & 15;
    const bool last = gi == g - 1;
    const double cx = d.tctr[3 * t], cy = d.tctr[3 * t + 1], cz = d.tctr[3 * t + 2];
    const float4 *nrm = NRM == 1 ? d.tn : d.sn;   // one set: a target's normal is its source normal
    double x[T], y[T], z[T];
    float nx[T], ny[T], nz[T];
    float are[NC][T], aim[NC][T];
    float2 ut[T];
#pragma unroll
    for (int k = 0; k < T; ++k) {
        // a slot past nt repeats target 0 with zero input: its source-side terms are zero, its own sums discarded
        const int ti = gi + g * k;
        const int i = i0 + (ti < nt ? ti : 0);
        x[k] = (d.txs[i] - cx) * scale;
        y[k] = (d.tys[i] - cy) * scale;
        z[k] = (d.tzs[i] - cz) * scale;
        nx[k] = ny[k] = nz[k] = 0.f;
        if (NRM != 3) {
            const float4 n = nrm[i];
            nx[k] = n.x;
            ny[k] = n.y;
            nz[k] = n.z;
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) are[c][k] = aim[c][k] = 0.f;
        const float2 uu = d.u[i];
        ut[k] = ti < nt ? make_float2(uu.x * uscale, uu.y * uscale) : make_float2(0.f, 0.f);
    }
    near_walk<true, NRM != 3>(
        d, waves[threadIdx.x >> 6].list, t, nrm,
        [&](const NearChunk &c, const NearRegs &rg) {
            const int steps = (c.cnt + R - 1) / R;
            near_stage_chunk(d, sm, rg, c.cnt, R, steps, steps | 1, cx, cy, cz, scale, uscale, NRM == 3 ? nullptr : snm,
                             NRM == 1 ? 1.f : -1.f);
        },
        [&](const NearChunk &c) {
            const int steps = (c.cnt + R - 1) / R, base = r * (steps | 1);
            if (c.s <= t) {
                // the box itself (r > 0 test) and lower neighbours without a reverse entry: ordered pairs
                if constexpr (NRM == 3) {
                    if (c.s == t)
                        near_range_grad<HELM, BIG, true, T>(sm, base, steps, x, y, z, are, aim);
                    else
                        near_range_grad<HELM, BIG, false, T>(sm, base, steps, x, y, z, are, aim);
                } else {
                    if (c.s == t)
                        near_range<HELM, NRM, BIG, true, T>(sm, snm, base, steps, x, y, z, nx, ny, nz, are[0], aim[0]);
                    else
                        near_range<HELM, NRM, BIG, false, T>(sm, snm, base, steps, x, y, z, nx, ny, nz, are[0], aim[0]);
                }
            } else {
                const int jb = r * steps;
                for (int q = 0; q < steps; ++q) {
                    const int sl = base + q;
                    const double sx = sm.x[sl], sy = sm.y[sl], sz = sm.z[sl];
                    const float2 us = sm.u[sl];
                    const float4 sn = NRM == 3 ? make_float4(0.f, 0.f, 0.f, 0.f) : snm[sl];
                    float sre[NC], sim[NC];
#pragma unroll
                    for (int m = 0; m < NC; ++m) sre[m] = sim[m] = 0.f;
#pragma unroll
                    for (int k = 0; k < T; ++k) {
                        float ar[NC], ai[NC];
#pragma unroll
                        for (int m = 0; m < NC; ++m) {
                            ar[m] = are[m][k];
                            ai[m] = aim[m][k];
                        }
                        near_pair_symd<HELM, BIG, NRM, NC>(x[k], y[k], z[k], nx[k], ny[k], nz[k], ut[k], sx, sy, sz,
                                                           sn, us, ar, ai, sre, sim);
#pragma unroll
                        for (int m = 0; m < NC; ++m) {
                            are[m][k] = ar[m];
                            aim[m][k] = ai[m];
                        }
                    }
#pragma unroll
                    for (int m = 0; m < NC; ++m) {
                        const float a = row_sum16(sre[m]), b = row_sum16(sim[m]);
                        if (last) (m == 0 ? sm.sp : sp12[m - 1])[jb + q] = make_float2(a, b);
                    }
                }
                wave_lds_fence();
                if (lane < c.cnt) {
#pragma unroll
                    for (int m = 0; m < NC; ++m) {
                        float2 *o = d.nsym + (int64_t)m * d.nsymn + c.off + c.rel + lane;
                        float2 a = (m == 0 ? sm.sp : sp12[m - 1])[lane];
                        if (!first) {
                            const float2 b = *o;
                            a.x += b.x;
                            a.y += b.y;
                        }
                        *o = a;
                    }
                }
            }
        });
#pragma unroll
    for (int c = 0; c < NC; ++c) near_reduce(waves, are[c], aim[c], g, R, nt, d.v + (int64_t)c * d.nx + i0);
}

template <bool HELM, bool BIG, int NRM>
__global__ void __launch_bounds__(512, 3)
k_near_sym_d(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    NearWave<NRM, true> *waves = reinterpret_cast<NearWave<NRM, true> *>(near_raw);
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int t = wk.y;
    const int ta = d.tstart[t], tz = d.tstart[t + 1];
    const double kr = (double)d.k_rev;
    const double scale = HELM ? kr : 1.0;
    const float uscale = (float)((1.0 / (4.0 * M_PI)) * (HELM ? kr * kr : 1.0));
    for (int i0 = ta; i0 < tz;) {
        const int nt = min(80, tz - i0);
        const int T = (nt + 15) >> 4;
        const bool first = i0 == ta;
        switch (T) {
            case 1: near_pass_symd<HELM, BIG, NRM, 1>(d, waves, t, i0, nt, first, scale, uscale); break;
            case 2: near_pass_symd<HELM, BIG, NRM, 2>(d, waves, t, i0, nt, first, scale, uscale); break;
            case 3: near_pass_symd<HELM, BIG, NRM, 3>(d, waves, t, i0, nt, first, scale, uscale); break;
            case 4: near_pass_symd<HELM, BIG, NRM, 4>(d, waves, t, i0, nt, first, scale, uscale); break;
            default: near_pass_symd<HELM, BIG, NRM, 5>(d, waves, t, i0, nt, first, scale, uscale); break;
        }
        i0 += nt;
    }
}

// v_i += the source-side sums that lower neighbour boxes computed for box b's points (list order).  Item
// (desc, box b).
__global__ void __launch_bounds__(64)
k_near_gather(const LDesc *__restrict__ descs, const IoEntry *__restrict__, const int4 *__restrict__ work) {
    const int4 wk = work[blockIdx.x];
    const LDesc &d = descs[wk.x];
    const int b = wk.y;
    const int ta = d.tstart[b], tz = d.tstart[b + 1];
    const int64_t e0 = d.near_ptr[b], e1 = d.near_ptr[b + 1];
    const int lane = threadIdx.x;
    for (int64_t eb = e0; eb < e1; eb += 64) {
        // the entries in the lanes; those with sums for this box in list order, four loads at a time
        int64_t off = -1;
        if (eb + lane < e1 && d.near_src[eb + lane] < b) off = d.near_off[eb + lane];
        const unsigned long long has = __ballot(off >= 0);
        for (int c = 0; c < d.ncomp; ++c) {
            const float2 *ns = d.nsym + (int64_t)c * d.nsymn - ta;
            float2 *vc = d.v + (int64_t)c * d.nx;
            for (int i = ta + lane; i - lane < tz; i += 64) {
                float2 a = make_float2(0.f, 0.f);
                unsigned long long m = has;
                while (m) {
                    float2 w[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        w[u] = make_float2(0.f, 0.f);
                        if (!m) continue;
                        const int e = __builtin_ctzll(m);
                        m &= m - 1;
                        const int64_t o = ((int64_t)__builtin_amdgcn_readlane((int)(off >> 32), e) << 32) |
                                          (uint32_t)__builtin_amdgcn_readlane((int)off, e);
                        if (i < tz) w[u] = ns[o + i];
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        a.x += w[u].x;
                        a.y += w[u].y;
                    }
                }
                if (i < tz) {
                    float2 o = vc[i];
                    o.x += a.x;
                    o.y += a.y;
                    vc[i] = o;
                }
            }
        }
    }
}

typedef void (*KernelFn)(const LDesc *, const IoEntry *, const int4 *);

KernelFn kernel_of(const Stage &S, int &threads) {
    threads = kThreads;
    switch (S.kern) {
        case K_PERM_IN: return k_perm_in;
        case K_AMAX: return S.a ? k_zero_amax : k_amax;
        case K_PERM_OUT: return k_perm_out;
        case K_FWD_PAIR:
            // a = PPT (+100: 64-thread blocks)
            if (S.a == 101) {
                threads = 64;
                return S.b ? k_pw_forward<1, 64, true> : k_pw_forward<1, 64, false>;
            }
            if (S.a == 4) return S.b ? k_pw_forward<4, kThreads, true> : k_pw_forward<4, kThreads, false>;
            if (S.a == 2) return S.b ? k_pw_forward<2, kThreads, true> : k_pw_forward<2, kThreads, false>;
            return S.b ? k_pw_forward<1, kThreads, true> : k_pw_forward<1, kThreads, false>;
        case K_FWD_PAIR_DL:
            if (S.a == 101) {
                threads = 64;
                return S.b ? k_pw_forward_dl<1, 64, true> : k_pw_forward_dl<1, 64, false>;
            }
            if (S.a == 4) return S.b ? k_pw_forward_dl<4, kThreads, true> : k_pw_forward_dl<4, kThreads, false>;
            if (S.a == 2) return S.b ? k_pw_forward_dl<2, kThreads, true> : k_pw_forward_dl<2, kThreads, false>;
            return S.b ? k_pw_forward_dl<1, kThreads, true> : k_pw_forward_dl<1, kThreads, false>;
        case K_FWD_RING:
            if (S.a == 4) return S.b ? k_pw_forward_rings<4, true> : k_pw_forward_rings<4, false>;
            return S.b ? k_pw_forward_rings<2, true> : k_pw_forward_rings<2, false>;
        case K_SUM: return k_sum_segments;
        case K_TRANSFER:
            // a = 1000 + direction pairs per tile (transfer_qt): class tables staged in LDS; else
            // a = PPT (+100: 64-thread blocks)
            switch (S.a) {
                case 1004: return k_pw_transfer_lds<4>;
                case 1002: return k_pw_transfer_lds<2>;
                case 1001: return k_pw_transfer_lds<1>;
                case 101: threads = 64; return k_pw_transfer<1, 64>;
                case 201: return k_pw_transfer_grp;
                case 301: return k_pw_transfer_sib;
                case 2: return k_pw_transfer<2, kThreads>;
                default: return k_pw_transfer<1, kThreads>;
            }
        case K_BWD_PAIR:
            // a = 100: 64-thread blocks
            if (S.a == 100) {
                threads = 64;
                return S.b ? k_pw_backward<64, true> : k_pw_backward<64, false>;
            }
            return S.b ? k_pw_backward<kThreads, true> : k_pw_backward<kThreads, false>;
        case K_BWD_RING:
            // inner loop unrolled by 4 (one point per thread) or 2 (two points per thread)
            // (a = 102: two points per thread in 128-thread blocks)
            if (S.a == 102) {
                threads = 128;
                return S.b ? k_pw_backward_rings<2, 2, true, 128> : k_pw_backward_rings<2, 2, false, 128>;
            }
            if (S.a == 2) return S.b ? k_pw_backward_rings<2, 2, true> : k_pw_backward_rings<2, 2, false>;
            return S.b ? k_pw_backward_rings<1, 4, true> : k_pw_backward_rings<1, 4, false>;
        case K_BSUM: return k_sum_parts;
        // a = waves per block
        case K_ANTERP: threads = 64 * std::max(1, S.a); return S.b ? k_lag_anterp_ord : k_lag_anterp;
        case K_ANTERP_DL: threads = 64 * std::max(1, S.a); return k_lag_anterp_dl;
        case K_DIRSCALE: return k_dir_scale;
        case K_DNCOMBINE: return k_dn_combine;
        case K_DLCOMBINE: return k_dl_combine;
        case K_MFMA32: return S.b ? k_lag_mfma<true> : k_lag_mfma<false>;
        case K_MFMA16:
            // a = rp / 32
            switch (S.a) {
                case 1: return S.b ? k_lag_mfma16<true, 1> : k_lag_mfma16<false, 1>;
                case 2: return S.b ? k_lag_mfma16<true, 2> : k_lag_mfma16<false, 2>;
                case 4: return S.b ? k_lag_mfma16<true, 4> : k_lag_mfma16<false, 4>;
                case 7: return S.b ? k_lag_mfma16<true, 7> : k_lag_mfma16<false, 7>;
                case 11: return S.b ? k_lag_mfma16<true, 11> : k_lag_mfma16<false, 11>;
                case 16: return S.b ? k_lag_mfma16<true, 16> : k_lag_mfma16<false, 16>;
                default: throw Error(FFM_EINTERNAL, "unknown node count");
            }
        case K_ACA: return S.b ? k_lag_project<true> : k_lag_project<false>;
        case K_EXPAND:
            // a = 1000 (long unit lists) + 100 (row tiles per wave) + waves
            threads = 64 * std::max(1, S.a % 100);
            if (S.a >= 1000) {
                if (S.a % 1000 < 200) return S.b ? k_lag_expand<true, 1, true> : k_lag_expand<false, 1, true>;
                return S.b ? k_lag_expand<true, 4, true> : k_lag_expand<false, 4, true>;
            }
            if (S.a < 200) return S.b ? k_lag_expand<true, 1, false> : k_lag_expand<false, 1, false>;
            return S.b ? k_lag_expand<true, 4, false> : k_lag_expand<false, 4, false>;
        case K_INTERP: threads = 64 * std::max(1, S.a); return k_lag_interp;
        // near-field kernels: a = BIG (symmetric ones BIG + 2 NRM) + 16 log2(waves per block)
        case K_NEAR:
            threads = 64 << (S.a >> 4);
            return S.b ? ((S.a & 1) ? k_near<true, true> : k_near<true, false>) : k_near<false, false>;
        case K_NEAR_SYM:
            // NRM 0: the kernel itself, 1: normal derivative at the targets, 2: at the sources, 3: the gradient
            threads = 64 << (S.a >> 4);
            switch ((S.a & 15) >> 1) {
                case 1:
                    return S.b ? ((S.a & 1) ? k_near_sym_d<true, true, 1> : k_near_sym_d<true, false, 1>)
                               : k_near_sym_d<false, false, 1>;
                case 2:
                    return S.b ? ((S.a & 1) ? k_near_sym_d<true, true, 2> : k_near_sym_d<true, false, 2>)
                               : k_near_sym_d<false, false, 2>;
                case 3:
                    return S.b ? ((S.a & 1) ? k_near_sym_d<true, true, 3> : k_near_sym_d<true, false, 3>)
                               : k_near_sym_d<false, false, 3>;
                default:
                    return S.b ? ((S.a & 1) ? k_near_sym<true, true> : k_near_sym<true, false>) : k_near_sym<false, false>;
            }
        case K_NEAR_GATHER: threads = 64; return k_near_gather;
        case K_NEAR_DL:
            threads = 64 << (S.a >> 4);
            return S.b ? ((S.a & 1) ? k_near_dl<true, true> : k_near_dl<true, false>) : k_near_dl<false, false>;
        case K_NEAR_DN:
            threads = 64 << (S.a >> 4);
            return S.b ? ((S.a & 1) ? k_near_dn<true, true> : k_near_dn<true, false>) : k_near_dn<false, false>;
        case K_NEAR_GRAD:
            threads = 64 << (S.a >> 4);
            return S.b ? ((S.a & 1) ? k_near_grad<true, true> : k_near_grad<true, false>) : k_near_grad<false, false>;
        case K_INTERP_DN: threads = 64 * std::max(1, S.a); return k_lag_interp_dn;
        case K_BWD_PAIR_DN:
            if (S.a == 100) {
                threads = 64;
                return S.b ? k_pw_backward_dn<64, true> : k_pw_backward_dn<64, false>;
            }
            return S.b ? k_pw_backward_dn<kThreads, true> : k_pw_backward_dn<kThreads, false>;
        case K_ZERO_OUT: return k_zero_io;
        case K_GSPREAD:
            switch (S.a) {
                case 4: return k_grid_spread<4>;
                case 5: return k_grid_spread<5>;
                case 6: return k_grid_spread<6>;
                case 7: return k_grid_spread<7>;
                case 8: return k_grid_spread<8>;
                default: throw Error(FFM_EINTERNAL, "unknown spreading width");
            }
        case K_GZ: return k_grid_z;
        case K_GPHI:
            // a = p / 16 for grids of at most 128 nodes per axis, 0 otherwise
            switch (S.a) {
                case 1: return k_grid_phi_s<1>;
                case 2: return k_grid_phi_s<2>;
                case 3: return k_grid_phi_s<3>;
                case 4: return k_grid_phi_s<4>;
                case 5: return k_grid_phi_r<5>;
                case 6: return k_grid_phi_r<6>;
                case 7: return k_grid_phi_r<7>;
                case 8: return k_grid_phi_r<8>;
                default: return k_grid_phi;
            }
        case K_GPHIT: return S.a == 1 ? k_grid_phit_wide : (S.a == 2 ? k_grid_phit_pair : k_grid_phit);
        case K_GZT: return k_grid_zt;
        case K_GINTERP:
            switch (S.a) {
                case 4: return k_grid_interp<4>;
                case 5: return k_grid_interp<5>;
                case 6: return k_grid_interp<6>;
                case 7: return k_grid_interp<7>;
                case 8: return k_grid_interp<8>;
                default: throw Error(FFM_EINTERNAL, "unknown spreading width");
            }
        default: throw Error(FFM_EINTERNAL, "unknown kernel variant");
    }
}

}  // namespace

size_t near_shmem(int kern, int a) {
    const size_t nw = (size_t)1 << (a >> 4);
    switch (kern) {
        case K_NEAR: return nw * sizeof(NearWave<0, false>);
        case K_NEAR_DN: return nw * sizeof(NearWave<1, false>);
        case K_NEAR_DL: return nw * sizeof(NearWave<2, false>);
        case K_NEAR_GRAD: return nw * sizeof(NearWave<3, false>);
        default: break;
    }
    switch ((a & 15) >> 1) {
        case 0: return nw * sizeof(NearWave<0, true>);
        case 1: return nw * sizeof(NearWave<1, true>);
        case 2: return nw * sizeof(NearWave<2, true>);
        default: return nw * sizeof(NearWave<3, true>);
    }
}

int stage_blocks_per_cu(int kern, int a, int b) {
    // a property of the compiled kernel and the device: queried once per (device, variant)
    static std::mutex mx;
    static std::map<std::tuple<int, int, int, int>, int> cache;
    int dev = 0;
    FFM_HIP(hipGetDevice(&dev));
    const auto key = std::make_tuple(dev, kern, a, b);
    {
        std::lock_guard<std::mutex> lk(mx);
        auto it = cache.find(key);
        if (it != cache.end()) return it->second;
    }
    Stage S;
    S.kern = kern;
    S.a = a;
    S.b = b;
    int threads = kThreads;
    KernelFn fn = kernel_of(S, threads);
    int nb = 0;
    FFM_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, threads, 0));
    nb = std::max(nb, 1);
    std::lock_guard<std::mutex> lk(mx);
    cache[key] = nb;
    return nb;
}

int device_cus() {
    static std::mutex mx;
    static std::map<int, int> cache;
    int dev = 0, n = 0;
    FFM_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lk(mx);
    auto it = cache.find(dev);
    if (it != cache.end()) return it->second;
    FFM_HIP(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev));
    return cache[dev] = std::max(n, 1);
}

void run_stage(const Stage &S, const LDesc *ddesc, const IoEntry *dio, hipStream_t st) {
    if (S.nitems == 0) return;
    FFM_CHECK(S.nitems < ((size_t)1 << 31), FFM_EINTERNAL, "stage grid too large");
    int threads = kThreads;
    KernelFn fn = kernel_of(S, threads);
    hipLaunchKernelGGL(fn, dim3((unsigned)S.nitems), dim3(threads), S.shmem, st, ddesc, dio, S.ditems);
    FFM_HIP(hipGetLastError());
}

// Record the end of a phase (timing plans only): the first call opens the apply.
void Plan::mark(int phase, hipStream_t st, const Stage *S) {
    if (tev.empty()) return;
    if (tused == (int)tev.size()) {
        // more launches than the events made with the plan (box batches, per-axis passes): one more event
        hipEvent_t e = nullptr;
        FFM_HIP(hipEventCreate(&e));
        tev.push_back(e);
        tphase.push_back(-1);
        tkern.push_back(make_int4(-1, 0, 0, 0));
        tblocks.push_back(0);
    }
    FFM_HIP(hipEventRecord(tev[tused], st));
    tphase[tused] = phase;
    tkern[tused] = S ? make_int4(S->kern, S->a, S->b, S->level) : make_int4(-1, 0, 0, 0);
    tblocks[tused] = S ? (int64_t)S->nitems : 0;
    ++tused;
}

void plan_apply(Plan &P, const void *wu, int dtype, float2 *v, hipStream_t st) {
    P.tused = 0;
    if (P.empty) {
        P.mark(-1, st);
        const int64_t nv = P.nx * P.ncomp();
        if (nv > 0) FFM_LAUNCH(k_zero_out, (int)((nv + kThreads - 1) / kThreads), kThreads, 0, st, v, nv);
        return;
    }
    // this apply's input and output go to the plan's I/O entry (pinned, copied in stream order); the
    // previous apply's copy has completed once its completion event has
    if (P.applied) FFM_HIP(hipEventSynchronize(P.done));
    if (P.pending) {
        // the plan's last GPU work runs on its planning stream: order this apply after it, and free its
        // temporaries once it is complete
        FFM_HIP(hipStreamWaitEvent(st, P.ready, 0));
        if (hipEventQuery(P.ready) == hipSuccess) {
            P.pending->release();
            P.pending.reset();
        }
    }
    P.hio->wu = wu;
    P.hio->vout = v;
    P.hio->dtype = dtype;
    FFM_HIP(hipMemcpyAsync(P.dio.p, P.hio, sizeof(IoEntry), hipMemcpyHostToDevice, st));
    P.mark(-1, st);
    for (const Stage &S : P.pre) {
        run_stage(S, P.ddesc.p, P.dio.p, st);
        P.mark(0, st, &S);
    }
    for (int l = 1; l <= P.leaf; ++l)
        for (const Stage &S : P.lev[l].stages) {
            run_stage(S, P.ddesc.p, P.dio.p, st);
            P.mark(S.tslot, st, &S);
        }
    for (const Stage &S : P.post) {
        run_stage(S, P.ddesc.p, P.dio.p, st);
        P.mark(S.tslot, st, &S);
    }
}

// The symbol of a stage's kernel as profilers print it (see kernel_of for the variants).
std::string kernel_name(int kern, int a, int b) {
    auto tf = [](int v) { return std::string(v ? "true" : "false"); };
    switch (kern) {
        case K_PERM_IN: return "k_perm_in";
        case K_AMAX: return a ? "k_zero_amax" : "k_amax";
        case K_PERM_OUT: return "k_perm_out";
        case K_FWD_PAIR:
            if (a == 101) return "k_pw_forward<1, 64, " + tf(b) + ">";
            return "k_pw_forward<" + std::to_string(a == 4 || a == 2 ? a : 1) + ", 256, " + tf(b) + ">";
        case K_FWD_PAIR_DL:
            if (a == 101) return "k_pw_forward_dl<1, 64, " + tf(b) + ">";
            return "k_pw_forward_dl<" + std::to_string(a == 4 || a == 2 ? a : 1) + ", 256, " + tf(b) + ">";
        case K_FWD_RING: return "k_pw_forward_rings<" + std::to_string(a == 4 ? 4 : 2) + ", " + tf(b) + ">";
        case K_SUM: return "k_sum_segments";
        case K_TRANSFER:
            if (a > 1000) return "k_pw_transfer_lds<" + std::to_string(a - 1000) + ">";
            if (a == 101) return "k_pw_transfer<1, 64>";
            if (a == 201) return "k_pw_transfer_grp";
            if (a == 301) return "k_pw_transfer_sib";
            return "k_pw_transfer<" + std::to_string(a == 2 ? 2 : 1) + ", 256>";
        case K_BWD_PAIR: return "k_pw_backward<" + std::to_string(a == 100 ? 64 : 256) + ", " + tf(b) + ">";
        case K_BWD_RING:
            if (a == 102) return "k_pw_backward_rings<2, 2, " + tf(b) + ", 128>";
            return a == 2 ? "k_pw_backward_rings<2, 2, " + tf(b) + ", 256>" : "k_pw_backward_rings<1, 4, " + tf(b) + ", 256>";
        case K_BSUM: return "k_sum_parts";
        case K_ANTERP: return b ? "k_lag_anterp_ord" : "k_lag_anterp";
        case K_ANTERP_DL: return "k_lag_anterp_dl";
        case K_DIRSCALE: return "k_dir_scale";
        case K_DNCOMBINE: return "k_dn_combine";
        case K_DLCOMBINE: return "k_dl_combine";
        case K_MFMA32: return "k_lag_mfma<" + tf(b) + ">";
        case K_MFMA16: return "k_lag_mfma16<" + tf(b) + ", " + std::to_string(a) + ">";
        case K_ACA: return "k_lag_project<" + tf(b) + ">";
        case K_EXPAND: return "k_lag_expand<" + tf(b) + (a % 1000 < 200 ? ", 1, " : ", 4, ") + tf(a >= 1000) + ">";
        case K_INTERP: return "k_lag_interp";
        case K_NEAR: return "k_near<" + tf(b) + ", " + tf(b && (a & 1)) + ">";
        case K_NEAR_SYM:
            if ((a & 15) >> 1)
                return "k_near_sym_d<" + tf(b) + ", " + tf(b && (a & 1)) + ", " + std::to_string((a & 15) >> 1) + ">";
            return "k_near_sym<" + tf(b) + ", " + tf(b && (a & 1)) + ">";
        case K_NEAR_GATHER: return "k_near_gather";
        case K_NEAR_DN: return "k_near_dn<" + tf(b) + ", " + tf(b && (a & 1)) + ">";
        case K_NEAR_GRAD: return "k_near_grad<" + tf(b) + ", " + tf(b && (a & 1)) + ">";
        case K_NEAR_DL: return "k_near_dl<" + tf(b) + ", " + tf(b && (a & 1)) + ">";
        case K_INTERP_DN: return "k_lag_interp_dn";
        case K_BWD_PAIR_DN: return "k_pw_backward_dn<" + std::to_string(a == 100 ? 64 : 256) + ", " + tf(b) + ">";
        case K_ZERO_OUT: return "k_zero_io";
        case K_GSPREAD: return a >= 4 && a <= 8 ? "k_grid_spread<" + std::to_string(a) + ">" : "";
        case K_GZ: return "k_grid_z";
        case K_GPHI:
            if (a >= 1 && a <= 4) return "k_grid_phi_s<" + std::to_string(a) + ">";
            return a >= 5 && a <= 8 ? "k_grid_phi_r<" + std::to_string(a) + ">" : "k_grid_phi";
        case K_GPHIT: return a == 1 ? "k_grid_phit_wide" : (a == 2 ? "k_grid_phit_pair" : "k_grid_phit");
        case K_GZT: return "k_grid_zt";
        case K_GINTERP: return a >= 4 && a <= 8 ? "k_grid_interp<" + std::to_string(a) + ">" : "";
        default: return "";
    }
}

}  // namespace ffm
