// Volume ray casting kernels for gfx950 (MI355X).
//
// G lanes per ray; a 64-lane wave covers a block of wave_w x (64/G/wave_w)
// pixels and a 256-thread workgroup a 2-D arrangement of four such blocks.
// For every pixel the kernel builds the ray in FP64, intersects it with the
// local box and the clipping planes (the kept scan points along a ray form
// one interval of the sample index k), then marches in FP32: at each scan
// point every active source is read at integer indices through its strided
// accessor, passed through its functor chain, interpolated (trilinear) or
// taken from the nearest cell, classified with its transfer table, weighted
// and mixed into one colour and opacity, and composited front to back until
// the opacity reaches the termination threshold.  This is the per-scan-point
// source loop of ISAAC (Matthes et al., Sec. 3.2, Fig. "pap" and the
// paragraph after it; functors Sec. 3.3, Tab. "functors").
//
// Source reads use raw buffer loads: a read outside the range the host
// derived from the declared extents returns 0 instead of touching memory.
// Transfer tables (256 x RGBA32F per source) live in LDS.
#include <hip/hip_runtime.h>

#include <limits.h>

#include <algorithm>
#include <mutex>

#include "isaac_internal.h"

namespace isaac {

namespace {

constexpr int kRsrcFlags = 0x00020000;   // raw buffer, 32-bit data format (gfx9 family)

// Source descriptors are wave-uniform by construction; readfirstlane keeps
// the buffer resource in SGPRs whatever the compiler could prove.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(uint64_t base, uint32_t n) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)base);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
    const uint64_t b = ((uint64_t)hi << 32) | lo;
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(b), (short)0,
                                             (int)__builtin_amdgcn_readfirstlane(n), kRsrcFlags);
}

__device__ __forceinline__ float ld_f32(__amdgpu_buffer_rsrc_t r, int off) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}

__device__ __forceinline__ float ld_scalar(__amdgpu_buffer_rsrc_t r, int off, int dtype) {
    if (dtype == DT_F32) return ld_f32(r, off);
    unsigned short h = __builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0);
    if (dtype == DT_F16) return (float)__builtin_bit_cast(_Float16, h);
    return __builtin_bit_cast(float, (uint32_t)h << 16);
}

// N voxels of one source (N = 1 nearest, 8 trilinear corners); off[i] is the
// byte offset of voxel i relative to voxel (0,0,0).  One uniform branch per
// call selects the load form, and all N loads are issued before any is used.
template <int N>
__device__ __forceinline__ void fetch(const DevSource& S, const int (&off)[N], float (&v)[N][4]) {
    const int f_dim = S.f_dim;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i][0] = v[i][1] = v[i][2] = v[i][3] = 0.f;
    if (S.packed && S.dtype == DT_F32) {
        // adjacent FP32 components: consecutive dword loads merge into x2/x3/x4 loads
        const __amdgpu_buffer_rsrc_t r = make_rsrc(S.base[0], S.num_records[0]);
        const int o = S.comp_off[0];
        if (f_dim == 1) {
#pragma unroll
            for (int i = 0; i < N; ++i) v[i][0] = ld_f32(r, off[i] + o);
        } else if (f_dim == 3) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                v[i][0] = ld_f32(r, off[i] + o);
                v[i][1] = ld_f32(r, off[i] + o + 4);
                v[i][2] = ld_f32(r, off[i] + o + 8);
            }
        } else if (f_dim == 2) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                v[i][0] = ld_f32(r, off[i] + o);
                v[i][1] = ld_f32(r, off[i] + o + 4);
            }
        } else {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                v[i][0] = ld_f32(r, off[i] + o);
                v[i][1] = ld_f32(r, off[i] + o + 4);
                v[i][2] = ld_f32(r, off[i] + o + 8);
                v[i][3] = ld_f32(r, off[i] + o + 12);
            }
        }
        return;
    }
    const int dtype = S.dtype;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if (c < f_dim) {
            const int k = S.packed ? 0 : c;
            const __amdgpu_buffer_rsrc_t r = make_rsrc(S.base[k], S.num_records[k]);
            const int o = S.comp_off[c];
#pragma unroll
            for (int i = 0; i < N; ++i) v[i][c] = ld_scalar(r, off[i] + o, dtype);
        }
    }
}

// pow for FP32 with IEEE special cases: exp2(y log2|x|), a negative base
// needs an integer exponent (odd exponents keep the sign), else NaN.
__device__ __forceinline__ float pow_f32(float x, float y) {
    if (y == 0.f) return 1.f;
    if (x == 1.f) return 1.f;
    float ax = fabsf(x);
    float r;
    if (ax == 0.f) {
        r = (y > 0.f) ? 0.f : __builtin_inff();
    } else {
        r = __builtin_amdgcn_exp2f(y * __builtin_amdgcn_logf(ax));
    }
    if (x < 0.f) {
        float yi = truncf(y);
        if (yi != y) return __builtin_nanf("");
        float half = 0.5f * yi;
        if (truncf(half) != half) r = -r;   // odd exponent
    }
    return r;
}

// Functor chain over N dates at once: one wave-uniform dispatch per functor,
// N dates of work inside.  D bounds the feature dimension at compile time
// (components D..3 are never touched); res[i] is component 0 of date i's
// result.
template <int N, int D = 4>
__device__ __forceinline__ void run_chain_n(const DevSource& S, float (&v)[N][4], float (&res)[N]) {
    const int n_ops = S.n_ops;
    for (int o = 0; o < n_ops; ++o) {
        const DevOp& op = S.ops[o];
        const int dim = op.dim;
        const float a[4] = {op.arg[0], op.arg[1], op.arg[2], op.arg[3]};
        switch (op.kind) {
        case OP_ADD:
#pragma unroll
            for (int c = 0; c < D; ++c)
                if (c < dim)
#pragma unroll
                    for (int i = 0; i < N; ++i) v[i][c] = v[i][c] + a[c];
            break;
        case OP_MUL:
#pragma unroll
            for (int c = 0; c < D; ++c)
                if (c < dim)
#pragma unroll
                    for (int i = 0; i < N; ++i) v[i][c] = v[i][c] * a[c];
            break;
        case OP_POW:
#pragma unroll
            for (int c = 0; c < D; ++c)
                if (c < dim)
#pragma unroll
                    for (int i = 0; i < N; ++i) v[i][c] = pow_f32(v[i][c], a[c]);
            break;
        case OP_SQRT:
#pragma unroll
            for (int c = 0; c < D; ++c)
                if (c < dim)
#pragma unroll
                    for (int i = 0; i < N; ++i)
                        v[i][c] = v[i][c] < 0.f ? __builtin_nanf("") : __builtin_amdgcn_sqrtf(v[i][c]);
            break;
        case OP_SQUARE:
#pragma unroll
            for (int c = 0; c < D; ++c)
                if (c < dim)
#pragma unroll
                    for (int i = 0; i < N; ++i) v[i][c] = v[i][c] * v[i][c];
            break;
        case OP_LENGTH:
#pragma unroll
            for (int i = 0; i < N; ++i) {
                float s = v[i][0] * v[i][0];
                if (D > 1 && dim > 1) s = fmaf(v[i][1], v[i][1], s);
                if (D > 2 && dim > 2) s = fmaf(v[i][2], v[i][2], s);
                if (D > 3 && dim > 3) s = fmaf(v[i][3], v[i][3], s);
                v[i][0] = __builtin_amdgcn_sqrtf(s);
            }
            break;
        case OP_SUM:
#pragma unroll
            for (int i = 0; i < N; ++i) {
                float s = v[i][0];
                if (D > 1 && dim > 1) s = s + v[i][1];
                if (D > 2 && dim > 2) s = s + v[i][2];
                if (D > 3 && dim > 3) s = s + v[i][3];
                v[i][0] = s;
            }
            break;
        default:
            break;
        }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) res[i] = v[i][0];
}

// The 8 trilinear corners run the bytecode in two groups of 4, which bounds
// the interpreter's live registers (more resident waves).
template <int N, int D = 4>
__device__ __forceinline__ void run_chain(const DevSource& S, float (&v)[N][4], float (&res)[N]) {
    if constexpr (N == 8) {
        float a[4][4], b[4][4], ra[4], rb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                a[i][c] = v[i][c];
                b[i][c] = v[i + 4][c];
            }
        run_chain_n<4, D>(S, a, ra);
        run_chain_n<4, D>(S, b, rb);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            res[i] = ra[i];
            res[i + 4] = rb[i];
        }
    } else {
        run_chain_n<N, D>(S, v, res);
    }
}

// Transfer-table lookup in a staged table (kTfLds values): clamp to [0,1]
// (NaN -> 0), 255 intervals, linear.  No contraction: the fraction is that of
// the rounded u in every caller, whatever the surrounding code lets the
// compiler fuse.  u is in [0, 255], so its fraction is exact and equals u - j;
// at u = 255 the lookup lands on the last entry, whose copy makes the slope 0,
// and returns T[255] itself.
__device__ __forceinline__ float4 classify(const float4* __restrict__ table, float x) {
#pragma clang fp contract(off)
    float t = fminf(fmaxf(x, 0.f), 1.f);    // max(NaN, 0) = 0
    float u = 255.f * t;
    int j = (int)u;
    float f = __builtin_amdgcn_fractf(u);
    const float4 a = table[j];              // T[j]
    const float4 b = table[j + 1];          // T[j+1]
    return make_float4(fmaf(f, b.x - a.x, a.x), fmaf(f, b.y - a.y, a.y), fmaf(f, b.z - a.z, a.z),
                       fmaf(f, b.w - a.w, a.w));
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return min(max(v, lo), hi); }

// FP64 ray setup.  Returns false if the ray misses the box or keeps no scan
// point; otherwise the kept sample indices are [*kb, *ke) and the FP32 ray is
// p(k) = pb + ((k + 1/2) * step) * d32.
struct RaySetup {
    float pb[3];           // global position of the ray at t0
    float d[3];
    int kb, ke;
    float t_first;         // ray parameter of scan point kb
};

// A set-up ray as stored by the setup passes (40 bytes).
struct RayRec {
    float pb[3];
    float d[3];
    int kb, ke;
    float t_first;
    int pixel;
};

// Scan point k in the volume's own index space: the global position minus the
// brick origin (an exact FP32 subtraction of an integer below the position).
__device__ __forceinline__ void point_at(const DevJob& J, const RaySetup& R, float tk, float (&p)[3]) {
    p[0] = fmaf(tk, R.d[0], R.pb[0]) - J.org[0];
    p[1] = fmaf(tk, R.d[1], R.pb[1]) - J.org[1];
    p[2] = fmaf(tk, R.d[2], R.pb[2]) - J.org[2];
}

// Trilinear cell coordinates u = p - 1/2 of scan point k in index space:
// the numbers point_at at (k + 1/2) step gives, minus 1/2, bit for bit, in
// fewer operations.  (k + 1/2) step and k step + step/2 are the same real
// number, rounded once either way; position - org is exact (an integer origin
// below 2^22, a position at most a voxel outside the brick), so subtracting
// org + 1/2 at once rounds the same value as subtracting org, then 1/2.
__device__ __forceinline__ void cell_at(const DevJob& J, const RaySetup& R, int k, float (&u)[3]) {
    const float tk = fmaf((float)k, (float)J.step, J.half_step);
    u[0] = fmaf(tk, R.d[0], R.pb[0]) - J.orgh[0];
    u[1] = fmaf(tk, R.d[1], R.pb[1]) - J.orgh[1];
    u[2] = fmaf(tk, R.d[2], R.pb[2]) - J.orgh[2];
}

__device__ __forceinline__ bool setup_ray(const DevJob& J, int px, int py, RaySetup& R) {
#pragma clang fp contract(off)
    const double x = (2.0 * (px + 0.5) / J.width - 1.0) * J.h * J.aspect;
    const double y = (1.0 - 2.0 * (py + 0.5) / J.height) * J.h;
    double o[3], d[3];
    if (J.ortho) {
        for (int a = 0; a < 3; ++a) {
            o[a] = J.eye[a] + x * J.right[a] + y * J.upp[a];
            d[a] = J.fwd[a];
        }
    } else {
        for (int a = 0; a < 3; ++a) {
            o[a] = J.eye[a];
            d[a] = J.fwd[a] + x * J.right[a] + y * J.upp[a];
        }
        const double n = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
        for (int a = 0; a < 3; ++a) d[a] = d[a] / n;
    }
    // slab test against the box [lo_a, hi_a] per axis
    auto slab = [&](const double* blo, const double* bhi, double& lo, double& hi) {
#pragma clang fp contract(off)
        lo = -__builtin_inf();
        hi = __builtin_inf();
        for (int a = 0; a < 3; ++a) {
            if (d[a] == 0.0) {
                if (o[a] < blo[a] || o[a] > bhi[a]) return false;
                continue;
            }
            const double ta = (blo[a] - o[a]) / d[a];
            const double tb = (bhi[a] - o[a]) / d[a];
            const double tn = ta < tb ? ta : tb;
            const double tf = ta < tb ? tb : ta;
            if (tn > lo) lo = tn;
            if (tf < hi) hi = tf;
        }
        return true;
    };
    // the step grid is anchored at the entry into the global box
    const double zero[3] = {0.0, 0.0, 0.0};
    double lo, hi;
    if (!slab(zero, J.gbox_hi, lo, hi)) return false;
    if (lo < 0.0) lo = 0.0;
    if (!(hi > lo)) return false;
    const double t0 = lo, t1 = hi, step = J.step;
    // scan points t_k = t0 + (k + 1/2) step with t_k < t1: k < (t1 - t0)/step - 1/2
    const double r = (t1 - t0) / step - 0.5;
    int kb = 0, ke = r > 0.0 ? (int)ceil(fmin(r, 2.0e9)) : 0;
    if (J.brick) {
        // a brick keeps the scan points inside its own box; neighbouring bricks
        // compute the shared crossing with the same expression, so every scan
        // point belongs to exactly one brick
        const double bl[3] = {(double)J.org[0], (double)J.org[1], (double)J.org[2]};
        const double bh[3] = {bl[0] + J.dims[0], bl[1] + J.dims[1], bl[2] + J.dims[2]};
        double blo, bhi;
        if (!slab(bl, bh, blo, bhi) || !(bhi > blo)) return false;
        kb = max(kb, (int)ceil(fmin(fmax((blo - t0) / step - 0.5, -1.0), 2.0e9)));
        ke = min(ke, (int)ceil(fmin(fmax((bhi - t0) / step - 0.5, -1.0), 2.0e9)));
    }
    // each plane keeps one interval of k: n.(o + t d) + d >= 0 is affine in t.
    // Bounds in closed form; a point this can misplace lies within FP64
    // rounding of the plane, far inside the decision margin
    for (int c = 0; c < J.n_clip; ++c) {
        const double* pl = J.clip[c];
        const double nd = pl[0] * d[0] + pl[1] * d[1] + pl[2] * d[2];
        const double no = pl[0] * o[0] + pl[1] * o[1] + pl[2] * o[2] + pl[3];
        if (nd == 0.0) {
            if (no < 0.0) ke = kb;
            continue;
        }
        const double kc = fmin(fmax((-no / nd - t0) / step - 0.5, -1.0), 2.0e9);
        if (nd > 0.0) kb = max(kb, (int)ceil(kc));          // kept for k >= kc
        else ke = min(ke, (int)floor(kc) + 1);              // kept for k <= kc
    }
    if (kb >= ke) return false;
    for (int a = 0; a < 3; ++a) {
        R.pb[a] = (float)(o[a] + t0 * d[a]);
        R.d[a] = (float)d[a];
    }
    R.kb = kb;
    R.ke = ke;
    R.t_first = (float)(t0 + ((double)kb + 0.5) * step);
    return true;
}

// One source at position p: nearest cell, or trilinear over the chain
// outputs of the 8 surrounding voxels (chain per fetched voxel, then blend).
template <int INTERP>
__device__ __forceinline__ float sample_source(const DevSource& S, const int dims[3], const float p[3]) {
    if (INTERP == 0) {
        const int qx = clampi((int)floorf(p[0]), 0, dims[0] - 1);
        const int qy = clampi((int)floorf(p[1]), 0, dims[1] - 1);
        const int qz = clampi((int)floorf(p[2]), 0, dims[2] - 1);
        const int off[1] = {qx * S.stride[0] + qy * S.stride[1] + qz * S.stride[2]};
        float v[1][4], r[1];
        fetch<1>(S, off, v);
        run_chain<1>(S, v, r);
        return r[0];
    }
    int i0[3], i1[3];
    float w[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float u = p[a] - 0.5f;
        const float fl = floorf(u);
        w[a] = u - fl;
        i0[a] = (int)fl;
        i1[a] = i0[a] + 1;
        if (S.guard < 1) {
            i0[a] = clampi(i0[a], 0, dims[a] - 1);
            i1[a] = clampi(i1[a], 0, dims[a] - 1);
        }
    }
    const int x0 = i0[0] * S.stride[0], x1 = i1[0] * S.stride[0];
    const int y0 = i0[1] * S.stride[1], y1 = i1[1] * S.stride[1];
    const int z0 = i0[2] * S.stride[2], z1 = i1[2] * S.stride[2];
    const int off[8] = {x0 + y0 + z0, x1 + y0 + z0, x0 + y1 + z0, x1 + y1 + z0,
                        x0 + y0 + z1, x1 + y0 + z1, x0 + y1 + z1, x1 + y1 + z1};
    float v[8][4], c[8];
    fetch<8>(S, off, v);
    run_chain<8>(S, v, c);
    const float c00 = fmaf(w[0], c[1] - c[0], c[0]);
    const float c10 = fmaf(w[0], c[3] - c[2], c[2]);
    const float c01 = fmaf(w[0], c[5] - c[4], c[4]);
    const float c11 = fmaf(w[0], c[7] - c[6], c[6]);
    const float c0 = fmaf(w[1], c10 - c00, c00);
    const float c1 = fmaf(w[1], c11 - c01, c01);
    return fmaf(w[2], c1 - c0, c0);
}

// A plain source (packed FP32 scalar, no functor, guard layers: a derived
// component, or such a source itself) at position p: sample_source's loads
// and arithmetic, without its run-time storage and chain handling (and so
// without the registers they hold).
template <int INTERP>
__device__ __forceinline__ float sample_plain(const DevSource& S, const int dims[3], const float p[3]) {
    const __amdgpu_buffer_rsrc_t r = make_rsrc(S.base[0], S.num_records[0]);
    const int o = S.comp_off[0];
    if (INTERP == 0) {
        const int qx = clampi((int)floorf(p[0]), 0, dims[0] - 1);
        const int qy = clampi((int)floorf(p[1]), 0, dims[1] - 1);
        const int qz = clampi((int)floorf(p[2]), 0, dims[2] - 1);
        return ld_f32(r, qx * S.stride[0] + qy * S.stride[1] + qz * S.stride[2] + o);
    }
    int i0[3], i1[3];
    float w[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const float u = p[a] - 0.5f;
        const float fl = floorf(u);
        w[a] = u - fl;
        i0[a] = (int)fl;
        i1[a] = i0[a] + 1;
    }
    const int x0 = i0[0] * S.stride[0], x1 = i1[0] * S.stride[0];
    const int y0 = i0[1] * S.stride[1], y1 = i1[1] * S.stride[1];
    const int z0 = i0[2] * S.stride[2], z1 = i1[2] * S.stride[2];
    const int off[8] = {x0 + y0 + z0, x1 + y0 + z0, x0 + y1 + z0, x1 + y1 + z0,
                        x0 + y0 + z1, x1 + y0 + z1, x0 + y1 + z1, x1 + y1 + z1};
    float c[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = ld_f32(r, off[i] + o);
    const float c00 = fmaf(w[0], c[1] - c[0], c[0]);
    const float c10 = fmaf(w[0], c[3] - c[2], c[2]);
    const float c01 = fmaf(w[0], c[5] - c[4], c[4]);
    const float c11 = fmaf(w[0], c[7] - c[6], c[6]);
    const float c0 = fmaf(w[1], c10 - c00, c00);
    const float c1 = fmaf(w[1], c11 - c01, c01);
    return fmaf(w[2], c1 - c0, c0);
}

template <int INTERP, bool PLAIN>
__device__ __forceinline__ float sample_any(const DevSource& S, const int dims[3], const float p[3]) {
    if constexpr (PLAIN) return sample_plain<INTERP>(S, dims, p);
    else return sample_source<INTERP>(S, dims, p);
}

// Compile-time source kinds of the specialized scan-point loop.
enum Kind : int { K_NONE = 0, K_F32x1 = 1, K_F32x3 = 2, K_F16x1 = 3, K_F16x3 = 4, K_BF16x1 = 5, K_BF16x3 = 6 };

template <int K> struct KindOf { static constexpr int dim = 1, dtype = DT_F32; };
template <> struct KindOf<K_F32x3> { static constexpr int dim = 3, dtype = DT_F32; };
template <> struct KindOf<K_F16x1> { static constexpr int dim = 1, dtype = DT_F16; };
template <> struct KindOf<K_F16x3> { static constexpr int dim = 3, dtype = DT_F16; };
template <> struct KindOf<K_BF16x1> { static constexpr int dim = 1, dtype = DT_BF16; };
template <> struct KindOf<K_BF16x3> { static constexpr int dim = 3, dtype = DT_BF16; };

// Voxel offsets of one source: nearest cell, or the 8 trilinear corners with
// the border clamp of guard-less sources.  24-bit multiplies (the host admits
// a signature only when every stride is below 2^23 bytes).
template <int INTERP, bool CLAMP = true>
__device__ __forceinline__ void corner_offsets(const DevSource& S, const int dims[3], const int (&i0)[3],
                                               int (&off)[INTERP ? 8 : 1]) {
    if (INTERP == 0) {
        off[0] = __mul24(i0[0], S.stride[0]) + __mul24(i0[1], S.stride[1]) + __mul24(i0[2], S.stride[2]);
        return;
    }
    int a0[3], a1[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        a0[a] = i0[a];
        a1[a] = i0[a] + 1;
        if (CLAMP && S.guard < 1) {
            a0[a] = clampi(a0[a], 0, dims[a] - 1);
            a1[a] = clampi(a1[a], 0, dims[a] - 1);
        }
    }
    const int x0 = __mul24(a0[0], S.stride[0]), x1 = __mul24(a1[0], S.stride[0]);
    const int y0 = __mul24(a0[1], S.stride[1]), y1 = __mul24(a1[1], S.stride[1]);
    const int z0 = __mul24(a0[2], S.stride[2]), z1 = __mul24(a1[2], S.stride[2]);
    off[0] = x0 + y0 + z0;
    off[1] = x1 + y0 + z0;
    off[2] = x0 + y1 + z0;
    off[3] = x1 + y1 + z0;
    off[4] = x0 + y0 + z1;
    off[5] = x1 + y0 + z1;
    off[6] = x0 + y1 + z1;
    off[7] = x1 + y1 + z1;
}

template <int K, int N>
__device__ __forceinline__ void fetch_kind(const DevSource& S, const int (&off)[N], float (&v)[N][4]) {
    constexpr int D = KindOf<K>::dim, T = KindOf<K>::dtype;
    const __amdgpu_buffer_rsrc_t r = make_rsrc(S.base[0], S.num_records[0]);
    const int o = S.comp_off[0];
#pragma unroll
    for (int i = 0; i < N; ++i) {
#pragma unroll
        for (int c = 0; c < 4; ++c) v[i][c] = 0.f;
#pragma unroll
        for (int c = 0; c < D; ++c) {
            if (T == DT_F32) v[i][c] = ld_f32(r, off[i] + o + 4 * c);
            else v[i][c] = ld_scalar(r, off[i] + o + 2 * c, T);
        }
    }
}

// The 8 corners of an FP32 scalar whose x neighbours are 4 bytes apart, in 4 loads.
__device__ __forceinline__ void fetch_f32_pairs(const DevSource& S, const int (&off)[8], float (&v)[8][4]) {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const __amdgpu_buffer_rsrc_t r = make_rsrc(S.base[0], S.num_records[0]);
    const int o = S.comp_off[0];
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
        const u32x2 x = __builtin_amdgcn_raw_buffer_load_b64(r, off[i] + o, 0, 0);
        const unsigned lo = x.x, hi = x.y;       // (bit_cast of a vector's element takes its first)
        v[i][0] = __builtin_bit_cast(float, lo);
        v[i + 1][0] = __builtin_bit_cast(float, hi);
#pragma unroll
        for (int c = 1; c < 4; ++c) v[i][c] = v[i + 1][c] = 0.f;
    }
}

// Sources of 16-bit values whose x neighbours are adjacent (2 D bytes apart): the
// D values of voxels x and x + 1 are 4 D consecutive bytes at an even address, and
// one aligned load of 8 (D = 1) or 16 bytes (D = 3) holds them, 4 loads for the 8
// corners instead of 8 D.  The window is moved down where it would pass the last
// dword of the range, so it is in bounds whatever the buffer's range check does
// with a load that straddles its end; `at` is where the values start in it
// (0, 2 or 4 bytes).  The first and the last dword of the range may hold two bytes
// that are not the source's (its base is 2-byte aligned): same dword, never used.
// 192^3 FP16 density, E and B in place at 1024 x 768: 674 -> 195 us a call (12
// loads a point instead of 56).
template <int D>
struct HalfPairs {
    static constexpr int n = D == 1 ? 2 : 4;     // dwords per load
    uint32_t w[4][n];
    int at[4];
};

template <int D>
__device__ __forceinline__ void load_half_pairs(const DevSource& S, const int (&off)[8], HalfPairs<D>& h) {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    const int pad = (int)(S.base[0] & 3);
    const uint32_t records = (S.num_records[0] + (uint32_t)pad + 3u) & ~3u;
    const __amdgpu_buffer_rsrc_t r = make_rsrc(S.base[0] & ~3ull, records);
    const int last = (int)records - 4 * HalfPairs<D>::n, o = S.comp_off[0] + pad;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int a = off[2 * i] + o, b = min(a & ~3, last);
        h.at[i] = a - b;
        if constexpr (D == 1) {
            const u32x2 x = __builtin_amdgcn_raw_buffer_load_b64(r, b, 0, 0);
            h.w[i][0] = x.x, h.w[i][1] = x.y;
        } else {
            const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(r, b, 0, 0);
            h.w[i][0] = x.x, h.w[i][1] = x.y, h.w[i][2] = x.z, h.w[i][3] = x.w;
        }
    }
}

template <int D, int T>
__device__ __forceinline__ void unpack_half_pairs(const HalfPairs<D>& h, float (&v)[8][4]) {
    auto widen = [](uint32_t bits, int hi) {     // the low or the high 16 bits
        if constexpr (T == DT_BF16) return __builtin_bit_cast(float, hi ? bits & 0xFFFF0000u : bits << 16);
        else return (float)__builtin_bit_cast(_Float16, (unsigned short)(hi ? bits >> 16 : bits & 0xFFFFu));
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t x[D];
#pragma unroll
        for (int k = 0; k < D; ++k)              // dword k of the 4 D bytes
            x[k] = (uint32_t)((((uint64_t)h.w[i][k + 1] << 32) | h.w[i][k]) >> (8 * h.at[i]));
#pragma unroll
        for (int c = 0; c < 4; ++c) v[2 * i][c] = v[2 * i + 1][c] = 0.f;
#pragma unroll
        for (int c = 0; c < D; ++c) {
            v[2 * i][c] = widen(x[c >> 1], c & 1);
            v[2 * i + 1][c] = widen(x[(D + c) >> 1], (D + c) & 1);
        }
    }
}

// The signatures whose sources are plain FP32 values side by side: n values
// per voxel, in (y, z) pairs or x fastest, with or without a border clamp.
template <int SIG> struct Il { static constexpr int n = 0; static constexpr bool paired = false, clamp = false; };
template <> struct Il<SIG_IL1> { static constexpr int n = 1; static constexpr bool paired = false, clamp = false; };
template <> struct Il<SIG_IL1C> { static constexpr int n = 1; static constexpr bool paired = false, clamp = true; };
template <> struct Il<SIG_IL2> { static constexpr int n = 2; static constexpr bool paired = false, clamp = false; };
template <> struct Il<SIG_IL3> { static constexpr int n = 3; static constexpr bool paired = false, clamp = false; };
template <> struct Il<SIG_IL3P> { static constexpr int n = 3; static constexpr bool paired = true, clamp = false; };
template <> struct Il<SIG_IL4> { static constexpr int n = 4; static constexpr bool paired = false, clamp = false; };

// The 8 trilinear corners (or the nearest cell) of such a volume, same corner
// order as corner_offsets.  A gather costs the texture-address unit one cycle
// per cache line its 64 lanes touch (at least 16 for more than 4 bytes a lane),
// whatever its width, so a load takes as many corners as are adjacent:
// one and two sources (4 and 8 bytes a voxel): both x corners in one load, 4
// loads instead of 8 (a batch of 64 FP32 scalars 1.88 -> 1.17 ms, bound by the
// address unit before) or, two derived sources, instead of 16 by the general
// loop (192 x 160 x 224 with a third clipped at 1280 x 720: 142 -> 47 us);
// three, x fastest, and four: one load per corner;
// three, PAIRED (layout 1, (y, z) pairs): the x + 1 corners are 48 bytes on (the
// loads' scalar offset); the y + 1 and z + 1 corners lie in the same pair or
// the next one depending on the parity of the index.  A wave's gathers of one
// corner touch fewer cache lines on oblique rays than in the x-fastest layout.
// A derived volume's y and z steps travel in the loads' scalar offset (its
// strides are not negative); a scalar read in place may have any strides, and
// its whole offset is subject to the buffer's range check.
template <int INTERP, int SIG>
__device__ __forceinline__ void fetch_il(const DevSource& S, const int dims[3], const int (&i0)[3],
                                         float (&v)[INTERP ? 8 : 1][4]) {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    constexpr int N = Il<SIG>::n;
    static_assert(!(Il<SIG>::paired && Il<SIG>::clamp), "derived pairs have guard layers");
    const __amdgpu_buffer_rsrc_t r = make_rsrc(S.base[0], S.num_records[0]);
    const int sx = __builtin_amdgcn_readfirstlane(S.stride[0]);
    const int sy = __builtin_amdgcn_readfirstlane(S.stride[1]);
    const int sz = __builtin_amdgcn_readfirstlane(S.stride[2]);
    auto f32 = [](unsigned b) { return __builtin_bit_cast(float, b); };
    // one voxel
    auto ld = [&](int vo, int so, float (&d)[4]) {
        if constexpr (N == 4) {
            const u32x4 b = __builtin_amdgcn_raw_buffer_load_b128(r, vo, so, 0);
            d[0] = f32(b.x), d[1] = f32(b.y), d[2] = f32(b.z), d[3] = f32(b.w);
        } else {
            d[0] = f32(__builtin_amdgcn_raw_buffer_load_b32(r, vo, so, 0));
            if constexpr (N > 1) d[1] = f32(__builtin_amdgcn_raw_buffer_load_b32(r, vo + 4, so, 0));
            if constexpr (N > 2) d[2] = f32(__builtin_amdgcn_raw_buffer_load_b32(r, vo + 8, so, 0));
        }
    };
    // voxels x and x + 1 (adjacent)
    auto ld_pair = [&](int vo, int so, float (&d0)[4], float (&d1)[4]) {
        if constexpr (N == 1) {
            const u32x2 b = __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, 0);
            d0[0] = f32(b.x), d1[0] = f32(b.y);
        } else if constexpr (N == 2) {
            const u32x4 b = __builtin_amdgcn_raw_buffer_load_b128(r, vo, so, 0);
            d0[0] = f32(b.x), d0[1] = f32(b.y), d1[0] = f32(b.z), d1[1] = f32(b.w);
        } else {
            ld(vo, so, d0);
            ld(vo, so + sx, d1);
        }
    };
    if constexpr (Il<SIG>::paired) {
        const int yl = i0[1] & 1, zl = i0[2] & 1;
        const int b0 = __mul24(i0[2] >> 1, sz) + __mul24(i0[1] >> 1, sy) + __mul24(i0[0], sx) + __mul24(zl, 24) +
                       __mul24(yl, 12) + S.comp_off[0];
        if constexpr (INTERP == 0) {
            ld(b0, 0, v[0]);
        } else {
            const int oy = __mul24(yl, sy - 24) + 12;   // y + 1: same pair (+12) or the next one
            const int oz = __mul24(zl, sz - 48) + 24;   // z + 1: same pair (+24) or the next one
            const int b2 = b0 + oy, b4 = b0 + oz, b6 = b4 + oy;
            ld_pair(b0, 0, v[0], v[1]);
            ld_pair(b2, 0, v[2], v[3]);
            ld_pair(b4, 0, v[4], v[5]);
            ld_pair(b6, 0, v[6], v[7]);
        }
    } else if constexpr (Il<SIG>::clamp && INTERP != 0) {
        // the x pair from the last place it fits; at a border both corners are the border voxel
        const int xb = clampi(i0[0], 0, dims[0] - 2);
        const int bx = __mul24(xb, sx) + S.comp_off[0];
        const int y0 = __mul24(clampi(i0[1], 0, dims[1] - 1), sy), y1 = __mul24(clampi(i0[1] + 1, 0, dims[1] - 1), sy);
        const int z0 = __mul24(clampi(i0[2], 0, dims[2] - 1), sz), z1 = __mul24(clampi(i0[2] + 1, 0, dims[2] - 1), sz);
        ld_pair(bx + y0 + z0, 0, v[0], v[1]);
        ld_pair(bx + y1 + z0, 0, v[2], v[3]);
        ld_pair(bx + y0 + z1, 0, v[4], v[5]);
        ld_pair(bx + y1 + z1, 0, v[6], v[7]);
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
            const float lo = v[i][0], hi = v[i + 1][0];
            v[i][0] = i0[0] > xb ? hi : lo;
            v[i + 1][0] = i0[0] < xb ? lo : hi;
        }
    } else {
        const int b0 = __mul24(i0[0], sx) + __mul24(i0[1], sy) + __mul24(i0[2], sz) + S.comp_off[0];
        if constexpr (INTERP == 0) {
            ld(b0, 0, v[0]);
        } else if constexpr (N == 1) {
            const int b1 = b0 + sz;
            ld_pair(b0, 0, v[0], v[1]);
            ld_pair(b0 + sy, 0, v[2], v[3]);
            ld_pair(b1, 0, v[4], v[5]);
            ld_pair(b1 + sy, 0, v[6], v[7]);
        } else {
            const int b1 = b0 + sz;
            ld_pair(b0, 0, v[0], v[1]);
            ld_pair(b0, sy, v[2], v[3]);
            ld_pair(b1, 0, v[4], v[5]);
            ld_pair(b1, sy, v[6], v[7]);
        }
    }
}

template <int N>
__device__ __forceinline__ float blend(const float (&c)[N], const float (&w)[3]) {
    if (N == 1) return c[0];
    const float c00 = fmaf(w[0], c[1] - c[0], c[0]);
    const float c10 = fmaf(w[0], c[3] - c[2], c[2]);
    const float c01 = fmaf(w[0], c[5] - c[4], c[4]);
    const float c11 = fmaf(w[0], c[7] - c[6], c[6]);
    const float c0 = fmaf(w[1], c10 - c00, c00);
    const float c1 = fmaf(w[1], c11 - c01, c01);
    return fmaf(w[2], c1 - c0, c0);
}

// ---------------------------------------------------------------------------
// Scan points.  point_generic evaluates one scan point with the runtime
// source loop (any sources); point<...> for a compile-time source signature,
// issuing every load before any is consumed (the source loop unrolled at
// compile time, as the paper does with template metaprogramming, Sec. 3.2).
// Both return the mixed premultiplied colour E and opacity S of the point and round alike at every step (the
// trilinear cell coordinates come from point_at and a subtraction of 1/2 in
// one, from cell_at in the other, which give the same numbers), so they give
// the same image bit for bit.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void mix_finish(float& S, float (&E)[3]) {
    if (S > 1.f) {
        const float inv = 1.f / S;
        E[0] *= inv;
        E[1] *= inv;
        E[2] *= inv;
        S = 1.f;
    }
}

template <int INTERP>
__device__ __forceinline__ void point_generic(const DevJob& J, const float4* __restrict__ s_tf, const RaySetup& R,
                                              int k, float (&E)[3], float& S) {
    const float tk = ((float)k + 0.5f) * (float)J.step;
    float p[3];
    point_at(J, R, tk, p);
    const int dims[3] = {J.dims[0], J.dims[1], J.dims[2]};
    S = 0.f;
    E[0] = E[1] = E[2] = 0.f;
    for (int s = 0; s < J.n_src; ++s) {
        const DevSource& src = J.src[s];
        const float x = sample_source<INTERP>(src, dims, p);
        const float4 c = classify(s_tf + s * kTfLds, x);
        const float wa = src.weight * c.w;
        S = fmaf(src.weight, c.w, S);
        E[0] = fmaf(wa, c.x, E[0]);
        E[1] = fmaf(wa, c.y, E[1]);
        E[2] = fmaf(wa, c.z, E[2]);
    }
    mix_finish(S, E);
}

// Cell indices and interpolation weights of scan point k (nearest: the clamped cell).
template <int INTERP>
__device__ __forceinline__ void locate(const DevJob& J, const RaySetup& R, int k, int (&i0)[3], float (&w)[3]) {
    float p[3];
    if (INTERP == 0) point_at(J, R, ((float)k + 0.5f) * (float)J.step, p);
    else cell_at(J, R, k, p);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (INTERP == 0) {
            i0[a] = clampi((int)floorf(p[a]), 0, J.dims[a] - 1);
            w[a] = 0.f;
        } else {
            const float fl = floorf(p[a]);
            w[a] = p[a] - fl;
            i0[a] = (int)fl;
        }
    }
}

template <int SIG> struct SigKinds { static constexpr int k0 = K_NONE, k1 = K_NONE, k2 = K_NONE; };
template <> struct SigKinds<SIG_F32x1> { static constexpr int k0 = K_F32x1, k1 = K_NONE, k2 = K_NONE; };
template <> struct SigKinds<SIG_PIC3_F32> { static constexpr int k0 = K_F32x1, k1 = K_F32x3, k2 = K_F32x3; };
template <> struct SigKinds<SIG_PIC3_F16> { static constexpr int k0 = K_F16x1, k1 = K_F16x3, k2 = K_F16x3; };
template <> struct SigKinds<SIG_PIC3_BF16> { static constexpr int k0 = K_BF16x1, k1 = K_BF16x3, k2 = K_BF16x3; };

// PS (per source): load, chain, blend and classify one source before the
// next one's loads; fewer live registers (more resident waves) at the cost of
// one memory round trip per source.  Same arithmetic either way.
template <int INTERP, int SIG, bool PS>
__device__ __forceinline__ void point(const DevJob& J, const float4* __restrict__ s_tf, const RaySetup& R, int k,
                                      float (&E)[3], float& S) {
    if constexpr (SIG == SIG_GENERIC) {
        point_generic<INTERP>(J, s_tf, R, k, E, S);
    } else {
        constexpr int K0 = SigKinds<SIG>::k0, K1 = SigKinds<SIG>::k1, K2 = SigKinds<SIG>::k2;
        constexpr int KS[3] = {K0, K1, K2};
        constexpr int NV = INTERP ? 8 : 1;
        constexpr int NS = (K0 != K_NONE) + (K1 != K_NONE) + (K2 != K_NONE);
        // the host admits the three-source signatures only with guard layers: no border clamp
        constexpr bool CL = SIG == SIG_F32x1;
        constexpr bool kHalf = (SIG == SIG_PIC3_F16 || SIG == SIG_PIC3_BF16) && INTERP != 0;
        const int dims[3] = {J.dims[0], J.dims[1], J.dims[2]};
        int i0[3];
        float w[3];
        locate<INTERP>(J, R, k, i0, w);
        S = 0.f;
        E[0] = E[1] = E[2] = 0.f;
        auto accumulate = [&](int s, float x) {
            const float4 cl = classify(s_tf + s * kTfLds, x);
            const float wa = J.src[s].weight * cl.w;
            S = fmaf(J.src[s].weight, cl.w, S);
            E[0] = fmaf(wa, cl.x, E[0]);
            E[1] = fmaf(wa, cl.y, E[1]);
            E[2] = fmaf(wa, cl.z, E[2]);
        };
        if constexpr (Il<SIG>::n > 0) {
            // the values of a voxel are adjacent
            float v[NV][4];
            fetch_il<INTERP, SIG>(J.src[0], dims, i0, v);
#pragma unroll
            for (int s = 0; s < Il<SIG>::n; ++s) {
                float c[NV];
#pragma unroll
                for (int i = 0; i < NV; ++i) c[i] = v[i][s];
                accumulate(s, blend<NV>(c, w));
            }
        } else if (kHalf && J.src[0].stride[0] == 2 && J.src[1].stride[0] == 6 && J.src[2].stride[0] == 6) {
            if constexpr (kHalf) {
                constexpr int T = KindOf<K0>::dtype;
                HalfPairs<1> h0;
                HalfPairs<3> h1, h2;
                int off[8];
                corner_offsets<INTERP, CL>(J.src[0], dims, i0, off);
                load_half_pairs(J.src[0], off, h0);
                corner_offsets<INTERP, CL>(J.src[1], dims, i0, off);
                load_half_pairs(J.src[1], off, h1);
                corner_offsets<INTERP, CL>(J.src[2], dims, i0, off);
                load_half_pairs(J.src[2], off, h2);
                float v[8][4], c[8];
                unpack_half_pairs<1, T>(h0, v);
                run_chain<8, 1>(J.src[0], v, c);
                accumulate(0, blend<8>(c, w));
                unpack_half_pairs<3, T>(h1, v);
                run_chain<8, 3>(J.src[1], v, c);
                accumulate(1, blend<8>(c, w));
                unpack_half_pairs<3, T>(h2, v);
                run_chain<8, 3>(J.src[2], v, c);
                accumulate(2, blend<8>(c, w));
            }
        } else if constexpr (PS) {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                int off[NV];
                float v[NV][4], c[NV];
                corner_offsets<INTERP, CL>(J.src[s], dims, i0, off);
                if (s == 0) fetch_kind<KS[0], NV>(J.src[0], off, v);
                else if (s == 1) fetch_kind<KS[1], NV>(J.src[1], off, v);
                else fetch_kind<KS[2], NV>(J.src[2], off, v);
                if (s == 0) run_chain<NV, KindOf<KS[0]>::dim>(J.src[0], v, c);
                else if (s == 1) run_chain<NV, KindOf<KS[1]>::dim>(J.src[1], v, c);
                else run_chain<NV, KindOf<KS[2]>::dim>(J.src[2], v, c);
                accumulate(s, blend<NV>(c, w));
            }
        } else {
            // every source's loads first, then chains, interpolation, classification
            float vals[3][NV][4];
            int off[NV];
            if (NS > 0) {
                corner_offsets<INTERP, CL>(J.src[0], dims, i0, off);
                // an FP32 scalar whose x neighbours are adjacent: both in one load
                bool pairs = false;
                if constexpr (SIG == SIG_PIC3_F32 && INTERP != 0) {
                    pairs = J.src[0].stride[0] == 4;
                    if (pairs) fetch_f32_pairs(J.src[0], off, vals[0]);
                }
                if (!pairs) fetch_kind<K0, NV>(J.src[0], off, vals[0]);
            }
            if (NS > 1) {
                corner_offsets<INTERP, CL>(J.src[1], dims, i0, off);
                fetch_kind<K1, NV>(J.src[1], off, vals[1]);
            }
            if (NS > 2) {
                corner_offsets<INTERP, CL>(J.src[2], dims, i0, off);
                fetch_kind<K2, NV>(J.src[2], off, vals[2]);
            }
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                float c[NV];
                if (s == 0) run_chain<NV, KindOf<KS[0]>::dim>(J.src[0], vals[0], c);
                else if (s == 1) run_chain<NV, KindOf<KS[1]>::dim>(J.src[1], vals[1], c);
                else run_chain<NV, KindOf<KS[2]>::dim>(J.src[2], vals[2], c);
                accumulate(s, blend<NV>(c, w));
            }
        }
        mix_finish(S, E);
    }
}

// A row of G points, one per lane of the group (G = 4: a quad, G = 16: a row of
// lanes), composited in order onto (C0, C1, C2, A), on every lane of the group:
// per point T = 1 - A and four fused multiply-adds that take the point's lane by
// DPP (quad_perm, row_newbcast).  In assembly, 5 instructions per point: the
// compiler does not fold a broadcast into fmac and issues 9.  The nop keeps the
// wait states a DPP read needs after a write of its source or of EXEC; nothing
// inside writes either.
#define ISAAC_OVER(DPP)                                                              \
    "v_sub_f32 %4, 1.0, %3\n\t"                                                      \
    "v_fmac_f32_dpp %0, %5, %4 " DPP " row_mask:0xf bank_mask:0xf\n\t"               \
    "v_fmac_f32_dpp %1, %6, %4 " DPP " row_mask:0xf bank_mask:0xf\n\t"               \
    "v_fmac_f32_dpp %2, %7, %4 " DPP " row_mask:0xf bank_mask:0xf\n\t"               \
    "v_fmac_f32_dpp %3, %8, %4 " DPP " row_mask:0xf bank_mask:0xf\n\t"
template <int G>
__device__ __forceinline__ void over_in_order(const float (&E)[3], float S, float& C0, float& C1, float& C2, float& A) {
    static_assert(G == 4 || G == 16, "a quad or a row");
    float t;
    if constexpr (G == 4) {
        asm("s_nop 4\n\t"
            ISAAC_OVER("quad_perm:[0,0,0,0]") ISAAC_OVER("quad_perm:[1,1,1,1]")
            ISAAC_OVER("quad_perm:[2,2,2,2]") ISAAC_OVER("quad_perm:[3,3,3,3]")
            : "+&v"(C0), "+&v"(C1), "+&v"(C2), "+&v"(A), "=&v"(t)
            : "v"(E[0]), "v"(E[1]), "v"(E[2]), "v"(S));
    } else {
        asm("s_nop 4\n\t"
            ISAAC_OVER("row_newbcast:0") ISAAC_OVER("row_newbcast:1") ISAAC_OVER("row_newbcast:2")
            ISAAC_OVER("row_newbcast:3") ISAAC_OVER("row_newbcast:4") ISAAC_OVER("row_newbcast:5")
            ISAAC_OVER("row_newbcast:6") ISAAC_OVER("row_newbcast:7") ISAAC_OVER("row_newbcast:8")
            ISAAC_OVER("row_newbcast:9") ISAAC_OVER("row_newbcast:10") ISAAC_OVER("row_newbcast:11")
            ISAAC_OVER("row_newbcast:12") ISAAC_OVER("row_newbcast:13") ISAAC_OVER("row_newbcast:14")
            ISAAC_OVER("row_newbcast:15")
            : "+&v"(C0), "+&v"(C1), "+&v"(C2), "+&v"(A), "=&v"(t)
            : "v"(E[0]), "v"(E[1]), "v"(E[2]), "v"(S));
    }
}
#undef ISAAC_OVER

// One lane per ray: its scan points one after another, front to back, to the first
// whose opacity reaches ert.  For launches of many rays that end after a few points:
// a row of points evaluated together (below) is mostly wasted on those, and the
// groups' waves are so many that starting them is the time (an opaque scalar at 1920 x
// 1080: 25 us a call against 44 with 16 lanes, 29 with 4; at 4K 46 against 58 with 4).
template <int INTERP, int SIG, bool PS>
__device__ __forceinline__ void march_one(const DevJob& J, const float4* __restrict__ s_tf, const RaySetup& R,
                                          float4& out, int& count) {
    float C0 = 0.f, C1 = 0.f, C2 = 0.f, A = 0.f;
    int n = 0;
    for (int k = R.kb; k < R.ke; ++k) {
        float E[3], S;
        point<INTERP, SIG, PS>(J, s_tf, R, k, E, S);
        const float T = 1.f - A;
        C0 = fmaf(E[0], T, C0);
        C1 = fmaf(E[1], T, C1);
        C2 = fmaf(E[2], T, C2);
        A = fmaf(S, T, A);
        ++n;
        if (A >= J.ert) break;
    }
    out = make_float4(C0, C1, C2, A);
    count = n;
}

// One lane per ray as far as the image goes: the scan points of a ray are
// composited one after another, front to back, with early termination at the
// first whose opacity reaches ert.  They are evaluated by a group of G lanes, a
// row of G points at a time (a lane alone on a ray waits for one gather after
// another, and a frame's rays are too few to fill the chip with one lane each);
// every lane of the group then composites the row in order, so the arithmetic,
// and the image, are those of a single lane.  Opacities do not decrease along
// a row, so a row whose last opacity is below ert holds no termination; the one
// row of a ray that does is composited again point by point.  A point past the
// ray's end has E = S = 0, which changes nothing.  Against a lane of its own per
// ray, which waited on one gather after another (144 waves for 256^2 pixels): one
// 64^3 scalar at 256^2 67 -> 23 us a call, three sources read in place at 512 x 300
// 910 -> 88, four derived at 720p 689 -> 129, one scalar at 4K 1395 -> 503.
template <int INTERP, int G, int SIG, bool PS>
__device__ __forceinline__ void march_ordered(const DevJob& J, const float4* __restrict__ s_tf, const RaySetup& R,
                                              int lane, float4& out, int& count) {
    const int g = lane & (G - 1);
    float C0 = 0.f, C1 = 0.f, C2 = 0.f, A = 0.f;
    int n = 0;
    for (int k0 = R.kb; k0 < R.ke; k0 += G) {
        const int k = k0 + g;
        const bool valid = k < R.ke;
        float E[3], S;
        point<INTERP, SIG, PS>(J, s_tf, R, valid ? k : R.ke - 1, E, S);
        if (!valid) E[0] = E[1] = E[2] = S = 0.f;
        float N0 = C0, N1 = C1, N2 = C2, NA = A;
        over_in_order<G>(E, S, N0, N1, N2, NA);
        if (NA >= J.ert) {
            for (int j = 0; j < G; ++j) {
                const float T = 1.f - A;
                C0 = fmaf(__shfl(E[0], j, G), T, C0);
                C1 = fmaf(__shfl(E[1], j, G), T, C1);
                C2 = fmaf(__shfl(E[2], j, G), T, C2);
                A = fmaf(__shfl(S, j, G), T, A);
                ++n;
                if (A >= J.ert) break;
            }
            break;
        }
        C0 = N0;
        C1 = N1;
        C2 = N2;
        A = NA;
        n += min(G, R.ke - k0);
    }
    out = make_float4(C0, C1, C2, A);
    count = n;
}

// Value of the lane D below inside a row of 16 lanes (DPP row_shr:D); a lane
// whose source would lie in another row reads 0.
template <int D>
__device__ __forceinline__ float lane_up(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x110 + D, 0xF, 0xF,
                                                                 true));
}

// Running front-to-back state of one ray composited by a group of G lanes.
struct RayAccum {
    float C0, C1, C2, A;
    int n;
};

// Composite one row of G scan points (k0 .. k0+G-1; lane g holds point
// k0 + g, `valid` when below R.ke) into acc: an inclusive scan of the
// front-to-back operator across the group, then termination at the first
// point whose cumulative opacity reaches ert.  Returns true when the ray is
// finished (termination, or no scan point left).
// Inclusive scan of the front-to-back operator over the G lanes of a group
// (lane g ends with the composite of lanes 0..g, lane 0 frontmost).
template <int G>
__device__ __forceinline__ void group_scan(int lane, float& c0, float& c1, float& c2, float& a) {
    const int g = lane & (G - 1);
    // inclusive scan inside each row of 16 lanes ...
#pragma unroll
    for (int d = 1; d < (G < 16 ? G : 16); d <<= 1) {
        float o0, o1, o2, oa;
        if (d == 1) {
            o0 = lane_up<1>(c0); o1 = lane_up<1>(c1); o2 = lane_up<1>(c2); oa = lane_up<1>(a);
        } else if (d == 2) {
            o0 = lane_up<2>(c0); o1 = lane_up<2>(c1); o2 = lane_up<2>(c2); oa = lane_up<2>(a);
        } else if (d == 4) {
            o0 = lane_up<4>(c0); o1 = lane_up<4>(c1); o2 = lane_up<4>(c2); oa = lane_up<4>(a);
        } else {
            o0 = lane_up<8>(c0); o1 = lane_up<8>(c1); o2 = lane_up<8>(c2); oa = lane_up<8>(a);
        }
        // with whole rows per group the shifted-in value of a row's first lanes
        // is 0 (bound_ctrl), the identity of the operator: no mask needed
        if (G >= 16 || (g & 15) >= d) {
            const float t = 1.f - oa;
            c0 = fmaf(t, c0, o0);
            c1 = fmaf(t, c1, o1);
            c2 = fmaf(t, c2, o2);
            a = fmaf(t, a, oa);
        }
    }
    // ... then each row appends the total of the rows before it in its group
    // (the last lane of the row below, after that row's own update)
#pragma unroll
    for (int r = 16; r < G; r <<= 1) {
        const int src = (lane & ~(2 * r - 1)) + r - 1;
        const float o0 = __shfl(c0, src, 64), o1 = __shfl(c1, src, 64), o2 = __shfl(c2, src, 64);
        const float oa = __shfl(a, src, 64);
        if (g & r) {
            const float t = 1.f - oa;
            c0 = fmaf(t, c0, o0);
            c1 = fmaf(t, c1, o1);
            c2 = fmaf(t, c2, o2);
            a = fmaf(t, a, oa);
        }
    }
}

// The lane index, opaque to the optimizer: masks and permute addresses made from
// it inside a loop are recomputed there (one instruction each) instead of held in
// registers through it.  k0 (the loop's) keeps it in the loop; volatile would too, but
// counts as a write to memory and keeps the job's fields from being read once
// before the loop.
__device__ __forceinline__ int fresh(int lane, int k0) {
    asm("" : "+v"(lane) : "v"(k0));
    return lane;
}

// One row of G scan points of a ray composited into acc.  A lane past the ray's
// last scan point (valid false) may carry any finite values (the callers give it
// the last point's sample): the scan is inclusive, so no kept lane's prefix
// depends on it, the termination ballot masks it, and the lane taken is never
// past the row's last kept point.
template <int G>
__device__ __forceinline__ bool row_composite(const DevJob& J, const RaySetup& R, int lane, int k0, bool valid,
                                              float c0, float c1, float c2, float a, RayAccum& acc) {
    group_scan<G>(lane, c0, c1, c2, a);
    const float T = 1.f - acc.A;
    const float n0 = fmaf(T, c0, acc.C0), n1 = fmaf(T, c1, acc.C1), n2 = fmaf(T, c2, acc.C2), na = fmaf(T, a, acc.A);
    const unsigned long long m = __builtin_amdgcn_ballot_w64(na >= J.ert) & __builtin_amdgcn_ballot_w64(valid);
    constexpr unsigned long long kGroupMask = G == 64 ? ~0ull : ((1ull << (G & 63)) - 1ull);
    const int first = fresh(lane, k0) & ~(G - 1);
    const unsigned long long bits = (m >> first) & kGroupMask;
    const bool stop = bits != 0;
    // the first terminating point, else the row's last kept one (k0 < R.ke, so
    // last >= 0; every set bit belongs to a kept point, i.e. lies at or below last)
    const int last = min(G, R.ke - k0) - 1;
    int sel;
    if constexpr (G <= 32) sel = __builtin_ctz((unsigned)bits | (1u << last));
    else sel = __builtin_ctzll(bits | (1ull << last));
    acc.n += sel + 1;
    auto from = [&](float x) {
        return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((first + sel) << 2, __builtin_bit_cast(int, x)));
    };
    acc.C0 = from(n0);
    acc.C1 = from(n1);
    acc.C2 = from(n2);
    acc.A = from(na);
    return stop || k0 + G >= R.ke;
}

// One row of the lanes-per-ray schedule: scan points k0 .. k0+G-1 (those
// below R.ke), composited into acc.  Returns true when the ray is finished.
template <int INTERP, int G, int SIG, bool PS>
__device__ __forceinline__ bool lanes_row(const DevJob& J, const float4* __restrict__ s_tf, const RaySetup& R,
                                          int lane, int k0, RayAccum& acc) {
    const int k = k0 + (fresh(lane, k0) & (G - 1));
    const bool valid = k < R.ke;
    float E[3], S;
    point<INTERP, SIG, PS>(J, s_tf, R, valid ? k : R.ke - 1, E, S);
    return row_composite<G>(J, R, lane, k0, valid, E[0], E[1], E[2], S, acc);
}

// Plain values side by side (Il<SIG>), G lanes per ray, software-pipelined:
// the corner loads of a lane's next scan point are issued before the current
// one is blended, classified and composited, so a row's memory latency
// overlaps the previous row's arithmetic.  The arithmetic is that of
// lanes_row, operation for operation.
template <int NV, int N>
__device__ __forceinline__ void il_mix(const DevJob& J, const float4* __restrict__ s_tf, const float (&v)[NV][4],
                                        const float (&w)[3], float (&E)[3], float& S) {
    S = 0.f;
    E[0] = E[1] = E[2] = 0.f;
#pragma unroll
    for (int s = 0; s < N; ++s) {
        float c[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i) c[i] = v[i][s];
        const float4 cl = classify(s_tf + s * kTfLds, blend<NV>(c, w));
        const float wa = J.src[s].weight * cl.w;
        S = fmaf(J.src[s].weight, cl.w, S);
        E[0] = fmaf(wa, cl.x, E[0]);
        E[1] = fmaf(wa, cl.y, E[1]);
        E[2] = fmaf(wa, cl.z, E[2]);
    }
    mix_finish(S, E);
}

template <int INTERP, int G, int SIG>
__device__ __forceinline__ void march_lanes_il(const DevJob& J, const float4* __restrict__ s_tf, const RaySetup& R,
                                               int lane, float4& out, int& count) {
    constexpr int NV = INTERP ? 8 : 1;
    const int dims[3] = {J.dims[0], J.dims[1], J.dims[2]};
    const int g = lane & (G - 1);
    int i0[3];
    float w[3], v[NV][4];
    locate<INTERP>(J, R, min(R.kb + g, R.ke - 1), i0, w);
    fetch_il<INTERP, SIG>(J.src[0], dims, i0, v);
    RayAccum acc = {0.f, 0.f, 0.f, 0.f, 0};
    for (int k0 = R.kb;; k0 += G) {
        // the next row's loads (clamped to the last scan point: always in bounds)
        int i0n[3];
        float wn[3], vn[NV][4];
        locate<INTERP>(J, R, min(k0 + G + g, R.ke - 1), i0n, wn);
        fetch_il<INTERP, SIG>(J.src[0], dims, i0n, vn);
        const bool valid = k0 + g < R.ke;
        float E[3], S;
        il_mix<NV, Il<SIG>::n>(J, s_tf, v, w, E, S);
        if (row_composite<G>(J, R, lane, k0, valid, E[0], E[1], E[2], S, acc))
            break;
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int c = 0; c < Il<SIG>::n; ++c) v[i][c] = vn[i][c];
        w[0] = wn[0];
        w[1] = wn[1];
        w[2] = wn[2];
    }
    out = make_float4(acc.C0, acc.C1, acc.C2, acc.A);
    count = acc.n;
}

// G lanes per ray: lane g evaluates scan points kb + g, kb + g + G, ...; each
// row of G points is composited in order with an inclusive scan of the
// associative front-to-back operator (C, A) o (C', A') = (C + (1-A) C',
// A + (1-A) A') across the group, then appended to the ray's running state.
// The first point whose cumulative opacity reaches ert ends the ray, exactly
// where the one-lane loop would stop.
template <int INTERP, int G, int SIG, bool PS>
__device__ __forceinline__ void march_lanes(const DevJob& J, const float4* __restrict__ s_tf, const RaySetup& R,
                                            int lane, float4& out, int& count) {
    RayAccum acc = {0.f, 0.f, 0.f, 0.f, 0};
    for (int k0 = R.kb;; k0 += G)
        if (lanes_row<INTERP, G, SIG, PS>(J, s_tf, R, lane, k0, acc)) break;
    out = make_float4(acc.C0, acc.C1, acc.C2, acc.A);
    count = acc.n;
}

template <int INTERP, bool ORD, int G, int SIG, bool PS>
__device__ __forceinline__ void march_sig(const DevJob& J, const float4* __restrict__ s_tf, const RaySetup& R,
                                          int lane, float4& out, int& count) {
    if constexpr (ORD && G == 1) march_one<INTERP, SIG, PS>(J, s_tf, R, out, count);
    else if constexpr (ORD) march_ordered<INTERP, G, SIG, PS>(J, s_tf, R, lane, out, count);
    else if constexpr (Il<SIG>::n > 0 && !PS) march_lanes_il<INTERP, G, SIG>(J, s_tf, R, lane, out, count);
    else march_lanes<INTERP, G, SIG, PS>(J, s_tf, R, lane, out, count);
}

template <int INTERP, bool ORD, int G, bool PS>
__device__ __forceinline__ void march_dispatch(const DevJob& J, const float4* __restrict__ s_tf, const RaySetup& R,
                                               int lane, float4& out, int& count) {
    switch (J.sig) {
    case SIG_F32x1: march_sig<INTERP, ORD, G, SIG_F32x1, PS>(J, s_tf, R, lane, out, count); break;
    case SIG_PIC3_F32: march_sig<INTERP, ORD, G, SIG_PIC3_F32, PS>(J, s_tf, R, lane, out, count); break;
    case SIG_PIC3_F16: march_sig<INTERP, ORD, G, SIG_PIC3_F16, PS>(J, s_tf, R, lane, out, count); break;
    case SIG_PIC3_BF16: march_sig<INTERP, ORD, G, SIG_PIC3_BF16, PS>(J, s_tf, R, lane, out, count); break;
    case SIG_IL3: march_sig<INTERP, ORD, G, SIG_IL3, PS>(J, s_tf, R, lane, out, count); break;
    case SIG_IL3P: march_sig<INTERP, ORD, G, SIG_IL3P, PS>(J, s_tf, R, lane, out, count); break;
    case SIG_IL1: march_sig<INTERP, ORD, G, SIG_IL1, PS>(J, s_tf, R, lane, out, count); break;
    case SIG_IL1C: march_sig<INTERP, ORD, G, SIG_IL1C, PS>(J, s_tf, R, lane, out, count); break;
    case SIG_IL2: march_sig<INTERP, ORD, G, SIG_IL2, PS>(J, s_tf, R, lane, out, count); break;
    case SIG_IL4: march_sig<INTERP, ORD, G, SIG_IL4, PS>(J, s_tf, R, lane, out, count); break;
    default: march_sig<INTERP, ORD, G, SIG_GENERIC, PS>(J, s_tf, R, lane, out, count); break;
    }
}

// Iso-surface mode (a listed feature, Sec. 3; the paper gives no algorithm):
// the first place where a source's interpolated chain output crosses its iso
// value between two consecutive scan points, placed by linear interpolation
// between them; opaque, coloured by the source's table at the iso value and
// lit by a headlight, 0.3 + 0.7 |cos| of the angle between the ray and the
// central-difference gradient (half a voxel each side).  The source loop is
// uniform, so every source's buffer resource stays scalar.
// The crossing of source s between scan points k - 1 and k, at fraction f of
// the step: opaque, the source's table colour at its iso value lit by a
// headlight from the central-difference gradient (half a voxel each side).
// s must be wave-uniform (the source's buffer resource is scalar).
template <int INTERP, bool PLAIN>
__device__ __forceinline__ float4 iso_shade(const DevJob& J, const float4* __restrict__ s_tf, const RaySetup& R,
                                            int s, int k, float f) {
    // no contraction: (k + 1/2) step - tp is rounded as written wherever this is inlined
#pragma clang fp contract(off)
    const int dims[3] = {J.dims[0], J.dims[1], J.dims[2]};
    const float step = (float)J.step;
    const DevSource& S = J.src[s];
    const float tp = ((float)(k - 1) + 0.5f) * step;
    const float ts = fmaf(f, ((float)k + 0.5f) * step - tp, tp);
    float q[3];
    point_at(J, R, ts, q);
    float g[3] = {0.f, 0.f, 0.f};
#pragma unroll 1
    for (int a = 0; a < 3; ++a) {           // one axis at a time keeps register use low
        const float hx = a == 0 ? 0.5f : 0.f, hy = a == 1 ? 0.5f : 0.f, hz = a == 2 ? 0.5f : 0.f;
        const float qp[3] = {q[0] + hx, q[1] + hy, q[2] + hz}, qm[3] = {q[0] - hx, q[1] - hy, q[2] - hz};
        const float d = sample_any<INTERP, PLAIN>(S, dims, qp) - sample_any<INTERP, PLAIN>(S, dims, qm);
        g[0] = a == 0 ? d : g[0];
        g[1] = a == 1 ? d : g[1];
        g[2] = a == 2 ? d : g[2];
    }
    const float gl = sqrtf(fmaf(g[0], g[0], fmaf(g[1], g[1], g[2] * g[2])));
    const float cosine = gl > 0.f ? fabsf(fmaf(g[0], R.d[0], fmaf(g[1], R.d[1], g[2] * R.d[2]))) / gl : 1.f;
    const float light = fmaf(0.7f, fminf(cosine, 1.f), 0.3f);
    const float4 c = classify(s_tf + s * kTfLds, S.iso);
    return make_float4(c.x * light, c.y * light, c.z * light, 1.f);
}

// G lanes per ray: lane g takes scan point k0 + g of each row of G points; its
// predecessor's values come from lane g - 1 (lane 0: the last point of the row
// before), so every lane tests its own pair of consecutive points at once and
// the ray's crossing is the first lane (then the first source in index order)
// that sees one: the point, source and fraction the one-lane loop finds, with
// the same arithmetic, in a fraction of its dependent steps (G = 1 is that loop,
// for launches of many short rays).  The crossing's lane shades, and passes colour
// and count to the group's first lane.
template <int INTERP, int G, bool PLAIN>
__device__ __forceinline__ void march_iso_lanes(const DevJob& J, const float4* __restrict__ s_tf,
                                                const RaySetup& R, int lane, float4& out, int& count) {
    const int dims[3] = {J.dims[0], J.dims[1], J.dims[2]};
    const float step = (float)J.step;
    const int g = lane & (G - 1), base = lane & ~(G - 1);
    constexpr unsigned long long kGroupMask = G == 64 ? ~0ull : ((1ull << (G & 63)) - 1ull);
    float carry[kMaxSources] = {};              // values at the last point of the previous row
    int sel = -1, my_s = -1, k = R.kb;
    float my_f = 0.f;
    for (int k0 = R.kb;; k0 += G) {
        k = k0 + g;
        const bool valid = k < R.ke;
        float p[3];
        point_at(J, R, ((float)(valid ? k : R.ke - 1) + 0.5f) * step, p);
        for (int s = 0; s < J.n_src; ++s) {
            const DevSource& S = J.src[s];
            const float x = sample_any<INTERP, PLAIN>(S, dims, p);
            float prev = carry[s];
            if constexpr (G > 1) {
                const float below = __shfl(x, base + ((g + G - 1) & (G - 1)), 64);
                if (g > 0) prev = below;
            }
            if (my_s < 0 && valid && k > R.kb && ((prev >= S.iso) != (x >= S.iso))) {
                my_s = s;
                my_f = (S.iso - prev) / (x - prev);
            }
            carry[s] = G > 1 ? __shfl(x, base + G - 1, 64) : x;
        }
        const unsigned long long bits = (__builtin_amdgcn_ballot_w64(my_s >= 0) >> base) & kGroupMask;
        if (bits) {
            sel = (int)__builtin_ctzll(bits);
            count = k0 + sel - R.kb + 1;
            break;
        }
        if (k0 + G >= R.ke) {
            count = R.ke - R.kb;
            break;
        }
    }
    // shade one source at a time: the source must be the same on every active lane
    // (its buffer resource is read as wave-uniform), whatever surface each ray found
    float4 c = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s = 0; s < J.n_src; ++s)
        if (g == sel && my_s == s) c = iso_shade<INTERP, PLAIN>(J, s_tf, R, s, k, my_f);
    const int src = base + (sel >= 0 ? sel : 0);
    out = make_float4(__shfl(c.x, src, 64), __shfl(c.y, src, 64), __shfl(c.z, src, 64), __shfl(c.w, src, 64));
}

__device__ __forceinline__ int find_job(const DevJob* __restrict__ jobs, int n_jobs, int tile) {
    int lo = 0, hi = n_jobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].tile_begin <= tile) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// First pixel of tile t of job J (G lanes share one ray), the same for the workgroup.
template <int G>
__device__ __forceinline__ void tile_origin(const DevJob& J, int t, int& x0, int& y0) {
    const int ty = t / J.tiles_x, tx = t - ty * J.tiles_x;
    x0 = __builtin_amdgcn_readfirstlane(J.cull[0] + tx * (J.wave_w * J.waves_x));
    y0 = __builtin_amdgcn_readfirstlane(J.cull[1] + ty * ((64 / G) / J.wave_w * (4 / J.waves_x)));
}

// Pixel of a thread in the tile at (x0, y0); false outside the image.  The widths are
// powers of two: shifts and masks, since every lane does this twice (as divisions it
// was some 140 instructions a time, 3 us of a frame of 21 thousand waves).
template <int G>
__device__ __forceinline__ bool pixel_of(const DevJob& J, int x0, int y0, int thread, int& px, int& py) {
    const int ray = (thread & 63) / G, wave = thread >> 6;
    const int w = __builtin_ctz(J.wave_w), h = __builtin_ctz(64 / G) - w, x = __builtin_ctz(J.waves_x);
    px = x0 + ((wave & (J.waves_x - 1)) << w) + (ray & (J.wave_w - 1));
    py = y0 + ((wave >> x) << h) + (ray >> w);
    return px <= J.cull[2] && py <= J.cull[3];
}

// Staging of a workgroup's transfer tables in LDS, a value per thread and source:
// the first three loaded to registers ahead, any others when they are stored.
struct StagedTables {
    float4 t0, t1, t2;
};

__device__ __forceinline__ float4 table_entry(const DevJob& J, const float4* __restrict__ tf_pool, int s) {
    static_assert(kBlockThreads == kTfEntries, "one table entry per thread");
    return tf_pool[(size_t)J.src[s].tf_slot * kTfEntries + threadIdx.x];
}

__device__ __forceinline__ StagedTables load_tables(const DevJob& J, const float4* __restrict__ tf_pool) {
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    StagedTables t;
    t.t0 = J.n_src > 0 ? table_entry(J, tf_pool, 0) : zero;
    t.t1 = J.n_src > 1 ? table_entry(J, tf_pool, 1) : zero;
    t.t2 = J.n_src > 2 ? table_entry(J, tf_pool, 2) : zero;
    return t;
}

__device__ __forceinline__ void store_tables(const DevJob& J, const float4* __restrict__ tf_pool,
                                             const StagedTables& t, float4* __restrict__ s_tf) {
    auto put = [&](int s, const float4& v) {
        s_tf[s * kTfLds + threadIdx.x] = v;
        if (threadIdx.x == kTfEntries - 1) s_tf[s * kTfLds + kTfEntries] = v;   // the last entry's copy
    };
    if (J.n_src > 0) put(0, t.t0);
    if (J.n_src > 1) put(1, t.t1);
    if (J.n_src > 2) put(2, t.t2);
    for (int s = 3; s < J.n_src; ++s) put(s, table_entry(J, tf_pool, s));
}

// One workgroup per tile, for one job or the tiles of many.  (Batches once ran a
// resident set of workgroups over a tile queue, to stage a job's tables once for
// many tiles: 1303 against 1256 us a call for 64 sub-volumes, 533 against 439 us for
// six served requests of one volume, 2 % the other way for 40 small ones.)
// Waves-per-SIMD hint: W = 0 leaves register allocation to the compiler and
// issues every load of a scan point at once; W > 0 asks for at least W
// resident waves per SIMD and evaluates the sources one after another.  The
// pipelined loop over one adjacent value and, bound, the loop over three fit the 64
// vector registers of 8 waves, since what a row needs of the lane index is made
// afresh (fresh()) and the pixel is not kept through the loop.
// SIGK >= 0: the kernel runs only that source signature (every job of the
// launch has it); SIGK = -1: it dispatches on each job's signature; SIGK = -2:
// iso-surface jobs; SIGK = -3: iso-surface jobs whose sources are all plain
// (sample_plain).
template <bool ORD, int G, int W, int SIGK>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(W > 0 ? W : 1, 8)))
void raycast_kernel(const DevJob* __restrict__ jobs, const float4* __restrict__ tf_pool, int n_jobs, int tile0) {
    extern __shared__ float4 s_tf[];
    const int lane = threadIdx.x & 63;
    const int tile = tile0 + (int)blockIdx.x;
    const int job = __builtin_amdgcn_readfirstlane(find_job(jobs, n_jobs, tile));
    const DevJob& J = jobs[job];
    // Loops over adjacent values: the tables travel while the ray record does, whether a
    // ray of the tile meets the box or not, so a workgroup waits for memory once before
    // its rows, not for the record, then for the tables (a wave lives 8.6 us on the
    // average; 8 bricks at 1920 x 1080 526 -> 517 us a call).  The longer loops over
    // sources in place (272 against 274 us) stage for the tiles that need them.
    constexpr bool kEarly = Il<SIGK>::n > 0;
    StagedTables tab;
    if constexpr (kEarly) tab = load_tables(J, tf_pool);
    // tiles cover the box's screen rectangle only (the fill kernel clears the rest)
    int x0, y0, px, py;
    const int t = tile - J.tile_begin;
    tile_origin<G>(J, SIGK <= -2 ? job_tile(t, job, J.tiles_x * J.tiles_y) : t, x0, y0);
    const bool in_image = pixel_of<G>(J, x0, y0, (int)threadIdx.x, px, py);
    RaySetup R;
    bool hit;
    if (J.rays) {
        // set up by the prepass, one lane per ray
        hit = false;
        if (in_image) {
            const int rw = J.cull[2] - J.cull[0] + 1;
            const RayRec& rr = static_cast<const RayRec*>(J.rays)[(py - J.cull[1]) * rw + (px - J.cull[0])];
            R.kb = rr.kb;
            R.ke = rr.ke;
            hit = R.kb < R.ke;
            if (hit) {
                for (int a = 0; a < 3; ++a) {
                    R.pb[a] = rr.pb[a];
                    R.d[a] = rr.d[a];
                }
                R.t_first = rr.t_first;
            }
        }
    } else {
        hit = in_image && setup_ray(J, px, py, R);
    }
    if (J.out_depth && in_image && (lane & (G - 1)) == 0)
        J.out_depth[(size_t)py * J.width + px] = hit ? R.t_first : __builtin_inff();
    if constexpr (kEarly) {
        store_tables(J, tf_pool, tab, s_tf);
        __syncthreads();
    } else if (__syncthreads_or(hit)) {
        store_tables(J, tf_pool, load_tables(J, tf_pool), s_tf);
        __syncthreads();
    }
    float4 c = make_float4(0.f, 0.f, 0.f, 0.f);
    int count = 0;
    if (hit) {
        if constexpr (SIGK == -2 || SIGK == -3) {
            constexpr bool PL = SIGK == -3;
            if (J.interp) march_iso_lanes<1, G, PL>(J, s_tf, R, lane, c, count);
            else march_iso_lanes<0, G, PL>(J, s_tf, R, lane, c, count);
        } else if constexpr (SIGK < 0) {
            if (J.interp) march_dispatch<1, ORD, G, (W > 0)>(J, s_tf, R, lane, c, count);
            else march_dispatch<0, ORD, G, (W > 0)>(J, s_tf, R, lane, c, count);
        } else {
            if (J.interp) march_sig<1, ORD, G, SIGK, (W > 0)>(J, s_tf, R, lane, c, count);
            else march_sig<0, ORD, G, SIGK, (W > 0)>(J, s_tf, R, lane, c, count);
        }
    }
    // the pixel again, from the thread index: nothing of it stays in registers
    // through the loop above
    int tid = (int)threadIdx.x;
    asm("" : "+v"(tid));
    if (pixel_of<G>(J, x0, y0, tid, px, py) && (tid & (G - 1)) == 0) {
        const size_t pix = (size_t)py * J.width + px;
        reinterpret_cast<float4*>(J.out)[pix] = c;
        if (J.out_samples) J.out_samples[pix] = count;
    }
}

// ---------------------------------------------------------------------------
// Pooled schedule (one job).  ray_setup_kernel sets up every pixel's ray and
// appends the rays that keep scan points to a compact list (the others get
// their empty output at once); raycast_pool_kernel keeps its waves resident
// and hands the listed rays to groups of G lanes as groups free up, so a
// wave's lanes stay busy whatever the lengths of its rays.  Each ray is
// composited row by row exactly as in the tiled schedule with G lanes per ray.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void ray_setup_kernel(const DevJob* __restrict__ jobs, RayRec* __restrict__ rays,
                                                        int* __restrict__ counters) {
    const DevJob& J = jobs[0];
    const int px = (int)(blockIdx.x * 16 + (threadIdx.x & 15));
    const int py = (int)(blockIdx.y * 16 + (threadIdx.x >> 4));
    const bool in_image = px < J.width && py < J.height;
    const bool in_rect = px >= J.cull[0] && px <= J.cull[2] && py >= J.cull[1] && py <= J.cull[3];
    RaySetup R;
    const bool hit = in_image && in_rect && setup_ray(J, px, py, R);
    // one append per wave
    const unsigned long long m = __ballot(hit);
    const int lane = (int)(threadIdx.x & 63);
    int base = 0;
    if (m) {
        const int first = __builtin_ctzll(m);
        if (lane == first) base = atomicAdd(&counters[0], __popcll(m));
        base = __shfl(base, first);
    }
    const size_t pix = (size_t)py * J.width + px;
    if (hit) {
        const int slot =
            base + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
        RayRec r;
        for (int a = 0; a < 3; ++a) {
            r.pb[a] = R.pb[a];
            r.d[a] = R.d[a];
        }
        r.kb = R.kb;
        r.ke = R.ke;
        r.t_first = R.t_first;
        r.pixel = (int)pix;
        rays[slot] = r;
    } else if (in_image) {
        reinterpret_cast<float4*>(J.out)[pix] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (J.out_samples) J.out_samples[pix] = 0;
        if (J.out_depth) J.out_depth[pix] = __builtin_inff();
    }
}

template <int INTERP, int G, int SIGK, bool PS>
__device__ __forceinline__ bool pool_row(const DevJob& J, const float4* __restrict__ s_tf, const RaySetup& R, int lane,
                                         int k0, RayAccum& acc) {
    if constexpr (SIGK >= 0) {
        return lanes_row<INTERP, G, SIGK, PS>(J, s_tf, R, lane, k0, acc);
    } else {
        switch (J.sig) {
        case SIG_F32x1: return lanes_row<INTERP, G, SIG_F32x1, PS>(J, s_tf, R, lane, k0, acc);
        case SIG_PIC3_F32: return lanes_row<INTERP, G, SIG_PIC3_F32, PS>(J, s_tf, R, lane, k0, acc);
        case SIG_PIC3_F16: return lanes_row<INTERP, G, SIG_PIC3_F16, PS>(J, s_tf, R, lane, k0, acc);
        case SIG_PIC3_BF16: return lanes_row<INTERP, G, SIG_PIC3_BF16, PS>(J, s_tf, R, lane, k0, acc);
        case SIG_IL3: return lanes_row<INTERP, G, SIG_IL3, PS>(J, s_tf, R, lane, k0, acc);
        case SIG_IL3P: return lanes_row<INTERP, G, SIG_IL3P, PS>(J, s_tf, R, lane, k0, acc);
        case SIG_IL1: return lanes_row<INTERP, G, SIG_IL1, PS>(J, s_tf, R, lane, k0, acc);
        case SIG_IL1C: return lanes_row<INTERP, G, SIG_IL1C, PS>(J, s_tf, R, lane, k0, acc);
        case SIG_IL2: return lanes_row<INTERP, G, SIG_IL2, PS>(J, s_tf, R, lane, k0, acc);
        case SIG_IL4: return lanes_row<INTERP, G, SIG_IL4, PS>(J, s_tf, R, lane, k0, acc);
        default: return lanes_row<INTERP, G, SIG_GENERIC, PS>(J, s_tf, R, lane, k0, acc);
        }
    }
}

template <int G, int W, int SIGK>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(W > 0 ? W : 1, 8)))
void raycast_pool_kernel(const DevJob* __restrict__ jobs, const float4* __restrict__ tf_pool,
                         const RayRec* __restrict__ rays, int* __restrict__ counters) {
    extern __shared__ float4 s_tf[];
    const DevJob& J = jobs[0];
    store_tables(J, tf_pool, load_tables(J, tf_pool), s_tf);
    __syncthreads();
    const int n_rays = __builtin_amdgcn_readfirstlane(counters[0]);   // the setup kernel's count
    const int lane = (int)(threadIdx.x & 63);
    const int leader = lane & ~(G - 1);
    constexpr int kChunk = 2 * (64 / G);                                 // rays taken at a time
    // the wave's local queue, at first the chunk of its own number; the atomics of all waves on
    // one counter take about 14 ns each, one after another (7168 waves: 100 us)
    const int wave = (int)blockIdx.x * (kBlockThreads / 64) + (int)(threadIdx.x >> 6);
    const int handed = (int)gridDim.x * (kBlockThreads / 64) * kChunk;
    int q_next = min(__builtin_amdgcn_readfirstlane(wave) * kChunk, n_rays), q_end = min(q_next + kChunk, n_rays);
    bool exhausted = false, live = false;
    RaySetup R;
    int pixel = 0, k0 = 0;
    RayAccum acc = {0.f, 0.f, 0.f, 0.f, 0};
    for (;;) {
        // hand queued rays to the idle groups, in lane order
        unsigned long long idle = __ballot(!live && lane == leader);
        while (idle && !exhausted) {
            if (q_next >= q_end) {
                int base = handed;
                if (handed < n_rays) {
                    if (lane == 0) base += atomicAdd(&counters[1], kChunk);
                    base = __shfl(base, 0);
                }
                if (base >= n_rays) {
                    exhausted = true;
                    break;
                }
                q_next = base;
                q_end = min(base + kChunk, n_rays);
            }
            const int take = min(__popcll(idle), q_end - q_next);
            const int rank = __popcll(idle & ((1ull << leader) - 1ull));
            if (!live && rank < take) {
                const RayRec& rr = rays[q_next + rank];
                for (int a = 0; a < 3; ++a) {
                    R.pb[a] = rr.pb[a];
                    R.d[a] = rr.d[a];
                }
                R.kb = rr.kb;
                R.ke = rr.ke;
                R.t_first = rr.t_first;
                pixel = rr.pixel;
                k0 = R.kb;
                acc = RayAccum{0.f, 0.f, 0.f, 0.f, 0};
                live = true;
            }
            q_next += take;
            idle = __ballot(!live && lane == leader);
        }
        if (!__ballot(live)) break;
        if (live) {
            const bool done = J.interp ? pool_row<1, G, SIGK, (W > 0)>(J, s_tf, R, lane, k0, acc)
                                       : pool_row<0, G, SIGK, (W > 0)>(J, s_tf, R, lane, k0, acc);
            k0 += G;
            if (done) {
                if (lane == leader) {
                    reinterpret_cast<float4*>(J.out)[pixel] = make_float4(acc.C0, acc.C1, acc.C2, acc.A);
                    if (J.out_samples) J.out_samples[pixel] = acc.n;
                    if (J.out_depth) J.out_depth[pixel] = R.t_first;
                }
                live = false;
            }
        }
    }
}

// Sort-last compositing of partial images: per pixel, order the layers by
// the ray parameter of their first scan point and apply the front-to-back
// operator (C, A) o (C', A') = (C + (1-A) C', A + (1-A) A').
struct CompositeArgs {
    const float4* rgba[kMaxLayers];
    const float* depth[kMaxLayers];
    int n;
    int64_t n_pixels;
    float4* out;
};

// A layer without a scan point at a pixel has depth +inf and colour
// (0,0,0,0); compositing it changes nothing (C + T*0 = C exactly), so a pixel
// reads the colours of its layers with a finite depth only, and a pixel no
// layer reaches (most of the frame) writes transparent black at once.  Bound by
// memory: N (the layer count rounded up to a power of two) is a compile-time
// constant so that the depths of a pixel are loaded together and sorted in
// registers by static index, then the colours' addresses and the colours
// together; with a run-time count each layer waited for the one before (8 layers
// at 1920 x 1080, a quarter covered: 43 -> 17.6 us).
template <int N>
__global__ __launch_bounds__(256) void composite_kernel(CompositeArgs a) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n_pixels;
         i += (int64_t)gridDim.x * blockDim.x) {
        float dep[N];
        int idx[N];
        int live = 0;
#pragma unroll
        for (int l = 0; l < N; ++l) {
            dep[l] = l < a.n ? a.depth[l][i] : __builtin_inff();
            idx[l] = l;
        }
#pragma unroll
        for (int l = 0; l < N; ++l) live += dep[l] < __builtin_inff();
        if (live == 0) {
            a.out[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            continue;
        }
#pragma unroll
        for (int l = 1; l < N; ++l) {            // insertion sort, stable
            const float dv = dep[l];
            bool go = true;
#pragma unroll
            for (int m = l - 1; m >= 0; --m) {   // entry m moves up past dv, or dv settles above it
                const bool up = go && dep[m] > dv;
                dep[m + 1] = up ? dep[m] : go ? dv : dep[m + 1];
                const int im = idx[m], iu = idx[m + 1];
                idx[m + 1] = up ? im : iu;
                idx[m] = up ? iu : im;
                go = up;
            }
            dep[0] = go ? dv : dep[0];
        }
        const float4* layer[N];
        float4 c[N];
#pragma unroll
        for (int l = 0; l < N; ++l)
            if (l < live) layer[l] = a.rgba[idx[l]];
#pragma unroll
        for (int l = 0; l < N; ++l)
            if (l < live) c[l] = layer[l][i];
        float Cr = 0.f, Cg = 0.f, Cb = 0.f, A = 0.f;
#pragma unroll
        for (int l = 0; l < N; ++l)              // the finite depths sort first
            if (l < live) {
                const float T = 1.f - A;
                Cr = fmaf(T, c[l].x, Cr);
                Cg = fmaf(T, c[l].y, Cg);
                Cb = fmaf(T, c[l].z, Cb);
                A = fmaf(T, c[l].w, A);
            }
        a.out[i] = make_float4(Cr, Cg, Cb, A);
    }
}

// Frame encode: premultiplied RGBA32F over an opaque background, quantized
// to 8 bits per channel, q = floor(clamp(v, 0, 1) * 255 + 1/2) with NaN -> 0.
// Every operation is a separately rounded FP32 operation (no contraction), so
// the integer codes are a fixed function of the input bits.
struct EncodeArgs {
    const float4* in;
    uchar4* out;
    int64_t n_pixels;
    float bg[3];
    int has_bg;
};

__device__ __forceinline__ unsigned char quantize8(float v) {
#pragma clang fp contract(off)
    const float c = v > 0.f ? fminf(v, 1.f) : 0.f;    // NaN -> 0
    return (unsigned char)(int)floorf(c * 255.f + 0.5f);
}

__global__ void encode_rgba8_kernel(EncodeArgs a) {
#pragma clang fp contract(off)
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n_pixels;
         i += (int64_t)gridDim.x * blockDim.x) {
        const float4 c = a.in[i];
        uchar4 q;
        if (a.has_bg) {
            const float t = 1.f - c.w;
            q.x = quantize8(c.x + t * a.bg[0]);
            q.y = quantize8(c.y + t * a.bg[1]);
            q.z = quantize8(c.z + t * a.bg[2]);
            q.w = 255;
        } else {
            q.x = quantize8(c.x);
            q.y = quantize8(c.y);
            q.z = quantize8(c.z);
            q.w = quantize8(c.w);
        }
        a.out[i] = q;
    }
}

// Derived volume: every voxel's chain output per source, computed once with
// the same fetch and chain code as the ray loop (so the values are the ones
// the loop would compute at that voxel, bit for bit).  A thread takes 4 voxels
// with their loads in flight together: one (x, y) in 4 consecutive z-slices
// (x-fastest layout), or, in the paired layout, both y parities of one stored
// y pair at one x and one z parity in 2 consecutive stored z pairs (its two
// records of a pair are adjacent; lanes alternate the z parity, then step x).
// A wave's stores are one contiguous run (x-fastest) or 64 adjacent record
// pairs, and its reads of a source cover whole runs of 64 or 2 x 32 x.
// SIG > 0: the sources have that signature's compile-time kinds; SIG = 0: N
// sources of at most D components each, any storage.
template <int SIG, int N, int D, bool PAIRED>
__device__ __forceinline__ void derive_voxels(const DeriveArgs& a, int xi, int slot, int yi, int zi0, int nz) {
    constexpr int kZ = 4;
    const int ex = a.ext[0], ey = a.ext[1];
    const int x = xi - a.g;
    int vy[kZ], vz[kZ];                        // volume indices of the 4 voxels
    int64_t rec[kZ];                           // their records (float index / n)
    bool need[kZ];
#pragma unroll
    for (int j = 0; j < kZ; ++j) {
        if (PAIRED) {
            // slot: the z parity; j: y parity (j & 1) in stored z pair zi0 + (j >> 1)
            const int zp = zi0 + (j >> 1);
            vy[j] = 2 * yi + (j & 1) - a.gp;
            vz[j] = 2 * zp + slot - a.gp;
            need[j] = (j >> 1) < nz && vy[j] >= -a.g && vy[j] < ey - a.g && vz[j] >= -a.g && vz[j] < a.ext[2] - a.g;
            rec[j] = (((int64_t)zp * a.ny2 + yi) * ex + xi) * 4 + 2 * slot + (j & 1);
        } else {
            vy[j] = yi - a.g;
            vz[j] = zi0 + j - a.g;
            need[j] = j < nz;
            rec[j] = ((int64_t)(zi0 + j) * ey + yi) * ex + xi;
        }
    }
    // The clip test: this latency-bound pass waits on each wave's chain of
    // dependent scalar reads before its loads, so planes are outermost (each read
    // once for the 4 voxels), not one read per voxel and plane.
    if (a.n_sets > 0) {
        // a kept scan point reads voxel centres less than one voxel away per axis
        // (1.5 for the iso-surface gradient), i.e. within 1.5 sqrt(3) < 3 of it
        // along any unit normal
        bool any[kZ] = {false, false, false, false};
        auto test = [&](const float* pl, bool use, bool (&inside)[kZ]) {
            const float n0 = pl[0], n1 = pl[1], n2 = pl[2], n3 = pl[3];
            const float base = n0 * (a.org[0] + x + 0.5f);
#pragma unroll
            for (int j = 0; j < kZ; ++j)
                inside[j] = inside[j] &&
                            (!use || base + n1 * (a.org[1] + vy[j] + 0.5f) + n2 * (a.org[2] + vz[j] + 0.5f) + n3 >= -3.f);
        };
        for (int k = 0; k < a.n_sets; ++k) {
            bool inside[kZ] = {true, true, true, true};
            const int np = a.n_planes[k];
            // the first two planes of a set are read whether used or not (the arrays
            // hold kMaxClip planes), so their loads go out together with the count
            test(a.planes[k][0], np > 0, inside);
            test(a.planes[k][1], np > 1, inside);
            for (int p = 2; p < np; ++p) test(a.planes[k][p], true, inside);
#pragma unroll
            for (int j = 0; j < kZ; ++j) any[j] = any[j] || inside[j];
        }
#pragma unroll
        for (int j = 0; j < kZ; ++j) need[j] = need[j] && any[j];
    }
    int first = -1;
#pragma unroll
    for (int j = kZ - 1; j >= 0; --j)
        if (need[j]) first = j;
    if (first < 0) return;
    // a voxel that is not needed reads the first needed one's address (harmless, never stored)
    int ry[kZ], rz[kZ];
#pragma unroll
    for (int j = 0; j < kZ; ++j) {
        ry[j] = need[j] ? vy[j] : vy[first];
        rz[j] = need[j] ? vz[j] : vz[first];
    }
    // a source without guard layers never has them read: its guard cells hold the border values
    auto offset = [&](const DevSource& S, int y, int z) {
        const int qx = S.guard < 1 ? clampi(x, 0, ex - 2 * a.g - 1) : x;
        const int qy = S.guard < 1 ? clampi(y, 0, ey - 2 * a.g - 1) : y;
        const int qz = S.guard < 1 ? clampi(z, 0, a.ext[2] - 2 * a.g - 1) : z;
        return qx * S.stride[0] + qy * S.stride[1] + qz * S.stride[2];
    };
    auto store = [&](int j, const float* o) {
        float* d = a.dst + rec[j] * N;
        if constexpr (N == 4) {
            *reinterpret_cast<float4*>(d) = make_float4(o[0], o[1], o[2], o[3]);
        } else if constexpr (N == 2) {
            *reinterpret_cast<float2*>(d) = make_float2(o[0], o[1]);
        } else {
#pragma unroll
            for (int s = 0; s < N; ++s) d[s] = o[s];
        }
    };
    float out[kZ][N];
    if constexpr (SIG == SIG_GENERIC) {
        // every component of every source first, as it is stored (the loads of a
        // component are one uniform branch on the storage width, and nothing waits
        // on them there), then the chains
        uint32_t raw[N][kZ][D];
#pragma unroll
        for (int s = 0; s < N; ++s) {
            const DevSource& S = a.src[s];
            int off[kZ];
#pragma unroll
            for (int j = 0; j < kZ; ++j) off[j] = offset(S, ry[j], rz[j]);
#pragma unroll
            for (int c = 0; c < D; ++c) {
#pragma unroll
                for (int j = 0; j < kZ; ++j) raw[s][j][c] = 0u;
                if (c < S.f_dim) {
                    const int k = S.packed ? 0 : c, o = S.comp_off[c];
                    const __amdgpu_buffer_rsrc_t r = make_rsrc(S.base[k], S.num_records[k]);
                    if (S.dtype == DT_F32) {
#pragma unroll
                        for (int j = 0; j < kZ; ++j)
                            raw[s][j][c] = __builtin_amdgcn_raw_buffer_load_b32(r, off[j] + o, 0, 0);
                    } else {
#pragma unroll
                        for (int j = 0; j < kZ; ++j)
                            raw[s][j][c] = __builtin_amdgcn_raw_buffer_load_b16(r, off[j] + o, 0, 0);
                    }
                }
            }
        }
#pragma unroll
        for (int s = 0; s < N; ++s) {
            float v[kZ][4], res[kZ];
            const int dtype = a.src[s].dtype;
#pragma unroll
            for (int j = 0; j < kZ; ++j)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const uint32_t b = c < D ? raw[s][j][c < D ? c : 0] : 0u;
                    if (dtype == DT_F32) v[j][c] = __builtin_bit_cast(float, b);
                    else if (dtype == DT_F16) v[j][c] = (float)__builtin_bit_cast(_Float16, (unsigned short)b);
                    else v[j][c] = __builtin_bit_cast(float, b << 16);
                }
            run_chain_n<kZ, D>(a.src[s], v, res);
#pragma unroll
            for (int j = 0; j < kZ; ++j) out[j][s] = res[j];
        }
    } else {
        constexpr int K0 = SigKinds<SIG>::k0, K1 = SigKinds<SIG>::k1, K2 = SigKinds<SIG>::k2;
        float v0[kZ][4], v1[kZ][4], v2[kZ][4];
        // every load of the 4 voxels first
#pragma unroll
        for (int j = 0; j < kZ; ++j) {
            float t[1][4];
            const int o0[1] = {offset(a.src[0], ry[j], rz[j])};
            fetch_kind<K0, 1>(a.src[0], o0, t);
            for (int c = 0; c < 4; ++c) v0[j][c] = t[0][c];
            if constexpr (K1 != K_NONE) {
                const int o1[1] = {offset(a.src[1], ry[j], rz[j])};
                fetch_kind<K1, 1>(a.src[1], o1, t);
                for (int c = 0; c < 4; ++c) v1[j][c] = t[0][c];
            }
            if constexpr (K2 != K_NONE) {
                const int o2[1] = {offset(a.src[2], ry[j], rz[j])};
                fetch_kind<K2, 1>(a.src[2], o2, t);
                for (int c = 0; c < 4; ++c) v2[j][c] = t[0][c];
            }
        }
#pragma unroll
        for (int j = 0; j < kZ; ++j) {
            float t[1][4], r[1];
            for (int c = 0; c < 4; ++c) t[0][c] = v0[j][c];
            run_chain<1, KindOf<K0>::dim>(a.src[0], t, r);
            out[j][0] = r[0];
            if constexpr (K1 != K_NONE) {
                for (int c = 0; c < 4; ++c) t[0][c] = v1[j][c];
                run_chain<1, KindOf<K1>::dim>(a.src[1], t, r);
                out[j][1] = r[0];
            }
            if constexpr (K2 != K_NONE) {
                for (int c = 0; c < 4; ++c) t[0][c] = v2[j][c];
                run_chain<1, KindOf<K2>::dim>(a.src[2], t, r);
                out[j][2] = r[0];
            }
        }
    }
    // one contiguous store per voxel
#pragma unroll
    for (int j = 0; j < kZ; ++j)
        if (need[j]) store(j, out[j]);
}

// Blocks of 256 threads cover consecutive threads of consecutive rows (y, or
// stored y pairs of 2 ex threads) of one slab (4 z-slices, or 2 stored z
// pairs); the slabs are laid over grid y and z, one per thread.  A loop over
// slabs, which no volume but one of more than 262,140 slices needed, made every
// argument of every source loop-invariant: the compiler held them all in scalar
// registers across it and spilled 25 to 146 of them, to vector registers and to
// scratch.  Straight-line code reads each argument where it is used: no variant
// spills, and eight waves fit per SIMD (5 or 6 with sources of 4 components).
// Bound by memory once that is so.  The general kernel (SIG_GENERIC), which also
// read one voxel at a time, a source after the other: FP16 component arrays of
// 213 x 187 x 241 with a third clipped 176 -> 50 us, two FP32 sources of 256^3
// with half clipped 123 -> 49 us (the specialized pass over all three 82 -> 80).
constexpr unsigned kDeriveSlabsY = 32768;
template <int SIG, int N, int D, bool PAIRED>
__global__ __launch_bounds__(256) void derive_kernel(DeriveArgs a) {
    const int ex = a.ext[0];
    const int row = PAIRED ? 2 * ex : ex;
    const int rows = PAIRED ? a.ny2 : a.ext[1];
    const int idx = (int)(blockIdx.x * 256 + threadIdx.x);
    if (idx >= row * rows) return;
    const int yi = idx / row;
    const int r = idx - yi * row;
    const int xi = PAIRED ? r >> 1 : r, slot = PAIRED ? r & 1 : 0;
    const int nzs = PAIRED ? a.nz2 : a.ext[2], per = PAIRED ? 2 : 4;
    const int zi0 = per * (int)(blockIdx.z * kDeriveSlabsY + blockIdx.y);
    if (zi0 >= nzs) return;
    derive_voxels<SIG, N, D, PAIRED>(a, xi, slot, yi, zi0, min(per, nzs - zi0));
}

// Ray setup of every pixel of each job's screen rectangle, one lane per ray,
// into the job's ray records (kb = ke = 0: no scan point); the ray-casting
// kernel then reads a record instead of repeating the FP64 setup on every
// lane of a ray's group.
__device__ __forceinline__ void ray_setup_dense(const DevJob& J, int block, int n_blocks) {
    const int rw = J.cull[2] - J.cull[0] + 1, rh = J.cull[3] - J.cull[1] + 1;
    if (rw <= 0 || rh <= 0) return;
    RayRec* rays = static_cast<RayRec*>(J.rays);
    for (int i = block * 256 + (int)threadIdx.x; i < rw * rh; i += n_blocks * 256) {
        const int ry = i / rw, rx = i - ry * rw;
        const int px = J.cull[0] + rx, py = J.cull[1] + ry;
        RaySetup R;
        RayRec r;
        if (setup_ray(J, px, py, R)) {
            for (int a = 0; a < 3; ++a) {
                r.pb[a] = R.pb[a];
                r.d[a] = R.d[a];
            }
            r.kb = R.kb;
            r.ke = R.ke;
            r.t_first = R.t_first;
        } else {
            for (int a = 0; a < 3; ++a) r.pb[a] = r.d[a] = 0.f;
            r.kb = r.ke = 0;
            r.t_first = 0.f;
        }
        r.pixel = py * J.width + px;
        rays[i] = r;
    }
}

// Clear the output of every pixel outside its job's screen rectangle (no ray
// there can meet the box): transparent black, 0 samples, depth +inf.
__device__ __forceinline__ void fill_outside(const DevJob& J, int block, int n_blocks) {
    const int n = J.width * J.height;
    for (int i = block * 256 + (int)threadIdx.x; i < n; i += n_blocks * 256) {
        const int py = i / J.width, px = i - py * J.width;
        if (px >= J.cull[0] && px <= J.cull[2] && py >= J.cull[1] && py <= J.cull[3]) continue;
        reinterpret_cast<float4*>(J.out)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (J.out_samples) J.out_samples[i] = 0;
        if (J.out_depth) J.out_depth[i] = __builtin_inff();
    }
}

__global__ __launch_bounds__(256) void fill_outside_kernel(const DevJob* __restrict__ jobs) {
    fill_outside(jobs[blockIdx.y], (int)blockIdx.x, (int)gridDim.x);
}

// The fill and the ray setup touch different memory: one launch runs both,
// workgroups [0, nb) filling and [nb, 2 nb) setting up rays.
__global__ __launch_bounds__(256) void prepass_kernel(const DevJob* __restrict__ jobs, int nb) {
    const DevJob& J = jobs[blockIdx.y];
    const int b = (int)blockIdx.x;
    if (b < nb)
        fill_outside(J, b, nb);
    else
        ray_setup_dense(J, b - nb, nb);
}

// One job: the fill and ray setup as above, reading the job block from the
// kernel arguments, and the block stored to device memory for the
// ray-casting launch that follows (no separate host-to-device copy).
__global__ __launch_bounds__(256) void prepass_one_kernel(const DevJob job, DevJob* __restrict__ dst, int nb,
                                                          int dense) {
    const int b = (int)blockIdx.x;
    if (b == 0) {
        const uint32_t* s = reinterpret_cast<const uint32_t*>(&job);
        uint32_t* d = reinterpret_cast<uint32_t*>(dst);
        for (int i = (int)threadIdx.x; i < (int)(sizeof(DevJob) / 4); i += 256) d[i] = s[i];
    }
    if (b < nb)
        fill_outside(job, b, nb);
    else if (dense)
        ray_setup_dense(job, b - nb, nb);
}

__global__ void reset_counter_kernel(int* c, int n) {
    if ((int)threadIdx.x < n) c[threadIdx.x] = 0;
}

// Copy a strided field (guard layers included) into a packed buffer of the
// same storage type.  One thread per voxel.
struct CopyArgs {
    const unsigned char* src[4];
    int64_t src_stride[3];
    unsigned char* dst;
    int64_t dst_stride[3];
    int esize, f_dim;
    int lo[3], ext[3];
};

__global__ __launch_bounds__(256) void strided_copy_kernel(CopyArgs a) {
    const int xi = (int)(blockIdx.x * 64 + threadIdx.x);
    const int yi = (int)(blockIdx.y * 4 + threadIdx.y);
    if (xi >= a.ext[0] || yi >= a.ext[1]) return;
    for (int zi = (int)blockIdx.z; zi < a.ext[2]; zi += (int)gridDim.z) {
        const int x = xi + a.lo[0];
        const int y = yi + a.lo[1];
        const int z = zi + a.lo[2];
        for (int c = 0; c < a.f_dim; ++c) {
            const unsigned char* s = a.src[c] + x * a.src_stride[0] + y * a.src_stride[1] + z * a.src_stride[2];
            unsigned char* d = a.dst + x * a.dst_stride[0] + y * a.dst_stride[1] + z * a.dst_stride[2] +
                               (int64_t)c * a.esize;
            if (a.esize == 4) *reinterpret_cast<uint32_t*>(d) = *reinterpret_cast<const uint32_t*>(s);
            else *reinterpret_cast<uint16_t*>(d) = *reinterpret_cast<const uint16_t*>(s);
        }
    }
}

}  // namespace

using KernelFn = void (*)(const DevJob*, const float4*, int, int);

// The variant (W) of a signature's loop under the hint for at least 4 waves per
// SIMD.  One or two adjacent values: the pipelined loop (60 and 78 vector
// registers, 8 and 6 waves) is the faster one (two derived sources at 720p 81
// against 88 us a call, a 48^3 scalar 20.7 against 22.4).  Scalar and vectors read
// in place: every source's loads together (105 to 113 registers, 4 waves) instead of a
// source after the other: 272 against 350 us for 192^3 FP32 at 1024 x 768.  Three
// and four adjacent values keep the loop with more waves (62 and 76 registers, 8 and 6
// waves, against 90 and 104, 5 and 4, pipelined: six served requests 587 against 613 us,
// four derived sources 76 against 79), the general loop its bound.
template <int SIGK>
constexpr int kHintW = Il<SIGK>::n >= 3 || SIGK == SIG_GENERIC ? 4 : 0;

// ordered: the image of one lane per ray, by one lane or groups of 4 or 16
template <int SIGK>
KernelFn pick_specialized(int ordered, int lanes, int hint) {
    constexpr int H = kHintW<SIGK>;
    // the general loop would spill under a bound of 4 waves with the composited row beside it
    constexpr int O = SIGK == SIG_GENERIC ? 0 : H;
    if (ordered)
        return lanes == 1   ? raycast_kernel<true, 1, O, SIGK>
               : lanes == 4 ? raycast_kernel<true, 4, O, SIGK>
                            : raycast_kernel<true, 16, O, SIGK>;
    switch (lanes) {
    case 64: return raycast_kernel<false, 64, 0, SIGK>;
    case 32: return raycast_kernel<false, 32, 0, SIGK>;
    case 16: return hint ? raycast_kernel<false, 16, H, SIGK> : raycast_kernel<false, 16, 0, SIGK>;
    case 8: return hint ? raycast_kernel<false, 8, H, SIGK> : raycast_kernel<false, 8, 0, SIGK>;
    case 4: return hint ? raycast_kernel<false, 4, H, SIGK> : raycast_kernel<false, 4, 0, SIGK>;
    default: return raycast_kernel<false, 2, 0, SIGK>;
    }
}

KernelFn pick_kernel(int mode, int sig, int ordered, int lanes, int hint) {
    // iso-surface jobs: sig -3 when every source is plain (packed FP32 scalars without
    // functors, guard layers), else the run-time source handling
    // (bound to 3 waves per SIMD it takes 157 registers; without the bound 170, and 2 waves:
    // one iso-surface of a guard-less 128^3 at 1024 x 768 105 against 129 us a call)
    if (mode == 1) {
        if (lanes == 1) return sig == -3 ? raycast_kernel<false, 1, 0, -3> : raycast_kernel<false, 1, 3, -2>;
        return sig == -3 ? raycast_kernel<false, 8, 0, -3> : raycast_kernel<false, 8, 3, -2>;
    }
    switch (sig) {
    case SIG_F32x1: return pick_specialized<SIG_F32x1>(ordered, lanes, hint);
    case SIG_PIC3_F32: return pick_specialized<SIG_PIC3_F32>(ordered, lanes, hint);
    case SIG_PIC3_F16: return pick_specialized<SIG_PIC3_F16>(ordered, lanes, hint);
    case SIG_PIC3_BF16: return pick_specialized<SIG_PIC3_BF16>(ordered, lanes, hint);
    case SIG_IL3: return pick_specialized<SIG_IL3>(ordered, lanes, hint);
    case SIG_IL3P: return pick_specialized<SIG_IL3P>(ordered, lanes, hint);
    case SIG_IL1: return pick_specialized<SIG_IL1>(ordered, lanes, hint);
    case SIG_IL1C: return pick_specialized<SIG_IL1C>(ordered, lanes, hint);
    case SIG_IL2: return pick_specialized<SIG_IL2>(ordered, lanes, hint);
    case SIG_IL4: return pick_specialized<SIG_IL4>(ordered, lanes, hint);
    case SIG_GENERIC: return pick_specialized<SIG_GENERIC>(ordered, lanes, 1);
    default:
        break;
    }
    // mixed signatures: the dispatching kernels (one lane-count each)
    if (ordered)
        return lanes == 1   ? raycast_kernel<true, 1, 0, -1>
               : lanes == 4 ? raycast_kernel<true, 4, 0, -1>
                            : raycast_kernel<true, 16, 0, -1>;
    switch (lanes) {
    case 64: return raycast_kernel<false, 64, 0, -1>;
    case 32: return raycast_kernel<false, 32, 0, -1>;
    case 16: return raycast_kernel<false, 16, 0, -1>;
    case 8: return raycast_kernel<false, 8, 0, -1>;
    case 4: return raycast_kernel<false, 4, 0, -1>;
    default: return raycast_kernel<false, 2, 0, -1>;
    }
}

int launch_prepass(const LaunchArgs& a, void* stream) {
    // pixels outside the jobs' screen rectangles, then (optionally) the rays inside them
    if (a.dense_setup)
        hipLaunchKernelGGL(prepass_kernel, dim3(2 * a.fill_blocks, (unsigned)a.n_jobs), dim3(256), 0,
                           (hipStream_t)stream, a.jobs, (int)a.fill_blocks);
    else
        hipLaunchKernelGGL(fill_outside_kernel, dim3(a.fill_blocks, (unsigned)a.n_jobs), dim3(256), 0,
                           (hipStream_t)stream, a.jobs);
    return hipGetLastError();
}

int launch_prepass_one(const DevJob& job, DevJob* dst, unsigned fill_blocks, int dense, void* stream) {
    static_assert(sizeof(DevJob) % 4 == 0 && sizeof(DevJob) + 16 <= 4096, "the job block is a kernel argument");
    hipLaunchKernelGGL(prepass_one_kernel, dim3((dense ? 2 : 1) * fill_blocks), dim3(256), 0, (hipStream_t)stream,
                       job, dst, (int)fill_blocks, dense);
    return hipGetLastError();
}

int launch_raycast(const LaunchArgs& a, void* stream) {
    // dynamic LDS: one staged table (kTfLds RGBA32F values) per active source of the widest job
    const size_t lds = (size_t)(a.max_src > 0 ? a.max_src : 1) * kTfLds * sizeof(float4);
    const KernelFn kernel = pick_kernel(a.mode, a.sig, a.ordered, a.lanes, a.waves_hint);
    constexpr int kMaxBlocks = 1 << 23;      // a grid holds fewer than 2^32 threads
    for (int tile0 = 0; tile0 < a.total_tiles; tile0 += kMaxBlocks) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)std::min(kMaxBlocks, a.total_tiles - tile0)), dim3(kBlockThreads),
                           lds, (hipStream_t)stream, a.jobs, reinterpret_cast<const float4*>(a.tf_pool), a.n_jobs,
                           tile0);
        if (tile0 > INT_MAX - kMaxBlocks) break;
    }
    return hipGetLastError();
}

using PoolFn = void (*)(const DevJob*, const float4*, const RayRec*, int*);

template <int SIGK>
PoolFn pick_pool_specialized(int lanes, int hint) {
    switch (lanes) {
    case 16: return hint ? raycast_pool_kernel<16, 4, SIGK> : raycast_pool_kernel<16, 0, SIGK>;
    case 8: return hint ? raycast_pool_kernel<8, 4, SIGK> : raycast_pool_kernel<8, 0, SIGK>;
    case 4: return hint ? raycast_pool_kernel<4, 4, SIGK> : raycast_pool_kernel<4, 0, SIGK>;
    default: return raycast_pool_kernel<2, 0, SIGK>;
    }
}

PoolFn pick_pool_kernel(int sig, int lanes, int hint) {
    switch (sig) {
    case SIG_F32x1: return pick_pool_specialized<SIG_F32x1>(lanes, hint);
    case SIG_PIC3_F32: return pick_pool_specialized<SIG_PIC3_F32>(lanes, hint);
    case SIG_PIC3_F16: return pick_pool_specialized<SIG_PIC3_F16>(lanes, hint);
    case SIG_PIC3_BF16: return pick_pool_specialized<SIG_PIC3_BF16>(lanes, hint);
    case SIG_IL3: return pick_pool_specialized<SIG_IL3>(lanes, hint);
    case SIG_IL3P: return pick_pool_specialized<SIG_IL3P>(lanes, hint);
    case SIG_GENERIC: return pick_pool_specialized<SIG_GENERIC>(lanes, hint);
    case SIG_IL1: return pick_pool_specialized<SIG_IL1>(lanes, hint);
    // their own loops keep 7 or 8 waves per SIMD, the dispatching one 3 (160^3 at 1280 x 720, 16
    // lanes, dispatching and own, us a call: a guard-less scalar 162 and 121, two derived sources
    // 187 and 141, four 204 and 202; with 2 lanes 475 and 407, 519 and 450, 412 and 374)
    case SIG_IL1C: return pick_pool_specialized<SIG_IL1C>(lanes, hint);
    case SIG_IL2: return pick_pool_specialized<SIG_IL2>(lanes, hint);
    case SIG_IL4: return pick_pool_specialized<SIG_IL4>(lanes, hint);
    default: break;
    }
    switch (lanes) {
    case 16: return raycast_pool_kernel<16, 0, -1>;
    case 8: return raycast_pool_kernel<8, 0, -1>;
    case 4: return raycast_pool_kernel<4, 0, -1>;
    default: return raycast_pool_kernel<2, 0, -1>;
    }
}

int launch_raycast_pooled(const DevJob* job_dev, int width, int height, const float* tf_pool, int max_src, int sig,
                          int lanes, int hint, void* rays, int* counters, int n_cu, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(reset_counter_kernel, dim3(1), dim3(64), 0, st, counters, 2);
    const dim3 sgrid((unsigned)((width + 15) / 16), (unsigned)((height + 15) / 16));
    hipLaunchKernelGGL(ray_setup_kernel, sgrid, dim3(256), 0, st, job_dev, static_cast<RayRec*>(rays), counters);
    const size_t lds = (size_t)(max_src > 0 ? max_src : 1) * kTfLds * sizeof(float4);
    const PoolFn k = pick_pool_kernel(sig, lanes, hint);
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, kBlockThreads, lds) != hipSuccess || per_cu < 1)
        per_cu = 1;
    hipLaunchKernelGGL(k, dim3((unsigned)(n_cu * per_cu)), dim3(kBlockThreads), lds, st, job_dev,
                       reinterpret_cast<const float4*>(tf_pool), static_cast<const RayRec*>(rays), counters);
    return hipGetLastError();
}

size_t ray_record_bytes() { return sizeof(RayRec); }

int launch_strided_copy(const void* const* src_comp, const int64_t* src_stride, void* dst,
                        const int64_t* dst_stride, int esize, int f_dim, const int32_t lo[3],
                        const int32_t ext[3], void* stream) {
    CopyArgs a;
    for (int c = 0; c < 4; ++c) a.src[c] = c < f_dim ? static_cast<const unsigned char*>(src_comp[c]) : nullptr;
    for (int k = 0; k < 3; ++k) {
        a.src_stride[k] = src_stride[k];
        a.dst_stride[k] = dst_stride[k];
        a.lo[k] = lo[k];
        a.ext[k] = ext[k];
    }
    a.dst = static_cast<unsigned char*>(dst);
    a.esize = esize;
    a.f_dim = f_dim;
    if (ext[0] <= 0 || ext[1] <= 0 || ext[2] <= 0) return hipSuccess;
    const dim3 grid((unsigned)((ext[0] + 63) / 64), (unsigned)((ext[1] + 3) / 4), (unsigned)std::min(ext[2], 65535));
    hipLaunchKernelGGL(strided_copy_kernel, grid, dim3(64, 4), 0, (hipStream_t)stream, a);
    return hipGetLastError();
}

int launch_composite(const float* const* rgba, const float* const* depth, int n_layers, int64_t n_pixels, float* out,
                     void* stream) {
    CompositeArgs a;
    for (int l = 0; l < kMaxLayers; ++l) {
        a.rgba[l] = l < n_layers ? reinterpret_cast<const float4*>(rgba[l]) : nullptr;
        a.depth[l] = l < n_layers ? depth[l] : nullptr;
    }
    a.n = n_layers;
    a.n_pixels = n_pixels;
    a.out = reinterpret_cast<float4*>(out);
    if (n_pixels <= 0) return hipSuccess;
    const int64_t blocks = (n_pixels + 255) / 256;
    void (*const k)(CompositeArgs) = n_layers <= 2   ? composite_kernel<2>
                                     : n_layers <= 4 ? composite_kernel<4>
                                     : n_layers <= 8 ? composite_kernel<8>
                                                     : composite_kernel<16>;
    hipLaunchKernelGGL(k, dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(256), 0, (hipStream_t)stream, a);
    return hipGetLastError();
}

int launch_encode_rgba8(const float* rgba, int64_t n_pixels, const float* bg, unsigned char* out, void* stream) {
    EncodeArgs a;
    a.in = reinterpret_cast<const float4*>(rgba);
    a.out = reinterpret_cast<uchar4*>(out);
    a.n_pixels = n_pixels;
    a.has_bg = bg != nullptr;
    for (int c = 0; c < 3; ++c) a.bg[c] = bg ? bg[c] : 0.f;
    const int64_t blocks = std::min<int64_t>((n_pixels + 255) / 256, 8192);
    if (blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(encode_rgba8_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, a);
    return hipGetLastError();
}

using DeriveFn = void (*)(DeriveArgs);

template <int N, bool PAIRED>
DeriveFn derive_general(int dim) {
    if (dim <= 1) return derive_kernel<SIG_GENERIC, N, 1, PAIRED>;
    if (dim <= 3) return derive_kernel<SIG_GENERIC, N, 3, PAIRED>;
    return derive_kernel<SIG_GENERIC, N, 4, PAIRED>;
}

DeriveFn derive_variant(const DeriveArgs& a, int sig) {
    int dim = 1;
    for (int s = 0; s < a.n; ++s) dim = std::max(dim, (int)a.src[s].f_dim);
    if (a.paired) {
        switch (sig) {
        case SIG_PIC3_F32: return derive_kernel<SIG_PIC3_F32, 3, 3, true>;
        case SIG_PIC3_F16: return derive_kernel<SIG_PIC3_F16, 3, 3, true>;
        case SIG_PIC3_BF16: return derive_kernel<SIG_PIC3_BF16, 3, 3, true>;
        default: return derive_general<3, true>(dim);
        }
    }
    // x fastest: the compiled kinds for three sources too, whose pass is shorter where a
    // launch is (100 volumes of 24^3, iso: 898 us a call by the general pass, 770; from 96^3 on
    // they take the same time)
    switch (a.n == 3 ? sig : (int)SIG_GENERIC) {
    case SIG_PIC3_F32: return derive_kernel<SIG_PIC3_F32, 3, 3, false>;
    case SIG_PIC3_F16: return derive_kernel<SIG_PIC3_F16, 3, 3, false>;
    case SIG_PIC3_BF16: return derive_kernel<SIG_PIC3_BF16, 3, 3, false>;
    default: break;
    }
    switch (a.n) {
    case 1: return derive_general<1, false>(dim);
    case 2: return derive_general<2, false>(dim);
    case 3: return derive_general<3, false>(dim);
    default: return derive_general<4, false>(dim);
    }
}

int launch_derive(const DeriveArgs& a, int sig, void* stream) {
    if (a.ext[0] <= 0 || a.ext[1] <= 0 || a.ext[2] <= 0) return hipSuccess;
    if (a.n < 1 || a.n > kMaxDerived || (a.paired && a.n != 3)) return hipErrorInvalidValue;
    if (a.paired && (a.gp < a.g || (a.gp & 1) || 2 * a.ny2 < a.ext[1] - a.g + a.gp ||
                     2 * a.nz2 < a.ext[2] - a.g + a.gp))
        return hipErrorInvalidValue;
    const int64_t slice = (int64_t)a.ext[0] * (a.paired ? 2 * (int64_t)a.ny2 : a.ext[1]);
    if (slice > (1LL << 30)) return hipErrorInvalidValue;
    const int slabs = a.paired ? (a.nz2 + 1) / 2 : (a.ext[2] + 3) / 4;
    const dim3 grid((unsigned)((slice + 255) / 256), std::min((unsigned)slabs, kDeriveSlabsY),
                    ((unsigned)slabs + kDeriveSlabsY - 1) / kDeriveSlabsY);
    hipLaunchKernelGGL(derive_variant(a, sig), grid, dim3(256), 0, (hipStream_t)stream, a);
    return hipGetLastError();
}

// Scratch of the render entry point that allocates nothing: the ray records of
// its set-up pass.  One copy per device, held until the process ends; every call
// on a device uses that device's copy, so calls that overlap on one device (other
// streams, other contexts) race.  Host code must not pass the array's name to a
// kernel (in host code it is a stand-in, not a device address): it takes the
// address noalloc_scratch() looked up for the device.
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

int noalloc_scratch(int device, void** ptr) {
    static std::mutex lock;
    static void* addr[kMaxDevices] = {};
    if (device < 0 || device >= kMaxDevices || !ptr) return hipErrorInvalidValue;
    std::lock_guard<std::mutex> guard(lock);
    if (!addr[device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));   // the current device's copy
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[device] = p;
    }
    *ptr = addr[device];
    return hipSuccess;
}

}  // namespace isaac
